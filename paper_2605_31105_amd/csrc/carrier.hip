// Carrier-concentration diagnostics of a local merge rule (App. B,
// "Quantitative Carrier Concentration"; Sec. 1 on span boundaries): every
// evicted token is assigned to the retained token whose key has the highest
// cosine similarity with its own (the key-similarity matching of D2O/KVMerger),
// and the loads a_i of the retained slots are summarised per unit.
//
// match_kernel: a block takes 128 or 256 consecutive cache positions of one unit
// (one or two 16-row tiles per wave in registers) and streams the unit's retained
// keys through LDS in tiles of 64, gathered through idx; the inverse norm of each
// retained key is formed while the tile is staged (NaN past the last slot, so
// that those never compare larger).  S = K_q K_ret^T runs on the bf16 MFMA
// (exact products, fp32 sums); a lane keeps, for each of its 4 or 8 rows, the best
// (S / ||k_i||, slot) over the keys it sees, in increasing slot order, and the
// 16 lanes that share a row settle the row at the end (equal values go to the
// lower slot).  Scaling by 1 / ||k_j|| is left out: it does not change the
// argmax.  Retained positions get -1.
// Bound by issue and latency: per 64 products the VALU takes a multiply, a
// compare and two selects (16 cycles of a SIMD) and the MFMAs 16, and staging a
// key costs every block the same.  The products of the next 16 keys are issued
// among the compares of the current ones, with one barrier per tile; the norm
// is a corrected hardware estimate, and row addresses are looked up
// a tile ahead.  Whole calls, 64 units of 32k tokens and 2048 keys: 1677 -> 1320 us
// (four row tiles per wave, at one block per compute unit, about 1600).
// stats_kernel: one block per unit; loads by LDS atomics, then b, b_eff, A_max,
// the Gini coefficient (exact integer sum of |a_i - a_j| over all pairs: with
// F(v) the number of loads <= v it is 2 sum_v F(v) (c - F(v)), from a histogram
// of the loads and one scan; over the pairs themselves with few slots and when a
// load reaches the histogram's size), and the boundary-carrier figures.  With 64 units of 32k
// tokens and 2048 slots: 147 -> 14 us.
#include <math.h>

#include <type_traits>

#include "grkv_device.h"
#include "grkv_internal.h"

namespace grkv {
namespace {

// Sum over N (8 or 16) consecutive lanes, in every one of them.
template <int N>
__device__ __forceinline__ float row_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, false));
  if (N == 16)
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, false));
  return v;
}

// 1 / sqrt(ss) with the square root and then the reciprocal rounded to nearest
// (Markstein's residual corrections of the hardware estimates; with estimates an
// ulp off either way, the result is within an ulp of the IEEE operations' and
// differs from it in about 1 of 10^7), 0 for ss = 0 or infinite; ss is scaled by a
// power of four where the estimate would leave its normal range.
__device__ __forceinline__ float inv_norm(float ss) {
  const bool tiny = ss < 0x1p-100f;
  const float x = tiny ? ss * 0x1p48f : ss;
  const float y = __builtin_amdgcn_rsqf(x);
  float q = x * y;
  q = fmaf(fmaf(-q, q, x), 0.5f * y, q);
  float r = __builtin_amdgcn_rcpf(q);
  r = fmaf(fmaf(-q, r, 1.f), r, r);
  r = fmaf(fmaf(-q, r, 1.f), r, r);
  if (tiny) r *= 0x1p24f;
  return ss > 0.f && ss < __builtin_huge_valf() ? r : 0.f;
}

constexpr int kMatchWaves = 8;
constexpr int kRetTile = 64;                   // retained keys per LDS tile

// RT: 16-row tiles per wave
template <int D, int RT>
__global__ __launch_bounds__(kMatchWaves * 64) void match_kernel(
    const u16* __restrict__ K, const int32_t* __restrict__ idx, int64_t n, int c,
    int32_t* __restrict__ assign) {
  constexpr int NTH = kMatchWaves * 64;
  constexpr int KS = D + 8;                      // LDS row stride (bf16)
  constexpr int CH = kRetTile * D / 8;           // 16-byte chunks of a tile
  constexpr int PER = CH / NTH;
  constexpr int CPR = D / 8;                     // chunks per key row
  constexpr int DS = D / 32, KT = kRetTile / 16;
  static_assert(CH % NTH == 0 && (CPR == 8 || CPR == 16), "whole tiles, rows of 8 or 16 lanes");
  __shared__ __attribute__((aligned(16))) u16 kt_s[2][kRetTile * KS];
  __shared__ float inv_s[2][kRetTile];
  const int u = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const u16* Ku = K + (size_t)u * n * D;
  const int32_t* iu = idx + (size_t)u * c;
  const int64_t r0 = ((int64_t)blockIdx.x * kMatchWaves + wave) * (16 * RT);   // this wave's first row

  // query rows of this wave: rows r0 + 16 rt + l16, k = 32 ks + 8 g ..
  uint4 qa[RT][DS];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int64_t r = min(r0 + 16 * rt + l16, n - 1);
#pragma unroll
    for (int ks = 0; ks < DS; ++ks)
      qa[rt][ks] = *reinterpret_cast<const uint4*>(Ku + (size_t)r * D + ks * 32 + 8 * g);
  }

  // register-staged retained tiles; chunk e of tile t: key t*64 + e / CPR.
  // The source rows of a tile are looked up one tile before its keys.
  uint4 reg[PER];
  uint32_t src[PER];
  auto rows = [&](int t) {   // (past the last slot: the last slot's row)
#pragma unroll
    for (int k = 0; k < PER; ++k)
      src[k] = (uint32_t)iu[min(t * kRetTile + (tid + k * NTH) / CPR, c - 1)];
  };
  auto load = [&]() {
#pragma unroll
    for (int k = 0; k < PER; ++k)
      reg[k] = reinterpret_cast<const uint4*>(Ku)[(size_t)src[k] * CPR + tid % CPR];
  };
  auto store = [&](int t) {
    const int buf = t & 1;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = tid + k * NTH;
      const int key = e / CPR, ch = e % CPR;
      *reinterpret_cast<uint4*>(&kt_s[buf][key * KS + ch * 8]) = reg[k];
      const uint32_t w4[4] = {reg[k].x, reg[k].y, reg[k].z, reg[k].w};
      float ss = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = __uint_as_float(w4[q] << 16), b = __uint_as_float(w4[q] & 0xffff0000u);
        ss = fmaf(a, a, fmaf(b, b, ss));
      }
      // the CPR chunks of a key sit in CPR consecutive lanes
      ss = row_sum<CPR>(ss);
      // 1 / ||k|| (the IEEE square root and division take the kernel past 128
      // registers, one block per compute unit less: 1342 -> 1845 us)
      if (ch == 0)
        inv_s[buf][key] = t * kRetTile + key >= c ? __builtin_nanf("") : inv_norm(ss);
    }
  };

  float best[RT][4];
  int bslot[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      best[rt][i] = -__builtin_huge_valf();
      bslot[rt][i] = 0;
    }

  const int ntiles = (c + kRetTile - 1) / kRetTile;
  rows(0);
  load();
  rows(1);
  store(0);
  load();
  rows(2);
  for (int t = 0; t < ntiles; ++t) {
    const int buf = t & 1;
    __syncthreads();   // tile t is in LDS, and every wave is done with tile t - 1
    if (t + 1 < ntiles) {   // (the loads run up to two tiles past the last: never stored)
      store(t + 1);
      load();
      rows(t + 3);
    }
    // acc[rt]: rows r0 + 16rt + 4g + i, key 16kt + l16
    auto products = [&](int kt, f32x4 (&acc)[RT], float& inv) {
      const int key = 16 * kt + l16;
      uint4 kb[DS];
#pragma unroll
      for (int ks = 0; ks < DS; ++ks)
        kb[ks] = *reinterpret_cast<const uint4*>(&kt_s[buf][key * KS + ks * 32 + 8 * g]);
      inv = inv_s[buf][key];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = zero4();
#pragma unroll
      for (int ks = 0; ks < DS; ++ks)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          acc[rt] = mfma_bf16(as_bf16x8(qa[rt][ks]), as_bf16x8(kb[ks]), acc[rt]);
    };
    auto compare = [&](int kt, const f32x4 (&acc)[RT], float inv) {
      const int slot = t * kRetTile + 16 * kt + l16;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = acc[rt][i] * inv;
          const bool up = v > best[rt][i];   // slots rise within a lane: a tie keeps the lower
          best[rt][i] = up ? v : best[rt][i];
          bslot[rt][i] = up ? slot : bslot[rt][i];
        }
    };
    f32x4 acc[2][RT];
    float inv[2];
    products(0, acc[0], inv[0]);
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      if (kt + 1 < KT) products(kt + 1, acc[(kt + 1) & 1], inv[(kt + 1) & 1]);
      compare(kt, acc[kt & 1], inv[kt & 1]);
    }
  }

  // settle each row over the 16 lanes holding it: larger value, then lower slot
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v = best[rt][i];
      int sl = bslot[rt][i];
#pragma unroll
      for (int off = 1; off < 16; off <<= 1) {
        const float ov = __shfl_xor(v, off);
        const int os = __shfl_xor(sl, off);
        if (ov > v || (ov == v && os < sl)) {
          v = ov;
          sl = os;
        }
      }
      const int64_t r = r0 + 16 * rt + 4 * g + i;
      if (l16 == 0 && r < n) {
        // retained position?  idx is ascending: binary search
        int lo = 0, hi = c;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (iu[mid] < r) lo = mid + 1;
          else hi = mid;
        }
        const bool ret = lo < c && iu[lo] == r;
        assign[(size_t)u * n + r] = ret ? -1 : sl;
      }
    }
}

constexpr int kStatsThreads = 1024;
constexpr int kMaxCarrierSlots = 8192;
constexpr int kPairSlots = 256;

// metrics [U][8] = {b, b_eff, A_max, Gini, boundary fraction, boundary share,
// enrichment, boundary / interior mean load}
__global__ __launch_bounds__(kStatsThreads) void stats_kernel(
    const int32_t* __restrict__ assign, const int32_t* __restrict__ idx, int64_t n, int c,
    int32_t* __restrict__ counts, float* __restrict__ metrics) {
  __shared__ int cnt[kMaxCarrierSlots];
  __shared__ uint32_t hist[kMaxCarrierSlots];
  __shared__ uint32_t scratch[16];
  __shared__ int large;
  __shared__ unsigned long long red[16][6];
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t* iu = idx + (size_t)u * c;
  for (int i = tid; i < c; i += kStatsThreads) cnt[i] = 0;
  __syncthreads();
  auto count = [&](auto batch_tag) {   // `batch` loads in flight
    constexpr int B = decltype(batch_tag)::value;
    for (int64_t j0 = tid; j0 < n; j0 += B * kStatsThreads) {
      int a[B];
#pragma unroll
      for (int k = 0; k < B; ++k) a[k] = assign[(size_t)u * n + min(j0 + k * kStatsThreads, n - 1)];
#pragma unroll
      for (int k = 0; k < B; ++k)
        if (j0 + k * kStatsThreads < n && a[k] >= 0 && a[k] < c) atomicAdd(&cnt[a[k]], 1);
    }
  };
  if (n <= 2 * kStatsThreads) count(std::integral_constant<int, 2>{});
  else count(std::integral_constant<int, 16>{});
  // few slots: every pair directly (100 slots: a call 1.3 us shorter than with the
  // histogram; 256 the same, 512 5 us longer)
  const bool direct = c <= kPairSlots;
  if (!direct)
    for (int i = tid; i < kMaxCarrierSlots; i += kStatsThreads) hist[i] = 0u;
  if (tid == 0) large = 0;
  __syncthreads();
  // per thread: sum a, sum a^2, max a, active, boundary slots, boundary load,
  // and the pair sum of |a_i - a_j| over its rows i
  unsigned long long s1 = 0, s2 = 0, amax = 0, act = 0, nb = 0, sb = 0, pair = 0;
  for (int i = tid; i < c; i += kStatsThreads) {
    const unsigned long long a = (unsigned long long)cnt[i];
    s1 += a;
    s2 += a * a;
    amax = a > amax ? a : amax;
    act += a > 0;
    const bool first = i == 0 || iu[i - 1] + 1 != iu[i];
    const bool last = i == c - 1 || iu[i] + 1 != iu[i + 1];
    if (first || last) {
      ++nb;
      sb += a;
    }
    if (counts) counts[(size_t)u * c + i] = (int32_t)a;
    if (direct) continue;
    if (a < (unsigned long long)kMaxCarrierSlots) atomicAdd(&hist[a], 1u);
    else large = 1;
  }
  __syncthreads();
  if (!direct && !large) {   // (block-uniform)
    constexpr int PER = kMaxCarrierSlots / kStatsThreads;
    uint32_t h[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      h[k] = hist[tid * PER + k];
      sum += h[k];
    }
    uint32_t total, F = block_exclusive_scan(sum, scratch, &total);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      F += h[k];
      pair += 2ull * F * (uint32_t)(c - (int)F);
    }
  } else {
    for (int i = tid; i < c; i += kStatsThreads)
      for (int j = 0; j < c; ++j) {
        const int dlt = cnt[i] - cnt[j];
        pair += (unsigned long long)(dlt < 0 ? -dlt : dlt);
      }
  }
  unsigned long long v[6] = {s1, s2, act, nb, sb, pair};
  for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] += __shfl_xor(v[k], off);
    const unsigned long long om = __shfl_xor(amax, off);
    amax = om > amax ? om : amax;
  }
  __shared__ unsigned long long redmax[16];
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) red[wave][k] = v[k];
    redmax[wave] = amax;
  }
  __syncthreads();
  if (tid == 0) {
    unsigned long long t[6] = {0, 0, 0, 0, 0, 0}, mx = 0;
    for (int w = 0; w < kStatsThreads / 64; ++w) {
      for (int k = 0; k < 6; ++k) t[k] += red[w][k];
      mx = redmax[w] > mx ? redmax[w] : mx;
    }
    const double tot = (double)t[0], cc = (double)c;
    const float nanf_ = __builtin_nanf("");
    float m[8];
    m[0] = (float)t[2];
    m[4] = (float)((double)t[3] / cc);
    if (t[0] > 0) {
      m[1] = (float)(tot * tot / (double)t[1]);
      m[2] = (float)((double)mx / (tot / cc));
      m[3] = (float)((double)t[5] / (2.0 * cc * tot));
      const double share = (double)t[4] / tot;
      m[5] = (float)share;
      m[6] = (float)(share / ((double)t[3] / cc));
      const double ni = cc - (double)t[3];
      if (t[3] > 0 && ni > 0) {
        const double mi = (tot - (double)t[4]) / ni;
        m[7] = mi > 0 ? (float)(((double)t[4] / (double)t[3]) / mi) : __builtin_huge_valf();
      } else {
        m[7] = nanf_;
      }
    } else {
      m[1] = m[2] = m[3] = m[5] = m[6] = m[7] = nanf_;
    }
    for (int k = 0; k < 8; ++k) metrics[(size_t)u * 8 + k] = m[k];
  }
}

// L_common = sum_u D_after_u ||Y_u||^2 / sum_u ||Y_u||^2 from the stats of a
// grkv_compress call (one block, fixed summation order).
__global__ __launch_bounds__(256) void lcommon_kernel(const float* __restrict__ stats, int U,
                                                      float* __restrict__ out) {
  __shared__ double rn[4], rd[4];
  const int tid = threadIdx.x;
  double num = 0, den = 0;
  for (int u = tid; u < U; u += 256) {
    num += (double)stats[u * 4 + 2] * stats[u * 4 + 0];
    den += (double)stats[u * 4 + 0];
  }
  for (int off = 32; off > 0; off >>= 1) {
    num += __shfl_xor(num, off);
    den += __shfl_xor(den, off);
  }
  if ((tid & 63) == 0) {
    rn[tid >> 6] = num;
    rd[tid >> 6] = den;
  }
  __syncthreads();
  if (tid == 0) {
    double a = 0, b = 0;
    for (int k = 0; k < 4; ++k) { a += rn[k]; b += rd[k]; }
    out[0] = b > 0 ? (float)(a / b) : 0.f;
  }
}

}  // namespace

bool carrier_supported(int dtype, int d, int c) {
  return dtype == GRKV_BF16 && (d == 64 || d == 128) && c >= 1 && c <= kMaxCarrierSlots;
}

hipError_t launch_carrier(const void* K, const int32_t* idx, int U, int64_t n, int c, int d,
                          const float* stats, int32_t* assign, int32_t* counts, float* metrics,
                          float* l_common, hipStream_t s) {
  // Two row tiles per wave (113 registers, two blocks per compute unit at d = 128)
  // read each key half as often, one starts sooner and fills the chip with fewer
  // positions.  One / two tiles, whole calls at d = 128 and 64: 64 units of 8192
  // positions with 384 slots 122 / 128 and 87 / 89 us, with 512 145 / 141 and 99 / 97,
  // with 1100 262 / 219 and 168 / 148; 40 units of 3400 positions (560 blocks of two
  // tiles) with 1100 slots 98 / 101 and 69 / 74; 8 of 8192 with 512 38 / 42 and 31 /
  // 36.  Where two tiles take one round at d = 128 and one tile a second past its
  // three blocks per compute unit: 132 of 706 with 255 41.8 / 39.3, 100 of 1000 with
  // 900 78.8 / 68.0, but 180 of 500 with 400 (720 blocks of one tile) 44.1 / 48.4.
  auto blocks = [&](int tiles) { return (n + 16 * tiles * kMatchWaves - 1) / (16 * tiles * kMatchWaves); };
  const int64_t b1 = U * blocks(1), b2 = U * blocks(2);
  const int rt = (b2 >= 1024 && c >= 512) || (d == 128 && b2 <= 512 && b1 > 768) ? 2 : 1;
  const dim3 grid((unsigned)blocks(rt), U);
#define GRKV_MATCH(DV, RTV)                                                                  \
  hipLaunchKernelGGL((match_kernel<DV, RTV>), grid, dim3(kMatchWaves * 64), 0, s,            \
                     (const u16*)K, idx, n, c, assign)
  if (d == 128) {
    if (rt == 2) GRKV_MATCH(128, 2);
    else GRKV_MATCH(128, 1);
  } else {
    if (rt == 2) GRKV_MATCH(64, 2);
    else GRKV_MATCH(64, 1);
  }
#undef GRKV_MATCH
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(stats_kernel, dim3(U), dim3(kStatsThreads), 0, s, assign, idx, n, c, counts,
                     metrics);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (stats && l_common) {
    hipLaunchKernelGGL(lcommon_kernel, dim3(1), dim3(256), 0, s, stats, U, l_common);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace grkv
