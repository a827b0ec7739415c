// Token scores of H2O, the token-based eviction method GRKV is paired with
// (Sec. 2: heavy hitters kept by accumulated attention scores; Sec. 4.3,
// compatibility).  A prefix token's score is the attention it receives,
// summed over every prompt position of every query head of its KV head's
// group, each row being the causal softmax of q_i K^T / sqrt(d) over keys
// 0..i:
//   s_j = sum_g sum_{i >= j} 2^(t_{g,i,j} - LSE2_{g,i}),  t = q . k log2(e) / sqrt(d).
// This is the work of a prefill attention without P.V (O(n^2 d) per head),
// done in two MFMA passes with no atomics, each with 8 waves per block:
//  * h2o_lse_kernel: a block takes 128 RT / G prompt positions of all G query
//    heads (head-major rows; a wave owns RT 16-row tiles as MFMA B operands in
//    registers) and streams the keys up to its last position through LDS in
//    tiles of 64, keeping per row and lane an integer reference exponent and an
//    fp64 sum of 2^(t - ref) (as the window's pass A does); the four lanes of
//    a row merge at the end into LSE2 (log2 domain).  Blocks run latest
//    positions first (most keys);
//  * h2o_colsum_kernel: a block takes 128 KT prefix keys (a wave: KT 16-key
//    tiles as A operands in registers) and streams the query tiles (128 / G
//    positions of all heads) at or after its first key, with their LSE2,
//    through LDS; P = 2^(t - LSE2) under the causal rule is summed per key, in
//    fp32 within a query tile and in fp64 across tiles; a 16-lane reduction at
//    the end gives the key's score.
// What bounds them: per 64 logits the VALU takes fma + exp + add (16 cycles of
// a SIMD, the exponential at half rate) and the MFMAs 16 more, so both passes
// are written to run the two side by side: the products of the next 16-wide
// tile are issued among the exponentials of the current one (the accumulators
// are double-buffered), one barrier per staged tile, and four stationary tiles
// per wave, so that one fragment read from LDS feeds four MFMAs (with one, as
// the column sums had it, the LDS reads took longer than the MFMAs).  Blocks
// are ordered tile-major over the units, longest first: unit-major, the last
// unit's long blocks started late and the column sums took 1.6 times the
// row pass for the same work.  Eight units of 32k tokens with 4 heads each,
// both passes: 13.1 -> 8.6 ms (two tiles per wave 10.0 ms).
// Calls with few blocks take fewer stationary tiles per wave (h2o_tiles).
// Causal masks are applied only on tiles that straddle the diagonal, and a
// wave skips the tiles that it sees nothing of.
// The scores then drive grkv_compress_scored (selection with pool width 1).
#include "grkv_device.h"
#include "grkv_internal.h"

#include <type_traits>

namespace grkv {
namespace {

constexpr int kH2oWaves = 8;
constexpr int kH2oTh = kH2oWaves * 64;
constexpr int kH2oKT = 64;          // keys per streamed key tile (LSE pass)
constexpr int kH2oQRows = 128;      // rows (positions x heads) of a streamed query tile

// ------------------------------------------------------------ row LSE ----
template <int D, int G, int RT>
__global__ __launch_bounds__(kH2oTh) void h2o_lse_kernel(const u16* __restrict__ q_all,
                                                         const u16* __restrict__ K, int U, int n,
                                                         float scale_log2, float* __restrict__ lse2) {
  constexpr int WR = 16 * RT;               // rows per wave
  constexpr int TQ = WR * kH2oWaves / G;    // prompt positions per block
  constexpr int KS = D + 8;                 // LDS row stride (bf16)
  constexpr int CH = kH2oKT * D / 8;        // 16-byte chunks of a key tile
  constexpr int PER = CH / kH2oTh;
  constexpr int KT = kH2oKT / 16;           // 16-key tiles per key tile
  constexpr int DS = D / 32;
  constexpr float NINF = -__builtin_huge_valf();
  static_assert(CH % kH2oTh == 0 && TQ >= WR && TQ % WR == 0, "whole tiles");
  __shared__ __attribute__((aligned(16))) u16 kt_s[2][kH2oKT * KS];
  const int nb = (n + TQ - 1) / TQ;
  const int u = blockIdx.x % U, p0 = (nb - 1 - (int)(blockIdx.x / U)) * TQ, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, gq = lane >> 4;
  const int head = (WR * wave) / TQ, pw0 = p0 + (WR * wave) % TQ;   // the wave's head, first position
  const u16* ku = K + (size_t)u * n * D;
  const u16* qh = q_all + ((size_t)u * G + head) * n * D;

  // the wave's rows: positions pw0 + 16 rt + l16 (B operand layout)
  bf16x8 qb[RT][DS];
  int pos[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    pos[rt] = pw0 + 16 * rt + l16;
    const int pr = min(pos[rt], n - 1);
#pragma unroll
    for (int ks = 0; ks < DS; ++ks)
      qb[rt][ks] = *reinterpret_cast<const bf16x8*>(qh + (size_t)pr * D + ks * 32 + 8 * gq);
  }
  // keys 0 .. min(n, p0 + TQ) - 1 in tiles of kH2oKT
  const int kend = min(n, p0 + TQ);
  const int ntiles = (kend + kH2oKT - 1) / kH2oKT;
  bf16x8 kr[PER];
  auto load_k = [&](int t) {   // (past the last tile: clamped rows, never used)
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = tid + k * kH2oTh;
      const int key = min(t * kH2oKT + e / (D / 8), n - 1), ch = e % (D / 8);
      kr[k] = *reinterpret_cast<const bf16x8*>(ku + (size_t)key * D + ch * 8);
    }
  };
  auto store_k = [&](u16* dst) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = tid + k * kH2oTh;
      *reinterpret_cast<bf16x8*>(dst + (e / (D / 8)) * KS + (e % (D / 8)) * 8) = kr[k];
    }
  };
  float nref[RT];   // minus the reference exponent (+inf before the first visible key)
  double srun[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    nref[rt] = -NINF;
    srun[rt] = 0.0;
  }
  load_k(0);
  store_k(kt_s[0]);
  load_k(1);
  for (int t = 0; t < ntiles; ++t) {
    const u16* cur = kt_s[t & 1];
    __syncthreads();   // tile t is in LDS, and every wave is done with tile t - 1
    store_k(kt_s[(t + 1) & 1]);
    load_k(t + 2);
    const int kt0 = t * kH2oKT;
    if (kt0 > pw0 + WR - 1) continue;   // no visible key for this wave (wave-uniform)
    // the causal test matters only on tiles that reach past the wave's first row
    const bool edge = kt0 + kH2oKT - 1 > pw0 || kt0 + kH2oKT > n;
    // acc[rt]: keys 64t + 16kt + 4gq + i, row 16rt + l16
    auto products = [&](int kt, f32x4 (&acc)[RT]) {
      bf16x8 kf[DS];
#pragma unroll
      for (int ks = 0; ks < DS; ++ks)
        kf[ks] = *reinterpret_cast<const bf16x8*>(cur + (16 * kt + l16) * KS + ks * 32 + 8 * gq);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = zero4();
#pragma unroll
      for (int ks = 0; ks < DS; ++ks)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = mfma_bf16(kf[ks], qb[rt][ks], acc[rt]);
    };
    // sums of 2^(t - ref) over the tile, per row tile
    auto tile_sums = [&](auto edge_tag, float (&a)[RT]) {
      constexpr bool EDGE = decltype(edge_tag)::value;
      f32x4 st[2][RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) a[rt] = 0.f;
      products(0, st[0]);
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        if (kt + 1 < KT) products(kt + 1, st[(kt + 1) & 1]);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float x = __builtin_amdgcn_exp2f(fmaf(st[kt & 1][rt][i], scale_log2, nref[rt]));
            if constexpr (EDGE) {
              const int key = kt0 + 16 * kt + 4 * gq + i;
              a[rt] += (key <= pos[rt] && key < n) ? x : 0.f;
            } else {
              a[rt] += x;
            }
          }
      }
    };
    float a[RT];
    if (edge) tile_sums(std::true_type{}, a);
    else tile_sums(std::false_type{}, a);
    bool moved = false;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) moved |= !(a[rt] <= 0x1p64f);
    // a new reference when a tile's sum leaves [0, 2^64] (also taken on the
    // lane's first visible key, while the reference is still -inf): rare, so
    // the tile's products are formed again
    if (__any(moved)) {
      float mx[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) mx[rt] = NINF;
#pragma unroll 1
      for (int kt = 0; kt < KT; ++kt) {
        f32x4 st[RT];
        products(kt, st);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int key = kt0 + 16 * kt + 4 * gq + i;
            if (key <= pos[rt] && key < n) mx[rt] = fmaxf(mx[rt], st[rt][i]);
          }
      }
      float b[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        b[rt] = 0.f;
        if (!(a[rt] <= 0x1p64f) && mx[rt] != NINF) {
          const float ref = ceilf(mx[rt] * scale_log2);
          srun[rt] = nref[rt] == -NINF ? 0.0 : ldexp(srun[rt], (int)(-nref[rt] - ref));
          nref[rt] = -ref;
        }
      }
#pragma unroll 1
      for (int kt = 0; kt < KT; ++kt) {
        f32x4 st[RT];
        products(kt, st);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int key = kt0 + 16 * kt + 4 * gq + i;
            const float x = __builtin_amdgcn_exp2f(fmaf(st[rt][i], scale_log2, nref[rt]));
            b[rt] += (key <= pos[rt] && key < n) ? x : 0.f;
          }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        if (!(a[rt] <= 0x1p64f)) a[rt] = b[rt];
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) srun[rt] += (double)a[rt];
  }
  // merge the four lanes of each row (exact power-of-two rescales)
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const float mref = -nref[rt];
    const float M = max_over_groups(mref);
    const double part = mref == NINF ? 0.0 : ldexp(srun[rt], (int)(mref - M));
    const double tot = sum_over_groups(part);
    if (gq == 0 && pos[rt] < n)
      lse2[((size_t)u * G + head) * n + pos[rt]] = (float)((double)M + log2(tot));
  }
}

// --------------------------------------------------------- column sums ----
template <int D, int G, int KT>
__global__ __launch_bounds__(kH2oTh) void h2o_colsum_kernel(
    const u16* __restrict__ q_all, const u16* __restrict__ K, const float* __restrict__ lse2,
    int U, int n, int P, float scale_log2, float* __restrict__ scores) {
  constexpr int TQ = kH2oQRows / G;         // positions per query tile
  constexpr int QS = D + 8;                 // LDS row stride (bf16) of Q rows
  constexpr int NR = kH2oQRows;             // rows of a query tile (head-major)
  constexpr int NRT = NR / 16;
  constexpr int CH = NR * D / 8;            // 16-byte chunks of a query tile
  constexpr int PER = CH / kH2oTh;
  constexpr int DS = D / 32;
  static_assert(CH % kH2oTh == 0 && NR <= kH2oTh && TQ % 16 == 0, "whole query tiles per block");
  __shared__ __attribute__((aligned(16))) u16 q_s[2][NR * QS];
  __shared__ float l_s[2][NR];
  const int u = blockIdx.x % U, k0 = blockIdx.x / U * 16 * KT * kH2oWaves, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, gq = lane >> 4;
  const u16* ku = K + (size_t)u * n * D;
  const u16* qu = q_all + (size_t)u * G * n * D;
  const float* lu = lse2 + (size_t)u * G * n;

  // this wave's keys (KT 16-key tiles) as A operands
  const int kb = k0 + 16 * KT * wave;
  bf16x8 kf[KT][DS];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    const int key = min(kb + 16 * kt + l16, n - 1);
#pragma unroll
    for (int ks = 0; ks < DS; ++ks)
      kf[kt][ks] = *reinterpret_cast<const bf16x8*>(ku + (size_t)key * D + ks * 32 + 8 * gq);
  }
  // query tiles at or after the block's first key
  const int qt0 = k0 / TQ, qt1 = (n + TQ - 1) / TQ;
  bf16x8 qr[PER];
  float lr = 0.f;
  auto load_q = [&](int qt) {   // (past the last tile: clamped rows, never used)
    const int pl0 = qt * TQ;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = tid + k * kH2oTh;
      const int row = e / (D / 8), ch = e % (D / 8);
      const int hg = row / TQ, pos = min(pl0 + row % TQ, n - 1);
      qr[k] = *reinterpret_cast<const bf16x8*>(qu + ((size_t)hg * n + pos) * D + ch * 8);
    }
    if (tid < NR) lr = lu[(size_t)(tid / TQ) * n + min(pl0 + tid % TQ, n - 1)];
  };
  auto store_q = [&](int b) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = tid + k * kH2oTh;
      *reinterpret_cast<bf16x8*>(&q_s[b][(e / (D / 8)) * QS + (e % (D / 8)) * 8]) = qr[k];
    }
    if (tid < NR) l_s[b][tid] = lr;
  };
  double col[KT][4];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int i = 0; i < 4; ++i) col[kt][i] = 0.0;
  load_q(qt0);
  store_q(0);
  load_q(qt0 + 1);
  for (int qt = qt0; qt < qt1; ++qt) {
    const int b = (qt - qt0) & 1;
    __syncthreads();   // tile qt is in LDS, and every wave is done with tile qt - 1
    store_q(b ^ 1);
    load_q(qt + 2);
    const int p0 = qt * TQ;
    if (p0 + TQ - 1 < kb) continue;   // before all of the wave's keys (wave-uniform)
    // the causal test and the end of the prompt matter only on tiles that
    // start before the wave's last key or run past n (wave-uniform)
    const bool edge = p0 < kb + 16 * KT - 1 || p0 + TQ > n;
    // acc[kt]: keys kb + 16kt + 4gq + i, row 16rt + l16 (head 16rt / TQ)
    auto products = [&](int rt, f32x4 (&acc)[KT], float& nl) {
      bf16x8 qf[DS];
#pragma unroll
      for (int ks = 0; ks < DS; ++ks)
        qf[ks] = *reinterpret_cast<const bf16x8*>(&q_s[b][(16 * rt + l16) * QS + ks * 32 + 8 * gq]);
      nl = -l_s[b][16 * rt + l16];
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) acc[kt] = zero4();
#pragma unroll
      for (int ks = 0; ks < DS; ++ks)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) acc[kt] = mfma_bf16(kf[kt][ks], qf[ks], acc[kt]);
    };
    float part[KT][4];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int i = 0; i < 4; ++i) part[kt][i] = 0.f;
    auto tile = [&](auto edge_tag) {
      constexpr bool EDGE = decltype(edge_tag)::value;
      f32x4 st[2][KT];
      float nl[2];
      auto consume = [&](int rt, const f32x4 (&t4)[KT], float nlr) {
        const int rpos = p0 + (16 * rt) % TQ + l16;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float x = __builtin_amdgcn_exp2f(fmaf(t4[kt][i], scale_log2, nlr));
            if constexpr (EDGE) {
              const int key = kb + 16 * kt + 4 * gq + i;
              part[kt][i] += (rpos < n && key <= rpos) ? x : 0.f;
            } else {
              part[kt][i] += x;
            }
          }
      };
      products(0, st[0], nl[0]);
#pragma unroll 1
      for (int rt = 0; rt < NRT - 2; rt += 2) {
        products(rt + 1, st[1], nl[1]);
        consume(rt, st[0], nl[0]);
        products(rt + 2, st[0], nl[0]);
        consume(rt + 1, st[1], nl[1]);
      }
      products(NRT - 1, st[1], nl[1]);
      consume(NRT - 2, st[0], nl[0]);
      consume(NRT - 1, st[1], nl[1]);
    };
    if (edge) tile(std::true_type{});
    else tile(std::false_type{});
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int i = 0; i < 4; ++i) col[kt][i] += (double)part[kt][i];
  }
  // sum over the 16 lanes (rows) sharing each key, in fp64
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double v = col[kt][i];
      v += __shfl_xor(v, 1);
      v += __shfl_xor(v, 2);
      v += __shfl_xor(v, 4);
      v += __shfl_xor(v, 8);
      const int key = kb + 16 * kt + 4 * gq + i;
      if (l16 == 0 && key < P) scores[(size_t)u * P + key] = (float)v;
    }
}

// Stationary 16-wide tiles per wave of a pass with `items` rows (or keys) per
// unit: four when that still gives two blocks per compute unit, else fewer
// (shorter blocks over more compute units).  Whole calls of 8 units of 4 heads, d =
// 128, one / two / four tiles, the rule's marked: the row pass at 8192 tokens 838 /
// 752 / 753* us, at 16384 2705 / 2350 / 2321*, one unit of 8192 473* / 510 / 607; the
// column sums at 8192 748* / 837 / 1227, at 16384 2523 / 2314* / 2935.  With 2 heads
// the four-tile column sums spill 7 registers and are still the fastest (16 units of
// 16384 2424 / 2248 / 2200*).  At d = 64 one tile less would be 6% faster at the line
// itself (8 units of 16384 1620 / 1727* / 2099) and 4% slower past it (2 heads, 24000
// 1720 / 1651* / 1840).
int h2o_tiles(int U, int64_t items) {
  for (int t = 4; t > 1; t /= 2)
    if (U * ((items + 128 * t - 1) / (128 * t)) >= 512) return t;
  return 1;
}

template <int D, int G, int T>
void launch_h2o_lse(const u16* q_all, const u16* K, int U, int n, float scale_log2, float* lse2,
                    hipStream_t s) {
  constexpr int TQ = 16 * T * kH2oWaves / G;
  hipLaunchKernelGGL((h2o_lse_kernel<D, G, T>), dim3((unsigned)((n + TQ - 1) / TQ) * U), dim3(kH2oTh), 0, s,
                     q_all, K, U, n, scale_log2, lse2);
}

template <int D, int G, int T>
void launch_h2o_colsum(const u16* q_all, const u16* K, const float* lse2, int U, int n, int P,
                       float scale_log2, float* scores, hipStream_t s) {
  constexpr int KB = 16 * T * kH2oWaves;
  hipLaunchKernelGGL((h2o_colsum_kernel<D, G, T>), dim3((unsigned)((P + KB - 1) / KB) * U), dim3(kH2oTh), 0, s,
                     q_all, K, lse2, U, n, P, scale_log2, scores);
}

template <int D, int G>
hipError_t launch_h2o_t(const u16* q_all, const u16* K, int U, int n, int P, float* lse2,
                        float* scores, hipStream_t s) {
  const float sc = (float)(1.4426950408889634 / __builtin_sqrt((double)D));
  switch (h2o_tiles(U, (int64_t)n * G)) {
    case 4: launch_h2o_lse<D, G, 4>(q_all, K, U, n, sc, lse2, s); break;
    case 2: launch_h2o_lse<D, G, 2>(q_all, K, U, n, sc, lse2, s); break;
    default: launch_h2o_lse<D, G, 1>(q_all, K, U, n, sc, lse2, s); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || P < 1) return e;
  switch (h2o_tiles(U, P)) {
    case 4: launch_h2o_colsum<D, G, 4>(q_all, K, lse2, U, n, P, sc, scores, s); break;
    case 2: launch_h2o_colsum<D, G, 2>(q_all, K, lse2, U, n, P, sc, scores, s); break;
    default: launch_h2o_colsum<D, G, 1>(q_all, K, lse2, U, n, P, sc, scores, s); break;
  }
  return hipGetLastError();
}

}  // namespace

bool h2o_supported(int dtype, int d, int G) {
  return dtype == GRKV_BF16 && (d == 64 || d == 128) && (G == 1 || G == 2 || G == 4 || G == 8);
}

hipError_t launch_h2o(const void* q_all, const void* K, int U, int G, int d, int64_t n, int P,
                      float* lse2, float* scores, hipStream_t s) {
#define GRKV_H2O(DV, GV)                                                                     \
  if (d == DV && G == GV)                                                                    \
    return launch_h2o_t<DV, GV>((const u16*)q_all, (const u16*)K, U, (int)n, P, lse2, scores, s);
  GRKV_H2O(64, 1) GRKV_H2O(64, 2) GRKV_H2O(64, 4) GRKV_H2O(64, 8)
  GRKV_H2O(128, 1) GRKV_H2O(128, 2) GRKV_H2O(128, 4) GRKV_H2O(128, 8)
#undef GRKV_H2O
  return hipErrorInvalidValue;
}

}  // namespace grkv
