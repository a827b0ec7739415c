// Adaptive per-head budgets (the head-wise allocation of Ada-KV, with which
// the paper pairs GRKV in Sec. 4): inside each layer the H heads share
// H (c - w) selected tokens, taken as the highest pooled SnapKV scores over
// all heads of the layer (ties to the lower head, then the lower position),
// and head h keeps w plus the number of its tokens taken.
//
// One block per layer (the entry point has no workspace, so blocks cannot
// share a layer).  Pooled scores are non-negative, so their fp32 bit patterns
// order like the values, and the k-th largest key T is found in one full
// sweep over the layer's scores:
//  * 8192 keys are sampled (in large layers four from each of 2048 cache
//    lines, since every line fetched costs as much as in a full sweep) and two
//    order statistics either side of rank k bisected in registers; they
//    bracket T;
//  * one sweep counts, per head, the keys at or above the bracket and appends
//    the keys inside it (a few percent) to LDS with their head, one LDS
//    atomic per wave and 32 keys per lane;
//  * radix rounds on those candidates find T, and they complete the per-head
//    counts of keys above T and equal to T (shared out in head order).
// What it costs is one compute unit's passes over the layer (1 MB at 8 heads of
// 32k): four sweeps, a histogram sweep per radix digit of the whole key and then
// the counts, took 95 us for 32 layers of 8 x 32k scores; the sample, its bisection
// and one sweep take 60.  The sample and the bisection are about 17 of them (by as
// much a call of tied scores, which stops after them, is longer than the radix).
// The bracket is used only when the exact counts confirm that it holds T and
// the candidates fit; otherwise (an unlucky sample, or heavily tied scores, which
// the sample itself shows) the
// radix select over the full keys runs: three digits of 11, 11 and 9 bits, one
// LDS histogram sweep per digit, then a counting sweep.
#include "grkv_device.h"
#include "grkv_internal.h"

namespace grkv {
namespace {

constexpr int kAdaThreads = 1024;
constexpr int kAdaMaxHeads = 128;
constexpr int kAdaUnroll = 32;    // independent loads in flight per thread
constexpr int kAdaBins = 2048;    // widest digit (11 bits)
// Each bin is kept in kAdaCopies copies (chosen by lane), so that lanes of a
// wave landing in one crowded bin (scores share few exponents) add to
// different words; the scan sums the copies.
constexpr int kAdaCopies = 16;

// The scores of one layer, kAdaUnroll coalesced loads per thread at a time;
// past the end the key is 0xFFFFFFFF, which no radix prefix of a finite
// non-negative score matches.
template <typename F>
__device__ __forceinline__ void for_keys(const uint32_t* __restrict__ key, int64_t N, F f) {
  for (int64_t e0 = 0; e0 < N; e0 += (int64_t)kAdaThreads * kAdaUnroll) {
    uint32_t x[kAdaUnroll];
#pragma unroll
    for (int k = 0; k < kAdaUnroll; ++k) {
      const int64_t e = e0 + (int64_t)k * kAdaThreads + threadIdx.x;
      x[k] = e < N ? key[e] : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int k = 0; k < kAdaUnroll; ++k) f(x[k]);
  }
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Sum over the 64 lanes of a wave (DPP within rows of 16, then the rows).
__device__ __forceinline__ uint32_t wave_sum_dpp(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, false);
  return (uint32_t)(__builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16) +
                    __builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48));
}

constexpr int kAdaWaves = kAdaThreads / 64;
constexpr int kAdaSamplePer = 8;
constexpr int kAdaSample = kAdaSamplePer * kAdaThreads;
constexpr uint32_t kAdaCand = 24576;   // candidates held in LDS
constexpr int64_t kAdaWhole = 12288;   // layers of up to this many keys: every key is one
// Ranks a bracket may span: its ends are rounded outwards, and the keys between
// two sampled ranks vary by their root times the sampling stride (1300 where four
// standard deviations of a rank just fit).
constexpr int64_t kAdaInside = 18432;
constexpr uint32_t kAdaTop = 0x7F800001u;
constexpr uint32_t kAdaSlack = 256u;
constexpr int64_t kAdaSparse = 65536;  // four samples span at least 32 keys (one line) from here

// LDS of the one-sweep search, over the histogram area of the full radix.
struct AdaLds {
  uint32_t key[kAdaCand];
  uint8_t head[kAdaCand];
  uint32_t part[2][2][kAdaWaves];   // alternating halves: one barrier per step
  uint32_t hist[256];
  uint32_t sh[4];
  uint32_t n;
};
static_assert(sizeof(AdaLds) <= sizeof(uint32_t) * kAdaBins * kAdaCopies, "fits the histogram area");

// T by the sampled bracket; gt and eq (zeroed) receive the per-head counts.
// Returns false, with gt and eq unchanged, when the bracket does not hold.
__device__ bool bracket_search(const uint32_t* __restrict__ key, int64_t N, int H, int P,
                               uint32_t kk, AdaLds& w, uint32_t* gt, uint32_t* eq) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int parity = 0;
  // block totals of two counts per thread
  auto totals = [&](uint32_t c0, uint32_t c1, uint32_t& t0, uint32_t& t1) {
    c0 = wave_sum_dpp(c0);
    c1 = wave_sum_dpp(c1);
    if (lane == 0) { w.part[parity][0][wave] = c0; w.part[parity][1][wave] = c1; }
    __syncthreads();
    t0 = t1 = 0;
#pragma unroll
    for (int q = 0; q < kAdaWaves; ++q) { t0 += w.part[parity][0][q]; t1 += w.part[parity][1][q]; }
    t0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)t0);
    t1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)t1);
    parity ^= 1;
  };
  // 1. the bracket [lo, hi): the samples about four or five standard deviations
  // + 8 ranks either side of rank r = k / stride (fewer where they would hold more
  // keys than fit), each bisected until few samples lie between its
  // ends (or kAdaSlack units in the last place) and kept on its safe side.  (Five, of independent samples, where four samples share a line:
  // scores of neighbouring positions go together.  With four and half the room
  // for candidates, 1 to 7% of such layers with scores in runs of 32 alike missed T
  // or did not fit, and calls of 32 of them took 141 us at 8 x 32k scores and 345 at
  // 8 x 93k, where the radix takes 95 and 250; now 67 and 123, and independent
  // scores 59.9 where they took 58.4.  Bisected to a fixed 2^-8 relative, scores
  // within a few percent of each other did not fit either: 142 us, now 64.)
  uint32_t lo = 0u, hi = kAdaTop;
  const bool whole = N <= kAdaWhole;   // every key is inside
  if (!whole) {
    // (few heads of fewer keys than that pattern is for: the radix's sweeps are as
    // short as the bisection; 30000 keys of one head 21.9 us against 25.1, 63366 31.5 /
    // 32.7, three heads of 10655 27 / 29, four of 5000 29 / 27)
    if (N < kAdaSparse && H <= (N <= (int64_t)kAdaThreads * kAdaUnroll ? 3 : 2)) return false;
    // sample i is key i * stride, or (layers of at least kAdaSparse keys) key
    // (i / 4) * 4 stride + 8 (i % 4): of four neighbouring samples' span, the
    // first 25 keys
    const int64_t stride = (N + kAdaSample - 1) / kAdaSample;
    const int ns = (int)((N + stride - 1) / stride);
    const bool sparse = N >= kAdaSparse;
    // (four standard deviations of a sampled rank at least: with fewer the
    // bracket often misses T, and the sweep is lost)
    const int r = (int)((int64_t)kk / stride);
    const float sd = sqrtf((float)r * (1.f - fminf((float)r / ns, 1.f)));
    const int delta = min((sparse ? 5 : 4) * (int)sd + 8, (int)(kAdaInside / (2 * stride)));
    if (delta < 4.f * sd + 1.f) return false;
    uint32_t sv[kAdaSamplePer];
#pragma unroll
    for (int m = 0; m < kAdaSamplePer; ++m) {
      const int i = tid + m * kAdaThreads;
      const int64_t j = sparse ? (int64_t)(i >> 2) * (4 * stride) + 8 * (i & 3) : (int64_t)i * stride;
      const uint32_t x = key[j < N ? j : N - 1];
      sv[m] = i < ns && j < N ? x : 0u;
    }
    const bool act[2] = {r - delta >= 0, r + delta < ns};
    const uint32_t J[2] = {(uint32_t)(r - delta), (uint32_t)(r + delta)};
    uint32_t L[2] = {0u, 0u}, U[2] = {kAdaTop, kAdaTop};
    // (samples at or above L and U: a bound is near enough once few lie between)
    uint32_t cL[2] = {(uint32_t)ns, (uint32_t)ns}, cU[2] = {0u, 0u};
    const uint32_t near = (uint32_t)(4 + delta / 32);
#pragma unroll 1
    for (int it = 0; it < 32; ++it) {
      const bool go0 = act[0] && cL[0] - cU[0] > near && U[0] - L[0] > kAdaSlack;
      const bool go1 = act[1] && cL[1] - cU[1] > near && U[1] - L[1] > kAdaSlack;
      if (!go0 && !go1) break;
      const uint32_t m0 = L[0] + (U[0] - L[0]) / 2, m1 = L[1] + (U[1] - L[1]) / 2;
      uint32_t c0 = 0, c1 = 0, t0, t1;
#pragma unroll
      for (int m = 0; m < kAdaSamplePer; ++m) {
        c0 += sv[m] >= m0;
        c1 += sv[m] >= m1;
      }
      totals(c0, c1, t0, t1);
      if (go0) { if (t0 > J[0]) { L[0] = m0; cL[0] = t0; } else { U[0] = m0; cU[0] = t0; } }
      if (go1) { if (t1 > J[1]) { L[1] = m1; cL[1] = t1; } else { U[1] = m1; cU[1] = t1; } }
    }
    if (act[0]) hi = U[0];
    if (act[1]) lo = L[1];
    if (!(lo < hi)) return false;
    // far more samples between the bounds than the ranks chosen: tied scores,
    // which would not fit (32 layers of 8 x 32k scores of two values 115 us, with the
    // sweep first 151)
    if ((int64_t)(cL[1] - cU[0]) * stride > 3 * (int64_t)kAdaCand / 2) return false;
  }
  // 2. one sweep: keys at or above hi counted, keys in [lo, hi) appended.  A
  // wave takes a segment of one head at a time (up to kAdaUnroll keys a lane;
  // shorter where the waves outnumber the heads), so layers of short heads
  // keep every lane's loads in flight: 8 heads of 3.3k keys 25 us a call (head
  // by head 48, the radix 39), 128 heads of 500 63 us (442, 336).
  __syncthreads();
  if (tid == 0) w.n = 0u;
  __syncthreads();
  const uint32_t width = hi - lo;
  uint32_t above = 0;   // (this wave's share)
  const int want = max((P + 64 * kAdaUnroll - 1) / (64 * kAdaUnroll), max(1, kAdaWaves / H));
  const int len = ((P + want - 1) / want + 63) / 64 * 64, nseg = (P + len - 1) / len;
  for (int q = wave; q < H * nseg; q += kAdaWaves) {
    const int h = q / nseg, e0 = (q - h * nseg) * len + lane, end = min(e0 - lane + len, P);
    const uint32_t* kh = key + (size_t)h * P;
    uint32_t x[kAdaUnroll];
#pragma unroll
    for (int k = 0; k < kAdaUnroll; ++k) x[k] = kh[min(e0 + k * 64, P - 1)];
    uint32_t ch = 0, in = 0;   // in, bit k: key k lies inside the bracket
#pragma unroll
    for (int k = 0; k < kAdaUnroll; ++k) {
      const bool live = e0 + k * 64 < end;
      ch += live && x[k] >= hi;
      in |= (uint32_t)(live && x[k] - lo < width) << k;
    }
    const uint32_t cnt = __builtin_popcount(in);
    uint32_t incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t t = __shfl_up(incl, off);
      if (lane >= off) incl += t;
    }
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    uint32_t base = 0;
    if (lane == 0 && tot) base = atomicAdd(&w.n, tot);
    uint32_t o = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + incl - cnt;
    if (whole) {
#pragma unroll
      for (int k = 0; k < kAdaUnroll; ++k)
        if ((in >> k & 1u) && o < kAdaCand) { w.key[o] = x[k]; w.head[o] = (uint8_t)h; ++o; }
    } else {
      // the few keys inside are read again (from cache): a test per key of
      // the 32 in registers costs more
      while (in) {
        const int k = __builtin_ctz(in);
        in &= in - 1;
        const uint32_t y = kh[e0 + k * 64];
        if (o < kAdaCand) { w.key[o] = y; w.head[o] = (uint8_t)h; }
        ++o;
      }
    }
    ch = wave_sum_dpp(ch);
    if (lane == 0 && ch) atomicAdd(&gt[h], ch);
    above += ch;
  }
  uint32_t chi, unused;
  totals(lane == 0 ? above : 0u, 0u, chi, unused);   // the barrier also publishes the candidates
  const uint32_t L = w.n;
  uint32_t clo = chi + L;
  if (L > kAdaCand || chi >= kk || clo < kk) {   // (block-uniform)
    __syncthreads();
    for (int h = tid; h < H; h += kAdaThreads) gt[h] = 0u;
    __syncthreads();
    return false;
  }
  // 3. radix rounds on the candidates' offsets: clo >= k > chi throughout
#pragma unroll 1
  for (int it = 0; it < 5 && hi - lo > 1; ++it) {
    const int bits = 32 - __builtin_clz(hi - lo - 1);   // hi - lo - 1 < 2^bits
    const int shift = bits > 8 ? bits - 8 : 0;
    if (tid < 256) w.hist[tid] = 0u;
    __syncthreads();
    for (uint32_t e = tid; e < L; e += kAdaThreads) {
      const uint32_t x = w.key[e];
      if (x - lo < hi - lo) atomicAdd(&w.hist[(x - lo) >> shift], 1u);
    }
    __syncthreads();
    if (wave == 0) {
      // lane l holds bins 4(63 - l) .. +3: a prefix sum over the lanes counts
      // the keys at or above each lane's bins
      const int b0 = 4 * (63 - lane);
      uint32_t h4[4], suf = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) { h4[i] = w.hist[b0 + i]; suf += h4[i]; }
      uint32_t incl = suf;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off);
        if (lane >= off) incl += t;
      }
      uint32_t abv = chi + incl - suf, bc = 0, bh = 0;
      int best = -1;
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        const uint32_t c = abv + h4[i];
        if (best < 0 && c >= kk) { best = b0 + i; bc = c; bh = abv; }
        abv = c;
      }
      const uint64_t hit = __ballot(best >= 0);   // not empty: clo >= k
      if (hit && lane == __builtin_ctzll(hit)) {
        const uint64_t nh = (uint64_t)lo + ((uint64_t)(best + 1) << shift);
        w.sh[0] = lo + ((uint32_t)best << shift);
        w.sh[1] = nh < hi ? (uint32_t)nh : hi;
        w.sh[2] = bc;
        w.sh[3] = bh;
      }
    }
    __syncthreads();
    lo = w.sh[0];
    hi = w.sh[1];
    clo = w.sh[2];
    chi = w.sh[3];
    __syncthreads();
  }
  const uint32_t T = lo;
  for (uint32_t e = tid; e < L; e += kAdaThreads) {
    const uint32_t x = w.key[e];
    if (x > T) atomicAdd(&gt[w.head[e]], 1u);
    if (x == T) atomicAdd(&eq[w.head[e]], 1u);
  }
  return true;
}

__global__ __launch_bounds__(kAdaThreads) void adaptive_kernel(const float* __restrict__ pooled,
                                                               int H, int P, int64_t kk, int w,
                                                               int32_t* __restrict__ budgets) {
  __shared__ __attribute__((aligned(16))) uint32_t hist[kAdaBins * kAdaCopies];
  __shared__ uint32_t scratch[kAdaThreads / 64];
  __shared__ uint32_t gt[kAdaMaxHeads], eq[kAdaMaxHeads];
  __shared__ uint32_t pick[2];
  const int l = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int64_t N = (int64_t)H * P;
  const uint32_t* key = reinterpret_cast<const uint32_t*>(pooled + (size_t)l * N);
  if (kk > N) kk = N;
  for (int h = tid; h < H; h += kAdaThreads) gt[h] = eq[h] = 0;

  __syncthreads();
  const bool done = kk > 0 && bracket_search(key, N, H, P, (uint32_t)kk,
                                             *reinterpret_cast<AdaLds*>(hist), gt, eq);
  __syncthreads();   // hist is the search's LDS

  // digits from the top: bits 30..20, 19..9, 8..0
  constexpr int kShift[3] = {20, 9, 0};
  constexpr int kBits[3] = {11, 11, 9};
  uint32_t prefix = 0;          // the digits of T found so far, in place
  uint32_t krem = (uint32_t)kk; // rank of T among the keys matching the prefix
  if (kk > 0 && !done) {
    // a layer that one batch of loads covers is read once for the three sweeps
    // (16000 scores in two heads 24.2 -> 22.2 us)
    const bool once = N <= (int64_t)kAdaThreads * kAdaUnroll;
    uint32_t held[kAdaUnroll];
    if (once) {
#pragma unroll
      for (int k = 0; k < kAdaUnroll; ++k) {
        const int e = k * kAdaThreads + tid;
        const uint32_t x = key[min((int64_t)e, N - 1)];
        held[k] = e < N ? x : 0xFFFFFFFFu;
      }
    }
#pragma unroll
    for (int lev = 0; lev < 3; ++lev) {
      const int shift = kShift[lev], nb = 1 << kBits[lev], top = shift + kBits[lev];
      for (int b = tid; b < nb * kAdaCopies; b += kAdaThreads) hist[b] = 0;
      __syncthreads();
      const uint32_t want = prefix >> top;
      const int copy = lane & (kAdaCopies - 1);
      auto add = [&](uint32_t x) {
        if ((x >> top) == want) atomicAdd(&hist[((x >> shift) & (nb - 1)) * kAdaCopies + copy], 1u);
      };
      if (once) {
#pragma unroll
        for (int k = 0; k < kAdaUnroll; ++k) add(held[k]);
      } else {
        for_keys(key, N, add);
      }
      // (no pick when the scores break the non-negative precondition: T = 0)
      if (tid == 0) pick[0] = pick[1] = 0u;
      __syncthreads();
      // suffix counts in descending bin order: thread t holds bins
      // nb-1-2t and nb-2-2t; T's digit is the bin where the count of keys at
      // or above it first reaches krem
      const int per = nb / kAdaThreads > 0 ? nb / kAdaThreads : 1;   // 2 or 1 bins
      uint32_t v[2] = {0u, 0u};
      const int b0 = nb - 1 - per * tid;
      auto bin = [&](int b) {
        uint32_t t = 0;
#pragma unroll
        for (int k = 0; k < kAdaCopies; ++k) t += hist[b * kAdaCopies + k];
        return t;
      };
      if (b0 >= 0) {
        v[0] = bin(b0);
        if (per == 2) v[1] = bin(b0 - 1);
      }
      uint32_t tot;
      const uint32_t before = block_exclusive_scan(v[0] + v[1], scratch, &tot);
      if (b0 >= 0) {
        if (before < krem && before + v[0] >= krem) {
          pick[0] = (uint32_t)b0;
          pick[1] = before;
        } else if (per == 2 && before + v[0] < krem && before + v[0] + v[1] >= krem) {
          pick[0] = (uint32_t)(b0 - 1);
          pick[1] = before + v[0];
        }
      }
      __syncthreads();
      prefix |= pick[0] << shift;
      krem -= pick[1];   // keys of higher digits already counted
      __syncthreads();   // pick and hist are rewritten by the next level
    }
  }
  const uint32_t T = prefix;

  // keys above T and equal to T, per head (one LDS add per wave and head)
  if (kk > 0 && !done) {
    for (int h = 0; h < H; ++h) {
      uint32_t a = 0, e = 0;
      for_keys(key + (size_t)h * P, P, [&](uint32_t x) {
        a += x != 0xFFFFFFFFu && x > T;
        e += x == T;
      });
      a = wave_sum(a);
      e = wave_sum(e);
      if (lane == 0) {
        if (a) atomicAdd(&gt[h], a);
        if (e) atomicAdd(&eq[h], e);
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    int64_t above = 0;
    for (int h = 0; h < H; ++h) above += gt[h];
    int64_t need = kk > 0 ? kk - above : 0;   // keys equal to T still to take
    for (int h = 0; h < H; ++h) {
      const int64_t tie = need > 0 ? (need < (int64_t)eq[h] ? need : (int64_t)eq[h]) : 0;
      need -= tie;
      budgets[(size_t)l * H + h] = w + (int32_t)(gt[h] + tie);
    }
  }
}

}  // namespace

hipError_t launch_adaptive_budgets(const float* pooled, int layers, int H, int P, int64_t kk,
                                   int w, int32_t* budgets, hipStream_t s) {
  if (H < 1 || H > kAdaMaxHeads) return hipErrorInvalidValue;
  hipLaunchKernelGGL(adaptive_kernel, dim3(layers), dim3(kAdaThreads), 0, s, pooled, H, P, kk, w,
                     budgets);
  return hipGetLastError();
}

}  // namespace grkv
