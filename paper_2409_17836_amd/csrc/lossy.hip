// The lossy steps LM-GC is composed with (Sec. 5.4, "Compatibility"):
// top-k sparsification by magnitude, linear quantisation to n-bit indices
// (Eq. 4) and SignSGD sign bits.  All three are streaming passes over a
// float32 vector and bound by HBM bandwidth.
//
// Top-k is a radix select on the magnitude key (the IEEE bits with the sign
// cleared, an unsigned integer whose order is the order of |v| for numbers).
// Two passes count the keys' leading 12 bits and, among the keys that share
// the threshold's, their next 11; no digit leaves the device: every block of
// a later kernel finds them in the histograms by itself (a suffix scan of 24
// KB, against a launch of its own).  The 23 bits known then settle all keys
// but the few that share them (n / 70000 for smooth distributions), so the
// third pass over the vector writes the output and collects those candidates,
// and a wave for each ranks it by key and index.  Vectors with more candidates
// than the list holds take the last 8 bits by a third counting pass, and a
// per-chunk count of the threshold's ties before an ordered write with a block
// scan: ties are kept in index order, lowest first.  Those are vectors with
// many equal magnitudes; of values with few mantissa bits, such as those that
// came from bf16 (8 million: 64 us against 42 for normal values), from a few
// hundred thousand on; and smooth ones beyond some 70 million.
#include <algorithm>
#include <mutex>

#include "common.h"

namespace lmgc {
namespace {

constexpr int kThreads = 256;
constexpr int kGridStride = 512;        // blocks of the min/max pass, whose partials each later block merges
constexpr int kTile = kThreads * 4;     // elements per block iteration
// top-k: digits of 12, 11 and 8 bits, blocks of 1024 threads
constexpr int kTopkThreads = 1024, kTopkTile = kTopkThreads * 4;
constexpr int kBinsA = 4096, kBinsB = 2048, kBinsC = 256;
constexpr int kShiftA = 19, kShiftB = 8;
constexpr int kMaxChunks = 1024;        // ordered chunks of the tie passes
constexpr int64_t kMergeMost = 128 << 10;  // elements up to which keys alike are added at once
constexpr uint32_t kMaxCand = 1000;     // keys that share the 23-bit prefix

// Scratch of a top-k call.  A and B are counted by the first two passes.  The
// candidate list takes what the workspace has left (`cap` entries, kMaxCand at
// most); with more candidates than that the last digit's counts take its place
// and the chunks' ties that of A.  The counts lie on whole cache lines, and the
// four words of the call after them: all blocks add to the former while they
// read the latter (before them, 1 million values in a narrow range took 39.4
// us, now 37.6).
struct TopkScratch {
  union {
    uint32_t a[kBinsA];
    uint32_t ties[kMaxChunks];
  };
  uint32_t b[kBinsB];
  union {
    uint64_t cand[kMaxCand + 2];  // 128 and 129 are the four words below
    struct {
      uint32_t c[kBinsC];
      uint32_t n_cand;
      uint32_t prefix, need, count;  // of topk_split_kernel, for the kernels after it
    };
  };
  __device__ uint64_t& entry(uint32_t i) { return cand[i < 128 ? i : i + 2]; }
};

__device__ inline uint32_t mag_key(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }

// Four consecutive elements starting at i (a multiple of 4); lanes past n
// read as +0 and are marked invalid through `valid` (number of valid lanes).
__device__ inline float4 load4(const float* __restrict__ v, int64_t i, int64_t n, int& valid) {
  if (i + 4 <= n) {
    valid = 4;
    return *reinterpret_cast<const float4*>(v + i);
  }
  float t[4] = {0.f, 0.f, 0.f, 0.f};
  valid = (int)(n > i ? n - i : 0);
  for (int e = 0; e < valid; e++) t[e] = v[i + e];
  return make_float4(t[0], t[1], t[2], t[3]);
}

// Calls f(i, x, valid) for the groups of four elements i, i + stride, ... < n
// (i a multiple of 4), the loads of four groups in flight at once.
template <class F>
__device__ inline void for_each4(const float* v, int64_t i, int64_t stride, int64_t n, F&& f) {
  for (; i + 3 * stride + 4 <= n; i += 4 * stride) {
    float4 x[4];
#pragma unroll
    for (int u = 0; u < 4; u++) x[u] = *reinterpret_cast<const float4*>(v + i + u * stride);
#pragma unroll
    for (int u = 0; u < 4; u++) f(i + u * stride, x[u], 4);
  }
  for (; i < n; i += stride) {
    int valid;
    const float4 x = load4(v, i, n, valid);
    f(i, x, valid);
  }
}

__device__ inline void store4(float* __restrict__ o, int64_t i, int valid, float4 x) {
  if (valid == 4) {
    *reinterpret_cast<float4*>(o + i) = x;
  } else {
    const float t[4] = {x.x, x.y, x.z, x.w};
    for (int e = 0; e < valid; e++) o[i + e] = t[e];
  }
}

// ------------------------------------------------------------------ top-k
// The digit of the key that `need` keys (by magnitude, largest first) reach:
// bin d with fewer than `need` keys in the bins above it and at least `need`
// with its own.  Every thread of the block gets d, how many keys of bin d are
// still needed, and its count.
struct Digit {
  uint32_t d, need, count;
};
template <int NB>
__device__ inline Digit find_digit(const uint32_t* __restrict__ hist, uint32_t need) {
  constexpr int PER = NB > kTopkThreads ? NB / kTopkThreads : 1, NW = kTopkThreads / 64;
  __shared__ uint32_t wsum[NW];
  __shared__ Digit res;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, b0 = threadIdx.x * PER;
  uint32_t c[PER], own = 0;
#pragma unroll
  for (int i = 0; i < PER; i++) {
    c[i] = b0 + i < NB ? hist[b0 + i] : 0u;
    own += c[i];
  }
  uint32_t suf = own;  // bins of this thread and of the wave's later ones
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_down(suf, d);
    if (lane + d < 64) suf += y;
  }
  if (lane == 0) wsum[wave] = suf;
  __syncthreads();
  for (int w = wave + 1; w < NW; w++) suf += wsum[w];
  uint32_t above = suf - own;
#pragma unroll
  for (int i = PER - 1; i >= 0; i--) {
    if (above < need && above + c[i] >= need) res = Digit{(uint32_t)(b0 + i), need - above, c[i]};
    above += c[i];
  }
  __syncthreads();
  const Digit r = res;
  __syncthreads();  // res and wsum may be used again
  return r;
}

// The threshold's leading 23 bits, the keys still to keep among those that
// share them, and how many share them.
__device__ inline Digit find_prefix(const TopkScratch* __restrict__ sc, uint32_t k) {
  const Digit a = find_digit<kBinsA>(sc->a, k);
  const Digit b = find_digit<kBinsB>(sc->b, a.need);
  return Digit{(a.d << (kShiftA - kShiftB)) | b.d, b.need, b.count};
}

__global__ __launch_bounds__(kTopkThreads) void topk_init_kernel(TopkScratch* sc) {
  for (int i = threadIdx.x; i < kBinsA; i += kTopkThreads) sc->a[i] = 0;
  for (int i = threadIdx.x; i < kBinsB; i += kTopkThreads) sc->b[i] = 0;
  if (threadIdx.x == 0) sc->n_cand = 0;
}

// Adds the block's elements to hist: keys whose bits above `top` equal prefix
// (all of them if top == 32), by their NB-valued digit at `shift`.  MERGE: a
// thread's four keys alike are one addition (LDS atomics that meet at one
// address run one after the other, and on short vectors of one magnitude they
// are what a pass takes: 60000 values 33 -> 26 us a call; longer ones would pay
// more for the comparison than they gain).
template <int NB, bool MERGE>
__device__ inline void count_keys(const float* __restrict__ v, int64_t n, int top, uint32_t prefix, int shift,
                                  uint32_t* __restrict__ hist) {
  __shared__ uint32_t lh[NB];
  for (int i = threadIdx.x; i < NB; i += kTopkThreads) lh[i] = 0;
  __syncthreads();
  // zeros (whole runs of them in sparse vectors, whose LDS atomics would all
  // meet at one address) are counted in a register
  uint32_t zeros = 0;
  const int64_t stride = (int64_t)gridDim.x * kTopkTile;
  for_each4(v, ((int64_t)blockIdx.x * kTopkThreads + threadIdx.x) * 4, stride, n,
            [&](int64_t, float4 x, int valid) __attribute__((always_inline)) {
              const float t[4] = {x.x, x.y, x.z, x.w};
              const bool alike = MERGE && valid == 4 && mag_key(t[0]) == mag_key(t[1]) &&
                                 mag_key(t[0]) == mag_key(t[2]) && mag_key(t[0]) == mag_key(t[3]);
              const uint32_t add = alike ? 4u : 1u;
#pragma unroll
              for (int e = 0; e < 4; e++) {
                const uint32_t key = mag_key(t[e]);
                const bool in = e < (alike ? 1 : valid) && (top == 32 || (key >> top) == prefix);
                if (in && key == 0) zeros += add;
                else if (in) atomicAdd(&lh[(key >> shift) & (NB - 1)], add);
              }
            });
  for (int d = 32; d >= 1; d >>= 1) zeros += __shfl_xor(zeros, d);
  if ((threadIdx.x & 63) == 0 && zeros) atomicAdd(&lh[0], zeros);
  __syncthreads();
  for (int i = threadIdx.x; i < NB; i += kTopkThreads) {
    const uint32_t c = lh[i];
    if (c) atomicAdd(&hist[i], c);
  }
}

template <bool MERGE>
__global__ __launch_bounds__(kTopkThreads) void topk_count_a_kernel(const float* __restrict__ v, int64_t n,
                                                                    TopkScratch* sc) {
  count_keys<kBinsA, MERGE>(v, n, 32, 0, kShiftA, sc->a);
}

template <bool MERGE>
__global__ __launch_bounds__(kTopkThreads) void topk_count_b_kernel(const float* __restrict__ v, int64_t n, uint32_t k,
                                                                    TopkScratch* sc) {
  const Digit a = find_digit<kBinsA>(sc->a, k);
  count_keys<kBinsB, MERGE>(v, n, kShiftA, a.d, kShiftB, sc->b);
}

// Keeps the keys above the prefix, zeroes those below, and keeps and lists the
// ones that share it.  With too many of those the vector is left to
// topk_write_kernel.
__global__ __launch_bounds__(kTopkThreads) void topk_split_kernel(const float* v, int64_t n, uint32_t k,
                                                                  uint32_t cap, TopkScratch* sc, float* out) {
  const Digit p = find_prefix(sc, k);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc->prefix = p.d;
    sc->need = p.need;
    sc->count = p.count;
  }
  if (p.count > cap) {
    if (blockIdx.x == 0 && threadIdx.x < kBinsC) sc->c[threadIdx.x] = 0;
    return;
  }
  const int64_t stride = (int64_t)gridDim.x * kTopkTile;
  for_each4(v, ((int64_t)blockIdx.x * kTopkThreads + threadIdx.x) * 4, stride, n,
            [&](int64_t i, float4 x, int valid) __attribute__((always_inline)) {
              float t[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
              for (int e = 0; e < 4; e++) {
                const uint32_t key = mag_key(t[e]), pre = key >> kShiftB;
                if (e < valid && pre == p.d) {  // larger keys first, then lower indices
                  const uint32_t at = atomicAdd(&sc->n_cand, 1u);
                  if (at < cap) sc->entry(at) = ((uint64_t)key << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)(i + e));
                }
                if (pre < p.d) t[e] = 0.0f;
              }
              store4(out, i, valid, make_float4(t[0], t[1], t[2], t[3]));
            });
}

// Few candidates: a wave per candidate ranks it and zeroes it if it comes
// after the `need`-th.  Many: the last digit's counts.
// (Overlapping calls on one scratch find each other's list and its length; the
// checks of the slot above and of the index here keep them in bounds, with
// wrong values and no more.)
template <bool MERGE>
__global__ __launch_bounds__(kTopkThreads) void topk_finish_kernel(const float* v, int64_t n, uint32_t cap,
                                                                   TopkScratch* sc, float* out) {
  const uint32_t need = sc->need, count = sc->count;
  if (count > cap) {
    count_keys<kBinsC, MERGE>(v, n, kShiftB, sc->prefix, 0, sc->c);
    return;
  }
  if (need == count) return;
  const int lane = threadIdx.x & 63;
  const uint32_t waves = gridDim.x * (kTopkThreads / 64);
  for (uint32_t i = blockIdx.x * (kTopkThreads / 64) + (threadIdx.x >> 6); i < count; i += waves) {
    const uint64_t mine = sc->entry(i);
    uint32_t rank = 0;
    for (uint32_t j = lane; j < count; j += 64) rank += sc->entry(j) > mine ? 1u : 0u;
    for (int d = 32; d >= 1; d >>= 1) rank += __shfl_xor(rank, d);
    const uint32_t at = 0xFFFFFFFFu - (uint32_t)mine;
    if (lane == 0 && rank >= need && at < n) out[at] = 0.0f;
  }
}

// The whole threshold key, and how many keys equal to it are kept.
__device__ inline Digit find_key(const TopkScratch* __restrict__ sc) {
  const Digit c = find_digit<kBinsC>(sc->c, sc->need);
  return Digit{(sc->prefix << kShiftB) | c.d, c.need, c.count};
}

// Per chunk: how many keys equal the threshold.
__global__ __launch_bounds__(kTopkThreads) void topk_tie_count_kernel(const float* __restrict__ v, int64_t n,
                                                                      int64_t chunk, uint32_t cap, TopkScratch* sc) {
  __shared__ uint32_t wsum[kTopkThreads / 64];
  if (sc->count <= cap) return;
  const uint32_t T = find_key(sc).d;
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
  uint32_t cnt = 0;
  for (int64_t i = c0 + threadIdx.x * 4; i < c1; i += kTopkTile) {
    int valid;
    const float4 x = load4(v, i, c1, valid);
    const float t[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int e = 0; e < 4; e++) cnt += (e < valid && mag_key(t[e]) == T) ? 1u : 0u;
  }
  for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (int w = 0; w < kTopkThreads / 64; w++) s += wsum[w];
    sc->ties[blockIdx.x] = s;
  }
}

// Ordered pass over one chunk: keep keys above T, and keys equal to T whose
// rank among equal keys (in index order) is below `need`.
__global__ __launch_bounds__(kTopkThreads) void topk_write_kernel(const float* v, int64_t n, int64_t chunk, uint32_t cap,
                                                                  const TopkScratch* __restrict__ sc, float* out) {
  constexpr int NW = kTopkThreads / 64;
  __shared__ uint32_t wtot[2][NW];
  __shared__ uint32_t base_sh;
  if (sc->count <= cap) return;
  const Digit th = find_key(sc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t T = th.d, need = th.need;
  // equal keys in the chunks before this one
  uint32_t before = 0;
  for (int b = threadIdx.x; b < (int)blockIdx.x; b += kTopkThreads) before += sc->ties[b];
  for (int d = 32; d >= 1; d >>= 1) before += __shfl_xor(before, d);
  if (lane == 0) wtot[0][wave] = before;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (int w = 0; w < NW; w++) s += wtot[0][w];
    base_sh = s;
  }
  __syncthreads();
  uint32_t running = base_sh;
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
  int buf = 1;
  for (int64_t i0 = c0; i0 < c1; i0 += kTopkTile) {
    const int64_t i = i0 + threadIdx.x * 4;
    int valid;
    const float4 x = load4(v, i, c1, valid);
    float t[4] = {x.x, x.y, x.z, x.w};
    uint32_t key[4], eq = 0;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      key[e] = mag_key(t[e]);
      eq += (e < valid && key[e] == T) ? 1u : 0u;
    }
    // inclusive scan of eq over the wave, then over the waves
    uint32_t inc = eq;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d);
      if (lane >= d) inc += y;
    }
    if (lane == 63) wtot[buf][wave] = inc;
    __syncthreads();
    uint32_t woff = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NW; w++) {
      const uint32_t s = wtot[buf][w];
      woff += (w < wave) ? s : 0u;
      tot += s;
    }
    uint32_t rank = running + woff + inc - eq;  // equal keys before this thread's first element
#pragma unroll
    for (int e = 0; e < 4; e++) {
      bool keep = e < valid && key[e] > T;
      if (e < valid && key[e] == T) {
        keep = rank < need;
        rank++;
      }
      if (!keep) t[e] = 0.0f;
    }
    if (valid > 0) store4(out, i, valid, make_float4(t[0], t[1], t[2], t[3]));
    running += tot;
    buf ^= 1;  // the next tile writes the other buffer; this one is read by all before then
  }
}

constexpr int kSmall = 8 * kTopkTile;

// The bin that most of the wave's lanes hold, if that is one of two lanes' and
// at least kCrowd hold it; kNoBin otherwise.
constexpr int kCrowd = 12;  // (the fullest of the first digit's bins has 3 of 64 normal values)
constexpr uint32_t kNoBin = 0xFFFFFFFFu;
__device__ inline uint32_t crowded_bin(uint32_t bin) {
  uint32_t hot = kNoBin;
  int most = kCrowd - 1;
#pragma unroll
  for (int c = 0; c < 2; c++) {
    const uint32_t b = __builtin_amdgcn_readlane(bin, 21 * c);
    const int same = __popcll(__ballot(bin == b));
    if (b != kNoBin && same > most) most = same, hot = b;
  }
  return hot;
}

// A thread's elements of topk_small_kernel, read again: the bin that the
// samples crowd in is counted in a register.
__device__ inline void count_crowded(const float* v, int n, bool sampled, uint32_t sample, uint32_t* h, int top, uint32_t prefix,
                                     int shift, int nb) {
  auto bin = [&](uint32_t key) __attribute__((always_inline)) {
    return top == 32 || (key >> top) == prefix ? (key >> shift) & (nb - 1) : kNoBin;
  };
  const uint32_t hot = crowded_bin(sampled ? bin(sample) : kNoBin);
  uint32_t mine = 0;
#pragma unroll 1
  for (int i = threadIdx.x * 4; i < n; i += kTopkTile) {
    int valid;
    const float4 x = load4(v, i, n, valid);
    const float t[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const uint32_t b = e < valid ? bin(mag_key(t[e])) : kNoBin;
      if (b == kNoBin) continue;
      if (b == hot) mine++;
      else atomicAdd(&h[b], 1u);
    }
  }
  for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d);
  if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&h[hot], mine);
}

// Vectors of at most kSmall values in one block: the values in registers,
// the three digits' counts in LDS, ties ranked by a block scan per tile.  One
// launch where the passes above are seven.  What bounds it is LDS atomics, which
// run one after the other where they meet at one address: 32768 normal values
// 13 us, but 97 us for zeros or a single magnitude (the passes: 23 and 33).  So
// beyond two tiles (28 us at the worst) a wave that finds a fifth of a sample of
// its keys in one bin of the first digit counts each digit's crowded bin in a
// register: 31 us; the look at the sample costs the others 0.3.  TILES: 2, 4 or
// 8, whole up to a half of them, so that few instructions are for values that
// are not there.
template <int TILES>
__global__ __launch_bounds__(kTopkThreads) void topk_small_kernel(const float* v, int n, uint32_t k, float* out) {
  constexpr int NW = kTopkThreads / 64, FULL = TILES > 2 ? TILES / 2 : 0;
  constexpr bool SPREAD = TILES > 2;
  __shared__ uint32_t ha[kBinsA], hb[kBinsB], hc[kBinsC], wtot[2][NW];
  for (int i = threadIdx.x; i < kBinsA; i += kTopkThreads) ha[i] = 0;
  for (int i = threadIdx.x; i < kBinsB; i += kTopkThreads) hb[i] = 0;
  if (threadIdx.x < kBinsC) hc[threadIdx.x] = 0;
  float x[TILES][4];
  int valid[TILES];
#pragma unroll
  for (int u = 0; u < TILES; u++) {
    const int64_t i = (int64_t)u * kTopkTile + threadIdx.x * 4;
    valid[u] = 4;  // the first FULL tiles are whole
    const float4 t = u < FULL ? *reinterpret_cast<const float4*>(v + i) : load4(v, i, n, valid[u]);
    x[u][0] = t.x, x[u][1] = t.y, x[u][2] = t.z, x[u][3] = t.w;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // one key of each lane, from four tiles and all places in a float4
  uint32_t sample = 0;
  bool sampled = false;
  if constexpr (SPREAD) {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if ((lane & 3) == e) sample = mag_key(x[e * TILES / 4][e]), sampled = e < valid[e * TILES / 4];
  }
  const bool crowded = SPREAD && crowded_bin(sampled ? sample >> kShiftA : kNoBin) != kNoBin;
  __syncthreads();
  auto count = [&](uint32_t* h, int top, uint32_t prefix, int shift, int nb) __attribute__((always_inline)) {
    if (SPREAD && __builtin_expect(crowded, 0)) {
      count_crowded(v, n, sampled, sample, h, top, prefix, shift, nb);
    } else {
#pragma unroll
      for (int u = 0; u < TILES; u++) {
        if (SPREAD && u == 3 * TILES / 4 && u * kTopkTile >= n) break;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const uint32_t key = mag_key(x[u][e]);
          if (e < valid[u] && (top == 32 || (key >> top) == prefix)) atomicAdd(&h[(key >> shift) & (nb - 1)], 1u);
        }
      }
    }
    __syncthreads();
  };
  count(ha, 32, 0, kShiftA, kBinsA);
  const Digit a = find_digit<kBinsA>(ha, k);
  count(hb, kShiftA, a.d, kShiftB, kBinsB);
  const Digit b = find_digit<kBinsB>(hb, a.need);
  const uint32_t pre = (a.d << (kShiftA - kShiftB)) | b.d;
  count(hc, kShiftB, pre, 0, kBinsC);
  const Digit c = find_digit<kBinsC>(hc, b.need);
  const uint32_t T = (pre << kShiftB) | c.d;
  uint32_t running = 0;
#pragma unroll
  for (int u = 0; u < TILES; u++) {
    if (u * kTopkTile >= n) break;
    uint32_t rank = 0;
    if (c.need < c.count) {  // some of the ties go
      uint32_t eq = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) eq += (e < valid[u] && mag_key(x[u][e]) == T) ? 1u : 0u;
      uint32_t inc = eq;
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d);
        if (lane >= d) inc += y;
      }
      if (lane == 63) wtot[u & 1][wave] = inc;
      __syncthreads();
      uint32_t woff = 0, tot = 0;
#pragma unroll
      for (int w = 0; w < NW; w++) {
        const uint32_t t = wtot[u & 1][w];
        woff += w < wave ? t : 0u;
        tot += t;
      }
      rank = running + woff + inc - eq;  // equal keys before this thread's first element
      running += tot;
    }
    float t[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const uint32_t key = mag_key(x[u][e]);
      const bool keep = key > T || (key == T && rank < c.need);
      if (key == T) rank++;
      t[e] = keep ? x[u][e] : 0.0f;
    }
    store4(out, (int64_t)u * kTopkTile + threadIdx.x * 4, valid[u], make_float4(t[0], t[1], t[2], t[3]));
  }
}

__global__ void fill_zero_kernel(float* __restrict__ out, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
  if (i < n) {
    const int valid = (int)(i + 4 <= n ? 4 : n - i);
    store4(out, i, valid, make_float4(0.f, 0.f, 0.f, 0.f));
  }
}

// ----------------------------------------------------------- quantisation
__global__ __launch_bounds__(kThreads) void minmax_kernel(const float* __restrict__ v, int64_t n,
                                                          LossyMinMax* __restrict__ part) {
  __shared__ LossyMinMax ws[kThreads / 64];
  float mn = INFINITY, mx = -INFINITY;
  uint32_t bad = 0;
  for_each4(v, ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4, (int64_t)gridDim.x * kTile, n,
            [&](int64_t, float4 x, int valid) __attribute__((always_inline)) {
              const float t[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
              for (int e = 0; e < 4; e++) {
                if (e < valid) {
                  bad += isfinite(t[e]) ? 0u : 1u;
                  mn = fminf(mn, t[e]);
                  mx = fmaxf(mx, t[e]);
                }
              }
            });
  for (int d = 32; d >= 1; d >>= 1) {
    mn = fminf(mn, __shfl_xor(mn, d));
    mx = fmaxf(mx, __shfl_xor(mx, d));
    bad += __shfl_xor(bad, d);
  }
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = LossyMinMax{mn, mx, bad, 0u};
  __syncthreads();
  if (threadIdx.x == 0) {
    LossyMinMax r = ws[0];
    for (int w = 1; w < kThreads / 64; w++) {
      r.mn = fminf(r.mn, ws[w].mn);
      r.mx = fmaxf(r.mx, ws[w].mx);
      r.nonfinite += ws[w].nonfinite;
    }
    part[blockIdx.x] = r;
  }
}

// Eq. 4 in float32: one rounding per operation, no contraction, round half
// to even.  span = max - min > 0; every index lands in [0, levels].
__device__ inline uint32_t eq4_index(float x, float mn, float span, float levels) {
#pragma clang fp contract(off)
  const float t = (x - mn) / span;
  return (uint32_t)__builtin_rintf(t * levels);
}

// Every block merges the min/max partials itself (at most 16 KB from L2; a
// launch of its own took 3 us and a gap); block 0 leaves the result in res for
// the host.  Nothing is written for a vector with NaN or infinite values.
template <typename IdxT>
__global__ __launch_bounds__(kThreads) void quantize_kernel(const float* __restrict__ v, int64_t n,
                                                            const LossyMinMax* __restrict__ part, int nparts,
                                                            LossyMinMax* __restrict__ res, float levels,
                                                            IdxT* __restrict__ idx) {
  __shared__ LossyMinMax ws[kThreads / 64];
  float mn = INFINITY, mx = -INFINITY;
  uint32_t bad = 0;
  for (int b = threadIdx.x; b < nparts; b += kThreads) {
    mn = fminf(mn, part[b].mn);
    mx = fmaxf(mx, part[b].mx);
    bad += part[b].nonfinite;
  }
  for (int d = 32; d >= 1; d >>= 1) {
    mn = fminf(mn, __shfl_xor(mn, d));
    mx = fmaxf(mx, __shfl_xor(mx, d));
    bad += __shfl_xor(bad, d);
  }
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = LossyMinMax{mn, mx, bad, 0u};
  __syncthreads();
  LossyMinMax r = ws[0];
  for (int w = 1; w < kThreads / 64; w++) {
    r.mn = fminf(r.mn, ws[w].mn);
    r.mx = fmaxf(r.mx, ws[w].mx);
    r.nonfinite += ws[w].nonfinite;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *res = r;
  if (r.nonfinite) return;
  mn = r.mn;
  mx = r.mx;
  const float span = mx - mn;
  for_each4(v, ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4, (int64_t)gridDim.x * kTile, n,
            [&](int64_t i, float4 x, int valid) __attribute__((always_inline)) {
              const float t[4] = {x.x, x.y, x.z, x.w};
              uint32_t q[4];
#pragma unroll
              for (int e = 0; e < 4; e++) q[e] = mx > mn ? eq4_index(t[e], mn, span, levels) : 0u;
              if (valid == 4) {
                if constexpr (sizeof(IdxT) == 1) {
                  *reinterpret_cast<uint32_t*>(idx + i) = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
                } else {
                  *reinterpret_cast<uint2*>(idx + i) = make_uint2(q[0] | (q[1] << 16), q[2] | (q[3] << 16));
                }
              } else {
                for (int e = 0; e < valid; e++) idx[i + e] = (IdxT)q[e];
              }
            });
}

// ------------------------------------------------------------------- signs
// Thread j packs values 8j..8j+7 into byte j, the first value in bit 7.
__global__ __launch_bounds__(kThreads) void sign_pack_kernel(const float* __restrict__ v, int64_t n,
                                                             uint8_t* __restrict__ out) {
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t i = j * 8;
  if (i >= n) return;
  int va, vb;
  const float4 a = load4(v, i, n, va);
  const float4 b = load4(v, i + 4, n, vb);
  const float t[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint32_t byte = 0;
#pragma unroll
  for (int e = 0; e < 8; e++) {
    const uint32_t s = (e < va + vb) ? (__float_as_uint(t[e]) >> 31) : 0u;
    byte |= s << (7 - e);
  }
  out[j] = (uint8_t)byte;
}

inline unsigned blocks_for(int64_t n, int64_t per_block) { return (unsigned)((n + per_block - 1) / per_block); }

}  // namespace

// ------------------------------------------------------------- launchers
// Top-k and min/max calls use the same bytes (one call at a time on a
// workspace): the top-k scratch, or the min/max partials and their result.
// Smaller workspaces are taken down to kLossyMinBytes, what earlier versions
// asked for: the candidate list is shorter in them (130 entries, enough for 9
// million normal values; beyond, the passes for many candidates run).
constexpr size_t kLossyBytes = std::max(sizeof(TopkScratch), (kGridStride + 1) * sizeof(LossyMinMax));
constexpr size_t kLossyMinBytes = 25632;
static_assert(kLossyBytes <= 32768, "the library-owned scratch holds it");
static_assert(offsetof(TopkScratch, count) + sizeof(uint32_t) <= kLossyMinBytes &&
                  (kGridStride + 1) * sizeof(LossyMinMax) <= kLossyMinBytes,
              "the smallest workspace holds everything but the whole candidate list");
size_t lossy_workspace_bytes() { return kLossyBytes; }
size_t lossy_min_workspace_bytes() { return kLossyMinBytes; }

int64_t topk_chunk(int64_t n) {
  // a multiple of the tile, so that only the vector's last float4 can be partial
  const int64_t per = (n + kMaxChunks - 1) / kMaxChunks;
  const int64_t c = (per + kTopkTile - 1) / kTopkTile * kTopkTile;
  return c > kTopkTile ? c : kTopkTile;
}

hipError_t launch_sparsify_topk(const float* v, int64_t n, int64_t k, float* out, void* ws, size_t ws_bytes,
                                hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (k <= 0) {
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks_for(n, kTile)), dim3(kThreads), 0, s, out, n);
    return hipGetLastError();
  }
  if (k > n) k = n;
  const uint32_t kk = (uint32_t)k;
  if (n <= kSmall) {
    const dim3 grid(1), block(kTopkThreads);
    if (n <= 2 * kTopkTile) hipLaunchKernelGGL(topk_small_kernel<2>, grid, block, 0, s, v, (int)n, kk, out);
    else if (n <= 4 * kTopkTile) hipLaunchKernelGGL(topk_small_kernel<4>, grid, block, 0, s, v, (int)n, kk, out);
    else hipLaunchKernelGGL(topk_small_kernel<8>, grid, block, 0, s, v, (int)n, kk, out);
    return hipGetLastError();
  }
  if (ws_bytes < kLossyMinBytes) return hipErrorInvalidValue;
  TopkScratch* sc = (TopkScratch*)ws;
  const uint32_t cap = (uint32_t)std::min<size_t>(kMaxCand, (ws_bytes - offsetof(TopkScratch, cand)) / sizeof(uint64_t) - 2);
  // one block per CU while the vector comes from the caches (each block also
  // adds its counts to the global ones), two beyond
  const unsigned most = n <= (32 << 20) ? 256 : 512;
  const dim3 g(std::min(most, blocks_for(n, kTopkTile))), block(kTopkThreads);
  const bool merge = n <= kMergeMost;
  hipLaunchKernelGGL(topk_init_kernel, dim3(1), block, 0, s, sc);
  if (merge) {
    hipLaunchKernelGGL(topk_count_a_kernel<true>, g, block, 0, s, v, n, sc);
    hipLaunchKernelGGL(topk_count_b_kernel<true>, g, block, 0, s, v, n, kk, sc);
  } else {
    hipLaunchKernelGGL(topk_count_a_kernel<false>, g, block, 0, s, v, n, sc);
    hipLaunchKernelGGL(topk_count_b_kernel<false>, g, block, 0, s, v, n, kk, sc);
  }
  hipLaunchKernelGGL(topk_split_kernel, g, block, 0, s, v, n, kk, cap, sc, out);
  // a wave ranks a candidate against all others in about a microsecond, so as
  // many waves as candidates, also where the vector has few blocks: 32769 values
  // of which about 1000 are candidates
  // 44 -> 32 us
  const dim3 gf(std::max(g.x, (kMaxCand * 64 + kTopkThreads - 1) / kTopkThreads));
  if (merge) hipLaunchKernelGGL(topk_finish_kernel<true>, gf, block, 0, s, v, n, cap, sc, out);
  else hipLaunchKernelGGL(topk_finish_kernel<false>, gf, block, 0, s, v, n, cap, sc, out);
  // these two return at once unless the candidates were too many
  const int64_t chunk = topk_chunk(n);
  const dim3 nchunks(blocks_for(n, chunk));
  hipLaunchKernelGGL(topk_tie_count_kernel, nchunks, block, 0, s, v, n, chunk, cap, sc);
  hipLaunchKernelGGL(topk_write_kernel, nchunks, block, 0, s, v, n, chunk, cap, (const TopkScratch*)sc, out);
  return hipGetLastError();
}

// ------------------------------------------------ library-owned scratch
// The scratch of lmgc_sparsify_topk_noalloc: a file-scope device array, one
// copy on every GPU the library runs on, held from module load until the
// process ends.  In host code `scratch` names a host-side stand-in, not a
// device address; the current device's copy is found with
// hipGetSymbolAddress (once per device, then cached) and only that address
// reaches the kernels.  The top-k kernels clear what must start at zero
// (state and histogram) themselves and write every tie count before reading
// it, so what an earlier call left there does not matter; calls that overlap
// on one GPU (two streams at once) race on it.
constexpr size_t kScratchBytes = 32768;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

hipError_t lossy_scratch(void** ptr, size_t* bytes) {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  *bytes = kScratchBytes;
  return hipSuccess;
}

LossyMinMax* lossy_minmax_slot(void* ws) { return (LossyMinMax*)ws + kGridStride; }

hipError_t launch_quantize_linear(const float* v, int64_t n, int bits, void* idx, void* ws, hipStream_t s) {
  if (n == 0) return hipSuccess;
  LossyMinMax* part = (LossyMinMax*)ws;
  const unsigned g = std::min<unsigned>(kGridStride, blocks_for(n, kTile));
  hipLaunchKernelGGL(minmax_kernel, dim3(g), dim3(kThreads), 0, s, v, n, part);
  const float levels = (float)((1u << bits) - 1u);
  const dim3 grid(std::min<unsigned>(2048, blocks_for(n, kTile))), block(kThreads);
  if (bits <= 8)
    hipLaunchKernelGGL(quantize_kernel<uint8_t>, grid, block, 0, s, v, n, (const LossyMinMax*)part, (int)g,
                       lossy_minmax_slot(ws), levels, (uint8_t*)idx);
  else
    hipLaunchKernelGGL(quantize_kernel<uint16_t>, grid, block, 0, s, v, n, (const LossyMinMax*)part, (int)g,
                       lossy_minmax_slot(ws), levels, (uint16_t*)idx);
  return hipGetLastError();
}

hipError_t launch_sign_pack(const float* v, int64_t n, uint8_t* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t nbytes = (n + 7) / 8;
  hipLaunchKernelGGL(sign_pack_kernel, dim3(blocks_for(nbytes, kThreads)), dim3(kThreads), 0, s, v, n, out);
  return hipGetLastError();
}

}  // namespace lmgc
