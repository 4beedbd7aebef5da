// Serialisation kernel: values -> hex-digit + separator token windows
// (Sec. 4, "Serialization").  Each thread produces four consecutive tokens of
// the window range at a time and stores them with one 16-byte and one 4-byte
// store; the value bytes it needs are read through the cache (nine tokens
// share one float32).  The bytes to move are 4/9 read and 5 written per token
// (one separator token; 4/10 and 5 with two).  What bounded it was the
// arithmetic: with a 64-bit division by the group's length and a digit lookup
// in the kernel arguments for every token, 4M values (9 tokens each) took 82
// us, 2.5 TB/s.  Now a block divides once, its threads multiply by the
// length's reciprocal, the token ids sit in LDS and the stores are
// non-temporal (the outputs are far larger than the caches): 33 us, 6.1 TB/s.
// Blocks that reach the end of the stream or of the range do the same with a
// comparison per token (with a division per token there, sixteen in sequence,
// that block alone took 10 us, the whole launch of a short vector; 2.6 now).
#include <type_traits>

#include "common.h"

namespace lmgc {
namespace {

struct SerialDev {
  int64_t n_tokens;
  int64_t whole_groups;  // groups of the stream that are not cut off by its end
  int32_t bpv, bpg, msb_first;
  int32_t last_digits;  // tokens before the separators of the group after those
  int32_t pad_id, nsep, sep[2];  // separator tokens after each group (bins 16, 17)
  int32_t hex[16];
};

constexpr int kThreads = 256;
// Ranges of up to this many tokens take four tokens per thread, longer ones
// sixteen (so a block's division is shared by more).  Per launch, four against
// sixteen per thread: 90 thousand tokens 2.6 / 4.9 us, 900 thousand 3.6 / 4.9,
// 2.7 million 5.5 / 6.3, 4.5 million 7.2 / 7.2, 18 million 23.0 / 17.7, 37.7
// million 45.6 / 33.4.
constexpr int64_t kShortRange = 1 << 22;

// magic = ceil(2^32 / G) for groups of G tokens: x / G = (x * magic) >> 32 for
// x * G < 2^32 (here x < G + kBlockTokens and G <= 512).
template <int kRounds>
__global__ __launch_bounds__(kThreads) void serialize_kernel(const uint8_t* __restrict__ vals, SerialDev p,
                                                             uint32_t magic, int64_t t0, int64_t n_local,
                                                             int32_t* __restrict__ tokens,
                                                             uint8_t* __restrict__ sym) {
  constexpr int kBlockTokens = kThreads * 4 * kRounds;  // four tokens per thread and round
  __shared__ int32_t ids[18];
  if (threadIdx.x < 16) ids[threadIdx.x] = p.hex[threadIdx.x];
  else if (threadIdx.x < 18) ids[threadIdx.x] = p.sep[threadIdx.x - 16];
  __syncthreads();
  const int64_t first = (int64_t)blockIdx.x * kBlockTokens;  // of the range
  const int64_t tb = t0 + first;                             // in the stream
  // token r of group g: the group's digits, then its separators
  const int32_t G = p.bpg > 0 ? 2 * p.bpg + p.nsep : 2, gb = p.bpg > 0 ? p.bpg : 1;
  const int64_t g0 = tb / G;
  const uint32_t r0 = (uint32_t)(tb - g0 * G);
  const uint32_t byte0 = (uint32_t)(g0 * gb & (p.bpv - 1));  // the block's first group's byte in its value (bpv is a
  const uint8_t* src = vals + (g0 * gb - byte0);             // power of two), and that value
  const uint32_t flip = p.msb_first ? p.bpv - 1 : 0;         // k -> bpv - 1 - k within a value
  auto block = [&](auto whole_tag) __attribute__((always_inline)) {
    constexpr bool WHOLE = decltype(whole_tag)::value;
    // where the stream ends, counted like x and g below
    const int64_t end = p.n_tokens - g0 * G, cut = p.whole_groups - g0;
    const uint32_t x_end = (uint32_t)(end < 0 ? 0 : end < (1 << 30) ? end : (1 << 30));
    const uint32_t g_cut = (uint32_t)(cut < 0 ? 0 : cut < (1 << 30) ? cut : (1 << 30));
#pragma unroll
    for (int u = 0; u < kRounds; u++) {
      const uint32_t x = r0 + (u * kThreads + threadIdx.x) * 4;
      uint32_t g = __umulhi(x, magic), r = x - g * G;
      int32_t tk[4];
      uint32_t packed = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const uint32_t digits = WHOLE || g < g_cut ? 2u * gb : (uint32_t)p.last_digits;
        uint32_t bin;
        if (!WHOLE && x + e >= x_end) {
          bin = 255;
        } else if (r >= digits) {
          bin = 16 + r - digits;
        } else {
          const uint32_t byte = byte0 + g * gb + (r >> 1);
          const uint8_t b = src[byte ^ flip];
          bin = (r & 1) ? (b & 15) : (b >> 4);
        }
        tk[e] = WHOLE || bin < 18 ? ids[bin] : p.pad_id;
        packed |= bin << (8 * e);
        if (++r == (uint32_t)G) {
          r = 0;
          g++;
        }
      }
      const int64_t base = first + ((int64_t)u * kThreads + threadIdx.x) * 4;
      if (WHOLE || base + 4 <= n_local) {
        typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(i32x4{tk[0], tk[1], tk[2], tk[3]}, reinterpret_cast<i32x4*>(tokens + base));
        if (sym) __builtin_nontemporal_store(packed, reinterpret_cast<uint32_t*>(sym + base));
      } else {
        for (int e = 0; e < 4; e++) {
          if (base + e >= n_local) break;
          tokens[base + e] = tk[e];
          if (sym) sym[base + e] = (uint8_t)(packed >> (8 * e));
        }
      }
    }
  };
  // the block's tokens all lie in the range and in whole groups of the stream
  if (first + kBlockTokens <= n_local && g0 + kBlockTokens / G + 2 <= p.whole_groups) block(std::true_type{});
  else block(std::false_type{});
}

template <int kRounds>
hipError_t launch_rounds(const void* values, int64_t n_values, const lmgc_serial_params& sp, int64_t first_window,
                         int64_t n_windows, int32_t* tokens, uint8_t* sym, hipStream_t s) {
  SerialDev p;
  p.bpv = sp.bytes_per_value;
  p.bpg = sp.bytes_per_group;
  p.msb_first = sp.msb_first;
  p.pad_id = sp.pad_id;
  p.nsep = sp.sep2_id >= 0 ? 2 : 1;
  p.sep[0] = sp.sep_id;
  p.sep[1] = sp.sep2_id;
  for (int i = 0; i < 16; i++) p.hex[i] = sp.hex_ids[i];
  const int64_t gb = p.bpg > 0 ? p.bpg : 1, nbytes = n_values * (int64_t)sp.bytes_per_value;
  p.whole_groups = nbytes / gb;
  p.last_digits = 2 * (int32_t)(nbytes % gb);
  p.n_tokens = 2 * nbytes + (p.bpg > 0 ? (nbytes + gb - 1) / gb * p.nsep : 0);
  const uint32_t G = p.bpg > 0 ? 2 * p.bpg + p.nsep : 2;
  const uint32_t magic = (uint32_t)(((1ull << 32) + G - 1) / G);
  const int64_t n_local = n_windows * sp.window, blocks = (n_local + kThreads * 4 * kRounds - 1) / (kThreads * 4 * kRounds);
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(serialize_kernel<kRounds>, dim3((unsigned)blocks), dim3(kThreads), 0, s, (const uint8_t*)values, p,
                     magic, first_window * sp.window, n_local, tokens, sym);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_serialize(const void* values, int64_t n_values, const lmgc_serial_params& sp,
                            int64_t first_window, int64_t n_windows, int32_t* tokens,
                            uint8_t* sym, hipStream_t s) {
  const int64_t n_local = n_windows * sp.window;
  if (n_local == 0) return hipSuccess;
  if (n_local <= kShortRange) return launch_rounds<1>(values, n_values, sp, first_window, n_windows, tokens, sym, s);
  return launch_rounds<4>(values, n_values, sp, first_window, n_windows, tokens, sym, s);
}

}  // namespace lmgc
