// Serialisation kernel: values -> hex-digit + separator token windows
// (Sec. 4, "Serialization").  Each thread produces four consecutive tokens of
// the window range at a time and stores them with one 16-byte and one 4-byte
// store; the value bytes it needs are read through the cache (nine tokens
// share one float32).  The bytes to move are 4/9 read and 5 written per token
// (one separator token; 4/10 and 5 with two).  What bounded it was the
// arithmetic: with a 64-bit division by the group's length and a digit lookup
// in the kernel arguments for every token, 4M values (9 tokens each) took 94
// us, 2.2 TB/s.  Now a block divides once, its threads multiply by the
// length's reciprocal, and the token ids sit in LDS (73 us); non-temporal
// stores, of outputs far larger than the caches, take it to 40 us, 5.1 TB/s.
#include "common.h"

namespace lmgc {
namespace {

struct SerialDev {
  int64_t n_values, n_tokens, nbytes;
  int32_t bpv, bpg, msb_first, W;
  int32_t pad_id, nsep, sep[2];  // separator tokens after each group (bins 16, 17)
  int32_t hex[16];
};

__device__ inline void token_at(const uint8_t* __restrict__ vals, const SerialDev& p, int64_t t,
                                int32_t& tok, uint8_t& sym) {
  if (t >= p.n_tokens) {
    tok = p.pad_id;
    sym = 255;
    return;
  }
  int64_t byte;
  int sep = -1, low = 0;
  if (p.bpg > 0) {
    const int64_t G = 2 * (int64_t)p.bpg + p.nsep;  // a full group's tokens
    const int64_t g = t / G;
    const int32_t r = (int32_t)(t - g * G);
    const int64_t b0 = g * p.bpg;
    const int64_t left = p.nbytes - b0;
    const int32_t nb = left < p.bpg ? (int32_t)left : p.bpg;
    if (r >= 2 * nb) {
      sep = r - 2 * nb;  // 0 or 1
      byte = 0;
    } else {
      byte = b0 + (r >> 1);
      low = r & 1;
    }
  } else {
    byte = t >> 1;
    low = (int)(t & 1);
  }
  if (sep >= 0) {
    tok = p.sep[sep];
    sym = (uint8_t)(16 + sep);
    return;
  }
  const int64_t i = byte / p.bpv;
  const int32_t k = (int32_t)(byte - i * p.bpv);
  const int32_t mem = p.msb_first ? (p.bpv - 1 - k) : k;
  const uint8_t b = vals[i * p.bpv + mem];
  const int nib = low ? (b & 15) : (b >> 4);
  tok = p.hex[nib];
  sym = (uint8_t)nib;
}

constexpr int kThreads = 256, kRounds = 4;  // four tokens per thread and round
constexpr int kBlockTokens = kThreads * 4 * kRounds;

// magic = ceil(2^32 / G) for groups of G tokens: x / G = (x * magic) >> 32 for
// x * G < 2^32 (here x < G + kBlockTokens and G <= 512).
__global__ __launch_bounds__(kThreads) void serialize_kernel(const uint8_t* __restrict__ vals, SerialDev p,
                                                             uint32_t magic, int64_t t0, int64_t n_local,
                                                             int32_t* __restrict__ tokens,
                                                             uint8_t* __restrict__ sym) {
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
  // the block's tokens all lie in the range and in whole groups of the stream
  const bool whole = first + kBlockTokens <= n_local && (g0 + kBlockTokens / G + 2) * (int64_t)gb <= p.nbytes;
  if (!whole) {
    for (int u = 0; u < kRounds; u++) {
      const int64_t base = first + ((int64_t)u * kThreads + threadIdx.x) * 4;
      for (int e = 0; e < 4 && base + e < n_local; e++) {
        int32_t tk;
        uint8_t sy;
        token_at(vals, p, t0 + base + e, tk, sy);
        tokens[base + e] = tk;
        if (sym) sym[base + e] = sy;
      }
    }
    return;
  }
  const uint8_t* src = vals + g0 * gb / p.bpv * p.bpv;   // value of the block's first group
  const uint32_t byte0 = (uint32_t)(g0 * gb % p.bpv);    // its byte in that value
  const uint32_t flip = p.msb_first ? p.bpv - 1 : 0;     // k -> bpv - 1 - k within a value
#pragma unroll
  for (int u = 0; u < kRounds; u++) {
    const uint32_t x = r0 + (u * kThreads + threadIdx.x) * 4;
    uint32_t g = __umulhi(x, magic), r = x - g * G;
    int32_t tk[4];
    uint32_t packed = 0;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      uint32_t bin;
      if (r >= 2u * gb) {
        bin = 16 + r - 2 * gb;
      } else {
        const uint32_t byte = byte0 + g * gb + (r >> 1);
        const uint8_t b = src[byte ^ flip];  // bpv is a power of two
        bin = (r & 1) ? (b & 15) : (b >> 4);
      }
      tk[e] = ids[bin];
      packed |= bin << (8 * e);
      if (++r == (uint32_t)G) {
        r = 0;
        g++;
      }
    }
    const int64_t base = first + ((int64_t)u * kThreads + threadIdx.x) * 4;
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(i32x4{tk[0], tk[1], tk[2], tk[3]}, reinterpret_cast<i32x4*>(tokens + base));
    if (sym) __builtin_nontemporal_store(packed, reinterpret_cast<uint32_t*>(sym + base));
  }
}

}  // namespace

hipError_t launch_serialize(const void* values, int64_t n_values, const lmgc_serial_params& sp,
                            int64_t first_window, int64_t n_windows, int32_t* tokens,
                            uint8_t* sym, hipStream_t s) {
  SerialDev p;
  p.n_values = n_values;
  p.bpv = sp.bytes_per_value;
  p.bpg = sp.bytes_per_group;
  p.msb_first = sp.msb_first;
  p.W = sp.window;
  p.pad_id = sp.pad_id;
  p.nsep = sp.sep2_id >= 0 ? 2 : 1;
  p.sep[0] = sp.sep_id;
  p.sep[1] = sp.sep2_id;
  for (int i = 0; i < 16; i++) p.hex[i] = sp.hex_ids[i];
  p.nbytes = n_values * (int64_t)sp.bytes_per_value;
  p.n_tokens = 2 * p.nbytes + (sp.bytes_per_group > 0
                                   ? (p.nbytes + sp.bytes_per_group - 1) / sp.bytes_per_group * p.nsep
                                   : 0);
  const int64_t t0 = first_window * sp.window;
  const int64_t n_local = n_windows * sp.window;
  if (n_local == 0) return hipSuccess;
  const int64_t blocks = (n_local + kBlockTokens - 1) / kBlockTokens;
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  const uint32_t G = sp.bytes_per_group > 0 ? 2 * sp.bytes_per_group + p.nsep : 2;
  const uint32_t magic = (uint32_t)(((1ull << 32) + G - 1) / G);
  hipLaunchKernelGGL(serialize_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s,
                     (const uint8_t*)values, p, magic, t0, n_local, tokens, sym);
  return hipGetLastError();
}

}  // namespace lmgc
