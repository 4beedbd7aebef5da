// float32 matrix product for float32 decoders: C = A[M, K] * B[N, K]^T with
// the same fused epilogues as the bf16 kernel.  Every output is one
// sequential, k-ordered FMA chain, so results do not depend on M or on other
// rows (a decoding step runs it on one row per window and gets the same
// values).
//
// v_mfma_f32_16x16x4_f32 is that chain: C + a0 b0, + a1 b1, + a2 b2, + a3 b3,
// each a fused multiply-add rounded to nearest even with denormals kept
// (measured against fmaf on the host: 5 million results over exponents from
// 2^-149 to 2^60, signed zeros and denormal sums, all bits equal; the reverse
// order differs in half of them).  So the matrix cores (150 TFLOP/s) take over
// from vector FMAs (79 without packed instructions) with the same bits.
//
// 64 x 64 tile, four waves of 16 rows x 64 columns: a wave holds both columns
// of each epilogue pair and a whole 64-column head group.  A lane's operand
// for MFMA s of a 16-wide stage is element k = 4 s + lane / 16, so LDS holds a
// row's elements as [k % 4][k / 4] and one 16-byte read gives all four.  Two
// LDS buffers, one barrier per stage, the next stage's global loads under the
// MFMAs.  Per launch at 36864 rows, vector FMAs before -> now: gate/up (K 128,
// N 1024) 144 -> 111 us, down (K 512, N 128) and O (128, 128) 58 -> 42 us on
// average, QKV 65 -> 53 us, head 43 -> 35 us; gate/up runs at 88 TFLOP/s, bound by
// fill and epilogue around its eight stages.  Slower or no different: 128-row
// tiles (gate/up -5 %, the others +5 %), XCD-contiguous tile order.
#include "epilogue.h"

namespace lmgc {
namespace {

constexpr int TM = 64, TN = 64, TK = 16;
constexpr int LD = TK + 4;  // LDS row in floats: 16 rows' 16-byte reads fall on 64 different banks

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int KIND>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A,
                                                       const float* __restrict__ Bw, int M, int K,
                                                       EpiArgs e) {
  __shared__ __attribute__((aligned(16))) float As[2][TM * LD];
  __shared__ __attribute__((aligned(16))) float Bs[2][TN * LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
  // loader: row tid / 4, k offset (tid % 4) * 4; element k = 4 s + q of
  // a row goes to slot 4 q + s
  const int lr = tid >> 2, ls = tid & 3;
  const float* pa = A + (int64_t)min(m0 + lr, M - 1) * K + 4 * ls;
  const float* pb = Bw + (int64_t)(n0 + lr) * K + 4 * ls;
  f32x4 va, vb;
  auto load = [&](int k0) __attribute__((always_inline)) {
    va = *reinterpret_cast<const f32x4*>(pa + k0);
    vb = *reinterpret_cast<const f32x4*>(pb + k0);
  };
  auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      As[buf][lr * LD + 4 * q + ls] = va[q];
      Bs[buf][lr * LD + 4 * q + ls] = vb[q];
    }
  };
  f32x4 acc[4];
#pragma unroll
  for (int j = 0; j < 4; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  load(0);
  store(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < K; k0 += TK) {
    const bool more = k0 + TK < K;
    if (more) load(k0 + TK);
    f32x4 b[4];
    const f32x4 a = *reinterpret_cast<const f32x4*>(&As[buf][(16 * wave + l16) * LD + 4 * kq]);
#pragma unroll
    for (int j = 0; j < 4; j++) b[j] = *reinterpret_cast<const f32x4*>(&Bs[buf][(16 * j + l16) * LD + 4 * kq]);
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
      for (int j = 0; j < 4; j++) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[j][s], acc[j], 0, 0, 0);
    buf ^= 1;
    if (more) {
      store(buf);
      __syncthreads();
    }
  }
  // lane: rows row0 .. row0 + 3, columns c0 + 16 j
  const int row0 = m0 + 16 * wave + 4 * kq, c0 = n0 + l16;
  if constexpr (KIND == EPI_HEAD) {
    bool ok[4];
    int aidx[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      ok[j] = c0 + 16 * j < e.N;
      aidx[j] = ok[j] ? alpha_index(e, c0 + 16 * j) : -1;
    }
    const bool any_alpha = __any(aidx[0] >= 0 || aidx[1] >= 0 || aidx[2] >= 0 || aidx[3] >= 0);
    float z[4][4];
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
      for (int j = 0; j < 4; j++) z[r][j] = ok[j] ? acc[j][r] : -INFINITY;
    head_rows4(e, z, aidx, any_alpha, row0, M, blockIdx.x, l16);
    return;
  }
  // pairs (c0, c0 + 32) and (c0 + 16, c0 + 48)
  using E = Epi<float, KIND, 0>;
  const ColInfo ci[2] = {E::column(e, c0), E::column(e, c0 + 16)};
  const int W = e.W > 0 ? e.W : 1;
  if (KIND == EPI_RESID || (KIND == EPI_QKV_ROPE && !e.step && (W & 3) == 0)) {
    // four rows of one window (the residual add needs no window): what the
    // epilogue reads is in flight together, before the first store
    const int b = row0 / W, p0 = row0 - b * W;
    typename E::Pre4 q[2];
#pragma unroll
    for (int p = 0; p < 2; p++) q[p] = E::template pre4<false>(e, ci[p], c0 + 16 * p, row0, M, p0);
#pragma unroll
    for (int p = 0; p < 2; p++) {
      const f32x4 l = acc[p], h = acc[p + 2];
      const float lo[4] = {l[0], l[1], l[2], l[3]}, hi[4] = {h[0], h[1], h[2], h[3]};
      E::template rows4<false>(e, ci[p], c0 + 16 * p, row0, M, b, p0, lo, hi, q[p]);
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int row = row0 + r;
    if (row >= M) continue;
    const int b = e.step ? row : row / W, pos = e.step ? e.dpos : row - b * W;
#pragma unroll
    for (int p = 0; p < 2; p++) E::row(e, ci[p], c0 + 16 * p, row, b, pos, acc[p][r], acc[p + 2][r]);
  }
}

template <int KIND>
void launch_kind(const float* A, const float* B, int M, int N_pad, int K, const EpiArgs& e, hipStream_t s) {
  const dim3 grid(N_pad / TN, (M + TM - 1) / TM), block(256);
  hipLaunchKernelGGL(gemm_f32_kernel<KIND>, grid, block, 0, s, A, B, M, K, e);
}

}  // namespace

hipError_t launch_gemm_f32(const float* A, const float* B, int M, int N_pad, int K,
                           const EpiArgs& e, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (K % TK != 0 || N_pad % TN != 0) return hipErrorInvalidValue;
  switch (e.kind) {
    case EPI_STORE_F32:
      launch_kind<EPI_STORE_F32>(A, B, M, N_pad, K, e, s);
      break;
    case EPI_RESID:
      launch_kind<EPI_RESID>(A, B, M, N_pad, K, e, s);
      break;
    case EPI_QKV_ROPE:
      launch_kind<EPI_QKV_ROPE>(A, B, M, N_pad, K, e, s);
      break;
    case EPI_QKV_BIAS:
      launch_kind<EPI_QKV_BIAS>(A, B, M, N_pad, K, e, s);
      break;
    case EPI_SWIGLU:
      launch_kind<EPI_SWIGLU>(A, B, M, N_pad, K, e, s);
      break;
    case EPI_BIAS_GELU:
      launch_kind<EPI_BIAS_GELU>(A, B, M, N_pad, K, e, s);
      break;
    case EPI_HEAD:
      launch_kind<EPI_HEAD>(A, B, M, N_pad, K, e, s);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace lmgc
