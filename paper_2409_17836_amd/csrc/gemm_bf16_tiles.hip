// bf16 matrix product with the fused epilogues on tiles smaller than
// gemm_bf16.hip's 256 x 256, for products whose 256 x 256 tiles leave CUs
// idle (short batches, narrow N) or whose K is too short to hide that
// kernel's epilogue.
//
// What bounds them: with few tiles, the bytes a CU pulls.  One CU fetches at
// most about 55 GB/s when the operands are not in its L2 (its outstanding
// misses are what is limited: 16, 64 or 128 KB of loads in flight gave the
// same rate in a streaming probe; L2 hits reach 130 GB/s), so a stage of a
// 64 x 64 tile (16 KB) takes 0.28 us however deep its ring is, and a product
// gets faster by spreading its bytes over more CUs.  Hence the range of
// tiles, from 32 x 32 (8 KB per 64 of K, 0.16 us) up; pick_gemm_tile chooses.
// M = 256 rows, against the 256 x 256 tile: GPT-2 down 56.5 -> 10.1 us, o
// 21.6 -> 4.3, up 23.3 -> 6.0; 7B o 76 -> 21, down 192 -> 51 us.  For large M
// the LM head at K = 768 gains from two 256 x 128 tiles per CU, one's
// exponentials under the other's MFMAs: 32768 rows 2.74 -> 2.40 ms.
//
// Layout as in gemm_bf16.hip: A rows of BK values with 16-byte chunks
// swizzled so that the 16 lanes of a ds_read_b128 cycle hit all banks, B as
// its 1 KB MFMA blocks, both by buffer loads straight into LDS; the per-tile
// buffer resource makes rows past M read as zero.  A ring of NS stages, one
// barrier per stage: at stage s the wave waits for its own loads of stage s
// (the younger stages stay in flight), the barrier makes them everyone's and
// ends every read of stage s - 1, whose buffer then takes stage s + NS - 1.
// Every output element is the same chain of 16x16x32 MFMAs over increasing
// k as in the other two bf16 kernels, so a row's results do not depend on
// which tile computed it.
#include "gemm_tile.h"

namespace lmgc {
namespace {

// WM x WN waves, each FM 16-row blocks by FN 16-column blocks; K in stages of
// BK through a ring of NS buffers.  FN = 4: 64 consecutive columns.  FN = 2
// (WN = 1): the blocks c and c + 32 of a 64-column group, which the epilogues
// pair; two such tiles make a group.
template <int WM, int WN, int FM, int FN, int BK, int NS>
struct Shape {
  static_assert(FN == 4 || (FN == 2 && WN == 1), "whole groups or one pair of blocks");
  static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
  static constexpr int TM = 16 * FM * WM, TN = 16 * FN * WN;
  static constexpr int CH = BK / 8;                  // 16-byte chunks of an A row
  static constexpr int NA = TM * BK / 512, NB = TN * BK / 512;  // 1 KB loads of a stage
  static constexpr int LA = NA / kWaves, LB = NB / kWaves;      // per wave
  static constexpr int kStage = (NA + NB) * 64;      // 16-byte units of a stage
  static_assert(NA % kWaves == 0 && NB % kWaves == 0, "whole loads per wave");
};

template <int KIND, int HD, int WM, int WN, int FM, int FN, int BK, int NS, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC) void gemm_tiles_kernel(const uint16_t* __restrict__ A,
                                                                       const uint16_t* __restrict__ Bw, int M,
                                                                       int K, int ntm, int ntn, EpiArgs e) {
  using S = Shape<WM, WN, FM, FN, BK, NS>;
  constexpr int CH = S::CH, KS = BK / 32, NL = S::LA + S::LB;
  __shared__ u32x4 lds[NS * S::kStage];

  int tm, tn;
  if (!map_tile<8>(blockIdx.x, gridDim.x, ntm, ntn, tm, tn)) return;
  const int m0 = tm * S::TM;
  const int n0 = FN == 4 ? tn * S::TN : (tn >> 1) * 64 + (tn & 1) * 16;  // first column (of a block)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int kq = lane >> 4;

  const __amdgpu_buffer_rsrc_t ra = make_rsrc(A + (int64_t)m0 * K, min(M - m0, S::TM) * K * 2);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(Bw + (int64_t)n0 * K, (FN == 4 ? S::TN : 48) * K * 2);
  auto swz = [](int row) __attribute__((always_inline)) { return CH == 8 ? (row >> 1) & 7 : (row >> 2) & 3; };
  static_assert(S::LA <= 8 && S::LB <= 8, "offset arrays");
  int va[8], vb[8];
#pragma unroll
  for (int i = 0; i < S::LA; i++) {
    const int q = wave * S::LA + i;
    const int row = q * (64 / CH) + lane / CH;
    va[i] = (row * K + ((lane % CH) ^ swz(row)) * 8) * 2;
  }
#pragma unroll
  for (int i = 0; i < S::LB; i++) {
    const int q = wave * S::LB + i;
    const int kc = q / (S::TN / 16), j = q % (S::TN / 16);
    vb[i] = ((FN == 4 ? j : 2 * j) * (K / 32) + kc) * 1024 + lane * 16;
  }
  auto load = [&](u32x4* buf, int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < S::LA; i++)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr_t)(buf + (wave * S::LA + i) * 64), 16, va[i], k0 * 2, 0, 0);
#pragma unroll
    for (int i = 0; i < S::LB; i++)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_ptr_t)(buf + (S::NA + wave * S::LB + i) * 64), 16, vb[i],
                                               k0 * 32, 0, 0);
  };
  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; i++)
#pragma unroll
    for (int j = 0; j < FN; j++) acc[i][j] = f32x4{};

  const int nk = K / BK;
  u32x4* wr = lds;  // buffer of the next stage to load
  u32x4* rd = lds;  // buffer of the next stage to read
  auto next = [&](u32x4* p) __attribute__((always_inline)) {
    p += S::kStage;
    return p == lds + NS * S::kStage ? lds : p;
  };
#pragma unroll
  for (int s = 0; s < NS - 1; s++) {
    if (s < nk) load(wr, s * BK);
    wr = next(wr);
  }
  bf16x8 fa[KS][FM], fb[KS][FN];
  auto fetch = [&](const u32x4* buf, int ks) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < FN; j++)
      fb[ks][j] = as_bf16x8(buf[S::NA * 64 + (ks * (S::TN / 16) + wn * FN + j) * 64 + lane]);
#pragma unroll
    for (int i = 0; i < FM; i++) {
      const int row = wm * 16 * FM + 16 * i + (lane & 15);
      fa[ks][i] = as_bf16x8(buf[row * CH + ((ks * 4 + kq) ^ swz(row))]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mma = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < FM; i++)
#pragma unroll
      for (int j = 0; j < FN; j++)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto compute = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ks++) fetch(rd, ks);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) mma(ks);
    rd = next(rd);
  };
  int s = 0;
  for (; s + NS - 1 < nk; s++) {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * NL));
    barrier();
    load(wr, (s + NS - 1) * BK);
    wr = next(wr);
    compute();
  }
  auto tail = [&](auto self, auto t_tag) __attribute__((always_inline)) -> void {
    constexpr int T = decltype(t_tag)::value;  // stages after this one
    if (nk > T) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(T * NL));
      barrier();
      compute();
    }
    if constexpr (T > 0) self(self, std::integral_constant<int, T - 1>{});
  };
  tail(tail, std::integral_constant<int, NS - 2>{});

  const int c0 = n0 + wn * 64 + (lane & 15);
  const int rb0 = m0 + wm * 16 * FM + 4 * kq;
  using E = Epi<uint16_t, KIND, HD>;
  if constexpr (KIND == EPI_HEAD) {
    static_assert(FN == 4, "a head group is 64 columns of one wave");
    bool ok[4];
    int aidx[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      ok[j] = c0 + 16 * j < e.N;
      aidx[j] = ok[j] ? alpha_index(e, c0 + 16 * j) : -1;
    }
    const bool any_alpha = __any(aidx[0] >= 0 || aidx[1] >= 0 || aidx[2] >= 0 || aidx[3] >= 0);
#pragma unroll
    for (int i = 0; i < FM; i++) {
      float z[4][4];
#pragma unroll
      for (int r = 0; r < 4; r++)
#pragma unroll
        for (int j = 0; j < 4; j++) z[r][j] = ok[j] ? acc[i][j][r] : -INFINITY;
      head_rows4(e, z, aidx, any_alpha, rb0 + 16 * i, M, (n0 >> 6) + wn, lane & 15);
    }
  } else {
    constexpr bool kQkv = KIND == EPI_QKV_ROPE || KIND == EPI_QKV_BIAS;
    constexpr int NP = FN / 2;  // column pairs (c, c + 32) of a lane
    ColInfo ci[NP];
#pragma unroll
    for (int p = 0; p < NP; p++) ci[p] = E::column(e, c0 + 16 * p);
    if constexpr (kQkv) {
#pragma unroll
      for (int p = 0; p < NP; p++) {
        ci[p].valid = __builtin_amdgcn_readfirstlane((int)ci[p].valid) != 0;
        ci[p].seg = __builtin_amdgcn_readfirstlane(ci[p].seg);
        ci[p].seg2 = __builtin_amdgcn_readfirstlane(ci[p].seg2);
        ci[p].head = __builtin_amdgcn_readfirstlane(ci[p].head);
        ci[p].head2 = __builtin_amdgcn_readfirstlane(ci[p].head2);
      }
    }
    const int W = e.W > 0 ? e.W : 1;
    auto rows = [&](auto full_tag) __attribute__((always_inline)) {
      constexpr bool FULL = decltype(full_tag)::value;
      // the reads of row blocks i + 1 .. i + PF are in flight while block i is
      // stored
      constexpr int PF = FM < 4 ? FM : 3;
      typename E::Pre4 q[PF][NP];
      auto fetch = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NP; p++)
          q[i % PF][p] = E::template pre4<FULL>(e, ci[p], c0 + 16 * p, rb0 + 16 * i, M, (rb0 + 16 * i) % W);
      };
#pragma unroll
      for (int i = 0; i < PF; i++) fetch(i);
#pragma unroll
      for (int i = 0; i < FM; i++) {
        const int r0 = rb0 + 16 * i;
        const int b = r0 / W, p0 = r0 - b * W;
#pragma unroll
        for (int p = 0; p < NP; p++) {
          const typename E::Pre4 qi = q[i % PF][p];
          const f32x4 l = acc[i][p], h = acc[i][p + NP];
          const float lo[4] = {l[0], l[1], l[2], l[3]}, hi[4] = {h[0], h[1], h[2], h[3]};
          E::template rows4<FULL>(e, ci[p], c0 + 16 * p, r0, M, b, p0, lo, hi, qi);
        }
        if (i + PF < FM) fetch(i + PF);
      }
    };
    if (m0 + S::TM <= M && n0 + (FN == 4 ? S::TN : 48) <= e.N) rows(std::true_type{});
    else rows(std::false_type{});
  }
}

template <int KIND, int HD, int WM, int WN, int FM, int FN, int BK, int NS, int OCC>
hipError_t launch_shape(const uint16_t* A, const uint16_t* B, int M, int N_pad, int K, const EpiArgs& e,
                        hipStream_t s) {
  using S = Shape<WM, WN, FM, FN, BK, NS>;
  const int ntm = (M + S::TM - 1) / S::TM, ntn = N_pad / S::TN;
  const dim3 grid((ntm * ntn + kXcds - 1) / kXcds * kXcds);
  hipLaunchKernelGGL((gemm_tiles_kernel<KIND, HD, WM, WN, FM, FN, BK, NS, OCC>), grid, dim3(S::kThreads), 0, s, A, B, M,
                     K, ntm, ntn, e);
  return hipGetLastError();
}

template <int KIND, int HD>
hipError_t launch_kind(GemmTile t, const uint16_t* A, const uint16_t* B, int M, int N_pad, int K, const EpiArgs& e,
                       hipStream_t s) {
  switch (t) {
    case GemmTile::k32x32:
      if constexpr (KIND != EPI_HEAD) return launch_shape<KIND, HD, 2, 1, 1, 2, 64, 8, 1>(A, B, M, N_pad, K, e, s);
      return hipErrorInvalidValue;
    case GemmTile::k64x64:
      return launch_shape<KIND, HD, 4, 1, 1, 4, 64, 5, 2>(A, B, M, N_pad, K, e, s);
    case GemmTile::k128x64:
      return launch_shape<KIND, HD, 4, 1, 2, 4, 64, 3, 2>(A, B, M, N_pad, K, e, s);
    case GemmTile::k128x128:
      return launch_shape<KIND, HD, 2, 2, 4, 4, 64, 2, 2>(A, B, M, N_pad, K, e, s);
    case GemmTile::k256x128:
      if constexpr (KIND == EPI_HEAD) return launch_shape<KIND, HD, 2, 2, 8, 4, 32, 3, 2>(A, B, M, N_pad, K, e, s);
      return hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace

// The tile whose modelled time is smallest.  A launch runs its tiles in
// rounds over the chip's CUs; a round takes `fixed` (launch ramp, first
// loads, epilogue) and, per 64 of K, `one` when each CU holds one tile or
// `two` when it holds two (the last round counts as `one` if at most a tile
// per CU is left).  The figures (microseconds) are fits to sweeps of the
// GPT-2, TinyLlama and 7B products over M = 8 .. 32768 on MI355X; in those the
// choice is the fastest tile or within 13 % of it.
GemmTile pick_gemm_tile(int kind, int M, int N_pad, int K) {
  struct Row {
    GemmTile t;
    int tm, tn, occ;
    double one, two, fixed;
  };
  static const Row rows[] = {
      {GemmTile::k32x32, 32, 32, 2, 0.164, 0.25, 2.4},   {GemmTile::k64x64, 64, 64, 2, 0.28, 0.45, 2.6},
      {GemmTile::k128x64, 128, 64, 2, 0.40, 0.72, 2.8},  {GemmTile::k128x128, 128, 128, 2, 0.78, 1.00, 3.0},
      {GemmTile::k256x128, 256, 128, 2, 1.50, 1.85, 3.0}, {GemmTile::k256x256, 256, 256, 1, 1.25, 1.25, 10.0},
  };
  constexpr int kCus = 256;
  const bool head = kind == EPI_HEAD;
  GemmTile best = GemmTile::k256x256;
  double best_us = 1e30;
  for (const Row& r : rows) {
    if (head ? r.t == GemmTile::k32x32 : r.t == GemmTile::k256x128) continue;
    const int64_t tiles = (int64_t)((M + r.tm - 1) / r.tm) * (N_pad / r.tn), slots = (int64_t)kCus * r.occ;
    const int64_t full = tiles / slots, rest = tiles - full * slots;
    // the head's epilogue (exponentials and row reductions) runs exposed on
    // the 256 x 256 tile, one wave per SIMD
    const double fixed = r.fixed + (head && r.t == GemmTile::k256x256 ? 3.0 : 0.0), nk = K / 64;
    const double us = full * (nk * r.two + fixed) + (rest ? nk * (rest > kCus ? r.two : r.one) + fixed : 0.0);
    if (us < best_us) {
      best_us = us;
      best = r.t;
    }
  }
  return best;
}

hipError_t launch_gemm_bf16_tiles(GemmTile t, const uint16_t* A, const uint16_t* B, int M, int N_pad, int K,
                                  const EpiArgs& e, hipStream_t s) {
  switch (e.kind) {
    case EPI_STORE_F32: return launch_kind<EPI_STORE_F32, 0>(t, A, B, M, N_pad, K, e, s);
    case EPI_HEAD: return launch_kind<EPI_HEAD, 0>(t, A, B, M, N_pad, K, e, s);
    case EPI_RESID: return launch_kind<EPI_RESID, 0>(t, A, B, M, N_pad, K, e, s);
    case EPI_SWIGLU: return launch_kind<EPI_SWIGLU, 0>(t, A, B, M, N_pad, K, e, s);
    case EPI_BIAS_GELU: return launch_kind<EPI_BIAS_GELU, 0>(t, A, B, M, N_pad, K, e, s);
    case EPI_QKV_ROPE:
      return e.hd == 128 ? launch_kind<EPI_QKV_ROPE, 128>(t, A, B, M, N_pad, K, e, s)
                         : launch_kind<EPI_QKV_ROPE, 64>(t, A, B, M, N_pad, K, e, s);
    case EPI_QKV_BIAS:
      return e.hd == 128 ? launch_kind<EPI_QKV_BIAS, 128>(t, A, B, M, N_pad, K, e, s)
                         : launch_kind<EPI_QKV_BIAS, 64>(t, A, B, M, N_pad, K, e, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lmgc
