// GEMM C = A*B for gfx950, two groups of wavefronts on alternate K steps, direct global->LDS loads.
//
// The tiles between the 256 x 256 of gemm_pp.hip and the small ones of gemm.hip: 128 columns by 128 to 256 rows. Same
// three levels as the paper's GEMM (arXiv 2503.14985, Sections 2.1-2.3); what differs from gemm_pp.hip
// is what the two wavefronts of a SIMD share. There each owns half of the tile's rows and works on every
// K step. Here four wavefronts (2 x 2, of 128 x 64 or 64 x 64 each) cover the whole tile, group 0 takes the even K
// steps and group 1 the odd ones, and their accumulators are added through LDS at the end (in that
// order). While one group multiplies its step the other one reads the operand fragments of the next
// (phases that end in a workgroup barrier, as in gemm_pp.hip).
//
// Why: reading fragments from LDS runs at 128 bytes per clock of a CU, and the fragments of a wavefront
// tile of m x n take 2 (m + n) bytes per k against m n / 1024 clocks of matrix work (four SIMDs): 128 B per
// clock for 64 x 64 and 171 for the 64 x 32 that two-group 128 x 128 tiles leave a wavefront, but 96 for
// 128 x 64. The two-group kernels' phases took what that predicts plus 230 clocks of barrier and latency:
// 0.436 us per 64 of K and 128 x 128 tile, 0.72 us for 256 x 128 as 4 x 2 wavefronts of 64 x 64 (built first).
//
// The tall tile also comes with 224, 192 and 160 rows (112, 96, 80 per wavefront): on a grid that fits one round of the chip, what is
// spent on padding rows is time (one round of 240 workgroups, 64 K steps, us, 256 / 224 / 192 / 160 rows: 51.6 / 48.7 / 47.4 / 44.5;
// 777 x 4096 x 14336 in two parts, four rows of tiles: 106.3 -> 99.0; 316 x 6784 x 10368 81.5 -> 66.2; 1142 x 4624 x 5480 97 -> 81;
// 708 x 7552 x 832 17.2 -> 13.1).
//
// LDS: a ring of R whole K steps (3 of 48 KB or less, 5 of 32 KB), operand tiles unpadded with the XOR swizzles of
// gemm_pp.hip. Step s lies in stage s % R and is read in phase s, by group s % 2, which is also the group
// that fetches it: step s + R - 1 in phase s, into the stage that the other group has read in phase s - 1.
//
// Requirements (checked by the host): those of gemm_pp.hip.
#include <type_traits>

#include "mlt_common.h"
#include "mlt_internal.h"

namespace mlt {

namespace {

constexpr int KP_NT = 512, KP_BK = 64;
constexpr int KP_GROUP_M = 4;                            // bands of 4 tile rows, as in gemm_pp.hip

template <int BM, int BN> struct KpTile {
  static constexpr int A_B = BM * KP_BK * 2, B_B = BN * KP_BK * 2, STAGE = A_B + B_B;
  static constexpr int R = BM > 128 ? 3 : 5;             // stages: as many as fit, odd (a group's steps are two apart)
  static constexpr int NL = STAGE / 1024 / 4;            // 1 KB loads per wavefront and step of its group
  static constexpr int NLA = A_B / 1024 / 4;             // of them from A
  static constexpr int S = BN + 4;                       // floats per row of a group's image of the result
  static constexpr int RPP = BM > 128 ? BM / 2 : 128;    // rows per pass of the epilogue: what two images leave room for
  static constexpr int IMG_B = 2 * RPP * S * 4;
  static constexpr int SMEM = R * STAGE > IMG_B ? R * STAGE : IMG_B;
};

}  // namespace

// TAIL: K is not a multiple of 64. K split across workgroups (part_steps > 0): as in gemm_tile_kernel.
template <typename Tag, bool TRANSB, int BM, int BN, bool TAIL>
__global__ __launch_bounds__(KP_NT, 2) void gemm_kp_kernel(
    int M, int N, int K_, const uint16_t* __restrict__ A_, int64_t lda, const uint16_t* __restrict__ B_, int64_t ldb,
    uint16_t* __restrict__ C_, int64_t ldc, int nbm, int nbn, int nxcd, int epi, const uint16_t* __restrict__ bias,
    int part_steps, int64_t part_stride) {
  typedef typename Elem<Tag>::vec8 V8;
  typedef KpTile<BM, BN> T;
  constexpr int BK = KP_BK, R = T::R, NL = T::NL, NLA = T::NLA;
  constexpr int AROW = BK * 2, BROW = BN * 2;            // bytes per row of the A (or N x K) tile, per k row of the K x N tile
  constexpr int WTM = BM / 2, WTN = BN / 2, TA = WTM / 16, TB = WTN / 16, NS = BK / 32;
  extern __shared__ __align__(16) char smem[];
  const uint16_t* A = A_;
  const uint16_t* B = B_;
  uint16_t* C = C_;
  int K = K_;
  // K split: an XCD takes the tiles of one part, or, where a part has a single row of tiles (no panel of B to share),
  // the same tiles of all parts (us, tiles / parts first: 777 x 4096 x 14336 108.2 / 106.2, 512 x 4096 x 14336 70.5 / 68.7, 1000 x 2048 x
  // 8192 45.1 / 43.5; 138 x 3840 x 14928 47.7 / 50.3)
  const int tiles = nbm * nbn;
  int logical;
  if (part_steps > 0) {
    int part;
    if (nbm > 1) {
      logical = logical_block(blockIdx.x, gridDim.x, nxcd);
      part = logical / tiles;
      logical -= part * tiles;
    } else {
      part = blockIdx.x / tiles;
      logical = logical_block(blockIdx.x - part * tiles, tiles, nxcd);
    }
    const int k_begin = part * part_steps * BK;            // < K_: the host launches no empty part
    A += k_begin;
    B += TRANSB ? (int64_t)k_begin : (int64_t)k_begin * ldb;
    K = K_ - k_begin < part_steps * BK ? K_ - k_begin : part_steps * BK;
    C = reinterpret_cast<uint16_t*>(reinterpret_cast<float*>(C_) + (int64_t)part * part_stride);
  } else {
    logical = logical_block(blockIdx.x, tiles, nxcd);
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, w = wave & 3;               // waves 0-3 / 4-7: one of each per SIMD
  const int wm = w >> 1, wn = w & 1;
  int tile_m, tile_n;
  tile_of_logical<KP_GROUP_M>(logical, nbm, nbn, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int KT = (K + BK - 1) / BK;
  const int k_tail = K - (KT - 1) * BK;                  // k values in the last step

  // ---- global -> LDS: wavefront w of a group fills blocks w*NLA .. of A and w*(NL-NLA) .. of B of the group's
  // steps; lane l owns the 16-byte slot l of a block (8 rows of 8 chunks; K x N: 4 k rows of 16 chunks)
  auto swz = [](int r) { return (r >> 1) & 7; };
  auto swz_kn = [](int k) { return 4 * (k & 3) + 2 * ((k >> 3) & 1); };
  static_assert(BN == 128, "16 chunks per k row of the K x N tile");
  const char* const a_base = reinterpret_cast<const char*>(A + (int64_t)m0 * lda);
  const char* const b_base = reinterpret_cast<const char*>(TRANSB ? B + (int64_t)n0 * ldb : B);
  const int64_t a_kstep = BK * 2, b_kstep = TRANSB ? (int64_t)BK * 2 : (int64_t)BK * ldb * 2;
  auto row_off = [&](int block, int origin, int rows, int64_t ld) -> uint32_t {
    const int r = block * 8 + lane / 8, c = (lane % 8) ^ swz(r);
    const int rr = origin + r < rows ? r : rows - 1 - origin;
    return (uint32_t)rr * (uint32_t)ld * 2u + (uint32_t)c * 16u;
  };
  uint32_t voff[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    if (i < NLA) {
      voff[i] = row_off(w * NLA + i, m0, M, lda);
    } else if (TRANSB) {
      voff[i] = row_off(w * (NL - NLA) + i - NLA, n0, N, ldb);
    } else {
      const int k = (w * (NL - NLA) + i - NLA) * 4 + lane / 16;
      const int col = n0 + ((lane % 16) ^ swz_kn(k)) * 8;
      voff[i] = (uint32_t)k * (uint32_t)ldb * 2u + (uint32_t)(col < N ? col : 0) * 2u;
    }
  }
  // (an operand that only one row or column of tiles reads is read exactly once: streaming form)
  const bool stream_a = nbn == 1, stream_b = nbm == 1;
  // last, partial K step: bytes that a chunk past K moves back to stay inside the matrix (zeroed in the
  // fragments); the lane hidden from the compiler, which would keep all values in registers otherwise
  auto tail_back = [&](int i) -> uint32_t {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    if (i < NLA || TRANSB) {
      const int r = (i < NLA ? w * NLA + i : w * (NL - NLA) + i - NLA) * 8 + ln / 8;
      const int c = (ln % 8) ^ swz(r);
      return c * 8 < k_tail ? 0u : (uint32_t)c * 16u;
    }
    const int k = (w * (NL - NLA) + i - NLA) * 4 + ln / 16;
    return k < k_tail ? 0u : (uint32_t)k * (uint32_t)ldb * 2u;
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
  auto issue = [&](int s, int stage) __attribute__((always_inline)) {
    const char* ap = a_base + (int64_t)s * a_kstep;
    const char* bp = b_base + (int64_t)s * b_kstep;
    const uint32_t da = lds0 + stage * T::STAGE + w * (NLA * 1024);
    const uint32_t db = lds0 + stage * T::STAGE + T::A_B + w * ((NL - NLA) * 1024);
    if (TAIL && s == KT - 1) {
#pragma unroll
      for (int i = 0; i < NL; ++i)
        load_lds16(i < NLA ? ap : bp, voff[i] - tail_back(i), i < NLA ? da + i * 1024 : db + (i - NLA) * 1024);
      return;
    }
    if (stream_a) {
#pragma unroll
      for (int i = 0; i < NLA; ++i) load_lds16_stream(ap, voff[i], da + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < NLA; ++i) load_lds16(ap, voff[i], da + i * 1024);
    }
    if (stream_b) {
#pragma unroll
      for (int i = NLA; i < NL; ++i) load_lds16_stream(bp, voff[i], db + (i - NLA) * 1024);
    } else {
#pragma unroll
      for (int i = NLA; i < NL; ++i) load_lds16(bp, voff[i], db + (i - NLA) * 1024);
    }
  };

  // ---- fragment addresses inside a stage: those of gemm_pp_kernel
  const int lq = lane & 15, h = lane >> 4;                // row (column) within a tile, k chunk of the slice
  int a_off[NS], b_off[4];
#pragma unroll
  for (int kk = 0; kk < NS; ++kk) a_off[kk] = (wm * WTM + lq) * AROW + (((4 * kk + h) ^ swz(lq)) * 16);
  if (TRANSB) {
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) b_off[kk] = T::A_B + (wn * WTN + lq) * AROW + (((4 * kk + h) ^ swz(lq)) * 16);
  } else {
    const int sl = lane & 15, krow = 8 * h + (sl >> 2), x = swz_kn(krow);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      b_off[j] = T::A_B + krow * BROW + (((wn * (WTN / 8) + 2 * j + ((sl & 3) >> 1)) ^ x) * 16) + 8 * (sl & 1);
  }
  static_assert(TB == 4, "b_off");

  f32x4 acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  V8 af[NS][TA], bf[NS][TB];

  // ---- schedule. Phase p ends at barrier p. Step s: read in phase s, multiplied in phase s + 1.
  int ld_stage = grp == 0 ? R - 1 : 0;                    // stage of step s + R - 1 = (s - 1) % R, s = grp
#pragma unroll
  for (int i = 0; i < (R - 1) / 2; ++i)
    if (grp + 2 * i < KT) issue(grp + 2 * i, grp + 2 * i);
  // a group's step s must have landed at barrier s - 1: of its loads only those of later steps may be in flight
  constexpr int LATER = (R - 3) / 2;                      // such steps, when all exist
  auto wait_step = [&](int s) __attribute__((always_inline)) {
    if (LATER > 0 && s + 2 * LATER < KT) __builtin_amdgcn_s_waitcnt(wait_imm(LATER * NL, 15));
    else __builtin_amdgcn_s_waitcnt(wait_imm(0, 15));
  };
  if (grp == 0) wait_step(0);
  MLT_BARRIER();
  if (grp == 1) {
    wait_step(1);
    MLT_BARRIER();
  }
  int stage = grp;                                        // of step s
  for (int s = grp; s < KT; s += 2) {
    // ---- memory phase s
    const char* st = smem + stage * T::STAGE;
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) {
#pragma unroll
      for (int i = 0; i < TA; ++i) af[kk][i] = lds_read8<V8>(st, a_off[kk] + i * 16 * AROW);
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        if (TRANSB) {
          bf[kk][j] = lds_read8<V8>(st, b_off[kk] + j * 16 * AROW);
        } else {
          const int o = b_off[j] + kk * 32 * BROW;
          bf[kk][j] = join_tr<V8>(lds_read_tr4(st, o), lds_read_tr4(st, o + 4 * BROW));
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (s + R - 1 < KT) issue(s + R - 1, ld_stage);
    __builtin_amdgcn_s_waitcnt(wait_imm(63, 0));
    if (TAIL && s == KT - 1) {
      // the 8 k values of a fragment's lane are all inside K or all past it; past it both operands become
      // zeros (one alone would leave 0 * Inf)
      const u32x4 zero4 = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int kk = 0; kk < NS; ++kk)
        if ((4 * kk + h) * 8 >= k_tail) {
#pragma unroll
          for (int i = 0; i < TA; ++i) af[kk][i] = __builtin_bit_cast(V8, zero4);
#pragma unroll
          for (int j = 0; j < TB; ++j) bf[kk][j] = __builtin_bit_cast(V8, zero4);
        }
    }
    MLT_BARRIER();
    __builtin_amdgcn_sched_barrier(0);
    // ---- compute phase s + 1
#pragma unroll
    for (int kk = 0; kk < NS; ++kk)
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = mfma16(af[kk][i], bf[kk][j], acc[i][j]);
    __builtin_amdgcn_sched_barrier(0);
    wait_step(s + 2);
    MLT_BARRIER();
    __builtin_amdgcn_sched_barrier(0);
    stage = stage + 2 >= R ? stage + 2 - R : stage + 2;
    ld_stage = ld_stage + 2 >= R ? ld_stage + 2 - R : ld_stage + 2;
  }
  if ((KT & 1) == grp) MLT_BARRIER();                     // KT + 1 phases for both groups

  // ---- epilogue: RPP rows at a time both groups park their accumulators in images of their own, and all
  // threads add the two and store row-contiguous pieces (see RowStore for what that is worth)
  float* const img = reinterpret_cast<float*>(smem);
  constexpr int S = T::S, RPP = T::RPP;
#pragma unroll
  for (int p = 0; p < BM / RPP; ++p) {
    if (p > 0) __syncthreads();
    if (BM == RPP || wm == p) {
      float* mine = img + (grp * RPP + (BM == RPP ? wm * WTM : 0) + 4 * h) * S + wn * WTN + lq;
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) *reinterpret_cast<f32_mem*>(mine + (i * 16 + r) * S + j * 16) = acc[i][j][r];
    }
    const int row0 = m0 + p * RPP;
    if (epi & (EPI_PART32 | EPI_ACC32)) {
      constexpr int CPT = BN / 4, NI = RPP * CPT / KP_NT;
      static_assert(RPP * CPT % KP_NT == 0, "whole passes");
      const int c = tid % CPT * 4, col = n0 + c;
      float* cp = reinterpret_cast<float*>(C) + (int64_t)(row0 + tid / CPT) * ldc + col;
      f32x4 old[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        old[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if ((epi & EPI_ACC32) && row0 + tid / CPT + i * (KP_NT / CPT) < M) {
          const float* src = cp + (int64_t)i * (KP_NT / CPT) * ldc;
          if (col + 4 <= N) old[i] = *reinterpret_cast<const f32x4_mem4*>(src);
          else
            for (int e = 0; e < 4; ++e)
              if (col + e < N) old[i][e] = src[e];
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int r = tid / CPT + i * (KP_NT / CPT);
        f32x4 v = *reinterpret_cast<const f32x4_mem*>(img + r * S + c);
        add4(v, *reinterpret_cast<const f32x4_mem*>(img + (RPP + r) * S + c));
        add4(v, old[i]);
        if (row0 + r < M) store_row4(v, cp + (int64_t)i * (KP_NT / CPT) * ldc, N - col, false);
      }
    } else {
      constexpr int CPT = BN / 8, NI = (RPP * CPT + KP_NT - 1) / KP_NT;
      const int c = tid % CPT * 8, col = n0 + c;
      __syncthreads();
      auto rows = [&](auto STREAM) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int r = tid / CPT + i * (KP_NT / CPT);
          const float* src = img + r * S + c;
          f32x4 lo = *reinterpret_cast<const f32x4_mem*>(src), hi = *reinterpret_cast<const f32x4_mem*>(src + 4);
          add4(lo, *reinterpret_cast<const f32x4_mem*>(src + RPP * S));
          add4(hi, *reinterpret_cast<const f32x4_mem*>(src + RPP * S + 4));
          if ((RPP * CPT % KP_NT == 0 || r < RPP) && row0 + r < M && col < N)
            store_row8<Tag, STREAM.value>(lo, hi, C + (int64_t)(row0 + r) * ldc + col, N - col, epi, bias ? bias + col : nullptr);
        }
      };
      if (epi & EPI_STREAM) rows(std::true_type{});
      else rows(std::false_type{});
    }
  }
}

template <typename Tag, bool TRANSB, int BM, int BN, bool TAIL>
static int launch_kp(const GemmArgs& g, hipStream_t s) {
  constexpr int SMEM = KpTile<BM, BN>::SMEM;
  auto kern = gemm_kp_kernel<Tag, TRANSB, BM, BN, TAIL>;
  static thread_local int configured_dev = -1;          // opt in to > 64 KB LDS once per device
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MLT_ERR_DEVICE;
  if (configured_dev != dev) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, SMEM) != hipSuccess) {
      (void)hipGetLastError();
      return MLT_ERR_LAUNCH;
    }
    configured_dev = dev;
  }
  const int nbm = (int)((g.M + BM - 1) / BM), nbn = (int)((g.N + BN - 1) / BN);
  if (g.parts <= 1) {
    hipLaunchKernelGGL(kern, dim3(nbm * nbn), dim3(KP_NT), SMEM, s, (int)g.M, (int)g.N, (int)g.K, g.A, g.lda, g.B, g.ldb,
                       g.C, g.ldc, nbm, nbn, device_xcds(), g.epi(), g.bias, 0, (int64_t)0);
    return hipGetLastError() == hipSuccess ? MLT_OK : MLT_ERR_LAUNCH;
  }
  // K split across workgroups: fp32 partial tiles into the scratch, then the fixed-order sum
  const int KT = (int)((g.K + KP_BK - 1) / KP_BK);
  const int part_steps = (KT + g.parts - 1) / g.parts;
  const int parts = (KT + part_steps - 1) / part_steps;    // no empty part
  hipLaunchKernelGGL(kern, dim3(nbm * nbn * parts), dim3(KP_NT), SMEM, s, (int)g.M, (int)g.N, (int)g.K, g.A, g.lda, g.B,
                     g.ldb, reinterpret_cast<uint16_t*>(g.scratch), g.N, nbm, nbn, device_xcds(), (int)EPI_PART32,
                     (const uint16_t*)nullptr, part_steps, g.M * g.N);
  if (hipGetLastError() != hipSuccess) return MLT_ERR_LAUNCH;
  return run_splitk_reduce(g, parts, g.M * g.N, s);
}

template <typename Tag, int BM>
static int run_kp_t(const GemmArgs& g, hipStream_t s) {
  if (g.K % KP_BK == 0) return g.transB ? launch_kp<Tag, true, BM, 128, false>(g, s) : launch_kp<Tag, false, BM, 128, false>(g, s);
  return g.transB ? launch_kp<Tag, true, BM, 128, true>(g, s) : launch_kp<Tag, false, BM, 128, true>(g, s);
}

template <typename Tag>
static int run_kp(const GemmArgs& g, int bm, hipStream_t s) {
  switch (bm) {
    case 256: return run_kp_t<Tag, 256>(g, s);
    case 224: return run_kp_t<Tag, 224>(g, s);
    case 192: return run_kp_t<Tag, 192>(g, s);
    case 160: return run_kp_t<Tag, 160>(g, s);
  }
  return run_kp_t<Tag, 128>(g, s);
}

int run_gemm_kp(const GemmArgs& g, int bm, hipStream_t s) {
  return g.dtype == MLT_BF16 ? run_kp<bf16_tag>(g, bm, s) : run_kp<f16_tag>(g, bm, s);
}

}  // namespace mlt
