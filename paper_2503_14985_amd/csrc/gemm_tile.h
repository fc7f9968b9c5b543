// The register-staged GEMM tile kernel, its second pass for a K split across workgroups, and their
// launcher. gemm.hip instantiates it for operands that allow aligned 16-byte accesses, gemm_any.hip
// for operands of any alignment.
#pragma once

#include <type_traits>

#include "mlt_common.h"
#include "mlt_internal.h"

namespace mlt {

// ------------------------------------------------------------------------------------------
// Main kernel. AL: requirements checked by the host: K % 8 == 0, lda % 8 == 0, ldb % 8 == 0,
// N % 8 == 0 when B is K x N row-major, A and B 16-byte aligned. !AL: K >= 8, and N >= 8 when B is
// K x N row-major, nothing else. M, N and K need not be multiples of the tile: out-of-range rows
// are clamped on load (their products land in accumulator rows/columns that are never stored) and
// the K tail is zero-filled.
//
// Operands of any alignment (!AL) take the same 16-byte global loads, at 2-byte alignment (the
// memory path splits an access that crosses a line, nothing else changes), and the same aligned
// LDS writes. A 16-byte chunk that would run over the end of its row is loaded from 8 elements
// before that end instead, so no access ever leaves the row, and shifted into place on its way to
// LDS: along k only in the last K step, along n (row-major B) only in the workgroups of the last
// column of tiles.
//
// LDS layout per stage (elements are 16-bit):
//   A tile   [BM][BK + 8]          k contiguous; the 16-byte pad makes the row stride 36 dwords,
//                                  so 16 consecutive rows at one k offset fall in 16 distinct
//                                  4-bank groups of the 64 banks
//   B tile   TRANSB:  [BN][BK + 8] same as A (global B is N x K, k contiguous)
//            !TRANSB: [BK][BN + 32] n contiguous, as in global memory; fragments are fetched with
//                                  the transposing LDS read; the 64-byte pad puts the 4 k-rows of
//                                  a 16-lane read group into disjoint bank ranges
// Two stages; global loads for step k+1 are issued before the MFMAs of step k, parked in
// registers and written to the other stage afterwards, one barrier per step.
// ------------------------------------------------------------------------------------------
template <typename Tag, int BM, int BN, int BK, int WM, int WN, bool TRANSB>
struct GemmTile {
  static constexpr int NT = WM * WN * 64;
  static constexpr int KC = BK / 8;                     // 16-byte chunks along k
  static constexpr int LDA_S = BK + 8;
  static constexpr int A_BYTES = BM * LDA_S * 2;
  static constexpr int LDB_S = TRANSB ? BK + 8 : BN + 32;
  static constexpr int B_BYTES = (TRANSB ? BN : BK) * LDB_S * 2;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int SMEM = 2 * STAGE;
  static constexpr int NA = BM * KC / NT;               // chunks per thread per stage
  static constexpr int NB = BN * KC / NT;
  static constexpr int TM = BM / WM / 32;               // MFMA tiles per wavefront
  static constexpr int TN = BN / WN / 32;
  static_assert(BM * KC % NT == 0 && BN * KC % NT == 0, "tile must split evenly over threads");
  static_assert(NT % KC == 0 && NT % (BN / 8) == 0, "a thread's chunks must share their column");
  static_assert(BK % 16 == 0 && BM % (WM * 32) == 0 && BN % (WN * 32) == 0, "MFMA tiling");
};

// K split across workgroups (part_steps > 0): the grid's y index is the part; part p takes the K
// steps p * part_steps .. of the problem and stores its fp32 partial tile (epi = EPI_PART32) into
// slice p of the scratch that C_ then points at (slices part_stride floats apart, row stride ldc);
// gemm_splitk_reduce_kernel adds the slices in a fixed order and applies the real epilogue.
// ACC: the form for an fp32 C that is added to (where there is one; the others can do it too).
template <typename Tag, int BM, int BN, int BK, int WM, int WN, bool TRANSB, int KS, bool AL, bool ACC>
__global__ __launch_bounds__(WM* WN * 64 * KS) void gemm_tile_kernel(
    int M, int N, int K_, const uint16_t* __restrict__ A_, int64_t lda,
    const uint16_t* __restrict__ B_, int64_t ldb, uint16_t* __restrict__ C_, int64_t ldc, int nbm,
    int nbn, int nxcd, int epi, const uint16_t* __restrict__ bias, int part_steps, int64_t part_stride) {
  typedef GemmTile<Tag, BM, BN, BK, WM, WN, TRANSB> Cfg;
  typedef typename Elem<Tag>::vec8 V8;
  typedef typename std::conditional<AL, u32x4_mem, u32x4_mem2>::type gmem16;   // a global 16-byte access
  extern __shared__ __align__(16) char smem_all[];
  const uint16_t* A = A_;
  const uint16_t* B = B_;
  uint16_t* C = C_;
  int K = K_;
  if (part_steps > 0) {
    const int part = blockIdx.y;
    const int k_begin = part * part_steps * BK;            // < K_: the host launches no empty part
    A += k_begin;
    B += TRANSB ? (int64_t)k_begin : (int64_t)k_begin * ldb;
    K = K_ - k_begin < part_steps * BK ? K_ - k_begin : part_steps * BK;
    C = reinterpret_cast<uint16_t*>(reinterpret_cast<float*>(C_) + (int64_t)part * part_stride);
  }

  // KS > 1: the workgroup holds KS groups of WM x WN wavefronts; group kg runs the whole pipeline
  // below on its own LDS stages over its own share of the K steps, and the groups' accumulators
  // are added through LDS at the end (see there). tid, wave: inside the group.
  const int kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / Cfg::NT);
  const int tid = KS == 1 ? (int)threadIdx.x : (int)threadIdx.x % Cfg::NT;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  char* const smem = smem_all + kg * Cfg::SMEM;
  int tile_m, tile_n;
  tile_of_block<8>(blockIdx.x, nbm, nbn, nxcd, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  // ---- per-thread staging assignments (fixed for the whole K loop)
  // Chunk c = tid + i*NT of a [rows][KC] tile is (row c / KC, k chunk c % KC). NT is a multiple of
  // KC, so the k chunk is the same for every i and row_i = row_0 + i * (NT / KC): LDS offsets
  // differ by compile-time constants and only the clamped global row pointers are per-i values.
  constexpr int RSTEP = Cfg::NT / Cfg::KC;              // tile rows between a thread's chunks
  const int st_row = tid / Cfg::KC, st_k = (tid % Cfg::KC) * 8;
  const uint16_t* a_src[Cfg::NA];
#pragma unroll
  for (int i = 0; i < Cfg::NA; ++i) {
    int grow = m0 + st_row + i * RSTEP;
    grow = grow < M ? grow : M - 1;
    a_src[i] = A + (int64_t)grow * lda + st_k;
  }
  const int a_dst = (st_row * Cfg::LDA_S + st_k) * 2;
  constexpr int A_DST_STEP = RSTEP * Cfg::LDA_S * 2;

  const uint16_t* b_src[TRANSB ? Cfg::NB : 1];
  int b_dst, b_k, b_drop = 0;
  const bool n_edge = !AL && !TRANSB && n0 + BN > N;     // some chunks of this tile run over the end of their row
  constexpr int NC = BN / 8;                            // 16-byte chunks along n (row-major B)
  constexpr int KSTEP = Cfg::NT / NC;                   // k rows between a thread's chunks
  constexpr int B_DST_STEP = (TRANSB ? RSTEP : KSTEP) * Cfg::LDB_S * 2;
  if (TRANSB) {
#pragma unroll
    for (int i = 0; i < Cfg::NB; ++i) {
      int grow = n0 + st_row + i * RSTEP;
      grow = grow < N ? grow : N - 1;
      b_src[i] = B + (int64_t)grow * ldb + st_k;
    }
    b_dst = Cfg::A_BYTES + (st_row * Cfg::LDB_S + st_k) * 2;
    b_k = st_k;
  } else {
    const int krow = tid / NC, nc = tid % NC;
    const int gcol = n0 + nc * 8;
    // a chunk outside the matrix reads column 0 instead; N % 8 == 0 (AL): no chunk is partly outside
    const int over = AL || gcol >= N ? 0 : (gcol + 8 > N ? gcol + 8 - N : 0);
    b_src[0] = B + (int64_t)krow * ldb + (gcol < N ? gcol - over : 0);
    b_drop = over;
    b_dst = Cfg::A_BYTES + (krow * Cfg::LDB_S + nc * 8) * 2;
    b_k = krow;
  }

  u32x4 ga[Cfg::NA], gb[Cfg::NB];
  const u32x4 zero4 = {0u, 0u, 0u, 0u};

  // Loads never branch per element: a chunk outside the matrix re-reads a valid address (row
  // clamp above, column 0 here). Only one K step can run past K; it takes the second form, in which
  // a chunk past K re-reads k = 0 (AL) or the 8 elements before K (!AL), to be zeroed or shifted on
  // the way to LDS.
  auto load_global_full = [&](int k0) {
#pragma unroll
    for (int i = 0; i < Cfg::NA; ++i) ga[i] = *reinterpret_cast<const gmem16*>(a_src[i] + k0);
#pragma unroll
    for (int i = 0; i < Cfg::NB; ++i) {
      if (TRANSB) gb[i] = *reinterpret_cast<const gmem16*>(b_src[i] + k0);
      else gb[i] = *reinterpret_cast<const gmem16*>(b_src[0] + (int64_t)(k0 + i * KSTEP) * ldb);
    }
  };
  auto load_global_tail = [&](int k0) {
    // k of this thread's chunk, relative to st_k: moved back inside the row
    const int ka = AL ? (k0 + st_k < K ? k0 : -st_k) : (k0 + st_k + 8 <= K ? k0 : K - 8 - st_k);
#pragma unroll
    for (int i = 0; i < Cfg::NA; ++i) ga[i] = *reinterpret_cast<const gmem16*>(a_src[i] + ka);
#pragma unroll
    for (int i = 0; i < Cfg::NB; ++i) {
      if (TRANSB) {
        gb[i] = *reinterpret_cast<const gmem16*>(b_src[i] + ka);
      } else {
        const int kr = k0 + i * KSTEP;                  // + b_k = the k row of this chunk
        gb[i] = *reinterpret_cast<const gmem16*>(b_src[0] + (int64_t)(kr + b_k < K ? kr : -b_k) * ldb);
      }
    }
  };
  // zeroes or shifts what a partial K step's chunks hold past K
  auto zero_k_tail = [&](int k0) {
    const int over = k0 + st_k + 8 - K;                  // elements of a k chunk that lie past K
#pragma unroll
    for (int i = 0; i < Cfg::NA; ++i) ga[i] = AL ? (over > 0 ? zero4 : ga[i]) : drop_elements(ga[i], over > 0 ? over : 0);
#pragma unroll
    for (int i = 0; i < Cfg::NB; ++i) {
      if (TRANSB) gb[i] = AL ? (over > 0 ? zero4 : gb[i]) : drop_elements(gb[i], over > 0 ? over : 0);
      else if (k0 + i * KSTEP + b_k >= K) gb[i] = zero4;
    }
  };
  auto store_lds = [&](int stage) {
    if (n_edge) {
#pragma unroll
      for (int i = 0; i < Cfg::NB; ++i) gb[i] = drop_elements(gb[i], b_drop);
    }
    char* base = smem + stage * Cfg::STAGE;
#pragma unroll
    for (int i = 0; i < Cfg::NA; ++i) *reinterpret_cast<u32x4_mem*>(base + a_dst + i * A_DST_STEP) = ga[i];
#pragma unroll
    for (int i = 0; i < Cfg::NB; ++i) *reinterpret_cast<u32x4_mem*>(base + b_dst + i * B_DST_STEP) = gb[i];
  };

  // ---- fragment addresses inside a stage
  // A fragment: row = wavefront row offset + 32*tm + lane%32, 8 consecutive k starting at
  // 8*(lane/32) inside each 16-wide k slice.
  const int a_frag = ((wm * (BM / WM) + (lane & 31)) * Cfg::LDA_S + 8 * (lane >> 5)) * 2;
  int b_frag;
  if (TRANSB) {
    b_frag = Cfg::A_BYTES + ((wn * (BN / WN) + (lane & 31)) * Cfg::LDB_S + 8 * (lane >> 5)) * 2;
  } else {
    // Transposing read: 16-lane group g = lane/16 serves columns 16*(g%2).. of the 32-wide tile
    // and k slots 8*(g/2)..; inside the group, lane s addresses k row s/4, columns 4*(s%4)..
    const int g = lane >> 4, s = lane & 15;
    const int krow = 8 * (g >> 1) + (s >> 2);
    const int col = wn * (BN / WN) + 16 * (g & 1) + 4 * (s & 3);
    b_frag = Cfg::A_BYTES + (krow * Cfg::LDB_S + col) * 2;
  }

  f32x16 acc[Cfg::TM][Cfg::TN];
#pragma unroll
  for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Fragments of k slice kk of a stage: TM A operands and TN B operands.
  auto load_frags = [&](const char* st, int kk, V8 (&af)[Cfg::TM], V8 (&bf)[Cfg::TN]) {
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
      af[i] = lds_read8<V8>(st, a_frag + (i * 32 * Cfg::LDA_S + kk * 16) * 2);
#pragma unroll
    for (int j = 0; j < Cfg::TN; ++j) {
      if (TRANSB) {
        bf[j] = lds_read8<V8>(st, b_frag + (j * 32 * Cfg::LDB_S + kk * 16) * 2);
      } else {
        const int off = b_frag + (kk * 16 * Cfg::LDB_S + j * 32) * 2;
        s16x4 lo = lds_read_tr4(st, off);
        s16x4 hi = lds_read_tr4(st, off + 4 * Cfg::LDB_S * 2);
        bf[j] = join_tr<V8>(lo, hi);
      }
    }
  };

  const int KT = (K + BK - 1) / BK;
  const bool ragged_k = (K % BK) != 0;                  // only the last step can be partial
  constexpr int NKK = BK / 16;
  static_assert(NKK == 4, "the schedule below is written for four k slices per stage");
  // This group's K steps: kg, kg + KS, kg + 2 KS, ... (all of them when KS == 1), so that at any
  // time the groups of a workgroup read neighbouring pieces of the same operand rows (with the
  // operands stored k-contiguous: KS x 128 contiguous bytes of every row instead of KS pieces far
  // apart); every group runs the loop KTG times so that all wavefronts meet at the same barriers,
  // idle once its steps are done.
  const int KTG = (KT + KS - 1) / KS;
  const int kt_begin = kg;
  const int kt_end = KT;
  // A partial K step is taken first, by the group it belongs to, so that the loop below never asks
  // (the question alone cost 512 x 4096 x 4096 2 %): such a group's steps are KT-1, kg, kg + KS, ...
  const bool tail_first = ragged_k && (KT - 1) % KS == kg;
  const int k_shift = tail_first ? KS * BK : 0;

  // Software pipeline. Stage s holds the group's i-th tile (s = i & 1). During step kt:
  //   slice 0: read fragments of slice 1 | MFMAs of slice 0
  //   slice 1: read fragments of slice 2 | MFMAs of slice 1 | write tile kt+1 (already in
  //            registers since the previous step) to the other stage | issue the global loads
  //            of tile kt+2 into the registers just freed
  //   slice 2: read fragments of slice 3 | MFMAs of slice 2 | barrier
  //   slice 3: read fragments of slice 0 of tile kt+1 | MFMAs of slice 3
  // The barrier sits where every wavefront has issued its last read of stage s and its writes
  // of tile kt+1, so after it stage s may be overwritten (in step kt+1) and tile kt+1 may be
  // read; its latency and that of the first fragment reads hide behind the MFMAs of slice 3.
  // An fp32 C that is added to: with several K groups a thread has few pieces of it, which are on their way through the whole K loop
  // (us, with loads behind the last step before: 440 x 928 x 440 6.1 / 5.7, 1024 x 1024 x 384 6.0 / 5.6, 328 x 2032 x 256 5.8 / 5.4). Without groups
  // the next tiles' pieces would wait for them (264 x 4000 x 256 6.3 / 6.7). A form of its own, because code that a small launch does not
  // reach costs it time too (512^3, 16-bit C, 4.87 / 4.95).
  constexpr int NTHR = Cfg::NT * KS, CPT4 = BN / 4, NC4 = BM * BN <= 128 * 128 ? (BM * CPT4 + NTHR - 1) / NTHR : 1;
  constexpr bool EARLY = ACC;
  static_assert(!ACC || (KS > 1 && NC4 <= 4), "few pieces of C per thread");
  f32x4 c32[EARLY ? NC4 : 1];
  auto load_c32 = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < (EARLY ? NC4 : 0); ++i) {
      const int it = (int)threadIdx.x + i * NTHR, r = it / CPT4, col = n0 + it % CPT4 * 4;
      c32[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (r >= BM || m0 + r >= M) continue;
      const float* src = reinterpret_cast<const float*>(C) + (int64_t)(m0 + r) * ldc + col;
      if (col + 4 <= N) c32[i] = *reinterpret_cast<const f32x4_mem4*>(src);
      else
        for (int e = 0; e < 4; ++e)
          if (col + e < N) c32[i][e] = src[e];
    }
  };

  const bool any = kt_begin < kt_end;
  if (any) {
    if (tail_first) load_global_tail((KT - 1) * BK); else load_global_full(kt_begin * BK);
    if (tail_first) zero_k_tail((KT - 1) * BK);
    store_lds(0);
    if (kt_begin + KS < kt_end) load_global_full((kt_begin + KS) * BK - k_shift);
  }
  if (EARLY) load_c32();
  __syncthreads();

  V8 af[2][Cfg::TM], bf[2][Cfg::TN];
  if (any) load_frags(smem, 0, af[0], bf[0]);

  auto mfma_slice = [&](int which) {
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::TN; ++j)
        acc[i][j] = mfma32(af[which][i], bf[which][j], acc[i][j]);
  };

  for (int it = 0; it < KTG; ++it) {
    const int kt = kt_begin + it * KS;
    const bool active = KS == 1 || kt < kt_end;
    const int cur = it & 1;
    const char* st = smem + cur * Cfg::STAGE;
    const char* nx = smem + (cur ^ 1) * Cfg::STAGE;
    const bool have_next = kt + KS < kt_end;

    if (active) {
      load_frags(st, 1, af[1], bf[1]);
      __builtin_amdgcn_sched_barrier(0);
      mfma_slice(0);
      __builtin_amdgcn_sched_barrier(0);

      load_frags(st, 2, af[0], bf[0]);
      __builtin_amdgcn_sched_barrier(0);
      mfma_slice(1);
      __builtin_amdgcn_sched_barrier(0);
      if (have_next) {
        store_lds(cur ^ 1);
        if (kt + 2 * KS < kt_end) load_global_full((kt + 2 * KS) * BK - k_shift);
      }
      __builtin_amdgcn_sched_barrier(0);

      load_frags(st, 3, af[1], bf[1]);
      __builtin_amdgcn_sched_barrier(0);
      mfma_slice(0);                                    // slice 2 lives in fragment set 0
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();

    if (active) {
      if (have_next) load_frags(nx, 0, af[0], bf[0]);
      __builtin_amdgcn_sched_barrier(0);
      mfma_slice(1);                                    // slice 3 lives in fragment set 1
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- epilogue, row-contiguous through LDS (see RowStore)
  if constexpr (BM * BN <= 128 * 128) {
    // The whole tile at once: every group parks its accumulators in its own image of the tile
    // ([row][BN + 8] floats: the two row groups of a 32x32 accumulator, 4 rows apart, in different
    // banks), and all threads of the workgroup then add the KS images in the order 0, 1, ... and store.
    // (The sum by group 0 alone, its partial values read one float at a time, and the store from
    // its registers took 0.9 us longer on 512 x 4096 x 4096.)
    constexpr int S = BN + 8;
    static_assert(KS * BM * S * 4 <= KS * Cfg::SMEM, "the images fit the stages");
    float* const red = reinterpret_cast<float*>(smem_all);
    if (KS > 1) __syncthreads();                          // (KS == 1: no stage is read after the loop's last barrier)
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          *reinterpret_cast<f32_mem*>(red + (kg * BM + wm * (BM / WM) + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * S +
                                      wn * (BN / WN) + j * 32 + (lane & 31)) = acc[i][j][r];
    __syncthreads();
    if (epi & (EPI_PART32 | EPI_ACC32)) {
      auto piece = [&](int it, const f32x4& old, bool load) __attribute__((always_inline)) {
        const int r = it / CPT4, c = it % CPT4 * 4;
        f32x4 v = *reinterpret_cast<const f32x4_mem*>(red + r * S + c);
#pragma unroll
        for (int g2 = 1; g2 < KS; ++g2) add4(v, *reinterpret_cast<const f32x4_mem*>(red + (g2 * BM + r) * S + c));
        if (!load) add4(v, old);
        if (m0 + r < M) store_row4(v, reinterpret_cast<float*>(C) + (int64_t)(m0 + r) * ldc + n0 + c, N - n0 - c, load && (epi & EPI_ACC32));
      };
      if constexpr (EARLY) {
#pragma unroll
        for (int i = 0; i < NC4; ++i) {
          const int it = (int)threadIdx.x + i * NTHR;
          if (BM * CPT4 % NTHR == 0 || it < BM * CPT4) piece(it, c32[i], false);
        }
      } else {
        for (int it = threadIdx.x; it < BM * CPT4; it += NTHR) piece(it, c32[0], true);
      }
    } else {
      constexpr int CPT = BN / 8;
      auto rows = [&](auto STREAM) __attribute__((always_inline)) {
        for (int it = threadIdx.x; it < BM * CPT; it += NTHR) {
          const int r = it / CPT, c = it % CPT * 8;
          const float* src = red + r * S + c;
          f32x4 lo = *reinterpret_cast<const f32x4_mem*>(src), hi = *reinterpret_cast<const f32x4_mem*>(src + 4);
#pragma unroll
          for (int g2 = 1; g2 < KS; ++g2) {
            add4(lo, *reinterpret_cast<const f32x4_mem*>(src + g2 * BM * S));
            add4(hi, *reinterpret_cast<const f32x4_mem*>(src + g2 * BM * S + 4));
          }
          if (m0 + r < M && n0 + c < N)
            store_row8<Tag, STREAM.value>(lo, hi, C + (int64_t)(m0 + r) * ldc + n0 + c, N - n0 - c, epi, bias ? bias + n0 + c : nullptr);
        }
      };
      if (epi & EPI_STREAM) rows(std::true_type{});
      else rows(std::false_type{});
    }
  } else {
    static_assert(KS == 1, "the large tiles have no K split inside the workgroup");
    constexpr int TJ = Cfg::TN < 2 ? Cfg::TN : 2;         // up to 64 columns at a time
    typedef RowStore<Tag, 32, TJ * 32, 8> Rows;
    static_assert(WM * WN * Rows::BYTES <= Cfg::SMEM, "the parking areas fit the LDS");
    float* park = reinterpret_cast<float*>(smem + wave * Rows::BYTES);
    // With 16 tiles per wavefront, code for both forms of the store is more than the compiler unrolls, and an accumulator with a
    // run-time index keeps all 256 in memory (4096 x 4096 x 4104 182 -> 1837 us): plain stores there.
    constexpr bool STREAMS = Cfg::TM * Cfg::TN < 16;
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
      for (int j0 = 0; j0 < Cfg::TN; j0 += TJ)
        Rows::template run<STREAMS>([&](float* lds) {
#pragma unroll
          for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              *reinterpret_cast<f32_mem*>(lds + (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * Rows::STRIDE + j * 32 + (lane & 31)) = acc[i][j0 + j][r];
        }, park, lane, m0 + wm * (BM / WM) + i * 32, n0 + wn * (BN / WN) + j0 * 32, M, N, C, ldc, epi, bias);
  }
}

// Second pass of a K split across workgroups: C = epilogue(sum over parts, in the order 0, 1, ...,
// of the fp32 partial products). One thread per four consecutive columns of a row;
// every part's values are requested before the first is added (up to P of them; a serial loop over
// the parts waits for one memory round trip after the other).
template <typename Tag, int P>
__global__ __launch_bounds__(256) void gemm_splitk_reduce_kernel(
    int M, int N, int parts, const float* __restrict__ ws, int64_t part_stride,
    uint16_t* __restrict__ C, int64_t ldc, int epi, const uint16_t* __restrict__ bias) {
  const int nq = (N + 3) / 4;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)M * nq) return;
  const int row = (int)(t / nq), col0 = (int)(t % nq) * 4;
  const float* src = ws + (int64_t)row * N + col0;
  const bool whole = col0 + 4 <= N;
  f32x4 v[P];
  if (whole) {
#pragma unroll
    for (int p = 0; p < P; ++p)
      v[p] = *reinterpret_cast<const f32x4_mem4*>(src + (int64_t)(p < parts ? p : 0) * part_stride);
  } else {
#pragma unroll
    for (int p = 0; p < P; ++p)
      for (int e = 0; e < 4; ++e) v[p][e] = col0 + e < N ? src[(int64_t)(p < parts ? p : 0) * part_stride + e] : 0.f;
  }
  float acc[4] = {v[0][0], v[0][1], v[0][2], v[0][3]};
#pragma unroll
  for (int p = 1; p < P; ++p)
    if (p < parts) { acc[0] += v[p][0]; acc[1] += v[p][1]; acc[2] += v[p][2]; acc[3] += v[p][3]; }
  if (epi & EPI_ACC32) {
    store_row4(f32x4{acc[0], acc[1], acc[2], acc[3]}, reinterpret_cast<float*>(C) + (int64_t)row * ldc + col0, N - col0, true);
    return;
  }
  const int act = (epi >> EPI_ACT_SHIFT) & EPI_ACT_MASK;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (bias && col0 + e < N) acc[e] += Elem<Tag>::to_f32(bias[col0 + e]);
    acc[e] = epi_act(acc[e], act);
  }
  uint16_t* cp = C + (int64_t)row * ldc + col0;
  if (whole) {
    *reinterpret_cast<u32x2_mem2*>(cp) = u32x2{Elem<Tag>::pack2(acc[0], acc[1]), Elem<Tag>::pack2(acc[2], acc[3])};
  } else {
    for (int e = 0; e < 4; ++e)
      if (col0 + e < N) cp[e] = Elem<Tag>::from_f32(acc[e]);
  }
}

template <typename Tag>
static int launch_splitk_reduce(const GemmArgs& g, int parts, int64_t part_stride, hipStream_t s) {
  const int64_t nthreads = g.M * ((g.N + 3) / 4);
  auto kern = parts <= 2 ? gemm_splitk_reduce_kernel<Tag, 2> : parts <= 4 ? gemm_splitk_reduce_kernel<Tag, 4>
                                                                          : gemm_splitk_reduce_kernel<Tag, 8>;
  hipLaunchKernelGGL(kern, dim3((unsigned)((nthreads + 255) / 256)), dim3(256), 0, s, (int)g.M, (int)g.N,
                     parts, g.scratch, part_stride, g.C, g.ldc, g.epi(), g.bias);
  return hipGetLastError() == hipSuccess ? MLT_OK : MLT_ERR_LAUNCH;
}

template <typename Tag, int BM, int BN, int BK, int WM, int WN, bool TRANSB, int KS, bool AL, bool ACC = false>
static int launch_tile(const GemmArgs& g, hipStream_t s) {
  typedef GemmTile<Tag, BM, BN, BK, WM, WN, TRANSB> Cfg;
  static_assert(Cfg::NT * KS <= 1024 && KS * Cfg::SMEM <= 160 * 1024, "one workgroup, one CU's LDS");
  auto kern = gemm_tile_kernel<Tag, BM, BN, BK, WM, WN, TRANSB, KS, AL, ACC>;
  static thread_local int configured_dev = -1;          // opt in to > 64 KB LDS once per device
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MLT_ERR_DEVICE;
  if (configured_dev != dev) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                            KS * Cfg::SMEM) != hipSuccess) {
      (void)hipGetLastError();
      return MLT_ERR_LAUNCH;
    }
    configured_dev = dev;
  }
  const int nbm = (int)((g.M + BM - 1) / BM), nbn = (int)((g.N + BN - 1) / BN);
  if (g.parts <= 1) {
    hipLaunchKernelGGL(kern, dim3(nbm * nbn), dim3(Cfg::NT * KS), KS * Cfg::SMEM, s, (int)g.M, (int)g.N,
                       (int)g.K, g.A, g.lda, g.B, g.ldb, g.C, g.ldc, nbm, nbn, device_xcds(), g.epi(), g.bias, 0,
                       (int64_t)0);
    return hipGetLastError() == hipSuccess ? MLT_OK : MLT_ERR_LAUNCH;
  }
  // K split across workgroups: fp32 partial tiles into the scratch, then the fixed-order sum
  const int KT = (int)((g.K + BK - 1) / BK);
  const int part_steps = (KT + g.parts - 1) / g.parts;
  const int parts = (KT + part_steps - 1) / part_steps;    // no empty part
  const int64_t part_stride = g.M * g.N;
  hipLaunchKernelGGL(kern, dim3(nbm * nbn, parts), dim3(Cfg::NT * KS), KS * Cfg::SMEM, s, (int)g.M,
                     (int)g.N, (int)g.K, g.A, g.lda, g.B, g.ldb, reinterpret_cast<uint16_t*>(g.scratch),
                     g.N, nbm, nbn, device_xcds(), (int)EPI_PART32, (const uint16_t*)nullptr, part_steps, part_stride);
  if (hipGetLastError() != hipSuccess) return MLT_ERR_LAUNCH;
  return launch_splitk_reduce<Tag>(g, parts, part_stride, s);
}

// KS: K-split groups per workgroup when B is stored N x K, KS_NN when it is stored K x N (whose
// padded stage is larger, so fewer groups fit the LDS).
template <typename Tag, bool AL, int BM, int BN, int BK, int WM, int WN, int KS = 1, int KS_NN = KS>
static int launch_tile_tb(const GemmArgs& g, hipStream_t s) {
  if constexpr (AL && KS > 1) {
    if (g.acc32 && g.parts <= 1)
      return g.transB ? launch_tile<Tag, BM, BN, BK, WM, WN, true, KS, AL, true>(g, s)
                      : launch_tile<Tag, BM, BN, BK, WM, WN, false, KS_NN, AL, true>(g, s);
  }
  return g.transB ? launch_tile<Tag, BM, BN, BK, WM, WN, true, KS, AL>(g, s)
                  : launch_tile<Tag, BM, BN, BK, WM, WN, false, KS_NN, AL>(g, s);
}

// The small-tile variants, which both kinds of operands share; -1: not one of them.
template <typename Tag, bool AL>
static int launch_small_tile(const GemmArgs& g, int variant, hipStream_t s) {
  switch (variant) {
    case GEMM_128_W8: return launch_tile_tb<Tag, AL, 128, 128, 64, 2, 4>(g, s);
    case GEMM_64X128_W8: return launch_tile_tb<Tag, AL, 64, 128, 64, 2, 4>(g, s);
    case GEMM_64_W4: return launch_tile_tb<Tag, AL, 64, 64, 64, 2, 2>(g, s);
    case GEMM_128_K2: return launch_tile_tb<Tag, AL, 128, 128, 64, 2, 4, 2>(g, s);
    case GEMM_64X128_K2: return launch_tile_tb<Tag, AL, 64, 128, 64, 2, 4, 2>(g, s);
    case GEMM_64_K4: return launch_tile_tb<Tag, AL, 64, 64, 64, 2, 2, 4, 3>(g, s);
    case GEMM_256_W8: return launch_tile_tb<Tag, AL, 256, 256, 64, 2, 4>(g, s);
  }
  return -1;
}

}  // namespace mlt
