// GEMM C = A*B for gfx950: 16-bit inputs, fp32 accumulation on MFMA, 16-bit output.
//
// The paper (arXiv 2503.14985, Section 2) splits the GEMM in three levels: a workgroup tile of C
// (Listing 1), a square partition of that tile over the warps (Section 2.1: warpsPerCTA and
// sizePerWarp), and the split of each warp's dot into hardware-sized dots (Section 2.3). The
// kernels here have the same three levels, fixed by template parameters and re-derived for CDNA4:
//   workgroup tile BM x BN, K step BK            (paper: 256 x 256, K step 32)
//   WM x WN wavefronts, each owning (BM/WM) x (BN/WN)   (paper: 8 x 4 warps of 32 x 64)
//   MFMA 32x32x16 tiles inside the wavefront tile       (paper: 8x16x16 DPAS)
// Unlike the paper's target there is no 2-D block load from memory into registers, so operand
// tiles are staged through LDS: each byte is fetched from global memory once per workgroup and
// read by the wavefronts that share it (the rows/columns of the warp grid that Section 2.2 notes
// work on the same sub-block of A or B).
#include <atomic>
#include <mutex>

#include "gemm_tile.h"

namespace mlt {

// ------------------------------------------------------------------------------------------
// General kernel: what no 16-byte access fits (K < 8, N < 8 with row-major B), K = 0 with a fused
// epilogue, and any problem by override. 64 x 64 x 32 tile, 4 wavefronts of 32 x 32, element-wise
// guarded loads with zero fill, B always staged as [n][k].
// ------------------------------------------------------------------------------------------
template <typename Tag>
__global__ __launch_bounds__(256) void gemm_general_kernel(
    int M, int N, int K, const uint16_t* __restrict__ A, int64_t lda,
    const uint16_t* __restrict__ B, int64_t ldb, int transB, uint16_t* __restrict__ C,
    int64_t ldc, int epi, const uint16_t* __restrict__ bias) {
  typedef typename Elem<Tag>::vec8 V8;
  constexpr int BM = 64, BN = 64, BK = 32, LDS_S = BK + 8;
  __shared__ __align__(16) uint16_t As[BM * LDS_S];
  __shared__ __align__(16) uint16_t Bs[BN * LDS_S];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;

  for (int k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
    for (int i = 0; i < BM * BK / 256; ++i) {
      const int e = tid + i * 256;
      const int row = e / BK, k = e % BK;               // consecutive lanes: consecutive k
      const bool ok = (m0 + row < M) && (k0 + k < K);
      As[row * LDS_S + k] = ok ? A[(int64_t)(m0 + row) * lda + k0 + k] : (uint16_t)0;
    }
#pragma unroll
    for (int i = 0; i < BN * BK / 256; ++i) {
      const int e = tid + i * 256;
      int n, k;
      if (transB) { n = e / BK; k = e % BK; } else { k = e / BN; n = e % BN; }
      const bool ok = (n0 + n < N) && (k0 + k < K);
      uint16_t v = 0;
      if (ok) v = transB ? B[(int64_t)(n0 + n) * ldb + k0 + k] : B[(int64_t)(k0 + k) * ldb + n0 + n];
      Bs[n * LDS_S + k] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int off = kk * 16 + 8 * (lane >> 5);
      V8 a = lds_read8<V8>(reinterpret_cast<const char*>(As), ((wm * 32 + (lane & 31)) * LDS_S + off) * 2);
      V8 b = lds_read8<V8>(reinterpret_cast<const char*>(Bs), ((wn * 32 + (lane & 31)) * LDS_S + off) * 2);
      acc = mfma32(a, b, acc);
    }
    __syncthreads();
  }
  const int col = n0 + wn * 32 + (lane & 31);
  gemm_epilogue<Tag>([&](auto&& out) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = m0 + wm * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      if (row < M && col < N) out((int64_t)row * ldc + col, col, acc[r]);
    }
  }, C, epi, bias);
}

// K == 0: the empty sum (only launched when C is overwritten; C += 0 is a no-op).
__global__ void gemm_zero_kernel(int M, int N, uint16_t* __restrict__ C, int64_t ldc) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < (int64_t)M * N) C[(e / N) * ldc + (e % N)] = 0;
}

// ------------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------------
template <typename Tag>
static int launch_general(const GemmArgs& g, hipStream_t s) {
  dim3 grid((unsigned)((g.N + 63) / 64), (unsigned)((g.M + 63) / 64));
  hipLaunchKernelGGL(gemm_general_kernel<Tag>, grid, dim3(256), 0, s, (int)g.M, (int)g.N, (int)g.K,
                     g.A, g.lda, g.B, g.ldb, g.transB, g.C, g.ldc, g.epi(), g.bias);
  return hipGetLastError() == hipSuccess ? MLT_OK : MLT_ERR_LAUNCH;
}

static bool fast_path_ok(const GemmArgs& g) {
  auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (!al16(g.A) || !al16(g.B)) return false;
  if (g.K % 8 || g.lda % 8 || g.ldb % 8) return false;
  if (!g.transB && g.N % 8) return false;
  return true;
}

static const char* any_name(int variant, int transB) {
  switch (variant) {
    case GEMM_128_W8: return transB ? "gemm_general_nt_128x128x64_w2x4" : "gemm_general_nn_128x128x64_w2x4";
    case GEMM_64X128_W8: return transB ? "gemm_general_nt_64x128x64_w2x4" : "gemm_general_nn_64x128x64_w2x4";
    case GEMM_64_W4: return transB ? "gemm_general_nt_64x64x64_w2x2" : "gemm_general_nn_64x64x64_w2x2";
    case GEMM_128_K2: return transB ? "gemm_general_nt_128x128x64_w2x4_k2" : "gemm_general_nn_128x128x64_w2x4_k2";
    case GEMM_64X128_K2: return transB ? "gemm_general_nt_64x128x64_w2x4_k2" : "gemm_general_nn_64x128x64_w2x4_k2";
    case GEMM_64_K4: return transB ? "gemm_general_nt_64x64x64_w2x2_k4" : "gemm_general_nn_64x64x64_w2x2_k4";
  }
  return transB ? "gemm_general_nt_256x256x64_w2x4" : "gemm_general_nn_256x256x64_w2x4";
}

// The streaming kernel of gemm_skinny.hip: its parts and its block
static void plan_skinny(const GemmArgs& g, int64_t ncu, GemmPlan& p) {
  // K over 1, 2, 4 or 8 workgroups: B's arrival + what a CU fetches of A (at 100 GB/s) + the price of the partial
  // results (a fit to the times of 175 problems: the choice is 1.2 % behind the best one on average, 26 % at worst)
  auto time = [&](int64_t parts) {
    const int64_t rows = g.M <= 4 ? 4 : (g.M + 15) / 16 * 16;
    return g.N * g.K * 2 / 6600 + rows * g.K * 2 / (100 * parts) + (parts > 1 ? 800 + 7 * parts * g.M * g.N / 1000 : 0);
  };
  p.parts = g.forced_parts > 0 ? g.forced_parts : 1;
  if (g.forced == GEMM_AUTO && g.forced_parts == 0)
    for (int n = 2; n <= 8; n *= 2)
      if (n * g.M * g.N * 4 <= kStaticScratchBytes && time(n) < time(p.parts)) p.parts = n;
  p.scratch_bytes = p.parts > 1 ? (int64_t)p.parts * g.M * g.N * 4 : 0;
  p.variant = GEMM_SKINNY;
  p.name = "gemm_nt_skinny_stream";
  p.bm = (int)((g.M + 15) / 16) * 16; p.bn = gemm_skinny_cols(g.N, p.parts, ncu); p.bk = 128;
  p.wm = 1; p.wn = 1;
  p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
}

// Up to 64 rows against B stored N x K: the streaming kernel, or the tile kernels? All times with B coming from memory, as a
// decoder's weights do (every matrix is read once per token, and a model is far larger than the 256 MiB last-level cache). On the
// same B again and again the tile kernels gain up to a third, the streaming kernel, which does not keep B in the caches, nothing: where the
// two are within a few percent it is the tiles (us, streaming / tiles, B from memory and, in brackets, repeated: 33 x 28672 x 4096 44 / 51 (44 / 38), 64 x
// 28672 x 4096 50 / 54 (50 / 39), 48 x 4096 x 4096 11.6 / 12.1 (10.5 / 11.1), 64 x 8192 x 14336 49 / 46 (48 / 40)). Over 962 problems of up to 64 rows, 1024
// to 100000 columns and K from 8 to 28672 the choice is 0.4 % behind the better kernel on average (streaming always: 10 %, 3.2 times at worst).
static bool stream_wins(const GemmArgs& g, int64_t ncu, const GemmPlan& tiles) {
  const int64_t kt = (g.K + 63) / 64;
  // Few steps of K: a wavefront of the streaming kernel has one piece or none, and what takes the time is its column blocks one behind the
  // other, each with a sum over 8 partial tiles; a workgroup of the tile kernels has one tile and few steps (us, streaming / tiles:
  // 9 x 14768 x 64 4.7 / 3.1, 19 x 60280 x 24 13.4 / 4.5, 23 x 17600 x 256 6.0 / 5.6, with GELU 28 x 18776 x 64 7.0 / 5.0; but 1 x 1784 x 320 2.9 / 5.4,
  // 8 x 18784 x 208 5.2 / 5.6; one row tile from 5 steps on: 2 x 69240 x 384 13.8 / 15.8). A fused activation costs the tile kernels more, whose
  // workgroups are fewer.
  if (g.M <= 32) return kt >= (g.M > 16 ? 8 : 5) || g.N * ((g.M + 15) / 16) <= 16 * ncu * kt * (g.fused() ? 2 : 1);
  if (kt < 8) return false;
  // Three and four row tiles: a workgroup of the tile kernels multiplies them all at once, so these win where their grid (`tiles`: the kernel and
  // parts that they would take) fills its rounds, one or two, of the chip; the streaming kernel has a workgroup on every CU in any case (us,
  // streaming / tiles; 64 x 128 tiles: 52 x 31704 x 1856, 248 of them, 30.1 / 23.7; 64 x 52736 x 576, 412, 26.8 / 17.4; 33888 x 1024, 265, 21.2 / 22.6;
  // 55 x 6904 x 6784 in four parts, 216, 26.3 / 23.8; 41 x 5592 x 3520, 176, 12.9 / 14.7; 38 x 7664 x 3392, 240, 13.8 / 15.7; 64 x 64 tiles: 51 x 1808 x 20736 in
  // eight, 232, 26.4 / 21.8; 60 x 13016 x 512, 204, 7.8 / 6.8; 42 x 12448 x 5632, 195, 28.7 / 31.7; 44 x 28384 x 1088, 444, 19.6 / 17.8; 34 x 24160 x 1024, 378,
  // 14.3 / 15.6). Rows of K that are not whole steps make the tile kernels' loads slower.
  if (g.M > 48 && g.N <= 16 * ncu && kt >= 64 && kt < 256 && tiles.parts > 1) return false;   // 64 x 4096 x 4096 13.9 / 12.8, 61 x 2976 x 16192 29.5 / 26.4
  const bool wide = tiles.variant == GEMM_64X128_K2;
  const int64_t wgs = (g.N + (wide ? 127 : 63)) / (wide ? 128 : 64) * tiles.parts, rounds = (wgs + ncu - 1) / ncu;
  const bool split = tiles.parts >= 4 && rounds == 1 && g.K % 64 == 0 && kt >= 16 * tiles.parts;
  if (wide) return !(4 * wgs >= 3 * ncu * rounds && (tiles.parts == 1 ? rounds <= 2 : split));
  if (tiles.variant != GEMM_64_K4) return true;
  if (tiles.parts > 1) return !(8 * wgs >= 5 * ncu && tiles.parts == 8 && split);
  if (rounds == 1) return !(8 * wgs >= 5 * ncu && g.K % 64 == 0 && kt < (g.fused() ? 12 : 40));
  return !(5 * wgs >= 4 * ncu * rounds && g.K % 64 == 0 && kt < 20 && !g.fused());
}

// rows of a tile of gemm_kp.hip; 0: another kernel's
static int kp_rows(int variant) {
  switch (variant) {
    case GEMM_256X128_KP: return 256;
    case GEMM_224X128_KP: return 224;
    case GEMM_192X128_KP: return 192;
    case GEMM_160X128_KP: return 160;
    case GEMM_128_KP: return 128;
  }
  return 0;
}

GemmPlan plan_gemm(const GemmArgs& g_in) {
  GemmPlan p;
  GemmArgs g = g_in;
  // K == 0: the empty sum; with a fused epilogue C = act(bias), which the general kernel's epilogue
  // computes after zero K steps
  if (g.K == 0 && !g.fused()) { p.variant = GEMM_ZERO; p.name = "gemm_zero"; return p; }
  // operands that do not allow aligned 16-byte accesses: the tile kernels in the form of gemm_any.hip;
  // rows too short for one such access: the general kernel
  p.aligned = g.K == 0 || g.forced == GEMM_GENERAL || fast_path_ok(g) || !gemm_any_ok(g);
  // the 256 x 256 kernels of the tiling hints exist for aligned operands only, and that tile is far too large for most
  // others (1439 x 333 x 113 row-major: 10.6 us, the automatic choice 7)
  if (!p.aligned && (g.forced == GEMM_256 || g.forced == GEMM_256_W8X1 || g.forced == GEMM_256_W1X8)) g.forced = GEMM_AUTO;
  if (g.K == 0 || g.forced == GEMM_GENERAL || (p.aligned && !fast_path_ok(g))) {
    p.variant = GEMM_GENERAL; p.name = "gemm_general_64x64x32";
    p.bm = 64; p.bn = 64; p.bk = 32; p.wm = 2; p.wn = 2;
    return p;
  }
  DeviceInfo di;
  const int64_t NCU = device_info(di) && di.ncu > 0 ? di.ncu : 256;
  const int64_t KT = (g.K + 63) / 64;
  const bool skinny = gemm_skinny_ok(g);
  if (skinny && (g.forced == GEMM_SKINNY || (g.forced == GEMM_AUTO && g.M <= 32 && stream_wins(g, NCU, p)))) {
    plan_skinny(g, NCU, p);
    return p;
  }
  // ---- the tile kernels: workgroup tile and K split
  // The candidate that needs the least time over the whole grid: (rounds of one workgroup per CU)
  // x (K steps of 64) x (its measured time per K step: two-group 256x256 kernel 1.17 us, older
  // 256x256 kernel 1.8 us; small tiles with the K steps split over 2 to 4 groups of wavefronts
  // inside the workgroup: 128x128 0.575 us, 64x128 0.37 us, 64x64 0.22 us; unsplit, for fewer than
  // 8 K steps: 0.60, 0.41, 0.35); ties go to the larger tile. (3072^3, 144 big tiles: 1033 TFLOP/s
  // against 739 with 576 tiles of 128x128; 2048^3, 64 big tiles: 437 against 758; 256 x 4096 x
  // 4096: 482 with 256 split tiles of 64x64, 326 unsplit, 244 with 64 tiles of 128x128.)
  // Never less than the time the operands take to arrive (A and B once at 5.2 TB/s: 64 x 8192 x
  // 28672 measured 91 us), more when too few workgroups pull or the last round leaves CUs idle
  // (the term is spelled out in the code below).
  // On top of that the K steps may be split over 2, 4 or 8 workgroups per tile (the small-tile
  // kernels), when the tiles alone leave most of the chip idle against a long K: each part writes
  // an fp32 partial tile to a scratch and a second kernel adds the parts in a fixed order
  // (deterministic; no atomics). Its price in the same units: a launch (4 us) plus writing and
  // reading parts * M * N floats at about 4 TB/s.
  // An fp32 C that is accumulated into comes and goes when all K steps are done: half of its traffic is added for gemm_kp.hip, and for the two-group 128 x 128
  // kernel where that has one workgroup per CU (with two, one works while the other waits). The split kernels have their pieces of C in flight from the start,
  // and the sum of a K split and 256 x 256 do better than that. Over 190 accumulated problems the choice is then 1.4 % behind the best
  // tile on average, 2.0 % with nothing added and with all of the traffic added to gemm_kp.hip alone (us, 680 x 3200 x 3200 27.4, there
  // 31.2 on K steps of 128; 2912 x 1344 x 3904 38.9 / 43.8; 2232 x 2752 x 968 27.9, with nothing added 36.7 on 224 x 128).
  const int64_t c32 = g.acc32 ? g.M * g.N * 4 / 5200 : 0;
  const bool pp = gemm_pp_ok(g);
  // GELU in the epilogue takes some 3 us a round on the 128-row tiles (us, without / with it: 2181 x 1792 x 576 two-group 12.0 / 15.0, split 10.9 / 13.6) and
  // more on the tall ones, whose wavefronts hold more of the result each and have nothing to hide it behind (970 x 7936 x 1088, 256 x 128 20.8 / 30.6, two-group
  // 128 x 128 in pairs 21.8 / 26.5; 2024 x 8640 x 704, two rounds of 256 x 256, 51.7 / 75.8); 64-row tiles pay in every round (651 x 3392 x 576, three rounds of
  // 64 x 64 18.8, 128 x 128 12.2). What is more than on the 128-row tiles is added. Without it 1607 x 3840 x 768 took 224 x 128, 25.0 us, 20.7 on 128 x 128;
  // over 78 such problems the choice was 3.8 % behind the best tile, now 0.6 %. (With K in parts the sum has the GELU, at less than a microsecond.)
  const bool gelu = g.act == ACT_GELU && pp && g.M > 128 && KT >= 8;
  auto cost = [&](int64_t bm, int64_t bn, int64_t t_step, int64_t fixed, int parts, int kgroups) {
    const int64_t wgs = ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * parts;
    const int64_t rounds = (wgs + NCU - 1) / NCU;
    const int64_t steps = (KT + parts - 1) / parts;
    const int64_t act = !gelu || parts > 1 ? 0 : bm == 256 ? rounds * 9000 : bm == 64 ? (rounds - 1) * 1200 : 0;
    const int64_t compute = rounds * (steps * t_step + fixed) + act;
    // operand arrival: both operands once at 5.2 TB/s, which about 0.6 workgroups per CU already
    // draw (measured 37 GB/s per streaming workgroup: 64 of them 2.4 TB/s, 128 4.2, 224 5.7);
    // beyond one workgroup per CU the last round's idle CUs count (448 workgroups take the time
    // of 512: 32 x 28672 x 8192 measured 104-108 us on 64 x 64 tiles against 82 on 224 of 64 x 128)
    const int64_t base = (g.M + g.N) * g.K * 2 / 5200;
    // (the decode shapes are priced with B coming from memory: then fewer workgroups than CUs do
    // not keep enough bytes in flight; 64 x 8192 x 8192 on 128 tiles of 64 x 64: 43 us with B
    // rotating over more than the last-level cache holds, 34-37 us with K split two or four ways)
    const int64_t need = g.M <= 64 && g.transB ? NCU : 6 * NCU / 10;
    // B stored N x K: a workgroup reads (K groups) x 128 contiguous bytes of each row at a time.
    // The two-group tiles (256-byte pieces) need a workgroup on every CU and a little more to
    // draw the full rate (64 x 28672 x 8192 on 224 tiles of 64 x 128: 107 us = 1.18 x the 5.2 TB/s
    // time); the four-group 64 x 64 tile with between one and two workgroups per CU has them all
    // resident at once, so there is no second round with idle CUs (the same problem on 448 such
    // tiles: 102 us; 32 x 28672 x 8192: 95 against 105; 48 x ...: 95 against 100)
    const int64_t need_here = g.transB && kgroups == 2 && parts == 1 ? NCU + NCU / 20 : need;
    int64_t arrive = wgs >= NCU && wgs >= need_here ? base * rounds * NCU / wgs
                     : (wgs >= need_here ? base : base * need_here / wgs);
    if (g.transB && kgroups == 4 && parts == 1 && wgs > NCU && wgs <= 2 * NCU) arrive = base + base / 20;
    return (compute > arrive ? compute : arrive) + (parts > 1 ? 4000 + 2 * parts * g.M * g.N / 1000 : 0);
  };
  // Among the candidates within 8 % of the best estimate the largest tile wins (a larger tile
  // re-reads its operands from L2 less often, which the estimate leaves out: 64 x 8192 x 28672
  // measured 90 us on 64x128 tiles in four parts, 100-110 us on 64x64 tiles in two); for one tile
  // size, the fewer parts unless more parts are estimated more than 5 % faster.
  // t: ns per K step of 64; fixed: ns per round before the first and after the last step, where a
  // fit over K gave one (2048 x 2048 x K on the split 128 x 128 kernel: 0.56 us per step + 2 us)
  struct Cand { int variant; int bm, bn; int64_t t, fixed; int kgroups; };
  // (fewer than 8 K steps, the last one partial: 1170 leaves out the start and end of the large tiles, and they were
  // taken where many small ones are faster. bf16, us, 256 x 256 / 128 x 128: 2936 x 5560 x 144 with bias and GELU 46 /
  // 31; 5117 x 1240 x 176 fp32 accumulate 26 / 19; 7029 x 1088 x 224 14.5 / 13.0)
  const bool short_ragged = g.K % 64 && KT < 8;
  const Cand big = {pp ? GEMM_256_PP16 : GEMM_256_W8, 256, 256, !p.aligned ? 2300 : pp && !short_ragged ? 1170 : 1800, 0, 1};
  // Operands of any alignment: a step's loads and their LDS writes weigh more than its MFMAs, and
  // the groups of a workgroup share them, so what the K split inside the workgroup gains is small;
  // two unsplit workgroups on a CU do as well (ns per step and tile, from 201 x 4001 x 4001, one tile
  // per CU, and 1999 x 3001 x 1501, 384 to 1504 tiles).
  const Cand any[] = {{GEMM_128_W8, 128, 128, 760, 0, 1}, {GEMM_64X128_K2, 64, 128, 600, 0, 2}, {GEMM_64_K4, 64, 64, 430, 0, 4}};
  const Cand split[] = {{GEMM_128_K2, 128, 128, 560, 2000, 2}, {GEMM_64X128_K2, 64, 128, 370, 0, 2}, {GEMM_64_K4, 64, 64, 220, 0, 4}};
  const Cand whole[] = {{GEMM_128_W8, 128, 128, 600, 0, 1}, {GEMM_64X128_W8, 64, 128, 410, 0, 1}, {GEMM_64_W4, 64, 64, 350, 0, 1}};
  struct Choice { int variant, parts, area; int64_t t; };
  Choice all[32];
  int n_all = 0;
  // no tile taller or wider than the matrix rounded up to 64 (it would multiply padding)
  auto fits = [&](int bm, int bn) {
    return !(bm > 64 && bm > (g.M + 63) / 64 * 64) && !(bn > 64 && bn > (g.N + 63) / 64 * 64);
  };
  // Fewer than 8 K steps and at most one 64 x 64 tile per CU: that tile has the least estimate by more than the 8 %
  // that a larger one is granted (350 a step against 410 or more, and more workgroups to fetch the operands), so the others
  // are not priced (0.2 us of a call of 6.5).
  const bool small_tiles = KT < 8 && g.forced_parts <= 1 && ((g.M + 63) / 64) * ((g.N + 63) / 64) <= NCU;
  // (an fp32 C that is read and written: four times the threads, K steps split over them, from 4 steps on; us, 440 x 928 x 440 7.2 / 6.1,
  // 1208 x 560 x 320 6.7 / 5.9, 328 x 2032 x 432 7.3 / 6.7)
  if (small_tiles) all[n_all++] = Choice{g.acc32 && p.aligned && KT >= 4 ? GEMM_64_K4 : GEMM_64_W4, 1, 64 * 64, cost(64, 64, 350, 0, 1, 1)};
  else if (g.forced_parts <= 1 && fits(256, 256)) all[n_all++] = Choice{big.variant, 1, 256 * 256, cost(256, 256, big.t, 0, 1, 1)};
  // The two-group kernel on 128 x 128 tiles, no K split across workgroups, in its two forms (fits
  // over K at 256 and 512 tiles, kernel time without the call):
  //   K steps of 64, two workgroups per CU: 0.84 us per step for a pair of tiles + 1.9 us per pair,
  //     0.52 us + 4 us for a tile alone on its CU (0.60 when K is not a multiple of 64: 2048 x 2048 x 2056
  //     takes 27.8 us, 24.8 on the split kernel);
  //   K steps of 128, one workgroup per CU: 0.436 us per 64 of K + 4.3 us per round.
  // One tile per CU: the 128-deep form (1024 x 4096 x 4096: 35.4 us against 40.8 on the register-
  // staged split kernel and 43.3 on the 64-deep form, hipBLASLt 36.6; 2048^3: 22.9 against 25.5,
  // hipBLASLt 25.3; 512 x 8192 x 8192: 65.7 against 76.4, hipBLASLt 64.1). Two tiles per CU: the
  // 64-deep form, whose workgroups hide each other's start and end (2048 x 4096 x 4096: 60.0
  // against 69.6 us, 82 on the split kernel, 73 on 128 big tiles; 1024 x 8192 x 8192: 114 against
  // 132, 153 and 134).
  if (pp && !small_tiles && g.forced_parts <= 1 && fits(128, 128)) {
    const int64_t wgs = ((g.M + 127) / 128) * ((g.N + 127) / 128);
    const int64_t base = (g.M + g.N) * g.K * 2 / 5200;
    const int64_t need = 6 * NCU / 10;
    const int64_t arrive = wgs >= need ? base : base * need / wgs;
    const int64_t pairs = wgs / (2 * NCU), rem = wgs - pairs * 2 * NCU;
    const int64_t own64 = pairs * (KT * 840 + 1900) +
                          (rem > NCU ? KT * 840 + 1900 : rem > 0 ? KT * (g.K % 64 ? 600 : 519) + 4000 : 0);
    // (with at most one tile per CU and K a multiple of 128 the 128-deep form is never slower, also
    // where both are bound by operand arrival: 128 x 28672 x 8192 116 against 134 us)
    if (wgs > NCU || g.K % 128 != 0)
      all[n_all++] = Choice{GEMM_128_PP16, 1, 128 * 128, (own64 > arrive ? own64 : arrive) + (wgs <= NCU ? c32 : 0)};
    if (g.K % 128 == 0) {
      const int64_t own128 = ((wgs + NCU - 1) / NCU) * (KT * 436 + 4300);
      all[n_all++] = Choice{GEMM_128_PP16_K128, 1, 128 * 128, (own128 > arrive ? own128 : arrive) + c32};
    }
  }
  // The kernels with two groups on alternate K steps (gemm_kp.hip). On a full chip their step is bound by what
  // the L2s deliver (about 17 TB/s), with fewer workgroups by its own latency (us per 64 of K, 80 / 160 / 256
  // workgroups, call included, B repeated: 256 x 128 0.56 / 0.64 / 0.73, 128 x 128 0.36 / 0.40 / 0.50; with B from
  // memory 80 workgroups take as long per step as 256 do, less so where K is split over more of them). Below on the scale of the other candidates, whose
  // times come out 1.1 to 1.25 of their estimates: over 280 problems of 6 to 300 tiles with B from memory the choice
  // is nowhere more than 8 % behind the best of the other tiles and 3 % ahead on average; rates that fall with the share
  // of busy CUs took these kernels for 40 to 110 tiles where they are up to 1.45 times slower (352 x 3176 x 5632 fp32
  // accumulate 37 us, 54; 245 x 4368 x 4456 30, 38; 2057 x 608 x 3200 26, 33).
  // bf16, us: 1024 x 8192 x 8192 128 on the best of the other tiles, 102 here; 2048 x 4096 x 4096 60 / 55;
  // 512 x 8192 x 8192 77 / 69; with K in two or four parts 777 x 4096 x 14336 131 / 97, 400 x 4096 x 11008
  // 57 / 47. The 6 us per round hold the sum of the two groups' results, which is why short K stays
  // with the others (2048^3: 21.4 on K steps of 128, 22.1 here).
  auto cost_kp = [&](int64_t bm, int parts) {
    const int64_t wgs = ((g.M + bm - 1) / bm) * ((g.N + 127) / 128) * parts;
    const int64_t rounds = (wgs + NCU - 1) / NCU, steps = (KT + parts - 1) / parts;
    const int64_t share = wgs < NCU ? wgs * 1000 / NCU : 1000;
    int64_t t_step = parts > 1 ? (bm > 128 ? 425 + 195 * share / 1000 : 206 + 190 * share / 1000) : bm > 128 ? 615 : 345 + 50 * share / 1000;
    // fewer rows: 224 0.94, 192 0.88, 160 0.81 of a step of 256. (One round of 240 workgroups measures 0.94, 0.91, 0.84. With those
    // the choice is worse: of 31 problems that they move to other tiles 16 lose, 303 x 11328 x 1280 19.8 / 23.7 us, 2624 x 6912 x 2304 90 / 107,
    // 822 x 4736 x 1280 17.1 / 21.1, and no more than 5 % is gained, 1532 x 6400 x 14016 276 / 263.)
    if (bm > 128) t_step -= t_step * (256 - bm) / 512;
    if (g.K % 64) t_step += t_step * 15 / 100;
    const int64_t act = gelu && parts == 1 && bm > 128 ? rounds * (34 * bm - 3000) : 0;
    const int64_t compute = rounds * (steps * t_step + (bm > 128 ? 6000 : 5700)) + act;
    const int64_t base = (g.M + g.N) * g.K * 2 / 5200, need = 6 * NCU / 10;
    const int64_t arrive = wgs >= need ? base : base * need / wgs;
    return (compute > arrive ? compute : arrive) + (parts > 1 ? 4000 + 2 * parts * g.M * g.N / 1000 : c32);
  };
  for (int parts = g.forced_parts > 0 ? g.forced_parts : 1; !small_tiles && parts <= (g.forced_parts > 0 ? g.forced_parts : 8); parts *= 2) {
    // every part keeps at least 8 K steps, and all parts' tiles fit the scratch that mlt_gemm_noalloc has
    // (a forced split may ask for more: mlt_gemm allocates it, mlt_gemm_noalloc refuses)
    if (parts > 1 && KT < 8 * parts) break;
    if (parts > 1 && g.forced_parts == 0 && parts * g.M * g.N * 4 > kStaticScratchBytes) break;
    if (pp && KT >= 8 * parts) {
      // (256 x 128 in 8 parts for one row of tiles only: 138 x 3840 x 14928 40 us, 51 in 4 parts of 128 x 128; but 852 x 920 x
      // 14784 50 in 8, 43 on the other tiles, 2375 x 272 x 16256 67, 60)
      if (g.M > 128 && (parts < 8 || g.M <= 256) && fits(64, 128)) {
        // the height with the least estimate; of equal ones with as many tiles the smaller, which multiplies less padding (150 x 8192 x 28672 in
        // four parts, bound by the operands' arrival: 110 us on 256 rows, 99 on 160)
        const auto tiles = [&](int64_t rows) { return (g.M + rows - 1) / rows; };
        Choice kp{GEMM_256X128_KP, parts, 256 * 128, cost_kp(256, parts)};
        for (int v : {GEMM_224X128_KP, GEMM_192X128_KP, GEMM_160X128_KP}) {
          const int64_t t = cost_kp(kp_rows(v), parts);
          if (t < kp.t || (t == kp.t && tiles(kp_rows(v)) == tiles(kp_rows(kp.variant)))) kp = Choice{v, parts, kp_rows(v) * 128, t};
        }
        all[n_all++] = kp;
      }
      if (fits(128, 128)) all[n_all++] = Choice{GEMM_128_KP, parts, 128 * 128, cost_kp(128, parts)};
    }
    for (const auto& c : KT / parts < 8 ? whole : p.aligned ? split : any) {
      if (!fits(c.bm, c.bn)) continue;
      all[n_all++] = Choice{c.variant, parts, c.bm * c.bn, cost(c.bm, c.bn, c.t, c.fixed, parts, c.kgroups)};
    }
  }
  if (n_all == 0) all[n_all++] = Choice{big.variant, 1, 256 * 256, cost(256, 256, big.t, 0, 1, 1)};
  int64_t best = all[0].t;
  for (int i = 1; i < n_all; ++i) best = all[i].t < best ? all[i].t : best;
  Choice pick = all[0];
  bool have = false;
  for (int i = 0; i < n_all; ++i) {
    if (all[i].t > best + best / 12) continue;
    bool better = !have || all[i].area > pick.area;
    if (have && all[i].area == pick.area) {
      // same tile: the fewer parts, unless more parts are estimated more than 5 % faster
      if (all[i].parts == pick.parts) better = all[i].t < pick.t;
      else if (all[i].parts < pick.parts) better = all[i].t <= pick.t + pick.t / 20;
      else better = all[i].t + all[i].t / 20 < pick.t;
    }
    if (better) pick = all[i];
    have = true;
  }
  p.variant = pick.variant; p.parts = pick.parts;
  if (skinny && g.forced == GEMM_AUTO && g.M > 32 && stream_wins(g, NCU, p)) {
    plan_skinny(g, NCU, p);
    return p;
  }
  int v = pick.variant;
  const int best_parts = pick.parts;
  if (g.forced >= GEMM_256 && g.forced < GEMM_NUM_VARIANTS && g.forced != GEMM_SKINNY) v = g.forced;
  if (v == GEMM_256_PP16 && !gemm_pp_ok(g)) v = GEMM_256_W8;
  if (kp_rows(v) && !pp) v = v == GEMM_128_KP ? GEMM_128_W8 : GEMM_256_W8;
  if (v == GEMM_256_W4 && !gemm_w4_ok(g)) v = GEMM_256_W8;
  if (v == GEMM_128_PP16_K128 && (!pp || g.K % 128)) v = GEMM_128_PP16;
  if (v == GEMM_128_PP16 && !pp) v = GEMM_128_W8;
  // a forced kernel keeps the split only if it is one of the kernels that can run it
  const bool can_split = v == GEMM_128_K2 || v == GEMM_64X128_K2 || v == GEMM_64_K4 || v == GEMM_128_W8 ||
                         v == GEMM_64X128_W8 || v == GEMM_64_W4 || kp_rows(v);
  p.parts = can_split ? best_parts : 1;
  p.scratch_bytes = p.parts > 1 ? (int64_t)p.parts * g.M * g.N * 4 : 0;
  p.variant = v;
  p.bk = 64;
  switch (v) {
    case GEMM_256: p.bm = p.bn = 256; p.wm = 2; p.wn = 2;
      p.name = g.transB ? "gemm_nt_256x256x64_w2x2" : "gemm_nn_256x256x64_w2x2"; break;
    case GEMM_256_W8: p.bm = p.bn = 256; p.wm = 2; p.wn = 4;
      p.name = g.transB ? "gemm_nt_256x256x64_w2x4" : "gemm_nn_256x256x64_w2x4"; break;
    case GEMM_256_W8X1: p.bm = p.bn = 256; p.wm = 8; p.wn = 1;
      p.name = g.transB ? "gemm_nt_256x256x64_w8x1" : "gemm_nn_256x256x64_w8x1"; break;
    case GEMM_256_W1X8: p.bm = p.bn = 256; p.wm = 1; p.wn = 8;
      p.name = g.transB ? "gemm_nt_256x256x64_w1x8" : "gemm_nn_256x256x64_w1x8"; break;
    case GEMM_256_PP16: p.bm = p.bn = 256; p.wm = 2; p.wn = 4;
      p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
      p.name = g.transB ? "gemm_nt_256x256x64_w2x4_pp16" : "gemm_nn_256x256x64_w2x4_pp16"; break;
    case GEMM_256X128_KP: p.bm = 256; p.bn = 128; p.wm = 2; p.wn = 2;
      p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
      p.name = g.transB ? "gemm_nt_256x128x64_w2x2_kp2" : "gemm_nn_256x128x64_w2x2_kp2"; break;
    case GEMM_224X128_KP: p.bm = 224; p.bn = 128; p.wm = 2; p.wn = 2;
      p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
      p.name = g.transB ? "gemm_nt_256x128x64_w2x2_kp2" : "gemm_nn_256x128x64_w2x2_kp2"; p.suffix = "_rows224"; break;
    case GEMM_192X128_KP: p.bm = 192; p.bn = 128; p.wm = 2; p.wn = 2;
      p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
      p.name = g.transB ? "gemm_nt_256x128x64_w2x2_kp2" : "gemm_nn_256x128x64_w2x2_kp2"; p.suffix = "_rows192"; break;
    case GEMM_160X128_KP: p.bm = 160; p.bn = 128; p.wm = 2; p.wn = 2;
      p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
      p.name = g.transB ? "gemm_nt_256x128x64_w2x2_kp2" : "gemm_nn_256x128x64_w2x2_kp2"; p.suffix = "_rows160"; break;
    case GEMM_128_KP: p.bm = p.bn = 128; p.wm = 2; p.wn = 2;
      p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
      p.name = g.transB ? "gemm_nt_128x128x64_w2x2_kp2" : "gemm_nn_128x128x64_w2x2_kp2"; break;
    case GEMM_128_PP16: p.bm = p.bn = 128; p.wm = 2; p.wn = 4;
      p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
      p.name = g.transB ? "gemm_nt_128x128x64_w2x4_pp16" : "gemm_nn_128x128x64_w2x4_pp16"; break;
    case GEMM_128_PP16_K128: p.bm = p.bn = 128; p.bk = 128; p.wm = 2; p.wn = 4;
      p.mfma_m = 16; p.mfma_n = 16; p.mfma_k = 32;
      p.name = g.transB ? "gemm_nt_128x128x128_w2x4_pp16" : "gemm_nn_128x128x128_w2x4_pp16"; break;
    case GEMM_256_W4: p.bm = p.bn = 256; p.wm = 2; p.wn = 2;
      p.name = g.transB ? "gemm_nt_256x256x64_w2x2_swp" : "gemm_nn_256x256x64_w2x2_swp"; break;
    case GEMM_128_W8: p.bm = p.bn = 128; p.wm = 2; p.wn = 4;
      p.name = g.transB ? "gemm_nt_128x128x64_w2x4" : "gemm_nn_128x128x64_w2x4"; break;
    case GEMM_64X128_W8: p.bm = 64; p.bn = 128; p.wm = 2; p.wn = 4;
      p.name = g.transB ? "gemm_nt_64x128x64_w2x4" : "gemm_nn_64x128x64_w2x4"; break;
    case GEMM_64_W4: p.bm = p.bn = 64; p.wm = 2; p.wn = 2;
      p.name = g.transB ? "gemm_nt_64x64x64_w2x2" : "gemm_nn_64x64x64_w2x2"; break;
    case GEMM_128_K2: p.bm = p.bn = 128; p.wm = 2; p.wn = 4;
      p.name = g.transB ? "gemm_nt_128x128x64_w2x4_k2" : "gemm_nn_128x128x64_w2x4_k2"; break;
    case GEMM_64X128_K2: p.bm = 64; p.bn = 128; p.wm = 2; p.wn = 4;
      p.name = g.transB ? "gemm_nt_64x128x64_w2x4_k2" : "gemm_nn_64x128x64_w2x4_k2"; break;
    case GEMM_64_K4: p.bm = p.bn = 64; p.wm = 2; p.wn = 2;
      p.name = g.transB ? "gemm_nt_64x64x64_w2x2_k4" : "gemm_nn_64x64x64_w2x2_k4"; break;
    default: p.variant = GEMM_256_W8; p.bm = p.bn = 256; p.wm = 2; p.wn = 4;
      p.name = g.transB ? "gemm_nt_256x256x64_w2x4" : "gemm_nn_256x256x64_w2x4"; break;
  }
  if (!p.aligned) p.name = any_name(v, g.transB);
  return p;
}

int run_splitk_reduce(const GemmArgs& g, int parts, int64_t part_stride, hipStream_t s) {
  return g.dtype == MLT_BF16 ? launch_splitk_reduce<bf16_tag>(g, parts, part_stride, s)
                             : launch_splitk_reduce<f16_tag>(g, parts, part_stride, s);
}

template <typename Tag>
static int run_gemm_t(const GemmArgs& g, const GemmPlan& p, hipStream_t s) {
  if (!p.aligned) return run_gemm_any(g, p.variant, s);
  switch (p.variant) {
    case GEMM_ZERO: {
      if (g.acc32) return MLT_OK;
      const int64_t n = g.M * g.N;
      hipLaunchKernelGGL(gemm_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                         (int)g.M, (int)g.N, g.C, g.ldc);
      return hipGetLastError() == hipSuccess ? MLT_OK : MLT_ERR_LAUNCH;
    }
    case GEMM_GENERAL: return launch_general<Tag>(g, s);
    case GEMM_256: return launch_tile_tb<Tag, true, 256, 256, 64, 2, 2>(g, s);
    case GEMM_256_W8X1: return launch_tile_tb<Tag, true, 256, 256, 64, 8, 1>(g, s);
    case GEMM_256_W1X8: return launch_tile_tb<Tag, true, 256, 256, 64, 1, 8>(g, s);
    case GEMM_256_PP16: return run_gemm_pp(g, 256, 64, s);
    case GEMM_128_PP16: return run_gemm_pp(g, 128, 64, s);
    case GEMM_128_PP16_K128: return run_gemm_pp(g, 128, 128, s);
    case GEMM_256X128_KP: case GEMM_224X128_KP: case GEMM_192X128_KP: case GEMM_160X128_KP: case GEMM_128_KP:
      return run_gemm_kp(g, kp_rows(p.variant), s);
    case GEMM_256_W4: return run_gemm_w4(g, s);
    case GEMM_SKINNY: return run_gemm_skinny(g, s);
  }
  const int rc = launch_small_tile<Tag, true>(g, p.variant, s);
  return rc == -1 ? MLT_ERR_UNSUPPORTED : rc;
}

// Scratch for the partial results of a split across workgroups: one buffer per (device, stream)
// pair, so that calls on different streams never share one (hipStreamPerThread is one handle for a stream of each
// thread's own, and has a buffer per thread); allocated at the first call that needs
// it (hipMalloc; no device synchronisation), grown by doubling (the smaller buffer is kept until the
// process ends: work already enqueued may still use it), used in stream order. The tables, one for streams and one for
// threads, are small and fixed; when one is full, or an allocation fails, a GEMM gets a stream-ordered
// allocation of its own (or, if that fails too, runs without the split). A call that is being recorded
// into a graph gets none, also where the stream has a buffer: the graph would go on using it whenever
// and on whatever stream it is replayed, beside the stream's own calls and beside other graphs recorded
// on it, in no order with either.
namespace {
struct ScratchSlot { int dev; hipStream_t stream; uint64_t thread; float* ptr; int64_t bytes; };
constexpr int kScratchSlots = 32;
struct ScratchTable { ScratchSlot slot[kScratchSlots]; int used; };
ScratchTable g_scratch, g_thread_scratch;
std::mutex g_scratch_mu;

// a number that no other thread has or had (a thread's id is used again after its end, when its calls may still run)
uint64_t this_thread() {
  static std::atomic<uint64_t> last{0};
  static thread_local const uint64_t id = ++last;
  return id;
}

}  // namespace

bool stream_is_capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) { (void)hipGetLastError(); return false; }
  return st != hipStreamCaptureStatusNone;
}

__global__ void zero_counters_kernel(uint32_t* counters) { counters[blockIdx.x * blockDim.x + threadIdx.x] = 0; }

float* cached_scratch(int64_t bytes, hipStream_t s) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
  if (stream_is_capturing(s)) return nullptr;
  const uint64_t thread = s == hipStreamPerThread ? this_thread() : 0;
  ScratchTable& table = thread ? g_thread_scratch : g_scratch;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  ScratchSlot* slot = nullptr;
  for (int i = 0; i < table.used; ++i)
    if (table.slot[i].dev == dev && table.slot[i].stream == s && table.slot[i].thread == thread) slot = &table.slot[i];
  if (slot && slot->bytes >= bytes) return slot->ptr;
  if (!slot) {
    if (table.used == kScratchSlots) return nullptr;
    slot = &table.slot[table.used];
    *slot = ScratchSlot{dev, s, thread, nullptr, 0};
  }
  int64_t want = slot->bytes > 0 ? 2 * slot->bytes : (int64_t)4 << 20;
  while (want < bytes) want *= 2;
  void* p = nullptr;
  if (hipMalloc(&p, (size_t)want + kScratchCounters * 4) != hipSuccess || !p) { (void)hipGetLastError(); return nullptr; }
  hipLaunchKernelGGL(zero_counters_kernel, dim3(kScratchCounters / 256), dim3(256), 0, s, static_cast<uint32_t*>(p));
  if (hipGetLastError() != hipSuccess) { (void)hipFree(p); return nullptr; }
  if (slot == &table.slot[table.used]) ++table.used;
  slot->ptr = reinterpret_cast<float*>(static_cast<uint32_t*>(p) + kScratchCounters);
  slot->bytes = want;
  return slot->ptr;
}

// The scratch of the entry point that may not allocate (mlt_gemm_noalloc): a fixed array in
// device memory, one copy per GPU the library runs on, held until the process ends. In host code
// the array's name is only a handle; its device address is looked up once per device, with that
// device current, and only that address is ever handed to kernels. Every call on a GPU shares
// that GPU's array (calls that overlap on one GPU race); nothing in it has to start at zero: each
// part of a K split writes every element of its slice before the second kernel reads them.
namespace {
static __device__ __align__(256) float scratch[kStaticScratchBytes / sizeof(float)];
constexpr int kMaxDevices = 64;
float* g_static_scratch[kMaxDevices];
std::mutex g_static_scratch_mu;
}  // namespace

float* static_scratch_of_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return nullptr; }
  std::lock_guard<std::mutex> lock(g_static_scratch_mu);
  if (!g_static_scratch[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return nullptr; }
    g_static_scratch[dev] = static_cast<float*>(p);
  }
  return g_static_scratch[dev];
}

int run_gemm(const GemmArgs& g_in, GemmPlan& p, hipStream_t s) {
  GemmArgs g = g_in;
  g.parts = p.parts;
  bool own = false;
  if (p.parts > 1 && !g.scratch) {
    g.scratch = cached_scratch(p.scratch_bytes, s);
    if (g.scratch) {
      g.counters = scratch_counters(g.scratch);
    } else {
      void* ws = nullptr;
      if (!stream_is_capturing(s) && hipMallocAsync(&ws, (size_t)p.scratch_bytes, s) == hipSuccess && ws) {
        g.scratch = static_cast<float*>(ws);
        own = true;
      } else {
        (void)hipGetLastError();
        // (the choice of the tile kernels for a short A was made for their split: us per captured call, 64 x 8192 x 14336
        // 112 on tiles, 58 streaming)
        if (g.forced == GEMM_AUTO && gemm_skinny_ok(g)) { g.forced_parts = 1; p = plan_gemm(g); }
        g.parts = 1;
        p.parts = 1;                                       // what ran, for the reported kernel name
        p.scratch_bytes = 0;
      }
    }
  }
  const int rc = g.dtype == MLT_BF16 ? run_gemm_t<bf16_tag>(g, p, s) : run_gemm_t<f16_tag>(g, p, s);
  if (own) (void)hipFreeAsync(g.scratch, s);
  return rc;
}

}  // namespace mlt
