// Skinny GEMM C = A*B for gfx950: M <= 64 rows (next-token decode shapes, Section 4.1 of the paper
// (arXiv 2503.14985): memory-bound GEMMs with a small m), B given as the N x K row-major array
// (k contiguous). The whole cost is reading B once from HBM, and the kernel is built around that stream:
//   * one workgroup of 8 wavefronts per CU, each with its even share of the columns of C (rows of the stored B),
//     contiguous, whatever their number, in blocks of up to 16. The wavefronts split K: wavefront w takes the
//     pieces of 128 k numbered w, w + 8, ..., so that at any time the workgroup reads 2 KB of each of its rows;
//   * every wavefront has an LDS ring of its own (20 KB) and is alone with it: it fetches its pieces of A and of
//     its columns of B straight into the ring (global_load_lds_dwordx4, 4 rows x 256 contiguous bytes per
//     instruction), several slots ahead, waits for the oldest by count, reads its MFMA fragments (16x16x32) and
//     refills it. No barrier until the end, no wavefront that only fetches, and A, which comes from L2, arrives in the
//     same stream as B, as far ahead (a CU's loads come back in order, so a load of A waits for the
//     loads of B in front of it wherever it goes);
//   * the rows of a piece are stored permuted (16-byte chunk c of row r at position c ^ r): the source
//     address of a lane is free, its LDS position is not, and the 16 lanes that read 16 rows at one k
//     position must hit 16 distinct bank groups;
//   * a wavefront starts some pieces into its share and goes round, each at another place: all of them walk through K
//     in step, and where the rows of B are a power of two long (K = 4096: 8 KB) the whole chip would read the same 2 KB
//     out of every 8 at a time, a part of the memory's channels (us, from the first piece / going round: 1 x 8192 x 4096 17.9 / 12.5, 16 x 8192 x
//     8192 28.8 / 25.4, 32 x 4096 x 8192 19.6 / 16.9, 16 x 28672 x 4096 39.6 / 36.7; 16 x 9000 x 2880 12.6 / 12.7). Not where rows do not start on
//     64 bytes: two wavefronts' neighbouring pieces then share a line, which comes from memory once only if both ask for it at the same
//     time (1 x 22912 x 7768 64.3 / 73.4, 15 x 8192 x 4104 14.8 / 16.5; but rows of 64 bytes' multiples, 1 x 8192 x 4128 16.4 / 15.3);
//   * with more than 16 columns a piece of A is fetched once for a group of up to 8 column blocks (4 from three row
//     tiles on), whose accumulators stay in registers;
//   * at the end the 8 partial tiles of a column block meet in LDS and are added in wavefront order.
//
// K may also be split over 2, 4 or 8 workgroups (PARTS): a workgroup then has that many times the columns and that part
// of K, so every CU fetches that much less of A, which all of them fetch in full otherwise (64 rows x 4096: 512 KB a CU
// beside 128 KB of B). The parts leave fp32 partial results in a scratch, and the one that comes last at a
// counter adds them in the order of the parts: no second launch, no atomics on values, the same bits on every run.
//
// What bounds it: what a CU's memory path takes (about 64 bytes per clock, A and B together: 1 x 4096 x 4096 7.4 us,
// 16 rows 8.3, 32 9.7, where a kernel that only reads B takes 6.4 and an empty one 2.0), for large B the
// memory (16 x 28672 x 8192 71 us = 6.6 TB/s), and for short calls the way to the first load and what follows the last one. Hence the
// order of the arguments (what the first loads need lies in their first 64 bytes and is read at once: 8 x 4096 x 1024 4.15 -> 3.93 us) and
// instances for one and for two column blocks, whose code is not spread over eight (3 x 3392 x 128 3.3 -> 3.1, 8 x 8192 x 1024 5.54 -> 5.43).
// The kernels before it, one with direct loads of 64 bytes per row into the
// operand registers, one with four fetching and four computing wavefronts and a barrier per 16 KB: 16 x 4096 x 4096
// 11.5 and 10.7 us, 16 x 28672 x 8192 123 and 83, 32 x 5120 x 5120 37 and 21.
#include "mlt_common.h"
#include "mlt_internal.h"

namespace mlt {

namespace {

constexpr int SK_NW = 8;              // wavefronts per workgroup = K split
constexpr int SK_NT = SK_NW * 64;
constexpr int SK_KP = 128;            // k values per piece
constexpr int SK_RING = 20 * 1024;    // LDS ring of a wavefront
constexpr int SK_SMEM = SK_NW * SK_RING;

// MT: 16-row tiles of A. AU, BU: load instructions (4 rows each) for a piece of a row tile, of a column block: 4, or
// fewer where no more rows or columns exist (each instruction costs a CU the same, whatever it fetches)
template <int MT, int AU, int BU> struct SkCfg {
  static constexpr int LU = AU > BU ? AU : BU;
  static constexpr int SLOT = LU * 1024;
  static constexpr int R = SK_RING / SLOT < 12 ? SK_RING / SLOT : 12;     // slots
  static constexpr int CB = 4 * BU;                                       // columns per block
  static constexpr int MAX_GB = BU < 4 ? 1 : MT <= 2 ? 8 : 4;             // blocks per group, at most
  static_assert(MAX_GB * MT * 1024 <= SK_RING, "a wavefront's partial tiles lie in its own ring");
  static_assert((R - 1) * LU < 63, "loads in flight are counted");
};

// share, rest: columns per workgroup, and how many of them have one more. GB: column blocks per group, at least those that a workgroup
// has or MAX_GB. PARTS: blockIdx.y is the part of K; `part` holds
// [part][M][N] floats, `counter` one zero per blockIdx.x (left as zero); without counters (null) another kernel adds the parts.
template <typename Tag, int MT, int AU, int BU, bool PARTS, int GB>
__global__ __launch_bounds__(SK_NT, 2) void gemm_skinny_kernel(
    int M, int N, int K, int share, int rest, int lda, int ldb, int act, const uint16_t* __restrict__ A,
    const uint16_t* __restrict__ B, uint16_t* __restrict__ C, int64_t ldc, const uint16_t* __restrict__ bias,
    float* __restrict__ part, uint32_t* __restrict__ counter) {
  asm volatile("" : : "s"(M), "s"(K), "s"(share), "s"(rest), "s"(lda), "s"(ldb), "s"(A), "s"(B));   // all read here, not one behind the other
  typedef typename Elem<Tag>::vec8 V8;
  typedef SkCfg<MT, AU, BU> L;
  constexpr int CB = L::CB, R = L::R;
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int bid = (int)blockIdx.x, c0 = bid * share + (bid < rest ? bid : rest), c1 = c0 + share + (bid < rest ? 1 : 0);
  const int nblk = GB == 1 ? 1 : (c1 - c0 + CB - 1) / CB;
  // pieces p0 .. p1 - 1, of them first = p0 + wave, first + 8, ..., from `start` on and then from the first again
  int p0 = 0, p1 = (K + SK_KP - 1) / SK_KP;
  if (PARTS) {
    const int per = (p1 + (int)gridDim.y - 1) / (int)gridDim.y;
    p0 = (int)blockIdx.y * per;
    p1 = p0 + per < p1 ? p0 + per : p1;
  }
  const int first = p0 + wave, mine = p1 > first ? (p1 - first + SK_NW - 1) / SK_NW : 0;
  const bool shared_lines = ((reinterpret_cast<uintptr_t>(B) | (uintptr_t)((uint32_t)ldb * 2u)) & 63) != 0;
  const int start = first + (shared_lines ? 0 : wave & (mine >= 8 ? 7 : mine >= 4 ? 3 : mine >= 2 ? 1 : 0)) * SK_NW;
  const uint32_t ring = (uint32_t)(uintptr_t)(lptr_t)smem + (uint32_t)wave * SK_RING;

  // load instruction i of a slot: rows 4 i .. 4 i + 3, lane l the chunk at position l % 16 of row 4 i + l / 16
  uint32_t va[AU], vb[BU];
#pragma unroll
  for (int i = 0; i < AU; ++i)
    va[i] = (uint32_t)(i * 4 + lane / 16) * (uint32_t)lda * 2u + (uint32_t)((lane % 16) ^ (i * 4 + lane / 16)) * 16u;
#pragma unroll
  for (int i = 0; i < BU; ++i)
    vb[i] = (uint32_t)(i * 4 + lane / 16) * (uint32_t)ldb * 2u + (uint32_t)((lane % 16) ^ (i * 4 + lane / 16)) * 16u;

  for (int base = 0; base < nblk; base += GB) {
    const int nb = GB == 1 ? 1 : nblk - base < GB ? nblk - base : GB;
    const int S = MT + nb, T = mine * S;                 // slots per piece (row tiles, then column blocks), in all
    f32x4 acc[GB][MT];
#pragma unroll
    for (int gb = 0; gb < GB; ++gb)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[gb][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // the cursor: the next slot of the stream to fetch, f_s of piece f_p, and its place
    int f_t = 0, f_s = 0, f_p = start;
    uint32_t f_slot = ring;
    int issued = 0, need = 0;                            // load instructions issued; up to the end of the slot in hand
    auto fetch = [&]() __attribute__((always_inline)) {
      if (f_t >= T) return;
      const int k0 = f_p * SK_KP;
      const bool tail = k0 + SK_KP > K;
      // rows past the matrix (past this workgroup's columns) and chunks past K: the piece's first chunk for all such
      // lanes, never stored or zeroed later; the instruction stays, and with it the count of loads in flight
      if (f_s < MT) {
        const char* src = reinterpret_cast<const char*>(A + (int64_t)(f_s * 16) * (uint32_t)lda + k0);
        const int rows = M - f_s * 16;
#pragma unroll
        for (int i = 0; i < AU; ++i) {
          const int row = i * 4 + lane / 16;
          uint32_t off = row < rows ? va[i] : 0u;
          if (tail && k0 + ((lane % 16) ^ row) * 8 >= K) off = 0u;
          load_lds16(src, off, f_slot + i * 1024u);
        }
        issued += AU;
      } else {
        const int n0 = c0 + (base + f_s - MT) * CB;
        const char* src = reinterpret_cast<const char*>(B + (int64_t)n0 * (uint32_t)ldb + k0);
        const int rows = c1 - n0;
#pragma unroll
        for (int i = 0; i < BU; ++i) {
          const int row = i * 4 + lane / 16;
          uint32_t off = row < rows ? vb[i] : 0u;
          if (tail && k0 + ((lane % 16) ^ row) * 8 >= K) off = 0u;
          load_lds16_stream(src, off, f_slot + i * 1024u);
        }
        issued += BU;
      }
      ++f_t;
      f_slot = f_slot == ring + (R - 1) * L::SLOT ? ring : f_slot + L::SLOT;
      if (++f_s == S) {
        f_s = 0;
        f_p = f_p + SK_NW < p1 ? f_p + SK_NW : first;
      }
    };
#pragma unroll
    for (int i = 0; i < R; ++i) fetch();

    // the next slot, of n loads: wait until it has landed (what was issued after it may be in flight), read its
    // fragments, refill its place
    uint32_t slot = ring;
    auto take = [&](u32x4 (&f)[4], int n) __attribute__((always_inline)) {
      need += n;
      int later = issued - need;
#ifdef MLT_DEBUG_BARRIERS
      later = 0;                                         // waits for all of them, so that a count that is too lax shows
#endif
      if (L::LU == 4 && later >= 16) __builtin_amdgcn_s_waitcnt(wait_imm(16, 15));
      else if (L::LU == 4 && later >= 12) __builtin_amdgcn_s_waitcnt(wait_imm(12, 15));
      else if (later >= 10) __builtin_amdgcn_s_waitcnt(wait_imm(10, 15));
      else if (later >= 8) __builtin_amdgcn_s_waitcnt(wait_imm(8, 15));
      else if (later >= 6) __builtin_amdgcn_s_waitcnt(wait_imm(6, 15));
      else if (later >= 4) __builtin_amdgcn_s_waitcnt(wait_imm(4, 15));
      else if (later >= 2) __builtin_amdgcn_s_waitcnt(wait_imm(2, 15));
      else if (later >= 1) __builtin_amdgcn_s_waitcnt(wait_imm(1, 15));
      else __builtin_amdgcn_s_waitcnt(wait_imm(0, 15));
      __builtin_amdgcn_sched_barrier(0);
      const int row = r16 & (4 * n - 1);                 // (fewer than 16 rows: repeated, never stored)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        f[j] = *(const MLT_LDS u32x4*)(uintptr_t)(slot + (uint32_t)row * 256u + (uint32_t)(((j * 4 + q) ^ row) << 4));
      __builtin_amdgcn_s_waitcnt(wait_imm(63, 0));
      __builtin_amdgcn_sched_barrier(0);
      fetch();
      __builtin_amdgcn_sched_barrier(0);
      slot = slot == ring + (R - 1) * L::SLOT ? ring : slot + L::SLOT;
    };
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    for (int i = 0, piece = start; i < mine; ++i, piece = piece + SK_NW < p1 ? piece + SK_NW : first) {
      const int k0 = piece * SK_KP;
      const bool tail = k0 + SK_KP > K;                  // chunks past K: zeros in both operands
      u32x4 af[MT][4];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) take(af[mt], AU);
      if (tail) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (k0 + j * 32 + 8 * q >= K) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) af[mt][j] = zero4;
          }
      }
#pragma unroll
      for (int gb = 0; gb < GB; ++gb)
        if (gb < nb) {
          u32x4 bf[4];
          take(bf, BU);
          if (tail) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (k0 + j * 32 + 8 * q >= K) bf[j] = zero4;
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              acc[gb][mt] = mfma16(__builtin_bit_cast(V8, af[mt][j]), __builtin_bit_cast(V8, bf[j]), acc[gb][mt]);
        }
    }
    // the partial tiles into the wavefront's own ring (all its loads have landed), then their sums
    float* own = reinterpret_cast<float*>(smem + wave * SK_RING);
#pragma unroll
    for (int gb = 0; gb < GB; ++gb)
      if (gb < nb) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int r = 0; r < 4; ++r) own[(gb * MT + mt) * 256 + (4 * q + r) * 16 + r16] = acc[gb][mt][r];
      }
    __syncthreads();
    // (one element at a time: a call of a few microseconds notices every line of code that it has to fetch)
    for (int e = tid; e < nb * MT * 256; e += SK_NT) {
      const int t = e >> 8, gr = t % MT * 16 + ((e >> 4) & 15), gc = c0 + (base + t / MT) * CB + (e & 15);
      if (gr < M && gc < c1 && (e & 15) < CB) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < SK_NW; ++w) sum += reinterpret_cast<const float*>(smem)[w * (SK_RING / 4) + e];
        if (PARTS) store_shared(part + ((int64_t)blockIdx.y * M + gr) * N + gc, sum);
        else C[(int64_t)gr * ldc + gc] = Elem<Tag>::from_f32(epi_act(bias ? sum + Elem<Tag>::to_f32(bias[gc]) : sum, act));
      }
    }
    if (base + GB < nblk) __syncthreads();
  }
  if (!PARTS || !counter) return;

  // the last part of these columns to get here adds them all
  if (!last_to_arrive(counter + bid, gridDim.y, reinterpret_cast<uint32_t*>(smem))) return;
  const int cols = c1 - c0, parts = (int)gridDim.y;
  // (EB elements of a thread at a time, all their parts requested before the first is used: each such round is a trip to
  // memory)
  constexpr int EB = MT == 1 ? 2 : 4;
  for (int e0 = tid; e0 < M * cols; e0 += EB * SK_NT) {
    float v[8][EB];
    int64_t at[EB];
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int e = e0 + i * SK_NT < M * cols ? e0 + i * SK_NT : e0;
      at[i] = (int64_t)(e / cols) * N + c0 + e % cols;
    }
#pragma unroll
    for (int p = 0; p < 8; ++p)
      if (p < parts) {
#pragma unroll
        for (int i = 0; i < EB; ++i) v[p][i] = load_shared(part + (int64_t)p * M * N + at[i]);
      }
#pragma unroll
    for (int p = 1; p < 8; ++p)
      if (p < parts) {
#pragma unroll
        for (int i = 0; i < EB; ++i) v[0][i] += v[p][i];
      }
#pragma unroll
    for (int i = 0; i < EB; ++i)
      if (e0 + i * SK_NT < M * cols) {
        const int gr = (e0 + i * SK_NT) / cols, gc = c0 + (e0 + i * SK_NT) % cols;
        C[(int64_t)gr * ldc + gc] = Elem<Tag>::from_f32(epi_act(bias ? v[0][i] + Elem<Tag>::to_f32(bias[gc]) : v[0][i], act));
      }
  }
}

template <typename Tag, int MT, int AU, int BU, bool PARTS, int GB>
int launch_skinny_blocks(const GemmArgs& g, unsigned nwg, hipStream_t s) {
  auto kern = gemm_skinny_kernel<Tag, MT, AU, BU, PARTS, GB>;
  static thread_local int configured_dev = -1;            // opt in to > 64 KB LDS once per device
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MLT_ERR_DEVICE;
  if (configured_dev != dev) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, SK_SMEM) != hipSuccess) {
      (void)hipGetLastError();
      return MLT_ERR_LAUNCH;
    }
    configured_dev = dev;
  }
  const int parts = PARTS ? g.parts : 1;
  hipLaunchKernelGGL(kern, dim3(nwg, (unsigned)parts), dim3(SK_NT), SK_SMEM, s, (int)g.M, (int)g.N, (int)g.K,
                     (int)(g.N / nwg), (int)(g.N % nwg), (int)g.lda, (int)g.ldb, g.act, g.A, g.B, g.C, g.ldc, g.bias, g.scratch, g.counters);
  if (hipGetLastError() != hipSuccess) return MLT_ERR_LAUNCH;
  return PARTS && !g.counters ? run_splitk_reduce(g, parts, g.M * g.N, s) : MLT_OK;
}

template <typename Tag, int MT, int AU, int BU, bool PARTS>
int launch_skinny(const GemmArgs& g, int64_t ncu, hipStream_t s) {
  constexpr int MAX_GB = SkCfg<MT, AU, BU>::MAX_GB;
  const int64_t want = ncu / (PARTS ? g.parts : 1) > 0 ? ncu / (PARTS ? g.parts : 1) : 1;
  const unsigned nwg = (unsigned)(g.N < want ? g.N : want);   // one workgroup per CU, every one with columns
  const int64_t blocks = ((g.N + nwg - 1) / nwg + 4 * BU - 1) / (4 * BU);
  if (blocks == 1) return launch_skinny_blocks<Tag, MT, AU, BU, PARTS, 1>(g, nwg, s);
  if (blocks == 2 && MAX_GB == 8) return launch_skinny_blocks<Tag, MT, AU, BU, PARTS, MAX_GB == 8 ? 2 : MAX_GB>(g, nwg, s);
  return launch_skinny_blocks<Tag, MT, AU, BU, PARTS, MAX_GB>(g, nwg, s);
}

template <typename Tag, int MT, int AU>
int run_skinny_cols(const GemmArgs& g, hipStream_t s) {
  DeviceInfo di;
  const int64_t ncu = device_info(di) && di.ncu > 0 ? di.ncu : 256;
  if (g.parts > 1) return launch_skinny<Tag, MT, AU, 4, true>(g, ncu, s);
  switch (gemm_skinny_cols(g.N, g.parts, ncu)) {
    case 4: return launch_skinny<Tag, MT, AU, 1, false>(g, ncu, s);
    case 8: return launch_skinny<Tag, MT, AU, 2, false>(g, ncu, s);
  }
  return launch_skinny<Tag, MT, AU, 4, false>(g, ncu, s);
}

template <typename Tag>
int run_skinny_t(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 4) return run_skinny_cols<Tag, 1, 1>(g, s);
  switch ((g.M + 15) / 16) {
    case 1: return run_skinny_cols<Tag, 1, 4>(g, s);
    case 2: return run_skinny_cols<Tag, 2, 4>(g, s);
    case 3: return run_skinny_cols<Tag, 3, 4>(g, s);
    case 4: return run_skinny_cols<Tag, 4, 4>(g, s);
  }
  return MLT_ERR_UNSUPPORTED;
}

}  // namespace

bool gemm_skinny_ok(const GemmArgs& g) {
  auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (!g.transB || g.acc32 || g.M > 64 || g.N < 1024) return false;
  if (!al16(g.A) || !al16(g.B)) return false;
  if (g.K % 8 || g.lda % 8 || g.ldb % 8) return false;
  // 32-bit byte offsets from a block's first row (and with them 32-bit row strides)
  return g.lda * 2 * 16 + g.K * 2 < ((int64_t)1 << 32) && g.ldb * 2 * 16 + g.K * 2 < ((int64_t)1 << 32);
}

int run_gemm_skinny(const GemmArgs& g, hipStream_t s) {
  return g.dtype == MLT_BF16 ? run_skinny_t<bf16_tag>(g, s) : run_skinny_t<f16_tag>(g, s);
}

}  // namespace mlt
