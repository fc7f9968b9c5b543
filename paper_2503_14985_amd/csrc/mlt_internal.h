// Host-side plumbing shared by the entry points and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mlt {

enum GemmVariant {
  GEMM_AUTO = -1, GEMM_ZERO = 0, GEMM_GENERAL = 1,
  GEMM_256 = 2,       // 256x256x64, 4 wavefronts (2x2) of 128x128 (tiling hint "square" with a ragged K)
  GEMM_256_W8 = 4,    // 256x256x64, 8 wavefronts (2x4) of 128x64 (big tiles when the direct loads do not apply)
  GEMM_SKINNY = 7,    // M <= 64, B stored N x K: B streamed through an LDS ring per wavefront, K split over 8 wavefronts
  GEMM_256_W4 = 10,   // 256x256x64, 4 wavefronts (2x2) of 128x128, software-pipelined, direct-to-LDS loads
  GEMM_256_PP16 = 11, // 256x256x64, 8 wavefronts (2x4), two-group schedule, direct-to-LDS loads, 16x16x32 MFMAs
  GEMM_256_W8X1 = 12, // 256x256x64, 8 wavefronts as 8x1: row strips of 32 x 256 ("horizontal")
  GEMM_256_W1X8 = 13, // 256x256x64, 8 wavefronts as 1x8: column strips of 256 x 32 ("vertical")
  GEMM_128_W8 = 14,   // 128x128x64, 8 wavefronts (2x4) of 64x32
  GEMM_64X128_W8 = 15, // 64x128x64, 8 wavefronts (2x4) of 32x32
  GEMM_64_W4 = 16,    // 64x64x64, 4 wavefronts (2x2) of 32x32
  GEMM_128_K2 = 17,   // 128x128x64, 2 groups of 8 wavefronts, each group half of the K steps
  GEMM_64X128_K2 = 18, // 64x128x64, 2 groups of 8 wavefronts
  GEMM_64_K4 = 19,    // 64x64x64, 4 groups of 4 wavefronts (3 when B is K x N), each group its share of the K steps
  GEMM_128_PP16 = 20, // 128x128x64, 8 wavefronts (2x4) of 64x32, two-group schedule, direct-to-LDS loads, two workgroups per CU
  GEMM_128_PP16_K128 = 21, // the same tile with K steps of 128 (one workgroup per CU, phases of twice the length)
  GEMM_256X128_KP = 22, // 256x128x64, two groups of 4 wavefronts (2x2) of 128x64 on alternate K steps, direct-to-LDS loads
  GEMM_128_KP = 23,   // 128x128x64, the same with 64x64 per wavefront
  GEMM_224X128_KP = 24, // 256x128 with 112, 96 or 80 rows per wavefront instead of 128
  GEMM_192X128_KP = 25,
  GEMM_160X128_KP = 26,
  GEMM_NUM_VARIANTS
};

struct GemmArgs {
  int64_t M, N, K;
  const uint16_t* A; int64_t lda;
  const uint16_t* B; int64_t ldb; int transB;
  uint16_t* C; int64_t ldc;
  int dtype;
  int forced;  // GemmVariant or GEMM_AUTO
  int acc32;   // 0: C is 16-bit and overwritten; 1: C is fp32 and accumulated into (C += A*B)
  const uint16_t* bias = nullptr;  // N elements of the input type added to every row (16-bit C only), or null
  int act = 0;                     // 0 none, 1 relu, 2 gelu: applied after the bias (16-bit C only)
  // K split across workgroups: the fp32 scratch the partial products go to (parts * M * N floats)
  // and the number of parts the plan asks for; run_gemm fills both in.
  float* scratch = nullptr;
  uint32_t* counters = nullptr;    // the scratch's kScratchCounters zeros (left as zeros), or null: a second kernel adds the parts
  int parts = 1;
  int forced_parts = 0;            // plan_gemm: 0 = the cost model's choice, 1 / 2 / 4 / 8 = forced
  // A result of 8 MB up to the 32 MB of the L2s, in rows of whole 128-byte lines, leaves in the non-temporal form. Plain, its lines stay dirty in
  // the L2s and are written back behind the kernel's end (the same bytes cross the L2 boundary either way). What counts is the call and the one
  // that reads C next (bf16, us, plain / non-temporal: the call; with a product of N x 1024 behind it; with C + R, element by element, behind it):
  //   4 MB,   1024 x 2048 x 1024    9.4 / 9.5      19.9 / 20.7    13.2 / 13.3     lines that the next call had still found in a cache
  //   6.4 MB,  777 x 4096 x 4096   36.6 / 35.8     68.0 / 71.3 *  41.2 / 40.9     (* N x 4096)
  //   12 MB,  6144 x 1024 x 1024   18.5 / 15.4     37.4 / 34.4    26.5 / 26.0
  //   16 MB,  4096 x 2048 x 1024   22.3 / 19.7     47.2 / 44.7    31.9 / 31.4
  //   24 MB,  3072 x 4096 x 3072   69.0 / 66.1    103.6 / 101.9   81.3 / 80.0
  //   32 MB,  2048 x 8192 x 4096   98.8 / 99.1    139.4 / 141.9  113.4 / 115.1
  //   64 MB,  4096 x 8192 x 2048  108.3 / 106.0   212.2 / 223.2  133.5 / 140.7    the last-level cache does not keep it
  //   128 MB, 8192 x 8192 x 1024  124.7 / 115.8   233.9 / 240.6  187.3 / 191.3
  // Rows that share lines lose: 7000 x 7000 x 1024 114 / 121, 14336 x 3000 x 512 61 / 67. An fp32 C that is accumulated
  // into gains nothing (4096 x 4096 x 2048 73.7 / 74.1) and may still be in the last-level cache (3072 x 912 x 416 11.6 / 13.8).
  bool stream_c() const {
    const int64_t bytes = M * N * 2;
    return !acc32 && bytes >= 8 << 20 && bytes < 32 << 20 && (reinterpret_cast<uintptr_t>(C) & 127) == 0 && ldc % 64 == 0;
  }
  int epi() const { return (acc32 ? 1 : act << 1) | (stream_c() ? 16 : 0); }   // the kernels' epilogue word
  bool fused() const { return bias != nullptr || act != 0; }
};

struct GemmPlan {
  int variant = GEMM_GENERAL;
  bool aligned = true;             // false: the forms of the tile kernels for operands of any alignment
  int parts = 1;                   // > 1: K split across workgroups, partial products through a scratch
  int64_t scratch_bytes = 0;       // parts * M * N * 4 when parts > 1
  const char* name = "";
  const char* suffix = "";         // of the reported name: a tile with fewer rows than the kernel's name says
  int bm = 0, bn = 0, bk = 0, wm = 0, wn = 0;
  int mfma_m = 32, mfma_n = 32, mfma_k = 16;
};

// mlt_gemm_noalloc: bytes of the fixed device array that takes the partial products of a K split
// across workgroups (no plan the library makes by itself needs more), and that
// array's address on the current device (nullptr if it cannot be had)
constexpr int64_t kStaticScratchBytes = (int64_t)32 << 20;
float* static_scratch_of_current_device();
// Counters (last_to_arrive in mlt_common.h) in front of every buffer that cached_scratch returns. The fixed array has none: calls
// that overlap there, against the rules, would leave them in disorder for all later ones.
constexpr int kScratchCounters = 16384;
inline uint32_t* scratch_counters(float* scratch) { return reinterpret_cast<uint32_t*>(scratch) - kScratchCounters; }

GemmPlan plan_gemm(const GemmArgs& g);
int run_gemm(const GemmArgs& g, GemmPlan& p, hipStream_t s);
bool gemm_pp_ok(const GemmArgs& g);            // gemm_pp.hip: can the two-group kernel take this problem?
int run_gemm_pp(const GemmArgs& g, int tile, int kstep, hipStream_t s);   // tile: 256 or 128; K step 64 or (tile 128 only) 128
int run_gemm_kp(const GemmArgs& g, int bm, hipStream_t s);   // gemm_kp.hip (where gemm_pp_ok): bm x 128, bm 256, 224, 192, 160 or 128; g.parts > 1: K split across workgroups
int run_splitk_reduce(const GemmArgs& g, int parts, int64_t part_stride, hipStream_t s);   // gemm.hip: the sum of the parts, with the epilogue
bool gemm_any_ok(const GemmArgs& g);           // gemm_any.hip: the tile kernels on operands of any alignment
int run_gemm_any(const GemmArgs& g, int variant, hipStream_t s);
bool gemm_w4_ok(const GemmArgs& g);            // gemm_w4.hip: whole K steps only
int run_gemm_w4(const GemmArgs& g, hipStream_t s);
bool gemm_skinny_ok(const GemmArgs& g);        // gemm_skinny.hip
// its columns per block: 16, or without a K split across workgroups the 4 or 8 that a CU has of a narrow matrix
inline int gemm_skinny_cols(int64_t N, int64_t parts, int64_t ncu) { return parts > 1 || N > 8 * ncu ? 16 : N > 4 * ncu ? 8 : 4; }
int run_gemm_skinny(const GemmArgs& g, hipStream_t s);

enum MhaVariant {
  MHA_AUTO = -1,
  MHA_PP32 = 0,   // two-group kernel, 32x32x16 MFMAs, one workgroup per (batch*head, query tile)
  MHA_PP16 = 1,   // the same on 16x16x32 MFMAs
  MHA_PS = 2,     // persistent form of the two-group kernel (unmasked, D = 128, at least two key tiles)
  MHA_K2 = 3,     // 128 query rows per workgroup, the keys split over two groups of wavefronts
  MHA_K4 = 4,     // 64 query rows per workgroup, the keys split over four groups
  MHA_NUM_VARIANTS
};

struct MhaArgs {
  int64_t B, H, Sq, Sk, D;
  const uint16_t *Q, *K, *V;
  uint16_t* O;
  float scale;
  int causal, dtype;
  int forced = MHA_AUTO;   // MhaVariant or MHA_AUTO
  int ps_grid = 0;         // persistent kernel: number of workgroups (0: one per CU)
  int forced_split = 0;    // MHA_K2 / MHA_K4: ranges of keys per item, from mlt_diag_force_key_split (0: automatic)
};

struct MhaPlan {
  const char* name = "";
  int bm = 0, bn = 0, waves = 0;
  bool supported = false;
  int mfma_size = 32;       // 32 = 32x32x16 MFMAs, 16 = 16x16x32
  bool persistent = false;  // one workgroup per CU walking through the items
  int key_groups = 1;       // > 1: the kernels of mha_ks.hip, bm = 256 / key_groups
  int nsplit = 1;           // > 1: their keys are split over that many workgroups as well, partial results through a scratch
};
bool mha_pp_ok(const MhaArgs& a);
int run_mha_pp(const MhaArgs& a, int mfma_size, hipStream_t s);
// mha_ks.hip; bm: 64 or 128 query rows per workgroup; nsplit > 1: scratch holds mha_ks_scratch_bytes
int run_mha_ks(const MhaArgs& a, int bm, int nsplit, float* scratch, hipStream_t s);
inline int64_t mha_ks_scratch_bytes(const MhaArgs& a, int nsplit) { return nsplit * a.B * a.H * a.Sq * (a.D + 2) * 4; }
bool mha_ps_ok(const MhaArgs& a);              // mha_pp.hip: can the persistent kernel take this problem?
int run_mha_ps(const MhaArgs& a, hipStream_t s);

// Process-wide overrides of the automatic kernel choice, for tuning and for the tests that must
// reach every kernel (mlt_diag_force_variant; initial values from MLT_GEMM_VARIANT /
// MLT_MHA_VARIANT / MLT_MHA_PS_GRID, read once).
struct Overrides { int gemm = GEMM_AUTO; int gemm_parts = 0; int mha = MHA_AUTO; int ps_grid = 0; int key_split = 0; };
Overrides& overrides();
// Device facts the launchers need, cached per thread for the current device.
struct DeviceInfo { int ncu = 0; int nxcd = 0; bool gfx950 = false; };
bool device_info(DeviceInfo& out);
// XCDs of the current device (hipDeviceAttributeNumberOfXccs; 8, the MI355X's, if it cannot be
// read). Only the workgroup -> tile maps use it: a wrong value costs L2 hits, never correctness.
int device_xcds();

// probe.hip: launches the register-only MFMA loop, returns the flop it will execute (< 0: launch failed)
double run_mfma_probe(int iters, int nblocks, const void* data, float* sink, int mfma_size, hipStream_t s);
int run_hbm_read_probe(const void* data, int64_t bytes, uint32_t* sink, int ncu, hipStream_t s);

MhaPlan plan_mha(const MhaArgs& a);
int run_mha(const MhaArgs& a, MhaPlan& p, hipStream_t s);

struct PagedArgs {
  int64_t B, H, D, block_size, max_blocks, num_blocks;
  const uint16_t *Q, *Kc, *Vc;
  const int32_t *block_table, *seq_lens;
  uint16_t* O;
  float scale;
  int dtype;
  int forced_split = 0;      // > 0: ranges of keys per (sequence, head), from mlt_diag_force_key_split
};
// Pieces of a paged decode dealt out by length: workgroup `id` of `total`, which the hardware puts on CU id % ncu (all are
// resident at once), takes the piece of this rank. Every second round of CUs runs backwards, the last full one among them.
__host__ __device__ inline int dealt_piece(int id, int total, int ncu) {
  const int round = id / ncu, full = total / ncu;
  return round < full && ((full - round) & 1) ? round * ncu + (ncu - 1 - (id - round * ncu)) : id;
}
// paged.hip; *nsplit_out: the number of key ranges per (sequence, head) that ran
int run_paged_decode(const PagedArgs& a, hipStream_t s, int* nsplit_out);
int plan_paged_split(const PagedArgs& a);                                       // key ranges per (sequence, head)
bool paged_by_length(const PagedArgs& a, int64_t nsplit, int64_t ncu);   // workgroups dealt out by sequence length?

// The library's own scratch memory for a stream of the current device: at least `bytes`, behind its counters, kept
// (and grown by doubling) from call to call, never freed; nullptr if it cannot be had, and while the
// stream records into a graph. Work of one stream that uses it is ordered by the stream.
float* cached_scratch(int64_t bytes, hipStream_t s);
bool stream_is_capturing(hipStream_t s);   // true while `s` records into a graph

}  // namespace mlt
