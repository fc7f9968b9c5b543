// Pieces shared by the attention-forward kernels for gfx950 (mha_pp.hip, mha_ks.hip): tile sizes,
// the direct global->LDS load, lane-pair exchanges, the workgroup->item map and the LDS layout of
// a K/V tile (paper: arXiv 2503.14985, Section 2.5, Algorithm 1 and Table 5).
#pragma once

#include "mlt_common.h"
#include "mlt_internal.h"

namespace mlt {

constexpr int PA_BM = 256;    // query rows per workgroup
constexpr int PA_BN = 64;     // keys per tile
constexpr int PA_NT = 512;
constexpr int PA_NS = 5;      // LDS ring slots (two-group kernels)
constexpr int PA_AHEAD = 3;   // tiles fetched ahead of the softmax phase that issues the fetch
constexpr float PA_LAZY_T = 8.f;   // log2 units a row maximum may grow before the reference point moves

// max / sum of a per-lane value with the one held by lane l ^ 32 (the other half of the keys of
// the same query): permlane32_swap fed the same register twice returns both halves' values.
__device__ __forceinline__ float both_halves_max(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float both_halves_sum(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
// O^T accumulators -> 16-byte pieces of O rows. A lane holds, of its query row, 4 consecutive d
// per register group g (d = 32t + 8g + 4h + 0..3, h = lane / 32): 8-byte pieces, which the lane
// with the other h interleaves. Swapping group g+1 of the lower lanes with group g of the upper
// ones (permlane32_swap, per packed register) leaves the lower lane with d = 32t + 8g + 0..7 and
// the upper lane with the next 8: one 16-byte store each instead of two 8-byte ones, and 32
// contiguous bytes per row and store instruction.
template <typename Tag>
__device__ __forceinline__ u32x4 o_piece16(const f32x16& acc, int g, float inv) {
  const uint32_t a0 = Elem<Tag>::pack2(acc[4 * g] * inv, acc[4 * g + 1] * inv);
  const uint32_t a1 = Elem<Tag>::pack2(acc[4 * g + 2] * inv, acc[4 * g + 3] * inv);
  const uint32_t b0 = Elem<Tag>::pack2(acc[4 * g + 4] * inv, acc[4 * g + 5] * inv);
  const uint32_t b1 = Elem<Tag>::pack2(acc[4 * g + 6] * inv, acc[4 * g + 7] * inv);
  auto s0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
  auto s1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
  return u32x4{(uint32_t)s0[0], (uint32_t)s1[0], (uint32_t)s0[1], (uint32_t)s1[1]};
}

__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_fmaxf(__builtin_fmaxf(a, b), c);       // v_max3_f32
}

// Workgroup id -> (batch*head, query tile): every XCD owns a contiguous range of the items, and
// the query tiles of one head are walked last tile first (with the causal mask it has the most
// work). All tiles of a head share one XCD's L2.
__device__ __forceinline__ void block_map(int bid, int total, int nq, int nxcd, int& bh, int& qt) {
  const int logical = logical_block(bid, total, nxcd);
  bh = logical / nq;
  qt = nq - 1 - logical % nq;
}

// The same for the masked problem, whose last query tiles take longest. An XCD's items, in the order above, are cut into chunks,
// and a chunk's are taken longest first, the last tiles of all its heads, then the tiles before them, and so on: the launch ends
// with short items, where whole heads, one after the other, left long items that started late to run alone (us, heads one by one / chunks, D = 128:
// 32 x 16 x 1024 242 / 201, 3 x 16 x 1693 58 / 48, 31 x 8 x 945 112 / 98; D = 64: 32 x 32 x 1024 258 / 227, 10 x 16 x 1778 100 / 91).
// cus (CUs per XCD, in bits 8 and up of nxcd_cus; 0 for other launches): all items are resident at once, one or two per CU, and
// the XCD's items i and i + cus share a CU. The longest that have to share one do so with the shortest, and those
// that do not are the longest of all (D = 64, 8 x 32 heads, 512 x 512: 24.2 -> 21.8 us).
struct MaskedMap {
  int per, rem;                 // items per XCD, and how many XCDs have one more
  int chunk;                    // 0: plain order (block_map)
  float r_nxcd, r_chunk, r_nq;  // reciprocals of the divisors
};
// a / b for 0 <= a < 2^20 (an integer division takes the start of a workgroup 0.1 us)
__host__ __device__ inline int small_div(int a, int b, float r) {
  int q = (int)((float)a * r);
  q -= q * b > a ? 1 : 0;
  return q + (a - q * b >= b ? 1 : 0);
}
__host__ __device__ inline void block_map_masked(int bid, int nq, int nxcd_cus, const MaskedMap& m, int& bh, int& qt) {
  const int nxcd = nxcd_cus & 255, cus = nxcd_cus >> 8;
  int k = small_div(bid, nxcd, m.r_nxcd);
  const int xcd = bid - k * nxcd;
  int first = xcd * m.per + (xcd < m.rem ? xcd : m.rem), n = m.per + (xcd < m.rem ? 1 : 0);
  if (cus > 0 && n >= cus && n <= 2 * cus) {
    const int two = n - cus;                               // CUs with two items
    k = k >= cus ? n - 1 - (k - cus) : k < two ? cus - two + k : k - two;
  } else {
    const int skip = small_div(k, m.chunk, m.r_chunk) * m.chunk;
    k -= skip;
    first += skip;
    n = n - skip < m.chunk ? n - skip : m.chunk;
  }
  // the k-th of the items first .. first + n - 1 by falling tile. Item i is tile nq - 1 - j, j = i % nq, of head i / nq: `rows` or
  // rows + 1 items of every j, one more of the n % nq values from j0 on (modulo nq)
  const int rows = small_div(n, nq, m.r_nq), more = n - rows * nq, h0 = small_div(first, nq, m.r_nq), j0 = first - h0 * nq;
  const int wrap = j0 + more - nq;
  auto before = [&](int j) {                               // items with a smaller j
    const int ext = wrap <= 0 ? (j - j0 < 0 ? 0 : j - j0 < more ? j - j0 : more) : (j < wrap ? j : wrap) + (j > j0 ? j - j0 : 0);
    return j * rows + ext;
  };
  int j = small_div(k, rows + 1, 1.f / (float)(rows + 1));     // (every j before the right one has at most rows + 1 items, ...
  if (rows > 0 && k > more) {                             // ... and all but `more` of them only `rows`)
    const int j1 = small_div(k - more, rows, 1.f / (float)rows);
    j = j1 > j ? j1 : j;
  }
  while (before(j + 1) <= k) ++j;
  bh = h0 + (j < j0 ? 1 : 0) + (k - before(j));
  qt = nq - 1 - j;
}
// Chunks of one launch's worth of resident workgroups for D = 128 and short sequences (their K and V are the 4 MB of an XCD's L2), of
// two otherwise (us, chunks of one / two / four: D = 128, 32 x 16 x 1024 201 / 204 / 221, 16 x 16 x 2048 313 / 322 / 325, 8 x 16 x 4096 543 /
// 537 / 550, 4 x 16 x 8192 1018 / 991 / 984; D = 64, 32 x 32 x 1024 231 / 227 / 231, 4 x 32 x 8192 1229 / 1171 / 1176; only the last two
// launches' worth sorted, the rest head by head: 235, 345 and 253 us for the three that begin with 32 and 16).
// The plain order stays where all items, or all but the shorter ones of the last head, are resident at once and not paired, where
// an XCD has no two heads, for launches too large for small_div, and for two or three tiles of which the last is at most half full: half of its workgroup's
// wavefronts have nothing to do, so the order of the tiles is not that of their lengths (11 x 16 x 640 44.8 us head by head, 52 sorted;
// 31 x 32 x 540, D = 64, 114, 118).
inline MaskedMap masked_map(int total, int nq, int Sq, int bm, bool causal, int D, int nxcd_cus, const DeviceInfo& di) {
  MaskedMap m{0, 0, 0, 0.f, 0.f, 0.f};
  const int nxcd = nxcd_cus & 255, ncu = di.ncu > 0 ? di.ncu : 256, per = total / nxcd, n = per + (total % nxcd ? 1 : 0);
  const int slots = ncu / nxcd * (D == 64 ? 2 : 1);
  if (!causal || nq < 2 || total >= 1 << 20 || slots < 1) return m;
  if (nxcd_cus < 256 && (8 * (n - slots) <= 5 * nq || n < 2 * nq || (nq <= 3 && 2 * (Sq - (nq - 1) * bm) <= bm))) return m;
  const int least = slots * (D == 128 && nq <= 8 ? 1 : 2), chunks = n >= least ? n / least : 1;
  m.per = per; m.rem = total % nxcd; m.chunk = (n + chunks - 1) / chunks;
  m.r_nxcd = 1.f / (float)nxcd; m.r_chunk = 1.f / (float)m.chunk; m.r_nq = 1.f / (float)nq;
  return m;
}
inline MaskedMap masked_map(int total, int nq, int Sq, int bm, bool causal, int D, int nxcd_cus) {
  DeviceInfo di;
  (void)device_info(di);
  return masked_map(total, nq, Sq, bm, causal, D, nxcd_cus, di);
}
// what a launch of `total` workgroups adds to the XCD count for that map
inline int paired_cus(int total, bool causal, int D, const DeviceInfo& di) {
  if (D != 64 || !causal || di.ncu <= 0 || di.nxcd <= 0) return 0;
  return total > di.ncu && total <= 2 * di.ncu ? di.ncu / di.nxcd << 8 : 0;
}
// The XCD word of a launch: their count, and for the kernels that decode it (all but the one on 16x16x32 MFMAs,
// which uses the plain map) the CUs for pairs.
inline int mha_xcd_word(int total, bool causal, int D, int mfma_size, const DeviceInfo& di) {
  return (di.nxcd > 0 ? di.nxcd : 8) + (mfma_size == 32 ? paired_cus(total, causal, D, di) : 0);
}
inline int mha_xcd_word(int total, bool causal, int D, int mfma_size) {
  DeviceInfo di;
  (void)device_info(di);
  return mha_xcd_word(total, causal, D, mfma_size, di);
}

template <int D> struct PaCfg {
  static constexpr int ROWB = D * 2;               // bytes per key row
  static constexpr int TILE_B = PA_BN * ROWB;      // one K or V tile
  static constexpr int SLOT_B = 2 * TILE_B;        // K tile then V tile
  static constexpr int SMEM = PA_NS * SLOT_B;      // 160 KB (D = 128) / 80 KB (D = 64)
  static constexpr int CPR = D / 8;                // 16-byte chunks per row
  static constexpr int RPB = 64 / CPR;             // rows per 1 KB block (one wavefront load)
  static constexpr int NBLK = PA_BN / RPB;         // blocks per tile
  static constexpr int LPW = NBLK / 8;             // loads per wavefront per tile and matrix
  static constexpr int NKK = D / 16;               // k slices of S^T = K Q^T
  static constexpr int NDT = D / 32;               // 32-row tiles of O^T
  // Swizzles. K rows are read 16 at a time at one chunk position (ds_read_b128), V rows 4 at a
  // time over 4 adjacent chunks (ds_read_b64_tr_b16); each must cover 16 distinct bank groups.
  static __device__ __forceinline__ int fk(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
  static __device__ __forceinline__ int fv(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }
};

}  // namespace mlt
