// Paged attention for decoding (arXiv 2503.14985, Section 3.2) for gfx950: one query per
// (sequence, head) over that sequence's keys and values, which live in fixed-size blocks of a cache
// and are found through a per-sequence block table.
//
// The paper's point about this kernel is its warp distribution: with a single query row there is
// nothing to split along the rows, so the KEYS are split over the warps of a workgroup, every warp
// runs the FlashAttention recurrence on its own cache blocks, and the partial maxima, sums and
// outputs are reduced across warps through shared local memory to one warp that stores the
// result (Listing 6). The same decomposition here, one level finer: a workgroup of 4 wavefronts
// owns one (sequence, head); the keys are cut into units of 16, wavefront w takes units w, w+4,
// ...; inside a wavefront each group of D/8 lanes owns one key row of a load (4 rows per 1 KB
// load for D = 128, 8 for D = 64) and keeps its OWN running maximum, sum and output slice, so
// nothing is exchanged between lanes except the D/8-lane sum of a dot product. All partial
// results (16 or 32 per workgroup) meet once, in LDS, at the end.
//
// With fewer (sequence, head) pairs than the chip needs workgroups, the same split goes one level
// up as well: the units of a sequence are cut into `nsplit` contiguous ranges, one workgroup per
// (sequence, head, range); each leaves its maximum, sum and unnormalised output slice (fp32) in a
// scratch buffer. Up to 8 ranges of a short launch are merged by the workgroup of the pair that comes last at a
// counter, more of them by a second small kernel, in the same fixed order, the way a workgroup merges its own
// partial results.
//
// The operation is bound by reading the cache once from HBM (2 * seq_len * D * 2 bytes per
// sequence and head), so there is no MFMA here (a 1-row product would waste it) and no LDS staging:
// 16-byte loads go straight to registers, one unit ahead of the arithmetic. Products use the
// packed dot instructions (v_dot2_f32_bf16 / v_dot2_f32_f16): q.k as four of them per lane and key,
// p.v as one per output element with the weight, rounded to the 16-bit type as in Listing 5's
// p.to(float16), in one half of the second operand.
#include "mlt_common.h"
#include "mlt_internal.h"

namespace mlt {

namespace {

constexpr int PG_NW = 4;            // wavefronts per workgroup
constexpr int PG_NT = PG_NW * 64;
constexpr int PG_UNIT = 16;         // keys per unit

// sum over the 16 (or 8) lanes that share a key row; every lane of the group gets the total
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, false));  // row_half_mirror
  if (LPR == 16)
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, false));  // row_mirror
  return x;
}

template <typename Tag> struct Dot2;
template <> struct Dot2<bf16_tag> {
  static __device__ __forceinline__ float f(uint32_t a, uint32_t b, float c) {
    typedef __attribute__((ext_vector_type(2))) __bf16 v2;
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2, a), __builtin_bit_cast(v2, b), c, false);
  }
};
template <> struct Dot2<f16_tag> {
  static __device__ __forceinline__ float f(uint32_t a, uint32_t b, float c) {
    typedef __attribute__((ext_vector_type(2))) _Float16 v2;
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(v2, a), __builtin_bit_cast(v2, b), c, false);
  }
};

// The sequence that comes `rank`-th when a batch is ordered by length, longest first (equal lengths: by
// index). B <= PG_NT; buf: PG_NT + 1 ints of LDS. Contains workgroup barriers; afterwards buf is free.
__device__ __forceinline__ int sequence_of_rank(const int32_t* seq_lens, int B, int rank, int* buf) {
  const int tid = threadIdx.x;
  const int mine = tid < B ? seq_lens[tid] : -0x7fffffff - 1;
  buf[tid] = mine;
  __syncthreads();
  if (tid < B) {
    int before = 0;
    for (int j = 0; j < B; ++j) {
      const int other = buf[j];
      before += other > mine || (other == mine && j < tid) ? 1 : 0;
    }
    if (before == rank) buf[PG_NT] = tid;
  }
  __syncthreads();
  const int b = __builtin_amdgcn_readfirstlane(buf[PG_NT]);
  __syncthreads();
  return b;
}

// O of one pair from its `nsplit` (at most MAXS) ranges at p, by all NT threads of a workgroup: group g of D threads adds the ranges
// g, g + 4, ... and the four sums meet in LDS in the order 0, 1, 2, 3. A sequence has at least one key, so range 0 is never
// empty and the maximum is finite. All of a thread's loads are requested at once: this is the memory round trips
// that it waits for (as a kernel of its own: a plain loop over 32 ranges 16 us, eight loads in flight 3.9; 64 ranges so 4.5).
// SHARED: the ranges come from workgroups of the same launch.
constexpr int PG_MAX_SPLIT = 64;
constexpr int PG_LAST_SPLIT = 8;    // ranges that the last of their workgroups merges, at most
template <typename Tag, int D, int MAXS, int NT, bool SHARED>
__device__ __forceinline__ void merge_ranges(const float* p, uint16_t* __restrict__ out, int nsplit, float* buf) {
  constexpr int NR = MAXS / 4, NG = 4 * D / NT;           // ranges of a group; groups of a thread
  float *sm = buf, *sl = sm + MAXS, *acc4 = sl + MAXS, *l4 = acc4 + 4 * D;
  const int tid = threadIdx.x, g0 = tid / D * NG, d = tid % D;
  auto get = [&](int i) __attribute__((always_inline)) { return SHARED ? load_shared(p + i) : p[i]; };
  float v[NG][NR];
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int n = 0; n < NG; ++n) v[n][i] = g0 + n + 4 * i < nsplit ? get((g0 + n + 4 * i) * (2 + D) + 2 + d) : 0.f;
  if (tid < MAXS) {
    sm[tid] = tid < nsplit ? get(tid * (2 + D)) : -__builtin_inff();
    sl[tid] = tid < nsplit ? get(tid * (2 + D) + 1) : 0.f;
  }
  __syncthreads();
  float M = sm[0];
#pragma unroll
  for (int s = 1; s < MAXS; ++s) M = __builtin_fmaxf(M, sm[s]);
#pragma unroll
  for (int n = 0; n < NG; ++n) {
    const int g = g0 + n;
    float acc = 0.f, L = 0.f;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const float wgt = __builtin_amdgcn_exp2f(sm[g + 4 * i] - M);         // empty ranges: exp2(-inf) = 0
      acc += v[n][i] * wgt;
      L += sl[g + 4 * i] * wgt;
    }
    acc4[g * D + d] = acc;
    if (d == 0) l4[g] = L;
  }
  __syncthreads();
  if (tid < D) out[d] = Elem<Tag>::from_f32((acc4[d] + acc4[D + d] + acc4[2 * D + d] + acc4[3 * D + d]) / (l4[0] + l4[1] + l4[2] + l4[3]));
}
// floats of LDS that it needs
constexpr int merge_floats(int maxs, int D) { return 2 * maxs + 4 * D + 4; }

// Which workgroup takes which sequence: hardware deals the workgroups of a launch to the CUs in turn, all of
// them at once up to 8 per CU, and with the batch in its own order the CUs' shares of keys differ by
// chance. A batch of 2 to PG_NT sequences with more workgroups than CUs is therefore dealt from the
// longest sequence to the shortest, every second round of CUs backwards, the last full one among them: an odd
// number of rounds leaves the first CUs with the shorter sequences, and they get what is over (27 x 32 of at most 9344
// keys, D = 64: 226 us with the first round forwards, 213 so, 212 in batch order). 64 sequences of 1024 to 4096
// keys, 32 heads, D = 128, shuffled: 456 -> 421 us (6.4 TB/s, as for equal lengths).
//
// SPLIT: blockIdx.y is the range of units this workgroup takes, and the result goes to `part`
// ([pair][range][2 + D] floats: maximum (log2 domain), sum, unnormalised outputs) instead of O; counters: a zero for each
// pair (left as zero), at which the last of its workgroups finds out that it is to merge them, or null: another kernel does.
// ORDER: by length, see above (ncu, B: only then).
template <typename Tag, int D, bool SPLIT, bool ORDER>
__global__ __launch_bounds__(PG_NT) void paged_decode_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ Kc,
    const uint16_t* __restrict__ Vc, const int32_t* __restrict__ block_table,
    const int32_t* __restrict__ seq_lens, uint16_t* __restrict__ O, float* part, uint32_t* __restrict__ counters, int H,
    int block_size, int max_blocks, int num_blocks, int B, int ncu, float c) {
  constexpr int LPR = D / 8;                 // lanes per key row (16 bytes each)
  constexpr int RPI = 64 / LPR;              // key rows per load instruction
  constexpr int NL = PG_UNIT / RPI;          // loads per unit and matrix
  constexpr int NSPLIT = PG_NW * RPI;        // partial results per workgroup
  __shared__ float sm[NSPLIT], sl[NSPLIT];
  __shared__ float so[NSPLIT][D];                        // (the rank search borrows it)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rgrp = lane / LPR, chunk = lane % LPR;
  const int nsplit = SPLIT ? (int)gridDim.y : 1;
  // which sequence, head and range
  int b, h, range = 0;
  if (ORDER) {
    const int pieces = H * nsplit, total = B * pieces;
    int id = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    id = dealt_piece(id, total, ncu);
    b = sequence_of_rank(seq_lens, B, id / pieces, reinterpret_cast<int*>(&so[0][0]));
    h = id % pieces / nsplit;
    range = id % nsplit;
  } else {
    b = blockIdx.x / H;
    h = blockIdx.x % H;
    if (SPLIT) range = blockIdx.y;
  }
  const int bh = b * H + h;

  int len = seq_lens[b];
  const int cap = max_blocks * block_size;
  len = len < 1 ? 1 : (len > cap ? cap : len);           // never trust it further than the table
  const int all_units = (len + PG_UNIT - 1) / PG_UNIT;
  const int upb = block_size / PG_UNIT;                  // units per cache block
  // the units this workgroup takes: all of them, or its range of a cut into gridDim.y ranges of
  // equal length (a multiple of the wavefront count; the last ranges of a short sequence are empty)
  int u_begin = 0, nunits = all_units;
  if (SPLIT) {
    const int per = ((all_units + nsplit - 1) / nsplit + PG_NW - 1) / PG_NW * PG_NW;
    u_begin = range * per;
    nunits = u_begin + per < all_units ? u_begin + per : all_units;
  }

  // this lane's 8 query elements, as packed pairs
  const u32x4 qv = *reinterpret_cast<const u32x4_mem*>(Q + (int64_t)bh * D + chunk * 8);

  // first element of unit u in the cache (block number clamped: a bad table entry may give a
  // wrong answer but never an access outside the cache)
  auto unit_base = [&](int u) -> int64_t {
    int pb = block_table[(int64_t)b * max_blocks + u / upb];
    pb = pb < 0 ? 0 : (pb >= num_blocks ? num_blocks - 1 : pb);
    return (((int64_t)pb * H + h) * block_size + (u % upb) * PG_UNIT) * D;
  };
  const int lane_off = rgrp * D + chunk * 8;             // + i * RPI * D for load i
  auto load_unit = [&](int u, u32x4 (&kf)[NL], u32x4 (&vf)[NL]) {
    const int64_t base = unit_base(u) + lane_off;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      kf[i] = load_stream16(Kc + base + i * RPI * D);     // the cache is read once: streaming loads
      vf[i] = load_stream16(Vc + base + i * RPI * D);
    }
  };

  float m = -__builtin_inff(), l = 0.f;                  // this row group's running maximum (log2 domain) and sum
  float o[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = 0.f;

  u32x4 kf[2][NL], vf[2][NL];
  if (u_begin + wave < nunits) load_unit(u_begin + wave, kf[0], vf[0]);
  int cur = 0;
  for (int u = u_begin + wave; u < nunits; u += PG_NW) {
    if (u + PG_NW < nunits) {
      if (cur == 0) load_unit(u + PG_NW, kf[1], vf[1]); else load_unit(u + PG_NW, kf[0], vf[0]);
    }
    // scores of this lane's keys of the unit: key position u*16 + i*RPI + rgrp
    float x[NL];
    float mx = m;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const u32x4 k = cur == 0 ? kf[0][i] : kf[1][i];
      float s = Dot2<Tag>::f(qv[0], k[0], 0.f);
      s = Dot2<Tag>::f(qv[1], k[1], s);
      s = Dot2<Tag>::f(qv[2], k[2], s);
      s = Dot2<Tag>::f(qv[3], k[3], s);
      s = row_sum<LPR>(s);
      const int p = u * PG_UNIT + i * RPI + rgrp;
      x[i] = p < len ? s * c : -__builtin_inff();
      mx = __builtin_fmaxf(mx, x[i]);
    }
    if (mx != -__builtin_inff()) {                        // else: nothing visible yet in this group
      const float alpha = __builtin_amdgcn_exp2f(m - mx);  // m = -inf gives 0
      l *= alpha;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] *= alpha;
      m = mx;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const float pw = __builtin_amdgcn_exp2f(x[i] - m);       // exp2(-inf) = 0 for masked keys
        const uint32_t pb16 = Elem<Tag>::from_f32(pw);           // weight rounded to the 16-bit type
        l += Elem<Tag>::to_f32((uint16_t)pb16);
        const uint32_t plo = pb16, phi = pb16 << 16;
        u32x4 v = cur == 0 ? vf[0][i] : vf[1][i];
        // slots past seq_len may hold anything (also NaN, and 0 * NaN is NaN): take zeros instead
        if (u * PG_UNIT + i * RPI + rgrp >= len) v = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          o[2 * w] = Dot2<Tag>::f(v[w], plo, o[2 * w]);           // low element of the pair times p
          o[2 * w + 1] = Dot2<Tag>::f(v[w], phi, o[2 * w + 1]);   // high element times p
        }
      }
    }
    cur ^= 1;
  }

  // ---- all partial results meet in LDS; D threads combine them
  const int sidx = wave * RPI + rgrp;
  if (chunk == 0) { sm[sidx] = m; sl[sidx] = l; }
#pragma unroll
  for (int e = 0; e < 8; ++e) so[sidx][chunk * 8 + e] = o[e];
  __syncthreads();
  if (tid < D) {
    float M = sm[0];
#pragma unroll
    for (int s = 1; s < NSPLIT; ++s) M = __builtin_fmaxf(M, sm[s]);
    // a range past the end of a short sequence saw no key at all: its sum and outputs are zeros
    // (the weights below must not become exp2(-inf - -inf))
    const float Mref = SPLIT && M == -__builtin_inff() ? 0.f : M;
    float L = 0.f, acc = 0.f;
#pragma unroll
    for (int s = 0; s < NSPLIT; ++s) {
      const float wgt = __builtin_amdgcn_exp2f(sm[s] - Mref);    // empty groups: exp2(-inf) = 0
      L += sl[s] * wgt;
      acc += so[s][tid] * wgt;
    }
    if (SPLIT) {
      float* out = part + ((int64_t)bh * nsplit + range) * (2 + D);
      if (!ORDER && counters) {
        if (tid == 0) { store_shared(out, M); store_shared(out + 1, L); }
        store_shared(out + 2 + tid, acc);
      } else {
        if (tid == 0) { out[0] = M; out[1] = L; }
        out[2 + tid] = acc;
      }
    } else {
      O[(int64_t)bh * D + tid] = Elem<Tag>::from_f32(acc / L);
    }
  }
  if (!SPLIT || ORDER || !counters) return;
  static_assert(merge_floats(PG_LAST_SPLIT, D) <= NSPLIT * D, "the merge works in so");
  if (!last_to_arrive(counters + bh, (uint32_t)nsplit, reinterpret_cast<uint32_t*>(sm))) return;
  merge_ranges<Tag, D, PG_LAST_SPLIT, PG_NT, true>(part + (int64_t)bh * nsplit * (2 + D), O + (int64_t)bh * D, nsplit, &so[0][0]);
}

// The merge as a kernel of its own, one workgroup per (sequence, head)
template <typename Tag, int D, int MAXS>
__global__ __launch_bounds__(4 * D) void paged_merge_kernel(const float* __restrict__ part,
                                                            uint16_t* __restrict__ O, int nsplit) {
  __shared__ float buf[merge_floats(MAXS, D)];
  const int64_t bh = blockIdx.x;
  merge_ranges<Tag, D, MAXS, 4 * D, false>(part + bh * nsplit * (2 + D), O + bh * D, nsplit, buf);
}

template <typename Tag, int D>
int launch_paged(const PagedArgs& a, int nsplit, float* part, hipStream_t s) {
  const float c = a.scale * 1.4426950408889634f;
  const unsigned pairs = (unsigned)(a.B * a.H);
  DeviceInfo di;
  const int64_t ncu = device_info(di) ? di.ncu : 0;
  const bool order = paged_by_length(a, nsplit, ncu);
  // Up to 8 ranges, and not by length: the last workgroup of a pair merges them, which saves the second launch (us, second
  // kernel / last workgroup: 1 x 8 pairs of 700 keys, D = 64, 4 ranges 7.8 / 6.0; 4 x 32 of 1024, D = 128, 4 ranges 14.5 / 13.9; 16 x 16 of 600, D = 64,
  // 2 ranges 11.8 / 11.1; 4 x 16 of 5440 in 8 equal). Its three trips to memory, one after the other (the written values, the counter, all the
  // ranges), cost as much as the launch with more ranges or where the CUs are still busy with other pieces (1 x 8, 32768 in
  // 64: 27.1 / 29.1; 1 x 32, 4096 in 32: 15.6 / 18.0; by length: 8 x 16, 32768 in 16 206 / 222, 10 x 32, 4096 in 6 67.9 / 71.0).
  uint32_t* counters = nsplit > 1 && nsplit <= PG_LAST_SPLIT && !order && pairs <= (unsigned)kScratchCounters ? scratch_counters(part) : nullptr;
  auto kern = nsplit > 1 ? (order ? paged_decode_kernel<Tag, D, true, true> : paged_decode_kernel<Tag, D, true, false>)
                         : (order ? paged_decode_kernel<Tag, D, false, true> : paged_decode_kernel<Tag, D, false, false>);
  hipLaunchKernelGGL(kern, dim3(pairs, nsplit > 1 ? (unsigned)nsplit : 1u), dim3(PG_NT), 0, s, a.Q, a.Kc, a.Vc,
                     a.block_table, a.seq_lens, a.O, nsplit > 1 ? part : (float*)nullptr, counters, (int)a.H, (int)a.block_size,
                     (int)a.max_blocks, (int)a.num_blocks, (int)a.B, (int)ncu, c);
  if (hipGetLastError() != hipSuccess) return MLT_ERR_LAUNCH;
  if (nsplit <= 1 || counters) return MLT_OK;
  auto merge = nsplit <= 8 ? paged_merge_kernel<Tag, D, 8> : nsplit <= 32 ? paged_merge_kernel<Tag, D, 32>
                                                                          : paged_merge_kernel<Tag, D, PG_MAX_SPLIT>;
  hipLaunchKernelGGL(merge, dim3(pairs), dim3(4 * D), 0, s, part, a.O, nsplit);
  return hipGetLastError() == hipSuccess ? MLT_OK : MLT_ERR_LAUNCH;
}

}  // namespace

// Whether a launch deals its workgroups by length. The rank search costs 1 to 2 us in front of the first load, so not for
// caches that are read in less than 30 us, 25 us in smaller pieces (17 x 32 pairs of at most 800 keys 26.9 us in batch order, 29.3 by length; 167 x 4
// of 1280, D = 64: 30, 32.6; 38 x 32 of 181: 16.1, 17.1). And every workgroup reads all
// B lengths, 25 ps for each on the whole chip. That has to stay below what the order gains: 0.5 to 0.6 of the reading over the
// workgroups per CU, nothing on short sequences. us in batch order / by length: 228 x 16 pairs of at most 256 keys, D = 128:
// 51 / 72; 76 x 16 of 400: 29 / 31; 206 x 16 of 544, D = 64: 49 / 61; 254 x 1 of 3456 in 6 ranges, D = 128: 54 / 60; but
// 246 x 4 of 1088, D = 128: 71 / 63; 208 x 4 of 608: 36 / 34; 230 x 8 of 2416, D = 64: 131 / 123.
bool paged_by_length(const PagedArgs& a, int64_t nsplit, int64_t ncu) {
  const int64_t wgs = a.B * a.H * nsplit, keys = a.max_blocks * a.block_size;
  if (ncu <= 0 || a.B < 2 || a.B > PG_NT || wgs <= ncu || keys < 512) return false;
  return a.B * a.H * keys * a.D * 4 >= ((int64_t)(nsplit > 1 ? 192 : 224) << 20) && wgs * nsplit * a.B * 10 < keys * a.D * 32;
}

// Ranges per (sequence, head), at most 64. Up to one workgroup per CU from the pairs alone: what brings the
// launch to two per CU, as long as a range of the longest possible sequence (the table's width) keeps 16
// units (256 keys); twice that for one sequence whose ranges are short anyway, down to 8 units
// (1 x 32 pairs, 4096 keys: 15.0 us with 16 ranges, 13.7 with 32). A batch, whose sequences differ in
// length, is cut finer, up to 8 pieces per CU and 32 units, also beyond one pair per CU: the pieces are dealt out by
// length, and the more there are the closer the CUs' shares come (us, lengths s/4 .. s, D = 128: 10 x 32, s = 4096:
// 102 uncut, 71 in 6 ranges; 8 x 16, 32768: 238 in 4, 208 in 16; 16 x 32, 4096: 118 uncut, 111 in 4; equal lengths
// 121 / 112, 335 / 331, 168 / 173). From three pairs per CU on the second kernel costs as much as that gains
// (24 x 32, 2048: 83.8 uncut, 86.3 in 2), from two and a half on for caches below 448 MiB (22 x 32, 2176, D = 64: 45.5, 47.4;
// but 83 x 8, 2816: 64, 56), and so it does where the cache is read in less than 20 us, or for a quarter more
// ranges and less (14 x 4, 5920: 26 in 10, 29 in 11; 4 x 16, 5440: 27 in 8, 28.7 in 10). Nor do the ranges of one sequence get finer from 32 units (D = 64: 64)
// on (1 x 32, 14848 keys: 42.8 in 16, 45.2 in 32; 7680 keys equal; D = 64, 12672 keys: 22.8, 21.5).
int plan_paged_split(const PagedArgs& a) {
  if (a.forced_split > 0) return a.forced_split > PG_MAX_SPLIT ? PG_MAX_SPLIT : a.forced_split;
  DeviceInfo di;
  const int64_t ncu = device_info(di) ? di.ncu : 256;
  const int64_t pairs = a.B * a.H;
  const int64_t max_units = (a.max_blocks * a.block_size + PG_UNIT - 1) / PG_UNIT;
  int64_t n = 1;
  if (pairs <= ncu) {
    n = (2 * ncu + pairs - 1) / pairs;
    if (n > max_units / 16) n = max_units / 16;
    if (a.B == 1 && n > 1 && max_units * a.D <= 4096 * n && max_units >= 16 * n) n *= 2;
  }
  const int64_t mib = pairs * max_units * PG_UNIT * a.D * 4 >> 20;
  const bool long_read = pairs <= ncu || mib >= (2 * pairs <= 5 * ncu ? 128 : 448);
  if (a.B > 1 && a.B <= PG_NT && pairs < 3 * ncu && long_read) {
    int64_t fine = 8 * ncu / pairs;
    if (fine > max_units / 32) fine = max_units / 32;
    if (4 * fine > 5 * n) n = fine;
  }
  if (n > PG_MAX_SPLIT) n = PG_MAX_SPLIT;
  return n < 1 ? 1 : (int)n;
}

int run_paged_decode(const PagedArgs& a, hipStream_t s, int* nsplit_out) {
  int nsplit = plan_paged_split(a);
  float* part = nullptr;
  if (nsplit > 1) {
    part = cached_scratch(a.B * a.H * nsplit * (2 + a.D) * (int64_t)sizeof(float), s);
    if (!part) nsplit = 1;                               // no scratch to be had: the plain form
  }
  if (nsplit_out) *nsplit_out = nsplit;
  if (a.dtype == MLT_BF16)
    return a.D == 128 ? launch_paged<bf16_tag, 128>(a, nsplit, part, s) : launch_paged<bf16_tag, 64>(a, nsplit, part, s);
  return a.D == 128 ? launch_paged<f16_tag, 128>(a, nsplit, part, s) : launch_paged<f16_tag, 64>(a, nsplit, part, s);
}

}  // namespace mlt
