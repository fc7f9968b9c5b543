// Attention forward: choice of the kernel for a problem (the kernels are in mha_pp.hip and mha_ks.hip).
//
// All of them follow the FlashAttention-2 forward of the paper (arXiv 2503.14985, Section 2.5,
// Algorithm 1) with the row-only partition of its warpsPerCTA = [numWarps, 1]: workgroup =
// 8 wavefronts x 32 query rows of one (batch, head), key tile 64; with few query rows for the chip, fewer
// rows and the keys split over groups of wavefronts.
#include <cmath>

#include "mha_tile.h"
#include "mlt_internal.h"

namespace mlt {

// 256 query rows per workgroup (mha_pp.hip) or 128 / 64 with the keys split over 2 / 4 groups of
// wavefronts (mha_ks.hip): the one with the least estimated time over the whole grid, ties within 5 % to
// the larger tile (it reads K and V from L2 less often). ns per 32 keys of a step and per workgroup, from
// fits over 40 problems of 1 to 256 heads, 1 to 2048 queries and 64 to 4096 keys; D = 64 puts two
// workgroups on a CU, which slow each other down and hide each other's start and end. Measured (bf16, us,
// 256 / 128 / 64 rows): 2 x 16 heads, 333 x 1501, D = 128: 36.3 / 29.7 / 20.3; 8 x 32, 100 x 1000: 34.7 / 29.4 /
// 32.4; 4 x 16, 600 x 2000: 51.9 / 73.2 / 69.3; 1 x 16, 2048 causal: 46.4 / 37.7 / 31.8; D = 64, 1 x 32, 333 x 1501:
// 28.8 / 22.8 / 15.0; 2 x 32, 1024: 22.8 / 26.6 / 29.7.
static void plan_key_groups(const MhaArgs& a, MhaPlan& p) {
  if (a.forced == MHA_K2 || a.forced == MHA_K4) {
    p.key_groups = a.forced == MHA_K4 ? 4 : 2;
    p.nsplit = a.forced_split > 0 ? (a.forced_split > 64 ? 64 : a.forced_split) : 1;
    return;
  }
  const int64_t heads = a.B * a.H;
  if (a.forced != MHA_AUTO || heads < 1 || a.Sq < 1) return;
  // with the mask the last query row sees min(Sq, Sk) keys (17 x 8 heads, 65 x 1994 causal, D = 128, priced with all
  // 1994: 64 rows, 11.8 us; 256 rows take 8.0)
  const int64_t keys = a.causal && a.Sq < a.Sk ? a.Sq : a.Sk, tiles = (keys + 31) / 32;
  // one key tile of the 256-row kernel and few workgroups: nothing to divide
  if (tiles <= 2 && heads * ((a.Sq + 255) / 256) <= 64) return;
  DeviceInfo di;
  const int64_t ncu = device_info(di) && di.ncu > 0 ? di.ncu : 256, nxcd = di.nxcd > 0 ? di.nxcd : 8;
  const bool one_round_of_256 = heads * ((a.Sq + 255) / 256) <= ncu;
  if (heads * ((a.Sq + 255) / 256) > 4 * ncu) return;             // enough of the large tiles
  const double arrive = (double)heads * (a.Sq + keys) * a.D * 4 / 5500;   // every tensor once at 5.5 TB/s
  auto cost = [&](int groups, int nsplit) -> int64_t {
    const int64_t bm = 256 / groups, nq = (a.Sq + bm - 1) / bm, wgs = heads * nq * nsplit;
    const int64_t t_step = a.D == 128 ? (groups == 1 ? 550 : groups == 2 ? 800 : 780) : (groups == 1 ? 525 : groups == 2 ? 650 : 700);
    const int64_t steps = (tiles + groups * nsplit - 1) / (groups * nsplit), longest = steps * t_step;
    // with the mask a workgroup sees its share of the keys only; the longest start first, or share their CU
    // with a short one (block_map_masked)
    const int64_t avg = a.causal && a.Sk >= a.Sq ? longest * (nq + 1) / (2 * nq) : longest;
    const int64_t rounds = (wgs + ncu - 1) / ncu;
    // start and end of a workgroup in a launch of several rounds: 256 rows of which more than half are not there cost as much
    // as if they were (928 heads, us, 256 / 128 rows: D = 128, 9 x 41 25 / 20, 68 x 68 causal 37 / 30, but 1024 heads, 128 x 128 44 / 47;
    // D = 64, 9 x 41 causal 13.0 / 8.5)
    const int64_t ends = groups > 1 && a.Sq <= 96 ? 5000 : 7000;
    int64_t t;
    if (rounds <= 1) t = longest + 7000;
    else if (a.D == 128) t = a.causal ? wgs * (avg * 5 / 4) / ncu + rounds * ends : rounds * (longest + ends);
    else if (a.causal) t = wgs * (rounds > 2 ? avg * 5 / 4 : avg) / ncu + (rounds + 1) / 2 * (ends - 1000) + 4000;
    else t = rounds * (avg + 3000) + 4000;
    if (t < longest + 7000) t = longest + 7000;
    // Masked items in a second, partly filled round of 128-row tiles, where the 256-row kernel needs one round. The term was fitted to
    // workgroups that went through the heads one by one, so that a long item could start behind another one; the figures are those of the order
    // of today, longest first (block_map_masked), in which the two share little. us, 64 / 128 / 256 rows: D = 128, 15 heads x
    // 3566 87 / 102 / 77, 9 x 5585 124 / 145 / 115, but 24 x 1290 26 / 27 / 32, 32 x 1055 28 / 23 / 28 and 24 x 2029 48 / 40 / 46; D = 64, 24 x 1394 18 / 22 / 27, 8 x
    // 4647 41 / 61 / 78, 16 x 2688 31 / 37 / 47, but 56 x 671 15 / 13 / 17, 48 x 1110 20 / 19 / 24. Over 260 such problems the choice is 4 % (D = 128) and
    // 14 % (D = 64) behind the best one; without the term 5 and 9 %, but half as long again at worst, where 64 rows are right.
    if (a.causal && groups == 2 && rounds == 2 && one_round_of_256 && (a.D == 128 || wgs < 2 * ncu)) {
      const int64_t extra = (wgs - ncu + nxcd - 1) / nxcd;
      if (heads % nxcd != 0 || (a.D == 128 && 4 * extra >= 3 * nq)) t += longest / 2;
      else if (a.D == 64) t += longest * (extra < nq ? extra : nq) * 7 / (10 * nq);
    }
    t = (int64_t)std::sqrt((double)t * t + arrive * arrive);       // the two overlap in part
    // the partial results' second kernel: a launch, and writing and reading them at 4 TB/s
    if (nsplit > 1) t += 3500 + 2 * nsplit * heads * a.Sq * (a.D + 2) / 1000;
    return t;
  };
  int64_t best = cost(1, 1);
  for (int groups = 2; groups <= 4; groups *= 2) {
    const int64_t t = cost(groups, 1);
    if (t + t / 20 < best) { best = t; p.key_groups = groups; }
  }
  // Few workgroups against many keys: the keys split over workgroups as well, as long as all of them fit one
  // round and a range keeps 4 steps (1 x 8 heads, 1 x 4096, D = 128: 37 us, 16 in four ranges; 3 x 16, 2 x 2831, D = 64:
  // 21.5 us, 11.8 in four ranges; 4 x 32, 1 x 4096: the operands' arrival takes as long either way, 40.6 against 44).
  if (p.key_groups != 4 || a.causal) return;
  const int64_t w64 = heads * ((a.Sq + 63) / 64);
  for (int n = 2; n <= 16; ++n) {
    if (w64 * n > ncu || tiles < 4 * 4 * n) break;
    const int64_t t = cost(4, n);
    if (t + t / 20 < best) { best = t; p.nsplit = n; }
  }
}

MhaPlan plan_mha(const MhaArgs& a) {
  MhaPlan p;
  // Sk * D * 2 has to fit the 32-bit per-lane byte offsets of the direct global->LDS loads
  if ((a.D != 64 && a.D != 128) || !mha_pp_ok(a)) return p;
  p.supported = true;
  p.bm = PA_BM; p.bn = PA_BN; p.waves = PA_NT / 64;
  // Default: 32x32x16 MFMAs. Measured for D = 128: the 16x16x32 form is 3 % faster in back-to-back
  // launches but 2 % slower when it alternates with the GEMM; for D = 64 it does not fit the 128
  // registers that let two workgroups share a CU (-6 %).
  p.mfma_size = a.forced == MHA_PP16 ? 16 : 32;
  // The persistent form runs only on request. Measured, unmasked, 2048 items, time per item
  // against the per-item kernel: D = 128 gains 25 % at 2 key tiles per item, 8 % at 4, 3 % at 8
  // and loses 1.5 % at 16, 3 % at 32 and 4 % at 64 (its loop carries the item bookkeeping). It is
  // not the automatic choice even for short sequences: it fetches the next item's Q operand with
  // loads the compiler cannot see into registers the compiler manages, which holds for the
  // compiler this library is built with (the build's own check of the generated code and the
  // parity tests say so) but is not a property of the source. D = 64 has no persistent form
  // (mha_ps_ok). Where the forced form cannot run, the default kernel does.
  p.persistent = a.forced == MHA_PS && mha_ps_ok(a);
  plan_key_groups(a, p);
  if (p.key_groups > 1) {
    static const char* const names[2][2][2] = {
        {{"mha_fwd_d64_128x32_k2_pp", "mha_fwd_d64_causal_128x32_k2_pp"}, {"mha_fwd_d64_64x32_k4_pp", "mha_fwd_d64_causal_64x32_k4_pp"}},
        {{"mha_fwd_d128_128x32_k2_pp", "mha_fwd_d128_causal_128x32_k2_pp"}, {"mha_fwd_d128_64x32_k4_pp", "mha_fwd_d128_causal_64x32_k4_pp"}}};
    p.bm = PA_BM / p.key_groups;
    p.waves = PA_NT / 64 / p.key_groups;                          // along the rows
    p.bn = 32;
    p.mfma_size = 32;
    p.name = names[a.D == 128][p.key_groups == 4][a.causal ? 1 : 0];
  } else if (p.persistent) {
    p.mfma_size = 32;
    p.name = "mha_fwd_d128_256x64_ps";
  } else if (p.mfma_size == 16) {
    if (a.D == 128) p.name = a.causal ? "mha_fwd_d128_causal_256x64_pp16" : "mha_fwd_d128_256x64_pp16";
    else p.name = a.causal ? "mha_fwd_d64_causal_256x64_pp16" : "mha_fwd_d64_256x64_pp16";
  } else {
    if (a.D == 128) p.name = a.causal ? "mha_fwd_d128_causal_256x64_pp" : "mha_fwd_d128_256x64_pp";
    else p.name = a.causal ? "mha_fwd_d64_causal_256x64_pp" : "mha_fwd_d64_256x64_pp";
  }
  return p;
}

int run_mha(const MhaArgs& a, MhaPlan& p, hipStream_t s) {
  if (!p.supported) return MLT_ERR_UNSUPPORTED;
  if (p.key_groups > 1) {
    float* scratch = nullptr;
    if (p.nsplit > 1) {
      scratch = cached_scratch(mha_ks_scratch_bytes(a, p.nsplit), s);
      if (!scratch) p.nsplit = 1;
    }
    return run_mha_ks(a, p.bm, p.nsplit, scratch, s);
  }
  if (p.persistent) return run_mha_ps(a, s);
  return run_mha_pp(a, p.mfma_size, s);
}

}  // namespace mlt
