// GEMM on operands of any alignment: odd K, N or leading dimensions, bases on any element. The same
// tile kernels as gemm.hip, whose 16-byte global accesses then need 2-byte alignment only and whose
// chunks at the end of a row are shifted into place (gemm_tile.h). What an
// unaligned access costs is small: 1999 x 3008 x 1536 (aligned) takes 33 us on the 128 x 128 tile, 1999 x
// 3002 x 1502 (rows on 4-byte boundaries) 34 us, 1999 x 3001 x 1501 (2-byte boundaries) 35-39 us. With
// element-wise loads (2 bytes per lane and instruction, no pipelining) the last one took 416 us.
// Bound by the LDS side of a K step (its stores, its fragment reads, the barrier), not by the loads.
#include "gemm_tile.h"

namespace mlt {

// K >= 8 (and N >= 8 with B stored K x N), so that a 16-byte access fits every row it reads.
bool gemm_any_ok(const GemmArgs& g) { return g.K >= 8 && (g.transB || g.N >= 8); }

int run_gemm_any(const GemmArgs& g, int variant, hipStream_t s) {
  const int rc = g.dtype == MLT_BF16 ? launch_small_tile<bf16_tag, false>(g, variant, s) : launch_small_tile<f16_tag, false>(g, variant, s);
  return rc == -1 ? MLT_ERR_UNSUPPORTED : rc;
}

}  // namespace mlt
