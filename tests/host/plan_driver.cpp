// Prints what the library's planning functions choose, without a device (they then assume 256 CUs, 8
// XCDs). One problem per line on stdin, one answer per line on stdout:
//   gemm M N K transB lda ldb fp32_accumulate fused noncontiguous_base   ->  name parts scratch_bytes
// (fused: 1 bias, 2 and ReLU, 3 and GELU; noncontiguous_base != 0: A starts on an odd element; "hint1", "hint2" instead of "gemm": with that tiling hint)
//   tile (as gemm)   ->  the same with the rows and columns of its workgroup tile in front
//   store M N ldc C fp32_accumulate   ->  1 if the result leaves in the non-temporal form
//   mha B H Sq Sk D causal   ->  name ranges
//   paged B H D block_size max_blocks   ->  ranges dealt_by_length ("paged_split": and a forced number of ranges)
//   xcdword workgroups causal D mfma_size   ->  what an attention launch passes as its XCD count
//   masked workgroups query_tiles Sq D   ->  head:tile of each workgroup of a masked attention launch
//   deal pieces CUs   ->  the rank of the piece that each workgroup takes
#include <stdio.h>
#include <string.h>

#include "../../paper_2503_14985_amd/csrc/mha_tile.h"

using namespace mlt;

int main() {
  char op[16];
  while (scanf("%15s", op) == 1) {
    if (!strcmp(op, "gemm") || !strcmp(op, "tile") || !strcmp(op, "hint1") || !strcmp(op, "hint2")) {
      long long M, N, K, lda, ldb;
      int tb, acc, fused, odd, forced = GEMM_AUTO;
      if (scanf("%lld %lld %lld %d %lld %lld %d %d %d", &M, &N, &K, &tb, &lda, &ldb, &acc, &fused, &odd) != 9) return 1;
      GemmArgs g{};
      g.M = M; g.N = N; g.K = K;
      g.A = (const uint16_t*)(0x100000 + (odd ? 2 : 0)); g.lda = lda;
      g.B = (const uint16_t*)0x200000; g.ldb = ldb; g.transB = tb;
      g.C = (uint16_t*)0x300000; g.ldc = N;
      if (!strcmp(op, "hint1")) forced = GEMM_256_W8X1;
      if (!strcmp(op, "hint2")) forced = GEMM_256_W1X8;
      g.forced = forced; g.acc32 = acc;
      if (fused) g.bias = (const uint16_t*)0x400000;
      g.act = fused > 1 ? fused - 1 : 0;
      const GemmPlan p = plan_gemm(g);
      if (!strcmp(op, "tile")) printf("%d %d ", p.bm, p.bn);
      printf("%s %d %lld\n", p.name, p.parts, (long long)p.scratch_bytes);
    } else if (!strcmp(op, "store")) {
      long long M, N, ldc, C;
      int acc;
      if (scanf("%lld %lld %lld %lld %d", &M, &N, &ldc, &C, &acc) != 5) return 1;
      GemmArgs g{};
      g.M = M; g.N = N; g.K = 1024; g.C = (uint16_t*)(uintptr_t)C; g.ldc = ldc; g.acc32 = acc;
      printf("%d\n", g.epi() & 16 ? 1 : 0);
    } else if (!strcmp(op, "mha")) {
      long long B, H, Sq, Sk, D;
      int causal;
      if (scanf("%lld %lld %lld %lld %lld %d", &B, &H, &Sq, &Sk, &D, &causal) != 6) return 1;
      MhaArgs a{};
      a.B = B; a.H = H; a.Sq = Sq; a.Sk = Sk; a.D = D;
      a.scale = 1.f; a.causal = causal;
      a.forced = MHA_AUTO;
      const MhaPlan p = plan_mha(a);
      printf("%s %d\n", p.name, p.nsplit);
    } else if (!strcmp(op, "paged") || !strcmp(op, "paged_split")) {
      long long B, H, D, block_size, max_blocks;
      if (scanf("%lld %lld %lld %lld %lld", &B, &H, &D, &block_size, &max_blocks) != 5) return 1;
      PagedArgs a{};
      a.B = B; a.H = H; a.D = D; a.block_size = block_size; a.max_blocks = max_blocks; a.num_blocks = B * max_blocks;
      if (op[5] == '_') scanf("%d", &a.forced_split);
      const int n = plan_paged_split(a);
      printf("%d %d\n", n, paged_by_length(a, n, 256) ? 1 : 0);
    } else if (!strcmp(op, "xcdword")) {
      int total, causal, D, mfma;
      if (scanf("%d %d %d %d", &total, &causal, &D, &mfma) != 4) return 1;
      DeviceInfo di;
      di.ncu = 256; di.nxcd = 8; di.gfx950 = true;
      printf("%d\n", mha_xcd_word(total, causal != 0, D, mfma, di));
    } else if (!strcmp(op, "masked")) {
      int total, nq, Sq, D;
      if (scanf("%d %d %d %d", &total, &nq, &Sq, &D) != 4) return 1;
      DeviceInfo di;
      di.ncu = 256; di.nxcd = 8; di.gfx950 = true;
      const int word = mha_xcd_word(total, true, D, 32, di);
      const MaskedMap m = masked_map(total, nq, Sq, 256, true, D, word, di);
      if (m.chunk <= 0) printf("plain");
      for (int b = 0; b < total && m.chunk > 0; ++b) {
        int bh, qt;
        block_map_masked(b, nq, word, m, bh, qt);
        printf("%d:%d ", bh, qt);
      }
      printf("\n");
    } else if (!strcmp(op, "deal")) {
      int total, ncu;
      if (scanf("%d %d", &total, &ncu) != 2) return 1;
      for (int id = 0; id < total; ++id) printf("%d ", dealt_piece(id, total, ncu));
      printf("\n");
    } else {
      return 1;
    }
  }
  return 0;
}
