"""The library's choice of kernels and splits, asked on the host (tests/host/plan_driver.cpp calls the
planning functions; no kernel runs and no device is needed)."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LIB_DIR = os.path.join(ROOT, "paper_2503_14985_amd")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    cmd = [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-x", "hip", os.path.join(ROOT, "tests", "host", "plan_driver.cpp"),
           "-x", "none", "-o", exe, os.path.join(LIB_DIR, "libmlt.so"), "-Wl,-rpath," + LIB_DIR]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    env = {k: v for k, v in os.environ.items() if not k.startswith("MLT_")}

    def ask(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=600, env=env)
        assert r.returncode == 0, r.stderr[-2000:]
        out = r.stdout.strip().split("\n")
        assert len(out) == len(lines)
        return out
    return ask


def gemm_line(M, N, K, transB, lda=None, ldb=None, acc=0, fused=0, odd=0):
    return "gemm %d %d %d %d %d %d %d %d %d" % (M, N, K, transB, lda or K, ldb or (K if transB else N), acc, fused, odd)


def test_no_split_of_its_own_needs_more_than_the_fixed_scratch(plan):
    """mlt_gemm_noalloc has 32 MiB for the partial products of a K split and refuses what needs more:
    no split that the library chooses by itself may, whatever the operands' alignment."""
    cases = [(2056, 2056, 8193, 0), (67, 16714, 9761, 1), (2100, 2100, 16001, 0), (2111, 2111, 8191, 1),
             (3001, 3001, 16385, 1), (3967, 4383, 24204, 0)]
    rng = random.Random(3)
    for _ in range(20000):
        size = lambda lo, hi: int(lo * (hi / lo) ** rng.random())
        cases.append((size(1, 6000), size(8, 30000), size(64, 60000), rng.randint(0, 1)))
    lines, shapes = [], []
    for i, (M, N, K, tb) in enumerate(cases):
        if i % 3 == 2:                                      # aligned operands
            N, K = N // 8 * 8, K // 8 * 8
        lines.append(gemm_line(M, N, K, tb, acc=i % 5 == 0, odd=i % 3 == 1))
        shapes.append((M, N, K, tb))
    split = 0
    for shape, ans in zip(shapes, plan(lines)):
        name, parts, scratch = ans.split()
        split += int(parts) > 1
        assert int(scratch) <= 32 << 20, (shape, ans)
        assert int(scratch) == (int(parts) * shape[0] * shape[1] * 4 if int(parts) > 1 else 0)
    assert split > 500                                       # the question was asked of real splits


@pytest.mark.parametrize("M,N,K,transB,acc,fused", [(1094, 13928, 72, 0, 0, 1), (2936, 5560, 144, 1, 0, 1), (417, 11424, 336, 0, 0, 1),
                                                    (5117, 1240, 176, 0, 1, 0), (2314, 2728, 176, 1, 1, 0), (7029, 1088, 224, 0, 0, 0)])
def test_a_short_ragged_k_takes_many_small_tiles(plan, M, N, K, transB, acc, fused):
    """Fewer than 8 K steps, the last one partial: 100 to 300 large tiles took up to 1.5 times as long."""
    assert "_128x128x64_w2x4" in plan([gemm_line(M, N, K, transB, acc=acc, fused=fused)])[0].split()[0]


@pytest.mark.parametrize("M,N,K,transB", [(2057, 608, 3200, 0), (241, 6680, 4096, 1), (245, 4368, 4456, 0), (352, 3176, 5632, 1), (2509, 704, 6744, 0),
                                          (460, 2648, 4224, 0)])
def test_few_tiles_are_not_left_to_the_two_k_groups_alone(plan, M, N, K, transB):
    """40 to 110 tiles of 128 x 128: without a split across workgroups the kernels with two groups on alternate K steps
    take up to 1.45 times as long as the best other one."""
    name, parts, _ = plan([gemm_line(M, N, K, transB)])[0].split()
    assert "kp2" not in name or int(parts) > 1


@pytest.mark.parametrize("D", [64, 128])
def test_causal_attention_is_priced_by_the_keys_it_sees(plan, D):
    """Keys past the last query row are masked for all rows: their number changes nothing in the choice."""
    for B, H, Sq in ((17, 8, 65), (4, 40, 67), (1, 32, 121), (1, 16, 600), (8, 32, 200)):
        assert len(set(plan(["mha %d %d %d %d %d 1" % (B, H, Sq, Sk, D) for Sk in (Sq, 2 * Sq, 1994, 30000)]))) == 1
    name = "mha_fwd_d%d_causal_256x64_pp 1" % D
    assert plan(["mha 17 8 65 1994 %d 1" % D, "mha 4 8 41 41 %d 1" % D]) == [name, name]


def test_masked_attention_avoids_a_partly_filled_second_round(plan):
    """128-row tiles that just overflow the chip, with heads that do not divide over the XCDs, start long items late."""
    ans = plan(["mha 1 %d %d %d %d 1" % c for c in ((12, 3403, 3403, 128), (22, 1574, 1574, 128), (29, 1809, 3928, 64), (40, 998, 998, 64),
                                                           (24, 1536, 1536, 128), (16, 2202, 2202, 64))])
    assert ["128x32_k2" in a for a in ans] == [False, False, False, False, True, True], ans
    # few rows of many heads, several rounds: 128-row tiles, whose workgroups start and end sooner
    assert ["128x32_k2" in a for a in plan(["mha 232 4 9 41 %d 1" % d for d in (64, 128)])] == [True, True]


def test_paged_decode_searches_ranks_only_where_the_lengths_are_few_for_the_keys(plan):
    """Every workgroup reads all B lengths: many short sequences took up to 1.4 times as long by length as in batch order."""
    ask = lambda cases: [a.split()[1] for a in plan(["paged %d %d %d %d %d" % c for c in cases])]
    assert ask([(228, 16, 128, 16, 16), (206, 16, 64, 32, 17), (76, 16, 128, 16, 25), (38, 32, 128, 16, 12), (300, 8, 128, 16, 256)]) == ["0"] * 5
    assert ask([(64, 32, 128, 16, 256), (246, 4, 128, 64, 17), (230, 8, 64, 16, 151), (10, 32, 128, 16, 256)]) == ["1"] * 4


def test_pieces_dealt_by_length_leave_the_remainder_to_the_cus_with_less(plan):
    """Piece lengths that fall evenly with the rank to a quarter; the hardware deals workgroup i to CU i % 256. Bounds: the
    most loaded CU over the mean, with the last full round backwards (forwards: 1.85, 1.55, 1.30, 1.18, 1.16 and 1.09
    for the first six)."""
    for total, bound in ((300, 1.37), (400, 1.07), (511, 1.01), (816, 1.07), (864, 1.06), (1000, 1.01), (512, 1.001), (2048, 1.001)):
        ranks = [int(x) for x in plan(["deal %d 256" % total])[0].split()]
        assert sorted(ranks) == list(range(total))
        load = [0.0] * 256
        for i, r in enumerate(ranks):
            load[i % 256] += 1.0 - 0.75 * r / total
        assert max(load) <= bound * sum(load) / 256, total


def test_paged_decode_is_cut_finer_only_where_that_gains(plan):
    ask = lambda cases: [int(a.split()[0]) for a in plan(["paged %d %d %d %d %d" % c for c in cases])]
    # one range, or the ranges that bring the launch to two workgroups per CU
    assert ask([(64, 32, 128, 16, 256), (24, 32, 128, 16, 128), (22, 32, 64, 16, 136), (14, 4, 128, 32, 185), (1, 32, 128, 64, 232)]) == [1, 1, 1, 10, 16]
    # finer
    assert ask([(1, 8, 128, 16, 2048), (1, 32, 128, 16, 256), (10, 32, 128, 16, 256), (8, 16, 128, 16, 2048), (20, 32, 128, 16, 128), (23, 32, 64, 64, 128),
                (6, 32, 64, 64, 36)]) == [64, 32, 6, 16, 3, 2, 4]


def test_routing_of_decode_gemms(plan):
    """Up to 64 rows against B stored N x K: B is streamed, with K over several workgroups where their few columns stand against
    a long K."""
    ask = lambda M, N, K, fused=0: plan([gemm_line(M, N, K, 1, fused=fused)])[0].rsplit(" ", 1)[0]
    for c in ((17, 6456, 5544), (24, 14336, 4096), (24, 14336, 4096, 1), (24, 4096, 2880), (16, 3584, 2048), (1, 4096, 2880), (1, 3072, 4096),
              (1, 1024, 8192), (1, 5120, 5120, 1), (1, 4096, 4096), (16, 4096, 4096), (30, 4096, 2048), (2, 3592, 4096), (40, 16384, 4096),
              (64, 28672, 4096), (64, 4096, 512), (48, 4096, 4096), (49, 4104, 4096), (64, 4096, 4032)):
        assert ask(*c) == "gemm_nt_skinny_stream 1", c
    for c, parts in (((17, 5120, 8192), 4), ((15, 1656, 11200, 1), 4), ((32, 2048, 8192), 4), ((24, 1024, 11200), 8), ((16, 1024, 28672), 8),
                     ((16, 1024, 28672, 1), 8), ((1, 1024, 28672, 1), 8), ((32, 1024, 28672), 8), ((50, 4800, 12608), 4)):
        assert ask(*c) == "gemm_nt_skinny_stream %d" % parts, c


@pytest.mark.parametrize("stream,tiles", [
    # up to 32 rows: columns per CU, row tiles, steps of 64 k (and a fused activation) against each other
    ((1, 4096, 64), (1, 4104, 64)), ((16, 8192, 128), (16, 8200, 128)), ((16, 8192, 72), (16, 8200, 72)), ((32, 4096, 128), (32, 4104, 128)),
    ((17, 2048, 64), (17, 2056, 64)), ((16, 60000, 264), (16, 60000, 256)), ((32, 14336, 448), (32, 14344, 448)), ((32, 30000, 456), (32, 30000, 448)), ((24, 8192, 128, 1), (24, 8200, 128, 1)),
    # 33 rows and more: 8 steps
    ((33, 4096, 456), (33, 4096, 448)), ((64, 4096, 512), (64, 5512, 72)),
    # 49 rows and more, at most 16 columns per CU, 64 to 255 steps
    ((48, 4096, 4096), (49, 4096, 4096)), ((64, 4104, 4096), (64, 4096, 4096)), ((64, 4096, 4032), (64, 1024, 16320)), ((64, 1024, 28608), (64, 1024, 16320)),
    # 64 x 128 tiles that fill three quarters of one or two rounds; one, in four or eight parts
    ((52, 24448, 1856), (52, 31704, 1856)), ((42, 33888, 1024), (64, 52736, 576)), ((41, 5592, 3520), (55, 6904, 6784)), ((37, 2928, 9664), (45, 3456, 9984)),
    ((45, 3456, 9992), (45, 3456, 9984)), ((38, 7664, 4032), (38, 7664, 4608)),
    # 64 x 64 tiles, in eight parts or few steps: five eighths of one round, four fifths of several
    ((34, 1112, 9984), (51, 1808, 20736)), ((60, 9216, 512), (60, 13016, 512)), ((60, 13016, 520), (60, 13016, 512)), ((42, 12448, 5632), (42, 12448, 2496)),
    ((42, 12448, 1024, 1), (42, 12448, 640, 1)), ((44, 28384, 1280), (44, 28384, 1216)), ((44, 24160, 1216), (44, 28384, 1216)), ((44, 28384, 640, 1), (44, 12448, 640, 1))])
def test_where_the_tile_kernels_take_over_from_the_streaming_kernel(plan, stream, tiles):
    ask = lambda M, N, K, fused=0: plan([gemm_line(M, N, K, 1, fused=fused)])[0]
    assert ask(*stream).startswith("gemm_nt_skinny_stream"), stream
    assert ask(*tiles).startswith("gemm_nt_64x"), (tiles, ask(*tiles))


def test_a_tiling_hint_on_unaligned_operands_is_the_automatic_choice(plan):
    for M, N, K, tb in ((1439, 333, 113, 0), (9, 18, 200, 0), (926, 10, 77, 1), (1999, 3001, 1501, 0), (64, 65, 3, 1)):
        line = gemm_line(M, N, K, tb)
        auto, h1, h2 = plan([line, line.replace("gemm", "hint1"), line.replace("gemm", "hint2")])
        assert auto == h1 == h2, (M, N, K, tb)
    assert "_w8x1" in plan([gemm_line(520, 776, 320, 0).replace("gemm", "hint1")])[0]


def test_only_kernels_that_decode_it_get_the_paired_maps_word(plan):
    """The masked D = 64 launches of 1 to 2 workgroups per CU carry the CUs per XCD above the XCD count; the kernel on 16x16x32
    MFMAs takes the word for the plain count."""
    ask = lambda *c: int(plan(["xcdword %d %d %d %d" % c])[0])
    assert [ask(t, 1, 64, 32) for t in (256, 257, 512, 513)] == [8, 8 + (32 << 8), 8 + (32 << 8), 8]
    assert [ask(t, 1, 64, 16) for t in (256, 257, 512, 513)] == [8] * 4
    assert ask(300, 0, 64, 32) == ask(300, 1, 128, 32) == 8


def test_the_batches_of_the_order_test_are_dealt_by_length(plan):
    from test_paged_order_gpu import CASES, longest
    lines = ["paged_split %d %d %d 16 %d %d" % (B, H, D, -(-longest(B, H, ranges, D) // 16), ranges) for B, H, ranges, D, _ in CASES]
    for (B, H, ranges, D, _), ans in zip(CASES, plan(lines)):
        assert ans == "%d %d" % (ranges, B <= 256), (B, H, ranges, D)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("heads,Sq", [(1024, 1024), (512, 2048), (128, 8192), (300, 1280), (161, 700), (64, 4096), (100, 768), (57, 1600), (64, 2048), (71, 2000),
                                      (29, 4096), (33, 1100), (10, 9472), (35, 512), (9, 12800), (257, 500), (86, 640), (1000, 540), (19, 999)])
def test_masked_attention_ends_with_short_items(plan, D, heads, Sq):
    """Every item once; and an XCD's workgroups, each started where one has ended (two per CU for D = 64), end together but for less
    than half of the longest item (head after head it was up to all of it)."""
    nq = -(-Sq // 256)
    ans = plan(["masked %d %d %d %d" % (heads * nq, nq, Sq, D)])[0]
    if ans == "plain":    # all resident at once, one per CU; no XCD has two heads; two or three tiles, the last not half full
        assert heads * nq <= (512 if D == 64 else 256) + 5 * nq or heads < 16 or (nq <= 3 and (Sq - 1) % 256 < 128)
        return
    items = [tuple(map(int, x.split(":"))) for x in ans.split()]
    assert sorted(items) == [(h, q) for h in range(heads) for q in range(nq)]
    for xcd in range(8):
        mine = [4 * (q + 1) for _, q in items[xcd::8]]
        if D == 64 and heads * nq <= 512:                   # pairs: the items i and i + 32 of an XCD share a CU
            pairs, alone = [a + b for a, b in zip(mine, mine[32:])], mine[max(0, len(mine) - 32):32]
            assert not pairs or max(pairs) - min(pairs) <= max(mine) / 2
            assert not alone or not pairs or min(alone) >= max(mine[:len(pairs)])
            continue
        load = [0] * (64 if D == 64 else 32)
        for c in mine:
            load[load.index(min(load))] += 2 + c
        assert max(load) <= sum(load) / len(load) + (2 + max(mine)) / 2
