"""What the calls of the C ABI launch, by kernel instance and grid, without a GPU: the program
tests/dispatch/launch_log.c takes the place of the HIP runtime's launch functions."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
F32, BF16 = 0, 1
OK, EUNSUPPORTED, EHIP = 0, -2, -4


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """launches(commands) -> per command (status, [(kernel, grid, threads), ...])"""
    from paper_2410_07348_amd import binding
    binding.load_library()
    lib = binding.lib_path()
    exe = str(tmp_path_factory.mktemp("dispatch") / "launch_log")
    subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "dispatch", "launch_log.c"), lib, "-ldl",
                    "-Wl,-rpath," + os.path.dirname(lib), "-Wl,--allow-shlib-undefined", "-o", exe], check=True)

    def run(commands):
        r = subprocess.run([exe], input="\n".join(commands) + "\n", capture_output=True, text=True, check=True)
        # (DF16b is __bf16, which older c++filts do not know)
        text = subprocess.run(["c++filt"], input=r.stdout.replace("DF16b", "t"), capture_output=True, text=True,
                              check=True).stdout
        out, cur = [], []
        for line in text.splitlines():
            if line.startswith("status "):
                out.append((int(line.split()[1]), cur))
                cur = []
            else:
                m = re.match(r"launch (?:void )?(?:moepp::)?(.*) (\d+) (\d+) (\d+) (\d+)$", line)
                name = re.sub(r"\(.*\)$", "", m.group(1)).replace("moepp::", "").replace("unsigned short", "bf16")
                cur.append((name, tuple(int(v) for v in m.groups()[1:4]), int(m.group(5))))
        assert len(out) == len(commands), text
        return out
    return run


def ctx(T, D, F, n_ffn, k=2, act=BF16, n_zero=1, n_copy=1, n_const=2):
    return "ctx %d %d %d %d %d %d %d %d %d" % (T, D, F, n_ffn, n_zero, n_copy, n_const, k, act)


def names(result):
    return [n for n, _, _ in result[1]]


@pytest.mark.parametrize("T,D,act", [(300, 768, BF16), (5000, 768, BF16), (300, 72, BF16), (5000, 64, F32), (30, 64, F32)])
def test_a_failed_router_leaves_nothing_for_the_permutation(launches, T, D, act):
    """When the router's launch fails its histogram was never written: a permutation that follows
    counts for itself."""
    r = launches([ctx(T, D, 64, 4, act=act), "fail 1", "route %d 2" % T, "fail 0", "permute %d 2" % T])
    assert r[2] == (EHIP, [])
    assert r[4][0] == OK
    assert names(r[4])[0] in ("k_perm_small", "k_perm_hist"), names(r[4])


@pytest.mark.parametrize("T,D,act,before", [(777, 4096, BF16, []), (300, 72, BF16, []), (30, 64, F32, []),
                                            (30, 64, F32, ["route 30 2", "permute 30 2"])])
def test_the_first_of_two_launches_may_fail(launches, T, D, act, before):
    """Routers that split D, and the statistics, are two kernels: a failure of the first one alone
    is reported, whether or not the runtime still knows of it after the second."""
    call = "permute" if before else "route"
    cmds = [ctx(T, D, 64, 4, act=act), "balance 0.75"] + before + ["fail 2", "%s %d 2" % (call, T)]
    assert launches(cmds)[-1] == (EHIP, [])


@pytest.mark.parametrize("T,D,k,act", [(1, 1 << 25, 2, BF16), (1, 1 << 25, 2, F32), (1000, 1 << 25, 4, F32), (64, 4096, 2, BF16)])
def test_combine_covers_any_width_within_the_grid(launches, T, D, k, act):
    """Pieces of a token lie along the grid's second dimension, which takes 65535 workgroups; whole
    accesses of 64 lanes, all columns covered."""
    r = launches([ctx(T, D, 64, 0, k=k, act=act, n_zero=1, n_copy=1, n_const=2), "combine %d %d" % (T, k)])
    (name, grid, threads), = r[1][1]
    assert name.startswith("k_combine") and threads == 256
    assert grid[0] == (T + 3) // 4 and grid[1] <= 65535 and grid[2] == 1
    if D == 4096:
        assert grid[1] == 8                      # one 16-byte access per lane and piece


# Weight-streaming FFN or tiles, by rows per expert, number of experts and bytes of weights; the
# first five are shapes of the GPU tests that are there for the weight-streaming kernels
@pytest.mark.parametrize("T,D,F,n_ffn,n_const,k,decode", [
    (48, 512, 512, 6, 2, 2, True), (40, 512, 768, 6, 2, 2, True), (64, 1024, 256, 8, 2, 2, True),
    (7, 256, 512, 3, 2, 3, True), (30, 1280, 1536, 4, 2, 2, True),
    (16, 4096, 5632, 2, 0, 2, True), (17, 4096, 5632, 2, 0, 2, False), (64, 768, 1024, 8, 0, 2, True),
    (56, 1536, 4096, 8, 0, 2, True), (64, 1536, 4096, 8, 0, 2, False), (48, 4096, 5632, 8, 0, 2, True),
    (52, 4096, 5632, 8, 0, 2, False), (80, 768, 1024, 16, 0, 2, True), (88, 768, 1024, 16, 0, 2, False),
    (64, 768, 2048, 16, 0, 2, True), (66, 768, 2048, 16, 0, 2, False), (64, 4096, 5632, 16, 2, 2, True),
    (100, 4096, 5632, 16, 2, 2, False), (64, 1000, 1416, 16, 2, 2, False)])
def test_which_ffn_takes_few_rows(launches, T, D, F, n_ffn, n_const, k, decode):
    zc = 1 if n_const else 0
    call = "forward %d %d" % (T, k)
    r = launches([ctx(T, D, F, n_ffn, k=k, n_zero=zc, n_copy=zc, n_const=n_const), call, "variant 2", call, "variant 3", call])
    for i, few in ((1, decode), (3, decode), (5, False)):
        if i > 1 and D % 128:
            assert r[i] == (EUNSUPPORTED, [])
            continue
        ffn = [n for n in names(r[i]) if n.startswith(("k_ffn", "k_grouped"))]
        want = ("k_ffn_decode<", "k_ffn_decode_combine<") if few else "k_grouped_gemm<"
        assert len(ffn) == 2 and all(n.startswith(want) for n in ffn), ffn
        assert not ffn[0].startswith("k_ffn_decode_combine<")


# 128-row tiles by rows per expert, T k / N + 1, alike with zero-computation experts and without
@pytest.mark.parametrize("T,D,F,n_ffn,n_const,tile", [
    (777, 4096, 5632, 16, 2, "128, 256"), (1025, 4096, 5632, 16, 2, "128, 256"), (1179, 4096, 5632, 16, 2, "128, 256"),
    (1180, 4096, 5632, 16, 2, "256, 256"), (1220, 4096, 5632, 16, 2, "256, 256"), (2359, 768, 2048, 32, 6, "128, 256"),
    (2360, 768, 2048, 32, 6, "256, 256"), (943, 1536, 4096, 16, 0, "128, 256"), (944, 1536, 4096, 16, 0, "256, 256"),
    (1024, 1536, 4096, 16, 0, "256, 256"),
    # 176 tiles of 256 rows, which without this rule would go to small ones
    (1180, 2048, 1408, 16, 2, "128, 256"), (1279, 2048, 1408, 16, 2, "128, 256"), (1280, 2048, 1408, 16, 2, "128, 128"),
    (255, 4096, 5632, 4, 0, "128, 256"), (256, 4096, 5632, 4, 0, "128, 128")])
def test_which_tiles_take_few_rows(launches, T, D, F, n_ffn, n_const, tile):
    zc = 1 if n_const else 0
    r = launches([ctx(T, D, F, n_ffn, n_zero=zc, n_copy=zc, n_const=n_const), "forward %d 2" % T])
    gemm1 = [n for n in names(r[1]) if n.startswith("k_grouped")][0]
    assert gemm1.startswith("k_grouped_gemm<Geo<%s," % tile), gemm1


def test_shapes_reach_the_instances_their_gpu_tests_name(launches):
    from test_gpu_ffn_edges import INSTANCES
    for kw, gemm1, gemm2 in INSTANCES:
        act, k = (F32 if kw.get("act") == "f32" else BF16), kw.get("k", 2)
        r = launches([ctx(kw["T"], kw["D"], kw["F"], kw["n_ffn"], k=k, act=act), "forward %d %d" % (kw["T"], k)])
        assert [n for n in names(r[1]) if n.startswith(("k_ffn", "k_grouped"))] == [gemm1, gemm2]


def test_float32_layers_on_split_operands(launches):
    """Which tiles, by rows per expert and widths; widths that are not multiples of 32 and few tiles stay
    with the float32 instruction."""
    from test_gpu_ffn_edges import F32_TILES, SPLIT_EXACT
    for kw, gemm1, gemm2 in F32_TILES:
        r = launches([ctx(kw["T"], kw["D"], kw["F"], kw["n_ffn"], k=kw.get("k", 2), act=F32),
                      "forward %d %d" % (kw["T"], kw.get("k", 2))])
        assert [n for n in names(r[1]) if n.startswith("k_ffn")] == [gemm1, gemm2], kw
    for T, D, F, gemm1, gemm2 in SPLIT_EXACT:
        r = launches([ctx(T, D, F, 4, k=1, act=F32, n_zero=0, n_copy=0, n_const=0), "forward %d 1" % T])
        assert [n for n in names(r[1]) if n.startswith("k_ffn")] == [gemm1, gemm2], (T, D, F)
    for D, F in ((768, 2048), (768, 2040), (760, 2048)):
        r = launches([ctx(2048, D, F, 8, act=F32), "forward 2048 2"])
        assert ["k_ffn_f32_split" in n for n in names(r[1]) if n.startswith("k_ffn")] == [(D, F) == (768, 2048)] * 2


@pytest.mark.parametrize("T,D,act,n_ffn,router", [
    (1, 768, BF16, 16, ["k_router_one"]), (16, 256, F32, 16, ["k_router_one"]),
    (2, 1024, BF16, 16, ["k_router_small_partial", "k_router_small_final_perm"]),
    (17, 256, BF16, 16, ["k_router_small_partial", "k_router_small_final_perm"]),
    (64, 4096, BF16, 40, ["k_router_small_partial", "k_router_small_final_perm"]),
    (65, 1024, BF16, 16, ["k_router_small_partial", "k_router_final"]), (65, 640, BF16, 16, ["k_router_block"]),
    (2048, 4096, BF16, 16, ["k_router_small_partial", "k_router_final"]), (2049, 768, BF16, 16, ["k_router_block"]),
    (4096, 4096, BF16, 16, ["k_router_small_partial", "k_router_final"]), (4097, 4096, BF16, 16, ["k_router_block"]),
    (8193, 1536, BF16, 16, ["k_router_mfma"]), (3000, 3080, BF16, 16, ["k_router_small_partial", "k_router_final"]),
    (5000, 1000, BF16, 16, ["k_router_small_partial", "k_router_final"]),
    (300, 1000, BF16, 56, ["k_router_small_partial", "k_router_final"]),
    (3000, 1032, F32, 16, ["k_router_small_partial", "k_router_final"]), (40000, 64, F32, 16, ["k_router_generic"])])
def test_which_router(launches, T, D, act, n_ffn, router):
    """By tokens, columns and type; the partial sums of every slice fit their 2.6 MB."""
    r = launches([ctx(T, D, 64, n_ffn, act=act), "route %d 2" % T])
    assert [n.split("<")[0] for n in names(r[1])] == router
    if router[0] == "k_router_small_partial":
        slices = r[1][1][0][1][0]
        assert slices <= 24 and slices * (T * (n_ffn + 8) + 3) * 4 <= 32 * 256 * 80 * 4


# (slices of D, blocks of tokens).  bf16: four to eight slices, as few rounds of 256 workgroups a slice as can be, more
# for a wide layer's few tokens; float32: as many as fit; always within the partial sums (T x rows x slices floats)
# and with a slice of 32 columns for every wave
@pytest.mark.parametrize("T,D,act,n_ffn,n_const,grid", [
    (80, 1536, BF16, 16, 2, (7, 5)), (300, 4096, BF16, 16, 2, (8, 10)), (1500, 4096, BF16, 16, 2, (5, 47)),
    (300, 776, BF16, 50, 6, (7, 10)), (2048, 4096, BF16, 16, 2, (8, 64)), (3000, 8192, BF16, 4, 0, (8, 94)),
    (1024, 4096, BF16, 32, 6, (8, 32)), (1200, 4096, BF16, 32, 6, (6, 38)), (2048, 4096, BF16, 32, 6, (4, 64)),
    (4096, 4096, BF16, 32, 6, (3, 128)), (300, 8192, BF16, 16, 2, (24, 10)), (1024, 8192, BF16, 16, 2, (8, 32)),
    (256, 128, F32, 50, 6, (2, 16)), (2048, 1056, F32, 16, 2, (9, 64)), (30000, 768, F32, 4, 0, (3, 938))])
def test_slices_of_the_router(launches, T, D, act, n_ffn, n_const, grid):
    r = launches([ctx(T, D, 64, n_ffn, act=act, n_const=n_const), "route %d 2" % T])
    assert names(r[1])[0].startswith("k_router_small_partial<") and r[1][1][0][1] == grid + (1,)
    rows = n_ffn + 2 + 3 * n_const
    assert grid[0] * (T * rows + 3) * 4 <= 32 * 256 * 80 * 4


MFMA = "k_router_mfma<%d, %d, %d, %d, %d>"


# blocks of 32 weight rows, tiles prefetched, tokens, waves per SIMD, groups of waves
@pytest.mark.parametrize("T,D,n_ffn,instance", [
    (300, 512, 6, (1, 4, 64, 2, 2)), (2100, 1024, 6, (1, 4, 64, 2, 2)), (257, 256, 3, (1, 2, 64, 2, 2)),
    (2100, 768, 6, (1, 2, 64, 2, 2)), (300, 640, 6, (1, 2, 64, 3, 1)), (2111, 1408, 3, (1, 2, 64, 3, 1)),
    (300, 512, 34, (2, 2, 64, 2, 2)), (2100, 768, 34, (2, 2, 64, 2, 2)), (2100, 1024, 34, (2, 2, 64, 2, 2)),
    (300, 640, 34, (2, 2, 64, 2, 1)), (2100, 1408, 34, (2, 2, 64, 2, 1)), (24576, 512, 6, (1, 4, 128, 2, 1))])
def test_instances_of_the_matrix_core_router(launches, T, D, n_ffn, instance):
    """The shapes of tests/test_gpu_router_numerics.py and tests/test_gpu_ffn_edges.py that are there for them, which ask
    for this router."""
    r = launches([ctx(T, D, 64, n_ffn, n_zero=2, n_copy=2), "variant 2", "route %d 2" % T])
    assert names(r[2]) == [MFMA % instance]


def test_the_lists_of_routers_name_the_kernels_they_reach(launches):
    from test_gpu_router_numerics import MATRIX_CORE, ROUTERS, SLICED, TWO_BLOCKS
    for act, T, D, variant in ROUTERS:
        r = launches([ctx(T, D, 64, 6, n_zero=2, n_copy=2, act=F32 if act == "f32" else BF16), "variant %d" % variant, "route %d 2" % T])
        assert names(r[2])[0].startswith("k_router_mfma<") == ((act, T, D, variant) in MATRIX_CORE), (act, T, D)
        assert (names(r[2])[-1].startswith("k_router_final<")) == ((act, T, D, variant) in SLICED), (act, T, D)
    for T, D in TWO_BLOCKS:
        r = launches([ctx(T, D, 64, 34, n_zero=2, n_copy=2), "variant 2", "route %d 2" % T])
        assert names(r[2])[0].startswith("k_router_mfma<2,"), (T, D)


# (n_ffn + 8 weight rows)
@pytest.mark.parametrize("T,D,act,n_ffn,tok", [
    # beside the matrix-core router
    (64, 256, BF16, 16, 0), (65, 128, BF16, 16, 16), (300, 640, BF16, 32, 16), (2049, 1408, BF16, 56, 16),
    (4096, 1408, BF16, 16, 16),
    (4097, 128, BF16, 16, 32), (4352, 4096, BF16, 32, 32), (8192, 256, BF16, 32, 32), (8193, 256, BF16, 16, 0),
    (300, 256, BF16, 57, 0),
    # beside the slices
    (65, 1000, BF16, 16, 16), (255, 1024, BF16, 16, 0), (256, 1024, BF16, 16, 16), (256, 1536, BF16, 16, 0),
    (1535, 1536, BF16, 8, 16),
    (1535, 2048, BF16, 16, 0), (1536, 2048, BF16, 16, 16), (1535, 1024, BF16, 32, 0), (2048, 1024, BF16, 32, 16),
    (2048, 1536, BF16, 32, 0),
    (2049, 1536, BF16, 32, 0), (1535, 1544, BF16, 8, 0), (1536, 1544, BF16, 8, 16), (4096, 1032, BF16, 32, 0),
    (4096, 2048, BF16, 16, 16), (2049, 4096, BF16, 16, 0), (2049, 4096, BF16, 8, 16),
    (300, 8, BF16, 8, 16), (4096, 1000, BF16, 32, 16), (4097, 1000, BF16, 8, 0), (4097, 512, BF16, 8, 32),
    (8192, 504, BF16, 56, 32),
    (4400, 520, BF16, 8, 0),
    # float32
    (65, 8, F32, 4, 16), (2048, 768, F32, 9, 16), (4096, 1024, F32, 16, 16), (4096, 1024, F32, 24, 16),
    (4096, 1032, F32, 8, 0),
    (4096, 512, F32, 56, 16), (4096, 520, F32, 25, 0), (4097, 256, F32, 4, 0), (300, 64, F32, 57, 0),
    (128, 1024, F32, 16, 0)])
def test_where_the_router_on_blocks_runs(launches, T, D, act, n_ffn, tok):
    """By tokens, columns, type and weight rows; variants keep the others, and the permutation has as many chunks as
    there were blocks (four chunks a workgroup), at most what its histogram's place and its kernel take."""
    r = launches([ctx(T, D, 64, n_ffn, act=act), "route %d 2" % T, "permute %d 2" % T, "variant 1", "route %d 2" % T])
    assert [n.startswith("k_router_block<") for n in names(r[1])][:1] == [tok > 0], names(r[1])
    assert "k_router_block" not in names(r[4])[0]
    if tok:
        (name, grid, threads), = r[1][1]
        assert grid == ((T + tok - 1) // tok, 1, 1) and name.split(",")[1].strip() == str(tok // 16)
        assert grid[0] <= 2048 and grid[0] * (n_ffn + 4) * 4 <= 32 * 256 * 80 * 4
        (name, perm, _), = r[2][1]
        assert name == "k_perm_scan_scatter" and perm == ((grid[0] + 3) // 4, 1, 1)


def test_blocks_of_the_gpu_tests(launches):
    """... and every instance is among them."""
    from test_gpu_router_block import BLOCK, INSTANCES
    reached = set()
    for act, T, D, n_ffn, n, k, inst in BLOCK:
        r = launches([ctx(T, D, 64, n_ffn, k=k, act=F32 if act == "f32" else BF16, n_zero=n, n_copy=n, n_const=n), "route %d %d" % (T, k)])
        m = re.match(r"k_router_block<(float|bf16), (\d), (\d), \d+, (\d+), (\d)>$", names(r[1])[0])
        assert m, (T, D, names(r[1]))
        got = (16 * int(m.group(2)),) + tuple(int(v) for v in m.groups()[2:])
        assert got == inst, (act, T, D, got)
        reached.add((act,) + got)
    assert reached == INSTANCES


def test_halves_of_wide_float32_tiles(launches):
    """As many workgroups as tiles at most (slots / 128 rows and one more per expert), and half of an XCD's CUs more on each."""
    from test_gpu_ffn_edges import F32_HALVES
    for kw, gemm1, gemm2 in F32_HALVES:
        T, D, F, n, k = kw["T"], kw["D"], kw["F"], kw["n_ffn"], kw.get("k", 2)
        r = launches([ctx(T, D, F, n, k=k, act=F32, n_zero=kw.get("n_zero", 1), n_copy=kw.get("n_copy", 1), n_const=kw.get("n_const", 2)),
                      "forward %d %d" % (T, k)])
        got = [(name, grid[0]) for name, grid, _ in r[1][1] if name.startswith("k_ffn")]
        for (name, grid), want, cols in zip(got, (gemm1, gemm2), (2 * F, D)):
            assert want in (None, name), (kw, got)
            if "128, 256" in name:
                assert grid == ((T * k // 128 + n) * -(-cols // 256) + 7) // 8 * 8 + 128


def test_halves_and_whole_tiles_of_the_gpu_test(launches):
    """Wide tiles in both calls, and as many as the test's own list of them has, which must be enough halves in the first."""
    from test_gpu_ffn_edges import F32_HALF_WHOLE, WIDE, tile_kinds
    for D, F, k, few, many, name in F32_HALF_WHOLE:
        halves = []
        for T in (few, many):
            r = launches([ctx(T, D, F, 4, k=k, act=F32, n_zero=0, n_copy=0, n_const=0), "forward %d %d" % (T, k)])
            gemm = [n for n in names(r[1]) if n.startswith("k_ffn")][name == "yffn"]
            assert gemm == WIDE % ("true" if name == "h" else "false"), gemm
            kinds = tile_kinds([(T * k + 3 - e) // 4 for e in range(4)], 2 * F if name == "h" else D)
            halves.append(sum(kinds.values()) / len(kinds))
        assert halves[0] > 0.25 and halves[1] == 0.0, halves


@pytest.mark.parametrize("T,D,F,n_ffn,k,together", [
    (1, 768, 2048, 16, 2, True), (2, 768, 2048, 16, 2, False), (1, 768, 2048, 16, 4, False), (16, 4096, 5632, 16, 2, True),
    (48, 4096, 5632, 16, 2, True),
    (49, 4096, 5632, 16, 2, False), (8, 2048, 2048, 16, 2, False), (4, 512, 512, 8, 2, True), (48, 3840, 256, 16, 2, True),
    (8, 3072, 2048, 16, 2, True), (18, 1024, 256, 16, 2, False), (6, 1024, 256, 16, 2, True),
    # more workgroups than the 256 CUs
    (1, 4352, 5632, 16, 2, False), (16, 4352, 5632, 16, 2, False), (16, 5120, 5632, 16, 2, False),
    (1, 5120, 2560, 16, 2, False),
    (1, 6144, 768, 16, 2, False), (16, 6144, 512, 16, 2, True), (4, 4352, 512, 16, 2, True), (16, 4352, 512, 16, 2, False)])
def test_which_calls_combine_in_gemm2(launches, T, D, F, n_ffn, k, together):
    """16 columns a workgroup; the step calls and the variants keep the two kernels."""
    call = "forward %d %d" % (T, k)
    r = launches([ctx(T, D, F, n_ffn, k=k), call, "ffn %d %d" % (T, k), "combine %d %d" % (T, k), "variant 2", call])
    last = [n for n in names(r[1]) if n.startswith(("k_ffn", "k_combine"))]
    if together:
        assert last[1:] == ["k_ffn_decode_combine<%d>" % (F // 256)] and r[1][1][-1][1] == (D // 16, 1, 1)
    for got in (last, [n for n in names(r[2]) + names(r[3])], [n for n in names(r[5]) if n.startswith(("k_ffn", "k_combine"))])[together:]:
        assert got[1].startswith("k_ffn_decode<false, ") and got[2].startswith("k_combine<"), got


def test_shapes_of_the_gpu_test_combine_in_gemm2(launches):
    from test_gpu_ffn_edges import DECODE_COMBINE
    for T, D, F, n_ffn, n, k in DECODE_COMBINE:
        r = launches([ctx(T, D, F, n_ffn, k=k, n_zero=n, n_copy=n, n_const=n), "forward %d %d" % (T, k)])
        assert names(r[1])[-1] == "k_ffn_decode_combine<%d>" % (F // 256), (T, D, F, names(r[1]))
