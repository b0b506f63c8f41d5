"""Kernels at the edges of their tiles and dispatch rules, every case against the oracle
on all tokens with the tolerances of tests/helpers.py: widths that leave a narrower last K
slab (D % 32, F % 32), fewer rows than a tile, groups that end inside one, token counts on
both sides of a rule."""
import numpy as np
import pytest

from workloads import LayerShape, make_inputs

from helpers import check_layer, gpu_forward, make_layer, sample_tokens

pytestmark = pytest.mark.gpu


def check(**kw):
    s = LayerShape("edge", n_zero=1, n_copy=1, n_const=2, seed=8100, **kw)
    print("shape", s, flush=True)
    inp = make_inputs(s)
    print("  ", check_layer(s, inp, gpu_forward(s, inp)), flush=True)


# 4 experts, top-2: weight streaming up to T = 32, above it tiles of 32 x 64 (GEMM1) and
# 32 x 32 (GEMM2); 64 x 128 tiles from 1024 of them on
@pytest.mark.parametrize("D,F", [(8, 8), (24, 40), (64, 32), (104, 72), (264, 1000), (768, 512)])
@pytest.mark.parametrize("T", [1, 2, 31, 32, 33, 257])
def test_f32(T, D, F):
    check(T=T, D=D, F=F, n_ffn=4, act="f32")


@pytest.mark.parametrize("T,D,F", [(4096, 520, 1032), (2500, 2048, 256), (2500, 96, 2080)])
def test_f32_large_tiles(T, D, F):
    check(T=T, D=D, F=F, n_ffn=4, act="f32", k=3)


# bf16 widths that are not multiples of 64 (zero-padded K loop), also with fewer than the
# four K tiles the ring starts with, and reductions of 64 (variants 0 and 2)
@pytest.mark.parametrize("D,F", [(8, 8), (24, 40), (72, 136), (128, 96), (104, 64), (520, 1032), (1000, 1416)])
@pytest.mark.parametrize("T", [1, 33, 127, 300])
def test_bf16_ragged_widths(T, D, F):
    check(T=T, D=D, F=F, n_ffn=4)


@pytest.mark.parametrize("D,F", [(64, 128), (128, 64), (64, 64)])
def test_bf16_short_reduction(D, F):
    check(T=900, D=D, F=F, n_ffn=4, k=3)


# routers between the few-token one (T <= 64) and the 128-token blocks (T >= 24576): blocks of 16 tokens in one
# kernel; the matrix-core one (variant 2) with two groups of waves (D = 128, 256, 512: one pass of its loop over K
# tiles, or two), one and two blocks of weight rows; slices of 32 columns (wider layers, more than 64 rows)
@pytest.mark.parametrize("D", [128, 256, 512, 1408, 1536, 4096, 72])
@pytest.mark.parametrize("n_ffn,n_const,k", [(3, 2, 2), (37, 7, 3), (52, 8, 8)])
@pytest.mark.parametrize("T", [257, 321])
def test_router(T, D, n_ffn, n_const, k, variant=0):
    s = LayerShape("edge", T=T, D=D, F=64, n_ffn=n_ffn, n_zero=1, n_copy=1, n_const=n_const, k=k,
                   bias="normal", seed=8200)
    inp = make_inputs(s)
    L = make_layer(s)
    cap = L.capacity(T, 1.1, 0.75)
    res = gpu_forward(s, inp, variant, layer=L, cap=cap, balance_tau=0.75)
    print("  ", s, check_layer(s, inp, res, cap=np.array(cap, np.int32), balance_tau=0.75), flush=True)


# the matrix-core router with several passes of its loop: one group of waves (D = 640, 1408), two (D = 768, 1024)
@pytest.mark.parametrize("n_ffn,n_const,k", [(3, 2, 2), (37, 7, 3)])
@pytest.mark.parametrize("T,D", [(257, 640), (2111, 768), (2111, 1024), (2111, 1408), (257, 128), (321, 256), (257, 512)])
@pytest.mark.parametrize("variant", [0, 2])
def test_matrix_core_router(T, D, n_ffn, n_const, k, variant):
    test_router(T, D, n_ffn, n_const, k, variant)


# the routers on slices of 32 columns: the whole router in one workgroup (T <= 16, up to 80 KB of x and
# weights) and in two kernels, blocks of 16 and 32 tokens, one to five blocks of 16 weight rows, a last
# slice of 8 columns, fewer slices than waves, more slices than fit in one pass of the waves, previous
# logits of more than one slice, no gating residual; with capacities, which the few-token permutation applies
@pytest.mark.parametrize("D", [8, 40, 264, 1000, 4096])
@pytest.mark.parametrize("n_ffn,n_const,k,act", [(3, 2, 2, "bf16"), (13, 4, 1, "f32"), (37, 7, 3, "bf16"), (52, 8, 8, "f32")])
@pytest.mark.parametrize("T", [1, 5, 16, 17, 64, 65, 257, 1025])
def test_sliced_router(T, D, n_ffn, n_const, k, act):
    s = LayerShape("edge", T=T, D=D, F=64, n_ffn=n_ffn, n_zero=1, n_copy=1, n_const=n_const, k=k, act=act,
                   bias="normal" if T % 2 else "none", residual=T != 5, seed=8500)
    inp = make_inputs(s)
    L = make_layer(s)
    cap = L.capacity(T, 1.1, 0.75)
    res = gpu_forward(s, inp, layer=L, cap=cap, balance_tau=0.75)
    print("  ", s, check_layer(s, inp, res, cap=np.array(cap, np.int32), balance_tau=0.75), flush=True)


# tile geometries of the bf16 FFN: 128x128 tiles (few tiles, or one round of 129 - 208 large
# ones), half tiles as the rest of a launch of large ones, weights past the caches (more than
# 256 MB of them), group sizes around the tile heights
@pytest.mark.parametrize("T,D,F,n_ffn,bias", [(40, 192, 320, 3, "none"), (300, 320, 192, 2, "normal"),
                                              (1300, 256, 256, 4, "normal"), (2600, 1024, 128, 16, "none"),
                                              (3000, 704, 1408, 5, "normal"), (700, 3072, 448, 33, "normal"),
                                              (1500, 64, 1000, 7, "none"), (1179, 1024, 512, 16, "none")])
def test_bf16_tile_geometries(T, D, F, n_ffn, bias):
    check(T=T, D=D, F=F, n_ffn=n_ffn, bias=bias)


# (700: 117 rows per expert, the most that take 128-row tiles, and groups beyond 128 rows)
@pytest.mark.parametrize("T", [130, 600, 700])
def test_bf16_streamed_weights(T):
    check(T=T, D=1536, F=4096, n_ffn=8)


# Kernel instances that take shapes of their own to reach, GEMM1 and GEMM2 (tests/test_dispatch_cpu.py
# checks that these shapes launch them): float32 tiles of 64 x 128 and 32 x 64 with and without a narrower
# last slab (widths that are not multiples of 32, which the split kernel does not take); 128 x 256 tiles with a narrower last slab of h; 256 x 256 tiles with streamed
# weights, which all run as half tiles in GEMM2 and leave 16 of 272 to them in GEMM1.
FULL, HALF = "Geo<256, 256, 2, 4, 32, 5, 4>", "Geo<128, 256, 2, 4, 32, 5, 4>"
INSTANCES = [
    (dict(T=4096, D=1024, F=1000, n_ffn=4, k=3, act="f32"), "k_ffn_f32<true, false, 64, 128, 2, 2>",
     "k_ffn_f32<false, true, 64, 128, 2, 2>"),
    (dict(T=4096, D=512, F=264, n_ffn=4, k=3, act="f32"), "k_ffn_f32<true, false, 32, 64, 2, 1>",
     "k_ffn_f32<false, true, 32, 64, 2, 2>"),
    (dict(T=4096, D=520, F=256, n_ffn=4, k=3, act="f32"), "k_ffn_f32<true, true, 32, 64, 2, 1>",
     "k_ffn_f32<false, false, 32, 64, 2, 2>"),
    (dict(T=4096, D=1032, F=512, n_ffn=4, k=3, act="f32"), "k_ffn_f32<true, true, 64, 128, 2, 2>",
     "k_ffn_f32<false, false, 64, 128, 2, 2>"),
    (dict(T=300, D=1000, F=424, n_ffn=40), "k_grouped_gemm<%s, true, void, true, false>" % HALF,
     "k_grouped_gemm<%s, false, void, true, false>" % HALF),
    (dict(T=2000, D=1536, F=2176, n_ffn=16), "k_grouped_gemm<%s, true, %s, false, true>" % (FULL, HALF),
     "k_grouped_gemm<%s, false, %s, false, true>" % (FULL, HALF)),
]


@pytest.mark.parametrize("kw", [i[0] for i in INSTANCES])
def test_instances(kw):
    s = LayerShape("edge", n_zero=1, n_copy=1, n_const=2, seed=8100, **kw)
    print("shape", s, flush=True)
    inp = make_inputs(s)
    res = gpu_forward(s, inp)
    if kw["n_ffn"] == 16:
        # the streamed launch: one tile of rows per expert, and a rest for the half tiles
        assert max(res["counts"][:16]) <= 256
        left = 16 * (2 * s.F // 256) % 256
        assert 0 < left <= 128 and 16 * (s.D // 256) <= 128
    print("  ", check_layer(s, inp, res, tok_list=sample_tokens(s, res["topk_idx"], 256)), flush=True)


# weight-streaming FFN: one fragment per workgroup in GEMM2 (few experts), two; several units per
# workgroup; both sides of T k = 16 n_ffn; the few-token router's one-workgroup end with
# 1 .. 64 tokens; a combine in pieces of a token
@pytest.mark.parametrize("T", [1, 2, 15, 16, 17, 32, 33, 63, 64])
@pytest.mark.parametrize("D,F,n_ffn", [(256, 512, 4), (1280, 256, 12), (512, 2048, 33)])
def test_bf16_few_rows(T, D, F, n_ffn):
    check(T=T, D=D, F=F, n_ffn=n_ffn, bias="normal")


# more workgroups of 16 columns than CUs: GEMM2 and the combine apart
def test_bf16_few_rows_of_a_wide_layer():
    check(T=9, D=6144, F=4352, n_ffn=2, k=3, bias="normal")


# SiLU of the ragged bf16 layers is as exact as expf and a division, which the plain FMA kernels have.  x has a
# single one and W3 is one, so both kernels see the same z = W1 exactly, and it runs through
# every bfloat16 of magnitude 2^-8 .. 88: h must be the same bit for bit, and within half a
# bfloat16 ulp (2^-9 of the value, and a few float32 ulps) of z / (1 + e^-z) * 1.
@pytest.mark.parametrize("T", [1, 300])
def test_ragged_silu(T):
    mag = (np.arange(0x3B80, 0x42B1, dtype=np.uint32) << 16).view(np.float32)
    z = np.concatenate([mag, -mag])
    s = LayerShape("silu", T=T, D=8, F=(z.size + 7) // 8 * 8, n_ffn=1, n_zero=0, n_copy=0, n_const=0, k=1,
                   residual=False, seed=8300)
    inp = make_inputs(s)
    inp["x"][:] = 0.0
    inp["x"][:, 3] = 1.0
    inp["w1"][:] = 0.0
    inp["w1"][0, :z.size, 3] = z
    inp["w3"][:] = 0.0
    inp["w3"][0, :, 3] = 1.0
    a, b = gpu_forward(s, inp), gpu_forward(s, inp, variant=1)
    want = z.astype(np.float64) / (1.0 + np.exp(-z.astype(np.float64)))
    err = np.abs(a["h"][:, :z.size] - want) / np.abs(want)
    print("silu error * 2^8", err.max() * 256, "differ", (a["h"] != b["h"]).sum(), flush=True)
    assert err.max() <= 1.0 / 256
    assert np.array_equal(a["h"], b["h"])


# float32 layers on split operands (D and F multiples of 32): 128 x 256 tiles, 128 x 128 and 64 x 64 ones, an
# odd and an even number of slabs, one slab, groups that end inside a tile, and the float32 instruction where it
# is faster; the rule is looked at in tests/test_dispatch_cpu.py
WIDE, SQUARE, SMALL = "k_ffn_f32_split<%s, 128, 256, 2, 4>", "k_ffn_f32_split<%s, 128, 128, %s>", "k_ffn_f32_split<%s, 64, 64, %s>"
PLAIN = "k_ffn_f32<false, false, 32, 32, 2, 2>"
F32_TILES = [
    (dict(T=4096, D=544, F=992, n_ffn=12), WIDE % "true", SMALL % ("false", "2, 2")),
    (dict(T=700, D=736, F=1024, n_ffn=6), "k_ffn_f32<true, false, 32, 64, 2, 1>", PLAIN),
    (dict(T=333, D=512, F=512, n_ffn=16, bias="normal"), SMALL % ("true", "4, 1"), PLAIN),
    (dict(T=3000, D=1024, F=256, n_ffn=4, k=3, bias="normal"), SMALL % ("true", "4, 1"), WIDE % "false"),
    (dict(T=2000, D=768, F=384, n_ffn=8, k=3), SQUARE % ("true", "4, 2"), SQUARE % ("false", "2, 4")),
    (dict(T=4096, D=1024, F=2048, n_ffn=8), WIDE % "true", WIDE % "false"),
    (dict(T=9000, D=32, F=96, n_ffn=8), SMALL % ("true", "4, 1"), PLAIN),
]


@pytest.mark.parametrize("kw", [i[0] for i in F32_TILES])
def test_f32_tiles(kw):
    s = LayerShape("edge", n_zero=1, n_copy=1, n_const=2, seed=8100, act="f32", **kw)
    print("shape", s, flush=True)
    inp = make_inputs(s)
    res = gpu_forward(s, inp)
    print("  ", check_layer(s, inp, res, tok_list=sample_tokens(s, res["topk_idx"], 256)), flush=True)


# (T, D, F, GEMM1, GEMM2) with 4 experts and nothing else: every instance
SPLIT_EXACT = [(3000, 1024, 512, SQUARE % ("true", "4, 2"), SQUARE % ("false", "2, 4")),
               (4096, 1024, 1024, SMALL % ("true", "4, 1"), SMALL % ("false", "2, 2")),
               (6000, 512, 512, WIDE % "true", SQUARE % ("false", "2, 4")),
               (2500, 2048, 256, SMALL % ("true", "4, 1"), WIDE % "false")]


def exact_shape(T, D, F):
    return LayerShape("edge", T=T, D=D, F=F, n_ffn=4, n_zero=0, n_copy=0, n_const=0, k=1, act="f32", residual=False, seed=8400)


def only(w, cols):
    """The columns `cols` of w, zeros elsewhere."""
    z = np.zeros_like(w)
    z[..., cols] = w[..., cols]
    return z


@pytest.mark.parametrize("scale", [1.0, 1e-18])
@pytest.mark.parametrize("n", [1, 4])
@pytest.mark.parametrize("T,D,F", [i[:3] for i in SPLIT_EXACT])
def test_f32_products_are_float32_products(T, D, F, n, scale):
    """Rows of h with n numbers that are not zero, down to 1e-36.  Every term of a sum is rounded with its
    addition, 2^-24 of what is added up, and that at most twice: once among the products of the first
    pieces, once with the others, whose own roundings are 2^-6 of that, seven a term; half the smallest
    float more where that is below the normal ones.  A lone term is rounded once."""
    s = exact_shape(T, D, F)
    inp = make_inputs(s)
    cols = [5, 77, 130, 201][:n]
    w1 = np.zeros_like(inp["w1"])
    w1[:, cols] = inp["w1"][:, cols]
    inp["w1"] = w1
    inp["x"] = (inp["x"] * scale).astype(np.float32)
    res = gpu_forward(s, inp)
    assert np.abs(res["h"][:, cols]).max() > 1e-3 * scale * scale and not np.delete(res["h"], cols, axis=1).any()
    worst = 0.0
    for e in range(s.n_ffn):
        rows = slice(res["offsets"][e], res["offsets"][e + 1])
        h, w2 = res["h"][rows][:, cols].astype(np.float64), inp["w2"][e][:, cols].astype(np.float64)
        err = np.abs(res["yffn"][rows] - h @ w2.T)
        bound = ((n if n > 1 else 0.5) * 2 + n * 7 / 64) * (2.0 ** -24 * (np.abs(h) @ np.abs(w2).T)) + n * 8 * 2.0 ** -150
        worst = max(worst, (err / bound).max())
    print("nonzero", n, "scale", scale, "error / bound", worst, flush=True)
    assert worst <= 1.0


@pytest.mark.parametrize("T,D,F", [i[:3] for i in SPLIT_EXACT])
def test_f32_small_activations(T, D, F):
    """x of 1e-36 in every third row and of 1e-41, below the normal numbers, in one, against large
    weights of one column: z and u are one product each, h = z u / (1 + e^-z), all within a few float32
    roundings (of the product, of e^-z, the sum, the division and the last product)."""
    s = exact_shape(T, D, F)
    inp = make_inputs(s)
    inp["w1"], inp["w3"] = only(inp["w1"], [9]) * np.float32(1e32), only(inp["w3"], [9]) * np.float32(1e32)
    x = inp["x"]
    x *= np.float32(1e-30)
    x[0::3] *= np.float32(1e-6)
    x[1::30] *= np.float32(1e-11)
    res = gpu_forward(s, inp)
    tok, worst = res["src_of"], 0.0
    for e in range(s.n_ffn):
        rows = slice(res["offsets"][e], res["offsets"][e + 1])
        xs = x[tok[rows], 9].astype(np.float64)[:, None]
        z, u = xs * inp["w1"][e][None, :, 9].astype(np.float64), xs * inp["w3"][e][None, :, 9].astype(np.float64)
        want = z / (1 + np.exp(-z)) * u
        big = np.abs(want) > 2.0 ** -120
        err = np.abs(res["h"][rows] - want)[big] / np.abs(want)[big]
        # e^-z: its argument is off by 2^-24 |z|
        worst = max(worst, (err * 2.0 ** 24 / (12 + np.abs(z)[big])).max())
    print("error / bound", worst, flush=True)
    assert worst <= 1.0


@pytest.mark.parametrize("T,D,F", [i[:3] for i in SPLIT_EXACT])
def test_f32_rows_do_not_depend_on_their_neighbours(T, D, F):
    """Tokens with an infinity, with NaN and with numbers below 2^-110 change no bit of another token's
    row of h and yffn, and weight rows of small numbers none of another column."""
    s = exact_shape(T, D, F)
    inp = make_inputs(s)
    inp["W_g"][:, 20:] = 0.0
    inp["w2"][:, :, 3] = 0.0
    a = gpu_forward(s, inp)
    odd = [T // 2, T // 3, T // 5]
    x = inp["x"]
    x[odd[0], 40], x[odd[1], 50] = np.inf, np.nan
    x[odd[2], 30:] *= np.float32(2.0 ** -118)
    inp["w1"][:, 3, 20:] *= np.float32(2.0 ** -118)
    inp["w2"][:, 5] *= np.float32(2.0 ** -118)
    b = gpu_forward(s, inp)
    assert (~np.isfinite(b["out_gate"]).all(axis=1)).sum() == 2          # (0 times an infinity or a NaN)
    # row of every token, whose only slot it is
    row = [np.argsort(r["src_of"]) for r in (a, b)]
    tok = np.array([t for t in range(T) if t not in odd])
    h, y = ([r[name][q[tok]] for r, q in zip((a, b), row)] for name in ("h", "yffn"))
    assert np.array_equal(np.delete(h[0], 3, axis=1), np.delete(h[1], 3, axis=1))
    assert np.array_equal(np.delete(y[0], 5, axis=1), np.delete(y[1], 5, axis=1))


# NaN of both signs, and with nothing but the lowest bits of the significand set
NANS = np.array([0x7fc00000, 0xffc00000, 0x7f800001, 0xff80ffff], np.uint32).view(np.float32)


def test_f32_largest_floats_infinities_and_nan():
    """The largest finite float does not overflow, and infinite or NaN operands give what the plain FMA
    kernels give: the same elements of h infinite (with their sign), NaN and finite."""
    s = LayerShape("edge", T=3000, D=1024, F=512, n_ffn=4, n_zero=0, n_copy=0, n_const=0, k=1, act="f32",
                   residual=False, seed=8400)
    inp = make_inputs(s)
    inp["W_g"][:, 5:12] = 0.0
    inp["w1"][:, :, 5] = 1e-30 * np.sign(inp["w1"][:, :, 5])        # 3.4e8, with the sign of the weight
    inp["w3"][:, :, 5] = 1e-33
    x = inp["x"]
    x[:, 5] = 0.0
    x[0::7, 5] = np.finfo(np.float32).min
    x[1::7, 5] = np.finfo(np.float32).max
    a, b = gpu_forward(s, inp), gpu_forward(s, inp, variant=1)
    assert np.isfinite(a["h"]).all() and np.array_equal(a["src_of"], b["src_of"])
    for name in ("h", "yffn"):
        ref = np.abs(b[name]).max(axis=1, keepdims=True)
        err = (np.abs(a[name] - b[name]) / ref).max()
        print(name, err, flush=True)
        assert err <= 1e-5, (name, err)
    x[2::7, 6] = np.inf
    x[3::7, 7] = -np.inf
    x[4::7, 8] = np.nan
    inp["w1"][0, 3, 9] = np.inf
    inp["w3"][1, 4, 10] = -np.inf
    for i, nan in enumerate(NANS):
        x[4 + 7 * i::28, 8] = nan
        inp["w1"][2, 10 + i, 9] = nan
        inp["w3"][3, 20 + i, 10] = nan
    a, b = gpu_forward(s, inp), gpu_forward(s, inp, variant=1)
    assert np.array_equal(a["src_of"], b["src_of"])
    for name in ("h", "yffn"):
        ha, hb = a[name], b[name]
        for what in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(what(ha), what(hb)), (name, what.__name__)
    rows = np.nonzero(np.isin(a["src_of"], np.arange(4, s.T, 7)))[0]
    assert np.isnan(a["h"][rows]).all()
    for i in range(len(NANS)):
        assert np.isnan(a["h"][a["offsets"][2]:a["offsets"][3], 10 + i]).all()
        assert np.isnan(a["h"][a["offsets"][3]:a["offsets"][4], 20 + i]).all()


# combine: instances for 2, 4 and 8 slots, in pieces of a token and whole
@pytest.mark.parametrize("k", [1, 3, 4, 5, 8])
@pytest.mark.parametrize("T,D,act", [(7, 1032, "bf16"), (7, 1032, "f32"), (2100, 520, "bf16"), (2100, 264, "f32")])
def test_combine_slots(T, D, k, act):
    check(T=T, D=D, F=64, n_ffn=6, k=k, act=act, bias="normal")


# pieces of a token where no, some or every zero-computation expert wants x
@pytest.mark.parametrize("n_zero,n_copy,n_const", [(0, 0, 0), (2, 0, 0), (0, 2, 0), (1, 0, 2)])
@pytest.mark.parametrize("T,D,act", [(65, 1032, "bf16"), (1000, 520, "f32")])
def test_combine_pieces(T, D, act, n_zero, n_copy, n_const):
    s = LayerShape("edge", T=T, D=D, F=64, n_ffn=4, n_zero=n_zero, n_copy=n_copy, n_const=n_const, act=act, seed=8100)
    inp = make_inputs(s)
    print("  ", s, check_layer(s, inp, gpu_forward(s, inp)), flush=True)


# wide float32 tiles whose last round runs as halves: (shape, GEMM1, GEMM2); last column tiles of 64 and of 160 columns, groups that
# end anywhere in a tile
F32_HALVES = [(dict(T=1683, D=608, F=1568, n_ffn=4, n_zero=0, n_copy=0, n_const=0), WIDE % "true", PLAIN),
              (dict(T=2048, D=1024, F=2048, n_ffn=8), WIDE % "true", SQUARE % ("false", "2, 4")),
              (dict(T=2507, D=928, F=1888, n_ffn=4, k=4, n_zero=0, n_copy=0, n_const=0), None, WIDE % "false")]


@pytest.mark.parametrize("kw", [i[0] for i in F32_HALVES])
def test_f32_halves_of_wide_tiles(kw):
    s = LayerShape("edge", **dict(dict(n_zero=1, n_copy=1, n_const=2, seed=8100, act="f32"), **kw))
    print("shape", s, flush=True)
    inp = make_inputs(s)
    res = gpu_forward(s, inp)
    print("  ", check_layer(s, inp, res, tok_list=sample_tokens(s, res["topk_idx"], 256)), flush=True)


def test_f32_rows_of_halves_do_not_depend_on_their_neighbours():
    """Three odd tokens (3366 of one slot: 836 to 848 rows per expert): no other token's row changes, nor with operands for
    the float32 instruction in a half."""
    for T in (3366, 3300, 3400):
        test_f32_rows_do_not_depend_on_their_neighbours(T, 608, 1568)


def tile_kinds(rows, cols):
    """{(expert, row block, column tile): run as halves} of the wide tiles of groups of `rows` rows: each of the eight
    XCDs takes a consecutive eighth of the list, row blocks fastest, and what whole rounds of 32 tiles leave there
    runs as halves where it is at most half a round."""
    tiles = [(e, m, n) for e, r in enumerate(rows) for n in range(-(-cols // 256)) for m in range(-(-r // 128))]
    per, kinds = -(-len(tiles) // 8), {}
    for x in range(0, len(tiles), per):
        mine = tiles[x:x + per]
        rest = len(mine) % 32
        for i, tile in enumerate(mine):
            kinds[tile] = 0 < rest <= 16 and i >= len(mine) - rest
    return kinds


# (D, F, slots, tokens, more of them): the last round of the named GEMM's wide tiles runs as halves with the former and whole
# with the latter; four experts, k = 1: token t goes to expert t % 4
F32_HALF_WHOLE = [(608, 1568, 1, 3366, 3700, "h"), (928, 1888, 4, 2900, 3100, "yffn")]


@pytest.mark.parametrize("D,F,k,few,many,name", F32_HALF_WHOLE)
def test_f32_halves_and_whole_tiles_are_the_same_numbers(D, F, k, few, many, name):
    s = LayerShape("edge", T=many, D=D, F=F, n_ffn=4, n_zero=0, n_copy=0, n_const=0, k=k, act="f32", residual=False, seed=8400)
    inp = make_inputs(s)
    if k == 1:
        inp["W_g"][:] = 8.0 * np.eye(4, D, dtype=np.float32)
        inp["x"][:, :4] = np.eye(4, dtype=np.float32)[np.arange(many) % 4]
    got, kinds = [], []
    for T in (few, many):
        r = gpu_forward(s.with_(T=T), dict(inp, x=inp["x"][:T]))
        rows = np.diff(r["offsets"])
        assert rows.sum() == T * k
        kinds.append(tile_kinds(rows, 2 * F if name == "h" else D))
        # the rows of the tokens both calls have, expert by expert
        got.append([(r["src_of"][o:o + n][r["src_of"][o:o + n] < few * k], {q: r[q][o:o + n][r["src_of"][o:o + n] < few * k]
                     for q in ("h", "yffn")}) for o, n in zip(r["offsets"][:-1], rows)])
    both = [t for t in kinds[0] if t in kinds[1]]
    changed = sum(kinds[0][t] != kinds[1][t] for t in both) / len(both)
    print("tiles that change kind", changed, "halves", sum(kinds[0].values()), sum(kinds[1].values()), flush=True)
    assert changed > 0.25
    for (src_a, a), (src_b, b) in zip(*got):
        assert np.array_equal(src_a, src_b)
        for q in ("h", "yffn") if name == "yffn" else ("h",):            # (the other GEMM2 is another kernel in the two calls)
            assert np.array_equal(a[q], b[q]), q


# GEMM2 with the combine in it: (T, D, F = 256 steps of a wave, FFN experts, others each, slots)
DECODE_COMBINE = [(1, 256, 256, 3, 1, 2), (48, 3840, 256, 16, 1, 2), (2, 512, 512, 4, 1, 7), (17, 4096, 768, 8, 2, 4),
                  (33, 4096, 1280, 12, 0, 2),
                  (1, 768, 2048, 16, 1, 2), (5, 3840, 2816, 4, 8, 8), (16, 4096, 4096, 6, 1, 2), (9, 3840, 4352, 2, 1, 3),
                  (9, 6144, 512, 2, 1, 3),
                  (3, 4096, 5632, 4, 1, 2), (2, 3840, 6144, 3, 1, 2)]


@pytest.mark.parametrize("T,D,F,n_ffn,n,k", DECODE_COMBINE)
@pytest.mark.parametrize("tight", [False, True])
def test_decode_with_the_combine(T, D, F, n_ffn, n, k, tight):
    """Against the oracle, and bit by bit what the separate kernels of the step calls give; slots dropped, too."""
    import torch
    from helpers import to_device
    s = LayerShape("edge", T=T, D=D, F=F, n_ffn=n_ffn, n_zero=n, n_copy=n, n_const=n, k=k, bias="normal", seed=8500 + T)
    print("shape", s, flush=True)
    inp = make_inputs(s)
    dev, L = to_device(s, inp), make_layer(s)
    cap = [max(0, c // 2) for c in L.capacity(T, 1.1, 0.75)] if tight else None
    res = gpu_forward(s, inp, layer=L, dev=dev, cap=cap)
    print("  ", check_layer(s, inp, res, cap=None if cap is None else np.array(cap, np.int32)), flush=True)
    packed = L.pack_experts(dev["w1"], dev["w3"], dev["w2"])
    L.route(dev["x"], dev["prev_gate"], dev["W_g"], dev["W_res"], dev["W_c"] if n else None)
    L.permute()
    L.expert_ffn(dev["x"], packed)
    out = L.combine(dev["x"], dev["const_vecs"] if n else None)
    torch.cuda.synchronize()
    assert np.array_equal(out.float().cpu().numpy().astype(np.float64), res["out"])
    R = int(res["offsets"][-1])
    for name, v in L.get_intermediates(R).items():
        assert np.array_equal(v.float().cpu().numpy(), res[name]), name


# SiLU of the float32 and ragged kernels: a wave whose arguments all have |z| <= 87 takes the shorter form. z is exact in
# every kernel (one 1 in x), near 0, up to 87, at the limit and far beyond it, alone and mixed in a wave. float32: e^-z
# and the quotient to 1.5 and 1 ulp of 2^-23 each at most, z = W1 exactly; h is compared where the true value is normal.
@pytest.mark.parametrize("act,D,F", [("f32", 32, 4096), ("f32", 40, 1000), ("bf16", 40, 1000)])
@pytest.mark.parametrize("far", [False, True])
def test_silu_near_and_far(act, D, F, far):
    rng = np.random.default_rng(8400)
    z = np.concatenate([np.exp2(rng.uniform(-20, 6.44, F - 8)) * rng.choice([-1, 1], F - 8),
                        [0.0, 87.0, -87.0, 1e-30, 86.99, -86.99, 0.5, -0.5]])
    if far:
        z[rng.permutation(F)[:F // 64]] = rng.choice([88.0, -88.0, 1e4, -1e4, 3e38, -3e38, 87.5, -87.5], F // 64)
    z = (np.float32(z).view(np.uint32) & (0xFFFF0000 if act == "bf16" else 0xFFFFFFFF)).view(np.float32)
    s = LayerShape("silu2", T=300, D=D, F=F, n_ffn=1, n_zero=0, n_copy=0, n_const=0, k=1, act=act, residual=False, seed=8401)
    inp = make_inputs(s)
    inp["x"][:] = 0.0
    inp["x"][:, 3] = 1.0
    inp["w1"][:] = 0.0
    inp["w1"][0, :, 3] = z
    inp["w3"][:] = 0.0
    inp["w3"][0, :, 3] = 1.0
    inp["w2"][:] = 0.0
    h = np.asarray(gpu_forward(s, inp)["h"], np.float64)
    z = z.astype(np.float64)
    with np.errstate(over="ignore"):
        want = z / (1.0 + np.exp(-z))
    bound = np.abs(want) * (1.0 / 256 if act == "bf16" else 2.5 * 2.0 ** -23) + 2.0 ** -126
    assert np.isfinite(h).all() and (np.abs(h - want) <= bound).all(), np.abs((h - want) / bound).max()


# sums of negative products that all underflow are a zero with its sign: silu(-0) is -0 here and in the plain kernels
def test_silu_keeps_the_sign_of_zero():
    s = LayerShape("silu3", T=300, D=32, F=64, n_ffn=1, n_zero=0, n_copy=0, n_const=0, k=1, act="f32", residual=False, seed=8402)
    inp = make_inputs(s)
    inp["x"][:] = 2.0 ** -100
    inp["w1"][:] = np.where(np.arange(s.F) % 3 == 1, -2.0 ** -100, 2.0 ** -100)[None, :, None]
    inp["w3"][:] = 2.0 ** 100
    a, b = (np.asarray(gpu_forward(s, inp, variant=v)["h"], np.float32) for v in (0, 1))
    print("zeros", (a == 0).all(), (b == 0).all(), "negative", np.signbit(a).sum(), np.signbit(b).sum(), flush=True)
    assert (a == 0).all() and np.signbit(b).any() and np.array_equal(np.signbit(a), np.signbit(b))
