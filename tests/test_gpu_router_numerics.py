"""The end of the routers (softmax, Top-K) on logits that are known exactly: every router the
dispatch can take, by size and type."""
import numpy as np
import pytest

from workloads import LayerShape, make_inputs

from helpers import gpu_forward

pytestmark = pytest.mark.gpu

# (act, T, D, variant).  Few tokens; blocks of 16 tokens in one kernel; slices of 32 columns beyond 64 tokens (wide layers,
# float32 and bf16, a bf16 width that the matrix-core router does not take); the matrix-core router, asked for where
# the automatic choice is another: blocks of 64 tokens, one and two groups of waves, several passes of its
# loop over K tiles, and blocks of 128 tokens (tests/test_dispatch_cpu.py looks at the instances)
MATRIX_CORE = [("bf16", 300, 640, 2), ("bf16", 2100, 768, 2), ("bf16", 2100, 1024, 2), ("bf16", 24576, 512, 0)]
SLICED = [("f32", 100, 1032, 0), ("bf16", 300, 3080, 0), ("bf16", 100, 2048, 0), ("bf16", 300, 4096, 0)]
ROUTERS = [("f32", 40, 64, 0), ("bf16", 40, 512, 0), ("f32", 100, 64, 0), ("bf16", 300, 1000, 0), ("bf16", 100, 768, 0),
           ("bf16", 300, 768, 0)] + SLICED + MATRIX_CORE


def one_hot_shape(act, T, D, **kw):
    kw = dict(dict(n_ffn=6, n_zero=2, n_copy=2, n_const=2, k=8, residual=False, seed=8400), **kw)
    return LayerShape("numerics", T=T, D=D, F=64, act=act, **kw)


def exact_logits(s, inp, col=5):
    """x[t] = 1 + t % 4 in one column, W_g[i] = -2.75 i there: logits -2.75 i (1 + t % 4), exact
    in float32 whatever the order of the sums."""
    inp["x"][:] = 0.0
    inp["x"][:, col] = 1.0 + np.arange(s.T) % 4
    inp["W_g"][:] = 0.0
    inp["W_g"][:, col] = -2.75 * np.arange(s.N)
    return -2.75 * np.arange(s.N)[None, :] * (1.0 + np.arange(s.T) % 4)[:, None]


@pytest.mark.parametrize("act,T,D,variant", ROUTERS)
def test_softmax_is_accurate_to_float32(act, T, D, variant):
    """Relative error, weight by weight, down to logits 77 apart: expf within 1 ulp (2^-23) in
    numerator and sum, N / 4 + 2 additions and a division of half an ulp each."""
    s = one_hot_shape(act, T, D)
    inp = make_inputs(s)
    L = exact_logits(s, inp)
    res = gpu_forward(s, inp, variant, balance_tau=0.75, intermediates=False)
    assert np.array_equal(res["out_gate"].astype(np.float64), L)
    assert np.array_equal(res["topk_idx"], np.tile(np.arange(s.k), (T, 1)))
    p = np.exp(L)                                   # the largest logit is 0
    p /= p.sum(axis=1, keepdims=True)
    bound = (2 + (s.N // 4 + 2 + 1) / 2) * 2.0 ** -23
    e_w = (np.abs(res["topk_w"] - p[:, :s.k]) / p[:, :s.k]).max()
    P = p.mean(axis=0)
    e_P = (np.abs(res["P"] - P) / P).max()
    print("router", act, T, D, "topk_w", e_w, "P", e_P, "bound", bound, flush=True)
    assert e_w <= bound
    assert e_P <= bound + 2.0 ** -24                # (added up in float64, rounded once)


# (variant 1: the router with one wave per token)
@pytest.mark.parametrize("act,T,D,variant", ROUTERS + [("f32", 40, 64, 1), ("bf16", 300, 512, 1)])
def test_a_nan_token_stays_alone(act, T, D, variant):
    """A NaN in one row of x makes all its logits NaN.  Its slots still go to k different experts
    (the lowest indices, as with equal logits), the counts add up, and every other token gets the
    bits it gets beside a token of zeros, whose logits are equal.  k > ceil(N / 4): the four
    threads of a token hold two experts each."""
    s = one_hot_shape(act, T, D, n_ffn=4, n_zero=1, n_copy=1, k=3)
    assert s.N == 8
    inp = make_inputs(s)
    t = T // 2 + 1
    inp["x"][t] = 0.0
    ref = gpu_forward(s, inp, variant, intermediates=False)
    inp["x"][t, 9] = np.nan
    res = gpu_forward(s, inp, variant, intermediates=False)
    print("nan token", act, T, D, res["topk_idx"][t].tolist(), res["counts"].tolist(), flush=True)
    assert res["topk_idx"][t].tolist() == [0, 1, 2]
    assert res["counts"].sum() == T * s.k
    for name in ("counts", "offsets", "row_of", "topk_idx"):
        assert np.array_equal(res[name], ref[name]), name
    others = np.arange(T) != t
    for name in ("out", "out_gate", "topk_w"):
        assert np.array_equal(res[name][others], ref[name][others]), name
        assert np.isnan(res[name][t]).all(), name


@pytest.mark.parametrize("act,T,D,variant", ROUTERS + [("f32", 40, 64, 1), ("bf16", 300, 512, 1)])
def test_masked_experts(act, T, D, variant):
    """A bias of -infinity on all experts but one: it takes weight 1, the other slots go to the
    masked experts of the lowest indices, each once, with weight 0."""
    s = one_hot_shape(act, T, D)
    inp = make_inputs(s)
    exact_logits(s, inp)
    inp["bias"] = np.full(s.N, -np.inf, np.float32)
    inp["bias"][4] = 0.0
    res = gpu_forward(s, inp, variant, intermediates=False)
    order = [4] + [i for i in range(s.N) if i != 4]
    assert np.array_equal(res["topk_idx"], np.tile(order[:s.k], (T, 1)))
    assert np.array_equal(res["topk_w"], np.tile([1.0] + [0.0] * (s.k - 1), (T, 1)))
    assert np.isfinite(res["out"]).all()


@pytest.mark.parametrize("act,T,D,variant", ROUTERS + [("bf16", 300, 512, 1)])
def test_infinite_router_operands(act, T, D, variant):
    """W_g = -infinity for one expert in a column where x is positive takes that expert out of the
    race, W_g = +infinity gives an infinite logit, and an infinite activation infinite logits of the
    weights' signs: not NaN, and nothing else changes."""
    s = one_hot_shape(act, T, D)
    inp = make_inputs(s)
    L = exact_logits(s, inp)
    inp["x"][:, 7] = 0.5
    inp["W_g"][3, 7] = -np.inf
    res = gpu_forward(s, inp, variant, intermediates=False)
    L[:, 3] = -np.inf
    assert np.array_equal(res["out_gate"].astype(np.float64), L)
    assert np.array_equal(res["topk_idx"], np.tile([i for i in range(s.N) if i != 3][:s.k], (T, 1)))
    assert np.isfinite(res["topk_w"]).all() and np.isfinite(res["out"]).all()
    inp["W_g"][3, 7] = np.inf
    res = gpu_forward(s, inp, variant, intermediates=False)
    assert np.all(res["out_gate"][:, 3] == np.inf) and np.all(res["topk_idx"][:, 0] == 3)
    inp["W_g"][3, 7] = 0.0
    sign = np.where(np.arange(s.N) % 3 == 1, -1.0, 1.0)
    inp["W_g"][:, 11] = 0.25 * sign
    inp["x"][T // 2, 11] = np.inf
    L = -2.75 * np.arange(s.N)[None, :] * (1.0 + np.arange(T) % 4)[:, None]
    L[T // 2] = np.inf * sign
    res = gpu_forward(s, inp, variant, intermediates=False)
    assert np.array_equal(res["out_gate"].astype(np.float64), L)


# (every router, the matrix-core one for one and two blocks of weight rows, and the few-token one in one
# workgroup)
@pytest.mark.parametrize("act,T,D,variant,n_ffn", [r + (6,) for r in ROUTERS] + [
    ("bf16", 300, 512, 2, 6), ("bf16", 300, 512, 2, 34), ("bf16", 300, 640, 2, 34), ("bf16", 2100, 768, 2, 34), ("bf16", 3, 64, 0, 6),
    ("f32", 3, 512, 0, 6)])
def test_infinite_previous_logits_stay_with_their_token(act, T, D, variant, n_ffn):
    """The gating residual is added to the logits of its own token and to nothing else: not to another
    token's, and not to the logits of the constant experts (a1)."""
    s = one_hot_shape(act, T, D, n_ffn=n_ffn, residual=True)
    inp = make_inputs(s)
    ref = gpu_forward(s, inp, variant)
    t = T // 2
    inp["prev_gate"][t, 1] = -np.inf
    inp["prev_gate"][t, 2] = np.nan
    res = gpu_forward(s, inp, variant)
    assert np.isnan(res["out_gate"][t]).all()
    others = np.arange(T) != t
    for name in ("out_gate", "topk_idx", "topk_w"):
        assert np.array_equal(res[name][others], ref[name][others]), name
    assert np.array_equal(res["alpha1"], ref["alpha1"])


# NaN of both signs, and with nothing but the lowest bits of the significand set
NANS = np.array([0x7fc00000, 0xffc00000, 0x7f800001, 0xff80ffff], np.uint32).view(np.float32)


@pytest.mark.parametrize("act,T,D,variant", ROUTERS + [("bf16", 3, 64, 0), ("bf16", 300, 512, 1)])
def test_nan_weights(act, T, D, variant):
    """A NaN among the weights of an expert makes its logit NaN, whatever the NaN's bits, and nothing
    else; a NaN in W_c the a1 of its constant expert."""
    s = one_hot_shape(act, T, D)
    inp = make_inputs(s)
    L = exact_logits(s, inp)
    inp["x"][:, 7] = 0.5
    inp["W_c"][:, :, 7] = 0.0
    ref = gpu_forward(s, inp, variant)
    for i, nan in enumerate(NANS):
        inp["W_g"][1 + 2 * i, 7] = nan
        L[:, 1 + 2 * i] = np.nan
        inp["W_c"][1, 1, 7] = nan
        res = gpu_forward(s, inp, variant)
        assert np.array_equal(res["out_gate"].astype(np.float64), L, equal_nan=True), hex(nan.view(np.uint32))
        assert np.isnan(res["topk_w"]).all()
        assert np.array_equal(res["alpha1"][:, 0], ref["alpha1"][:, 0])
        assert np.isnan(res["alpha1"][:, 1]).all()


# (every router but the matrix-core one, whose three bf16 pieces of a weight end at 2^-133)
@pytest.mark.parametrize("exponent", [-118, -130, -145])
@pytest.mark.parametrize("act,T,D,variant", [r for r in ROUTERS if r not in MATRIX_CORE] +
                         [("bf16", 3, 64, 0), ("bf16", 1500, 1536, 0), ("bf16", 300, 512, 1)])
def test_small_weights_keep_their_bits(act, T, D, variant, exponent):
    """Logits of one product each, of a weight with all its significand bits down to the smallest
    float32 and a small integer: the product rounded to float32 once."""
    s = one_hot_shape(act, T, D)
    inp = make_inputs(s)
    exact_logits(s, inp)
    w = np.ldexp(1.0 + (2 * np.arange(s.N) + 1) * 0.0713, exponent).astype(np.float32)
    inp["W_g"][:, 5] = w
    res = gpu_forward(s, inp, variant, intermediates=False)
    want = (w[None, :] * inp["x"][:, 5:6].astype(np.float64)).astype(np.float32)
    assert np.array_equal(res["out_gate"], want)


# the matrix-core router with two blocks of 32 weight rows: one and two groups of waves, one and several passes
TWO_BLOCKS = [(300, 512), (300, 640), (2100, 768), (2100, 1024), (2100, 1408)]


@pytest.mark.parametrize("T,D", TWO_BLOCKS)
def test_two_blocks_of_weight_rows(T, D, variant=2, act="bf16"):
    """Exact logits -i (1 + t % 4) / 4 of 40 experts: the softmax as accurate as with one block, and infinite
    and NaN weights of experts in the second block stay where they are."""
    s = one_hot_shape(act, T, D, n_ffn=34)
    assert s.N == 40
    inp = make_inputs(s)
    exact_logits(s, inp)
    inp["W_g"][:, 5] = -0.25 * np.arange(s.N)
    inp["x"][:, 7] = 0.5
    L = -0.25 * np.arange(s.N)[None, :] * (1.0 + np.arange(T) % 4)[:, None]
    res = gpu_forward(s, inp, variant, intermediates=False)
    assert np.array_equal(res["out_gate"].astype(np.float64), L)
    assert np.array_equal(res["topk_idx"], np.tile(np.arange(s.k), (T, 1)))
    p = np.exp(L)
    p /= p.sum(axis=1, keepdims=True)
    err = (np.abs(res["topk_w"] - p[:, :s.k]) / p[:, :s.k]).max()
    print("router", T, D, "topk_w", err, flush=True)
    assert err <= (2 + (s.N // 4 + 2 + 1) / 2) * 2.0 ** -23
    inp["W_g"][33, 7] = np.inf
    inp["W_g"][36, 7] = -np.inf
    res = gpu_forward(s, inp, variant, intermediates=False)
    L[:, 33], L[:, 36] = np.inf, -np.inf
    assert np.array_equal(res["out_gate"].astype(np.float64), L)
    assert np.all(res["topk_idx"][:, 0] == 33)
    for nan in NANS:
        inp["W_g"][33, 7], inp["W_g"][36, 7] = 0.0, nan
        res = gpu_forward(s, inp, variant, intermediates=False)
        L[:, 33], L[:, 36] = -0.25 * 33 * (1.0 + np.arange(T) % 4), np.nan
        assert np.array_equal(res["out_gate"].astype(np.float64), L, equal_nan=True)
