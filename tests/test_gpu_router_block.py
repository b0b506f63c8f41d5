"""The router that takes a block of 16 or 32 tokens per workgroup, at the edges of its blocks and of its rule, against the
oracle, and what tests/test_gpu_router_numerics.py asks of every router.  Needs a real MI355X: run with -m gpu."""
import numpy as np
import pytest

import test_gpu_router_numerics as numerics
from helpers import check_layer, gpu_forward, make_layer
from test_gpu_parity import say, small_shape
from workloads import make_inputs

pytestmark = pytest.mark.gpu

# (type, tokens, columns, FFN experts, others each, slots) -> tokens of a workgroup, blocks of 16 weight rows, waves, sets of
# sums; one more slice than whole rounds of the waves, one wave with work, a chunk of 16 slots
BLOCK = [("f32", 65, 256, 4, 1, 2, (16, 1, 16, 2)), ("f32", 4096, 264, 4, 1, 3, (16, 1, 16, 2)),
         ("f32", 333, 1024, 7, 1, 2, (16, 1, 16, 2)),
         ("f32", 256, 8, 4, 1, 2, (16, 1, 16, 2)), ("f32", 777, 512, 16, 2, 1, (16, 2, 8, 2)),
         ("f32", 70, 40, 20, 1, 4, (16, 2, 8, 2)),
         ("f32", 4081, 520, 10, 2, 2, (16, 2, 16, 2)), ("f32", 300, 1000, 20, 2, 3, (16, 2, 16, 2)),
         ("f32", 1025, 512, 48, 2, 8, (16, 4, 8, 2)),
         ("f32", 4095, 288, 29, 1, 2, (16, 4, 8, 2)),
         ("bf16", 97, 264, 8, 1, 2, (16, 1, 8, 1)), ("bf16", 1999, 1000, 8, 1, 8, (16, 1, 16, 2)),
         ("bf16", 2050, 4096, 8, 1, 2, (16, 1, 16, 2)),
         ("bf16", 2305, 256, 8, 1, 2, (16, 1, 8, 1)), ("bf16", 2305, 384, 14, 1, 4, (16, 2, 8, 1)),
         ("bf16", 65, 8, 16, 1, 2, (16, 2, 8, 1)),
         ("bf16", 4096, 1024, 16, 2, 2, (16, 2, 8, 1)), ("bf16", 300, 1000, 20, 2, 1, (16, 2, 16, 2)),
         ("bf16", 1536, 2048, 18, 2, 3, (16, 2, 16, 2)),
         ("bf16", 4095, 768, 32, 2, 2, (16, 4, 8, 1)), ("bf16", 257, 776, 40, 2, 8, (16, 4, 8, 2)), ("bf16", 2048, 1024, 30, 2, 2, (16, 4, 8, 2)),
         ("bf16", 2311, 256, 48, 1, 8, (16, 4, 8, 1)),
         ("bf16", 300, 512, 48, 3, 2, (16, 4, 8, 1)), ("bf16", 4353, 256, 3, 1, 2, (32, 1, 8, 1)),
         ("bf16", 4097, 504, 3, 1, 2, (32, 1, 8, 1)),
         ("bf16", 8191, 256, 16, 1, 8, (32, 2, 8, 1)), ("bf16", 4400, 640, 32, 3, 2, (32, 4, 8, 1)),
         ("bf16", 8192, 1408, 30, 2, 1, (32, 4, 8, 1))]
# all there are
INSTANCES = {("f32", 16, 1, 16, 2), ("f32", 16, 2, 8, 2), ("f32", 16, 2, 16, 2), ("f32", 16, 4, 8, 2),
             ("bf16", 16, 1, 8, 1), ("bf16", 16, 1, 16, 2),
             ("bf16", 16, 2, 8, 1), ("bf16", 16, 2, 16, 2), ("bf16", 16, 4, 8, 1), ("bf16", 16, 4, 8, 2),
             ("bf16", 32, 1, 8, 1),
             ("bf16", 32, 2, 8, 1), ("bf16", 32, 4, 8, 1)}


@pytest.mark.parametrize("act,T,D,n_ffn,n_other,k,inst", BLOCK)
@pytest.mark.parametrize("residual", [True, False])
def test_blocks_against_the_oracle(act, T, D, n_ffn, n_other, k, inst, residual):
    """Logits, weights, a1, the permutation of the histogram the blocks leave (also under capacities), the statistics."""
    s = small_shape("block", T=T, D=D, F=64, act=act, n_ffn=n_ffn, n_zero=n_other, n_copy=n_other, n_const=n_other, k=k,
                    residual=residual, bias="normal" if residual else "none", seed=T + D)
    inp = make_inputs(s)
    L = make_layer(s)
    cap = L.capacity(s.T, 1.1, 0.75) if k <= 2 else None
    res = gpu_forward(s, inp, layer=L, cap=cap, balance_tau=0.75)
    say("  ", check_layer(s, inp, res, cap=None if cap is None else np.array(cap, np.int32), balance_tau=0.75))


@pytest.mark.parametrize("act,T,D", [("f32", 100, 512), ("bf16", 300, 1000), ("bf16", 2400, 512), ("bf16", 4400, 512),
                                     ("f32", 300, 1024), ("bf16", 300, 640), ("bf16", 2100, 1024), ("bf16", 4097, 72)])
def test_numbers_of_the_other_routers(act, T, D):
    numerics.test_softmax_is_accurate_to_float32(act, T, D, 0)
    numerics.test_a_nan_token_stays_alone(act, T, D, 0)
    numerics.test_masked_experts(act, T, D, 0)
    numerics.test_infinite_router_operands(act, T, D, 0)
    numerics.test_infinite_previous_logits_stay_with_their_token(act, T, D, 0, 6)
    numerics.test_nan_weights(act, T, D, 0)
    numerics.test_small_weights_keep_their_bits(act, T, D, 0, -130)


@pytest.mark.parametrize("T,D", [(2400, 512), (4400, 512), (300, 640), (300, 776)])
def test_more_than_32_experts(T, D):
    numerics.test_two_blocks_of_weight_rows(T, D, 0)
    numerics.test_infinite_previous_logits_stay_with_their_token("bf16", T, D, 0, 34)


def test_more_than_32_experts_in_float32():
    numerics.test_two_blocks_of_weight_rows(300, 512, 0, "f32")
    numerics.test_infinite_previous_logits_stay_with_their_token("f32", 300, 512, 0, 34)
