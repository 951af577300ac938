"""The split-int8 general forward over pairs a <= b (t and its swapped copy stacked)
against the NumPy model of the digit scheme and the oracle, through the C ABI."""
import numpy as np
import pytest

import oracle
from paper_2310_04559_amd.inputs import integer_inputs, random_general
from tests import split_model
from tests.gpu_common import announce, dev, host, rel_fro

pytestmark = pytest.mark.gpu
I8 = 3


def _run(native, L, t, R0, **kw):
    import torch

    R = dev(R0)
    native.cc_ladder_residual(dev(L), dev(t), R, I8, opts=native.make_opts(**kw))
    torch.cuda.synchronize()
    return host(R)


# v^2 within one chunk of 16384 contracted indices: the swapped rows carry the same
# digits and exponents as the direct scheme's, so the model's sums come out to the
# rounding of the drains; odd v, 2 o^2 past one tile, one and two blocks
@pytest.mark.parametrize("o,v,P,a_block", [(4, 64, 70, 0), (9, 67, 33, 0), (3, 71, 20, 40)])
@pytest.mark.parametrize("exchange", [False, True])
@pytest.mark.parametrize("slices,depth", [(5, 1), (4, 2)])
def test_stacked_matches_the_model(gpu_lib, o, v, P, a_block, exchange, slices, depth):
    announce("i8-stacked", o, v, P, "a_block", a_block, "exchange", exchange, slices, depth)
    L, t, _ = random_general(o, v, P, 5000 + o + v)
    x = np.ascontiguousarray(t.transpose(0, 1, 3, 2)) if exchange else t
    R0 = np.random.default_rng(25).standard_normal(t.shape)
    got = _run(gpu_lib, L, t, R0, a_block=a_block, exchange=exchange, split_slices=slices,
               split_depth=depth)
    assert rel_fro(got - R0, split_model.ladder_i8(L, x, slices, depth)) < 1e-12


def test_stacked_two_chunks_and_integers(gpu_lib):
    # v = 130: two chunks of contracted indices, whose digits the swap regroups
    announce("i8-stacked-chunks")
    L, t, _ = random_general(4, 130, 9, 5100)
    err = rel_fro(_run(gpu_lib, L, t, np.zeros_like(t)), oracle.ladder_forward(L, t))
    assert err < 1e-9
    L, t = integer_inputs(3, 72, 5, 5101)
    assert np.array_equal(_run(gpu_lib, L, t, np.zeros_like(t)), oracle.ladder_forward(L, t))
