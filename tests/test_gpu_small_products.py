"""GPU parity of products on the small-grid kernels (register-direct waves with K
shared between them, 64-row direct-to-LDS tiles) at their edges, through the C ABI."""
import numpy as np
import pytest

import oracle
from paper_2310_04559_amd.inputs import random_general
from tests.gpu_common import TOL, announce, dev, host, rel_fro

pytestmark = pytest.mark.gpu

# o^2 rows x v^2 (or pair) columns: 400 x 4096 takes 64 x 128 tiles, its pairs 64 x 64
# where rows are aligned; odd v reads unaligned rows and, row-contiguous, a last
# column that has no pair; o = 1 and v = 2, 3 leave most of a sub-tile empty; P = 17 is
# one K-step and a remainder, v^2 = 1600 and 1681 = 105 * 16 + 1 share K between waves
SHAPES = [(20, 64, 30), (7, 63, 17), (1, 2, 5), (2, 3, 17), (6, 40, 64), (6, 41, 33), (11, 32, 49)]


@pytest.mark.parametrize("o,v,P", SHAPES)
@pytest.mark.parametrize("flags", [{}, {"pair_symmetric": True},
                                   {"pair_symmetric": True, "plus_minus": True}])
def test_small_forward(gpu_lib, o, v, P, flags):
    import torch

    announce("small-forward", o, v, P, flags)
    L, t, _ = random_general(o, v, P, 3000 + o + v)
    if flags:
        t = 0.5 * (t + t.transpose(1, 0, 3, 2))
    R0 = np.random.default_rng(21).standard_normal(t.shape)
    ref = oracle.ladder_forward(L, t)
    for precision in (0, 1):
        R = dev(R0)
        gpu_lib.cc_ladder_residual(dev(L), dev(t), R, precision, opts=gpu_lib.make_opts(**flags))
        torch.cuda.synchronize()
        assert rel_fro(host(R) - R0, ref) < TOL[precision], precision


@pytest.mark.parametrize("o,v,P", SHAPES)
def test_small_backward(gpu_lib, o, v, P):
    import torch

    announce("small-backward", o, v, P)
    L, t, lam = random_general(o, v, P, 3100 + o + v)
    dL_ref, dt_ref = oracle.ladder_backward(L, t, lam)
    for precision in (0, 1):
        dL, dt = dev(np.zeros_like(L)), dev(np.zeros_like(t))
        gpu_lib.cc_ladder_backward(dev(L), dev(t), dev(lam), dL, dt, precision)
        torch.cuda.synchronize()
        assert rel_fro(host(dL), dL_ref) < TOL[precision], precision
        assert rel_fro(host(dt), dt_ref) < TOL[precision], precision


@pytest.mark.parametrize("o,v,P", [(6, 44, 70), (6, 45, 70), (4, 50, 530)])
def test_float32_symmetric_build_is_the_blocked_one(gpu_lib, o, v, P):
    # one block forms half the integral and mirrors it, and pads odd rows; blocks of 4
    # virtuals form all of it: the same float32 sums, so the same bits (P = 530: two
    # drain chunks of the build)
    import torch

    announce("float32-symmetric-build", o, v, P)
    L, t, _ = random_general(o, v, P, 3200 + v)
    got = []
    for a_block in (0, 4):
        R = dev(np.zeros_like(t))
        gpu_lib.cc_ladder_residual(dev(L), dev(t), R, 1, opts=gpu_lib.make_opts(a_block=a_block))
        torch.cuda.synchronize()
        got.append(host(R))
    assert np.array_equal(got[0], got[1])
