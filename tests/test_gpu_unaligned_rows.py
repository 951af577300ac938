"""GPU parity of large products on rows that are not 16-byte aligned (odd v, odd o^2):
the dword loads of the direct-to-LDS kernels on each of their tiles, through the C ABI."""
import numpy as np
import pytest

import oracle
from paper_2310_04559_amd.inputs import random_general
from tests.gpu_common import TOL, announce, dev, host, rel_fro

pytestmark = pytest.mark.gpu

# v^2 = 3969 or 3721 columns and K (1 and 9 past whole K-steps; o^2 = 441 and 2025 as K of
# the hole-hole ladder leave 9 of 16): 64 x 128 tiles (o^2 = 400, 441; float32 pairs 64 x 64)
# and 128 x 256 (2025, 2116), which do not divide the output
FORWARD = [(20, 63, 30), (46, 61, 17)]
HOLE = [(21, 63, 17), (45, 61, 17)]


@pytest.mark.parametrize("o,v,P", FORWARD)
@pytest.mark.parametrize("flags", [{}, {"pair_symmetric": True}])
def test_unaligned_forward(gpu_lib, o, v, P, flags):
    import torch

    announce("unaligned-forward", o, v, P, flags)
    L, t, _ = random_general(o, v, P, 3300 + o)
    if flags:
        t = 0.5 * (t + t.transpose(1, 0, 3, 2))
    R0 = np.random.default_rng(22).standard_normal(t.shape)
    ref = oracle.ladder_forward(L, t)
    for precision in (0, 1):
        R = dev(R0)
        gpu_lib.cc_ladder_residual(dev(L), dev(t), R, precision, opts=gpu_lib.make_opts(**flags))
        torch.cuda.synchronize()
        assert rel_fro(host(R) - R0, ref) < TOL[precision], precision


@pytest.mark.parametrize("o,v,P", FORWARD[:1])
def test_unaligned_backward(gpu_lib, o, v, P):
    import torch

    announce("unaligned-backward", o, v, P)
    L, t, lam = random_general(o, v, P, 3400 + o)
    dL_ref, dt_ref = oracle.ladder_backward(L, t, lam)
    for precision in (0, 1):
        dL, dt = dev(np.zeros_like(L)), dev(np.zeros_like(t))
        gpu_lib.cc_ladder_backward(dev(L), dev(t), dev(lam), dL, dt, precision)
        torch.cuda.synchronize()
        assert rel_fro(host(dL), dL_ref) < TOL[precision], precision
        assert rel_fro(host(dt), dt_ref) < TOL[precision], precision


@pytest.mark.parametrize("o,v,P", HOLE)
def test_unaligned_hole_ladder(gpu_lib, o, v, P):
    import torch

    announce("unaligned-hole", o, v, P)
    _, t, R0 = random_general(o, v, P, 3500 + o)
    Loo = np.random.default_rng(23).standard_normal((P, o, o))
    ref = oracle.hole_ladder(Loo, t)
    for precision in (0, 1):
        R = dev(R0)
        gpu_lib.cc_hole_ladder(dev(Loo), dev(t), R, precision)
        torch.cuda.synchronize()
        assert rel_fro(host(R) - R0, ref) < TOL[precision], precision
