"""The float64 forward folded over the exchange of both virtual pairs against the
oracle: any vectors and amplitudes, one and several blocks, through the C ABI."""
import numpy as np
import pytest

import oracle
from paper_2310_04559_amd.inputs import integer_inputs, random_general
from tests.gpu_common import TOL, announce, dev, host, rel_fro

pytestmark = pytest.mark.gpu


def _run(native, L, t, R0, **kw):
    import torch

    seen = []
    fn = native.TRACE_FN(lambda user, phase, block, end, stream: seen.append((phase, block, end)))
    R = dev(R0)
    native.cc_ladder_residual(dev(L), dev(t), R, 0, opts=native.make_opts(trace=fn, **kw))
    torch.cuda.synchronize()
    # the folded route is the one that prepares amplitudes in the float64 form
    return host(R), (0, 0, 1) in seen, 1 + max(b for p, b, _ in seen if p == 2)


# v from the smallest folded size on, odd and even; the scratch of 30 virtuals
# (a_block) holds three folded blocks, that of one or seven virtuals none worth it (the
# direct route, whose flags are tested with it)
FOLDED = [(20, 64, 100, 0), (9, 71, 263, 0), (16, 72, 20, 30), (12, 81, 50, 30)]
DIRECT = [(9, 71, 60, 1), (16, 64, 200, 7), (20, 63, 100, 0)]


@pytest.mark.parametrize("o,v,P,a_block,folded,exchange,pairsym",
                         [(*c, True, x, p) for c in FOLDED for x in (False, True)
                          for p in (False, True)] +
                         [(*c, False, False, False) for c in DIRECT])
def test_folded_forward(gpu_lib, o, v, P, a_block, folded, exchange, pairsym):
    announce("fold", o, v, P, "a_block", a_block, "exchange", exchange, "pairsym", pairsym)
    L, t, _ = random_general(o, v, P, 4000 + o + v)
    if pairsym:
        t = 0.5 * (t + t.transpose(1, 0, 3, 2))
    R0 = np.random.default_rng(22).standard_normal(t.shape)
    got, prep, blocks = _run(gpu_lib, L, t, R0, a_block=a_block, exchange=exchange,
                             pair_symmetric=pairsym)
    ref = oracle.exchange_forward(L, t) if exchange else oracle.ladder_forward(L, t)
    assert rel_fro(got - R0, ref) < TOL[0]
    if not pairsym and not exchange:
        assert prep == folded
        assert blocks == 3 or not (folded and a_block)


def test_folded_forward_integer_exact(gpu_lib):
    # halves of integer sums below 2**53 are exact
    announce("fold-int")
    L, t = integer_inputs(16, 72, 20, 4100)
    got, prep, _ = _run(gpu_lib, L, t, np.zeros_like(t))
    assert prep and np.array_equal(got, oracle.ladder_forward(L, t))


def test_folded_forward_non_finite_rows_stay_apart(gpu_lib):
    # an infinite amplitude spoils its own (i, j) and no other; there nothing is finite
    announce("fold-inf")
    L, t, _ = random_general(16, 72, 20, 4200)
    t[1, 2, 3, 5] = np.inf
    got, prep, _ = _run(gpu_lib, L, t, np.zeros_like(t))
    ok = np.ones((16, 16), dtype=bool)
    ok[1, 2] = False
    assert prep
    assert np.isfinite(got[ok]).all() and not np.isfinite(got[1, 2]).any()
    t[1, 2, 3, 5] = 0.0
    assert rel_fro(got[ok], oracle.ladder_forward(L, t)[ok]) < TOL[0]


# the folded adjoint: even and odd v (the odd one copies L to aligned rows), more and
# fewer rows than one tile; a_block = 40 holds W in two blocks and keeps the direct route
@pytest.mark.parametrize("o,v,P,a_block", [(6, 64, 30, 0), (13, 71, 41, 0), (3, 97, 12, 0),
                                           (6, 64, 30, 40)])
@pytest.mark.parametrize("exchange", [False, True])
def test_folded_backward(gpu_lib, o, v, P, a_block, exchange):
    import torch

    announce("fold-backward", o, v, P, "a_block", a_block, "exchange", exchange)
    L, t, lam = random_general(o, v, P, 4300 + o + v)
    dL0 = np.random.default_rng(23).standard_normal(L.shape)
    dt0 = np.random.default_rng(24).standard_normal(t.shape)
    dL, dt = dev(dL0), dev(dt0)
    gpu_lib.cc_ladder_backward(dev(L), dev(t), dev(lam), dL, dt, 0,
                               opts=gpu_lib.make_opts(a_block=a_block, exchange=exchange))
    torch.cuda.synchronize()
    ref = oracle.exchange_backward(L, t, lam) if exchange else oracle.ladder_backward(L, t, lam)
    assert rel_fro(host(dL) - dL0, ref[0]) < TOL[0]
    assert rel_fro(host(dt) - dt0, ref[1]) < TOL[0]


def test_folded_backward_integer_exact(gpu_lib):
    import torch

    announce("fold-backward-int")
    L, t = integer_inputs(5, 66, 7, 4400)
    lam = integer_inputs(5, 66, 7, 4401)[1]
    dL, dt = dev(np.zeros_like(L)), dev(np.zeros_like(t))
    gpu_lib.cc_ladder_backward(dev(L), dev(t), dev(lam), dL, dt, 0)
    torch.cuda.synchronize()
    dL_ref, dt_ref = oracle.ladder_backward(L, t, lam)
    assert np.array_equal(host(dL), dL_ref) and np.array_equal(host(dt), dt_ref)


# pair-symmetric t and lam: rows i <= j (none i < j at o = 1), gathered from the
# pair-pair integral with symmetric vectors; v from the smallest folded size on, odd and
# even; a_block = 20 keeps the direct route
@pytest.mark.parametrize("o,v,P,a_block", [(5, 16, 20, 0), (1, 21, 9, 0), (7, 33, 41, 0),
                                           (12, 64, 30, 0), (5, 40, 20, 20)])
@pytest.mark.parametrize("exchange", [False, True])
@pytest.mark.parametrize("symv", [False, True])
def test_folded_pair_symmetric_backward(gpu_lib, o, v, P, a_block, exchange, symv):
    import torch

    announce("fold-backward-pairsym", o, v, P, "a_block", a_block, exchange, "symv", symv)
    L, t, lam = random_general(o, v, P, 4500 + o + v)
    t, lam = (0.5 * (x + x.transpose(1, 0, 3, 2)) for x in (t, lam))
    if symv:
        L = 0.5 * (L + L.transpose(0, 2, 1))
    dL0 = np.random.default_rng(26).standard_normal(L.shape)
    dt0 = np.random.default_rng(27).standard_normal(t.shape)
    dL, dt = dev(dL0), dev(dt0)
    gpu_lib.cc_ladder_backward(dev(L), dev(t), dev(lam), dL, dt, 0,
                               opts=gpu_lib.make_opts(a_block=a_block, exchange=exchange,
                                                      pair_symmetric=True, symmetric_vectors=symv))
    torch.cuda.synchronize()
    ref = oracle.exchange_backward(L, t, lam) if exchange else oracle.ladder_backward(L, t, lam)
    assert rel_fro(host(dL) - dL0, ref[0]) < TOL[0]
    assert rel_fro(host(dt) - dt0, ref[1]) < TOL[0]
