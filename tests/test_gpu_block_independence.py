"""R bit for bit independent of how the integral is cut into blocks, through the C ABI:
every sum over the contracted indices is formed in one order that the sizes fix."""
import numpy as np
import pytest

import oracle
from paper_2310_04559_amd.inputs import random_general
from tests.gpu_common import TOL, announce, dev, host, rel_fro

pytestmark = pytest.mark.gpu


def _residual(native, Ld, td, precision, **kw):
    import torch

    R = torch.zeros_like(td)
    native.cc_ladder_residual(Ld, td, R, precision, opts=native.make_opts(**kw))
    torch.cuda.synchronize()
    return R


# one block against several of the +- forward with symmetric vectors: K in one range and
# in several, scratch beside the packed vectors for all rows of the products and for few
# of them (P of 2 and 4)
@pytest.mark.parametrize("o,v,P,precision", [(9, 71, 263, 0), (13, 97, 341, 0), (13, 97, 341, 1),
                                             (12, 40, 60, 0), (12, 40, 60, 1), (30, 33, 2, 0),
                                             (20, 33, 4, 1), (1, 35, 9, 0)])
@pytest.mark.parametrize("exchange", [False, True])
def test_plus_minus_symmetric_vectors(gpu_lib, o, v, P, precision, exchange):
    import torch

    announce("blocks-pm-symv", o, v, P, "precision", precision, "exchange", exchange)
    L, t, _ = random_general(o, v, P, 6000 + o + v)
    L = 0.5 * (L + L.transpose(0, 2, 1))
    t = 0.5 * (t + t.transpose(1, 0, 3, 2))
    Ld, td = dev(L), dev(t)
    kw = dict(pair_symmetric=True, plus_minus=True, symmetric_vectors=True, exchange=exchange)
    one = _residual(gpu_lib, Ld, td, precision, **kw)
    ref = oracle.exchange_forward(L, t) if exchange else oracle.ladder_forward(L, t)
    assert rel_fro(host(one), ref) < TOL[precision]
    for a_block in (v - 1, v // 2, v // 5):
        assert torch.equal(_residual(gpu_lib, Ld, td, precision, a_block=a_block, **kw), one), a_block


# long rows: the two products of one block in a launch each, on tiles of 160 and 128 rows,
# against blocks in one launch; and, of few vectors in several blocks, cut once more into
# virtuals whose partial sums the packed vectors' room holds
@pytest.mark.parametrize("o,v,P,symv", [(16, 256, 3, False), (16, 261, 40, True), (25, 256, 30, True)])
def test_plus_minus_long_rows(gpu_lib, o, v, P, symv):
    import torch

    announce("blocks-pm-long", o, v, P, "symv", symv)
    L, t, _ = random_general(o, v, P, 6050 + o + v)
    L = 0.5 * (L + L.transpose(0, 2, 1))
    t = 0.5 * (t + t.transpose(1, 0, 3, 2))
    Ld, td = dev(L), dev(t)
    kw = dict(pair_symmetric=True, plus_minus=True, symmetric_vectors=symv)
    one = _residual(gpu_lib, Ld, td, 0, **kw)
    pairs = [(0, 0), (v - 1, v - 1), (0, v - 1), (v - 1, 0), (127, 128), (v // 2, 3), (31, 32), (200, 77)]
    ref = np.stack(list(oracle.ladder_pairs(L, t, pairs)))
    got = one[:, :, [a for a, _ in pairs], [b for _, b in pairs]].permute(2, 0, 1)
    assert rel_fro(host(got), ref) < TOL[0]
    for a_block in (v - 1, v // 2, v // 3):
        assert torch.equal(_residual(gpu_lib, Ld, td, 0, a_block=a_block, **kw), one), a_block


def _folded(native, Ld, td, **kw):
    """Whether the float64 forward is folded: it then prepares amplitudes without being
    the exchange partner, or runs in other blocks than the plan's."""
    seen = []
    fn = native.TRACE_FN(lambda user, phase, block, end, stream: seen.append((phase, block)))
    _residual(native, Ld, td, 0, trace=fn, **kw)
    blocks = 1 + max(b for p, b in seen if p == 2)
    return blocks > 1 if kw.get("exchange") else (0, 0) in seen


# the float64 forward: folded sizes (46 occupied with 64 virtuals: 2 o^2 > v^2, no room for
# partial sums) and sizes of the direct route; explicit blocks, and scratch down to the
# folded route's least, which is what one virtual per block asks for
@pytest.mark.parametrize("o,v,P,pairsym,folded", [
    (9, 71, 263, False, True), (20, 64, 100, False, True), (12, 81, 50, False, True),
    (46, 64, 20, False, True), (46, 72, 30, True, True), (30, 72, 50, True, True),
    (16, 64, 200, False, False), (12, 100, 300, True, False), (9, 71, 60, False, False)])
@pytest.mark.parametrize("exchange", [False, True])
def test_float64_forward(gpu_lib, o, v, P, pairsym, folded, exchange):
    import torch

    announce("blocks-float64", o, v, P, "pairsym", pairsym, "exchange", exchange)
    L, t, _ = random_general(o, v, P, 6100 + o + v)
    if pairsym:
        t = 0.5 * (t + t.transpose(1, 0, 3, 2))
    Ld, td = dev(L), dev(t)
    kw = dict(pair_symmetric=pairsym, exchange=exchange)
    one = _residual(gpu_lib, Ld, td, 0, **kw)
    ref = oracle.exchange_forward(L, t) if exchange else oracle.ladder_forward(L, t)
    assert rel_fro(host(one), ref) < TOL[0]
    if folded or not exchange:  # (the swapped copy tips the scales at some of the direct sizes)
        assert _folded(gpu_lib, Ld, td, **kw) == folded
    for a_block in (1, 7, v // 3, v - 1):
        assert torch.equal(_residual(gpu_lib, Ld, td, 0, a_block=a_block, **kw), one), a_block
    full, _ = gpu_lib.cc_ladder_workspace_query(o, v, P, 0, opts=gpu_lib.make_opts(**kw))
    least, _ = gpu_lib.cc_ladder_workspace_query(o, v, P, 0, opts=gpu_lib.make_opts(a_block=1, **kw))
    for budget in (full - 1, (full + least) // 2, least):
        assert torch.equal(_residual(gpu_lib, Ld, td, 0, hbm_budget=budget, **kw), one), budget
    if folded and not exchange:  # less scratch than the folded route needs: the direct one
        small = _residual(gpu_lib, Ld, td, 0, hbm_budget=least - 1, **kw)
        assert rel_fro(host(small), ref) < TOL[0]
        assert not _folded(gpu_lib, Ld, td, hbm_budget=least - 1, **kw)


# split-int8 past one chunk of 16384 contracted indices, which the stacked route's swapped
# copy of t regroups: the stacked route's sizes (v >= 3 o) and the direct one's
@pytest.mark.parametrize("o,v,P", [(4, 130, 9), (12, 133, 40), (44, 129, 6)])
@pytest.mark.parametrize("exchange", [False, True])
@pytest.mark.parametrize("slices", [4, 5])
def test_split_int8_forward(gpu_lib, o, v, P, exchange, slices):
    import torch

    announce("blocks-int8", o, v, P, "exchange", exchange, "slices", slices)
    L, t, _ = random_general(o, v, P, 6200 + o + v)
    Ld, td = dev(L), dev(t)
    kw = dict(exchange=exchange, split_slices=slices)
    one = _residual(gpu_lib, Ld, td, 3, **kw)
    for a_block in (1, v // 3, v - 1):
        assert torch.equal(_residual(gpu_lib, Ld, td, 3, a_block=a_block, **kw), one), a_block
    full, _ = gpu_lib.cc_ladder_workspace_query(o, v, P, 3, opts=gpu_lib.make_opts(**kw))
    least, _ = gpu_lib.cc_ladder_workspace_query(o, v, P, 3, opts=gpu_lib.make_opts(a_block=1, **kw))
    for budget in (full - 1, (full + least) // 2, least):
        assert torch.equal(_residual(gpu_lib, Ld, td, 3, hbm_budget=budget, **kw), one), budget
    if o < 20:
        ref = oracle.exchange_forward(L, t) if exchange else oracle.ladder_forward(L, t)
        assert rel_fro(host(one), ref) < (4e-8 if slices == 4 else 1e-9)


# the float64 adjoint: folded (amplitudes prepared, nothing swapped back at the end) in a
# plan of one block, from 64 virtuals on and 16 with pair-symmetric t and lam
@pytest.mark.parametrize("o,v,P,a_block,pairsym,symv,folded", [
    (6, 64, 30, 0, False, False, True), (3, 97, 12, 0, False, False, True),
    (6, 63, 30, 0, False, False, False), (6, 64, 30, 40, False, False, False),
    (5, 16, 20, 0, True, False, True), (7, 33, 41, 0, True, True, True),
    (5, 15, 20, 0, True, False, False), (5, 40, 20, 20, True, False, False)])
@pytest.mark.parametrize("exchange", [False, True])
def test_adjoint_route(gpu_lib, o, v, P, a_block, pairsym, symv, folded, exchange):
    import torch

    announce("route-adjoint", o, v, P, a_block, "pairsym", pairsym, "symv", symv, "exchange", exchange)
    Ld = torch.zeros(P, v, v, dtype=torch.float64, device="cuda")
    td = torch.zeros(o, o, v, v, dtype=torch.float64, device="cuda")
    seen = []
    fn = gpu_lib.TRACE_FN(lambda user, phase, block, end, stream: seen.append((phase, block)))
    gpu_lib.cc_ladder_backward(
        Ld, td, td.clone(), torch.zeros_like(Ld), torch.zeros_like(td), 0,
        opts=gpu_lib.make_opts(a_block=a_block, pair_symmetric=pairsym, symmetric_vectors=symv,
                               exchange=exchange, trace=fn))
    torch.cuda.synchronize()
    assert ((0, 1) not in seen if exchange else (0, 0) in seen) == folded
