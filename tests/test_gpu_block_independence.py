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
