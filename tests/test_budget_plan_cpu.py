"""The unlimited plan is the plan under any budget that holds it, which is what lets
the autograd wrapper skip the allocator statistics when the plan is small."""
import random

from paper_2310_04559_amd import native


def test_unlimited_plan_is_the_plan_of_any_budget_that_holds_it():
    rng = random.Random(7)
    flags = [{}, {"pair_symmetric": True}, {"exchange": True},
             {"pair_symmetric": True, "plus_minus": True},
             {"pair_symmetric": True, "symmetric_vectors": True},
             {"pair_symmetric": True, "plus_minus": True, "symmetric_vectors": True}]
    seen = 0
    for _ in range(600):
        o, v, P = rng.randint(1, 40), rng.randint(1, 300), rng.randint(1, 1500)
        prec, bwd, kw = rng.choice(range(4)), rng.random() < 0.3, rng.choice(flags)
        opts = native.make_opts(**kw)
        try:
            whole = native.cc_ladder_workspace_query(o, v, P, prec, backward=bwd, opts=opts)
        except native.LadderError:
            continue
        for extra in (0, 1, rng.randint(1, 1 << 33)):
            assert native.cc_ladder_workspace_query(o, v, P, prec, backward=bwd, opts=opts,
                                                    hbm_budget=whole[0] + extra) == whole
            seen += 1
    assert seen > 600


def test_float32_pads_are_left_out_where_they_do_not_fit():
    # odd v: rows padded to whole 16-byte chunks; a scratch sized without the pads
    # still holds the same blocks
    for o, v, P in ((3, 21, 30), (5, 97, 200), (2, 203, 11)):
        for bwd in (False, True):
            whole, n = native.cc_ladder_workspace_query(o, v, P, "fp32", backward=bwd)
            less, m = native.cc_ladder_workspace_query(o, v, P, "fp32", backward=bwd,
                                                       hbm_budget=whole - 1)
            assert n == m == v and less < whole
