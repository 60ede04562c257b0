"""The flop model behind every TFLOP/s figure (paper_1207_4461_amd/flops.py): its per-pair
counts equal the closed forms its docstring derives, the direct-pass counts are fixed, and
the split's pair counts add up to the workload's pairs at the two extremes of gamma."""
import numpy as np

from paper_1207_4461_amd import flops as F
from paper_1207_4461_amd import inputs as I


def test_forward_counts_follow_the_closed_forms():
    for p in range(1, 40):
        assert F.flops_forward_pair(p, 1) == 95 + 12 * p
        assert F.flops_forward_pair(p, 2) == 114 + 16 * p
        assert F.flops_forward_pair(p, 3) == 128 + 23 * p


def test_counts_grow_with_the_order_and_fuse_below_the_sum():
    for kind in (1, 2, 3):
        for fn in (F.flops_forward_pair, F.flops_tape_pair, F.flops_adjoint_pair,
                   F.flops_fused_pair, F.flops_grad_pair):
            c = [fn(p, kind) for p in range(0, 30)]
            assert all(b > a for a, b in zip(c, c[1:])), fn.__name__
    for p in (4, 12, 20):
        # S and D in one pass share the geometry and the seed
        for fn in (F.flops_forward_pair, F.flops_fused_pair):
            assert fn(p, 3) < fn(p, 1) + fn(p, 2)


def test_direct_pass_counts():
    assert (F.flops_far_pair(1), F.flops_far_pair(2), F.flops_far_pair(3)) == (85, 91, 99)
    assert F.interactions(10, 7, 3) == 140 and F.interactions(10, 7, 1) == 70


def test_split_pair_counts_at_the_extremes():
    P, os_ = 12, 2
    nodes = I.panel_nodes(I.star((5, 0.25, 0.0)), P)
    qs = 16 * os_
    near, far = F.split_pairs(nodes, os_, 2, 1e150)          # every panel near
    assert (near, far) == (2 * 16 * P * qs * P, 0)
    cnt = F.near_panel_counts(nodes, 1e-9)                    # each panel near only itself
    assert np.array_equal(cnt, np.ones(P, dtype=cnt.dtype))
    near, far = F.split_pairs(nodes, os_, 2, 1e-9)
    # far panels lend their 16 nodes, whatever the oversampling
    assert (near, far) == (2 * 16 * qs * P, (P - 1) * 16 * 16 * P)


def test_near_pairs():
    """A bounded number of panels per panel, with and without groups; all where nothing resolves."""
    from paper_1207_4461_amd import inputs as I

    for P in (96, 320, 640):
        pb = I.make_problem("near", I.star((5, 0.25, 0.3)), P, 10.0, 6, 0, 3, 1, oversample=2)
        assert 3 <= F.near_pairs(pb.nodes, pb.k, pb.r, 2, 2, 0) / (P * 16 * 2 * 32) <= 24
    assert F.near_pairs(pb.nodes, 1e5, pb.r, 2, 2, 0) == (640 * 16) ** 2 * 4


def test_expansions_apply():
    assert not F.expansions_apply(95, 8, 2, 24, 3) and F.expansions_apply(96, 4, 2, 12, 3)
    assert not F.expansions_apply(96, 3, 1, 4, 1) and F.expansions_apply(96, 3, 1, 4, 1, True)
    assert F.expansions_apply(4096, 1, 1, 0, 1)


def test_expansions_apply_in_a_small_batch():
    """A batch of less than 20 GFLOP over every pair takes them from 160 panels on."""
    small = F.all_pairs_work(120, 4, 1, 6, 1)
    assert small == (16 * 120) ** 2 * 4 * F.flops_forward_pair(6, 1) < 2e10
    assert not F.expansions_apply(120, 4, 1, 6, 1, True, small)
    assert F.expansions_apply(160, 4, 1, 6, 1, True, small)


def test_near_pairs_where_the_expansions_are_off():
    """Half of the pairs near: all of them for the adjoint, the near ones for the forward; the
    distance of unresolved panels squares without a warning."""
    import warnings

    from paper_1207_4461_amd import inputs as I

    pb = I.make_problem("near", I.star((5, 0.25, 0.3)), 290, 84.0, 6, 1, 1, 17)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        every = (290 * 16) ** 2 * 4
        assert F.near_pairs(pb.nodes, 84.0, 0.5, 4, 1, 1, adjoint=True) == every
        assert 0.4 * every < F.near_pairs(pb.nodes, 84.0, 0.5, 4, 1, 1) < 0.9 * every
        assert F.near_pairs(pb.nodes, 300.0, 0.5, 4, 1, 1) == every
