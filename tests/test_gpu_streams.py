"""Launches of one plan that overlap: on more streams than the plan has counter sets, with partial sums
of K splits, and in captured graphs (more of them than there are sets for) beside eager launches, each
with an output of its own.  Every output must hold the bits that the plan writes alone.  Launches over the
dies' queues with every tile size, with K splits and on a group's own grid.  And the order of capture and
first execution of a group."""

import numpy as np
import pytest
import torch

from paper_2201_01257_amd import core as tm

pytestmark = pytest.mark.gpu


def long_plan(k_tiles=(200, 56), k_splits=1):
    # 576 tiles of 128 x 128: more items than resident workgroups; 256 summed indices and more (about
    # 60 us) make them long enough for the queues, and so do parts of that length
    m, k = tm.Space.explicit([1500, 1500]), tm.Space.explicit(list(k_tiles))
    A, B, C = tm.Tensor([m, k]), tm.Tensor([k, m]), tm.Tensor([m, m])
    g = torch.Generator(device="cuda").manual_seed(11)
    for t in (A, B):
        t.data.copy_(torch.randn(t.data.shape, dtype=torch.float64, device="cuda", generator=g))
    plan = tm.Plan(C, "ij", A, "ik", B, "kj")
    plan.set_config(3, k_splits)
    assert plan.stats()["persistent"] == (1 if sum(k_tiles) // k_splits >= 256 else 0)
    plan.execute(1.0, 0.0)
    torch.cuda.synchronize()
    want = C.data.clone()
    ref = A.to_dense() @ B.to_dense()
    assert abs(C.to_dense() - ref).max() <= 1e-11 * abs(ref).max()
    return plan, C, want


# one part from the queues; two parts from a plain launch; two parts from the queues
@pytest.mark.parametrize("k_tiles,k_splits", [((200, 56), 1), ((40, 40), 2), ((256, 256), 2)])
def test_launches_on_more_streams_than_counter_sets(k_tiles, k_splits):
    plan, C, want = long_plan(k_tiles, k_splits)
    streams = [torch.cuda.Stream() for _ in range(12)]
    outs = [torch.full_like(want, float("nan")) for _ in range(36)]
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        C.bind(out)
        plan.execute(1.0, 0.0, stream=streams[i % 12].cuda_stream)
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        assert torch.equal(out, want), i


def test_captured_launches_beside_eager_ones():
    plan, C, want = long_plan()
    outs = [torch.full_like(want, float("nan")) for _ in range(30)]
    graphs = []
    for out in outs[:26]:  # two more than there are sets for captured launches
        C.bind(out)
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            plan.execute(1.0, 0.0)
    streams = [torch.cuda.Stream() for _ in range(4)]
    for _ in range(2):
        for out in outs:
            out.fill_(float("nan"))
        torch.cuda.synchronize()
        for i, out in enumerate(outs):
            with torch.cuda.stream(streams[i % 4]):
                if i < len(graphs):
                    graphs[i].replay()
                else:
                    C.bind(out)
                    plan.execute(1.0, 0.0)
        torch.cuda.synchronize()
        for i, out in enumerate(outs):
            assert torch.equal(out, want), i


def test_contractions_after_one_screening():
    plan, C, want = long_plan()
    plan.screen()
    for _ in range(3):  # no screening in between to clear the counters
        C.data.fill_(float("nan"))
        plan.contract(1.0, 0.0)
        torch.cuda.synchronize()
        assert torch.equal(C.data, want)


# (configuration, K splits): whether the launch takes its items from the queues (more items than resident
# workgroups, 40 us and more each)
@pytest.mark.parametrize("config,k_splits,persistent", [(3, 1, 1), (1, 1, 1), (2, 1, 1), (0, 1, 1), (4, 1, 1), (12, 1, 1), (13, 1, 1),
                                                        (9, 1, 1), (3, 2, 1), (1, 2, 1), (1, 3, 0)])
def test_queues_with_every_tile_size_and_splits(config, k_splits, persistent):
    m, n, k = tm.Space.explicit([1530, 1517]), tm.Space.explicit([1290, 1803]), tm.Space.explicit([300, 301, 299])
    A, B, C = tm.Tensor([m, k]), tm.Tensor([k, n]), tm.Tensor([m, n])
    g = torch.Generator(device="cuda").manual_seed(5)
    for t in (A, B, C):
        t.data.copy_(torch.randn(t.data.shape, dtype=torch.float64, device="cuda", generator=g))
    a, b, c0 = (t.to_dense() for t in (A, B, C))
    plan = tm.Plan(C, "ij", A, "ik", B, "kj")
    plan.set_config(config, k_splits)
    assert plan.stats()["persistent"] == persistent
    for _ in range(2):
        plan.execute(0.5, 1.0)
    torch.cuda.synchronize()
    # a sum of K products in another order: 2 (K + 2) u of the sum of magnitudes, for each of two executions
    err, bound = np.abs(C.to_dense() - (a @ b + c0)), 4 * (a.shape[1] + 2) * 2.0 ** -53 * (np.abs(a) @ np.abs(b) + np.abs(c0))
    assert (err <= bound).all()


@pytest.mark.parametrize("grid", [1, 7, 100])
def test_group_on_a_grid_of_fewer_workgroups_than_items(grid):
    m, k = tm.Space.explicit([200, 171]), tm.Space.explicit([16, 40])
    plans = []
    for (sa, la), (sb, lb) in ((([m, k], "ik"), ([k, m], "kj")), (([k, m], "ki"), ([m, k], "jk"))):
        A, B, C = tm.Tensor(sa), tm.Tensor(sb), tm.Tensor([m, m])
        for t in (A, B):
            t.data.normal_()
        plans.append(tm.Plan(C, "ij", A, la, B, lb, bind=False))
    group = tm.Group(plans)
    group.set_config(9)
    group.execute([1.0, 1.0], [0.0, 0.0])
    torch.cuda.synchronize()
    want = [p.out.data.clone() for p in plans]
    group.set_config(9, grid)
    assert group.stats()["work_items"] > 2 * grid
    for _ in range(2):
        for p in plans:
            p.out.data.fill_(float("nan"))
        group.execute([1.0, 1.0], [0.0, 0.0])
        torch.cuda.synchronize()
        for p, w in zip(plans, want):
            assert torch.equal(p.out.data, w)


def test_group_of_several_layouts_is_executed_before_it_is_captured():
    m, k = tm.Space.explicit([30, 34]), tm.Space.explicit([20, 24])
    plans = []
    for (sa, la), (sb, lb) in ((([m, k], "ik"), ([k, m], "kj")), (([k, m], "ki"), ([m, k], "jk"))):
        A, B, C = tm.Tensor(sa), tm.Tensor(sb), tm.Tensor([m, m])
        for t in (A, B):
            t.data.normal_()
        plans.append(tm.Plan(C, "ij", A, la, B, lb, bind=False))
    group = tm.Group(plans)
    with pytest.raises(tm.TammError) as e:
        group.capture([1.0, 1.0], [0.0, 0.0])
    assert e.value.status == "TAMM_ERR_UNSUPPORTED"
    group.execute([1.0, 1.0], [0.0, 0.0])
    torch.cuda.synchronize()
    want = [p.out.data.clone() for p in plans]
    group.capture([1.0, 1.0], [0.0, 0.0])
    for _ in range(2):
        for p in plans:
            p.out.data.fill_(float("nan"))
        group.execute([1.0, 1.0], [0.0, 0.0])
        torch.cuda.synchronize()
        for p, w in zip(plans, want):
            assert torch.equal(p.out.data, w)
    group = tm.Group(plans[:1])  # of one layout: captured at once
    group.capture([1.0], [0.0])
    group.execute([1.0], [0.0])
    torch.cuda.synchronize()
    assert torch.equal(plans[0].out.data, want[0])
