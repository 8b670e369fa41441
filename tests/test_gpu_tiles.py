"""Float64 tiles of every size a configuration can have (whole tiles, the even cuts of a block's end,
the smallest blocks), in both operand orientations, with and without K splits, and the queues of a
persistent launch, against float64 products computed by NumPy; and the reduced precisions' chunks.

The tolerance (float64) is that of a sum of K products in another order: 2 K u (u = 2^-53) of the sum of
magnitudes, element by element."""

import numpy as np
import pytest
import torch

from paper_2201_01257_amd import core as tm

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def matrices(m, k, n, a_kc, b_kc, m_tiles, n_tiles, k_tiles, seed):
    rng = np.random.default_rng(seed)
    A, B = rng.standard_normal((m, k)), rng.standard_normal((k, n))
    sm, sk, sn = (tm.Space.explicit(t) for t in (m_tiles, k_tiles, n_tiles))
    ta = tm.Tensor([sm, sk] if a_kc else [sk, sm]).from_dense(A if a_kc else A.T)
    tb = tm.Tensor([sn, sk] if b_kc else [sk, sn]).from_dense(B.T if b_kc else B)
    return A, B, ta, "ik" if a_kc else "ki", tb, "jk" if b_kc else "kj", tm.Tensor([sm, sn])


def check(C, A, B, alpha, beta, C0):
    got, ref = C.to_dense(), alpha * (A @ B) + beta * C0
    bound = 2 * (A.shape[1] + 2) * U * (abs(alpha) * (np.abs(A) @ np.abs(B)) + abs(beta * C0))
    bad = np.abs(got - ref) > bound
    assert not bad.any(), (int(bad.sum()), np.argwhere(bad)[:3].tolist())


@pytest.mark.parametrize("a_kc", [True, False])
@pytest.mark.parametrize("b_kc", [True, False])
@pytest.mark.parametrize("ext", [(1, 1), (15, 33), (16, 17), (32, 31), (48, 96), (63, 65), (80, 129), (127, 160), (200, 130)])
def test_every_tile_size(ext, a_kc, b_kc):
    m, n = ext
    # blocks of the extent itself and of one row and column more, three summed tiles (one odd)
    A, B, ta, la, tb, lb, C = matrices(2 * m + 1, 45, 2 * n + 1, a_kc, b_kc, [m, m + 1], [n, n + 1], [16, 24, 5], seed=m * 1000 + n)
    C0 = np.random.default_rng(7).standard_normal((2 * m + 1, 2 * n + 1))
    plan = tm.Plan(C, "ij", ta, la, tb, lb)
    for config in range(plan.config_count()):
        for ks in (1, 3):
            plan.set_config(config, ks)
            C.from_dense(C0)
            plan.execute(0.5, 1.0)
            torch.cuda.synchronize()
            check(C, A, B, 0.5, 1.0, C0)


@pytest.mark.parametrize("extent", [1024 * 4, 1024 * 4 - 3])
def test_persistent_launch_takes_every_item_once(extent):
    # more 128 x 128 tiles than resident workgroups, each long enough for the queues; unequal blocks
    tiles = [extent // 2 + 40, extent - extent // 2 - 40]
    A, B, ta, la, tb, lb, C = matrices(extent, 256, extent, True, False, tiles, tiles, [200, 56], seed=5)
    plan = tm.Plan(C, "ij", ta, la, tb, lb)
    for config, ks in ((3, 1), (1, 1), (3, 2)):
        plan.set_config(config, ks)
        assert plan.stats()["work_items"] > 512
        for _ in range(3):  # every launch starts its queues afresh
            C.data.fill_(float("nan"))
            plan.execute(1.0, 0.0)
            torch.cuda.synchronize()
        check(C, A, B, 1.0, 0.0, np.zeros_like(C.to_dense()))


def test_group_of_a_long_sum_and_a_wide_product():
    # a member with few output elements and a long sum is cut into small tiles beside a wide one
    plans, refs = [], []
    for m, k, n in ((150, 3000, 70), (900, 64, 1300), (33, 5, 17)):
        A, B, ta, la, tb, lb, C = matrices(m, k, n, True, False, [m // 2, m - m // 2], [n], [k // 2, k - k // 2], seed=m)
        plans.append(tm.Plan(C, "ij", ta, la, tb, lb, bind=False))
        refs.append((C, A, B))
    group = tm.Group(plans)
    for config in [-1] + list(range(plans[0].config_count())):
        group.set_config(config)
        for C, _, _ in refs:
            C.data.fill_(float("nan"))
        group.execute([1.5, 1.0, -1.0], [0.0] * 3)
        torch.cuda.synchronize()
        for (C, A, B), alpha in zip(refs, (1.5, 1.0, -1.0)):
            check(C, A, B, alpha, 0.0, np.zeros((A.shape[0], B.shape[1])))


@pytest.mark.parametrize("precision", ["f32", "bf16x3", "bf16x4_aligned"])
@pytest.mark.parametrize("a_kc,b_kc", [(True, True), (True, False), (False, True), (False, False)])
@pytest.mark.parametrize("ext", [(1, 17), (64, 65), (129, 63), (200, 130)])
def test_reduced_precision_chunks_and_windows(ext, a_kc, b_kc, precision):
    # summed tiles of every remainder of a chunk and of one 256-long window and a little more or
    # less; small integers, which every precision holds and sums exactly (sums below 2^24)
    m, n = ext
    k_tiles = [[16, 8, 256, 520], [7, 1, 255, 257, 33]][m % 2]
    k = sum(k_tiles)
    rng = np.random.default_rng(m)
    A, B = rng.integers(-8, 9, (m + 3, k)).astype(float), rng.integers(-8, 9, (k, n + 5)).astype(float)
    sm, sk, sn = (tm.Space.explicit(t) for t in ([m, 3], k_tiles, [5, n]))
    ta = tm.Tensor([sm, sk] if a_kc else [sk, sm]).from_dense(A if a_kc else A.T)
    tb = tm.Tensor([sn, sk] if b_kc else [sk, sn]).from_dense(B.T if b_kc else B)
    C = tm.Tensor([sm, sn], device="cuda")
    plan = tm.Plan(C, "ij", ta, "ik" if a_kc else "ki", tb, "jk" if b_kc else "kj", precision=precision)
    for config in range(plan.config_count()):
        for ks in (1, 2):
            plan.set_config(config, ks)
            C.data.fill_(float("nan"))
            plan.execute(1.0, 0.0)
            torch.cuda.synchronize()
            assert np.array_equal(C.to_dense(), A @ B), (plan.config_name(), ks)
