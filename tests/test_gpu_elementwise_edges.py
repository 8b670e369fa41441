"""Transposed AddOps at the edges of their 32-wide tiles and chains of AddOps over small planes, against
NumPy.  Factors are powers of two, so every term is exact and every sum
rounds once, in order: the comparison is exact."""

import numpy as np
import pytest
import torch

from paper_2201_01257_amd import core as tm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext", [(1, 1), (31, 33), (32, 64), (33, 65), (64, 32), (97, 127), (5, 200)])
@pytest.mark.parametrize("labels", ["jik", "kji", "ikj"])
@pytest.mark.parametrize("beta", [0.0, 0.5])
def test_transposed_add(ext, labels, beta):
    rng = np.random.default_rng(ext[0])
    sizes = dict(i=3, j=ext[0], k=ext[1])
    spaces = {c: tm.Space.explicit([n, 2]) for c, n in sizes.items()}
    full = {c: n + 2 for c, n in sizes.items()}
    X = rng.standard_normal([full[c] for c in labels])
    Z = rng.standard_normal([full[c] for c in "ijk"])
    x = tm.Tensor([spaces[c] for c in labels]).from_dense(X)
    z = tm.Tensor([spaces[c] for c in "ijk"]).from_dense(Z)
    if beta == 0.0:
        z.data.fill_(float("nan"))  # not read
    tm.Add(z, "ijk", x, labels).execute(-2.0, beta)
    torch.cuda.synchronize()
    ref = -2.0 * X.transpose([labels.index(c) for c in "ijk"]) + (beta * Z if beta else 0.0)
    assert np.array_equal(z.to_dense(), ref)


@pytest.mark.parametrize("i_tiles,j_tiles", [([1], [1]), ([16, 3], [16, 15]), ([16, 17], [16]), ([32, 9], [32, 31])])
def test_chain_of_planes(i_tiles, j_tiles):
    # planes of at most 256 elements (four per workgroup, a last workgroup partly filled), of 272 and
    # of 1024 (one per workgroup)
    rng = np.random.default_rng(len(i_tiles))
    si, sj, sb = (tm.Space.explicit(t) for t in (i_tiles, j_tiles, [3, 2]))
    n = dict(b=5, i=sum(i_tiles), j=sum(j_tiles))
    X, Y, Z = (rng.standard_normal([n[c] for c in l]) for l in ("bij", "bji", "bij"))
    x, y, z = (tm.Tensor(s).from_dense(v) for s, v in (([sb, si, sj], X), ([sb, sj, si], Y), ([sb, si, sj], Z)))
    chain = tm.Scheduler()
    chain.add(tm.Add(z, "bij", x, "bij"), -2.0, 0.5)
    chain.add(tm.Add(z, "bij", y, "bji"), 0.25, 1.0)
    chain.add(tm.Add(z, "bij", x, "bij"), 4.0, 1.0)
    chain.build()
    assert chain.info()["fused_ops"] == 3
    chain.bind_workspace(z.data.device)
    chain.execute()
    torch.cuda.synchronize()
    assert np.array_equal(z.to_dense(), 0.5 * Z + -2.0 * X + 0.25 * Y.transpose(0, 2, 1) + 4.0 * X)
