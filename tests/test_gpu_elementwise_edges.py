"""Transposed AddOps at the edges of their 32-wide tiles, against NumPy.  Factors are powers of two,
so every result has one correctly rounded value: the comparison is exact."""

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
