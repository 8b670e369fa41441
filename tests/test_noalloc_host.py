"""The workspace rules of the allocation-free one-shot contraction (host analysis, structure-only
tensors): what it does to the plan that tamm_contract keeps for the same contraction."""

import ctypes

import pytest
import torch

from paper_2201_01257_amd import _lib
from paper_2201_01257_amd import core as tm
from paper_2201_01257_amd.synth import TERMS

lib = _lib.load()


def statement(term, n_occ, n_vir, tile_occ, tile_vir):
    (_, op, ol), (_, lp, ll), (_, rp, rl), _ = TERMS[term]
    o = tm.Space.spin(n_occ - n_occ // 2, n_occ // 2, tile_occ)
    v = tm.Space.spin(n_vir - n_vir // 2, n_vir // 2, tile_vir)
    t = [tm.Tensor([dict(o=o, v=v)[c] for c in p], device=None) for p in (op, lp, rp)]
    return t[0], ol, t[1], ll, t[2], rl


def workspace(args, precision):
    n = ctypes.c_size_t()
    out, ol, lhs, ll, rhs, rl = args
    tm.check(lib.tamm_contract_workspace_size(out._h, ol.encode(), lhs._h, ll.encode(), rhs._h, rl.encode(),
                                              tm.PRECISIONS[precision], ctypes.byref(n)))
    return n.value


def noalloc_status(args, precision):
    """What the call ends with: it gets past the host analysis to the missing GPU or storage, or not."""
    with pytest.raises(tm.TammError) as e:
        tm.contract_noalloc(*args, 1.0, 0.0, precision, stream=None if torch.cuda.is_available() else 0)
    return e.value.status


def test_noalloc_leaves_the_plan_of_contract_as_it_is():
    # long items from the dies' queues, and partial sums of more than the scratch array
    args = statement("ladder", 32, 160, 32, 32)
    before = workspace(args, "f64")
    assert before > _lib.NOALLOC_WORKSPACE_BYTES
    noalloc_status(args, "f64")
    assert workspace(args, "f64") == before


def test_a_refused_call_leaves_no_plan_behind():
    m, k = tm.Space.fixed(64, 1), tm.Space.fixed(2048, 1)
    C, A, B = tm.Tensor([m, m], device=None), tm.Tensor([m, k], device=None), tm.Tensor([k, m], device=None)
    args = (C, "ij", A, "ik", B, "kj")
    workspace(args, "f64")
    plans = tm.contract_cache_count()
    assert noalloc_status(args, "f64") == "TAMM_ERR_WORKSPACE"
    assert tm.contract_cache_count() == plans


# Unsplit, each of these fits the scratch array; the K splits that tamm_contract's plan takes do not, in
# float32 for the first eight and in float64 for the first six.
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(22, 119, 13, 41), (22, 125, 12, 36), (30, 150, 30, 30), (25, 173, 24, 38), (32, 160, 32, 32),
                                   (32, 160, 16, 40), (20, 160, 20, 64), (8, 200, 8, 50), (40, 200, 40, 40), (12, 40, 3, 3)])
def test_noalloc_runs_what_fits_without_splits(shape, precision):
    args = statement("ladder", *shape)
    plan = tm.Plan(*args, precision=precision, bind=False)
    plan.set_config(3, 1)
    assert plan.workspace_size() <= _lib.NOALLOC_WORKSPACE_BYTES
    assert noalloc_status(args, precision) != "TAMM_ERR_WORKSPACE"
