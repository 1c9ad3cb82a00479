"""Reads on every way that a transfer takes: the pinned block of a handle that
has read often, sizes around it, and destinations in pinned memory."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2308_08085_amd import abi, workloads as W

pytestmark = pytest.mark.gpu


def _sim(dim, q, side, storage, levels=2):
    case = W.cavity(dim, q, side, levels, 100.0, storage=storage, seed=11, cap=(side // 4) ** dim * 2)
    g = abi.AmrLbm(case)
    g.set_root_rho_u(case.initial_rho_u())
    g.step(2)
    return g


def _read_pinned(g, kind, like):
    b = torch.zeros(like.nbytes, dtype=torch.uint8, pin_memory=True)
    abi._check(abi.load().amr_fields(g._h, abi.AMR_GET, kind, 0, C.c_void_p(b.data_ptr()), b.numel()))
    return b.numpy().view(like.dtype).reshape(like.shape)


# rho and u of 8 KB, 62 KB and 74 KB (the block holds 64), 0.7 MB and 2 MB
@pytest.mark.parametrize("dim,q,side,storage", [(2, 9, 16, "f64"), (2, 9, 44, "f32s"), (2, 9, 48, "f64"),
                                                (3, 19, 28, "f16s"), (3, 27, 40, "f32s")])
def test_small_and_pinned_reads(dim, q, side, storage):
    """the same values before the handle has its pinned block, with it, and into
    pinned memory of the caller"""
    g = _sim(dim, q, side, storage)
    first = (g.rho_u_out(), g.output()["f"], g.get_block_f_all(), g.mesh())
    for _ in range(40):
        g.mass_mom()  # the block comes with the 32nd small read
    ru, f, blocks, mesh = g.rho_u_out(), g.output()["f"], g.get_block_f_all(), g.mesh()
    assert np.array_equal(first[0], ru) and np.array_equal(first[1], f) and np.array_equal(first[2], blocks)
    for k in ("level", "status", "X", "nbr", "nbrc", "gap"):
        assert np.array_equal(first[3][k], mesh[k]), k
    out = g.output()
    assert np.array_equal(out["f"], blocks[out["blk"], out["cell"]])
    assert np.array_equal(_read_pinned(g, abi.F_RHO_U, ru), ru)
    assert np.array_equal(_read_pinned(g, abi.F_F, f), f)
    assert np.array_equal(_read_pinned(g, abi.F_BLOCK_F, blocks), blocks)
    assert np.array_equal(_read_pinned(g, abi.F_NBR, np.ascontiguousarray(mesh["nbr"].T)), mesh["nbr"].T)
    # the tags go up through the same block as the effective tags come back
    tags = np.zeros(g.cap, np.int8)
    tags[[0, 3]] = 1
    eff = g.tag(tags_in=tags)
    assert np.array_equal(eff, tags)
    assert g.adapt()["n_refine"] == 2
    m = g.mesh()
    assert np.array_equal(np.flatnonzero(m["status"] == 1), [0, 3]) and len(m["ids"][1]) == 2 * 2 ** dim
    out = g.output()
    assert np.array_equal(out["f"], g.get_block_f_all()[out["blk"], out["cell"]])
    g.close()
