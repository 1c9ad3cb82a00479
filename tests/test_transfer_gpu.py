"""Field reads of every size: one small block of pinned memory, the runtime's own
path, and the pinned ring with several chunks and host threads must all return
the same values."""
import threading

import numpy as np
import pytest

from paper_2308_08085_amd import abi, workloads as W

pytestmark = pytest.mark.gpu


def _sim(case, layers):
    g = abi.AmrLbm(case)
    g.set_root_rho_u(case.initial_rho_u())
    if layers:
        tags = np.zeros(g.cap, np.int8)
        tags[: layers] = 1
        g.tag(tags_in=tags)
        g.adapt()
    g.step(2)
    return g


def _check(g, f, cells):
    """the list of output cells and their fields, from the block-wise read"""
    m, blocks = g.mesh(), f
    out = g.output()
    assert np.array_equal(out["blk"], cells[:, 0]) and np.array_equal(out["cell"], cells[:, 1])
    assert np.array_equal(out["f"], blocks[out["blk"], out["cell"]])
    assert np.all(m["status"][out["blk"]] == 0)
    key = out["blk"].astype(np.int64) * g.mb + out["cell"]
    assert np.all(np.diff(key) > 0)
    ru = g.rho_u_out()
    assert np.array_equal(ru[:, 0], out["rho"]) and np.array_equal(ru[:, 1: 1 + g.dim], out["u"])
    rho = out["f"].sum(1)
    assert np.max(np.abs(ru[:, 0] - rho)) < 1e-13  # 27 terms of order 0.1, FP64


# sides: one chunk in pinned memory; the runtime's path; the ring with a few
# chunks; the ring with more chunks than slots (61 MB of populations)
@pytest.mark.parametrize("dim,q,side,storage", [(2, 9, 16, "f64"), (2, 9, 100, "f32"), (3, 19, 28, "f16s"),
                                                (3, 27, 68, "f32s")])
def test_reads_of_every_size(dim, q, side, storage):
    g = _sim(W.cavity(dim, q, side, 2, 100.0, storage=storage, seed=7, cap=(side // 4) ** dim * 2), 3)
    cells = g._fields(abi.AMR_GET, abi.F_CELLS, np.zeros((g.n_out(), 2), np.int32))
    for _ in range(2):  # again once the handle has read enough for the ring
        _check(g, g.get_block_f_all(), cells)
    g.close()


def test_reads_from_two_threads():
    """one handle per thread and stream, reading together: whichever finds the
    ring in use takes the other path"""
    case = W.cavity(3, 19, 48, 1, 100.0, storage="f32s", seed=9, cap=12 ** 3)
    sims = [_sim(case, 0) for _ in range(3)]
    want = sims[0].output()
    got = [[] for _ in sims]

    def read(i):
        for _ in range(4):
            got[i].append(sims[i].output())

    threads = [threading.Thread(target=read, args=(i,)) for i in range(len(sims))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for outs in got:
        assert len(outs) == 4
        for o in outs:
            for k in want:
                assert np.array_equal(o[k], want[k]), k
    for g in sims:
        g.close()
