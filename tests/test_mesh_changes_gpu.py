"""Mesh changes that follow each other without a step: every population of
every active block, ghost cells included, must come through each of them."""
import numpy as np
import pytest

from paper_2308_08085_amd import workloads as W

from meshcheck import random_tags
from parity_util import Pair

pytestmark = pytest.mark.gpu


def _cases():
    out = [W.cavity(2, 9, 32, 4, 100.0, cap=2000, name="2d_walls", seed=31)]
    c = W.cavity(2, 9, 16, 3, 100.0, cap=600, name="2d_periodic", seed=32)
    c.periodic = (1, 1, 0)
    out.append(c)
    c = W.cavity(2, 9, 24, 3, 100.0, cap=1000, name="2d_cubic", seed=33)
    c.interp = 1
    out.append(c)
    out.append(W.cylinder(2, 9, (32, 16), 4, 8, 3, 100.0, cap=800, name="2d_solid", storage="f64", seed=34))
    out.append(W.cavity(3, 19, 16, 3, 100.0, cap=3000, name="3d_walls", seed=35))
    c = W.cavity(3, 27, 12, 3, 100.0, cap=1500, name="3d_periodic_xz", seed=36)
    c.periodic = (1, 0, 1)
    out.append(c)
    out.append(W.cylinder(3, 27, (16, 12, 8), 4, 4, 3, 100.0, cap=1200, name="3d_solid", storage="f64", seed=37))
    return out


@pytest.mark.parametrize("case", _cases(), ids=lambda c: c.name)
def test_changes_without_a_step(case):
    """blocks whose neighbours are removed become the edge of their level and
    keep what streamed from them; a second synchronisation then reads it"""
    p = Pair(case)
    rng = np.random.default_rng(41)
    coarsened = 0
    for it in range(10):
        p.tag_replay(random_tags(case, p.o.mesh(), rng, 0.35, 0.3))
        coarsened += p.adapt()["n_coarsen"]
        p.check_mesh("after change %d" % it)
        p.assert_parity(1e-12, "%s, change %d" % (case.name, it))
        if it % 4 == 3:
            p.step(2)
            p.assert_parity(1e-12, "%s, steps after change %d" % (case.name, it))
    assert coarsened > 0
