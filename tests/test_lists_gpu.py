"""Ordered lists of the mesh: the counts of every 1024 indexes are added up by
each workgroup, or, from 1024 workgroups on, scanned by one in between."""
import numpy as np
import pytest

from paper_2308_08085_amd import workloads as W

from meshcheck import random_tags
from parity_util import Pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,scanned", [(349000, False), (350000, True)], ids=["added", "scanned"])
def test_lists_of_a_large_mesh(cap, scanned):
    """three levels over 300 x 300 root blocks: 3 * cap indexes of the level
    lists on both sides of 1024 * 1024; tables equal the oracle's, populations
    as everywhere within 1e-12"""
    assert ((3 * cap + 1023) // 1024 > 1024) == scanned
    case = W.cavity(2, 9, 1200, 3, 1000.0, cap=cap, name="lists", seed=12)
    p = Pair(case)
    rng = np.random.default_rng(5)
    for it in range(3):
        p.tag_replay(random_tags(case, p.o.mesh(), rng, 0.15, 0.4))
        p.adapt()
        p.check_mesh("after adapt %d" % it)
        p.step(1)
    p.assert_parity(1e-12, "large mesh")
