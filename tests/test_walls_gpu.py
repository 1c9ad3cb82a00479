"""Blocks that meet no, one or several walls: a sweep keeps the data of a block
that meets one face or solid only apart from the general look-up.  Boxes one or
two blocks thick put opposite faces, edges and corners into one block, and 2-D
waves of four blocks get every mix of them."""
import numpy as np
import pytest

from paper_2308_08085_amd import workloads as W

from parity_util import Pair

pytestmark = pytest.mark.gpu


def _case(dim, q, root, periodic, outflow, solid):
    c = W.cavity(dim, q, 16, 2, 50.0, cap=700, name="walls", seed=31)
    c.root = root if dim == 3 else (root[0], root[1], 1)
    c.periodic = periodic
    # every face moves along itself at a speed of its own
    u = [[0.0] * 3 for _ in range(6)]
    for f in range(2 * dim):
        for a in range(dim):
            if a != f // 2:
                u[f][a] = 0.002 * (f + 1) * (-1) ** a
    kind = [W.FACE_VELOCITY] * 6
    if outflow >= 0:
        kind[outflow], u[outflow] = W.FACE_OUTFLOW, [0.0] * 3
    c.face_kind, c.face_u = tuple(kind), tuple(tuple(v) for v in u)
    if solid:
        n = c.root[0] * c.root[1] * c.root[2]
        s = np.zeros(n, np.uint8)
        s[n // 2] = 1
        c.solid = s
    return c


@pytest.mark.parametrize("dim,q", [(2, 9), (3, 19), (3, 27)])
@pytest.mark.parametrize("root,periodic,outflow,solid", [
    ((1, 1, 1), (0, 0, 0), -1, False),   # every face in one block
    ((5, 1, 2), (0, 0, 0), 1, False),    # opposite faces, outflow
    ((3, 4, 3), (1, 0, 1), -1, False),   # one face per block, inner blocks between
    ((5, 5, 3), (1, 1, 1), -1, True),    # a solid only
    ((5, 3, 3), (0, 0, 1), 1, True)],    # solid and faces in one block
    ids=["all", "opposite", "one", "solid", "mixed"])
def test_walls_against_the_oracle(dim, q, root, periodic, outflow, solid):
    """as the other comparisons in FP64: every population within 1e-12 of the
    oracle's, on one level and with half the blocks refined"""
    p = Pair(_case(dim, q, root, periodic, outflow, solid))
    p.step(6)
    p.assert_parity(1e-12, "one level")
    m = p.o.mesh()
    tags = np.zeros(len(m["level"]), np.int8)
    tags[(m["level"] == 0) & (m["status"] == 0) & (np.arange(len(tags)) % 2 == 0)] = 1
    p.tag_replay(tags)
    p.adapt()
    p.check_mesh("refined")
    p.step(6)
    p.assert_parity(1e-12, "two levels")
