"""Momentum exchange added by sweeps that store past the caches."""
import numpy as np
import pytest

from paper_2308_08085_amd import abi, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,q,storage", [(2, 9, "f64"), (2, 9, "f16s"), (3, 19, "bf16s"), (3, 27, "f32s"),
                                           (3, 27, "f16s"), (3, 27, "f64")])
def test_exchange_in_streamed_sweep_equals_separate_pass(dim, q, storage):
    """with every level stored past the caches, the finest level's sweep adds
    the exchange itself; profiled steps run the separate pass: same sums and
    fields bit for bit"""
    if dim == 2:
        case = W.cylinder(2, 9, (64, 32), 8, 16, 3, 100.0, storage=storage, cap=3000, seed=19)
    else:
        case = W.cylinder(3, q, (32, 16, 16), 4, 8, 3, 100.0, storage=storage, cap=12000, seed=20)
    out = []
    for profile in (True, False):
        g = abi.AmrLbm(case)
        g.stream_bytes(0)
        g.set_root_rho_u(case.initial_rho_u())
        for _ in range(case.lmax - 1):
            g.tag(abi.TAG_DISTANCE, d_spec=case.d_spec, freeze=1)
            g.adapt()
        g.step(6, profile=profile)
        F = g.force()
        assert np.abs(F[case.lmax - 1, :dim]).max() > 0
        out.append((F, g.get_block_f_all()))
        g.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
