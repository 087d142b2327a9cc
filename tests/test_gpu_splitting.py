"""The splitting of a small level in one workgroup: states, rounds, numbering
and everything built from them equal the oracle's, at row counts around the
rows a thread keeps (1024, 2048, 4096 and past the limit), with couplings that
fit the workgroup's LDS and with more (the launch-by-launch rounds take over)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from nair_inputs.random_blocks import layered_block_triangular
from test_gpu_parity import build_pair, compare_hierarchies, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,deps,theta", [(130, 3, 0.5), (1023, 3, 0.5), (1024, 2, 0.2), (1025, 4, 0.5), (2048, 3, 0.75),
                                           (2049, 3, 0.1), (4095, 2, 0.5), (4096, 3, 0.3), (4097, 3, 0.3),
                                           (4000, 15, 1e-6)])
def test_splitting(nb, deps, theta):
    _say(f"test: splitting of {nb} rows, {deps} couplings a row, theta {theta}")
    rp, ci, va, _, _ = layered_block_triangular(nb, 1, 20, deps=deps, seed=nb, back_edges=nb // 50)
    G, O = build_pair(nb, 1, rp, ci, va, degree=0, theta=theta, max_levels=2, max_coarse_dofs=16)
    assert G.info()["levels"] == 2
    compare_hierarchies(G, O)
