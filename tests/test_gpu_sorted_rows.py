"""Symbolic products and column merges by sorted rows: the collector's row of
R (A P) has nsrc (nf + 1) + 1 products from nf + 1 inner slots, its row of A
nf + 1 blocks to merge, an F row nsrc + 1; the cases lie at the edges between a
quarter, half and whole wave per row, several keys per lane, and a workgroup
per row.  Long matrices take 64-bit keys (more block columns than fit beside a
product's number).  The hierarchy equals the oracle's bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_parity import build_pair, compare_hierarchies, _say
from test_gpu_spgemm_rows import arrow

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsrc,nf", [(3, 4), (4, 3), (1, 14), (1, 15), (1, 30), (4, 7), (1, 31), (9, 6), (8, 7), (1, 62),
                                     (1, 63), (1, 64), (8, 15), (15, 16), (16, 15), (2, 63), (2, 64), (1, 255),
                                     (1, 256), (73, 6), (16, 31), (33, 30), (32, 31), (63, 64), (3, 1023)])
def test_row_lengths(nsrc, nf):
    _say(f"test: sorted rows, {nsrc * (nf + 1) + 1} products from {nf + 1} slots")
    nb, rp, ci, va, cf = arrow(nf, nsrc, 1, seed=nf)
    G, O = build_pair(nb, 1, rp, ci, va, degree=1, cf_override=cf, max_levels=2, max_coarse_dofs=1, drop=0.0)
    compare_hierarchies(G, O)


def test_wide_keys():
    n = 13_000_000
    _say(f"test: sorted rows, {n} block columns")
    rng = np.random.default_rng(11)
    i = np.arange(n, dtype=np.int64)
    back = np.where(i % 3 == 0, 2, 1)
    first = np.maximum(i - back, 0)
    keep = i >= 2
    rp = np.zeros(n + 1, dtype=np.int32)
    np.cumsum(1 + keep, out=rp[1:])
    ci = np.empty(rp[-1], dtype=np.int32)
    va = np.empty(rp[-1])
    d = rp[1:] - 1
    ci[d] = i
    va[d] = rng.uniform(1.0, 2.0, n)
    ci[rp[:-1][keep]] = first[keep]
    va[rp[:-1][keep]] = -rng.uniform(0.3, 0.9, int(keep.sum()))
    G, O = build_pair(n, 1, rp, ci, va.reshape(-1, 1, 1), degree=1)
    assert O.level(0).nc >= 1 << 22
    compare_hierarchies(G, O)
