"""Short rows (levels below 32,768 lanes): sweeps and restrictions that read a
row's first 16 columns beside its header give the bits of those that go
through A's and Z's own index arrays (sweep_copy = "all"), at one lane group
per row: rows below, at and past 16 blocks, every instantiated block size and a
run-time one, FC relaxation, FP32 storage, F-cycles and the scalar form."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from nair_inputs import make_config
from nair_inputs.random_blocks import layered_block_triangular
from test_gpu_parity import to_dev, _say
from test_gpu_sweep import one_group_table, same_solves

pytestmark = pytest.mark.gpu


def short_plain(rp, ci, va, bs, **kw):
    import paper_1704_05001_amd as P
    d = to_dev(rp, ci, va)
    return [P.Hierarchy(*d, bs, P.Params(tuning=one_group_table(), sweep_copy=c, **kw))
            for c in ("off", "all")]


@pytest.mark.parametrize("bs", [1, 4, 5, 9, 16, 25, 32])
@pytest.mark.parametrize("deps", [3, 15, 16, 18])
def test_short_rows_change_no_bit(bs, deps):
    _say(f"test: short rows, blocks of {bs}, {deps} couplings a row")
    rp, ci, va, _, _ = layered_block_triangular(250, bs, 12, deps=deps, seed=bs)
    kw = dict(degree=2)
    if bs == 9:
        kw = dict(degree=0, relax=1)
    if bs == 5:
        kw = dict(degree=3, precision="fp32")
    same_solves(*short_plain(rp, ci, va, bs, **kw), np.random.default_rng(3).uniform(-1, 1, (len(rp) - 1) * bs))


@pytest.mark.parametrize("kw", [{}, dict(faces=False), dict(cycle="F"), dict(form="scalar")])
def test_short_rows_transport(kw):
    _say(f"test: short rows, transport {kw}")
    S, k = make_config("dg_q2_256_curved", N=48)
    same_solves(*short_plain(S.rowptr, S.colidx, S.vals, S.bs, **dict(dict(degree=k), **kw)), S.rhs)
