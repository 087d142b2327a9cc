"""Collapsed coarse cycle: below the finest level, the first level of at most 2048
unknowns (1024 block rows) has its cycle as one dense matrix.  One cycle and its transpose match
the oracle's, and solves take the oracle's iterations, for every block size the
kernels are instantiated for and run-time ones, F and FC relaxation, no, one and
three extra sweeps, V- and F-cycles, the scalar form, FP32 storage, and orders
around the rule's edge and the kernels' 64 columns."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from nair_inputs import make_config
from nair_inputs.random_blocks import layered_block_triangular
from test_gpu_parity import build_pair, _say, np_, check_solve, small_dg

pytestmark = pytest.mark.gpu


def check_cycles(G, O, n, seed):
    for trans in (False, True):
        v = np.random.default_rng(seed + trans).uniform(-1, 1, n)
        e = np_((G.vcycle_T if trans else G.vcycle)(torch.from_numpy(v).cuda()))
        eo = (O.vcycle_T if trans else O.vcycle)(v)
        assert np.abs(e - eo).max() <= 1e-12 * np.abs(eo).max()


@pytest.mark.parametrize("bs,nb,kw", [(1, 2500, {}), (1, 3400, {}), (1, 300, dict(relax=1)), (2, 900, {}), (3, 700, dict(degree=0)),
                                      (4, 700, {}), (6, 330, dict(relax=1)), (9, 300, dict(degree=3)),
                                      (12, 200, {}), (16, 160, {}), (25, 130, dict(degree=1, relax=1)), (32, 90, {})])
def test_cycles_match_the_oracle(bs, nb, kw):
    _say(f"test: collapsed cycle bs={bs} nb={nb} {kw}")
    rp, ci, va, _, _ = layered_block_triangular(nb, bs, 24, deps=3, seed=bs + nb, zero_entries=0.3)
    kw = dict(dict(degree=2, max_coarse_dofs=24), **kw)
    for cyc in ("V", "F"):
        G, O = build_pair(nb, bs, rp, ci, va, gpu_kw=dict(cycle=cyc), **kw)
        assert O.num_levels >= 3
        check_cycles(G, O, nb * bs, 50 + bs)


@pytest.mark.parametrize("N", [21, 22, 27])
def test_orders_around_the_rule(N):
    """Q2: the level the rule picks changes as the meshes grow past 2048 unknowns per level."""
    _say(f"test: collapsed cycle Q2 N={N}")
    S = small_dg(N, 2, seed=N)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, degree=2)
    check_cycles(G, O, S.n, N)
    check_solve(G, O, S.rhs)
    check_solve(G, O, np.random.default_rng(N).uniform(-1, 1, S.n), trans=True)


def test_scalar_form_and_fp32():
    _say("test: collapsed cycle, scalar form and FP32 storage")
    S, k = make_config("dg_q1_32", N=24)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, gpu_kw=dict(form="scalar"), degree=k)
    check_cycles(G, O, S.n, 3)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, gpu_kw=dict(precision="fp32"), degree=k)
    xg, rg = G.solve(torch.from_numpy(S.rhs).cuda(), rtol=1e-10)
    xo, ho, so = O.solve(S.rhs, 1e-10, 200)
    assert rg.status == so and abs(rg.iters - len(ho)) <= 2
    assert np.abs(np_(xg) - xo).max() <= 1e-8 * np.abs(xo).max()
