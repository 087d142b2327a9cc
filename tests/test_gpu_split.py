"""Split F sweeps (levels of at least 32,768 lanes): the sweeps from the split
copy keep the part that does not change between sweeps and skip the rows that
are final; they give the bits of the sweeps that read A itself and form
everything anew (sweep_copy = "off"), at one lane group per row, for every
block size the kernels are instantiated for and a run-time one, face rectangles and
blocks by their nonzero rows, FC relaxation, one to four sweeps, FP32 storage,
F-cycles, the scalar form and batches; and splittings whose F-F couplings end
at depth 0 or 1, where fewer sweeps run.  With the default lane groups the
solves match the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from nair_inputs import make_config, make_batch, concat_systems
from nair_inputs.random_blocks import layered_block_triangular
from test_gpu_parity import build_pair, to_dev, _say, check_solve
from test_gpu_sweep import one_group_table, same_solves

pytestmark = pytest.mark.gpu


def on_off(rp, ci, va, bs, sys_nb=None, **kw):
    import paper_1704_05001_amd as P
    d = to_dev(rp, ci, va)
    on = P.Hierarchy(*d, bs, P.Params(tuning=one_group_table(), **kw), sys_nb=sys_nb)
    off = P.Hierarchy(*d, bs, P.Params(tuning=one_group_table(), sweep_copy="off", **kw), sys_nb=sys_nb)
    large = [l for l in range(on.num_levels) if on.level(l, fields=())["sweep_nnzb"] >= 0]
    assert large, "no level is large enough"
    assert all(off.level(l, fields=())["sweep_nnzb"] == -1 for l in large)
    return on, off, large


@pytest.mark.parametrize("name,N,kw", [("dg_q2_256_curved", 96, {}), ("dg_q2_256_curved", 96, dict(faces=False)),
                                       ("dg_q2_256_curved", 80, dict(relax=1)),
                                       ("dg_q2_256_curved", 80, dict(precision="fp32")),
                                       ("dg_q2_256_curved", 80, dict(precision="fp32", faces=False)),
                                       ("dg_q2_256_curved", 72, dict(degree=0)),
                                       ("dg_q2_256_curved", 72, dict(degree=3)),
                                       ("dg_q2_256_curved", 72, dict(degree=1, cycle="F")),
                                       ("dg_q1_32", 130, {}), ("dg_q1_32", 120, dict(faces=False, degree=2)),
                                       ("dg_q1_32", 120, dict(form="scalar")),
                                       ("dg_q3_256_curved_sigma", 60, {}),
                                       ("dg_q4_512_jitter", 48, {}),
                                       ("dg_q4_512_jitter", 40, dict(faces=False, precision="fp32"))])
def test_split_sweeps_change_no_bit(name, N, kw):
    _say(f"test: split sweeps {name} N={N} {kw}")
    S, k = make_config(name, N=N)
    kw = dict(dict(degree=k), **kw)
    on, off, large = on_off(S.rowptr, S.colidx, S.vals, S.bs, **kw)
    r = same_solves(on, off, S.rhs)
    _say(f"  levels {large}, {r.iters} iterations, identical")


@pytest.mark.parametrize("bs", [3, 6, 8, 12])
def test_split_sweeps_dense_blocks(bs):
    _say(f"test: split sweeps, dense blocks of {bs}")
    rp, ci, va, _, _ = layered_block_triangular(33000 // bs + 300, bs, 30, deps=3, seed=bs)
    on, off, _ = on_off(rp, ci, va, bs, degree=2)
    same_solves(on, off, np.random.default_rng(3).uniform(-1, 1, (len(rp) - 1) * bs))


@pytest.mark.parametrize("period", [2, 3, 4])
def test_splittings_of_bounded_depth(period):
    """C on every period-th diagonal of an upwind grid: F-F chains of period - 2 couplings."""
    _say(f"test: split sweeps, F-F depth {period - 2}")
    from nair_inputs import dg_quad
    N = 70
    S = dg_quad(N, 2, (0.8, 0.6), seed_perm=None)
    c = np.arange(N * N)
    cf = (((c % N) + c // N) % period == 0).astype(np.int8)
    on, off, _ = on_off(S.rowptr, S.colidx, S.vals, S.bs, degree=2, cf_override=cf)
    same_solves(on, off, S.rhs)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, degree=2, cf_override=cf)
    check_solve(G, O, S.rhs)


def test_split_sweeps_batched():
    _say("test: split sweeps, batch")
    systems, k = make_batch("dg_q2_angles64_uneven", sizes=(40, 33, 8), nang=5)
    rp, ci, va, rhs, sys_nb = concat_systems(systems)
    bt = torch.from_numpy(rhs).cuda()
    for prec in ("fp64", "fp32"):
        on, off, _ = on_off(rp, ci, va, systems[0].bs, sys_nb=sys_nb, degree=k, precision=prec)
        x1, r1 = on.solve_batch(bt)
        x2, r2 = off.solve_batch(bt)
        assert [r.iters for r in r1] == [r.iters for r in r2]
        assert torch.equal(x1, x2)


def test_split_sweeps_against_the_oracle():
    _say("test: split sweeps, oracle parity")
    S, k = make_config("dg_q4_512_jitter", N=44)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, degree=k)
    check_solve(G, O, S.rhs)
    G.autotune(reps=2)
    check_solve(G, O, S.rhs)
