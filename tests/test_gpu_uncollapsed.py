"""Cycles that visit several levels below the finest one by one.  A single system's
levels of at most 2048 unknowns are one dense matrix, which small meshes reach on the
first or second coarse level; here at least two coarse levels are visited, or the
systems are batched (a batch is not collapsed).  F-cycles (their residuals on coarse
levels), FC relaxation, transposed cycles, FP32 storage with split levels below the
finest, against the oracle; sweep copies on small coarse levels bit for bit.  And the
collapsed matrix under FP32 storage, forward and transposed."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from nair_inputs import concat_systems, make_batch, make_config
from test_gpu_parity import build_pair, compare_hierarchies, _say, check_solve
from test_gpu_batch import build_batch, check_batch_solve
from test_gpu_collapse import check_cycles
from test_gpu_fp32 import _fp32_vs_oracle
from test_gpu_sweep import one_group_table, pair, same_solves

pytestmark = pytest.mark.gpu


def visited(G):
    """Coarse levels of a single system's hierarchy that its cycles visit one by one."""
    n = 0
    for l in range(1, G.num_levels):
        lv = G.level(l, fields=())
        if lv["coarsest"] or (lv["nb"] * lv["bs"] <= 2048 and lv["nb"] <= 1024):
            break
        n += 1
    return n


CASES = [("dg_q2_256_curved", 64, {}), ("dg_q1_32", 70, {}), ("dg_q3_256_curved_sigma", 48, {}),
         ("dg_q4_512_jitter", 24, {}), ("dg_q1_32", 64, dict(form="scalar"))]


@pytest.mark.parametrize("name,N,gpu_kw", CASES)
@pytest.mark.parametrize("cycle,relax", [("F", 0), ("V", 1), ("F", 1)])
def test_cycles_and_solves_match_the_oracle(name, N, gpu_kw, cycle, relax):
    _say(f"test: visited coarse levels {name} N={N} {gpu_kw} {cycle} relax={relax}")
    S, k = make_config(name, N=N)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, gpu_kw=dict(cycle=cycle, **gpu_kw), degree=k,
                      relax=relax)
    assert visited(G) >= 2
    check_cycles(G, O, S.n, 11)
    check_solve(G, O, S.rhs)
    check_solve(G, O, np.random.default_rng(12).uniform(-1, 1, S.n), trans=True)


@pytest.mark.parametrize("cycle,relax", [("V", 0), ("F", 0), ("V", 1), ("F", 1)])
@pytest.mark.parametrize("name,N", [("dg_q2_256_curved", 90), ("dg_q4_512_jitter", 60)])
def test_fp32_with_a_split_coarse_level(name, N, cycle, relax):
    """Level 1 has at least 32,768 lanes: its sweeps read a split copy, an F-cycle's residual and the C
    sweep A's float values, which only these two keep there."""
    _say(f"test: FP32, split coarse level {name} N={N} {cycle} relax={relax}")
    S, k = make_config(name, N=N)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, gpu_kw=dict(cycle=cycle, precision="fp32"), degree=k,
                      relax=relax)
    lv = G.level(1, fields=())
    assert lv["nb"] * lv["bs"] >= 32768 and lv["sweep_nnzb"] >= 0
    compare_hierarchies(G, O)
    _fp32_vs_oracle(G, O, S.rhs)
    _fp32_vs_oracle(G, O, np.random.default_rng(13).uniform(-1, 1, S.n), trans=True)


@pytest.mark.parametrize("cycle,relax", [("V", 0), ("F", 0), ("V", 1), ("F", 1)])
@pytest.mark.parametrize("name,N", [("dg_q1_32", 32), ("dg_q2_256_curved", 20)])
def test_fp32_collapsed(name, N, cycle, relax):
    _say(f"test: FP32, collapsed {name} N={N} {cycle} relax={relax}")
    S, k = make_config(name, N=N)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, gpu_kw=dict(cycle=cycle, precision="fp32"), degree=k,
                      relax=relax)
    assert visited(G) <= 1
    _fp32_vs_oracle(G, O, S.rhs)
    _fp32_vs_oracle(G, O, np.random.default_rng(14).uniform(-1, 1, S.n), trans=True)


@pytest.mark.parametrize("name,N,kw", [("dg_q2_256_curved", 48, {}), ("dg_q2_256_curved", 48, dict(relax=1)),
                                       ("dg_q2_256_curved", 48, dict(precision="fp32")),
                                       ("dg_q2_256_curved", 48, dict(faces=False, cycle="F")),
                                       ("dg_q1_32", 70, dict(cycle="F")), ("dg_q3_256_curved_sigma", 30, {}),
                                       ("dg_q4_512_jitter", 24, dict(precision="fp32"))])
def test_sweep_copies_of_coarse_levels_change_no_bit(name, N, kw):
    _say(f"test: sweep copy on/off, visited coarse levels {name} N={N} {kw}")
    S, k = make_config(name, N=N)
    on, off = pair(S.rowptr, S.colidx, S.vals, S.bs, degree=k, tuning=one_group_table(), **kw)
    assert visited(on) >= 2
    same_solves(on, off, S.rhs)
    same_solves(on, off, np.random.default_rng(15).uniform(-1, 1, S.n), trans=True)


@pytest.mark.parametrize("kw", [{}, dict(relax=1), dict(cycle="F"), dict(precision="fp32"),
                                dict(cycle="F", precision="fp32", relax=1)])
def test_sweep_copies_in_a_batch_change_no_bit(kw):
    _say(f"test: sweep copy on/off, batch {kw}")
    systems, k = make_batch("dg_q2_angles64_uneven", sizes=(14, 20), nang=2)
    rp, ci, va, rhs, sys_nb = concat_systems(systems)
    on, off = pair(rp, ci, va, systems[0].bs, sys_nb=sys_nb, degree=k, tuning=one_group_table(), **kw)
    bt = torch.from_numpy(rhs).cuda()
    for trans in (False, True):
        x1, r1 = on.solve_batch(bt, trans=trans)
        x2, r2 = off.solve_batch(bt, trans=trans)
        assert [r.iters for r in r1] == [r.iters for r in r2]
        assert torch.equal(x1, x2)


@pytest.mark.parametrize("kw", [dict(relax=1), dict(cycle="F"), dict(cycle="F", relax=1)])
def test_batches_match_the_oracle(kw):
    _say(f"test: batch of two systems against the oracle {kw}")
    systems, k = make_batch("dg_q2_angles64_uneven", sizes=(14, 20), nang=2)
    gpu_kw = {a: v for a, v in kw.items() if a == "cycle"}
    G, Os, rhs = build_batch(systems, gpu_kw=gpu_kw, degree=k, **{a: v for a, v in kw.items() if a != "cycle"})
    check_batch_solve(G, Os, systems, rhs)
    check_batch_solve(G, Os, systems, np.random.default_rng(16).uniform(-1, 1, rhs.size), trans=True)
