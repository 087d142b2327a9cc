"""NaN and infinities in one cycle of a collapsed hierarchy: they reach what depends
on the entry that holds them, no block more than the oracle's cycle, which visits the
levels one by one, and every other entry is the oracle's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from nair_inputs import make_config
from test_gpu_parity import build_pair, np_, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("name,N,kw", [("dg_q1_32", 32, {}), ("dg_q1_32", 32, dict(cycle="F")),
                                       ("dg_q2_256_curved", 24, {}), ("dg_q2_256_curved", 24, dict(precision="fp32"))])
def test_what_does_not_depend_stays_finite(name, N, kw, bad):
    _say(f"test: {bad} in a cycle, {name} N={N} {kw}")
    S, k = make_config(name, N=N)
    G, O = build_pair(S.nb, S.bs, S.rowptr, S.colidx, S.vals, gpu_kw=kw, degree=k)
    C = np.flatnonzero(O.level(0).cf == 1)
    tol = 1e-4 if kw.get("precision") == "fp32" else 1e-12
    reach = []
    for trans in (False, True):
        g = G.vcycle_T if trans else G.vcycle
        o = O.vcycle_T if trans else O.vcycle
        for I in C[::max(1, len(C) // 12)]:
            v = np.random.default_rng(3).uniform(-1, 1, S.n)
            v[I * S.bs] = bad
            with np.errstate(all="ignore"):
                eo = o(v).reshape(S.nb, S.bs)
            e = np_(g(torch.from_numpy(v).cuda())).reshape(S.nb, S.bs)
            out_g, out_o = ~np.isfinite(e).all(axis=1), ~np.isfinite(eo).all(axis=1)
            assert out_g[I] and not (out_g & ~out_o).any(), (trans, I, out_g.sum(), out_o.sum())
            assert np.abs(e[~out_o] - eo[~out_o]).max(initial=0.0) <= tol * np.abs(eo[~out_o]).max(initial=1.0)
            reach.append(int(out_g.sum()))
    assert min(reach) < S.nb // 10   # (some entry reaches a small part only)
