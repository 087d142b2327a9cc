"""Dense inverses of directly solved systems: orders around the tile, panel and
rows-per-thread edges of the two elimination kernels, dense random operators
(every column needs a row exchange), several orders in one batch, and singular
operators, against numpy's inverse.

Tolerance: both inverses come from eliminations with partial pivoting, whose
error is of the order n eps kappa |inv|; the bar is 4 n eps kappa max|inv|."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_parity import to_dev, _say, np_

pytestmark = pytest.mark.gpu


def dense_blocks(nb, bs, seed, shift=0):
    """All nb x nb blocks, entries U[-1, 1]; columns from `shift`."""
    rng = np.random.default_rng(seed)
    A = rng.uniform(-1.0, 1.0, (nb * bs, nb * bs))
    rp = (np.arange(nb + 1) * nb).astype(np.int32)
    ci = np.tile(np.arange(nb) + shift, nb).astype(np.int32)
    va = np.ascontiguousarray(A.reshape(nb, bs, nb, bs).transpose(0, 2, 1, 3).reshape(nb * nb, bs, bs))
    return A, rp, ci, va


def check_inverse(inv, A):
    ref = np.linalg.inv(A)
    n = len(A)
    bar = 4 * n * np.finfo(float).eps * np.linalg.norm(A, 2) * np.linalg.norm(ref, 2) * np.abs(ref).max()
    err = np.abs(inv - ref).max()
    assert err <= bar, (n, err, bar)


@pytest.mark.parametrize("nb,bs", [(1, 1), (3, 5), (16, 1), (1, 17), (9, 9), (5, 25), (127, 1), (32, 4), (43, 3),
                                   (10, 25), (57, 9), (32, 16), (27, 19), (64, 16), (41, 25), (128, 16), (82, 25)])
def test_inverse_of_dense_operators(nb, bs):
    _say(f"test: dense inverse nb={nb} bs={bs} n={nb * bs}")
    import paper_1704_05001_amd as P
    A, rp, ci, va = dense_blocks(nb, bs, 100 + nb * bs)
    H = P.Hierarchy(*to_dev(rp, ci, va), bs, P.Params(max_coarse_dofs=4096))
    lv = H.level(0)
    assert lv["coarsest"]
    inv = np_(lv["dense_inv"])
    check_inverse(inv, A)
    # one cycle is the product with the inverse (transposed: with its transpose)
    b = np.random.default_rng(7).uniform(-1, 1, nb * bs)
    for trans in (False, True):
        e = np_((H.vcycle_T if trans else H.vcycle)(torch.from_numpy(b).cuda()))
        want = (inv.T if trans else inv) @ b
        assert np.abs(e - want).max() <= 1e-12 * np.abs(inv).sum(axis=0 if trans else 1).max()


def test_batch_of_orders():
    """Orders below and above 128, 512 and 1024 in one batch: one LDS launch and two groups of panel launches."""
    _say("test: dense inverses, batch of orders")
    import paper_1704_05001_amd as P
    bs, sizes = 4, [3, 32, 33, 128, 40, 129, 256, 300, 1]
    parts, off, z = [], 0, 0
    for k, nb in enumerate(sizes):
        A, rp, ci, va = dense_blocks(nb, bs, 40 + k, shift=off)
        parts.append((A, rp[:-1] + z, ci, va))
        off += nb
        z += len(ci)
    rp = np.concatenate([p[1] for p in parts] + [[z]]).astype(np.int32)
    ci = np.concatenate([p[2] for p in parts])
    va = np.concatenate([p[3] for p in parts])
    H = P.Hierarchy(*to_dev(rp, ci, va), bs, P.Params(max_coarse_dofs=4096), sys_nb=sizes)
    lv = H.level(0)
    inv, sy = np_(lv["dense_inv"]).reshape(-1), H.systems(0)
    for k, p in enumerate(parts):
        n = sizes[k] * bs
        o = int(sy["dense_off"][k])
        check_inverse(inv[o:o + n * n].reshape(n, n), p[0])


@pytest.mark.parametrize("nb,bs", [(8, 4), (64, 4), (90, 9)])
@pytest.mark.parametrize("where", ["row", "column"])
def test_singular_operators_are_refused(nb, bs, where):
    _say(f"test: singular dense operator n={nb * bs} zero {where}")
    import paper_1704_05001_amd as P
    A, rp, ci, va = dense_blocks(nb, bs, 5)
    A[(nb * bs - 2,) if where == "row" else (slice(None), nb * bs - 2)] = 0.0
    va = np.ascontiguousarray(A.reshape(nb, bs, nb, bs).transpose(0, 2, 1, 3).reshape(nb * nb, bs, bs))
    with pytest.raises(P.NairError) as e:
        P.Hierarchy(*to_dev(rp, ci, va), bs, P.Params(max_coarse_dofs=4096))
    assert e.value.status == "ESINGULAR"
