"""Two devices in one process: a hierarchy on each, whose setups need more than 64 KiB
of dynamic LDS a workgroup (splitting in one launch, dense inverse of up to 128
unknowns), which a device grants for itself."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from nair_inputs import make_config

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(torch.cuda.device_count() < 2, reason="needs two devices")]


def test_a_second_device_gets_what_the_first_gets():
    import paper_1704_05001_amd as P
    S, k = make_config("dg_q2_256_curved", N=40)
    out = []
    for dev in (0, 1):
        with torch.cuda.device(dev):
            d = [torch.from_numpy(a).cuda() for a in (S.rowptr, S.colidx, S.vals, S.rhs)]
            H = P.Hierarchy(*d[:3], S.bs, P.Params(degree=k))
            x, r = H.solve(d[3])
            out.append((x.cpu().numpy(), r.iters, r.status))
            H.close()
    assert out[0][1:] == out[1][1:] and np.array_equal(out[0][0], out[1][0])
