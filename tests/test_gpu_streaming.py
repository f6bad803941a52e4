"""Stores past the caches or through them (chosen by the size of a mesh's data):
a periodic state repeated along the axes gives in every copy the bits of the
single one, whichever way the two meshes take."""
import numpy as np
import pytest

from paper_2306_12891_amd import inputs as I
from test_gpu_parity import G

pytestmark = pytest.mark.gpu


# 55 thousand nodes; 442 thousand (ordinary stores); 3.5 million (streaming)
@pytest.mark.parametrize("rep", [(2, 2, 2), (4, 4, 4)])
@pytest.mark.parametrize("kw", [dict(equations=0, vol_flux=0), dict(equations=1, mu=1e-2, vol_flux=1),
                                dict(equations=0, vol_flux=0, blending=1),
                                dict(equations=1, mu=1e-2, vol_flux=0, blending=1),
                                dict(equations=1, mu=1e-2, vol_flux=1, precision=1)])
def test_repeated_state(kw, rep):
    import torch

    from paper_2306_12891_amd import dg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kw = dict(kw)
    N, ne, hi = 5, (8, 8, 4), (1.0, 1.0, 0.5)
    mu = kw.pop("mu", 0.0)
    one = I.random_smooth(N, ne, hi=hi, seed=5, noise=0.02)
    n = one.reshape(ne[2], ne[1], ne[0], *one.shape[1:])
    many = np.tile(n, (rep[2], rep[1], rep[0], 1, 1, 1, 1)).reshape(-1, *one.shape[1:])
    out = []
    for m, h, U in ((ne, hi, one), (tuple(a * b for a, b in zip(ne, rep)), tuple(a * b for a, b in zip(hi, rep)), many)):
        op = dg.DG(m, N, hi=h, gamma=G, mu=mu, surf_flux=dg.LLF, **kw)
        V = torch.from_numpy(np.ascontiguousarray(U)).cuda()
        op.rk_steps(V, 1e-3, 3)
        out.append(V.cpu().numpy().reshape(m[2], m[1], m[0], *one.shape[1:]))
        op.close()
    a, b = out
    for kz, ky, kx in ((0, 0, 0), (rep[2] - 1, rep[1] - 1, rep[0] - 1)):
        sub = b[kz * ne[2]:(kz + 1) * ne[2], ky * ne[1]:(ky + 1) * ne[1], kx * ne[0]:(kx + 1) * ne[0]]
        assert np.array_equal(sub, a)
