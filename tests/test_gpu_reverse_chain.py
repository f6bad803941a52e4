"""Where the reverse Runge-Kutta step keeps its cotangents: the result must not
depend on whether U_bar_n is a new array, U_bar_np1 itself or an array that
overlaps it, nor on recorded or recomputed stages."""
import pytest

from paper_2306_12891_amd import inputs as I
from test_gpu_parity import G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(equations=0), dict(equations=1, mu=1e-2), dict(equations=1, mu=1e-2, blending=1)])
def test_cotangent_arrays(kw):
    import torch

    from paper_2306_12891_amd import dg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kw = dict(kw)
    N, nelem = 4, (3, 2, 2)
    op = dg.DG(nelem, N, gamma=G, mu=kw.pop("mu", 0.0), vol_flux=dg.KG, surf_flux=dg.LLF, **kw)
    U = torch.from_numpy(I.random_smooth(N, nelem, seed=2, noise=0.02)).cuda()
    w = torch.from_numpy(I.random_directions(tuple(U.shape), 1)).cuda()
    dt = op.max_dt(U, 0.3)
    ref = op.rk_step_vjp(U, dt, w)
    Y = torch.empty((5,) + tuple(U.shape), dtype=torch.float64, device="cuda")
    op.rk_step_record(U.clone(), dt, Y)
    a = w.clone()
    assert torch.equal(op.rk_step_vjp(U, dt, a, out=a), ref)
    n = U.numel()
    for shift in (7, n // 2):
        buf = torch.zeros(n + shift, dtype=torch.float64, device="cuda")
        src, dst = buf[:n].view(U.shape), buf[shift:].view(U.shape)
        src.copy_(w)
        assert torch.equal(op.rk_step_vjp_recorded(Y, dt, src, out=dst), ref)
