"""The buffers that dg_set_options takes beforehand: options may change inside
the capture of a stream, whether the library was told of that stream or not; a
buffer that a step could not get is not asked for in every later step."""
import ctypes

import pytest

from paper_2306_12891_amd import inputs as I
from test_gpu_deferred import torch_cuda  # noqa: F401
from test_gpu_parity import G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("told", [True, False])
@pytest.mark.parametrize("equations", ["EULER", "NS"])
def test_options_inside_a_capture(torch_cuda, told, equations):  # noqa: F811
    """A context without options has neither buffer; captured, it gets none with
    the stream told (Python binding), and the library allocates without breaking
    the capture of a stream that it does not know of."""
    torch = torch_cuda
    from paper_2306_12891_amd import dg
    N, nelem, kw = 4, (3, 2, 2), dict(equations=getattr(dg, equations), vol_flux=dg.PI, surf_flux=dg.ROE)
    U0 = torch.from_numpy(I.random_smooth(N, nelem, seed=4, noise=0.01)).cuda()
    ref = dg.DG(nelem, N, gamma=G, mu=1e-2, **kw)
    dt = ref.max_dt(U0, 0.3)
    want = ref.rk_steps(U0.clone(), dt, 3)
    op = dg.DG(nelem, N, gamma=G, mu=1e-2)
    U = U0.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        if told:
            op.set_options(**kw)
        else:
            o = dg.default_options()
            for k, v in kw.items():
                setattr(o, k, v)
            assert op.raw_call("dg_set_options", ctypes.byref(o)) == dg.DG_OK
        op.rk_steps(U, dt, 3)
    for _ in range(3):
        U.copy_(U0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(U, want)


def test_refused_buffer_is_not_asked_for_again(torch_cuda):  # noqa: F811
    """The third state is taken where it is at most an eighth of the free memory;
    a step that found less does not look again, until the options are set."""
    torch = torch_cuda
    from paper_2306_12891_amd import dg
    N, nelem = 7, (24, 24, 24)
    op = dg.DG(nelem, N, gamma=G)
    U = torch.from_numpy(I.density_wave(N, nelem)).cuda()
    state = U.numel() * 8
    op.time_derivative(U)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = lambda: (torch.cuda.synchronize(), torch.cuda.mem_get_info()[0])[1]  # noqa: E731
    rest = torch.empty(free() - 4 * state, dtype=torch.uint8, device="cuda")
    before = free()
    op.rk_step(U, 1e-4)
    assert before - free() < state // 2
    del rest
    torch.cuda.empty_cache()
    before = free()
    op.rk_step(U, 1e-4)
    assert before - free() < state // 2
    op.set_options()
    assert before - free() >= state
