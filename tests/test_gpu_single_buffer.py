"""Steps without the second face buffer or the third state (no memory, or a first
call under stream capture): the same bits as with them.

A context reaches that state for real: it is built with the two-pass lifting,
which takes no second face buffer, and only inside a capture, where nothing is
allocated, its options ask for the deferred exchange.  That the buffer was not
there is checked afterwards: the first call outside the capture takes it."""
import pytest

from paper_2306_12891_amd import inputs as I
from test_gpu_deferred import CASES, make, state, torch_cuda  # noqa: F401
from test_gpu_parity import G

pytestmark = pytest.mark.gpu

MESHES = [(2, (20, 16, 16)), (5, (10, 8, 8)), (7, (8, 6, 6))]  # a buffer of 4 MB at least


def takes_memory(torch, call, least):
    """The call allocates at least that much outside PyTorch's pool."""
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    call()
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] >= least


def captured(torch, calls):
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        calls()
    return g


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("N,nelem", MESHES)
def test_single_face_buffer(torch_cuda, case, N, nelem):  # noqa: F811
    torch = torch_cuda
    from paper_2306_12891_amd import dg
    kw, wall, warp = CASES[case]
    U0 = state(torch, N, nelem, 3 * N)
    w = torch.from_numpy(I.random_directions(tuple(U0.shape), 5)).cuda()
    new_record = lambda: torch.empty((5,) + tuple(U0.shape), dtype=torch.float64, device="cuda")  # noqa: E731

    ref = make(torch, case, N, nelem)
    dt = ref.max_dt(U0, 0.3)
    want = {"two": ref.rk_steps(U0.clone(), dt, 2), "three": ref.rk_steps(U0.clone(), dt, 3),
            "ut": ref.time_derivative(U0), "vjp": ref.rk_step_vjp(U0, dt, w), "Y": new_record()}
    want["recorded"] = ref.rk_step_record(U0.clone(), dt, want["Y"])

    op = dg.DG(nelem, N, gamma=G, mu=1e-2, equations=dg.NS, vol_flux=dg.PI, surf_flux=dg.ROE,
               lifting=dg.LIFT_TWO_PASS)
    op.rk_step_vjp(U0, dt, w)  # the reverse mode's buffers
    if kw.get("blending"):
        op.set_options(equations=dg.EULER, blending=1)
        op.vjp(U0, w)
        op.set_options(equations=dg.NS, blending=0)
    if warp:
        op.set_geometry(torch.from_numpy(I.warped_coordinates(N, nelem, amp=warp)).cuda())
    if wall is not None:
        op.set_wall_model(wall, 1.0, 0.4)
    got = {k: torch.empty_like(v) for k, v in want.items()}

    def calls():
        op.set_options(lifting=dg.LIFT_SPLIT, **kw)
        op.rk_steps(got["two"], dt, 2)
        op.rk_steps(got["three"], dt, 3)
        op.time_derivative(U0, out=got["ut"])
        op.rk_step_vjp(U0, dt, w, out=got["vjp"])
        op.rk_step_record(got["recorded"], dt, got["Y"])

    g = captured(torch, calls)
    for _ in range(3):
        for k in ("two", "three", "recorded"):
            got[k].copy_(U0)
        for k in ("ut", "vjp", "Y"):
            got[k].zero_()
        g.replay()
        ref.rk_step(U0.clone(), dt)  # work of its own between the replays
        torch.cuda.synchronize()
        for k in want:
            assert torch.equal(got[k], want[k]), k
    n1, elems = N + 1, op.n_elems
    takes_memory(torch, lambda: op.rk_step(got["two"], dt), elems * (24 * n1 ** 2 + n1 ** 3 // 2) * 8)


@pytest.mark.parametrize("N,nelem", MESHES)
def test_without_third_state(torch_cuda, N, nelem):  # noqa: F811
    torch = torch_cuda
    from paper_2306_12891_amd import dg
    U0 = state(torch, N, nelem, 11)
    ref = dg.DG(nelem, N, gamma=G, surf_flux=dg.LLF)
    dt = ref.max_dt(U0, 0.3)
    want = ref.rk_steps(U0.clone(), dt, 3)
    op = dg.DG(nelem, N, gamma=G)
    U = U0.clone()
    g = captured(torch, lambda: op.rk_steps(U, dt, 3))
    for _ in range(3):
        U.copy_(U0)
        g.replay()
        ref.rk_step(U0.clone(), dt)
        torch.cuda.synchronize()
        assert torch.equal(U, want)
    takes_memory(torch, lambda: op.rk_step(U, dt), U0.numel() * 8)
