"""Rounding of a Runge-Kutta step with the deferred viscous exchange.

With the recorded stage states Y_k and the operator's own U_t at them, the step
U_n + sum_k B_k dt G_k is formed in extended precision; what rk_step returns
differs from it by the roundings of the state alone.  A state is rounded once per
stage, five times in a step, each time uniformly over one unit in the last place:
the root mean square over many nodes is sqrt(5 / 12) of that unit, with 5 % for
the sample.  So it must be at the nodes that get the neighbours' half of the
viscous term one launch later, too, where a second rounding would make it
sqrt(10 / 12).  And each stage state is the rounded sum of the one before and its
increment: the state after the first stage, which has one rounding, is off by half
a unit at most (and what the increment's own rounding adds).  Values that change
their binade, or by more than a twentieth in one stage, are left out.
"""
import numpy as np
import pytest

from paper_2306_12891_amd import inputs as I
from test_gpu_deferred import CASES, make, torch_cuda  # noqa: F401
from test_gpu_parity import G

pytestmark = pytest.mark.gpu

A = [0.0, -567301805773.0 / 1357537059087.0, -2404267990393.0 / 2016746695238.0,
     -3550918686646.0 / 2091501179385.0, -1275806237668.0 / 842570457699.0]
B = [1432997174477.0 / 9575080441755.0, 5161836677717.0 / 13612068292357.0,
     1720146321549.0 / 2090206949498.0, 3134564353537.0 / 4481467310338.0,
     2277821191437.0 / 14882151754819.0]


def state(N, nelem):
    """Smooth state with a mean flow in all directions, jumps between elements."""
    X = I.random_smooth(N, nelem, seed=31 * N, noise=1e-3, mach=0.1)
    rho, u = X[:, 0], [X[:, 1 + d] / X[:, 0] + 0.6 for d in range(3)]
    p = (G - 1.0) * (X[:, 4] - 0.5 * (X[:, 1] ** 2 + X[:, 2] ** 2 + X[:, 3] ** 2) / rho)
    return I.from_primitive(rho, *u, p, G)


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("N", [3, 5, 7])
def test_step_rounds_no_more_than_one_update_per_stage(torch_cuda, case, N):  # noqa: F811
    torch = torch_cuda
    nelem = (6, 5, 4) if N == 3 else (4, 3, 3)
    op = make(torch, case, N, nelem)
    U0 = torch.from_numpy(state(N, nelem)).cuda()
    dt = op.max_dt(U0, 0.05)
    U1 = U0.clone()
    Y = torch.empty((5,) + tuple(U0.shape), dtype=torch.float64, device="cuda")
    op.rk_step_record(U1, dt, Y)
    got, stages = U1.cpu().numpy(), Y.cpu().numpy()
    assert np.array_equal(stages[0], U0.cpu().numpy())
    ref, reg, use = U0.cpu().numpy().astype(np.longdouble), 0.0, np.ones(got.shape, dtype=bool)
    for k in range(5):
        reg = np.longdouble(A[k]) * reg + op.time_derivative(Y[k]).cpu().numpy()
        inc = np.longdouble(B[k] * dt) * reg
        ref = ref + inc
        if k == 0:
            first = ref
        use &= (np.abs(inc) < 0.05 * np.abs(got)) & (np.frexp(stages[k])[1] == np.frexp(got)[1])
    one = np.abs((stages[1] - first) / np.spacing(np.abs(stages[1])))[use]
    assert np.mean(one > 0.5) < 0.02 and one.max() < 0.6
    err = ((got - ref) / np.spacing(np.abs(got))).astype(float)
    ix = np.arange(N + 1)
    end = (ix == 0) | (ix == N)
    boundary = np.broadcast_to(end[:, None, None] | end[None, :, None] | end[None, None, :], got.shape)
    for what, m in (("boundary", use & boundary), ("inner", use & ~boundary)):
        assert m.sum() > 1000, (what, m.sum())
        rms = np.sqrt(np.mean(err[m] ** 2))
        assert rms <= 1.05 * np.sqrt(5.0 / 12.0), f"{what} nodes: {rms:.3f} units in the last place"
