"""GPU: the kernels of small launches -- a quarter of an element group per
workgroup (stage, right-hand side, the adjoint's products) and the whole sweep
of a small mesh in one launch -- give bit for bit what the split kernel
(WADG_KERNEL_SPLIT) gives, which the oracle tests cover.  Sizes at their edges:
one to four sets of 16 elements with ragged and full last sets, the largest
mesh of one workgroup and the next one, several groups with a ragged last one,
and every compiled quadrature (other numbers of pieces per phase)."""

import numpy as np
import pytest

from workloads import periodic_quad_mesh, c2_layered

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def W():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import paper_1608_03836_amd as pkg
    return pkg


CASES = [  # (N, nq1 - N, K1D, S, nsteps)
    (3, 2, 2, 3, 2), (3, 2, 4, 1, 3), (3, 2, 5, 2, 1), (3, 2, 6, 2, 2), (3, 2, 8, 2, 2),
    (3, 2, 9, 2, 2), (3, 2, 17, 1, 1), (3, 1, 7, 2, 2), (3, 3, 6, 1, 2), (3, 3, 8, 2, 1),
    (1, 1, 3, 2, 2), (1, 2, 8, 2, 1), (1, 3, 9, 3, 2), (2, 1, 7, 1, 2), (2, 2, 8, 2, 2),
    (2, 3, 5, 2, 1), (4, 1, 6, 2, 1), (4, 2, 6, 1, 2), (4, 2, 9, 2, 1), (4, 3, 7, 1, 1),
]


@pytest.mark.parametrize("N,dq,K1D,S,nsteps", CASES)
def test_small_launches_bitwise(W, N, dq, K1D, S, nsteps):
    print("CASE", f"quarter N={N} nq1={N + dq} K1D={K1D} S={S} nsteps={nsteps}", flush=True)
    mesh = periodic_quad_mesh(K1D, N, eps=0.05, warp="skew", rotate_seed=K1D)
    sol = W.Solver(mesh, nq1=N + dq, c2=c2_layered)
    sol.set_c2_scale(1.25)
    rng = np.random.default_rng(K1D + S)
    Q0 = rng.standard_normal((S, 3, mesh.Np, mesh.K))
    dt = 0.1 / (K1D * (N + 1) ** 2)
    out = []
    for kern in (W.WADG_KERNEL_SPLIT, W.WADG_KERNEL_AUTO):
        sol.set_kernel(kern)
        Q = sol.upload(Q0)
        # padding lanes hold no state, whatever their contents
        lanes = Q.view(S, -1, 3 * mesh.Np, 64)
        if mesh.K % 64:
            lanes[:, -1, :, mesh.K % 64:] = float("nan")
        dQ = sol.rhs(Q, S)
        Q32 = Q.clone()
        sol.integrate(Q, S, dt, nsteps)
        sol.integrate_fp32(Q32, S, dt, nsteps)
        chk = sol.forward_checkpoints(sol.upload(Q0[:1]), 2, dt, nsteps)
        grad, d = sol.adjoint(chk, sol.upload(Q0[-1:]), 2, dt, nsteps)
        out.append([sol.download(Q, S), sol.download(dQ, S), sol.download(Q32, S),
                    sol.download(chk, 3), sol.download(grad, 1), d])
    for a, b in zip(*out):
        assert np.all(np.isfinite(a))
        assert np.array_equal(a, b)


def test_one_launch_sweep_under_capture(W):
    """The one-launch sweep recorded into a HIP graph: every replay advances
    the state as an eager call does."""
    import torch
    mesh = periodic_quad_mesh(4, 3, eps=0.05, warp="skew", rotate_seed=2)
    sol = W.Solver(mesh, c2=c2_layered)
    S, dt = 3, 0.1 / 64
    Q0 = sol.upload(np.random.default_rng(1).standard_normal((S, 3, mesh.Np, mesh.K)))
    eager, Q, work = Q0.clone(), Q0.clone(), sol.workspace(S)
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        sol.integrate(eager.clone(), S, dt, 2, work=work)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=side):
        sol.integrate(Q, S, dt, 2, work=work)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        sol.integrate(eager, S, dt, 2)
        torch.cuda.synchronize()
        assert torch.equal(Q, eager)
