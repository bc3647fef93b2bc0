"""GPU: the one-launch sweep of small meshes in more than one launch -- many
steps, which would hold their CUs throughout, or more slices than a launch has
lanes for -- gives the split kernel's bits, and no launch takes more than a
bounded share of the steps."""

import numpy as np
import pytest

from graph_nodes import kernel_nodes
from workloads import periodic_quad_mesh, c2_layered

pytestmark = pytest.mark.gpu


def _solver(N, nq1, K1D):
    import paper_1608_03836_amd as W
    mesh = periodic_quad_mesh(K1D, N, eps=0.05, warp="skew", rotate_seed=K1D)
    return W, mesh, W.Solver(mesh, nq1=nq1, c2=c2_layered)


@pytest.mark.parametrize("S,nsteps,launches", [(1, 512, 1), (1, 513, 2), (256, 1024, 2),
                                               (257, 1024, 4), (3000, 100, 3)])
def test_many_steps_are_cut(S, nsteps, launches):
    print("CASE", f"sweep launches S={S} nsteps={nsteps}", flush=True)
    W, mesh, sol = _solver(3, 5, 4)
    Q, w, w32 = sol.empty_state(S), sol.workspace(S), sol.workspace_fp32(S)
    for call in (lambda s: sol.integrate(Q, S, 1e-3, nsteps, work=w, stream=s),
                 lambda s: sol.integrate_fp32(Q, S, 1e-3, nsteps, work=w32, stream=s)):
        assert kernel_nodes(call) == [(S, 256)] * launches


@pytest.mark.parametrize("K1D,S,nsteps", [(4, 2, 514), (5, 600, 172)])
def test_cut_sweep_equals_split(K1D, S, nsteps):
    print("CASE", f"cut sweep K1D={K1D} S={S} nsteps={nsteps}", flush=True)
    W, mesh, sol = _solver(3, 5, K1D)
    Q0 = np.random.default_rng(K1D).standard_normal((S, 3, mesh.Np, mesh.K))
    dt, out = 0.1 / (K1D * 16), []
    for kernel in (W.WADG_KERNEL_SPLIT, W.WADG_KERNEL_AUTO):
        sol.set_kernel(kernel)
        Q, Q32 = sol.upload(Q0), sol.upload(Q0)
        sol.integrate(Q, S, dt, nsteps)
        sol.integrate_fp32(Q32, S, dt, nsteps)
        out.append((sol.download(Q, S), sol.download(Q32, S)))
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)


def test_more_slices_than_a_launch_has_lanes():
    """Recorded, never run: no launch of an accepted size passes 2^32 lanes."""
    from paper_1608_03836_amd import binding as B
    S = 11_500_000
    print("CASE", f"sweep launches S={S}", flush=True)
    W, mesh, sol = _solver(1, 4, 5)                  # two sets of three waves
    Q = 1 << 40                                      # (addresses of nothing)
    for call in (lambda s: B.wadg_integrate(sol.ctx, Q, 2 * Q, S, 1e-3, 1, s),
                 lambda s: B.wadg_integrate_fp32(sol.ctx, Q, 2 * Q, S, 1e-3, 1, s)):
        nodes = kernel_nodes(call)
        assert sum(g for g, _ in nodes) == S
        assert all(g * b < 2 ** 32 for g, b in nodes)
