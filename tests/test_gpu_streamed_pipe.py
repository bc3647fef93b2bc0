"""GPU: automatic FP64 stages and right-hand sides whose geometry does not fit
on chip run, with enough slices per workgroup, on the form of the pipelined
kernel that streams it; they equal the split kernel's bit for bit at every
such degree and quadrature, on either side of that rule, on ragged groups, a
mesh numbered at random, and with and without non-temporal stores."""

import numpy as np
import pytest

from workloads import periodic_quad_mesh, c2_layered
from test_gpu_scattered import Renumbered

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nq1,K1D,S,random", [
    (4, 5, 33, 30, False), (4, 6, 41, 23, False), (4, 7, 33, 30, False), (3, 6, 33, 30, False),
    (4, 6, 41, 23, True), (3, 6, 110, 2, False), (4, 5, 90, 3, False), (4, 6, 50, 6, False),
    (4, 6, 128, 20, False), (4, 5, 160, 3, False)])
def test_streamed_pipe_equals_split(N, nq1, K1D, S, random):
    import torch
    import paper_1608_03836_amd as W
    print("CASE", f"streamed pipe N={N} nq1={nq1} K1D={K1D} S={S} random={random}", flush=True)
    mesh = periodic_quad_mesh(K1D, N, eps=0.05, warp="skew", rotate_seed=K1D)
    if random:
        mesh = Renumbered(mesh, np.random.default_rng(K1D).permutation(K1D * K1D))
    sol = W.Solver(mesh, nq1=nq1, c2=c2_layered)
    g = torch.Generator(device="cuda").manual_seed(K1D)
    Q0 = torch.randn(S * sol.slice_doubles, dtype=torch.float64, device="cuda", generator=g)
    lanes = Q0.view(S, -1, 3 * (N + 1) ** 2, 64)
    if sol.K % 64:
        lanes[:, -1, :, sol.K % 64:] = float("nan")    # padding holds no state
    real = torch.ones(sol.K, dtype=torch.bool, device="cuda")
    real = torch.nn.functional.pad(real, (0, -sol.K % 64)).view(1, -1, 1, 64).expand_as(lanes)
    out = []
    for kernel in (W.WADG_KERNEL_SPLIT, W.WADG_KERNEL_AUTO):
        sol.set_kernel(kernel)
        Q, dq = Q0.clone(), sol.empty_state(S)
        sol.integrate(Q, S, 1e-3, 2)                     # first, middle and last stages
        sol.rhs(Q0, S, out=dq)
        out.append((Q.view_as(lanes)[real], dq))
    assert torch.isfinite(out[0][0]).all() and torch.isfinite(out[0][1]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
