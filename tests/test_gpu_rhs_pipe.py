"""GPU: an automatic right-hand side runs on the pipelined kernel where its LDS
plan fits; it equals the split kernel's bit for bit on one slice, short and
long slice runs and ragged groups, with and without non-temporal stores."""

import numpy as np
import pytest

from workloads import periodic_quad_mesh, c2_layered

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,dq,K1D,S", [(3, 2, 40, 1), (3, 2, 33, 30), (3, 1, 25, 70), (2, 3, 29, 40),
                                        (1, 1, 41, 37), (3, 2, 128, 44)])
def test_rhs_pipelined_equals_split(N, dq, K1D, S):
    import torch
    import paper_1608_03836_amd as W
    print("CASE", f"rhs N={N} nq1={N + dq} K1D={K1D} S={S}", flush=True)
    mesh = periodic_quad_mesh(K1D, N, eps=0.05, warp="skew", rotate_seed=K1D)
    sol = W.Solver(mesh, nq1=N + dq, c2=c2_layered)
    g = torch.Generator(device="cuda").manual_seed(K1D)
    Q = torch.randn(S * sol.slice_doubles, dtype=torch.float64, device="cuda", generator=g)
    lanes = Q.view(S, -1, 3 * mesh.Np, 64)
    if mesh.K % 64:
        lanes[:, -1, :, mesh.K % 64:] = float("nan")    # padding holds no state
    want, got = sol.empty_state(S), sol.empty_state(S)
    sol.set_kernel(W.WADG_KERNEL_SPLIT)
    sol.rhs(Q, S, out=want)
    sol.set_kernel(W.WADG_KERNEL_AUTO)
    sol.rhs(Q, S, out=got)
    assert torch.isfinite(want).all()
    assert torch.equal(got, want)      # the padding lanes of both keep their zeros
