"""GPU: the norms' four-at-a-time reduction at its edges: fewer values than one
pass of the lanes, a pass and a remainder, and a ragged last group whose
padding lanes hold NaN."""

import numpy as np
import pytest

from workloads import periodic_quad_mesh

pytestmark = pytest.mark.gpu

# Sums of squares in chains of at most n / 16384 + 70 additions: 4e-14 at the
# largest n here, and as much for the reference's own.
RTOL = 1e-13


@pytest.mark.parametrize("N,K1D,S", [(1, 2, 3), (3, 9, 2), (2, 50, 65), (3, 64, 2), (4, 37, 1)])
def test_norms_ragged(N, K1D, S):
    import paper_1608_03836_amd as W
    print("CASE", f"norms N={N} K1D={K1D} S={S}", flush=True)
    mesh = periodic_quad_mesh(K1D, N, eps=0.05)
    sol = W.Solver(mesh)
    rng = np.random.default_rng(K1D)
    A, Bs = (rng.standard_normal((S, 3, mesh.Np, mesh.K)) for _ in range(2))
    tA, tB = sol.upload(A), sol.upload(Bs)
    if mesh.K % 64:
        for t in (tA, tB):
            t.view(S, -1, 3 * mesh.Np, 64)[:, -1, :, mesh.K % 64:] = float("nan")
    for Bn, t in ((Bs, tB), (np.zeros_like(Bs), None)):
        out = sol.norms(tA, t, S)
        d, b = (A - Bn).reshape(S, -1), Bn.reshape(S, -1)
        np.testing.assert_allclose(out[:, 0], np.linalg.norm(d, axis=1), rtol=RTOL, atol=0)
        np.testing.assert_allclose(out[:, 1], np.linalg.norm(b, axis=1), rtol=RTOL, atol=0)
        assert np.array_equal(out[:, 2], np.abs(d).max(axis=1)) and np.all(out[:, 3] == 1.0)
