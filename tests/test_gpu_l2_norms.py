"""GPU: the L2 norms' kernels at their edges: a wave per item, per field and per
field and array, with ragged and full last groups, a non-finite value in a real
lane of A alone or in padding, more partials than a lane adds at a time, and
more items than one launch has lanes for."""

import numpy as np
import pytest

from oracle import WADGOracle
from workloads import periodic_quad_mesh

pytestmark = pytest.mark.gpu


# The geometries agree to 1e-12 relative; the sums, of at most 49 additions a
# lane, 9 per item and 11 per slice, to 1e-14.
RTOL = 1e-12


@pytest.mark.parametrize("N,nq1,K1D,S", [(1, 2, 7, 3), (1, 3, 8, 2), (1, 4, 130, 1), (2, 3, 9, 2),
                                         (2, 5, 130, 1), (3, 5, 9, 2), (4, 6, 8, 1)])
def test_l2_norms(N, nq1, K1D, S):
    import paper_1608_03836_amd as W
    print("CASE", f"l2 norms N={N} nq1={nq1} K1D={K1D} S={S}", flush=True)
    mesh = periodic_quad_mesh(K1D, N, eps=0.05)
    sol, o = W.Solver(mesh, nq1=nq1), WADGOracle(mesh, nq1=nq1)
    rng = np.random.default_rng(K1D)
    A, B = (rng.standard_normal((S, 3, mesh.Np, mesh.K)) for _ in range(2))
    tA, tB = sol.upload(A), sol.upload(B)
    if mesh.K % 64:
        for t in (tA, tB):
            t.view(S, -1, 3 * mesh.Np, 64)[:, -1, :, mesh.K % 64:] = float("nan")

    def norm(X):
        return np.array([o.l2_norm(x, nq=nq1) for x in X])

    np.testing.assert_allclose(sol.l2_norms(tA, tB, S), np.stack([norm(A - B), norm(B)], 1),
                               rtol=RTOL, atol=0)
    np.testing.assert_allclose(sol.l2_norms(tA, None, S), np.stack([norm(A), 0 * norm(A)], 1),
                               rtol=RTOL, atol=0)
    # a real lane of A, in the last group: only its slice's norm of A - B
    want = sol.l2_norms(tA, tB, S)
    tA.view(S, -1, 3 * mesh.Np, 64)[S - 1, -1, 2 * mesh.Np, (mesh.K - 1) % 64] = float("nan")
    with pytest.raises(W.WadgError) as e:
        sol.l2_norms(tA, tB, S)
    assert e.value.status == W.binding.WADG_E_NONFINITE
    got = sol.l2_norms(tA, tB, S, check_finite=False)
    assert np.isnan(got[S - 1, 0]) and np.array_equal(got[:, 1], want[:, 1])
    assert np.array_equal(got[:S - 1], want[:S - 1])


def test_more_items_than_a_launch_has_lanes():
    """22.5 million slices of one group (138 GB): past 2^32 lanes with three
    waves per item as with six.  All but three slices are zero."""
    import gc
    import torch
    import paper_1608_03836_amd as W
    S, mesh = 22_500_000, periodic_quad_mesh(8, 1, eps=0.05)
    sol = W.Solver(mesh, nq1=2)
    n1 = sol.slice_doubles
    gc.collect()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GB of free device memory")
    print("CASE", f"l2 norms S={S}", flush=True)
    at = [0, 11_300_000, S - 1]
    some = sol.upload(np.random.default_rng(1).standard_normal((3, 3, mesh.Np, mesh.K)))
    want = sol.l2_norms(some, some, 3)
    A = torch.zeros(S * n1, dtype=torch.float64, device="cuda")
    for i, s in enumerate(at):
        A[s * n1:(s + 1) * n1] = some[i * n1:(i + 1) * n1]
    pair, alone = sol.l2_norms(A, A, S), sol.l2_norms(A, None, S)
    sol._scratch = None
    del A
    torch.cuda.empty_cache()
    expect = np.zeros((S, 2))
    expect[at] = want
    assert np.array_equal(pair, expect)                    # ||A - A|| = 0, ||A||
    assert np.array_equal(alone, expect[:, ::-1])          # ||A||, 0
