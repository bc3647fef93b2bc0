"""GPU: on a mesh numbered at random the launches walk the slices in another
order over the XCDs; the same physical problem on the row-numbered mesh gives
the same bits, element by element (the order of launch never enters a value),
with several slice runs per group, one, and the split kernel's items."""

import numpy as np
import pytest

from workloads import periodic_quad_mesh, c2_layered

pytestmark = pytest.mark.gpu


class Renumbered:
    """Element k of the mesh is element order[k] of `m`."""

    def __init__(self, m, order):
        at = np.argsort(order)
        self.N, self.x, self.y = m.N, m.x[order], m.y[order]
        self.etoe, self.etof = at[m.etoe[order]].astype(np.int32), m.etof[order]


@pytest.mark.parametrize("N,dq,K1D,S", [(3, 2, 24, 40), (3, 2, 66, 9), (2, 2, 33, 30), (4, 2, 20, 19),
                                        (1, 2, 60, 17)])
def test_random_numbering_bitwise(N, dq, K1D, S):
    import paper_1608_03836_amd as W
    print("CASE", f"scattered N={N} nq1={N + dq} K1D={K1D} S={S}", flush=True)
    rows = periodic_quad_mesh(K1D, N, eps=0.05, warp="skew", rotate_seed=3)
    order = np.random.default_rng(K1D).permutation(rows.K)
    Q0 = np.random.default_rng(S).standard_normal((S, 3, rows.Np, rows.K))
    dt = 0.1 / (K1D * (N + 1) ** 2)
    out = []
    for mesh, perm in ((rows, np.arange(rows.K)), (Renumbered(rows, order), order)):
        sol = W.Solver(mesh, nq1=N + dq, c2=c2_layered)
        Q = sol.upload(Q0[..., perm])
        Q32 = Q.clone()
        dQ = sol.rhs(Q, S)
        sol.integrate(Q, S, dt, 1)
        sol.integrate_fp32(Q32, S, dt, 1)
        got = np.empty((3,) + Q0.shape)
        for a, t in zip(got, (dQ, Q, Q32)):
            a[..., perm] = sol.download(t, S)
        out.append(got)
    assert np.all(np.isfinite(out[0]))
    assert np.array_equal(out[0], out[1])
