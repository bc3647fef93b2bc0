"""GPU: the L2 norms' kernel at its edges: more items than one launch has lanes
for."""

import numpy as np
import pytest

from workloads import periodic_quad_mesh

pytestmark = pytest.mark.gpu


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
