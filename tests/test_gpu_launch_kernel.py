"""GPU: wadg_launch_kernel names the kernel that a call runs, read off the
workgroups that the call launches: 512 threads (pipelined), a workgroup per 16
elements (quarter) or per slice (whole sweep), else four waves per item (split)
or the resident kernel's ranges."""

import pytest

from graph_nodes import kernel_nodes
from workloads import periodic_quad_mesh

pytestmark = pytest.mark.gpu


def launched(W, sol, S, rhs=False, fp32=False):
    """The kernel of the second stage (of the only launch) of a call."""
    Q = sol.empty_state(S)
    if rhs:
        out = sol.empty_state(S)
        nodes = kernel_nodes(lambda s: sol.rhs(Q, S, out=out, stream=s))
    else:
        work = sol.workspace_fp32(S) if fp32 else sol.workspace(S)
        run = sol.integrate_fp32 if fp32 else sol.integrate
        nodes = kernel_nodes(lambda s: run(Q, S, 1e-3, 1, work=work, stream=s))
    if not rhs and len(nodes) == 1 and nodes[0][0] == S:
        return W.WADG_KERNEL_SWEEP
    G, sets = -(-sol.K // 64), -(-sol.K // 16)
    stages = nodes[:] if rhs else [n for n in nodes if nodes.count(n) >= 4]
    assert stages, nodes
    grid, threads = stages[0]
    if threads == 512:
        return W.WADG_KERNEL_PIPE
    if grid == sets * S and threads == 64 * (1 + (2 * sol.nq1 + 3) // 4):
        return W.WADG_KERNEL_QUARTER
    assert (grid, threads) == (G * S, 256), nodes
    return W.WADG_KERNEL_SPLIT


@pytest.mark.parametrize("N,nq1,K1D,S,rhs,fp32", [
    (3, 5, 4, 100, False, False), (3, 5, 4, 100, False, True), (3, 5, 4, 100, True, False),
    (3, 5, 9, 4, False, False), (3, 5, 64, 40, False, False), (3, 5, 64, 40, False, True),
    (3, 5, 64, 1, False, False), (3, 5, 64, 40, True, False), (3, 5, 100, 1, True, False),
    (4, 6, 50, 32, False, False), (4, 6, 50, 32, True, False), (4, 6, 50, 6, False, False),
    (3, 6, 64, 64, False, False), (3, 6, 9, 2, True, False), (2, 4, 81, 24, False, True)])
def test_launch_kernel_names_what_runs(N, nq1, K1D, S, rhs, fp32):
    import paper_1608_03836_amd as W
    print("CASE", f"launch kernel N={N} nq1={nq1} K1D={K1D} S={S} rhs={rhs} fp32={fp32}",
          flush=True)
    sol = W.Solver(periodic_quad_mesh(K1D, N, eps=0.05), nq1=nq1)
    assert sol.kernel_in_use(rhs=rhs, fp32=fp32, S=S) == launched(W, sol, S, rhs, fp32)
    for kernel in (W.WADG_KERNEL_STREAMED, W.WADG_KERNEL_SPLIT):
        sol.set_kernel(kernel)
        assert sol.kernel_in_use(rhs=rhs, fp32=fp32, S=S) == kernel


def test_launch_kernel_refuses():
    import paper_1608_03836_amd as W
    sol = W.Solver(periodic_quad_mesh(4, 3, eps=0.05))
    for S, rhs, fp32 in ((0, False, False), (1, True, True)):
        with pytest.raises(W.WadgError) as e:
            W.wadg_launch_kernel(sol.ctx, S, rhs, fp32)
        assert e.value.status == W.binding.WADG_E_INVALID
    with pytest.raises(W.WadgError):
        sol.set_kernel(W.WADG_KERNEL_QUARTER)


# Where the quarter kernel stops to pay: (N, nq1, K1D, S, rhs, fp32), kernel
QUARTER_EDGES = [
    (3, 5, 64, 2, False, True, "QUARTER"), (3, 5, 64, 4, False, True, "PIPE"),
    (4, 7, 17, 43, False, True, "PIPE"), (4, 5, 48, 4, False, True, "QUARTER"),
    (3, 5, 127, 1, False, True, "QUARTER"), (1, 2, 64, 1, False, True, "QUARTER"),
    (1, 2, 64, 2, False, True, "PIPE"), (1, 4, 64, 2, False, True, "QUARTER"),
    (2, 3, 32, 4, False, True, "QUARTER"), (2, 3, 32, 5, False, True, "PIPE"),
    (3, 6, 64, 1, False, False, "QUARTER"), (3, 6, 78, 1, False, False, "SPLIT"),
    (3, 6, 78, 1, True, False, "QUARTER"), (2, 3, 32, 6, False, False, "PIPE"),
    (3, 5, 78, 1, False, False, "QUARTER")]


@pytest.mark.parametrize("N,nq1,K1D,S,rhs,fp32,kernel", QUARTER_EDGES)
def test_quarter_kernel_where_it_is_faster(N, nq1, K1D, S, rhs, fp32, kernel):
    import paper_1608_03836_amd as W
    print("CASE", f"quarter edge N={N} nq1={nq1} K1D={K1D} S={S} rhs={rhs} fp32={fp32}",
          flush=True)
    sol = W.Solver(periodic_quad_mesh(K1D, N, eps=0.05), nq1=nq1)
    assert launched(W, sol, S, rhs, fp32) == getattr(W, "WADG_KERNEL_" + kernel)
    assert sol.kernel_in_use(rhs=rhs, fp32=fp32, S=S) == getattr(W, "WADG_KERNEL_" + kernel)


# Where a sweep in one workgroup per slice stops to pay
SWEEP_EDGES = [  # N, nq1, K1D, S, fp32, in one launch
    (3, 5, 6, 2048, True, True), (3, 5, 6, 2049, True, False), (3, 5, 6, 7281, True, False),
    (3, 5, 6, 7282, True, True), (3, 5, 6, 2048, False, True), (3, 5, 6, 3640, False, False),
    (3, 5, 6, 3641, False, True), (3, 6, 6, 4096, True, True), (3, 4, 6, 4096, True, True),
    (4, 6, 6, 4096, False, True), (4, 7, 6, 1, False, False), (4, 7, 6, 256, False, True),
    (4, 7, 6, 257, False, False), (4, 7, 6, 1024, True, True), (4, 7, 5, 1024, False, True),
    (3, 6, 8, 256, False, True), (3, 6, 8, 257, False, False), (3, 6, 8, 512, True, True),
    (3, 5, 8, 96, False, False), (3, 5, 8, 97, False, True), (3, 6, 8, 64, False, False),
    (3, 5, 8, 512, False, True), (3, 5, 8, 513, False, False), (2, 4, 6, 1024, False, True),
    (2, 4, 6, 1025, True, False)]


@pytest.mark.parametrize("N,nq1,K1D,S,fp32,one", SWEEP_EDGES)
def test_one_launch_sweep_where_it_is_faster(N, nq1, K1D, S, fp32, one):
    """The rule's edges, and the split kernel's bits on both sides of them."""
    import torch
    import paper_1608_03836_amd as W
    print("CASE", f"sweep edge N={N} nq1={nq1} K1D={K1D} S={S} fp32={fp32}", flush=True)
    sol = W.Solver(periodic_quad_mesh(K1D, N, eps=0.05, warp="skew", rotate_seed=K1D), nq1=nq1)
    assert (launched(W, sol, S, fp32=fp32) == W.WADG_KERNEL_SWEEP) == one
    g = torch.Generator(device="cuda").manual_seed(K1D)
    Q0 = torch.randn(S * sol.slice_doubles, dtype=torch.float64, device="cuda", generator=g)
    out = []
    for kernel in (W.WADG_KERNEL_SPLIT, W.WADG_KERNEL_AUTO):
        sol.set_kernel(kernel)
        Q = Q0.clone()
        (sol.integrate_fp32 if fp32 else sol.integrate)(Q, S, 0.1 / (K1D * (N + 1) ** 2), 2)
        out.append(Q.view(S, -1, 3 * (N + 1) ** 2, 64)[..., :sol.K])
    assert torch.isfinite(out[0]).all() and torch.equal(*out)
