"""GPU: the run length a batch is created with, read off the workgroups that a
stage launches."""

import numpy as np
import pytest

from graph_nodes import kernel_nodes
from workloads import periodic_quad_mesh

pytestmark = pytest.mark.gpu


def _batch(N, nq1, count, shapes):
    """count problems of 4 to 256 elements, 8 to 128 slices."""
    import paper_1608_03836_amd as W
    r = np.random.default_rng(shapes)
    nodes = np.exp(r.uniform(np.log(64), np.log(4096), count))
    k1d = np.clip(np.round(np.sqrt(nodes) / 4.0), 2, 16).astype(int)
    S = [int(s) for s in r.integers(8, 129, count)]
    return W.Batch([periodic_quad_mesh(int(k), N, eps=0.05) for k in k1d], S, nq1=nq1)


def _workgroups(batch):
    import torch
    Q = torch.zeros(batch.total, dtype=torch.float64, device="cuda")
    work, dt = batch.workspace(), np.full(len(batch.S), 1e-3)
    batch.integrate(Q, dt, 1, work=work)              # (uploads the step sizes)
    nodes = kernel_nodes(lambda s: batch.integrate(Q, dt, 1, work=work, stream=s))
    return max(nodes, key=nodes.count)


@pytest.mark.parametrize("N,nq1,count,shapes,kept", [
    (1, 2, 152, 6310, True), (1, 2, 241, 7046, True), (2, 4, 84, 8804, True),
    (1, 3, 3, 2, False), (3, 5, 250, 4, False)])
def test_default_runs_leave_16_for_a_clear_gain(N, nq1, count, shapes, kept):
    print("CASE", f"batch default N={N} nq1={nq1} count={count}", flush=True)
    batch = _batch(N, nq1, count, shapes)
    default = _workgroups(batch)
    batch.set_runs(16)
    assert (default == _workgroups(batch)) == kept


def test_tune_times_the_schedule_it_finds():
    """1,280 slices of one group: runs of 5 keep every CU busy for 7 steps, the
    nearest lengths for 10 and more, and the created batch has them."""
    import torch
    import paper_1608_03836_amd as W
    print("CASE batch tune", flush=True)
    batch = W.Batch([periodic_quad_mesh(8, 3, eps=0.05)], [1280])
    created = _workgroups(batch)
    Q = torch.zeros(batch.total, dtype=torch.float64, device="cuda")
    for runs in (None, 5, 16):                        # as created; the caller's; a slower one
        if runs:
            batch.set_runs(runs)
        _, _, tuned, us = batch.tune(Q, np.full(1, 1e-3), reps=10)
        assert tuned == 5 and us > 0.0
        assert _workgroups(batch) == created
