"""GPU: the run lengths and placement a batch is created with -- one problem,
few problems (whose runs are dealt over the XCDs) and many (a problem per XCD)
-- give the split kernel's bits."""

import numpy as np
import pytest

from workloads import make_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("members", [[12], [3], [3, 12], [0, 1, 2, 10, 12], list(range(40, 140))])
def test_default_runs_equal_split(members):
    import paper_1608_03836_amd as W
    print("CASE", f"batch runs {len(members)} from {members[0]}", flush=True)
    probs = make_batch(members=members)
    batch = W.Batch([p.mesh for p in probs], [p.S for p in probs])
    outs = []
    for runs in (None, 0):                       # as created; the item schedule
        if runs is not None:
            batch.set_runs(runs)
        Q = batch.upload([p.Q0 for p in probs])
        batch.integrate(Q, [p.dt for p in probs], 2)
        outs.append(batch.download(Q))
    for a, b in zip(*outs):
        assert np.isfinite(b).all() and np.array_equal(a, b)
