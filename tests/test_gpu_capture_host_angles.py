"""A captured forward call with host angles: at every size of the matrices a replay
takes those of the plan's last forward call (few matrices are sent by kernel argument
outside a capture only)."""
import numpy as np
import pytest

import qf_inputs as qi
from oracle import sim
from tests.gpu_helpers import TOL, maxabs, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,layers,dtype", [(4, 1, "c64"), (4, 2, "c128"), (8, 12, "c64")])
def test_replay_takes_the_last_calls_angles(n, layers, dtype):
    import torch

    import paper_2409_17716_amd as qf
    c = qi.hea(3, n, layers, 5, pairs=[(0, 1)], clock=False)
    p = qf.plan_for(c, dtype)
    t = qf.new_state(n, 3, dtype)
    p.forward(t, c.theta)  # allocations before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream(), capture_error_mode="thread_local"):
        p.forward(t, c.theta)

    def replay(theta):
        qf.qf_state_init(t, n, 3, None)
        torch.cuda.synchronize()
        graph.replay()
        assert maxabs(to_np(t), sim.run(c, theta=theta)) <= TOL[dtype]
    replay(c.theta)
    replay(c.theta)
    other = c.theta + 0.3
    qf.qf_state_init(t, n, 3, None)
    p.forward(t, other)
    assert maxabs(to_np(t), sim.run(c, theta=other)) <= TOL[dtype]
    replay(other)
    replay(other)
