"""Rows claimed for the distinct nodes of a step: with claim words per XCD and, on graphs with more nodes than these are kept
for, with one word per node; all blocks referring to a handful of nodes, and few of them referring to the same."""
import pytest

from gpu_common import GpuSide, OracleSide, batch_np, compare_state, compare_step, custom_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_nodes,batch,replicas", [(7, 700, 1), (7, 130, 3), (4_194_304, 60, 1), (4_194_305, 60, 1), (2_097_153, 40, 2)])
def test_claims(n_nodes, batch, replicas):
    P = custom_problem(n_nodes=n_nodes, E=4 * batch * replicas, d_mem=4, d_time=2, d_edge=1, d_static=0, n_heads=1, k=5, batch=batch, seed=9)
    G = GpuSide(P, n_replicas=replicas); Or = OracleSide(P, n_replicas=replicas)
    for s in range(3):
        b = [batch_np(P, (s * replicas + r) * batch, (s * replicas + r + 1) * batch) for r in range(replicas)]
        g = G.step(b, lr=0.01)
        o = Or.step(b, lr=0.01, gpu=g)
        compare_step(g, o, label=f"claims {n_nodes} {batch} step {s}")
    for r in range(replicas):
        compare_state(G.state_np(r), Or.states[r])
