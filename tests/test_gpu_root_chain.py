"""Where the attention output and G lie inside the root chain and where they are products of their own: columns of a root's
weighted sums at and past 1,024, 1,536 and 2,304, few events and 600, one batch and two, both tile heights, against the oracle."""
import pytest

import synth
from gpu_common import GpuSide, OracleSide, batch_np, compare_state, compare_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_edge,heads,batch,replicas,wide", [
    (500, 2, 17, 1, False), (501, 2, 17, 1, False), (501, 2, 17, 1, True), (501, 2, 300, 2, False), (1140, 2, 600, 1, False),
    (1141, 2, 600, 1, True), (372, 4, 600, 1, False), (373, 4, 600, 1, False), (245, 4, 33, 2, True),
])
def test_wide_rows_of_weighted_sums(d_edge, heads, batch, replicas, wide):
    from paper_2307_07649_amd import tgnn
    P = synth.custom_problem(n_nodes=60, E=3 * batch * replicas, d_mem=32, d_time=12, d_edge=d_edge, d_static=0, n_heads=heads, k=4,
                             batch=batch, seed=d_edge)
    G = GpuSide(P, n_replicas=replicas, flags=tgnn.FLAG_WIDE_ROOT_TILES if wide else 0); Or = OracleSide(P, n_replicas=replicas)
    for s in range(3):
        b = [batch_np(P, (s * replicas + r) * batch, (s * replicas + r + 1) * batch - r * (batch // 3)) for r in range(replicas)]
        g = G.step(b, lr=0.01)
        o = Or.step(b, lr=0.01, gpu=g)
        compare_step(g, o, label=f"root chain {d_edge} {heads} {batch} step {s}")
    for r in range(replicas):
        compare_state(G.state_np(r), Or.states[r])
