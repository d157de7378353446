"""The fp32 products A B^T of the separate launches, through a memory update whose nodes are too wide for the node path: 32-column
stages, chunks of four and an odd last 16 columns of the inner dimension, and both sides of every row count where tiles or
kernels change (gemm_nt_few_kernel, gemm_nt_kernel with tiles of 16 and of 32 columns; gemm_nt_counted_kernel, which chooses by a
row count that only the device knows)."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import GpuSide, OracleSide, batch_np, compare_state, compare_step, custom_problem, rel_err
from oracle import tgnn_oracle as O

pytestmark = pytest.mark.gpu

# Sums of K <= 1,029 fp32 products of weights below 1 / sqrt(K) and inputs of a few units at most, so that sums and partial sums are
# of a few units as well.  Each of K roundings is off by up to 2^-24 of the partial sum; as they fall either way that is about
# sqrt(K) 2^-24, 2e-6 per unit at the largest K (K 2^-24 times the sum of all magnitudes, which they would reach if they all
# fell the same way, is 1e-3).  Five times that; the gates do not enlarge it.
TOL = 1e-5


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# inner dimension 2 * 130 + 1 + d_edge: 272 (17 slabs of 16), 273, 288 (nine whole stages), 289, 384 (three whole chunks), 385,
# 1,029 (nine chunks, the last of one stage)
@pytest.mark.parametrize("d_edge", [11, 12, 27, 28, 123, 124, 768])
@pytest.mark.parametrize("n", [1, 16, 63, 64, 65, 1536, 1537, 4096, 4097])   # (52 tiles of 16 columns per 64 rows: one block up to 1,536)
def test_wide_memory_update(d_edge, n):
    from paper_2307_07649_amd import tgnn
    d = synth.ModelDims(n_nodes=50, d_mem=130, d_time=1, d_edge=d_edge, d_static=0, n_heads=1, k=10, batch=130)
    p32 = synth.gen_params(d, seed=3, random_phase=True)
    ctx = tgnn.Context(d.n_nodes, d.d_mem, d.d_time, d.d_edge, d.d_static, d.n_heads, d.k, d.batch)
    rng = np.random.default_rng(n + d_edge)
    mem = rng.uniform(-1, 1, (n, d.d_mem)).astype(np.float32); mail = rng.uniform(-1, 1, (n, 2 * d.d_mem)).astype(np.float32)
    ef = rng.standard_normal((n, d.d_edge)).astype(np.float32)
    has = (rng.random(n) < 0.8).astype(np.int32)
    mem_ts = rng.uniform(0, 1e6, n); mail_ts = mem_ts + rng.uniform(0, 1e6, n)
    s, _ = ctx.tgnn_gru_update(tgnn.Params.from_numpy(p32), dict(mem=dev(mem), mail=dev(mail), mail_efeat=dev(ef), mem_ts=dev(mem_ts),
                                                                  mail_ts=dev(mail_ts), has_mail=dev(has)))
    p = O.to_f64(p32)
    x = np.concatenate([mail, O.time_encode(mail_ts - mem_ts, p["time_w"], p["time_b"]), ef], axis=1).astype(np.float64)
    ref = O.gru_cell(x, mem.astype(np.float64), p["gru_wih"], p["gru_whh"], p["gru_bih"], p["gru_bhh"])
    assert rel_err(s.cpu().numpy(), np.where(has[:, None] > 0, ref, mem)) <= TOL


# Steps whose distinct nodes are few or many beside the same bound on their number (kernel for few rows, tiles of 32 columns):
# memory wider than the node path holds, where the GRU products are counted ones (52 tiles per 64 rows, the limit between 576 and
# 577 rows), with the inner dimensions of above for the kernel for few rows; and a time encoding of ten column tiles, whose
# gradient is one (limit between 3,264 and 3,265 rows).  Uniform graphs late in the stream: nearly every slot its own node.
# (At least eight time columns: the gradient of a single phase can cancel to nothing.  With one, the second of these steps on 640 nodes
# has -2.0e-8 from terms whose magnitudes add up to 1.5e-3, of which a rounding, 2^-24, is 0.45 % of the result.  With eight, the
# magnitudes are up to 77 times the tensor's largest entry in any of these steps, a rounding of them 4.6e-6, of 1e-4 allowed.)
@pytest.mark.parametrize("d_mem,d_time,d_edge,n_nodes,batch,rows", [(130, 8, e, 577, 80, (513, 576)) for e in (4, 5, 20, 21, 116, 117, 761)]
                         + [(130, 8, 3, 640, 120, (577, 640)), (130, 8, 3, 5000, 60, (1000, 1980)), (32, 130, 3, 4000, 160, (2000, 3264)),
                            (32, 130, 3, 12000, 200, (3265, 6600))])
def test_counted_rows(d_mem, d_time, d_edge, n_nodes, batch, rows):
    first = 14 * n_nodes
    P = custom_problem(n_nodes=n_nodes, E=first + 3 * batch, d_mem=d_mem, d_time=d_time, d_edge=d_edge, d_static=0, n_heads=2, k=10,
                       batch=batch, seed=5)
    G = GpuSide(P); Or = OracleSide(P)
    seen = []
    for s in range(3):
        b = batch_np(P, first + s * batch, first + (s + 1) * batch)
        g = G.step([b], lr=0.01)
        o = Or.step([b], lr=0.01, gpu=g)
        compare_step(g, o, label=f"counted rows {d_mem} {d_edge} {n_nodes} step {s}")
        seen.append(len(np.unique(np.concatenate([b["src"], b["dst"], b["neg"], g["nbr"][g["nbr"] >= 0]]))))
    assert rows[0] <= min(seen) and max(seen) <= rows[1], seen
    compare_state(G.state_np(), Or.states[0])
