"""The node path (UPDT and the per-node projections on split bf16 operands) at the row counts where its tiling changes, at
widths with remainders in every block size, and the separate launches that take over where it does not fit."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import GpuSide, OracleSide, batch_np, compare_state, compare_step, custom_problem, rel_err
from oracle import tgnn_oracle as O

pytestmark = pytest.mark.gpu

# A pre-activation is a sum of K <= 1,600 products whose factors are at most 1/sqrt(K) and a few units: fp32 sums are off by
# less than K 2^-24 times the largest product, 9.5e-6 here in the worst case and under 1e-6 in practice; the gates and the
# projections that follow do not enlarge that.
NODE_TOL = 1e-5


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def dims(d_mem, d_time, d_edge, d_static=0, H=1, k=10, batch=400):
    return synth.ModelDims(n_nodes=50, d_mem=d_mem, d_time=d_time, d_edge=d_edge, d_static=d_static, n_heads=H, k=k, batch=batch)


def make(d):
    from paper_2307_07649_amd import tgnn
    p32 = synth.gen_params(d, seed=3, random_phase=True)
    ctx = tgnn.Context(d.n_nodes, d.d_mem, d.d_time, d.d_edge, d.d_static, d.n_heads, d.k, d.batch)
    return tgnn, ctx, p32, tgnn.Params.from_numpy(p32)


# rows: one tile, a remainder of one row, both sides of every change of row blocks and column groups (252 workgroups); inputs
# of 1,080 columns, whose tiles hold two row blocks, and of 1,242 and 1,500, which hold one: there the workgroups go through
# several units beyond 8,064 and 4,032 rows, with one column group and (under 4,032) with several
ROWS = [1, 15, 16, 17, 1008, 1009, 1344, 1345, 2017, 4033, 6049, 8065, 12097, 13200]


@pytest.mark.parametrize("widths,n", [((100, 100, 172), n) for n in ROWS]
                         + [(w, n) for w in ((128, 1, 255), (16, 5, 0), (7, 30, 3)) for n in (1, 17, 1345, 4033, 12097)]
                         + [((100, 100, 780), n) for n in (1009, 2017, 4032, 4033, 8065)]
                         + [((16, 10, 1200), n) for n in (33, 4100)] + [((100, 100, 1200), n) for n in (1345, 4033, 9000)])
def test_gru_update_row_counts(widths, n):
    d = dims(*widths)
    tgnn, ctx, p32, params = make(d)
    rng = np.random.default_rng(n)
    mem = rng.uniform(-1, 1, (n, d.d_mem)).astype(np.float32); mail = rng.uniform(-1, 1, (n, 2 * d.d_mem)).astype(np.float32)
    ef = rng.standard_normal((n, d.d_edge)).astype(np.float32)
    has = (rng.random(n) < 0.8).astype(np.int32)
    mem_ts = rng.uniform(0, 1e6, n); mail_ts = mem_ts + rng.uniform(0, 1e6, n)
    s, tau = ctx.tgnn_gru_update(params, dict(mem=dev(mem), mail=dev(mail), mail_efeat=dev(ef) if d.d_edge else torch.empty(n, 0, device="cuda"),
                                              mem_ts=dev(mem_ts), mail_ts=dev(mail_ts), has_mail=dev(has)))
    p = O.to_f64(p32)
    x = np.concatenate([mail, O.time_encode(mail_ts - mem_ts, p["time_w"], p["time_b"]), ef], axis=1).astype(np.float64)
    ref = O.gru_cell(x, mem.astype(np.float64), p["gru_wih"], p["gru_whh"], p["gru_bih"], p["gru_bhh"])
    ref = np.where(has[:, None] > 0, ref, mem)
    assert rel_err(s.cpu().numpy(), ref) <= NODE_TOL
    assert np.array_equal(tau.cpu().numpy(), np.where(has > 0, mail_ts, mem_ts))


# results over the inputs: a program that updates its staged rows in place, with one and with several column groups per tile
@pytest.mark.parametrize("n,tau_over", [(17, "mem_ts"), (1009, "mail_ts"), (4033, "mem_ts")])
def test_gru_update_in_place(n, tau_over):
    import ctypes
    d = dims(100, 100, 172)
    tgnn, ctx, _, params = make(d)
    rng = np.random.default_rng(n)
    mem_ts = rng.uniform(0, 1e6, n)
    rows = dict(mem=dev(rng.uniform(-1, 1, (n, d.d_mem)).astype(np.float32)), mail=dev(rng.uniform(-1, 1, (n, 2 * d.d_mem)).astype(np.float32)),
                mail_efeat=dev(rng.standard_normal((n, d.d_edge)).astype(np.float32)), mem_ts=dev(mem_ts),
                mail_ts=dev(mem_ts + rng.uniform(0, 1e6, n)), has_mail=dev((rng.random(n) < 0.8).astype(np.int32)))
    s, tau = ctx.tgnn_gru_update(params, rows)
    ptr = [rows[x].data_ptr() for x in ("mem", "mail", "mail_efeat", "mem_ts", "mail_ts", "has_mail")]
    rc = tgnn._lib.tgnn_gru_update(ctx.h, ctypes.byref(params.c), n, *ptr, rows["mem"].data_ptr(), rows[tau_over].data_ptr(),
                                   torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    assert torch.equal(rows["mem"], s) and torch.equal(rows[tau_over], tau)


# node rows 11 R of the stand-alone attention call: R lies inside every interval of the split into row blocks of 16, 32 and 64
# and eight to two column groups (512 workgroups: changes at 1,024, 1,360, 2,048, 2,720, 4,096, 5,440 and 8,192 rows), with
# remainders; one to three heads, a head boundary inside a column block, static columns (eight k slabs: the same splits, with 32
# rows at most)
@pytest.mark.parametrize("widths,R", [((100, 100, 172, 0, 2), R) for R in (1, 3, 93, 110, 186, 220, 300, 373, 600, 745, 1200)]
                         + [((100, 100, 131, 100, 2), R) for R in (3, 93, 110, 186, 220, 300, 373, 600, 745)]
                         + [((30, 9, 5, 3, 3), R) for R in (3, 745)])
def test_projections_row_counts(widths, R):
    d = dims(*widths)
    tgnn, ctx, p32, params = make(d)
    rng = np.random.default_rng(R)
    k = d.k
    x_root = rng.uniform(-1, 1, (R, d.d_x)).astype(np.float32); x_nbr = rng.uniform(-1, 1, (R, k, d.d_x)).astype(np.float32)
    e = rng.standard_normal((R, k, d.d_edge)).astype(np.float32); dt = rng.uniform(0, 3e5, (R, k))
    cnt = rng.integers(0, k + 1, R).astype(np.int32); cnt[0] = k
    z = ctx.tgnn_temporal_attn_fwd(params, dev(x_root), dev(x_nbr.reshape(R * k, -1)), dev(e.reshape(R * k, -1)),
                                   dev(dt.reshape(-1)), dev(cnt))
    mask = np.arange(k)[None] < cnt[:, None]
    ref, _ = O.attention_fwd(O.to_f64(p32), x_root.astype(np.float64), x_nbr * mask[..., None], e * mask[..., None], dt * mask,
                             cnt.astype(np.int64), d.n_heads)
    assert rel_err(z.cpu().numpy(), ref) <= NODE_TOL


# more tiles than run at once: the ones left over after the whole rounds in one to four (update) or to nine (projections) column
# groups, 64-row tiles and 32-row ones
@pytest.mark.parametrize("n", [12145, 14000, 16200, 20000])
def test_gru_update_last_round(n):
    test_gru_update_row_counts((100, 100, 172, 0, 1, 10, 700), n)


@pytest.mark.parametrize("widths,R", [((100, 100, 172, 0, 2, 10, 700), 1495), ((100, 100, 172, 0, 2, 10, 700), 1700), ((100, 100, 131, 100, 2), 760),
                                      ((100, 100, 131, 100, 2), 1100)])
def test_projections_last_round(widths, R):
    test_projections_row_counts(widths, R)


# where the node path does not fit: a memory wider than eight column blocks, a GRU input wider than the LDS tile, node rows
# of more than eight k slabs; and one just inside (a single row block per tile)
@pytest.mark.parametrize("shape", [
    dict(d_mem=130, d_time=10, d_edge=4, d_static=0, n_heads=2, k=4),
    dict(d_mem=16, d_time=10, d_edge=2500, d_static=0, n_heads=1, k=3),
    dict(d_mem=20, d_time=10, d_edge=6, d_static=300, n_heads=2, k=4),
    dict(d_mem=16, d_time=10, d_edge=1200, d_static=0, n_heads=1, k=3),
])
def test_step_at_the_limits_of_the_node_path(shape):
    P = custom_problem(n_nodes=60, E=240, batch=40, seed=5, **shape)
    G = GpuSide(P); Or = OracleSide(P)
    for s in range(4):
        b = batch_np(P, s * 40, (s + 1) * 40)
        g = G.step([b], lr=0.01)
        o = Or.step([b], lr=0.01, gpu=g)
        compare_step(g, o, label=f"{shape} step {s}")
    compare_state(G.state_np(), Or.states[0])
