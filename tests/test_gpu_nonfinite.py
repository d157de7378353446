"""Infinite, NaN and very large operands in the products on split bf16 operands, and infinite weights in padded ones.  In fp32 an infinite pre-activation takes its
gate to the limit and a product with an infinite factor is infinite; a number above 3.38e38 is finite, though it rounds to
infinity in bf16.  The kernels give what fp32 arithmetic gives, in these rows and in the ones beside them."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import GpuSide, OracleSide, batch_np
from oracle import tgnn_oracle as O

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]

INF, NAN, HUGE = np.inf, np.nan, 3.4e38
assert np.float32(HUGE) < np.float32(INF) and HUGE > 3.39e38


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def same(got, ref, tol):
    """NaNs and infinities in the same places, everything else within tol of the largest finite magnitude."""
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    ref = np.where(np.abs(ref) > np.finfo(np.float32).max, np.copysign(INF, ref), ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(got), got, 0), np.where(np.isinf(ref), ref, 0))
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= tol * np.abs(ref[ok]).max()


# rows: a tile with four column groups (and k parts), two row blocks, three row blocks in rounds; a width that is no multiple
# of four; no edge features
@pytest.mark.parametrize("widths,n", [((100, 100, 172), 33), ((100, 100, 172), 2100), ((100, 100, 172), 13000), ((30, 7, 5), 1500),
                                      ((128, 16, 0), 4100)])
def test_gru_update(widths, n):
    from paper_2307_07649_amd import tgnn
    dm, dt, de = widths
    d = synth.ModelDims(n_nodes=50, d_mem=dm, d_time=dt, d_edge=de, d_static=0, n_heads=1, k=10, batch=400)
    p32 = synth.gen_params(d, seed=3, random_phase=True)
    ctx = tgnn.Context(d.n_nodes, dm, dt, de, 0, 1, 10, 400)
    rng = np.random.default_rng(n)
    mem = rng.uniform(-1, 1, (n, dm)).astype(np.float32); mail = rng.uniform(-1, 1, (n, 2 * dm)).astype(np.float32)
    ef = rng.standard_normal((n, de)).astype(np.float32)
    has = (rng.random(n) < 0.8).astype(np.int32)
    rows = rng.permutation(n)[:14]
    for r, v in zip(rows, (INF, -INF, HUGE, -HUGE, NAN)):
        mail[r, rng.integers(2 * dm)] = v
    for r, v in zip(rows[5:], (INF, HUGE, -HUGE, NAN)):
        mem[r, rng.integers(dm)] = v
    if de:
        for r, v in zip(rows[9:], (INF, -INF, HUGE, -HUGE, NAN)):
            ef[r, rng.integers(de)] = v
    has[rows[:13]] = 1; has[rows[13]] = 0       # (a row without a mail keeps its memory)
    mem_ts = rng.uniform(0, 1e6, n); mail_ts = mem_ts + rng.uniform(0, 1e6, n)
    s, _ = ctx.tgnn_gru_update(tgnn.Params.from_numpy(p32),
                               dict(mem=dev(mem), mail=dev(mail), mail_efeat=dev(ef) if de else torch.empty(n, 0, device="cuda"),
                                    mem_ts=dev(mem_ts), mail_ts=dev(mail_ts), has_mail=dev(has)))
    p = O.to_f64(p32)
    x = np.concatenate([mail, O.time_encode(mail_ts - mem_ts, p["time_w"], p["time_b"]), ef], axis=1).astype(np.float64)
    ref = O.gru_cell(x, mem.astype(np.float64), p["gru_wih"], p["gru_whh"], p["gru_bih"], p["gru_bhh"])
    ref = np.where(has[:, None] > 0, ref, mem)
    assert np.isfinite(ref[rows[:4]]).all()                       # what infinite gates leave is finite
    # (the row with a huge memory entry would set the scale of all)
    big = np.zeros(n, bool); big[rows[5:9]] = True
    same(s.cpu().numpy()[~big], ref[~big], 1e-5)
    same(s.cpu().numpy()[big], ref[big], 1e-5)


# node rows of 16 (small R), 32 and 64 per tile, of four and of eight k slabs
@pytest.mark.parametrize("widths,R", [((100, 100, 172, 0, 2), 5), ((100, 100, 172, 0, 2), 300), ((100, 100, 172, 0, 2), 900),
                                      ((100, 20, 31, 100, 2), 300), ((30, 9, 5, 3, 3), 97)])
def test_projections_and_their_weight_gradients(widths, R):
    from paper_2307_07649_amd import tgnn
    dm, dt_, de, ds, H = widths
    k = 10
    d = synth.ModelDims(n_nodes=50, d_mem=dm, d_time=dt_, d_edge=de, d_static=ds, n_heads=H, k=k, batch=400)
    p32 = synth.gen_params(d, seed=3, random_phase=True)
    ctx = tgnn.Context(d.n_nodes, dm, dt_, de, ds, H, k, 400)
    params = tgnn.Params.from_numpy(p32); grads = tgnn.Params.zeros_like(params)
    rng = np.random.default_rng(R)
    x_root = rng.uniform(-1, 1, (R, d.d_x)).astype(np.float32); x_nbr = rng.uniform(-1, 1, (R, k, d.d_x)).astype(np.float32)
    e = rng.standard_normal((R, k, de)).astype(np.float32); dt = rng.uniform(0, 3e5, (R, k))
    cnt = rng.integers(0, k + 1, R).astype(np.int32); cnt[0] = k
    dz = rng.standard_normal((R, dm)).astype(np.float32)
    # without neighbours the row's merge part is all there is: infinite, or of the order of the entry.  dz: a huge gradient
    j = 3
    for r, v in ((1, INF), (2, -INF), (3, HUGE)):
        x_root[r, j] = v; cnt[r] = 0
    cnt[4] = 0
    z = ctx.tgnn_temporal_attn_fwd(params, dev(x_root), dev(x_nbr.reshape(R * k, -1)), dev(e.reshape(R * k, -1)), dev(dt.reshape(-1)),
                                   dev(cnt)).cpu().numpy()
    mask = np.arange(k)[None] < cnt[:, None]
    p = O.to_f64(p32)
    ref, cache = O.attention_fwd(p, x_root.astype(np.float64), x_nbr * mask[..., None], e * mask[..., None], dt * mask,
                                 cnt.astype(np.int64), H)
    c = int(np.argmax(ref[4])); dz[4, c] = HUGE
    assert ref[4, c] > 0.01 and np.isinf(ref[1]).any() and np.isfinite(ref[3]).all() and ref[3].max() > 1e35
    own = np.zeros(R, bool); own[3] = True                        # (its own scale)
    same(z[~own], ref[~own], 1e-5)
    same(z[own], ref[own], 1e-5)
    dr, dn = ctx.tgnn_temporal_attn_bwd(params, dev(dz), grads)
    g, _, _ = O.attention_bwd(p, cache, dz.astype(np.float64), H)
    gg = grads.numpy()
    # the infinite entries of x reach column j of the weights that x meets, the huge gradient row c of W_o and b_o; all
    # other entries are as they would be without either
    for n in ("wo", "bo"):
        same(np.delete(gg[n], c, axis=0), np.delete(g[n], c, axis=0), 2e-5)
        same(gg[n][c], g[n][c], 2e-5)
    assert np.isfinite(np.delete(g["wo"], dm + j, axis=1)).all() and not np.isfinite(g["wo"][:, dm + j]).any()
    assert np.array_equal(np.isfinite(gg["wq"]), np.isfinite(g["wq"]))
    # (W_v meets the node rows of roots, too, with a gradient of zero: column j may be NaN)
    same(np.delete(gg["wv"], j, axis=1), np.delete(g["wv"], j, axis=1), 2e-5)
    same(gg["bv"], g["bv"], 2e-5)


# More tiles than workgroups (512 at a time, two column groups): the rows that a workgroup looks at once more are in its second
# tile, 32 rows high with eight k slabs and 64 with four.  Weights of column j are so small that a huge entry there leaves
# projections of ordinary size; the split operands cannot take the entry.
@pytest.mark.parametrize("widths,R", [((100, 20, 31, 100, 2), 800), ((100, 20, 0, 0, 2), 1600)])
def test_projections_in_rounds(widths, R):
    from paper_2307_07649_amd import tgnn
    dm, dt_, de, ds, H = widths
    k, j = 10, 3
    d = synth.ModelDims(n_nodes=50, d_mem=dm, d_time=dt_, d_edge=de, d_static=ds, n_heads=H, k=k, batch=600)
    p32 = synth.gen_params(d, seed=3, random_phase=True)
    for n, c in (("wk", j), ("wv", j), ("wq", j), ("wo", dm + j)):
        p32[n][:, c] *= np.float32(2.0 ** -122)
    ctx = tgnn.Context(d.n_nodes, dm, dt_, de, ds, H, k, 600)
    params = tgnn.Params.from_numpy(p32)
    rng = np.random.default_rng(R)
    x_root = rng.uniform(-1, 1, (R, d.d_x)).astype(np.float32); x_nbr = rng.uniform(-1, 1, (R, k, d.d_x)).astype(np.float32)
    e = rng.standard_normal((R, k, de)).astype(np.float32); dt = rng.uniform(0, 3e5, (R, k))
    cnt = np.full(R, k, np.int32)
    for r in (0, 1, R - 40, R - 39, R - 1):      # a slot of the first rows and of the last ones
        x_nbr[r, r % k, j] = HUGE if r % 2 else -HUGE
    x_root[2, j] = HUGE
    z = ctx.tgnn_temporal_attn_fwd(params, dev(x_root), dev(x_nbr.reshape(R * k, -1)), dev(e.reshape(R * k, -1)) if de else None,
                                   dev(dt.reshape(-1)), dev(cnt)).cpu().numpy()
    p = O.to_f64(p32)
    ref, _ = O.attention_fwd(p, x_root.astype(np.float64), x_nbr.astype(np.float64), e.astype(np.float64), dt, cnt.astype(np.int64), H)
    assert np.isfinite(ref).all()
    same(z, ref, 1e-5)


def test_training_step_with_an_infinite_mail():
    """A node whose cached mail has an infinite and a huge entry: the memory that the step writes is finite, and so are the
    gradients outside of the two columns of W_ih that these entries meet."""
    P = synth.custom_problem(n_nodes=40, E=600, d_mem=36, d_time=10, d_edge=7, d_static=0, n_heads=2, k=5, batch=60, seed=2)
    G = GpuSide(P); Or = OracleSide(P)
    for s in range(3):
        G.step([batch_np(P, 60 * s, 60 * (s + 1))], lr=0.0); Or.step([batch_np(P, 60 * s, 60 * (s + 1))], lr=0.0)
    b = batch_np(P, 180, 240)
    v = int(b["src"][0])
    assert Or.states[0]["mail_eid"][v] >= 0
    for i, x in ((5, INF), (50, -HUGE)):
        G.state.mail[v, i] = x; Or.states[0]["mail"][v, i] = np.float64(np.float32(x))
    g = G.step([b], lr=0.0); o = Or.step([b], lr=0.0, gpu=g)
    st = G.state_np()
    assert np.isfinite(st["mem"]).all() and np.isfinite(Or.states[0]["mem"]).all()
    same(st["mem"], Or.states[0]["mem"], 1e-4)
    same(st["mail"], Or.states[0]["mail"], 1e-4)
    assert abs(g["loss"] - o["loss"]) <= 1e-4 * abs(o["loss"])
    for n in ("gru_wih", "gru_whh", "gru_bih", "gru_bhh", "wv", "bv", "wo", "bo", "dec_ws", "dec_wd", "dec_b1", "dec_w2"):
        a, r = g["grads"][n], o["grads"][n]
        if n == "gru_wih":
            a, r = np.delete(a, (5, 50), axis=1), np.delete(r, (5, 50), axis=1)
        same(a, r, 1e-4)


# the classification head pads its products to 64 columns and classes: the last column's and the last class's weights infinite
@pytest.mark.parametrize("d_mem,classes", [(20, 5), (64, 56), (100, 64)])
def test_infinite_output_weights_of_the_classification_head(d_mem, classes):
    P = synth.custom_problem(n_nodes=40, E=120, d_mem=d_mem, d_time=8, d_edge=4, d_static=0, n_heads=2, k=3, batch=40,
                             n_classes=classes, n_true=1, seed=classes)
    P["params"]["dec_w2"] = P["params"]["dec_w2"].copy()
    P["params"]["dec_w2"][classes - 1, d_mem - 1] = INF
    P["params"]["dec_b1"] = P["params"]["dec_b1"].copy()
    P["params"]["dec_b1"][-1] = 5.0                      # (the unit that meets the infinite weight is on)
    G = GpuSide(P)
    g = G.step([batch_np(P, 0, 40)], lr=0.0)
    h = g["h1"].astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = h @ np.where(np.isinf(P["params"]["dec_w2"]), 0, P["params"]["dec_w2"]).astype(np.float64).T + P["params"]["dec_b2"]
        ref[:, -1] += h[:, -1] * INF
    assert (h[:, -1] > 0).all()
    same(g["logits"], ref, 1e-5)
    # d loss / d hidden: a sum over the classes with one infinite term, in the last hidden unit only
    gb = g["grads"]["dec_b1"]
    assert np.isfinite(gb[:-1]).all() and not np.isfinite(gb[-1])
