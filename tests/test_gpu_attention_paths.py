"""The attention kernels' middle path (groups of four slots) against the generic path, which it replaces up to four heads,
d_e + d_t <= 320 and d_o <= 128: the same terms in the same order, so the outputs are equal bit for bit; gradients against
each other (their sums over roots are split differently from run to run).  Both against the oracle."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import GpuSide, OracleSide, batch_np, compare_state, compare_step, custom_problem, rel_err
from oracle import tgnn_oracle as O

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# (d_mem, d_time, d_edge, heads, k): k around the groups of four and the largest; columns around the rounds of 64 and the
# limits of the kernels of one, two and five rounds, no edge features, a time block inside one round and across two; widths past
# the limits (generic on both sides)
@pytest.mark.parametrize("shape", [
    (12, 5, 3, 3, 1), (12, 5, 0, 4, 4), (72, 50, 33, 3, 17), (100, 100, 186, 4, 11), (128, 128, 192, 4, 20), (112, 64, 0, 4, 32),
    (66, 63, 65, 1, 13), (64, 64, 64, 2, 12), (33, 1, 256, 3, 5), (130, 20, 10, 2, 12), (40, 129, 192, 4, 6), (40, 9, 4, 5, 7),
    (32, 8, 0, 1, 11), (39, 33, 32, 3, 5), (24, 100, 29, 1, 12),
])
def test_middle_path_equals_the_generic_path(shape, R=53):
    from paper_2307_07649_amd import tgnn
    dm, dt_, de, H, k = shape
    d = synth.ModelDims(n_nodes=50, d_mem=dm, d_time=dt_, d_edge=de, d_static=0, n_heads=H, k=k, batch=R)
    p32 = synth.gen_params(d, seed=3, random_phase=True)
    params = tgnn.Params.from_numpy(p32)
    rng = np.random.default_rng(k)
    host = dict(x_root=rng.uniform(-1, 1, (R, dm)).astype(np.float32), x_nbr=rng.uniform(-1, 1, (R * k, dm)).astype(np.float32),
                e=rng.standard_normal((R * k, de)).astype(np.float32), dt=rng.uniform(0, 3e5, R * k))
    x_root, x_nbr, e, dt = (dev(host[n]) for n in ("x_root", "x_nbr", "e", "dt"))
    cnt = rng.integers(0, k + 1, R).astype(np.int32); cnt[0] = k; cnt[1] = 0
    host["dz"] = rng.standard_normal((R, dm)).astype(np.float32)
    dz = dev(host["dz"])
    out = []
    for flags in (0, tgnn.FLAG_GENERIC_ATTN):
        ctx = tgnn.Context(d.n_nodes, dm, dt_, de, 0, H, k, R, flags=flags)
        grads = tgnn.Params.zeros_like(params)
        z = ctx.tgnn_temporal_attn_fwd(params, x_root, x_nbr, e, dt, dev(cnt)).cpu().numpy()
        dr, dn = ctx.tgnn_temporal_attn_bwd(params, dz, grads)
        out.append((z, dr.cpu().numpy(), dn.cpu().numpy(), grads.numpy()))
    (z0, r0, n0, g0), (z1, r1, n1, g1) = out
    assert np.array_equal(z0, z1)
    # fp32 sums of at most 53 x 32 terms in another order: 16 roundings of the largest entry
    assert rel_err(r0, r1) <= 2e-6 and rel_err(n0, n1) <= 2e-6
    for n in ("wv", "bv", "wo", "bo", "wq", "wk", "time_w", "time_b"):
        assert np.abs(g0[n] - g1[n]).max() <= 2e-5 * np.abs(g1[n]).max(), n
    # the oracle, in 64 bits: sums of at most 340 products per score and 32 slots, as in the projections (1e-5); weight
    # gradients over 53 roots, with sixteen roundings of the terms that cancel in the softmax's backward pass
    p = O.to_f64(p32)
    mask = (np.arange(k)[None] < cnt[:, None])
    ref, cache = O.attention_fwd(p, host["x_root"].astype(np.float64), host["x_nbr"].reshape(R, k, dm) * mask[..., None],
                                 host["e"].reshape(R, k, de) * mask[..., None], host["dt"].reshape(R, k) * mask, cnt.astype(np.int64), H)
    assert rel_err(z0, ref) <= 1e-5
    g, dxr, dxn = O.attention_bwd(p, cache, host["dz"].astype(np.float64), H)
    assert rel_err(r0, dxr[:, :dm]) <= 2e-5 and rel_err(n0.reshape(R, k, dm), dxn[:, :, :dm] * mask[..., None]) <= 2e-5
    for n in ("wv", "bv", "wo", "bo", "wq", "wk", "time_w", "time_b"):
        floor = 16 * 2.0 ** -24 * float(cache["abs_terms"][n].max()) if n in cache["abs_terms"] else 0.0
        assert np.abs(g0[n] - g[n]).max() <= 2e-5 * np.abs(g[n]).max() + floor, n


# many roots: a wavefront per root in the kernels of one, two and five rounds of columns (and a workgroup per root up to 400 of five)
@pytest.mark.parametrize("shape,R", [((32, 8, 0, 1, 11), 1500), ((32, 8, 0, 1, 11), 1501), ((36, 50, 33, 3, 17), 1200),
                                     ((36, 50, 33, 3, 17), 1201), ((40, 100, 186, 4, 11), 400), ((40, 100, 186, 4, 11), 401)])
def test_middle_path_row_counts(shape, R):
    from paper_2307_07649_amd import tgnn
    dm, dt_, de, H, k = shape
    d = synth.ModelDims(n_nodes=50, d_mem=dm, d_time=dt_, d_edge=de, d_static=0, n_heads=H, k=k, batch=R)
    params = tgnn.Params.from_numpy(synth.gen_params(d, seed=3, random_phase=True))
    rng = np.random.default_rng(R)
    x_root, x_nbr = (dev(rng.uniform(-1, 1, (n, dm)).astype(np.float32)) for n in (R, R * k))
    e, dt = dev(rng.standard_normal((R * k, de)).astype(np.float32)), dev(rng.uniform(0, 3e5, R * k))
    cnt = dev(rng.integers(0, k + 1, R).astype(np.int32))
    dz = dev(rng.standard_normal((R, dm)).astype(np.float32))
    out = []
    for flags in (0, tgnn.FLAG_GENERIC_ATTN):
        ctx = tgnn.Context(d.n_nodes, dm, dt_, de, 0, H, k, R, flags=flags)
        z = ctx.tgnn_temporal_attn_fwd(params, x_root, x_nbr, e, dt, cnt).cpu().numpy()
        dr, dn = ctx.tgnn_temporal_attn_bwd(params, dz, tgnn.Params.zeros_like(params))
        out.append((z, dr.cpu().numpy(), dn.cpu().numpy()))
    (z0, r0, n0), (z1, r1, n1) = out
    assert np.array_equal(z0, z1)
    assert rel_err(r0, r1) <= 2e-6 and rel_err(n0, n1) <= 2e-6   # (as above)


# a root more than the workgroup per root takes: the wavefront-per-root kernels of one, two and five rounds of columns, and of few
# neighbours; every gradient, against the generic path and the oracle (tolerances of above: sums over up to 17,425 rows)
@pytest.mark.parametrize("shape,R", [((32, 8, 0, 1, 11), 1350), ((32, 8, 0, 1, 11), 1351), ((33, 8, 20, 3, 8), 1181), ((36, 50, 33, 3, 17), 1024),
                                     ((36, 50, 33, 3, 17), 1025), ((36, 40, 60, 3, 5), 901), ((40, 100, 186, 4, 11), 401), ((36, 8, 0, 3, 4), 590),
                                     ((36, 8, 0, 3, 4), 591), ((36, 40, 60, 3, 3), 451), ((40, 100, 100, 4, 4), 201)])
def test_middle_path_gradients_around_the_row_counts(shape, R):
    test_middle_path_equals_the_generic_path(shape, R)


# the same kernels in a training step: rows looked up by node, the slot sort's fill pass beside them
@pytest.mark.parametrize("dm,dt_,de,H,k,batch", [(32, 8, 0, 1, 11, 450), (32, 8, 0, 1, 11, 451), (36, 50, 33, 3, 17, 341), (36, 50, 33, 3, 17, 342),
                                                 (36, 8, 0, 3, 4, 196), (36, 8, 0, 3, 4, 197), (40, 100, 186, 4, 11, 134)])
def test_middle_path_steps(dm, dt_, de, H, k, batch):
    P = custom_problem(n_nodes=500, E=8 * batch, d_mem=dm, d_time=dt_, d_edge=de, d_static=0, n_heads=H, k=k, batch=batch, seed=6)
    G = GpuSide(P); Or = OracleSide(P)
    for s in range(4, 7):
        b = batch_np(P, s * batch, (s + 1) * batch)
        g = G.step([b], lr=0.01)
        o = Or.step([b], lr=0.01, gpu=g)
        compare_step(g, o, label=f"middle path {dm} {k} {batch} step {s}")
    compare_state(G.state_np(), Or.states[0])
