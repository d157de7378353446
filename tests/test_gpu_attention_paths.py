"""The attention kernels' middle path (groups of four slots) against the generic path, which it replaces up to four heads,
d_e + d_t <= 320 and d_o <= 128: the same terms in the same order, so the outputs are equal bit for bit; gradients against
each other (their sums over roots are split differently from run to run)."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import rel_err

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# (d_mem, d_time, d_edge, heads, k): k around the groups of four and the largest; columns around the rounds of 64 and the
# limits, no edge features, a time block inside one round and across two; widths past the limits (generic on both sides)
@pytest.mark.parametrize("shape", [
    (12, 5, 3, 3, 1), (12, 5, 0, 4, 4), (72, 50, 33, 3, 17), (100, 100, 186, 4, 11), (128, 128, 192, 4, 20), (112, 64, 0, 4, 32),
    (66, 63, 65, 1, 13), (64, 64, 64, 2, 12), (33, 1, 256, 3, 5), (130, 20, 10, 2, 12), (40, 129, 192, 4, 6), (40, 9, 4, 5, 7),
])
def test_middle_path_equals_the_generic_path(shape):
    from paper_2307_07649_amd import tgnn
    dm, dt_, de, H, k = shape
    R = 53
    d = synth.ModelDims(n_nodes=50, d_mem=dm, d_time=dt_, d_edge=de, d_static=0, n_heads=H, k=k, batch=R)
    p32 = synth.gen_params(d, seed=3, random_phase=True)
    params = tgnn.Params.from_numpy(p32)
    rng = np.random.default_rng(k)
    x_root = dev(rng.uniform(-1, 1, (R, dm)).astype(np.float32)); x_nbr = dev(rng.uniform(-1, 1, (R * k, dm)).astype(np.float32))
    e = dev(rng.standard_normal((R * k, de)).astype(np.float32)); dt = dev(rng.uniform(0, 3e5, R * k))
    cnt = rng.integers(0, k + 1, R).astype(np.int32); cnt[0] = k; cnt[1] = 0
    dz = dev(rng.standard_normal((R, dm)).astype(np.float32))
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
