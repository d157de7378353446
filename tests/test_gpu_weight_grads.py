"""The weight-gradient products (columns by columns over all rows, on split bf16 operands) at the row counts where their
chunking changes and at tile widths with every kind of remainder, through the attention's backward call."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import rel_err
from oracle import tgnn_oracle as O

pytestmark = pytest.mark.gpu

# A gradient entry is a sum over M <= 133,100 rows; the fp32 partial sums of a wavefront hold at most 1,024 of them (a quarter of
# the longest chunk) and are off by a random walk of roundings, sqrt(1024) 2^-24 = 1.9e-6 of the sum's magnitude, and so are at
# most 512 chunks' sums that follow; cancellation raises that a few times.
GRAD_TOL = 2e-5


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# rows: below one 32-row step, both sides of a step, of a wavefront's and of a workgroup's share, of one chunk; widths: one
# head and several (their columns begin inside a 16-byte piece), remainders of 64 on both sides of 16, 32 and 48
@pytest.mark.parametrize("widths,R", [((100, 100, 172, 2), R) for R in (1, 2, 3, 11, 12, 31, 33, 127, 129, 2400)]
                         + [(w, R) for w in ((17, 12, 3, 1), (48, 40, 9, 3), (66, 47, 0, 2), (128, 33, 90, 4)) for R in (5, 187)])
def test_weight_gradients(widths, R):
    from paper_2307_07649_amd import tgnn
    dm, dt_, de, H = widths
    k = 10
    d = synth.ModelDims(n_nodes=50, d_mem=dm, d_time=dt_, d_edge=de, d_static=0, n_heads=H, k=k, batch=max((R + 2) // 3, 1))
    p32 = synth.gen_params(d, seed=3, random_phase=True)
    ctx = tgnn.Context(d.n_nodes, dm, dt_, de, 0, H, k, d.batch)
    params, grads = tgnn.Params.from_numpy(p32), None
    grads = tgnn.Params.zeros_like(params)
    rng = np.random.default_rng(R)
    x_root = rng.uniform(-1, 1, (R, dm)).astype(np.float32); x_nbr = rng.uniform(-1, 1, (R, k, dm)).astype(np.float32)
    e = rng.standard_normal((R, k, de)).astype(np.float32); dt = rng.uniform(0, 3e5, (R, k))
    cnt = rng.integers(0, k + 1, R).astype(np.int32); cnt[0] = k
    dz = rng.standard_normal((R, dm)).astype(np.float32)
    ctx.tgnn_temporal_attn_fwd(params, dev(x_root), dev(x_nbr.reshape(R * k, -1)), dev(e.reshape(R * k, -1)), dev(dt.reshape(-1)),
                               dev(cnt))
    mask = np.arange(k)[None] < cnt[:, None]
    p = O.to_f64(p32)
    _, cache = O.attention_fwd(p, x_root.astype(np.float64), x_nbr * mask[..., None], e * mask[..., None], dt * mask,
                               cnt.astype(np.int64), H)
    ctx.tgnn_temporal_attn_bwd(params, dev(dz), grads)
    # (a ReLU input within rounding of zero may be gated the other way: none at these seeds)
    g, _, _ = O.attention_bwd(p, cache, dz.astype(np.float64), H)
    gg = grads.numpy()
    for n in ("wq", "wk", "wv", "bv", "wo", "bo"):
        floor = 16 * 2.0 ** -24 * float(cache["abs_terms"][n].max()) if n in cache["abs_terms"] else 0.0
        err = float(np.abs(gg[n] - g[n]).max())
        assert err <= GRAD_TOL * float(np.abs(g[n]).max()) + floor, (n, err, float(np.abs(g[n]).max()))


# narrow tiles over so many rows that the shortest chunks would be more than the 64 that add to one tile; and, with 133,100 rows,
# over more than 64 of the longest: a bit of the masks stands for several
@pytest.mark.parametrize("widths,R", [((8, 2, 1, 1), 2400), ((4, 1, 0, 2), 1700), ((4, 1, 0, 2), 12100)])
def test_weight_gradients_many_chunks(widths, R):
    test_weight_gradients(widths, R)
