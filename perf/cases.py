"""Timed workloads of the library, taken through the public binding (paper_2307_07649_amd.tgnn): training steps of
every kind, evaluation passes and the stand-alone operators, from a 200-event mini-batch to four 4,000-event ones.

A case is a dict of plain values.  `prepare` draws everything a trainer holds before it asks for a step (graph, edge
features, node memory as it stands in the middle of the event stream, weights, the mini-batches of the rest of the
stream), `run` does one call of a training or evaluation loop: the next mini-batch(es) in chronological order; at the end
of the stream the loop goes back to its first mini-batch with the memory as it was kept there, as passes over a
validation split or trainers that resume from a checkpoint do.
"""
import math

import numpy as np
import torch

from paper_2307_07649_amd import tgnn

# A mini-batch's values unless a case says otherwise: one replica, one negative destination per event, no static memory,
# plain SGD, one step per call.  n_src == 0: both endpoints over all nodes; otherwise sources are [0, n_src) and
# destinations [n_src, nodes), the recipe of the user-item graphs.
DEFAULTS = dict(n_src=0, skew_src=1.05, skew_dst=1.05, t_max=2.7e6, d_static=0, heads=2, k=10, replicas=1, negatives=1,
                classes=0, steps=1, adam=False, lr=1e-4)


def listed():
    return [dict(DEFAULTS, **c) for c in (
        # the smallest workload of the benchmark: a step is launches and latency, little else
        dict(name="tiny-step", path="train", nodes=1000, events=20_000, batch=200, d_mem=32, d_time=32, d_edge=16, heads=1,
             skew_src=0.0, skew_dst=0.0),
        # the ordinary user-item graph at the usual local batch size, one call per step
        dict(name="bipartite-step", path="train", nodes=9227, n_src=8227, skew_src=1.2, skew_dst=1.5, events=157_474,
             batch=600, d_mem=100, d_time=100, d_edge=172),
        # a denser graph with pre-trained static node memory, trained with Adam
        dict(name="static-memory-adam", path="train", nodes=10_984, n_src=10_000, skew_src=1.1, skew_dst=1.3,
             events=672_447, batch=600, d_mem=100, d_time=100, d_edge=172, d_static=100, adam=True),
        # memory parallelism: eight time-shifted replicas in one step
        dict(name="eight-replicas", path="train", nodes=10_984, n_src=10_000, skew_src=1.1, skew_dst=1.3, events=672_447,
             batch=600, d_mem=100, d_time=100, d_edge=172, d_static=100, replicas=8),
        # the large dense graph with the large batch, four consecutive steps per call: the headline of the benchmark
        dict(name="large-steps", path="train", nodes=16_682, events=2_000_000, t_max=1.4e5, batch=4000, d_mem=100,
             d_time=100, d_edge=186, steps=4),
        # a graph without edge features
        dict(name="no-edge-features", path="train", nodes=7144, n_src=7047, skew_src=0.9, skew_dst=1.0, t_max=2.6e7,
             events=411_749, batch=600, d_mem=100, d_time=100, d_edge=0, d_static=100, steps=4),
        # epoch parallelism on one GPU: four negative sets per positive mini-batch
        dict(name="epoch-parallel", path="train", nodes=9227, n_src=8227, skew_src=1.2, skew_dst=1.5, events=157_474,
             batch=600, d_mem=100, d_time=100, d_edge=172, negatives=4),
        # validation: every true destination ranked among 49 sampled ones
        dict(name="evaluation", path="eval", nodes=9227, n_src=8227, skew_src=1.2, skew_dst=1.5, events=157_474, batch=600,
             d_mem=100, d_time=100, d_edge=172, negatives=49),
        # edge classification with 56 classes
        dict(name="edge-classes", path="train", nodes=16_682, events=2_000_000, t_max=1.4e5, batch=4000, d_mem=100,
             d_time=100, d_edge=130, classes=56),
        # widths, head count and neighbour count that are no multiple of anything, a ragged batch
        dict(name="odd-widths", path="train", nodes=3001, events=60_000, batch=333, d_mem=72, d_time=50, d_edge=33,
             d_static=20, heads=3, k=17),
        # the operators one by one, as a program that builds its own step calls them: sample, gather, memory update,
        # attention forward and backward, write-back
        dict(name="operators", path="operators", nodes=9227, n_src=8227, skew_src=1.2, skew_dst=1.5, events=157_474,
             batch=600, d_mem=100, d_time=100, d_edge=172),
    )]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: batches of 32 to 4,000 events, memory widths 24 to 128, up to 20 neighbours, 4 heads,
    8 replicas, 49 negative destinations, 64 classes, at most the roots and widths of the large listed case."""
    largest = next(c for c in listed() if c["name"] == "large-steps")
    while True:
        c = dict(DEFAULTS, path=rng.choice(["train", "train", "train", "train", "eval", "operators"]))
        c["nodes"] = _log_int(rng, 500, 17_000)
        if rng.random() < 0.5:
            c["n_src"] = int(c["nodes"] * rng.uniform(0.5, 0.95))
        c["skew_src"], c["skew_dst"] = round(rng.uniform(0.0, 1.3), 2), round(rng.uniform(0.0, 1.5), 2)
        c["batch"] = _log_int(rng, 32, 4000)
        c["events"] = min(2_000_000, c["batch"] * _log_int(rng, 60, 500) + rng.randrange(c["batch"]))
        c["heads"] = rng.choice([1, 2, 2, 2, 4])
        c["d_mem"] = c["heads"] * rng.randint(24 // c["heads"], 128 // c["heads"])
        c["d_time"] = rng.randint(16, 128)
        c["d_edge"] = rng.choice([0, rng.randint(4, 64), rng.randint(65, 192), rng.randint(65, 192)])
        c["d_static"] = rng.choice([0, 0, rng.randint(8, 128)])
        c["k"] = rng.choice([10, 10, 10, rng.randint(3, 20)])
        c["t_max"] = 10.0 ** rng.uniform(4, 7.4)
        kind = rng.choice(["plain", "plain", "replicas", "negatives", "classes", "steps", "adam"])
        if c["path"] == "eval":
            c["negatives"] = _log_int(rng, 2, 49)
        elif c["path"] == "operators":
            c["d_static"] = 0
        elif kind == "replicas":
            c["replicas"] = rng.randint(2, 8)
        elif kind == "negatives":
            c["negatives"] = rng.randint(2, 8)
        elif kind == "classes":
            c["classes"] = rng.randint(2, 64)
        elif kind == "steps":
            c["steps"] = rng.randint(2, 8)
        elif kind == "adam":
            c["adam"] = True
        if c["path"] == "operators":
            c["batch"] = min(c["batch"], 1000) // 4 * 4   # every slot is a row of its own there; the operators' arguments
                                                          # are slices by role, which have to stay 16-byte aligned
        roots = _roots(c) * c["steps"]
        w, most = work(c), work(largest)
        if (roots <= 48_000 and roots * c["k"] <= 480_000 and c["events"] >= 8 * c["replicas"] * c["batch"]
                and w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]):
            return c


def _roots(c):
    return c["batch"] * c["replicas"] * (2 if c["classes"] else 2 + c["negatives"])


def _shapes(c):
    """Parameter tensors in the library's order: name -> (shape, fan_in)."""
    m, t, e, s = c["d_mem"], c["d_time"], c["d_edge"], c["d_static"]
    x, i = m + s, 2 * m + t + e
    kv, C = x + e + t, c["classes"]
    return {"time_w": ((t,), 0), "time_b": ((t,), 0),
            "gru_wih": ((3 * m, i), i), "gru_whh": ((3 * m, m), m), "gru_bih": ((3 * m,), i), "gru_bhh": ((3 * m,), m),
            "wq": ((m, x + t), x + t), "bq": ((m,), x + t), "wk": ((m, kv), kv), "bk": ((m,), kv),
            "wv": ((m, kv), kv), "bv": ((m,), kv), "wo": ((m, m + x), m + x), "bo": ((m,), m + x),
            "dec_ws": ((m, m), m), "dec_wd": ((m, m), m), "dec_b1": ((m,), m),
            "dec_w2": ((C, m) if C else (m,), m), "dec_b2": ((C or 1,), m)}


def _bucket(c):
    """A parameter set whose tensors are views of one flat buffer (one bucket to save, clear or exchange)."""
    shapes = _shapes(c)
    size = {n: (math.prod(s) + 3) // 4 * 4 for n, (s, _) in shapes.items()}      # 16-byte aligned views
    flat = torch.zeros(sum(size.values()), device="cuda")
    views, off = {}, 0
    for n, (s, _) in shapes.items():
        views[n] = flat[off:off + math.prod(s)].view(s)
        off += size[n]
    return flat, tgnn.Params(views)


def _init_params(c, gen):
    flat, params = _bucket(c)
    for n, (shape, fan_in) in _shapes(c).items():
        if n == "time_w":
            i = torch.arange(c["d_time"], dtype=torch.float64, device="cuda")
            params.t[n].copy_(10.0 ** (-9.0 * i / max(c["d_time"] - 1, 1)))
        elif n != "time_b":
            b = 1.0 / math.sqrt(fan_in)
            params.t[n].uniform_(-b, b, generator=gen)
    return flat, params


def _zipf(n, a, size, gen):
    """Ids in [0, n) with probability proportional to rank^-a under a random map from rank to id."""
    cdf = torch.arange(1, n + 1, dtype=torch.float64, device="cuda").pow(-a).cumsum(0)
    u = torch.rand(size, dtype=torch.float64, device="cuda", generator=gen) * cdf[-1]
    rank = torch.searchsorted(cdf, u).clamp_(max=n - 1)
    return torch.randperm(n, device="cuda", generator=gen)[rank]


def _rows(values, M, n):
    """[M * n, ...] -> M contiguous, 16-byte aligned pieces of n rows."""
    v = values[:M * n].reshape(M, -1)
    pitch = (v.shape[1] + 3) // 4 * 4
    out = torch.zeros(M, pitch, dtype=v.dtype, device=v.device)
    out[:, :v.shape[1]] = v
    return [out[i, :v.shape[1]] for i in range(M)]


_STREAM = None


def _stream():
    """The stream of the training program: one, not the default stream."""
    global _STREAM
    if _STREAM is None:
        _STREAM = torch.cuda.Stream()
    return _STREAM


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    N, E, n, J = c["nodes"], c["events"], c["batch"], c["negatives"]
    dst_lo = c["n_src"]
    src = _zipf(c["n_src"] or N, c["skew_src"], E, gen)
    dst = _zipf(N - dst_lo, c["skew_dst"], E, gen) + dst_lo
    if not c["n_src"]:
        dst = torch.where(dst == src, (dst + 1) % N, dst)
    src, dst = src.int(), dst.int()
    ts = (torch.rand(E, dtype=torch.float64, device="cuda", generator=gen) * c["t_max"]).sort().values
    efeat = torch.randn(E, c["d_edge"], device="cuda", generator=gen) if c["d_edge"] else None
    static = 0.1 * torch.randn(N, c["d_static"], device="cuda", generator=gen) if c["d_static"] else None
    graph = tgnn.Graph(src.cpu().numpy(), dst.cpu().numpy(), ts.cpu().numpy(), N, efeat)
    pflat, params = _init_params(c, gen)
    gflat, grads = _bucket(c)
    evaluating = c["path"] == "eval"
    ctx = tgnn.Context(N, c["d_mem"], c["d_time"], c["d_edge"], c["d_static"], c["heads"], c["k"], n,
                       n_replicas=c["replicas"], flags=0 if evaluating else tgnn.FLAG_OVERWRITE_GRADS, max_neg_sets=J,
                       n_classes=c["classes"])
    if c["adam"]:
        ctx.tgnn_set_optimizer(1, tgnn.Params.zeros_like(params), tgnn.Params.zeros_like(params))

    # the full mini-batches of the second half of the stream, resident on the device
    first = E // n // 2
    M, lo = E // n - first, first * n
    neg = torch.randint(dst_lo, N, (M * n * J,), dtype=torch.int32, device="cuda", generator=gen)
    eid = torch.arange(E, dtype=torch.int32, device="cuda")
    cols = [_rows(src[lo:], M, n), _rows(dst[lo:], M, n), _rows(neg, M, n * J), _rows(eid[lo:], M, n), _rows(ts[lo:], M, n)]
    batches = [[tgnn.Batch(*(col[i] for col in cols), replica=r) for i in range(M)] for r in range(c["replicas"])]
    labels = None
    if c["classes"]:      # a few true classes per event, the popular ones more often
        like = 6.0 / (1.0 + torch.arange(c["classes"], device="cuda")) / math.log(c["classes"] + 1.0)
        labels = torch.rand(M * n, c["classes"], device="cuda", generator=gen) < like
        labels = [y.view(n, c["classes"]) for y in _rows(labels.float(), M, n)]

    # node memory and mails as they stand before a mini-batch; replica r begins at mini-batch r shift
    shift = -(-M // c["replicas"])
    owner = torch.repeat_interleave(torch.arange(N, device="cuda"), graph.indptr.diff())

    def memory_before(event):
        past = torch.bincount(owner[graph.eid < event], minlength=N)     # a node's events so far, oldest first in its list
        has, last = past > 0, (graph.indptr[:-1] + past - 1).clamp_(min=0)
        mem = (torch.rand(N, c["d_mem"], device="cuda", generator=gen) - 0.5) * has[:, None]
        mail = (torch.rand(N, 2 * c["d_mem"], device="cuda", generator=gen) - 0.5) * has[:, None]
        return dict(mem=mem, mem_ts=torch.where(past > 1, graph.ts[(last - 1).clamp_(min=0)], 0.0), mail=mail,
                    mail_ts=torch.where(has, graph.ts[last], 0.0), mail_eid=torch.where(has, graph.eid[last], -1).int())

    kept = memory_before(lo)
    st = tgnn.State(N, c["d_mem"], c["replicas"], static)
    for r in range(c["replicas"]):
        for name, v in (kept if r == 0 else memory_before(lo + r * shift % M * n)).items():
            getattr(st, name)[r * N:(r + 1) * N] = v
    s = dict(case=c, ctx=ctx, graph=graph, st=st, params=params, pflat=pflat, grads=grads, gflat=gflat, batches=batches,
             labels=labels, kept=kept, step=0, shift=shift, M=M, loss=torch.zeros(8, device="cuda"),
             rank=torch.zeros(n, device="cuda"), rr=torch.zeros(1, device="cuda"),
             logits=torch.zeros(n * (1 + J), device="cuda") if evaluating else None,
             winner=torch.zeros(2 * n, dtype=torch.int32, device="cuda") if evaluating else None)
    if c["path"] == "operators":
        s["dz"] = torch.randn(3 * n, c["d_mem"], device="cuda", generator=gen) / (3 * n)
    return s


def _at_start(s, i):
    """The replicas that are at the first mini-batch in step i."""
    return [r for r in range(s["case"]["replicas"]) if (i + r * s["shift"]) % s["M"] == 0]


def _next(s):
    """The next step's mini-batches, one per replica; a replica that is through the stream goes back to its beginning."""
    i = s["step"]
    s["step"] = i + 1
    for r in _at_start(s, i) if i > 0 else ():
        N = s["case"]["nodes"]
        for name, v in s["kept"].items():
            getattr(s["st"], name)[r * N:(r + 1) * N].copy_(v)
    which = [(i + r * s["shift"]) % s["M"] for r in range(s["case"]["replicas"])]
    return [s["batches"][r][m] for r, m in enumerate(which)], which


def _memory(s):
    st = s["st"]
    return dict(mem=st.mem, mem_ts=st.mem_ts, mail=st.mail, mail_ts=st.mail_ts, mail_eid=st.mail_eid)


def _run_operators(s):
    c, ctx, g, st, p = s["case"], s["ctx"], s["graph"], s["st"], s["params"]
    (b,), _ = _next(s)
    n, k, R = b.n, c["k"], 3 * b.n
    root, t = torch.cat([b.src, b.dst, b.neg]), b.t.repeat(3)
    nbr, eid, _, cnt = ctx.tgnn_sample_recent(g, root, t)
    s_new, tau = ctx.tgnn_gru_update(p, ctx.tgnn_gather_memory(g, st, 0, torch.cat([root, nbr.view(-1)])))
    e_nbr = g.efeat[eid.view(-1).clamp(min=0)] if c["d_edge"] else None
    dt = t[:, None] - tau[R:].view(R, k)
    z = ctx.tgnn_temporal_attn_fwd(p, s_new[:R], s_new[R:], e_nbr, dt, cnt)
    ctx.tgnn_zero_params(s["grads"])
    d_root, d_nbr = ctx.tgnn_temporal_attn_bwd(p, s["dz"], s["grads"])
    winner = ctx.tgnn_memory_writeback(st, 0, b.src, b.dst, b.eid, b.t, s_new[:n], s_new[n:2 * n], tau[:n], tau[n:2 * n])
    return dict(_memory(s), z=z, grads=s["gflat"], d_root=d_root, d_nbr=d_nbr, winner=winner)


def run(s):
    c, ctx = s["case"], s["ctx"]
    with torch.cuda.stream(_stream()):
        if c["path"] == "operators":
            return _run_operators(s)
        if c["path"] == "eval":
            b, _ = _next(s)
            ctx.tgnn_eval_step(s["graph"], s["st"], s["params"], b, c["negatives"], s["rank"], s["rr"],
                               out_logits=s["logits"], out_winner=s["winner"])
            # (ranks are halves of whole numbers: their bits are compared as whole values)
            return dict(_memory(s), logits=s["logits"], rank=s["rank"].view(torch.int32), winner=s["winner"])
        args = (s["graph"], s["st"], s["params"], s["grads"])
        if c["steps"] > 1:
            todo = []
            for _ in range(c["steps"]):
                if todo and _at_start(s, s["step"]):     # the stream ends here: what is left of it goes first
                    ctx.tgnn_train_steps(*args, todo, lr=c["lr"], out_loss=s["loss"])
                    todo = []
                todo.append(_next(s)[0])
            ctx.tgnn_train_steps(*args, todo, lr=c["lr"], out_loss=s["loss"])
        elif c["classes"]:
            b, which = _next(s)
            ctx.tgnn_train_step_edge_class(*args, b, [s["labels"][m] for m in which], lr=c["lr"], out_loss=s["loss"])
        elif c["negatives"] > 1:
            ctx.tgnn_train_step_epoch_parallel(*args, _next(s)[0], c["negatives"], lr=c["lr"], out_loss=s["loss"])
        else:
            ctx.tgnn_train_step(*args, _next(s)[0], lr=c["lr"], out_loss=s["loss"])
        return dict(_memory(s), loss=s["loss"], grads=s["gflat"], params=s["pflat"])


def work(case):
    """Bytes and operations of one pass that no implementation of the step avoids: memory update and node parts of the
    projections once per distinct node, everything else once per root or neighbour slot; inputs read once, outputs
    written once.  The number of distinct nodes among a step's slots is taken as an eighth of the slots, at most all."""
    c = dict(DEFAULTS, **case)
    m, t, e, x = c["d_mem"], c["d_time"], c["d_edge"], c["d_mem"] + c["d_static"]
    B, R, k, H = c["batch"] * c["replicas"], _roots(c), c["k"], c["heads"]
    ev = e + t
    ops = c["path"] == "operators"
    U = R * (1 + k) if ops else min(c["nodes"] * c["replicas"], max(R * (1 + k) // 8, 64))
    pairs = B * (c["classes"] or 1 + c["negatives"])
    fwd = 2 * (U * (2 * m + t + e + m) * 3 * m + U * x * 4 * m + U * m * ev          # memory update, node parts, u = q W
               + R * k * (2 * H * ev + 2 * m) + R * ev * m                            # scores and weighted sums, output
               + R * m * m)                                                           # merge layer
    if not ops:
        fwd += 2 * (R * m * m + pairs * m)                                            # decoder
    if c["path"] == "eval":
        flops = fwd
    elif ops:
        flops = fwd + 2 * (2 * R * m * m + 4 * R * ev * m + R * k * (3 * H * ev + 4 * m) + 2 * U * x * 4 * m)
    else:
        flops = 3 * fwd
    n_par = sum(math.prod(s) for s, _ in _shapes(c).values())
    events = min(R * k, U * k)                                       # distinct events among the neighbour slots, about
    nbytes = (U * (12 * m + 4 * e + 28) + U * 4 * c["d_static"]   # memory, mails and their edge features, static
              + events * 4 * e + R * (16 * k + 128)                           # edge features of the slots, neighbour lists
              + min(2 * B, c["nodes"] * c["replicas"]) * (12 * m + 20)        # write-back
              + 4 * n_par * (1 if c["path"] == "eval" else 2 if ops else 7 if c["adam"] else 3) + 4 * pairs)
    if ops:   # the operators' own results: staged rows, updated memory, attention inputs, outputs and gradients
        nbytes += 4 * (U * (3 * m + e) + U * 2 * m + R * k * e + R * 2 * m + U * m)
    return {"bytes": float(nbytes * c["steps"]), "flops": float(flops * c["steps"])}


def tolerance(case):
    """Measured by moving every weight by up to half a rounding (a relative 6e-8) and comparing: logits and memory move by
    at most 5e-7 (2-norm) and 2e-6 (largest), gradients by 5e-7 and 3e-5 as long as no ReLU changes sides.  A training
    step has up to a few million ReLU inputs, now and then one within rounding of zero; when it is gated the other way
    the gradients of one event change: 1.4e-3 and 5e-2 seen on eight replicas.  Four times each.  Two scores within
    rounding of each other may swap ranks."""
    if case["path"] == "eval":
        return {"rel": 2e-6, "max": 1e-5, "differ": 1e-3}
    return {"rel": 5e-3, "max": 0.2}
