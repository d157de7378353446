"""GPU parity of the edge-classification step (tgnn_train_step_edge_class) and of the evaluation pass (tgnn_eval_step,
reciprocal rank among sampled negative destinations) against the oracle."""
import numpy as np
import pytest
import torch

from gpu_common import GpuSide, OracleSide, batch_np, compare_state, compare_step, make_problem, rel_err, TOL
from oracle import tgnn_oracle as O
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    dict(n_nodes=60, E=900, d_mem=16, d_time=8, d_edge=5, d_static=0, n_heads=2, k=5, batch=50, n_classes=7, n_true=2),
    # the task's own widths (Sec. 4 "Datasets"): 56 classes, 6 of them true, 130 edge features
    dict(n_nodes=300, E=1500, d_mem=100, d_time=100, d_edge=130, d_static=0, n_heads=2, k=10, batch=120, n_classes=56,
         n_true=6),
    dict(n_nodes=80, E=600, d_mem=132, d_time=12, d_edge=0, d_static=4, n_heads=2, k=4, batch=40, n_classes=1, n_true=1),
])
def test_edge_classification_steps_against_the_oracle(shape):
    P = synth.custom_problem(**shape, seed=31)
    d = P["d"]
    G = GpuSide(P); Or = OracleSide(P)
    n_steps = P["E"] // d.batch
    for s in range(n_steps):
        b = batch_np(P, s * d.batch, (s + 1) * d.batch)
        assert b["labels"].shape == (d.batch, d.n_classes)
        g = G.step([b], lr=0.05)
        o = Or.step([b], lr=0.05, gpu=g)
        assert g["logits"].shape == (d.batch, d.n_classes) and len(g["cnt"]) == 2 * d.batch
        compare_step(g, o, label=f"edge classification C={d.n_classes} step {s}")
    compare_state(G.state_np(), Or.states[0], label="edge classification state")
    moved = False
    for n, v in G.params.numpy().items():
        assert v.shape == Or.p[n].shape and rel_err(v, Or.p[n]) <= 1e-4, n
        moved |= n == "dec_w2" and np.abs(v - P["params"][n]).max() > 0
    assert moved


def test_edge_classification_two_replicas_and_entry_point_checks():
    import torch
    from paper_2307_07649_amd import tgnn
    P = synth.custom_problem(n_nodes=70, E=800, d_mem=24, d_time=8, d_edge=6, d_static=0, n_heads=2, k=5, batch=40,
                             n_classes=9, n_true=3, seed=5)
    d = P["d"]
    G = GpuSide(P, n_replicas=2); Or = OracleSide(P, n_replicas=2)
    for s in range(4):
        bs = [batch_np(P, (2 * s + r) * d.batch, (2 * s + r + 1) * d.batch - 7 * r) for r in range(2)]   # ragged second batch
        g = G.step(bs, lr=0.02)
        o = Or.step(bs, lr=0.02, gpu=g)
        compare_step(g, o, label=f"edge classification 2 replicas step {s}")
    # a context with a classification head refuses the link-prediction step, and the other way round
    b = batch_np(P, 0, d.batch)
    bl = [tgnn.Batch(b["src"], b["dst"], b["neg"], b["eid"], b["t"])]
    with pytest.raises(tgnn.TgnnError):
        G.ctx.tgnn_train_step(G.graph, G.state, G.params, G.grads, bl, lr=0.0, out_loss=G.loss)
    P0 = synth.custom_problem(n_nodes=70, E=800, d_mem=24, d_time=8, d_edge=6, d_static=0, n_heads=2, k=5, batch=40, seed=5)
    G0 = GpuSide(P0)
    y = torch.zeros(d.batch, 9, device="cuda")
    with pytest.raises(tgnn.TgnnError):
        G0.ctx.tgnn_train_step_edge_class(G0.graph, G0.state, G0.params, G0.grads, bl, [y], lr=0.0, out_loss=G0.loss)


@pytest.mark.parametrize("J,shape", [
    (49, dict(n_nodes=200, E=1200, d_mem=32, d_time=16, d_edge=8, d_static=0, n_heads=2, k=10, batch=60)),
    (49, dict(n_nodes=300, E=600, d_mem=100, d_time=100, d_edge=172, d_static=0, n_heads=2, k=10, batch=50)),
    (1, dict(n_nodes=90, E=600, d_mem=20, d_time=6, d_edge=3, d_static=5, n_heads=1, k=4, batch=40)),
])
def test_evaluation_pass_against_the_oracle(J, shape):
    """Scores of the true and the J sampled destinations against the oracle's forward pass (1e-4 of the largest score);
    the ranks are an integer decision taken on floating-point scores, so both sides take it on the same scores: the
    oracle's rank function applied to the GPU's own logits must reproduce the GPU's ranks exactly, and the sum of the
    reciprocal ranks to fp32 rounding; memory after the pass as after training steps; parameters untouched."""
    P = synth.custom_problem(**shape, seed=17)
    d = P["d"]
    rng = np.random.default_rng(3)
    G = GpuSide(P, max_neg_sets=J); Or = OracleSide(P)
    before = G.params.numpy()
    n_steps = min(6, P["E"] // d.batch)
    for s in range(n_steps):
        b = batch_np(P, s * d.batch, (s + 1) * d.batch)
        b["neg"] = rng.integers(0, d.n_nodes, (J, d.batch)).astype(np.int32)
        if s == 2:
            b["neg"][0] = b["dst"]                      # ties with the true destination: half a rank each
        g = G.eval_step([b], J)
        o = Or.step([b], lr=0.0)
        ref = o["outs"][0]["logits"]
        assert rel_err(g["logits"], ref) <= TOL, s
        assert np.array_equal(g["winner"], o["winners"][0]) and np.array_equal(g["cnt"], o["outs"][0]["cnt"])
        B = d.batch
        rank, mrr = O.reciprocal_rank(g["logits"][:B].astype(np.float64), g["logits"][B:].reshape(J, B).astype(np.float64))
        assert np.array_equal(g["rank"], rank.astype(np.float32)), s
        assert abs(g["rr_sum"] / B - mrr) <= 1e-6
        if s == 2:    # a negative destination that IS the true destination scores exactly the same: half a rank each
            lg = g["logits"]
            assert np.array_equal(lg[B:2 * B], lg[:B]) and (np.abs(g["rank"] * 2 % 2 - 1) < 1e-6).sum() > B // 2
        # and against the oracle's own scores, wherever no two scores are within rounding of each other
        o_rank, _ = O.reciprocal_rank(ref[:B], ref[B:].reshape(J, B))
        gap = np.abs(ref[B:].reshape(J, B) - ref[:B][None, :])
        safe = (gap > 1e-4 * np.abs(ref).max()).all(0) | (s == 2)
        assert np.array_equal(g["rank"][safe & (s != 2)], o_rank[safe & (s != 2)].astype(np.float32))
    compare_state(G.state_np(), Or.states[0], label="state after evaluation")
    assert all(np.array_equal(before[n], v) for n, v in G.params.numpy().items())
    assert not any(np.any(v) for v in G.grads.numpy().values())


def test_empty_batches_and_argument_errors():
    import torch
    from paper_2307_07649_amd import tgnn
    P = synth.custom_problem(n_nodes=50, E=300, d_mem=16, d_time=8, d_edge=4, d_static=0, n_heads=2, k=4, batch=30,
                             n_classes=5, n_true=2, seed=2)
    d = P["d"]
    G = GpuSide(P)
    e = batch_np(P, 0, 0)
    empty = tgnn.Batch(e["src"], e["dst"], e["neg"], e["eid"], e["t"])
    y0 = torch.zeros(0, 5, device="cuda")
    G.loss.fill_(7.0)
    before = G.state_np()
    G.ctx.tgnn_train_step_edge_class(G.graph, G.state, G.params, G.grads, [empty], [y0], lr=0.1, out_loss=G.loss)
    torch.cuda.synchronize()
    assert float(G.loss[0]) == 0.0 and all(np.array_equal(before[k], v) for k, v in G.state_np().items())
    b = batch_np(P, 0, d.batch)
    full = tgnn.Batch(b["src"], b["dst"], b["neg"], b["eid"], b["t"])
    with pytest.raises(tgnn.TgnnError):          # a batch with events needs its targets
        G.ctx.tgnn_train_step_edge_class(G.graph, G.state, G.params, G.grads, [full], [None], lr=0.0, out_loss=G.loss)
    # evaluation: more negative sets than the context was created for; an empty batch ranks nothing
    P1 = synth.custom_problem(n_nodes=50, E=300, d_mem=16, d_time=8, d_edge=4, d_static=0, n_heads=2, k=4, batch=30, seed=2)
    G1 = GpuSide(P1, max_neg_sets=3)
    rank = torch.zeros(30, device="cuda"); rr = torch.full((1,), 2.5, device="cuda")
    with pytest.raises(tgnn.TgnnError):
        G1.ctx.tgnn_eval_step(G1.graph, G1.state, G1.params, [full], 4, rank, rr)
    G1.ctx.tgnn_eval_step(G1.graph, G1.state, G1.params, [empty], 3, rank, rr)
    torch.cuda.synchronize()
    assert float(rr[0]) == 2.5 and not rank.any()
    with pytest.raises(tgnn.TgnnError):          # the evaluation pass is link prediction: not on a classification context
        G.ctx.tgnn_eval_step(G.graph, G.state, G.params, [full], 1, rank, rr)


def test_training_and_evaluation_steps_alternate_on_one_context():
    """Train, evaluate, train ... on one context and one stream (each kind of step replays its own captured graph): the
    state an evaluation step leaves is the one the next training step starts from, on both sides."""
    P = synth.custom_problem(n_nodes=120, E=1200, d_mem=32, d_time=16, d_edge=8, d_static=0, n_heads=2, k=6, batch=60, seed=23)
    d = P["d"]
    J = 5
    rng = np.random.default_rng(1)
    G = GpuSide(P, max_neg_sets=J); Or = OracleSide(P)
    for s in range(12):
        b = batch_np(P, s * d.batch, (s + 1) * d.batch)
        if s % 3 == 1:
            b["neg"] = rng.integers(0, d.n_nodes, (J, d.batch)).astype(np.int32)
            g = G.eval_step([b], J)
            o = Or.step([b], lr=0.0)
            assert rel_err(g["logits"], o["outs"][0]["logits"]) <= TOL, s
            assert np.array_equal(g["winner"], o["winners"][0])
        else:
            g = G.step([b], lr=0.05)
            o = Or.step([b], lr=0.05, gpu=g)
            compare_step(g, o, label=f"train/eval alternating step {s}")
    compare_state(G.state_np(), Or.states[0], label="train/eval alternating")
    for n, v in G.params.numpy().items():
        assert rel_err(v, Or.p[n]) <= 1e-4, n


def test_edge_classification_with_adam():
    """Adam on a context with a classification head (the output layer's tensors are [C, d_o] and [C] there): on every
    step the oracle's Adam, given the GPU's own parameters, moments and gradients, reproduces the GPU's update."""
    from paper_2307_07649_amd import tgnn
    P = synth.custom_problem(n_nodes=60, E=600, d_mem=24, d_time=8, d_edge=5, d_static=0, n_heads=2, k=5, batch=40,
                             n_classes=11, n_true=3, seed=8)
    d = P["d"]
    G = GpuSide(P); Or = OracleSide(P)
    m = tgnn.Params.zeros_like(G.params); v = tgnn.Params.zeros_like(G.params)
    b1, b2, eps = (float(np.float32(x)) for x in (0.9, 0.999, 1e-8))
    G.ctx.tgnn_set_optimizer(1, m, v, b1, b2, eps)
    Or.use_adam(b1, b2, eps)
    for s in range(6):
        b = batch_np(P, s * d.batch, (s + 1) * d.batch)
        before = (G.params.numpy(), m.numpy(), v.numpy())
        g = G.step([b], lr=1e-3)
        o = Or.step([b], lr=1e-3, gpu=g)
        compare_step(g, o, label=f"edge classification + Adam step {s}")
        p1 = {n: x.astype(np.float64) for n, x in before[0].items()}
        st = dict(m={n: x.astype(np.float64) for n, x in before[1].items()},
                  v={n: x.astype(np.float64) for n, x in before[2].items()}, t=s)
        O.adam(p1, {n: x.astype(np.float64) for n, x in g["grads"].items()}, st, 1e-3, b1, b2, eps)
        after = (G.params.numpy(), m.numpy(), v.numpy())
        for n in p1:
            assert after[0][n].shape == p1[n].shape
            assert rel_err(after[0][n], p1[n]) <= 1e-6 and rel_err(after[1][n], st["m"][n]) <= 1e-6, (s, n)
            assert rel_err(after[2][n], st["v"][n]) <= 1e-6, (s, n)
    moved = np.abs(G.params.numpy()["dec_w2"] - P["params"]["dec_w2"]) > 0      # (hidden units that never fire stay put)
    assert moved.shape == (11, 24) and moved.all(axis=0).sum() > 12 and moved.any(axis=1).all()


def test_classification_evaluation_pass_against_the_oracle():
    """tgnn_eval_step_edge_class between training steps on one context: logits against the oracle's forward pass, the
    tp / fp / fn counts exactly those of the oracle's counting function on the GPU's own logits (and on the oracle's,
    where no logit is within rounding of zero), memory advanced, parameters untouched by the evaluation steps."""
    P = synth.custom_problem(n_nodes=90, E=900, d_mem=32, d_time=16, d_edge=6, d_static=0, n_heads=2, k=5, batch=50,
                             n_classes=13, n_true=4, seed=41)
    d = P["d"]
    G = GpuSide(P); Or = OracleSide(P)
    total = np.zeros(3, np.int64)
    for s in range(12):
        b = batch_np(P, s * d.batch, (s + 1) * d.batch)
        if s % 2 == 1:
            before = G.params.numpy()
            g = G.eval_class_step([b])
            o = Or.step([b], lr=0.0)
            ref = o["outs"][0]["logits"]
            assert rel_err(g["logits"], ref) <= TOL, s
            assert np.array_equal(g["winner"], o["winners"][0])
            assert g["counts"] == O.f1_micro_counts(g["logits"], b["labels"]), s
            if np.abs(ref).min() > 1e-4 * np.abs(ref).max():
                assert g["counts"] == O.f1_micro_counts(ref, b["labels"]), s
            assert sum(g["counts"][i] for i in (0, 2)) == int(b["labels"].sum())         # tp + fn = the true labels
            assert all(np.array_equal(before[n], v) for n, v in G.params.numpy().items())
            total += g["counts"]
        else:
            g = G.step([b], lr=0.05)
            o = Or.step([b], lr=0.05, gpu=g)
            compare_step(g, o, label=f"classification train/eval step {s}")
    compare_state(G.state_np(), Or.states[0], label="classification train/eval")
    assert total[0] + total[1] > 0          # the head does predict something


def test_evaluation_pass_two_replicas_ragged_batches():
    """Two memory replicas in one evaluation call, batches of different lengths: scores, ranks (pair layout per batch) and
    the memory of both replicas."""
    P = synth.custom_problem(n_nodes=100, E=1000, d_mem=24, d_time=8, d_edge=4, d_static=3, n_heads=3, k=6, batch=50, seed=29)
    d = P["d"]
    J = 7
    rng = np.random.default_rng(5)
    G = GpuSide(P, n_replicas=2, max_neg_sets=J); Or = OracleSide(P, n_replicas=2)
    for s in range(5):
        bs = []
        for r in range(2):
            lo = (2 * s + r) * d.batch; hi = lo + d.batch - 13 * r
            b = batch_np(P, lo, hi)
            b["neg"] = rng.integers(0, d.n_nodes, (J, hi - lo)).astype(np.int32)
            bs.append(b)
        g = G.eval_step(bs, J)
        o = Or.step(bs, lr=0.0)
        ref = np.concatenate([x["logits"] for x in o["outs"]])
        assert rel_err(g["logits"], ref) <= TOL, s
        assert np.array_equal(g["winner"], np.concatenate(o["winners"]))
        off_l = off_e = 0
        for b in bs:
            n = len(b["src"])
            lg = g["logits"][off_l:off_l + (1 + J) * n].astype(np.float64)
            rank, _ = O.reciprocal_rank(lg[:n], lg[n:].reshape(J, n))
            assert np.array_equal(g["rank"][off_e:off_e + n], rank.astype(np.float32)), s
            off_l += (1 + J) * n; off_e += n
        assert abs(g["rr_sum"] - float((1.0 / g["rank"].astype(np.float64)).sum())) <= 1e-4
    for r in range(2):
        compare_state(G.state_np(r), Or.states[r], label=f"evaluation replica {r}")


# the classification head's tiles: events around a tile of 16, classes and widths around 16 and 64, the widest of both
@pytest.mark.parametrize("d_mem,heads,classes,batch", [(8, 1, 1, 1), (16, 2, 16, 15), (20, 1, 17, 16), (64, 2, 63, 17),
                                                       (66, 2, 65, 33), (256, 2, 256, 18)])
def test_classification_head_tile_edges(d_mem, heads, classes, batch):
    P = synth.custom_problem(n_nodes=40, E=6 * batch, d_mem=d_mem, d_time=8, d_edge=4, d_static=0, n_heads=heads, k=3, batch=batch,
                       n_classes=classes, n_true=1, seed=classes)
    G = GpuSide(P); Or = OracleSide(P)
    for s in range(4):
        b = batch_np(P, s * batch, (s + 1) * batch)
        g = G.step([b], lr=0.01)
        o = Or.step([b], lr=0.01, gpu=g)
        compare_step(g, o, label=f"{classes} classes, {d_mem} wide, {batch} events, step {s}")


# one wavefront per event (J < 8) and four, pairs around a round of each, the most negatives, widths on both sides of 64
@pytest.mark.parametrize("J,d_mem,batch", [(1, 8, 1), (7, 64, 5), (8, 65, 6), (27, 100, 3), (28, 128, 3), (63, 130, 2), (64, 256, 2)])
def test_rank_kernel_pair_counts(J, d_mem, batch):
    P = synth.custom_problem(n_nodes=40, E=6 * batch, d_mem=d_mem, d_time=8, d_edge=4, d_static=0, n_heads=1, k=3, batch=batch, seed=J)
    G = GpuSide(P, max_neg_sets=J); Or = OracleSide(P)
    rng = np.random.default_rng(J)
    for s in range(4):
        b = batch_np(P, s * batch, (s + 1) * batch)
        b["neg"] = rng.integers(0, 40, (J, batch)).astype(np.int32)
        g = G.eval_step([b], J)
        ref = Or.step([b], lr=0.0)["outs"][0]["logits"]
        assert rel_err(g["logits"], ref) <= TOL
        rank, mrr = O.reciprocal_rank(g["logits"][:batch].astype(np.float64), g["logits"][batch:].reshape(J, batch).astype(np.float64))
        assert np.array_equal(g["rank"], rank.astype(np.float32)) and abs(g["rr_sum"] / batch - mrr) <= 1e-6


# the sum of the reciprocal ranks is carried on by the caller: below, at and above one block of 256 events, one wavefront
# per event and four
@pytest.mark.parametrize("J,batch", [(49, 255), (49, 256), (3, 700), (49, 600)])
def test_reciprocal_rank_sum_added_to_a_large_one(J, batch):
    from paper_2307_07649_amd import tgnn
    P = synth.custom_problem(n_nodes=300, E=3 * batch, d_mem=16, d_time=8, d_edge=4, d_static=0, n_heads=1, k=3, batch=batch, seed=J)
    G = GpuSide(P, max_neg_sets=J)
    rng = np.random.default_rng(J)
    start = float(2 ** 17)
    rank = torch.empty(batch, device="cuda"); rr = torch.full((1,), start, device="cuda")
    want = start
    for s in range(3):
        b = batch_np(P, s * batch, (s + 1) * batch)
        neg = rng.integers(0, 300, J * batch).astype(np.int32)
        G.ctx.tgnn_eval_step(G.graph, G.state, G.params, [tgnn.Batch(b["src"], b["dst"], neg, b["eid"], b["t"])], J, rank, rr)
        want += float((1.0 / rank.cpu().numpy().astype(np.float64)).sum())
    # 256 events are one addition to the large sum, of half an ulp (2^-7) each; what they add up to is exact to 1e-5
    assert abs(float(rr.item()) - want) <= 3 * ((batch + 255) // 256) * (2.0 ** -7 + 1e-5)
