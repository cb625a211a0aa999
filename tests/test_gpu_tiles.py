"""The branches of the launch rules that the parity cases' own shapes do not reach, at their edges."""
import hashlib

import numpy as np
import pytest
import torch

from paper_2408_10746_amd import binding as pb
from paper_2408_10746_amd import inputs
from paper_2408_10746_amd.inputs import Workload

pytestmark = pytest.mark.gpu

from tests.test_gpu_parity import TOL, check_against_oracle, make_session, oracle_batch  # noqa: E402


def tiles_of(w, lens):
    ctx = pb.pac_create(w.L, w.d, w.n_max, w.r, w.C, w.B, w.N, pb.PAC_BF16 if w.cache_dtype == "bf16" else pb.PAC_F32)
    try:
        return pb.pac_step_tiles(ctx, lens[:w.B], w.B)
    finally:
        pb.pac_destroy(ctx)


# 256 x 256 tiles with a last one part empty along the token rows, along d (0.75 and 4.75 tiles) and along r (0.75 and 1.75
# tiles), a last 64-token step of few valid tokens
LARGE_TILES = [
    # the projection alone
    (Workload("p1", L=28, d=192, n_max=140, B=3, r=448, C=4, N=3, cache_dtype="bf16", len_lo=110), dict(proj=256, grads=128)),
    # all three
    (Workload("p2", L=48, d=1216, n_max=300, B=3, r=192, C=2, N=3, cache_dtype="bf16", len_lo=250), dict(proj=256, tokens=256, grads=256, rows=1, sg=1)),
    (Workload("p3", L=24, d=1216, n_max=300, B=3, r=448, C=5, N=3, cache_dtype="bf16", len_lo=250), dict(proj=256, tokens=256, grads=256, rows=1, sg=1)),
    # the contractions over the tokens alone, both results split over them
    (Workload("p4", L=12, d=1216, n_max=500, B=8, r=160, C=3, N=8, cache_dtype="bf16", len_lo=400), dict(tokens=256, grads=128, se=2, sg=2)),
    (Workload("p5", L=4, d=1952, n_max=1000, B=6, r=256, C=3, N=6, cache_dtype="bf16", len_lo=960), dict(proj=128, tokens=256, grads=128)),
    # vector gradients as whole rows in the launch of the token splits' sums
    (Workload("p6", L=3, d=2560, n_max=100, B=2, r=448, C=3, N=2, cache_dtype="bf16", len_lo=80), dict(proj=128, tokens=128, grads=128, rows=1, se=2, sg=2)),
]


@pytest.mark.parametrize("w,tiles", LARGE_TILES, ids=[w.name for w, _ in LARGE_TILES])
def test_wide_contractions_on_large_tiles(w, tiles):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    got = tiles_of(w, lens)
    assert {k: got[k] for k in tiles} == tiles, got
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens)
    sess.cache_fill(ids, acts, lens)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["bf16"], what=w.name)


# The layer-by-layer chains over several groups of layers: 256 x 256 tiles (c1), K steps of 32 and a last group of two layers
# (c2), many tokens on few weights, where the groups' sums do not fit beside each other (c3), five groups of which the last
# holds one layer, on a few rows (c4), a group that is not a power of two wide (c5), a first part of two groups and a last
# group of one layer (c6).
@pytest.mark.parametrize("w,plan", [
    (Workload("c1", L=8, d=32, n_max=180, B=30, r=512, C=2, N=30, cache_dtype="bf16", len_lo=160), (4, 2, 1, 1, 256, 256)),
    (Workload("c2", L=14, d=96, n_max=90, B=5, r=160, C=3, N=5, cache_dtype="bf16", len_lo=3), (3, 6, 1, 1, 128, 128)),
    (Workload("c3", L=14, d=32, n_max=4200, B=2, r=160, C=2, N=2, cache_dtype="bf16", len_lo=3900), (3, 6, 0, 2, 128, 128)),
    (Workload("c4", L=9, d=64, n_max=23, B=1, r=384, C=4, N=1, cache_dtype="bf16", len_lo=0), (5, 2, 1, 1, 128, 128)),
    (Workload("c5", L=20, d=64, n_max=130, B=8, r=192, C=2, N=8, cache_dtype="bf16", len_lo=40), (4, 5, 1, 1, 128, 128)),
    (Workload("c6", L=9, d=32, n_max=120, B=20, r=512, C=2, N=20, cache_dtype="bf16", len_lo=110), (5, 2, 1, 2, 128, 256)),
], ids=lambda v: getattr(v, "name", None))
def test_chains_over_groups_of_layers(w, plan):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens)
    assert tuple(pb.pac_chain_plan(sess.ctx, lens[:w.B], w.B).values()) == plan
    sess.cache_fill(ids, acts, lens)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["bf16"], what=w.name)


# The logit shares of the layer-by-layer chains: loads without a branch up to four classes, per class above.
@pytest.mark.parametrize("C", [1, 4, 5, 16])
def test_chain_class_counts(C):
    w = Workload(f"k{C}", L=9, d=64, n_max=37, B=3, r=160, C=C, N=3, cache_dtype="bf16", len_lo=5)
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens)
    assert pb.pac_step_path(sess.ctx) == 2
    sess.cache_fill(ids, acts, lens)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["bf16"], what=w.name)


# fp32: 16-row tiles with 8, 6 (the second column chunk part empty), 4 and 6 column blocks per workgroup; K of 2 .. 10
# units over eight wavefronts, a last row tile of a few rows.  64 x 64 tiles where they fill the chip: K in long steps (f6)
# and in short ones (f7).
@pytest.mark.parametrize("w,rows", [
    (Workload("f1", L=2, d=96, n_max=130, B=32, r=128, C=3, N=32, cache_dtype="f32", len_lo=128), 16),
    (Workload("f2", L=2, d=160, n_max=68, B=32, r=160, C=2, N=32, cache_dtype="f32", len_lo=62), 16),
    (Workload("f3", L=3, d=64, n_max=68, B=32, r=128, C=2, N=32, cache_dtype="f32", len_lo=62), 16),
    (Workload("f4", L=2, d=32, n_max=130, B=32, r=96, C=5, N=32, cache_dtype="f32", len_lo=128), 16),
    (Workload("f5", L=2, d=288, n_max=9, B=3, r=64, C=2, N=3, cache_dtype="f32", len_lo=1), 16),
    (Workload("f6", L=2, d=64, n_max=75, B=32, r=512, C=2, N=32, cache_dtype="f32", len_lo=70), 64),
    (Workload("f7", L=2, d=96, n_max=140, B=32, r=512, C=3, N=32, cache_dtype="f32", len_lo=135), 64),
    # one layer (no dpre launch for its sums to ride on) and five (the two arrays of the side gradient take turns)
    (Workload("f8", L=1, d=64, n_max=40, B=3, r=32, C=2, N=3, cache_dtype="f32", len_lo=7), 16),
    (Workload("f9", L=5, d=96, n_max=70, B=7, r=64, C=3, N=7, cache_dtype="f32", len_lo=7), 16),
], ids=lambda w: getattr(w, "name", None))
def test_fp32_contractions(w, rows):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    assert tiles_of(w, lens)["proj"] == rows
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens)
    sess.cache_fill(ids, acts, lens)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["f32"], what=w.name)


# fp32 in the Gram-matrix formulation: adapter widths of each instantiation, d of a last tile and a last chunk half empty (96,
# 288, 352), samples of less than one and of several 16-row tiles, fewer than 16 rows in all (t1), 32-row projection tiles (t4),
# a partial last chunk of the vector parts' classes (16), layers whose chains need two wavefronts a unit (t5, and r > 96), token
# splits (t7).
@pytest.mark.parametrize("w", [
    Workload("t1", L=2, d=64, n_max=5, B=2, r=32, C=2, N=2, cache_dtype="f32", len_lo=1),
    Workload("t2", L=4, d=96, n_max=37, B=3, r=32, C=3, N=3, cache_dtype="f32", len_lo=9),
    Workload("t3", L=5, d=288, n_max=33, B=5, r=96, C=16, N=5, cache_dtype="f32", len_lo=15),
    Workload("t4", L=16, d=128, n_max=130, B=12, r=64, C=4, N=12, cache_dtype="f32", len_lo=126),
    Workload("t5", L=31, d=128, n_max=40, B=3, r=64, C=3, N=3, cache_dtype="f32", len_lo=17),
    Workload("t6", L=3, d=352, n_max=50, B=3, r=128, C=1, N=3, cache_dtype="f32", len_lo=3),
    Workload("t7", L=2, d=64, n_max=400, B=8, r=32, C=3, N=8, cache_dtype="f32", len_lo=250),
    Workload("t8", L=3, d=416, n_max=40, B=3, r=192, C=5, N=3, cache_dtype="f32", len_lo=30),
    Workload("t9", L=2, d=512, n_max=20, B=2, r=256, C=3, N=2, cache_dtype="f32"),
], ids=lambda w: w.name)
def test_fp32_gram(w):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    params = inputs.random_params(w, up_scale=0.3)
    got = []
    for flags in (0, pb.PAC_FLAG_SPLIT_LAUNCH):
        sess = make_session(w, lens=lens, flags=flags)
        sess.cache_fill(ids, acts, lens)
        pb.pac_profile_begin(sess.ctx)
        check_against_oracle(w, sess, ids, acts, lens, labels, params, TOL["f32"], what=w.name)
        assert any(k.startswith("g_tokred") and n for k, (_, n) in pb.pac_profile_end(sess.ctx).items())
        got.append((sess.loss.clone(), sess.logits.clone(), sess.grads.clone()))
        sess.loss_grad(ids, torch.from_numpy(labels).to(sess.dev), want_grads=False)
        assert torch.equal(sess.loss, got[0][0]) and torch.equal(sess.logits, got[0][1])
    for a, b in zip(got[0], got[1]):
        assert torch.equal(a, b)
    # a smaller batch on the same workspace, and a training step with the last two sums left to the optimizer
    sel = ids[:max(1, w.B - 1)]
    check_against_oracle(w, sess, sel, acts[sel], None if lens is None else lens[sel], labels[sel], params, TOL["f32"], what=w.name)
    loss, grads = sess.loss.clone(), sess.grads.clone()
    sess.step(sel, torch.from_numpy(labels[sel]).to(sess.dev))
    assert torch.equal(sess.loss, loss) and torch.equal(sess.grads, grads)


# What the cases above leave out of the fp32 Gram-matrix formulation: 32-row projection tiles at each width that has them
# (i1-i3: last tiles of 18 to 32 rows), token splits and their sum at each width (i4-i8: ragged last splits), the most layers
# that fit (i9-i12: 60, 16, 14 and 8).
@pytest.mark.parametrize("w,plan", [
    (Workload("i1", L=16, d=64, n_max=96, B=11, r=32, C=3, N=11, cache_dtype="f32", len_lo=82), (1, 32, 1, 1)),
    (Workload("i2", L=16, d=192, n_max=96, B=11, r=96, C=3, N=11, cache_dtype="f32", len_lo=82), (1, 32, 1, 1)),
    (Workload("i3", L=14, d=512, n_max=96, B=13, r=128, C=3, N=13, cache_dtype="f32", len_lo=82), (1, 32, 1, 2)),
    (Workload("i4", L=2, d=128, n_max=400, B=8, r=64, C=3, N=8, cache_dtype="f32", len_lo=300), (1, 16, 8, 1)),
    (Workload("i5", L=2, d=192, n_max=400, B=8, r=96, C=3, N=8, cache_dtype="f32", len_lo=300), (1, 16, 8, 1)),
    (Workload("i6", L=2, d=256, n_max=400, B=8, r=128, C=3, N=8, cache_dtype="f32", len_lo=300), (1, 16, 8, 2)),
    (Workload("i7", L=2, d=384, n_max=300, B=4, r=192, C=3, N=4, cache_dtype="f32", len_lo=201), (1, 16, 7, 2)),
    (Workload("i8", L=2, d=512, n_max=300, B=4, r=256, C=3, N=4, cache_dtype="f32", len_lo=201), (1, 16, 3, 2)),
    (Workload("i9", L=60, d=64, n_max=20, B=2, r=32, C=3, N=2, cache_dtype="f32", len_lo=3), (1, 16, 1, 1)),
    (Workload("i10", L=16, d=192, n_max=9, B=1, r=96, C=3, N=1, cache_dtype="f32"), (1, 16, 1, 1)),
    (Workload("i11", L=14, d=256, n_max=9, B=1, r=128, C=3, N=1, cache_dtype="f32"), (1, 16, 1, 2)),
    (Workload("i12", L=8, d=768, n_max=64, B=4, r=192, C=3, N=4, cache_dtype="f32", len_lo=30), (1, 16, 1, 2)),
], ids=lambda v: getattr(v, "name", None))
def test_fp32_gram_widths_and_depths(w, plan):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens)
    assert tuple(pb.pac_f32_plan(sess.ctx, lens, w.B).values()) == plan
    sess.cache_fill(ids, acts, lens)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["f32"], what=w.name)


# The per-layer 16-row tiles at the longest K, by flag where the Gram-matrix formulation would be taken (q1: two wavefronts of
# eight with a unit more than the others; q2) and at a width without it (q3).
@pytest.mark.parametrize("w,flags", [
    (Workload("q1", L=2, d=288, n_max=9, B=3, r=64, C=2, N=3, cache_dtype="f32", len_lo=1), pb.PAC_FLAG_PER_LAYER),
    (Workload("q2", L=3, d=768, n_max=33, B=3, r=96, C=3, N=3, cache_dtype="f32", len_lo=9), pb.PAC_FLAG_PER_LAYER),
    (Workload("q3", L=2, d=768, n_max=40, B=3, r=160, C=3, N=3, cache_dtype="f32", len_lo=9), 0),
], ids=lambda v: getattr(v, "name", None))
def test_fp32_per_layer_tiles_at_long_k(w, flags):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens, flags=flags)
    assert not pb.pac_f32_plan(sess.ctx, lens, w.B)["gram"] and pb.pac_step_tiles(sess.ctx, lens, w.B)["proj"] == 16
    sess.cache_fill(ids, acts, lens)
    pb.pac_profile_begin(sess.ctx)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["f32"], what=w.name)
    assert not any(k.startswith("g_") and n for k, (_, n) in pb.pac_profile_end(sess.ctx).items())


# One context whose calls take different formulations: steps on the whole batch the Gram-matrix formulation, all others the
# per-layer kernels (b1), or steps the one and forward-only calls the other (b2).
@pytest.mark.parametrize("w,whole,short", [
    (Workload("b1", L=5, d=512, n_max=64, B=4, r=256, C=3, N=4, cache_dtype="f32", len_lo=3), (1, 0), (0, 0)),
    (Workload("b2", L=13, d=256, n_max=64, B=4, r=128, C=3, N=4, cache_dtype="f32", len_lo=3), (1, 0), (1, 0)),
], ids=lambda v: getattr(v, "name", None))
def test_fp32_formulation_by_batch(w, whole, short):
    lens = np.array([64, 3, 64, 61], dtype=np.int32)
    ids, acts, labels = np.arange(w.B), inputs.batch_acts(w, np.arange(w.B)), inputs.labels(w)[:w.B]
    params = inputs.random_params(w, up_scale=0.3)
    sess = make_session(w, lens=lens)
    sess.cache_fill(ids, acts, lens)
    runs_gram = lambda p: any(k.startswith("g_chain") and n for k, (_, n) in p.items())
    for sel, form in ((ids, whole), (ids[1:2], short)):
        assert tuple(pb.pac_f32_plan(sess.ctx, lens[sel], len(sel), g)["gram"] for g in (True, False)) == form
        lab = torch.from_numpy(labels[sel]).to(sess.dev)
        pb.pac_profile_begin(sess.ctx)
        _, loss, _, _ = check_against_oracle(w, sess, sel, acts[sel], lens[sel], labels[sel], params, TOL["f32"], what=w.name)
        assert runs_gram(pb.pac_profile_end(sess.ctx)) == bool(form[0])
        logits, grads = sess.logits[:len(sel) * w.C].clone(), sess.grads.clone()
        pb.pac_profile_begin(sess.ctx)
        sess.loss_grad(sel, lab, want_grads=False)
        assert runs_gram(pb.pac_profile_end(sess.ctx)) == bool(form[1])
        assert abs(float(sess.loss) - loss) <= TOL["f32"] * abs(loss)
        assert torch.linalg.norm(sess.logits[:len(sel) * w.C] - logits) <= TOL["f32"] * torch.linalg.norm(logits)
        sess.step(sel, lab, keep_grads=False)  # its gradient lies where the formulation's own workspace has it
        assert torch.allclose(sess.m, 0.1 * grads, rtol=1e-5, atol=0)
        sess.set_params(params)


@pytest.mark.parametrize("w", [Workload("b4", L=31, d=128, n_max=26, B=1, r=32, C=3, N=1, cache_dtype="f32"),
                               Workload("b5", L=13, d=256, n_max=64, B=4, r=128, C=3, N=4, cache_dtype="f32", len_lo=3)],
                         ids=lambda w: w.name)
def test_fp32_on_the_per_layer_kernels_workspace(w):
    """A workspace too small for the Gram-matrix formulation gets the per-layer kernels, and their bits."""
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, lab = inputs.batch_acts(w, ids), torch.from_numpy(inputs.labels(w)[ids]).cuda()
    params = inputs.random_params(w, up_scale=0.3)
    per_layer, sess = make_session(w, lens=lens, flags=pb.PAC_FLAG_PER_LAYER), make_session(w, lens=lens)
    assert pb.pac_f32_plan(sess.ctx, lens, w.B)["gram"] and per_layer.ws_bytes < sess.ws_bytes
    sess.ws_bytes = per_layer.ws_bytes
    sess.ws = torch.empty(sess.ws_bytes, dtype=torch.uint8, device=sess.dev)
    got = []
    for s in (per_layer, sess):
        s.cache_fill(ids, acts, lens)
        s.set_params(params)
        s.step(ids, lab)
        step = [t.clone() for t in (s.loss, s.grads, s.params)]
        s.set_params(params)
        s.loss_grad(ids, lab)
        got.append(step + [s.loss.clone(), s.logits.clone(), s.grads.clone()])
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_fp32_gram_within_the_static_workspace():
    """The per-layer kernels would need more than the static entry has, so every batch takes the Gram-matrix formulation."""
    from paper_2408_10746_amd.runtime import _stream_handle
    w = Workload("b3", L=5, d=2208, n_max=2, B=2, r=256, C=3, N=2, cache_dtype="f32")
    ids, acts, labels = np.arange(w.B), inputs.batch_acts(w, np.arange(w.B)), inputs.labels(w)[:w.B]
    sess = make_session(w)
    assert pb.pac_f32_plan(sess.ctx, None, 1, False)["gram"] and sess.ws_bytes <= pb.PAC_STATIC_WORKSPACE_BYTES
    sess.cache_fill(ids, acts)
    params = inputs.random_params(w, up_scale=0.3)
    lab = torch.from_numpy(labels).to(sess.dev)
    check_against_oracle(w, sess, ids, acts, None, labels, params, TOL["f32"], what=w.name)
    sess.step(ids, lab)
    want = [t.clone() for t in (sess.loss, sess.grads, sess.params)]
    sess.set_params(params)
    pb.pac_adapter_step_static(sess.ctx, sess.cache.data_ptr(), ids, lab.data_ptr(), sess.params.data_ptr(), sess.m.data_ptr(),
                               sess.v.data_ptr(), 0, sess.hp, sess.loss.data_ptr(), sess.grads.data_ptr(), _stream_handle())
    for a, b in zip(want, (sess.loss, sess.grads, sess.params)):
        assert torch.equal(a, b)


def test_fp32_gram_error_is_no_larger_than_per_layer():
    """Gradients against float64 in both fp32 formulations: deep narrow adapters, few rows and many, where the Gram-matrix
    formulation has the longest sums and uses the same rounded products (Q, V) for every token.  Geometric means over the
    configurations, of the whole gradient and of the gates' and head's parts; every sum's order is fixed, and so are they."""
    rng = np.random.default_rng(7)
    shapes = []
    while len(shapes) < 48:
        r = int(rng.choice([32, 64, 96, 128]))
        L, d = int(rng.integers(5, {32: 48, 64: 30, 96: 16, 128: 14}[r])), 32 * int(rng.integers(r // 16, 20))
        n, B = int(rng.integers(2, 80)), int(rng.integers(1, 6))
        if L * d * r * n * B < 2e8:
            shapes.append((L, d, r, n, B))
    logs = np.zeros((len(shapes), 3))
    for i, (L, d, r, n, B) in enumerate(shapes):
        w = Workload(f"e{i}", L=L, d=d, n_max=n, B=B, r=r, C=2 + i % 3, N=B, cache_dtype="f32", len_lo=max(1, n // 2))
        lens, ids = inputs.lengths(w), np.arange(B)
        acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
        params = inputs.random_params(w, up_scale=0.3)
        _, ref = oracle_batch(w, acts, lens, labels, params)
        ref = np.asarray(ref["grads"], dtype=np.float64)
        gates = np.arange(1, L + 1) * w.layer_block - 1
        parts = [slice(None), gates, slice(L * w.layer_block, None)]
        err = []
        for flags in (0, pb.PAC_FLAG_PER_LAYER):
            sess = make_session(w, lens=lens, flags=flags)
            sess.cache_fill(ids, acts, lens)
            sess.set_params(params)
            sess.loss_grad(ids, torch.from_numpy(labels).to(sess.dev))
            g = sess.grads.cpu().numpy().astype(np.float64)
            err.append([np.linalg.norm(g[q] - ref[q]) / np.linalg.norm(ref[q]) for q in parts])
        logs[i] = np.log(err[0]) - np.log(err[1])
    ratio = np.exp(logs.mean(0))
    print("error, Gram-matrix formulation / per-layer kernels: all %.3f, gates %.3f, head %.3f" % tuple(ratio))
    assert (ratio <= 1.0).all(), ratio


# What the fp32 launches do for each class: four at a time, a last group of one, two, three and four.
@pytest.mark.parametrize("C", [2, 4, 5, 7, 16])
def test_fp32_gram_class_counts(C):
    w = Workload(f"tc{C}", L=3, d=320, n_max=37, B=3, r=64, C=C, N=3, cache_dtype="f32", len_lo=5)
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, labels = inputs.batch_acts(w, ids), inputs.labels(w)[ids]
    sess = make_session(w, lens=lens)
    sess.cache_fill(ids, acts, lens)
    check_against_oracle(w, sess, ids, acts, lens, labels, inputs.random_params(w, up_scale=0.3), TOL["f32"], what=w.name)


# Every sum behind a gradient has a fixed order, and a launch rule or a faster load is no reason for other results: SHA-1 of
# the gradients' bits.  The rows of the vector gradients: two threads each with 2, 6 and 8 chunks of 16 bytes, four with 5,
# eight with 5.
GRADIENT_BITS = [
    (Workload("v1", L=3, d=96, n_max=40, B=3, r=32, C=3, N=3, cache_dtype="bf16", len_lo=9), "bf07fed9679412bf56da923467881f94334387db"),
    (Workload("v2", L=5, d=160, n_max=50, B=4, r=96, C=4, N=4, cache_dtype="bf16", len_lo=17), "fcc7a8818c9045ccd5ce0796d3e563ec6c8a488b"),
    (Workload("v3", L=4, d=128, n_max=33, B=6, r=128, C=5, N=6, cache_dtype="bf16", len_lo=30), "cfee8560e57df98e45a329d77ae95239dfc47066"),
    (Workload("v4", L=6, d=192, n_max=70, B=3, r=160, C=2, N=3, cache_dtype="bf16", len_lo=20), "b65bb0db09c5898d574722af252de0d5bd5a0335"),
    (Workload("v5", L=3, d=160, n_max=45, B=4, r=320, C=3, N=4, cache_dtype="bf16", len_lo=11), "ea5613cd8f4175923a991598be845cc257956889"),
]


# Per-layer path: with PAC_FLAG_SPLIT_LAUNCH every part of the joined launches is a launch of its own class, with the same
# bits.  fp32 on 16-row tiles with one layer and with five, on 64 x 64 tiles; bf16 by flag.
@pytest.mark.parametrize("w,flags", [
    (Workload("l1", L=1, d=64, n_max=40, B=3, r=32, C=2, N=3, cache_dtype="f32", len_lo=7), 0),
    (Workload("l5", L=5, d=96, n_max=70, B=7, r=64, C=3, N=7, cache_dtype="f32", len_lo=7), 0),
    (Workload("l3", L=3, d=64, n_max=75, B=32, r=512, C=2, N=32, cache_dtype="f32", len_lo=70), 0),
    (Workload("b3", L=3, d=96, n_max=50, B=5, r=64, C=3, N=5, cache_dtype="bf16", len_lo=9), pb.PAC_FLAG_PER_LAYER),
], ids=lambda v: getattr(v, "name", None))
def test_per_layer_split_launches(w, flags):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    acts, lab = inputs.batch_acts(w, ids), torch.from_numpy(inputs.labels(w)[ids]).cuda()
    got, launches = [], []
    for split in (0, pb.PAC_FLAG_SPLIT_LAUNCH):
        sess = make_session(w, lens=lens, flags=flags | split)
        assert pb.pac_step_path(sess.ctx) == 0
        sess.cache_fill(ids, acts, lens)
        sess.set_params(inputs.random_params(w, up_scale=0.5))
        pb.pac_profile_begin(sess.ctx)
        sess.loss_grad(ids, lab)
        torch.cuda.synchronize()
        launches.append({k: n for k, (_, n) in pb.pac_profile_end(sess.ctx).items() if k.startswith(("head_bwd", "bwd_", "reduce"))})
        got.append((sess.loss.clone(), sess.logits.clone(), sess.grads.clone()))
    assert launches[0] == {"head_bwd": 1, "bwd_dpre": w.L, "bwd_layer": w.L, "reduce": 1}
    assert launches[1] == {"head_bwd": 1, "bwd_dpre": w.L + 1, "bwd_wgrad": w.L, "bwd_dx": w.L, "reduce": w.L}
    for a, b in zip(got[0], got[1]):
        assert torch.equal(a, b)


def gradients(w):
    lens, ids = inputs.lengths(w), np.arange(w.B)
    sess = make_session(w, lens=lens)
    sess.cache_fill(ids, inputs.batch_acts(w, ids), lens)
    sess.set_params(inputs.random_params(w, up_scale=0.3))
    sess.loss_grad(ids, torch.from_numpy(inputs.labels(w)[ids]).to(sess.dev))
    return sess.grads.cpu().numpy()


@pytest.mark.parametrize("w,sha1", GRADIENT_BITS, ids=[w.name for w, _ in GRADIENT_BITS])
def test_gradients_keep_their_bits(w, sha1):
    assert hashlib.sha1(gradients(w).tobytes()).hexdigest() == sha1
