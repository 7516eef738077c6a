"""float32 models at the edges of the matrix-core tiles, against the float64 oracle.

The tile edges: rows and columns that are no multiple of 16, reduction lengths
that are no multiple of 16 (scalar operand loads), widths beyond the fused
norm's 512, both head dimensions, grouped heads, and enough rows for every tile
height (16 rows on eight or four waves, 32 rows).
"""
import math

import numpy as np
import pytest
import torch

from oracle import forward as of
from oracle import vocab as ov
from paper_2608_22646_amd import binding as B
from paper_2608_22646_amd import synth

pytestmark = pytest.mark.gpu


def config(d, heads, kv, hd, ff, vocab):
    return synth.ModelConfig("f32-edge", n_layers=2, d_model=d, n_heads=heads, n_kv_heads=kv, head_dim=hd, d_ff=ff,
                             vocab=vocab, rope_base=10000.0, dtype="f32", lm_head_std=5.0 / math.sqrt(d),
                             norm_gain_std=0.2)


@pytest.mark.parametrize("Bn,L,row0,rows,shape", [
    (1, 17, 1, 9, (250, 4, 2, 64, 333, 777)),      # scalar loads, every dimension ragged
    (1, 1, 0, 1, (256, 2, 1, 128, 88, 100)),       # a single position
    (3, 45, 7, 32, (528, 4, 2, 128, 352, 1031)),   # norm in its own launch
    (2, 301, 200, 33, (512, 6, 3, 64, 720, 2048)), # widest fused norm
    (4, 530, 3, 64, (256, 4, 4, 64, 704, 4099)),   # 32-row tiles
])
def test_forward_matches_float64(gpu_lib, Bn, L, row0, rows, shape):
    cfg = config(*shape)
    w = synth.make_weights(cfg, "cpu")
    model = B.Model(cfg, [t.cuda() for t in w])
    x = synth.make_ints((Bn, L), 5, 0, cfg.vocab)
    conf, arg, lg = model.forward(x.cuda(), row0, rows, logits=True)
    ref = of.forward(cfg, [t.numpy().astype(np.float64) for t in w], x.numpy(), rows=np.arange(row0, row0 + rows))
    got = lg.cpu().numpy().astype(np.float64)
    # a stored float32 value is the rounding of a float64 sum; two layers of such
    # roundings (2^-24 relative each, ~20 per path) on logits of spread 5
    assert np.abs(got - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max() / 5)
    c_ref, a_ref = ov.confidence_argmax(got, cfg.mask_id)
    np.testing.assert_allclose(conf.cpu().numpy(), c_ref, rtol=2e-6)
    np.testing.assert_array_equal(arg.cpu().numpy(), a_ref)


def test_scores_of_minus_infinity_drop_out(gpu_lib):
    """Keys whose scores are -inf take no part, also where whole 16-key tiles are of that kind."""
    cfg = config(256, 4, 4, 64, 64, 64)
    model = B.Model(cfg, [t.cuda() for t in synth.make_weights(cfg, "cpu")])
    L, pos, dead = 64, 40, 32
    ws, kv, lay = model.workspace(1, L, 1), model.kv_cache(1, L), model.layout(1, L, 1)
    n = cfg.n_kv_heads * L * cfg.head_dim
    K = kv[:4 * n].view(torch.float32).view(cfg.n_kv_heads, L, cfg.head_dim)
    V = kv[4 * n:8 * n].view(torch.float32).view(cfg.n_kv_heads, cfg.head_dim, L)
    kv.zero_()
    K.copy_(synth.make_normal(K.shape, 7))
    V.copy_(synth.make_normal(V.shape, 8))
    x = synth.make_ints((1, L), 3, 0, cfg.vocab).cuda()
    q = ws[lay.q:lay.q + 4 * 256].view(torch.float32).view(4, 1, 64)
    for _ in range(2):  # the first pass only yields q; its signs then make every dead key's score -inf
        model.embed_rows(x, pos, 1, ws)
        model.layer_kv(0, 0, 1, L, pos, 1, kv, ws)
        K[:, :dead] = torch.where(q > 0, -math.inf, math.inf).expand(-1, dead, -1)
    got = ws[lay.attn:lay.attn + 4 * 256].view(torch.float32).double().cpu().numpy().reshape(4, 64)
    qd = q.double().cpu().numpy()[:, 0]
    kk, vv = K.double().cpu().numpy()[:, dead:], V.double().cpu().numpy()[:, :, dead:]
    sc = (qd[:, None] * kk).sum(-1) / 8.0
    p = np.exp(sc - sc.max(-1, keepdims=True))
    ref = ((p / p.sum(-1, keepdims=True))[:, None] * vv).sum(-1)
    np.testing.assert_allclose(got, ref, rtol=1e-6, atol=1e-6)


def windowed(cfg, w, x, row0, rows):
    """Layer 0's attention half on a window of the sequence x over a random cache: (q, K, V^T, attention output)
    in float64, and a function that runs the half again."""
    model = B.Model(cfg, [t.cuda() for t in w])
    L, H, hd = x.shape[1], cfg.n_heads, cfg.head_dim
    ws, kv, lay = model.workspace(1, L, rows), model.kv_cache(1, L), model.layout(1, L, rows)
    n = cfg.n_kv_heads * L * hd
    K = kv[:4 * n].view(torch.float32).view(cfg.n_kv_heads, L, hd)
    V = kv[4 * n:8 * n].view(torch.float32).view(cfg.n_kv_heads, hd, L)
    kv.zero_()
    K.copy_(synth.make_normal(K.shape, 7))
    V.copy_(synth.make_normal(V.shape, 8))
    model.embed_rows(x.cuda(), row0, rows, ws)

    def run():
        model.layer_kv(0, 0, 1, L, row0, rows, kv, ws)
        q = ws[lay.q:lay.q + 4 * H * rows * hd].view(torch.float32).view(H, rows, hd)
        out = ws[lay.attn:lay.attn + 4 * rows * H * hd].view(torch.float32).view(rows, H, hd).transpose(0, 1)
        return [t.double().cpu().numpy() for t in (q, K, V, out)]
    return K, run


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("first", [0, 48, 96])
def test_nan_keys_reach_every_query(gpu_lib, hd, first):
    """A whole 16-key tile of NaN keys, also where it is the first its wave sees."""
    cfg = config(256, 4, 2, hd, 64, 64)
    K, run = windowed(cfg, synth.make_weights(cfg, "cpu"), synth.make_ints((1, 150), 3, 0, cfg.vocab), 120, 20)
    assert np.isfinite(run()[3]).all()
    K[:, first:first + 16] = math.nan
    assert np.isnan(run()[3]).all()


@pytest.mark.parametrize("hd", [64, 128])
def test_queries_without_a_score_leave_the_others_alone(gpu_lib, hd):
    """Some queries of a 16-query tile are NaN (their projection overflows float32), so none of their scores counts;
    the others' results are the float64 ones."""
    cfg = config(256, 4, 2, hd, 64, 64)
    w = synth.make_weights(cfg, "cpu")
    L, row0, rows, bad = 150, 110, 32, 5
    w[0][:, 3] = 0.0
    w[0][bad, 3] = 3.0  # column 3 of h, and with it a q pair of every head, is that token's alone
    for h in range(cfg.n_heads):
        for j in (7, 7 + hd // 2):
            w[2][h * hd + j] = 0.0
            w[2][h * hd + j, 3] = 3e38
    x = synth.make_ints((1, L), 3, bad + 1, cfg.vocab)
    at = [1, 2, 9, 16, 31]
    x[0, [row0 + i for i in at]] = bad
    _, run = windowed(cfg, w, x, row0, rows)
    q, K, V, out = run()
    good = np.setdiff1d(np.arange(rows), at)
    assert np.isnan(out[:, at]).all()
    rep = cfg.n_heads // cfg.n_kv_heads
    for h in range(cfg.n_heads):
        sc = q[h, good] @ K[h // rep].T / math.sqrt(hd)
        p = np.exp(sc - sc.max(-1, keepdims=True))
        ref = (p / p.sum(-1, keepdims=True)) @ V[h // rep].T
        # float64 sums on both sides: what differs is one float32 rounding of values of size ~1
        np.testing.assert_allclose(out[h, good], ref, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("hd", [64, 128])
def test_longest_sequence(gpu_lib, hd):
    """A window at the end of 8000 positions; one more is refused."""
    cfg = config(256, 4, 2, hd, 64, 64)
    w, L, rows = synth.make_weights(cfg, "cpu"), 8000, 3
    _, run = windowed(cfg, w, synth.make_ints((1, L), 3, 0, cfg.vocab), L - rows, rows)
    q, K, V, out = run()
    for h in range(cfg.n_heads):
        sc = q[h] @ K[h // 2].T / math.sqrt(hd)
        p = np.exp(sc - sc.max(-1, keepdims=True))
        np.testing.assert_allclose(out[h], (p / p.sum(-1, keepdims=True)) @ V[h // 2].T, rtol=1e-6, atol=1e-6)
    with pytest.raises(B.DllmError, match="8000"):
        windowed(cfg, w, synth.make_ints((1, L + 1), 3, 0, cfg.vocab), L - rows, rows)


def test_head_timing_holds_the_reduction(gpu_lib):
    """PROF_HEAD is the head's GEMM and reduction: nearly all of a forward without layers over a wide vocabulary."""
    cfg = synth.ModelConfig("f32-head", n_layers=0, d_model=16, n_heads=1, n_kv_heads=1, head_dim=64, d_ff=16,
                            vocab=400000, rope_base=10000.0, dtype="f32")
    model = B.Model(cfg, [t.cuda() for t in synth.make_weights(cfg, "cpu")])
    x, ws = synth.make_ints((1, 1), 3, 0, cfg.vocab).cuda(), model.workspace(1, 1, 1)
    model.forward(x, 0, 1, ws=ws)
    a, b = torch.cuda.Event(True), torch.cuda.Event(True)
    model.prof_enable([B.PROF_HEAD])
    a.record()
    for _ in range(10):
        model.forward(x, 0, 1, ws=ws)
    b.record()
    b.synchronize()
    ms, n = model.prof_read(B.PROF_HEAD)
    assert n == 10 and ms > 0.5 * a.elapsed_time(b)
