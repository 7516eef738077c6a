"""The few-row GEMM (packed weights, at most 64 rows) at the edges of its plans.

Every stage of a layer against the oracle (gpu_stages), at widths whose 32-row
groups divide into every group count a workgroup takes, leave remainders, or
give some waves no slice of K; one and two row operands, whole and partial; the
attention kernels that write its operand-order input, at even and odd lengths
(an odd length's V^T rows start in the middle of a dword) with one and several
key splits and waves without a tile; and the split residual sums folded into the
next norm against the separate reduction.
"""
import math

import numpy as np
import pytest
import torch

from gpu_stages import check_layer, check_layer_cached
from paper_2608_22646_amd import binding as B
from paper_2608_22646_amd import synth

pytestmark = pytest.mark.gpu


def model_of(d, heads, kv, ff, layers=1):
    cfg = synth.ModelConfig("rows-edge", n_layers=layers, d_model=d, n_heads=heads, n_kv_heads=kv, head_dim=128,
                            d_ff=ff, vocab=1000, rope_base=10000.0, dtype="bf16", lm_head_std=5 / math.sqrt(d),
                            norm_gain_std=0.1)
    w = synth.make_weights(cfg, "cpu")
    return cfg, B.Model(cfg, [t.cuda() for t in w]).pack_weights(), [t.to(torch.float32).numpy() for t in w]


# (d, heads, kv heads, d_ff): 256 = eight groups, one 16-k slice per wave; 2304 =
# 72 groups; d_ff 18944 = 1184 gate/up groups (five a workgroup at 32 rows)
SHAPES = [(256, 2, 2, 128), (2304, 18, 2, 1408), (3584, 28, 4, 18944)]
# q/k/v two groups a workgroup and gate/up three, and the other way round
WIDE = [(512, 32, 32, 12288), (512, 48, 48, 8192)]


@pytest.mark.parametrize("shape", SHAPES + WIDE)
@pytest.mark.parametrize("Bn,L", [(1, 1), (1, 31), (2, 17), (1, 64)])
def test_full_forward_of_few_rows(gpu_lib, shape, Bn, L):
    cfg, model, w = model_of(*shape)
    ws = model.workspace(Bn, L, min(L, 32))
    model.embed(synth.make_ints((Bn, L), 3, 0, cfg.vocab).cuda(), ws)
    check_layer(model, cfg, w, ws, Bn, L, 0)


@pytest.mark.parametrize("d,offset", [(8448, 0), (512, 1)])
@pytest.mark.parametrize("Bn,L", [(1, 5), (2, 31)])
def test_half_layers_of_wide_rows_and_of_gains_at_any_element(gpu_lib, d, offset, Bn, L):
    """Rows beyond the vector norms' 8192 columns, and gains that are not 16-byte aligned."""
    cfg = synth.ModelConfig("norm-edge", n_layers=1, d_model=d, n_heads=2, n_kv_heads=2, head_dim=128, d_ff=128,
                            vocab=1000, rope_base=10000.0, dtype="bf16", norm_gain_std=0.1)
    w = synth.make_weights(cfg, "cpu")
    dev = [t.cuda() for t in w]
    for i in (1, 6):  # the layer's two gains
        dev[i] = torch.cat([dev[i][:offset], dev[i]])[offset:]
    model = B.Model(cfg, dev).pack_weights()
    ws = model.workspace(Bn, L, 0)
    model.embed(synth.make_ints((Bn, L), 3, 0, cfg.vocab).cuda(), ws)
    check_layer(model, cfg, [t.to(torch.float32).numpy() for t in w], ws, Bn, L, 0)


@pytest.mark.parametrize("shape", SHAPES[1:])
@pytest.mark.parametrize("Bn,L,row0,rows", [(1, 77, 40, 32), (1, 515, 483, 32), (16, 33, 0, 4), (3, 50, 9, 16), (1, 200, 101, 64), (2, 96, 64, 32)])
def test_cached_rows(gpu_lib, shape, Bn, L, row0, rows):
    cfg, model, w = model_of(*shape)
    kv, ws = model.kv_cache(Bn, L), model.workspace(Bn, L, rows)
    x = synth.make_ints((Bn, L), 4, 0, cfg.vocab).cuda()
    model.embed(x, ws)
    model.layer_kv(0, 2, Bn, L, 0, L, kv, ws)
    model.embed_rows(x.flip(1).contiguous(), row0, rows, ws)
    check_layer_cached(model, cfg, w, ws, kv, Bn, L, row0, rows, 0)


# 32 rows and fewer: the keys of a head over four workgroups at these lengths; more: the key-group kernel
@pytest.mark.parametrize("L,rows", [(515, 20), (544, 32), (515, 50)])
@pytest.mark.parametrize("first", [0, 128, 256])
def test_nan_keys_reach_every_query(gpu_lib, L, rows, first):
    """NaN keys that fill all tiles of one workgroup's share."""
    cfg, model, _ = model_of(512, 4, 2, 128)
    kv, ws = model.kv_cache(1, L), model.workspace(1, L, rows)
    x = synth.make_ints((1, L), 4, 0, cfg.vocab).cuda()
    model.embed(x, ws)
    model.layer_kv(0, 2, 1, L, 0, L, kv, ws)
    out = ws[model.layout(1, L, rows).attn:][:rows * 512 * 2].view(torch.bfloat16)
    K = kv[:2 * 2 * L * 128].view(torch.bfloat16).view(2, L, 128)
    for nan in (False, True):
        if nan:
            K[:, first:first + 128] = math.nan
        model.embed_rows(x, L - rows, rows, ws)
        model.layer_kv(0, 0, 1, L, L - rows, rows, kv, ws)
        assert (torch.isnan(out) if nan else torch.isfinite(out)).all()


@pytest.mark.parametrize("rows", [5, 32, 64])
def test_folded_residual_sums_equal_the_reduction(gpu_lib, rows):
    cfg, model, _ = model_of(3584, 28, 4, 1408, layers=2)
    L, row0 = 130, 40
    x = synth.make_ints((1, L), 6, 0, cfg.vocab).cuda()
    kv, ws = model.kv_cache(1, L), model.workspace(1, L, rows)
    model.forward_kv(x, row0, rows, kv, refresh=True, ws=ws)
    kv2 = B.device_buffer(kv.numel()).copy_(kv)
    _, _, fused = model.forward_kv(x, row0, rows, kv, refresh=False, ws=ws, logits=True)
    model.embed_rows(x, row0, rows, ws)
    for l in range(cfg.n_layers):
        model.layer_kv(l, 2, 1, L, row0, rows, kv2, ws)
    h = ws[model.layout(1, L, rows).h:][:rows * cfg.d_model * 4].view(torch.float32).view(rows, -1).clone()
    _, _, calls = model.head_noalloc(h, 1, rows, 0, rows, logits=True)
    assert torch.equal(fused.view(torch.int32), calls.view(torch.int32))
    assert torch.equal(kv, kv2)


@pytest.mark.parametrize("rows", [33, 64, 65, 128, 129, 224, 256])
@pytest.mark.parametrize("V,mask", [(1000, 999), (515, 512), (257, 0)])
def test_head_rows_and_vocabulary_edges(gpu_lib, monkeypatch, rows, V, mask):
    """The head kernels' row counts and vocabulary remainders, with and without the logits buffer: the mask id first,
    in the last partial group or alone past a whole tile; confidences against float64 of the kernel's own logits."""
    d = 256
    cfg = synth.ModelConfig("head-edge", n_layers=0, d_model=d, n_heads=2, n_kv_heads=2, head_dim=128, d_ff=128,
                            vocab=V, rope_base=10000.0, dtype="bf16", lm_head_std=5 / math.sqrt(d))
    w = [t.cuda() for t in synth.make_weights(cfg, "cpu")]
    c = B.model_cfg(cfg)
    c.mask_id = mask
    monkeypatch.setattr(B, "model_cfg", lambda _: c)
    model = B.Model(cfg, w)
    h = synth.make_normal((rows, d), 9).cuda()
    Bn = 4 if rows % 4 == 0 else 1
    conf, arg, lg = model.head_noalloc(h, Bn, rows // Bn, 0, rows // Bn, logits=True)
    conf2, arg2, _ = model.head_noalloc(h, Bn, rows // Bn, 0, rows // Bn)
    assert torch.equal(conf.view(torch.int32), conf2.view(torch.int32)) and torch.equal(arg, arg2)
    x = lg.view(rows, V).double().cpu().numpy()
    x[:, mask] = -np.inf
    p = 1.0 / np.exp(x - x.max(-1, keepdims=True)).sum(-1)
    # float32 exponentials and sums of up to 1000 terms: a few 2^-24 each
    np.testing.assert_allclose(conf.view(-1).cpu().numpy(), p, rtol=3e-6)
    np.testing.assert_array_equal(arg.view(-1).cpu().numpy(), x.argmax(-1))
