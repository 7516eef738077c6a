"""Sequence lengths that are no multiple of 8, through each attention kernel.

V^T rows then start at any multiple of two bytes: the streaming kernels read a
copy with padded rows, and the q/k/v epilogue stores v one value per lane.
Every stage of a layer against the oracle (gpu_stages), for full forwards (one
query group per workgroup and several, batches whose sequences start anywhere)
and for cached windows of more than 32 rows.
"""
import math

import numpy as np
import pytest
import torch

from gpu_stages import check_layer, check_layer_cached
from paper_2608_22646_amd import binding as B
from paper_2608_22646_amd import synth

pytestmark = pytest.mark.gpu

CFG = synth.ModelConfig("ragged-bf16", n_layers=1, d_model=512, n_heads=4, n_kv_heads=2, head_dim=128, d_ff=768,
                        vocab=1000, rope_base=10000.0, dtype="bf16", lm_head_std=5 / math.sqrt(512), norm_gain_std=0.1)


@pytest.fixture(scope="module")
def small():
    w = synth.make_weights(CFG, "cpu")
    return B.Model(CFG, [t.cuda() for t in w]), [t.to(torch.float32).numpy() for t in w]


# L = 33 .. 64: one streaming workgroup a head; (1, 65) .. (1, 2999) the key-group kernel
# with 64 queries a workgroup, (4, 1045) with 96; (16, 509) the four-wave and (4, 8201) the eight-wave streaming kernel
@pytest.mark.parametrize("Bn,L", [(1, 33), (3, 63), (1, 65), (2, 101), (1, 515), (1, 2999), (4, 1045), (16, 509),
                                  (4, 8201)])
def test_full_layer(gpu_lib, small, Bn, L):
    model, w = small
    ws = model.workspace(Bn, L, 0)
    model.embed(synth.make_ints((Bn, L), 5, 0, CFG.vocab).cuda(), ws)
    rows = None if Bn * L <= 300 else np.sort(np.random.default_rng(0).choice(Bn * L, 96, replace=False))
    check_layer(model, CFG, w, ws, Bn, L, 0, rows=rows)


@pytest.mark.parametrize("Bn,L,row0,rows", [(1, 203, 101, 64), (2, 97, 30, 40), (3, 130, 67, 50)])
def test_cached_window(gpu_lib, small, Bn, L, row0, rows):
    model, w = small
    kv, ws = model.kv_cache(Bn, L), model.workspace(Bn, L, rows)
    x = synth.make_ints((Bn, L), 4, 0, CFG.vocab).cuda()
    model.embed(x, ws)
    model.layer_kv(0, 2, Bn, L, 0, L, kv, ws)
    model.embed_rows(x.flip(1).contiguous(), row0, rows, ws)
    check_layer_cached(model, CFG, w, ws, kv, Bn, L, row0, rows, 0)


@pytest.mark.parametrize("L,rows", [(45, 40), (203, 50)])  # a streaming workgroup a head; the key-group kernel
def test_a_nan_value_stays_in_its_dimension(gpu_lib, small, L, rows):
    """What lies behind a V^T row in the last tile takes no part, not even as 0 * NaN."""
    model, _ = small
    kv, ws = model.kv_cache(1, L), model.workspace(1, L, rows)
    x = synth.make_ints((1, L), 4, 0, CFG.vocab).cuda()
    model.embed(x, ws)
    model.layer_kv(0, 2, 1, L, 0, L, kv, ws)
    n = (2 * L * 128 * 2 + 255) // 256 * 256
    kv[n:n + 2 * 128 * L * 2].view(torch.float16).view(2, 128, L)[:, 70, :5] = math.nan
    model.embed_rows(x, L - rows, rows, ws)
    model.layer_kv(0, 0, 1, L, L - rows, rows, kv, ws)
    out = ws[model.layout(1, L, rows).attn:][:rows * 512 * 2].view(torch.bfloat16).view(rows, 4, 128)
    nan = torch.isnan(out)
    assert nan[:, :, 70].all() and int(nan.sum()) == rows * 4
