"""The 256-row GEMM tiles (16 x 16 x 32 MFMAs) at the edges of their range.

Every stage of a layer against the oracle (gpu_stages) on models without packed
weights, at row counts that leave a few rows in the last tile and sequences that
start anywhere in one.  In order: 256 x 256 for gate/up and the down projection
split over K; 256 x 256 for q/k/v and both residual projections, 256 x 192 for
gate/up; 256 x 192 for q/k/v (q and k, and k and v, in one tile) and both residual
projections; 256 x 256 throughout, v^T in whole 16-byte pieces.
"""
import math

import numpy as np
import pytest
import torch

from gpu_stages import check_layer
from paper_2608_22646_amd import binding as B
from paper_2608_22646_amd import synth

pytestmark = pytest.mark.gpu


# (d, heads, kv heads, d_ff), sequences, length
@pytest.mark.parametrize("shape,Bn,L", [((512, 4, 2, 4096), 1, 8201), ((1024, 8, 2, 1152), 3, 2733),
                                        ((768, 8, 2, 640), 3, 5461), ((768, 8, 2, 640), 8, 2504)])
def test_full_layer(gpu_lib, shape, Bn, L):
    d, heads, kv, ff = shape
    cfg = synth.ModelConfig("tiles-bf16", n_layers=1, d_model=d, n_heads=heads, n_kv_heads=kv, head_dim=128, d_ff=ff,
                            vocab=1000, rope_base=10000.0, dtype="bf16", lm_head_std=5 / math.sqrt(d), norm_gain_std=0.1)
    w = synth.make_weights(cfg, "cpu")
    model = B.Model(cfg, [t.cuda() for t in w])
    M = Bn * L
    ws = model.workspace(Bn, L, 0)
    model.embed(synth.make_ints((Bn, L), 5, 0, cfg.vocab).cuda(), ws)
    rows = np.unique(np.concatenate([np.random.default_rng(0).choice(M, 60, replace=False), np.arange(M - 12, M)]))
    check_layer(model, cfg, [t.float().numpy() for t in w], ws, Bn, L, 0, rows=rows)


# activations of the down projection beyond 2 GiB, the end of 32-bit buffer offsets (row 56680 at 18944 columns), in
# one K range (65536 rows) and split over K (65792): every stage of rows around there and in the last sequences
@pytest.mark.parametrize("L", [4096, 4112])
def test_activations_beyond_two_gib(gpu_lib, L):
    cfg = synth.ModelConfig("large-bf16", n_layers=1, d_model=256, n_heads=2, n_kv_heads=2, head_dim=128, d_ff=18944,
                            vocab=1000, rope_base=10000.0, dtype="bf16", lm_head_std=5 / 16, norm_gain_std=0.1)
    w = synth.make_weights(cfg, "cpu")
    model = B.Model(cfg, [t.cuda() for t in w])
    Bn, edge = 16, 2 ** 31 // (2 * cfg.d_ff)
    ws = model.workspace(Bn, L, 0)
    model.embed(synth.make_ints((Bn, L), 5, 0, cfg.vocab).cuda(), ws)
    rows = np.unique(np.concatenate([np.arange(edge - 6, edge + 6), np.random.default_rng(0).integers(edge, Bn * L, 24),
                                     np.arange(Bn * L - 6, Bn * L)]))
    check_layer(model, cfg, [t.float().numpy() for t in w], ws, Bn, L, 0, rows=rows)


def test_weights_beyond_two_gib_are_refused(gpu_lib):
    """A weight tensor past the end of 32-bit buffer offsets: the layer half that reads it is refused, the other runs."""
    cfg = synth.ModelConfig("wide-bf16", n_layers=1, d_model=4096, n_heads=2, n_kv_heads=2, head_dim=128, d_ff=262272,
                            vocab=1000, rope_base=10000.0, dtype="bf16")
    w = [torch.zeros(shape, dtype=torch.bfloat16, device="cuda") for _, shape, _ in synth.weight_specs(cfg)]
    model = B.Model(cfg, w)
    ws = model.workspace(1, 40, 0)
    model.embed(synth.make_ints((1, 40), 5, 0, cfg.vocab).cuda(), ws)
    model.layer(0, 0, 1, 40, ws)
    for part in (1, 2):
        with pytest.raises(B.DllmError, match="2 GiB"):
            model.layer(0, part, 1, 40, ws)
