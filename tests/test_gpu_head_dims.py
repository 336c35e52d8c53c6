"""The attention at every head_dim it accepts (multiples of 8: bf16 up to 128, float32 up to 64). bf16: QK remainders
of 0, 8, 16 and 24 columns, denominators in a padding row or in a block of their own, swizzled and plain LDS rows;
float32: padded to 32, 48 or 64 columns, split and unsplit."""
import math

import numpy as np
import pytest

import oracle
from paper_2505_20600_amd import workloads as W
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,dtype", [(h, "bf16") for h in range(8, 129, 8)] + [(h, "fp32") for h in range(8, 65, 8)])
@pytest.mark.parametrize("split", ["1", "100000"], ids=["unsplit", "split"])
def test_block_at_every_head_dim_matches_oracle(hd, dtype, split, monkeypatch):
    """Three key tiles with a ragged tail (T = 138), a request that fills two query tiles and leaves waves of the
    second without rows, a request of one masked token; cached keys grow along the sequence, so that running maxima
    rise by more than the rescale threshold after the first tile."""
    monkeypatch.setenv("MS_ATTN_SPLIT_TARGET", split)
    d = hd * 64 // math.gcd(hd, 64)
    shape = W.ModelShape(f"hd{hd}", 1, d, d // hd, 2, 9, 15, n_text=3, dtype=dtype, batch=2)
    ws = W.stack_weights(shape, 300 + hd, random_ln=True, std=0.03)
    stored = W.to_bf16_values if dtype == "bf16" else lambda v: np.asarray(v, np.float32)
    # queries of standard deviation 2: scores up to ~20 in the exp2 domain
    ws[0]["w_qkv"][:d] = stored(ws[0]["w_qkv"][:d] * (2.0 / (0.03 * math.sqrt(d))))
    xt = W.template_hidden(shape, 300 + hd)
    kv = np.stack([W.synthetic_kv_cache(shape, 300 + hd, 0)])
    kv[0, :, :, 0] = stored(kv[0, :, :, 0] * np.linspace(0.1, 4.0, shape.n_tokens, dtype=np.float32)[None, :, None])
    yc = W.synthetic_y_cache(shape, 300 + hd)
    mask = np.zeros((2, shape.n_image), np.uint8)
    mask[0, W.rng(300, 3, hd).permutation(shape.n_image)[:130]] = 1
    mask[1, 77] = 1
    x = W.edited_hidden(shape, 300 + hd, xt, mask)
    y, kv_gpu, _ = G.run_stack(shape, mask, x, kv, yc, ws)
    y_ref, kv_ref = oracle.masked_stack(x, mask, kv, yc, ws, shape, return_kv=True, round_p=dtype == "bf16")
    G.assert_close(y, y_ref, dtype, f"head_dim {hd} output", blocks=1, inp=x)
    G.assert_close(kv_gpu[0], kv_ref[0], dtype, f"head_dim {hd} K/V", blocks=1)


@pytest.mark.parametrize("hd,dtype", [(40, "bf16"), (64, "bf16"), (72, "bf16"), (128, "bf16"), (64, "fp32")])
@pytest.mark.parametrize("split", ["1", "100000"], ids=["unsplit", "split"])
@pytest.mark.parametrize("far", [(0,), (1,), (0, 1)], ids=["first", "second", "first-two"])
def test_key_tiles_far_from_the_others_match_oracle(hd, dtype, split, far, monkeypatch):
    """Three key tiles; every cached key of the tiles `far` scores -inf, the type's lowest value, large negative or
    large positive values against every query (one request each, the last with plain keys), so that a whole key range
    weighs nothing, or all others do, and a maximum jumps by far more than a score's digits hold. The queries are
    a bias in one column, so that the scores are products of two numbers."""
    monkeypatch.setenv("MS_ATTN_SPLIT_TARGET", split)
    lowest = -3.3895313892515355e38      # bf16; float32's own is below it
    values = [-np.inf, lowest, -2e37, -1e7, 1e12, None]
    d = hd * 64 // math.gcd(hd, 64)
    shape = W.ModelShape(f"far{hd}", 1, d, d // hd, 2, 9, 15, dtype=dtype, batch=len(values))
    ws = W.stack_weights(shape, 500 + hd, random_ln=True, std=0.03)
    stored = W.to_bf16_values if dtype == "bf16" else lambda v: np.asarray(v, np.float32)
    ws[0]["w_qkv"][:d] = 0.0
    ws[0]["b_qkv"][:d] = 0.0
    ws[0]["b_qkv"][0:d:hd] = 8.0
    xt = W.template_hidden(shape, 500 + hd)
    kv = np.stack([W.synthetic_kv_cache(shape, 500 + hd, 0)])
    keys = np.concatenate([np.arange(64 * t, 64 * t + 64) for t in far])
    for b, v in enumerate(values):
        if v is not None:
            # two values, so that the large positive ones are told apart (the weights of the lower are 0)
            kv[0, b, keys, 0, 0:d:hd] = v
            kv[0, b, keys[1::2], 0, 0:d:hd] = v if np.isinf(v) else stored(np.float32([0.9 * v]))
    kv[0, :, :, 0] = np.where(np.isfinite(kv[0, :, :, 0]), stored(kv[0, :, :, 0]), kv[0, :, :, 0])
    yc = W.synthetic_y_cache(shape, 500 + hd)
    mask = np.zeros((len(values), shape.n_image), np.uint8)
    mask[:, [129, 131, 134] if 1 in far else [64, 100, 127, 130]] = 1
    x = W.edited_hidden(shape, 500 + hd, xt, mask)
    y, _, _ = G.run_stack(shape, mask, x, kv, yc, ws, return_kv=False)
    y_ref = oracle.masked_stack(x, mask, kv, yc, ws, shape, round_p=dtype == "bf16")
    assert np.isfinite(y_ref).all()
    for b, v in enumerate(values):
        G.assert_close(y[b], y_ref[b], dtype, f"head_dim {hd}, keys of {v}", blocks=1, inp=x[b])
