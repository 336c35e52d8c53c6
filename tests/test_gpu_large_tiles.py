"""The large GEMM tiles under the QKV epilogue (16-byte stores of the K/V columns through the row table, tiles that
straddle the Q columns' end, K/V only, more tiles than CUs), which the planner picks for wide models and many rows and
the other tests' small models do not reach; and the deeper stage variants under the epilogues that stage bf16."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

import oracle
from paper_2505_20600_amd import maskstep as MS
from paper_2505_20600_amd import workloads as W
from tests import gpu_helpers as G
from tests.test_gpu_block_calls import STD, _mask
from tests.test_gpu_ops import STAGED, _err, _ref

pytestmark = pytest.mark.gpu
LARGE = [(256, 256), (256, 192), (192, 192)]

# 1728 QKV columns, the Q part ending at 576: inside a 256-wide tile, on the edge of a 192-wide one
SHAPES = [
    W.ModelShape("one_stream", 1, 576, 8, 2, 23, 21, dtype="bf16", batch=2),
    W.ModelShape("two_streams", 1, 576, 8, 2, 19, 17, n_text=37, dual_stream=True, dtype="bf16", batch=2),
]


@pytest.mark.parametrize("tile", LARGE, ids=lambda t: f"{t[0]}x{t[1]}")
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
@pytest.mark.parametrize("form", ["resident", "y"])
def test_block_through_large_tiles_matches_oracle(tile, shape, form, monkeypatch):
    """Ragged rows per stream; the cached rows stay bit for bit (K/V cache) or are recomputed (Y cache, no Q columns)."""
    monkeypatch.setenv("MS_GEMM_TILE", f"{tile[0]}x{tile[1]}")
    ws = W.stack_weights(shape, 130, random_ln=True, std=STD)
    xt = W.template_hidden(shape, 130)
    yc = W.synthetic_y_cache(shape, 130)
    mask = _mask(shape, 0.6, 33)
    x = W.edited_hidden(shape, 130, xt, mask)
    if form == "y":
        cache = W.to_bf16_values(W.rng(130, 6, 0).standard_normal((1, shape.batch, shape.n_image, shape.d_model)))
        kv = oracle.kv_cache_of_inputs(cache, mask, ws, shape)
    else:
        cache = kv = np.stack([W.synthetic_kv_cache(shape, 130, 0)])
    _, snaps, rows = G.run_block_by_block(shape, mask, x, cache, yc, ws, form=form)
    G.check_blocks(shape, snaps, rows, lambda l, b: kv[l][b], ws, f"{shape.name} {tile} {form}",
                   loaded_exact=form == "resident")


@pytest.mark.parametrize("tile", LARGE, ids=lambda t: f"{t[0]}x{t[1]}")
def test_recompute_over_more_tiles_than_cus(tile, monkeypatch):
    """About 15600 unmasked rows x 1152 K/V columns: workgroups take several tiles each, every output row through the
    row table; rows of masked and text tokens keep what they held. Bound: the output's own rounding (2^-8 of the
    largest value covers it and one flip of the LayerNorm's)."""
    monkeypatch.setenv("MS_GEMM_TILE", f"{tile[0]}x{tile[1]}")
    shape = W.ModelShape("recompute", 1, 576, 8, 2, 64, 64, n_text=3, dtype="bf16", batch=4)
    B, T, N, d, nt = shape.batch, shape.n_tokens, shape.n_image, shape.d_model, shape.n_text
    w = G.dev_weights(W.stack_weights(shape, 131, random_ln=True, std=0.03), shape)[0]
    mask = _mask(shape, 0.05, 34)
    g = torch.Generator(device=G.DEV).manual_seed(131)
    yin = torch.randn(B, N, d, device=G.DEV, generator=g).bfloat16()
    kv = torch.full((B, T, 2, d), 7.0, device=G.DEV, dtype=torch.bfloat16)
    step = G.new_step(shape, mask)
    step.recompute_kv(0, w, yin, kv)
    torch.cuda.synchronize()
    step.close()
    a = F.layer_norm(yin.float(), (d,), w["ln1_g"].float(), w["ln1_b"].float(), shape.ln_eps).bfloat16().float()
    ref = torch.full((B, T, 2, d), 7.0, device=G.DEV)
    out = a.reshape(B * N, d) @ w["w_qkv"][d:].float().t().contiguous() + w["b_qkv"][d:].float()
    keep = torch.as_tensor(mask, device=G.DEV) != 0
    ref[:, nt:] = torch.where(keep[:, :, None, None], ref[:, nt:], out.reshape(B, N, 2, d))
    assert torch.equal(kv[:, :nt], ref[:, :nt].bfloat16())
    assert torch.equal(kv[:, nt:][keep], ref[:, nt:][keep].bfloat16())
    assert _err(kv, ref) <= 2 ** -8


@pytest.mark.parametrize("tile,stages", STAGED, ids=lambda v: f"{v[0]}x{v[1]}" if isinstance(v, tuple) else f"s{v}")
@pytest.mark.parametrize("epi", [MS.MS_EPI_BIAS, MS.MS_EPI_BIAS_GELU], ids=["bias", "gelu"])
def test_stage_variants_that_stage_bf16(tile, stages, epi, monkeypatch):
    """Outputs staged as bf16 in the stages' own LDS; widths that leave half a 16-byte store. Bound as in
    test_linear_region_pipeline_edges."""
    monkeypatch.setenv("MS_GEMM_STAGES", str(stages))
    g = torch.Generator(device=G.DEV).manual_seed(tile[0] + 2 * tile[1] + stages)
    M, N, K = 300, 516, 704
    A = torch.randn(M, K, device=G.DEV, generator=g).bfloat16()
    Wt = (torch.randn(N, K, device=G.DEV, generator=g) * 0.05).bfloat16()
    b = (torch.randn(N, device=G.DEV, generator=g) * 0.05).bfloat16()
    out = torch.full((M + 1, N), float("nan"), device=G.DEV, dtype=torch.bfloat16)
    MS.ms_linear(A, Wt, b, out[:M], epilogue=epi, tile=tile, ksplit=1)
    torch.cuda.synchronize()
    assert _err(out[:M], _ref(A, Wt, b, None, epi)) <= 2 ** -8
    assert bool(out[M].isnan().all())
