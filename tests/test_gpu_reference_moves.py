"""Logits that leave the reference of a row's exponentials behind, by little, by much and by more than the range of an
exponential, rising, falling and late in the row."""
import math

import numpy as np
import pytest

from oracle import sparse_attention
from oracle.attention import sparse_attention_lse
from tests.parity_utils import assert_parity, cut_rows, from_dev, to_dev, whole_rows
from workloads import f32_to_bf16_bits

pytestmark = pytest.mark.gpu

STEPS = {  # powers of two above the first keys, per sixteenth of the row
    "rising by 6": np.arange(16) * 6.0,
    "rising by 20": np.arange(16) * 20.0,
    "jumps of 50": np.array([0, 0, 50, 50, 0, 0, 100, 0, 90, 150, 150, 0, 0, 200, 0, 10]) * 1.0,
    "a jump of 300": np.array([0] * 9 + [300] + [0] * 5 + [290]) * 1.0,
    "falling": -np.arange(16) * 40.0,
    "late by 100": np.array([0] * 15 + [100]) * 1.0,
}


@pytest.mark.parametrize("D,bq,bk", [(128, 128, 128), (64, 128, 64), (128, 64, 64), (64, 64, 128), (128, 128, 96)])
@pytest.mark.parametrize("steps", list(STEPS))
@pytest.mark.parametrize("max_blocks", [None, 3])
def test_reference_moves(lib, D, bq, bk, steps, max_blocks):
    import torch

    print(f"reference D={D} {bq}x{bk} {steps} max_blocks={max_blocks}", flush=True)
    H, N = 2, 16 * bk - 21
    rng = np.random.default_rng(D + bq + bk)
    scale = 1 / math.sqrt(D)
    x = [(g * rng.standard_normal((1, H, N, D))).astype(np.float32) for g in (1.0, 1.0, 1.0)]
    x[0][..., 0] = np.where(np.arange(N) % 3 == 0, 4.0, 2.0)  # every third query moves twice as far
    x[1][..., 0] = (STEPS[steps] * math.log(2) / (4.0 * scale))[np.arange(N) // bk]
    q, k, v = (f32_to_bf16_bits(a) for a in x)
    nbq, nbk = -(-N // bq), 16
    mask = np.ones((H, nbq, nbk), np.uint8)
    mask[1, :, 1::3] = 0
    none = np.full((H, nbq), -1, np.int32)
    dp = lib.compile_pattern(mask, None, H, N, bq, bk).to_device(intervals=max_blocks is None)
    dp = whole_rows(dp) if max_blocks is None else cut_rows(dp, max_blocks)
    out = torch.full((1, H, N, D), math.nan, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, H, N), math.nan, dtype=torch.float32, device="cuda")
    lib.sparse_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, dp, scale, lse=lse)
    torch.cuda.synchronize()
    assert_parity(from_dev(out), sparse_attention(q, k, v, mask, none, scale, bq, bk))
    want = sparse_attention_lse(q, k, mask, none, scale, bq, bk)
    # fp32 logits of up to 300 carry an error of some 2^-24 of their size and of that of the products they are summed from
    assert np.abs(lse.cpu().numpy() - want).max() <= 5e-3


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("steps", list(STEPS))
@pytest.mark.parametrize("split", [False, True], ids=["whole", "split"])
def test_reference_moves_in_anchor_rows(lib, D, steps, split):
    import torch

    print(f"reference, anchor rows D={D} {steps} split={split}", flush=True)
    H, (F, Hs, Ws) = 2, (2, 20, 50)
    N = F * Hs * Ws
    rng = np.random.default_rng(D)
    scale = 1 / math.sqrt(D)
    x = [rng.standard_normal((1, H, N, D)).astype(np.float32) for _ in range(3)]
    x[0][..., 0] = np.where(np.arange(N) % 3 == 0, 4.0, 2.0)
    x[1][..., 0] = (STEPS[steps] * math.log(2) / (4.0 * scale))[np.arange(N) * 16 // N]
    q, k, v = (f32_to_bf16_bits(a) for a in x)
    amap = lib.anchor_map(N, F, Hs, Ws, Hs).to_device()  # every row is an anchor
    n_split, nbytes = lib.anchor_split_plan(1, N, D, H, amap.n_q)
    assert n_split > 1
    workspace = torch.full((nbytes // 4,), math.nan, dtype=torch.float32, device="cuda") if split else None
    out = torch.full((1, H, N, D), math.nan, dtype=torch.bfloat16, device="cuda")
    lib.anchor_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, torch.arange(H, dtype=torch.int32, device="cuda"), amap, scale,
                        workspace=workspace)
    torch.cuda.synchronize()
    mask, none = np.ones((H, 16, 16), np.uint8), np.full((H, 16), -1, np.int32)
    assert_parity(from_dev(out), sparse_attention(q, k, v, mask, none, scale, 128, 128))


def test_large_values_behind_a_move(lib):
    """Values so large that probabilities far above 2^8 would overflow their products."""
    import torch

    print("reference large values", flush=True)
    N, D, scale = 1024, 128, 0.1
    rng = np.random.default_rng(5)
    x = [rng.standard_normal((1, 1, N, D)).astype(np.float32) for _ in range(3)]
    x[0][..., 0] = 4.0
    x[1][..., 0] = np.where(np.arange(N) < 600, 0.0, 50 * math.log(2) / (4.0 * scale))
    x[2] *= np.float32(2.0 ** 100)
    q, k, v = (f32_to_bf16_bits(a) for a in x)
    mask, none = np.ones((1, 8, 8), np.uint8), np.full((1, 8), -1, np.int32)
    out = torch.empty((1, 1, N, D), dtype=torch.bfloat16, device="cuda")
    lib.sparse_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, lib.compile_pattern(mask, None, 1, N, 128, 128).to_device(), scale)
    torch.cuda.synchronize()
    want = sparse_attention(q, k, v, mask, none, scale, 128, 128)
    got = out.double().cpu().numpy()
    assert np.isfinite(got).all() and np.linalg.norm(got - want) / np.linalg.norm(want) < 8e-3
