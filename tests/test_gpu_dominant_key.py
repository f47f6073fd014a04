"""The largest probability of a row is exact where the exponentials' reference is (or has just moved to) its logit: a row
that two keys share alike keeps no rounding but the one of the smaller key's probability."""
import math

import numpy as np
import pytest

from tests.parity_utils import bits_to_f64, cut_rows, from_dev, to_dev, whole_rows
from workloads import f32_to_bf16_bits

pytestmark = pytest.mark.gpu

# Key A has weight 1, key B 2^-x with x in (0, 0.2), all others less than 2^-30; the values are 1, -1 and 0, so a row is
# (1 - w) / (1 + w).  bf16 rounds w, in (0.87, 1), by 2^-9 at most, which moves the row by 2 / (1 + w)^2 <= 0.572 of that;
# the row itself, below 0.0693, is rounded by 2^-13 * 2 at most.  1e-5: fp32 logits of some 40.
BOUND = 0.572 * 2.0 ** -9 + 2.0 ** -12 + 1e-5


def two_keys(D, N, a, b, seed):
    """q, k, v bits [1, 1, N, D], scale and the rows: logits (powers of two) of 4 to 8 at key a, up to 0.2 less at key b, -30
    elsewhere, in every phase."""
    rng = np.random.default_rng(seed)
    q, k, v = (np.zeros((1, 1, N, D), np.float32) for _ in range(3))
    q[0, 0, :, 0] = 4 + rng.integers(0, 128, N) / 32   # exact in bf16
    q[0, 0, :, 1] = rng.integers(0, 128, N) / 4096
    q[0, 0, :, 2] = -(1 + rng.integers(0, 100, N)) / 512
    q[0, 0, :, 3] = 1
    k[0, 0, :, 3] = -30
    k[0, 0, [a, b], 0] = k[0, 0, [a, b], 1] = 1
    k[0, 0, [a, b], 3] = 0
    k[0, 0, b, 2] = 1
    v[0, 0, a], v[0, 0, b] = 1, -1
    w = np.exp2(q[0, 0, :, 2].astype(np.float64))
    return [f32_to_bf16_bits(x) for x in (q, k, v)], math.log(2), ((1 - w) / (1 + w))[:, None]


@pytest.mark.parametrize("split", [False, True], ids=["whole", "split"])
@pytest.mark.parametrize("D", [64, 128])
def test_anchor_rows(lib, D, split):
    import torch

    print(f"dominant key, anchor rows D={D} split={split}", flush=True)
    F, Hs, Ws = 2, 20, 40
    N = F * Hs * Ws
    (q, k, v), scale, want = two_keys(D, N, 300, 1100, 3)
    amap = lib.anchor_map(N, F, Hs, Ws, Hs).to_device()  # every row is an anchor
    n_split, nbytes = lib.anchor_split_plan(1, N, D, 1, amap.n_q)
    assert n_split > 1
    workspace = torch.full((nbytes // 4,), math.nan, dtype=torch.float32, device="cuda") if split else None
    out = torch.full((1, 1, N, D), math.nan, dtype=torch.bfloat16, device="cuda")
    lib.anchor_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, torch.zeros(1, dtype=torch.int32, device="cuda"), amap, scale,
                        workspace=workspace)
    torch.cuda.synchronize()
    err = np.abs(bits_to_f64(from_dev(out))[0, 0] - want).max()
    print(f"  largest error {err:.3e}, bound {BOUND:.3e}", flush=True)
    assert err <= BOUND


@pytest.mark.parametrize("split", [False, True], ids=["whole", "split"])
@pytest.mark.parametrize("D", [64, 128])
def test_anchor_rows_behind_keys_without_mass(lib, D, split):
    """Leading keys whose logits are -inf have no weight."""
    import torch
    from oracle.anchor import dense_rows
    from oracle import bf16_bits_to_f64

    print(f"anchor rows behind -inf D={D} split={split}", flush=True)
    F, Hs, Ws = 2, 20, 40
    N, first = F * Hs * Ws, 700
    rng = np.random.default_rng(4)
    x = [rng.standard_normal((1, 1, N, D)).astype(np.float32) for _ in range(3)]
    x[0][..., 0] = 3.0
    x[1][0, 0, :first, 0] = -3e38
    q, k, v = (f32_to_bf16_bits(a) for a in x)
    amap = lib.anchor_map(N, F, Hs, Ws, Hs).to_device()
    n_split, nbytes = lib.anchor_split_plan(1, N, D, 1, amap.n_q)
    workspace = torch.full((nbytes // 4,), math.nan, dtype=torch.float32, device="cuda") if split else None
    out = torch.full((1, 1, N, D), math.nan, dtype=torch.bfloat16, device="cuda")
    lib.anchor_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, torch.zeros(1, dtype=torch.int32, device="cuda"), amap, 1.0,
                        workspace=workspace)
    torch.cuda.synchronize()
    qf, kf, vf = (bf16_bits_to_f64(a[0, 0]) for a in (q, k, v))
    want = dense_rows(qf, kf[first:], vf[first:], 1.0)
    got = bits_to_f64(from_dev(out))[0, 0]
    assert np.isfinite(got).all() and np.abs(got - want).max() <= 2e-2 and np.linalg.norm(got - want) <= 8e-3 * np.linalg.norm(want)


@pytest.mark.parametrize("D,bq,bk", [(128, 128, 128), (128, 128, 192), (128, 128, 96), (128, 64, 64), (64, 128, 64), (64, 64, 128)])
@pytest.mark.parametrize("max_blocks", [None, 2])
def test_sparse_rows(lib, D, bq, bk, max_blocks):
    import torch

    print(f"dominant key, sparse rows D={D} {bq}x{bk} max_blocks={max_blocks}", flush=True)
    N = 1600
    (q, k, v), scale, want = two_keys(D, N, 700, 1100, 5)
    nbq, nbk = -(-N // bq), -(-N // bk)
    dp = lib.compile_pattern(np.ones((1, nbq, nbk), np.uint8), None, 1, N, bq, bk).to_device(intervals=True)
    dp = whole_rows(dp) if max_blocks is None else cut_rows(dp, max_blocks)
    out = torch.full((1, 1, N, D), math.nan, dtype=torch.bfloat16, device="cuda")
    lib.sparse_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, dp, scale)
    torch.cuda.synchronize()
    err = np.abs(bits_to_f64(from_dev(out))[0, 0] - want).max()
    print(f"  largest error {err:.3e}, bound {BOUND:.3e}", flush=True)
    assert err <= BOUND
