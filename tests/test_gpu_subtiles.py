"""The end of a row's stream of sub-tiles: rows of every small number of kept blocks (an odd or even number of
sub-tiles, a lone one), rows around the 64 cached columns, and a ragged last key block, against the oracle."""
import math

import numpy as np
import pytest

from oracle import sparse_attention
from tests.parity_utils import assert_parity, from_dev, to_dev, whole_rows
from workloads import f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,bq,bk", [(128, 128, 64), (64, 128, 64), (64, 64, 64), (128, 64, 64), (128, 128, 128),
                                     (128, 64, 128), (128, 128, 192), (128, 128, 96), (128, 128, 160)])
@pytest.mark.parametrize("intervals,rows", [(False, "whole"), (True, "whole"), (False, "one part"), (True, "one part"),
                                            (False, "planned")])
def test_every_short_row(lib, D, bq, bk, intervals, rows):
    import torch

    print(f"sub-tiles D={D} {bq}x{bk} intervals={intervals} {rows}", flush=True)
    counts = [0, 1, 2, 3, 4, 5, 6, 63, 64, 65, 66]
    nbk = 67
    N = nbk * bk - 29  # short last key block
    nbq = -(-N // bq)
    rng = np.random.default_rng(7 * D + bq + bk)
    q, k, v = (f32_to_bf16_bits((g * rng.standard_normal((1, 1, N, D))).astype(np.float32)) for g in (2.0, 2.0, 1.0))
    mask = np.zeros((1, nbq, nbk), np.uint8)
    for r in range(nbq):
        n = counts[r % len(counts)]
        if n == 0:
            continue
        cols = rng.choice(nbk - 1, size=n - 1, replace=False).tolist() + [nbk - 1] if r % 2 else rng.choice(
            nbk, size=n, replace=False)
        mask[0, r, cols] = 1
    assert set(mask[0].sum(1).tolist()) == set(counts)
    hp = lib.compile_pattern(mask, None, 1, N, bq, bk)
    dp = hp.to_device(intervals=intervals)
    if rows == "whole":
        whole_rows(dp)
    elif rows == "one part":
        dp._plan(True, 1000)
        assert set(dp._plans[1][1].cpu().numpy()[:, 2].tolist()) - {-1} == set(counts)
    out = torch.full((1, 1, N, D), math.nan, dtype=torch.bfloat16, device="cuda")
    lib.sparse_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, dp, 1 / math.sqrt(D))
    torch.cuda.synchronize()
    assert_parity(from_dev(out), sparse_attention(q, k, v, mask, np.full((1, nbq), -1, np.int32), 1 / math.sqrt(D), bq, bk))
