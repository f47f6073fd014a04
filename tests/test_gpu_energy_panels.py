"""The one-pass block energies where the call is large enough for workgroups of 256 queries, at ragged lengths and
odd numbers of query blocks, against fp64 and against the same call with a workspace that only the 128-query form
(or the 64-query one) fits.  Tolerance: fp32 sums of fp32 exponentials of logits below 64 (2^-18 in the exponent)."""
import math

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [129, 640, 901])
@pytest.mark.parametrize("D,bq,bk", [(128, 128, 128), (128, 128, 64), (128, 64, 128), (128, 64, 64),
                                     (64, 128, 128), (64, 128, 64), (64, 64, 128), (64, 64, 64)])
def test_block_energy_wide_workgroups(lib, D, bq, bk, N):
    import torch

    print(f"energy panels D={D} bq={bq} bk={bk} N={N}", flush=True)
    H = 4200 // -(-N // 256)  # 256-query units: more than twice the workgroups of a 256-CU device at four per CU
    gen = torch.Generator(device="cuda").manual_seed(N + D + bq + bk)
    q, k = (torch.randn(1, H, N, D, device="cuda", generator=gen).mul_(1.5).to(torch.bfloat16) for _ in range(2))
    scale = -1 / math.sqrt(D) if N == 640 else 1 / math.sqrt(D)
    nbytes = lib.block_energy_workspace_bytes(N, bq, bk)
    full, small = (torch.full((b // 4,), float("nan"), device="cuda") for b in (nbytes, nbytes // 1024 * 300))
    got = lib.block_energy(q, k, bq, bk, scale, workspace=full)
    again = lib.block_energy(q, k, bq, bk, scale, workspace=full)
    narrow = lib.block_energy(q, k, bq, bk, scale, workspace=small)
    torch.cuda.synchronize()
    assert torch.equal(got, again)
    torch.testing.assert_close(got, narrow, rtol=2e-5, atol=1e-9)
    for h in (0, H // 2, H - 1):
        p = torch.softmax((q[0, h].double() @ k[0, h].double().T) * scale, 1)
        rows = torch.arange(N, device="cuda")
        e = torch.zeros(N, -(-N // bk), dtype=torch.float64, device="cuda").index_add_(1, rows // bk, p)
        e = torch.zeros(-(-N // bq), e.shape[1], dtype=torch.float64, device="cuda").index_add_(0, rows // bq, e)
        e /= torch.bincount(rows // bq)[:, None]
        torch.testing.assert_close(got[0, h].double(), e, rtol=2e-5, atol=1e-9)
