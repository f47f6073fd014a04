"""The one-pass block energies where the call is large enough for workgroups of two query blocks, at ragged lengths
and odd numbers of query blocks, against fp64, and bit for bit against the form with one query block (a workspace of
one slice) and against one head alone; the form that a call takes is asserted.  Tolerance: fp32 sums of fp32
exponentials of logits below 64 (2^-18 in the exponent).  A second test has logits that outgrow the reference of the
exponentials late in a row: up to 2^8 in the exponent, sums of D products in fp32, so 2^-14 with a few ulps, and 2e-4
relative."""
import math

import pytest

pytestmark = pytest.mark.gpu


def _same_bits(a, b):
    import torch

    assert torch.equal(a.contiguous().view(torch.int32), b.contiguous().view(torch.int32))


def _workspaces(lib, B, H, N, D, bq, bk):
    """Workspaces of the recommended size, of one slice (one narrow workgroup) and of four times the recommended size,
    NaN-filled, after a look at the form that each gives."""
    import torch

    nbytes = lib.block_energy_workspace_bytes(N, bq, bk)
    sizes = nbytes, nbytes // 1024, 4 * nbytes
    one, two = lib.ENERGY_ONE_BLOCK, lib.ENERGY_ONE_BLOCK if (D, bq, bk) == (64, 128, 64) else lib.ENERGY_TWO_BLOCKS
    assert [lib.block_energy_onepass_form(B, H, N, D, bq, bk, n) for n in sizes] == [two, one, two]
    return [torch.full((n // 4,), float("nan"), device="cuda") for n in sizes]


def _energy64(q, k, bq, bk, scale):
    import torch

    N = q.shape[0]
    p = torch.softmax((q.double() @ k.double().T) * scale, 1)
    rows = torch.arange(N, device="cuda")
    e = torch.zeros(N, -(-N // bk), dtype=torch.float64, device="cuda").index_add_(1, rows // bk, p)
    e = torch.zeros(-(-N // bq), e.shape[1], dtype=torch.float64, device="cuda").index_add_(0, rows // bq, e)
    return e / torch.bincount(rows // bq)[:, None]


# 3800-4100 units of 256 queries: rounds of 512 workgroups, two per CU.  With blocks of 128, D = 64 and key blocks of 64
# the wide form is not built.
@pytest.mark.parametrize("N,H", [(129, 4096), (901, 1024), (4100, 225)])
@pytest.mark.parametrize("D,bq,bk", [(128, 128, 128), (128, 128, 64), (128, 64, 128), (128, 64, 64),
                                     (64, 128, 128), (64, 128, 64), (64, 64, 128), (64, 64, 64)])
def test_block_energy_wide_workgroups(lib, D, bq, bk, N, H):
    import torch

    print(f"energy panels D={D} bq={bq} bk={bk} N={N}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N + D + bq + bk)
    q, k = (torch.randn(1, H, N, D, device="cuda", generator=gen).mul_(1.5).to(torch.bfloat16) for _ in range(2))
    scale = -1 / math.sqrt(D) if N == 901 else 1 / math.sqrt(D)
    full, narrow, big = _workspaces(lib, 1, H, N, D, bq, bk)
    got = lib.block_energy(q, k, bq, bk, scale, workspace=full)
    for workspace in (full, narrow, big):
        _same_bits(got, lib.block_energy(q, k, bq, bk, scale, workspace=workspace))
    for h in (0, H // 2, H - 1):
        _same_bits(got[:, h:h + 1], lib.block_energy(q[:, h:h + 1].contiguous(), k[:, h:h + 1].contiguous(), bq, bk, scale,
                                                     workspace=full))
        torch.testing.assert_close(got[0, h].double(), _energy64(q[0, h], k[0, h], bq, bk, scale), rtol=2e-5, atol=1e-9)


# 576 units of 128 queries: one round of 512 workgroups and lone ones behind it
@pytest.mark.parametrize("N,H,bq", [(1100, 64, 128), (1024, 72, 128), (260, 192, 128), (1100, 64, 64), (140, 288, 64)])
@pytest.mark.parametrize("late", [0, 129])
def test_block_energy_overlapped(lib, N, H, bq, late):
    import torch

    print(f"energy overlapped N={N} H={H} bq={bq} late={late}", flush=True)
    D = bk = 128
    gen = torch.Generator(device="cuda").manual_seed(N + bq + late)
    q, k = (torch.randn(1, H, N, D, device="cuda", generator=gen) for _ in range(2))
    if late:
        q *= torch.tensor([0.05, 1.0, 6.0, 12.0], device="cuda")[torch.randint(0, 4, (1, H, N, 1), device="cuda",
                                                                               generator=gen)]
        k[:, :, :late] *= 0.2
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    scale = (2.5 if late else 1.5) / math.sqrt(D)
    nbytes = lib.block_energy_workspace_bytes(N, bq, bk)
    assert lib.block_energy_onepass_form(1, H, N, D, bq, bk, nbytes) == lib.ENERGY_OVERLAPPED
    assert lib.block_energy_onepass_form(1, H, N, D, bq, bk, nbytes // 1024) == lib.ENERGY_ONE_BLOCK
    full, narrow = (torch.full((n // 4,), float("nan"), device="cuda") for n in (nbytes, nbytes // 1024))
    got = lib.block_energy(q, k, bq, bk, scale, workspace=full)
    _same_bits(got, lib.block_energy(q, k, bq, bk, scale, workspace=narrow))
    _same_bits(got, lib.block_energy(q, k, bq, bk, scale, workspace=full))
    for h in (0, H - 1):
        torch.testing.assert_close(got[0, h].double(), _energy64(q[0, h], k[0, h], bq, bk, scale),
                                   rtol=2e-4 if late else 2e-5, atol=1e-9)


# the first key that outgrows the keys before it by more than the safe range: in the second tile, around the edges of
# tiles and sub-tiles, in the ragged last tile only
@pytest.mark.parametrize("N,late", [(700, 130), (700, 255), (700, 256), (700, 415), (675, 640), (675, 674)])
@pytest.mark.parametrize("D,bk", [(128, 128), (128, 64), (64, 128)])
def test_block_energy_late_large_logits(lib, D, bk, N, late):
    import torch

    print(f"energy late logits D={D} bk={bk} N={N} late={late}", flush=True)
    H = 1365  # x 3 units
    gen = torch.Generator(device="cuda").manual_seed(N + D + bk + late)
    q, k = (torch.randn(1, H, N, D, device="cuda", generator=gen) for _ in range(2))
    # rows of very different reach: some move their references more than once, others never, in either half of 64
    reach = torch.tensor([0.05, 1.0, 6.0, 12.0], device="cuda")[torch.randint(0, 4, (1, H, -(-N // 32), 1), device="cuda",
                                                                              generator=gen)]
    q *= reach.repeat_interleave(32, 2)[:, :, :N]
    k[:, :, :late] *= 0.2
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    scale = (-1 if late == 255 else 1) * 2.5 / math.sqrt(D)
    full, narrow, _ = _workspaces(lib, 1, H, N, D, 128, bk)
    got = lib.block_energy(q, k, 128, bk, scale, workspace=full)
    _same_bits(got, lib.block_energy(q, k, 128, bk, scale, workspace=narrow))
    for h in (0, 1, H - 1):
        torch.testing.assert_close(got[0, h].double(), _energy64(q[0, h], k[0, h], 128, bk, scale), rtol=2e-4, atol=1e-9)
