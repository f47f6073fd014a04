"""The forward with its rows cut along the keys against the oracle: every block shape, both list forms, cuts of every
size, and the state that its parts share."""
import math

import numpy as np
import pytest

from oracle import sparse_attention
from oracle.attention import sparse_attention_lse
from tests.parity_utils import assert_parity, assert_repeats_bitwise, from_dev, to_dev
from workloads import f32_to_bf16_bits, random_mask

pytestmark = pytest.mark.gpu


def _qkv(seed, B, H, N, D, gain=2.0):
    rng = np.random.default_rng(seed)
    return [f32_to_bf16_bits((g * rng.standard_normal((B, H, N, D))).astype(np.float32)) for g in (gain, gain, 1.0)]


def _pattern(lib, mask, repeat, H, N, bq, bk, max_blocks, intervals=False, **kw):
    dp = lib.compile_pattern(mask, repeat, H, N, bq, bk).to_device(intervals=intervals, **kw)
    dp._plan(True, max_blocks)
    assert dp._plans
    return dp


@pytest.mark.parametrize("D,bq,bk", [(128, 128, 128), (128, 128, 64), (128, 128, 96), (128, 128, 160), (128, 128, 192),
                                     (128, 64, 128), (128, 64, 64), (64, 128, 128), (64, 128, 64), (64, 64, 128),
                                     (64, 64, 64)])
@pytest.mark.parametrize("max_blocks,intervals", [(1, False), (2, True), (3, False), (4, True), (0, True)])
def test_cut_rows(lib, D, bq, bk, max_blocks, intervals):
    import torch

    print(f"split D={D} {bq}x{bk} max_blocks={max_blocks} intervals={intervals}", flush=True)
    B, H, N = 2, 2, 13 * bk - 37
    nbq, nbk = -(-N // bq), -(-N // bk)
    mask, repeat = random_mask(bk, H, nbq, nbk, 0.6, 0.2, tail_partial=N % bq != 0)
    mask[0, 1, :] = 0
    mask[1, 0, :] = 1
    scale = (-1 if max_blocks == 2 else 1) / math.sqrt(D)
    dp = _pattern(lib, mask, repeat, H, N, bq, bk, max_blocks, intervals)
    lse = torch.full((B, H, N), math.nan, dtype=torch.float32, device="cuda")
    out = torch.full((B, H, N, D), math.nan, dtype=torch.bfloat16, device="cuda")
    # Other inputs from call to call, whose workspaces the allocator puts in one place: parts that a call left would show in the
    # next one's result.  The third call has the bits of the first (the arrivals were re-armed).
    first = None
    for seed in (0, 1, 0):
        q, k, v = _qkv(D + bq + bk + seed, B, H, N, D)
        lib.sparse_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, dp, scale, lse=lse)
        torch.cuda.synchronize()
        got, got_lse = from_dev(out), lse.cpu().numpy()
        if seed == 0 and first is not None:
            assert (got == first).all()
            break
        first = got if first is None else first
        assert_parity(got, sparse_attention(q, k, v, mask, repeat, scale, bq, bk))
        assert_repeats_bitwise(got, repeat, bq, N)
        want_lse = sparse_attention_lse(q, k, mask, repeat, scale, bq, bk)
        kept = np.isfinite(want_lse)
        assert (np.isneginf(got_lse) == ~kept).all() and np.abs(got_lse[kept] - want_lse[kept]).max() <= 5e-3


def test_f16_strided_head_subset(lib):
    import torch

    print("split f16 strided head_map", flush=True)
    B, H, N, D = 1, 5, 1500, 128
    rng = np.random.default_rng(3)
    x = [torch.from_numpy((g * rng.standard_normal((B, N, H, D))).astype(np.float16)).cuda().transpose(1, 2)
         for g in (2.0, 2.0, 1.0)]
    heads = [4, 1]
    mask, repeat = random_mask(9, 2, 12, 12, 0.7, 0.2, tail_partial=True)
    out = torch.full((B, N, H, D), 7.0, dtype=torch.float16, device="cuda").transpose(1, 2)
    lib.sparse_attn_fwd(*x, out, _pattern(lib, mask, repeat, 2, N, 128, 128, 3, head_map=heads), 0.088)
    torch.cuda.synchronize()
    s = torch.einsum("bhqd,bhkd->bhqk", x[0][:, heads].double().cpu(), x[1][:, heads].double().cpu()) * 0.088
    t = torch.arange(N) // 128
    see = torch.from_numpy(mask).bool()[:, t][:, :, t]
    p = torch.softmax(s[0].masked_fill(~see, -math.inf), -1).nan_to_num(0.0)
    want = p @ x[2][0, heads].double().cpu()
    for h in range(2):
        for r in range(12):
            if repeat[h, r] >= 0:
                n = min(128, N - 128 * r)
                want[h, 128 * r:128 * r + n] = want[h, 128 * repeat[h, r]:128 * repeat[h, r] + n]
    got = out[0, heads].double().cpu()
    assert (got - want).abs().max() <= 2e-2 and (got - want).norm() / want.norm() <= 1.2e-3
    assert (out[:, [0, 2, 3]] == 7.0).all()


def test_parts_without_mass(lib):
    """Keys whose logits are -inf, over whole parts and at the start of a row, have no weight."""
    import torch

    print("split parts at -inf", flush=True)
    N, D = 1280, 128
    q, k, v = _qkv(11, 1, 1, N, D)
    q[..., 0] = f32_to_bf16_bits(np.full(1, 3.0, np.float32))
    low = np.isin(np.arange(N) // 128, [0, 1, 4, 5, 9])
    k[0, 0, low, 0] = f32_to_bf16_bits(np.full(1, -3e38, np.float32))
    mask = np.ones((1, 10, 10), np.uint8)
    none = np.full((1, 10), -1, np.int32)
    for max_blocks in (1, 2, 1000):
        out = torch.empty((1, 1, N, D), dtype=torch.bfloat16, device="cuda")
        lib.sparse_attn_fwd(to_dev(q), to_dev(k), to_dev(v), out, _pattern(lib, mask, none, 1, N, 128, 128, max_blocks), 0.1)
        torch.cuda.synchronize()
        mask2 = mask.copy()
        mask2[:, :, [0, 1, 4, 5, 9]] = 0
        assert_parity(from_dev(out), sparse_attention(q, k, v, mask2, none, 0.1, 128, 128))


def test_streams_and_graphs(lib):
    """Calls on more streams than there are spare arrivals, and a captured call beside eager ones, give one result."""
    import torch

    print("split streams and graph", flush=True)
    H, N, D = 4, 2000, 128
    q, k, v = (to_dev(x) for x in _qkv(13, 1, H, N, D))
    mask, repeat = random_mask(14, H, 16, 16, 0.6, 0.2, keep_diagonal=True, tail_partial=True)
    dp = _pattern(lib, mask, repeat, H, N, 128, 128, 2)
    want = torch.empty_like(q)
    lib.sparse_attn_fwd(q, k, v, want, dp, 0.088)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(10)]
    outs = [torch.zeros_like(q) for _ in streams]
    torch.cuda.synchronize()
    for _ in range(5):
        for s, o in zip(streams, outs):
            with torch.cuda.stream(s):
                lib.sparse_attn_fwd(q, k, v, o, dp, 0.088)
    torch.cuda.synchronize()
    assert all(torch.equal(o.view(torch.int16), want.view(torch.int16)) for o in outs)
    captured, eager = torch.zeros_like(q), torch.zeros_like(q)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=streams[0]):
        lib.sparse_attn_fwd(q, k, v, captured, dp, 0.088)
        lib.sparse_attn_fwd(q, k, v, captured, dp, 0.088)
    for _ in range(4):
        captured.zero_()
        eager.zero_()
        torch.cuda.synchronize()
        graph.replay()
        with torch.cuda.stream(streams[0]):
            lib.sparse_attn_fwd(q, k, v, eager, dp, 0.088)
        torch.cuda.synchronize()
        assert torch.equal(captured.view(torch.int16), want.view(torch.int16))
        assert torch.equal(eager.view(torch.int16), want.view(torch.int16))


def test_no_memory_for_the_workspace(lib):
    """A call whose workspace cannot be had runs with whole rows; one that has gone wrong otherwise says so as without a
    plan."""
    import torch

    from paper_2603_05503_amd.binding import CalibattError

    print("split without memory", flush=True)
    H, N, D = 4, 2000, 128
    q, k, v = (to_dev(x) for x in _qkv(15, 1, H, N, D))
    mask, repeat = random_mask(16, H, 16, 16, 0.6, 0.2, keep_diagonal=True, tail_partial=True)
    hp = lib.compile_pattern(mask, repeat, H, N, 128, 128)
    want, out = torch.empty_like(q), torch.empty_like(q)
    lib.sparse_attn_fwd(q, k, v, want, hp.to_device(persistent=False), 0.088)
    dp = _pattern(lib, mask, repeat, H, N, 128, 128, 2)
    assert dp._plans[1][0].n_slots * 67584 > 4 << 20  # more than what the allocator's small blocks could hold
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)
        held = []
        with pytest.raises(torch.OutOfMemoryError):  # take what is left of the blocks that the allocator has
            for _ in range(1000):
                held.append(torch.empty(1 << 20, dtype=torch.float32, device="cuda"))
        lib.sparse_attn_fwd(q, k, v, out, dp, 0.088)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))
    for block_q in (-128, 64, 1 << 30):
        with pytest.raises(CalibattError):
            lib.sparse_attn_fwd(q, k, v, out, dp, 0.088, block_q=block_q)
