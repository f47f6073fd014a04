"""The grouped call of the spatial similarity (tokens that share their partner computed together) against the form that
takes one token per lane: the same bits, for every way the tokens can fall into groups of three, of two, and pairs."""
import ctypes as C
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _partner(kind, lib, rows, cols, rng):
    n = rows * cols
    if kind.startswith("anchors"):
        return lib.anchor_partner(1, rows, cols, int(kind[7:]))
    if kind == "self":
        return np.arange(n, dtype=np.int32)
    if kind == "random":
        return rng.integers(0, n, n).astype(np.int32)
    if kind == "few":  # short runs, some of them their own partner, some with a partner outside the run
        return (rng.integers(0, 3, n) * (n // 3)).astype(np.int32)
    if kind == "one":
        return np.full(n, n // 2, np.int32)
    if kind.startswith("period"):  # of p rows the first p - 1 have the first one as their partner, the last is its own
        p, row = int(kind[6:]), np.arange(n) // cols
        return (np.arange(n) - np.where(row % p == p - 1, 0, row % p * cols)).astype(np.int32)
    if kind.startswith("runs"):  # runs of these lengths, with a partner inside, in another column or outside [0, n)
        out = np.empty((rows, cols), np.int32)
        for x in range(cols):
            y = 0
            while y < rows:
                length = int(rng.choice([int(c) for c in kind[4:]]))
                inside = (y + int(rng.integers(min(length, rows - y)))) * cols + x
                out[y:y + length, x] = rng.choice([inside, rng.integers(n), n + 2])
                y += length
        return out.reshape(-1)
    assert kind == "wild"  # clamped to [0, N)
    return rng.choice(np.array([-5, 0, n - 1, n + 3, 1 << 30], np.int32), n).astype(np.int32)


# heads, rows, cols, text tokens, D, partner map, tokens per group in the form that the device chooses (1: pairs)
CASES = [
    (1, 1, 1, 0, 64, "self", 1),
    (2, 7, 5, 3, 128, "anchors2", 1),
    (300, 9, 43, 0, 128, "self", 3),
    (300, 9, 43, 2, 64, "self", 3),
    (200, 64, 11, 1, 64, "one", 3),
    (300, 130, 3, 7, 128, "anchors1", 2),  # runs longer than a segment of 64 rows
    (256, 130, 5, 0, 64, "anchors1", 3),
    (300, 13, 31, 64, 128, "random", 1),
    (300, 13, 31, 0, 64, "few", 1),
    (300, 6, 70, 11, 64, "wild", 1),
    (300, 24, 16, 5, 128, "anchors1", 3),
    (300, 24, 16, 0, 64, "anchors1", 3),
    (300, 25, 16, 0, 128, "one", 2),
    (100, 47, 33, 3, 128, "runs123456789", 2),
    (256, 47, 33, 0, 64, "runs3369", 3),
    (256, 47, 33, 3, 128, "runs34569", 3),
    (100, 47, 33, 3, 128, "runs24", 2),
    (100, 47, 33, 0, 64, "runs24", 2),
    (100, 50, 33, 0, 128, "period5", 3),  # groups of three and lone tokens
    (100, 49, 33, 1, 64, "period5", 3),
    (256, 49, 33, 1, 128, "period4", 2),  # groups of two and lone tokens
    (256, 48, 33, 0, 64, "period4", 2),
]


def _form(lists, H, n, cus):
    """Tokens per group in the form that the device takes, from the numbers of groups that it left behind."""
    n2, n3, lone = np.frombuffer(lists[:12].cpu().numpy().tobytes(), np.int32).tolist()

    def up(a, b):
        return -(-a // b)

    def rows(groups, lanes, queries):
        return up(up(H * (up(groups, 128) + up(up(lone, lanes), 128)), 8), cus) * queries

    rows1, rows2, rows3 = up(up(H * up(n, 128), 8), cus) * 2, rows(n2, 3, 3), rows(n3, 4, 4)
    return 1 if rows1 < min(rows2, rows3) else 2 if rows2 <= rows3 else 3


@pytest.mark.parametrize("H,rows,cols,text,D,kind,form", CASES)
def test_grouped_matches_single_tokens(lib, H, rows, cols, text, D, kind, form):
    import torch

    print(f"grouped similarity H={H} rows={rows} cols={cols} text={text} D={D} {kind}", flush=True)
    raw = lib.load_library()
    rng = np.random.default_rng(rows * cols + D)
    n, N = rows * cols, rows * cols + text
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k = (torch.randn(1, H, N, D, device="cuda", generator=gen).mul_(2.0).to(torch.bfloat16) for _ in range(2))
    partner = torch.from_numpy(_partner(kind, lib, rows, cols, rng)).cuda()
    out = []
    for lists in (None, torch.full((36 * n + 16,), 0x5A, dtype=torch.uint8, device="cuda")):
        triples = torch.full((1, H, n, 3), float("nan"), device="cuda")
        score = torch.full((1, H), float("nan"), device="cuda")
        st = raw.calibatt_spatial_similarity_grouped(
            q.data_ptr(), k.data_ptr(), 1, H, N, D, partner.data_ptr(), n, cols, 1 / math.sqrt(D), triples.data_ptr(),
            None if lists is None else lists.data_ptr(), 0 if lists is None else lists.numel(), score.data_ptr(),
            C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        torch.cuda.synchronize()
        out.append((triples, score))
    assert _form(lists, H, n, torch.cuda.get_device_properties(0).multi_processor_count // 8) == form
    assert bool(torch.isfinite(out[0][0]).all())
    assert torch.equal(out[0][0].view(torch.int32), out[1][0].view(torch.int32))
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))
    # the single-token form against fp64 (tolerance of sums of probabilities whose logits carry fp32 rounding)
    p = torch.softmax((q[0, -1].double() @ k[0, -1].double().T) / math.sqrt(D), 1)
    a = partner.clamp(0, N - 1).long()
    want = torch.stack([(p[:n] * p[a]).sum(1), (p[:n] ** 2).sum(1), (p[a] ** 2).sum(1)], 1)
    torch.testing.assert_close(out[0][0][0, -1].double(), want, rtol=1e-3, atol=1e-9)


def _both_forms(lib, q, k, partner, cols, scale):
    """Triples of the form without and with groups, which have the same bits."""
    import torch

    raw = lib.load_library()
    _, H, N, D = q.shape
    n = partner.numel()
    out = []
    for nbytes in (0, 36 * n + 16):
        lists = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
        triples = torch.full((1, H, n, 3), float("nan"), device="cuda")
        score = torch.empty((1, H), device="cuda")
        st = raw.calibatt_spatial_similarity_grouped(
            q.data_ptr(), k.data_ptr(), 1, H, N, D, partner.data_ptr(), n, cols, scale, triples.data_ptr(),
            lists.data_ptr() if nbytes else None, nbytes, score.data_ptr(),
            C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        torch.cuda.synchronize()
        out.append(triples)
    assert torch.equal(out[0].view(torch.int32), out[1].view(torch.int32))
    return out[0][0]


def _triples64(q, k, partner, scale):
    import torch

    a = partner.long()
    p = [torch.softmax((q[0, h].double() @ k[0, h].double().T) * scale, 1)[:a.numel()] for h in range(q.shape[1])]
    return torch.stack([torch.stack([(x * x[a]).sum(1), (x ** 2).sum(1), (x[a] ** 2).sum(1)], 1) for x in p])


@pytest.mark.parametrize("D", [64, 128])
def test_late_large_logits(lib, D):
    """Logits that are exact in fp32 and whose first 64 keys lie some 40 powers of two below the rest.  Relative error of
    the sums, rms: 2.6e-7 (D = 128) with sums relative to the true maximum and one addition after the other, which the
    sums here stay below; an argument of an exponential that is 32 too large alone adds a rounding of 2^-20 / sqrt(3)."""
    import torch

    print(f"similarity late logits D={D}", flush=True)
    H, N, cols = 4, 2048, 32
    gen = torch.Generator(device="cuda").manual_seed(N + D)
    q, k = (torch.randint(-3, 4, (1, H, N, D), device="cuda", generator=gen).float() for _ in range(2))
    q[..., 0] = 4.0
    k[..., 0] = torch.where(torch.arange(N, device="cuda") < 64, -72.0 if D == 128 else -50.0, 0.0)
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    partner = torch.from_numpy(lib.anchor_partner(2, 32, cols, 5)).cuda()
    got, want = _both_forms(lib, q, k, partner, cols, 1 / math.sqrt(D)), _triples64(q, k, partner, 1 / math.sqrt(D))
    assert float((got.double() / want - 1).pow(2).mean().sqrt()) < 3e-7


@pytest.mark.parametrize("n_out", [32, 40, 64, 200])
@pytest.mark.parametrize("D", [64, 128])
def test_first_keys_at_minus_infinity(lib, D, n_out):
    """The logits of the first keys overflow to -inf: they have no mass, like keys that are not there."""
    import torch

    print(f"similarity -inf D={D} n_out={n_out}", flush=True)
    H, N, cols = 2, 333, 37
    gen = torch.Generator(device="cuda").manual_seed(N + D)
    q, k = (torch.randn(1, H, N, D, device="cuda", generator=gen) for _ in range(2))
    q[..., 0] = 2.0 ** 70
    k[..., 0] = 0.0
    k[:, :, :n_out, 0] = -2.0 ** 70
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    partner = torch.from_numpy(lib.anchor_partner(1, 9, cols, 2)).cuda()
    got, want = _both_forms(lib, q, k, partner, cols, 1 / math.sqrt(D)), _triples64(q, k, partner, 1 / math.sqrt(D))
    torch.testing.assert_close(got.double(), want, rtol=1e-4, atol=1e-12)


def test_grouped_refuses_what_does_not_fit(lib):
    import torch

    raw = lib.load_library()
    one = C.c_void_p(16)
    f = raw.calibatt_spatial_similarity_grouped
    assert f(one, one, 1, 1, 8, 64, one, 8, 2, 1.0, one, C.c_void_p(8), 1000, one, None) == -2
    assert f(one, one, 1, 1, 8, 64, one, 8, 2, 1.0, one, one, -1, one, None) == -2
    assert f(one, one, 1, 1, 8, 64, one, 8, 2, 1.0, one, one, 36 * 8 + 15, one, None) == -7
    n = C.c_int64(0)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for H, n_tok, want in ((1, 8, 0), (2 * cus, 100, 0), (2 * cus + 1, 100, 0), (2 * cus, 512, 0), (2 * cus, 513, 18484),
                           (2, 128 * cus, 0), (2, 128 * cus + 1, 36 * (128 * cus + 1) + 16)):
        assert raw.calibatt_similarity_lists_bytes(1, H, n_tok, C.byref(n)) == 0 and n.value == want


def test_temporaries_belong_to_the_stream_of_the_call(lib):
    """What the binding allocates for a call on another stream comes from that stream's memory: a block of the current
    stream may still be in use by earlier work there."""
    import torch

    n, cols, H, D = 65536, 256, 2, 64
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k = (torch.randn(1, H, n, D, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    partner = torch.from_numpy(lib.anchor_partner(2, n // 2 // cols, cols, 9)).cuda()
    triples = torch.empty((1, H, n, 3), device="cuda")
    nbytes = C.c_int64(0)
    assert lib.load_library().calibatt_similarity_lists_bytes(1, H, n, C.byref(nbytes)) == 0 and nbytes.value > 1 << 21
    want = lib.spatial_similarity(q, k, partner, cols, 0.1, workspace=triples)
    want_triples = triples.clone()
    torch.cuda.synchronize()
    q2, k2 = (x[:, :, :512].contiguous() for x in (q, k))
    side = torch.cuda.Stream()
    triples.fill_(0)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()

    def segments():
        return [s for s in torch.cuda.memory_snapshot() if s["stream"] == side.cuda_stream]

    before = sum(s["total_size"] for s in segments())
    score = lib.spatial_similarity(q, k, partner, cols, 0.1, workspace=triples, stream=side.cuda_stream)
    assert sum(s["total_size"] for s in segments()) - before >= nbytes.value  # the lists: more than a segment of small blocks
    energy = lib.block_energy(q2, k2, 128, 128, 0.1, stream=side.cuda_stream)
    mask = lib.select_blocks_device(energy, 0.9, stream=side.cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(score, want) and torch.equal(triples, want_triples)
    for t in (score, energy, mask):
        assert any(s["address"] <= t.data_ptr() < s["address"] + s["total_size"] for s in segments())


@pytest.mark.parametrize("D", [64, 128])
def test_long_runs_are_cut(lib, D):
    """Runs of up to 64 rows stay whole wherever they lie; longer ones, whose tokens would walk past all of their rows, end
    at every 64th row."""
    import torch

    print(f"grouped similarity: long runs D={D}", flush=True)
    raw = lib.load_library()
    lengths = [64, 65, 63, 3, 200, 1, 64, 66, 129, 30, 64, 1, 2, 128, 70]
    rows, cols, H = sum(lengths), 7, 1
    n = rows * cols
    N = n + len(lengths)
    rng = np.random.default_rng(8)
    partner, want = np.empty((rows, cols), np.int64), np.zeros(3, np.int64)
    for x in range(cols):
        y = 0
        for i in rng.permutation(len(lengths)):
            end = y + lengths[i]
            kind = rng.integers(3)  # the partner is a token of the run, a token of another column or one behind the grid
            row = int(rng.integers(y, end)) if kind == 0 else -1
            partner[y:end, x] = row * cols + x if kind == 0 else y * cols + (x + 1) % cols if kind == 1 else n + i
            cuts = [y] + ([c for c in range(y + 1, end) if c % 64 == 0] if end - y > 64 else []) + [end]
            for lo, hi in zip(cuts, cuts[1:]):
                inside = lo <= row < hi
                tokens = hi - lo - inside
                want += [-(-tokens // 2), -(-tokens // 3), inside and tokens == 0]
            y = end
    partner = torch.from_numpy(partner.reshape(-1).astype(np.int32)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k = (torch.randn(1, H, N, D, device="cuda", generator=gen).mul_(2.0).to(torch.bfloat16) for _ in range(2))
    out = []
    for lists in (None, torch.full((36 * n + 16,), 0x5A, dtype=torch.uint8, device="cuda")):
        triples = torch.full((1, H, n, 3), float("nan"), device="cuda")
        score = torch.full((1, H), float("nan"), device="cuda")
        assert raw.calibatt_spatial_similarity_grouped(
            q.data_ptr(), k.data_ptr(), 1, H, N, D, partner.data_ptr(), n, cols, 1 / math.sqrt(D), triples.data_ptr(),
            None if lists is None else lists.data_ptr(), 0 if lists is None else lists.numel(), score.data_ptr(),
            C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        torch.cuda.synchronize()
        out.append((triples, score))
    assert np.frombuffer(lists[:12].cpu().numpy().tobytes(), np.int32).tolist() == want.tolist()
    assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(*out))
