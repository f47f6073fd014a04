"""The mixed groups of the spatial similarity (threes and, at the end of a run, twos): the bits of the form that takes one
token per lane, for runs of every length that it cuts, partners inside and outside of them, and lone tokens beside them."""
import ctypes as C
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _partner(kind, frames, rows, cols):
    """Anchor rows of the library's map, or runs of the given lengths whose partner is their first, last or no token."""
    f, y, x = (a.reshape(-1) for a in np.meshgrid(np.arange(frames), np.arange(rows), np.arange(cols), indexing="ij"))
    period = int(kind[1:])
    start = y // period * period
    last = np.minimum(start + period, rows) - 1
    row = {"f": start, "l": last, "o": (start + rows // 2) % rows}[kind[0]]
    return ((f * rows + row) * cols + (x if kind[0] != "o" else (x + 1) % cols)).astype(np.int32)


def _mixed(lists, H, n, cus):
    words = np.frombuffer(lists.cpu().numpy().tobytes(), np.int32)
    n2, n3, lone, m3 = words[:4].tolist()
    m2 = int(words[3 + 9 * n]) if lone < n else 0

    def up(a, b):
        return -(-a // b)

    def rows(groups, lanes):
        return up(up(H * (up(groups, 128) + up(up(lone, lanes), 128)), 8), cus) * lanes

    u3, u2, u1 = up(m3, 128), up(m2, 128), up(up(lone, 4), 128)
    least = min(up(up(H * up(n, 128), 8), cus) * 2, rows(n2, 3), rows(n3, 4))
    units = u3 + u2 + u1
    mine = up(up(H * units, 8), cus) * (46 * (u3 + u1) + 30 * u2)
    return m3 > 0 and m2 > 0 and units <= up(n, 128) + 1 and mine * 10 < 96 * units * least


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kind,frames,rows,cols,mixed", [
    ("l6", 3, 29, 41, True), ("o5", 4, 40, 40, True), ("f6", 4, 30, 40, False), ("f8", 3, 40, 40, False),
    ("a5", 18, 30, 32, None), ("f9", 4, 46, 40, None), ("o8", 3, 64, 33, None),
    ("f6", 1, 1100, 5, None),  # many runs in a column
    ("f2", 4, 30, 40, False),  # runs of one token
])
def test_mixed_groups(lib, D, kind, frames, rows, cols, mixed):
    import torch

    print(f"mixed similarity D={D} {kind} {frames}x{rows}x{cols}", flush=True)
    raw = lib.load_library()
    H, n = 224, frames * rows * cols
    N = n + 37
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k = (torch.randn(1, H, N, D, device="cuda", generator=gen).mul_(2.0).to(torch.bfloat16) for _ in range(2))
    partner = lib.anchor_partner(frames, rows, cols, 5) if kind == "a5" else _partner(kind, frames, rows, cols)
    partner = torch.from_numpy(partner).cuda()
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
    took = _mixed(lists, H, n, torch.cuda.get_device_properties(0).multi_processor_count // 8)
    print("mixed", took, flush=True)
    assert mixed is None or took == mixed
    for a, b in zip(*out):
        assert bool(torch.isfinite(a).all()) and torch.equal(a.view(torch.int32), b.view(torch.int32))
