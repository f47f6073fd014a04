"""The plan of a split forward: every kept block of every computed row in exactly one part, in order."""
import ctypes as C

import numpy as np
import pytest

from paper_2603_05503_amd import binding
from workloads import random_mask


def _records(plan):
    split, parts = plan
    assert parts.shape == (split.n_parts, 12) and split.n_parts % 8 == 0
    live = parts[parts[:, 0] >= 0]
    assert (parts[parts[:, 0] < 0] == -1).all()
    return split, live


@pytest.mark.parametrize("H,N,bq,bk,density,order", [(1, 1, 128, 128, 1.0, 4), (3, 1000, 64, 64, 0.4, 1), (2, 5000, 128, 96, 0.7, 4),
                                                     (9, 3000, 128, 192, 0.2, 3), (5, 4000, 64, 128, 1.0, 0)])
@pytest.mark.parametrize("max_blocks", [0, 1, 2, 3, 7, 1000])
@pytest.mark.parametrize("intervals", [False, True])
def test_parts_cover_every_row(lib, H, N, bq, bk, density, order, max_blocks, intervals):
    nbq, nbk = -(-N // bq), -(-N // bk)
    mask, repeat = random_mask(N + bk, H, nbq, nbk, density, 0.2 if nbq > 3 else 0.0, tail_partial=N % bq != 0)
    mask[0, nbq // 2, :] = 0  # an empty row
    hp = lib.compile_pattern(mask, repeat, H, N, bq, bk, order)
    iv_ptr = hp.encode_intervals()[0] if intervals else None
    split, rec = _records(hp.plan_split(2, max_blocks, iv_ptr))
    assert split.B == 2
    item_of = {int(i): w for w, i in enumerate(hp.work)}
    slots, cut_rows = [], []
    assert sorted(set(rec[:, 0].tolist())) == sorted(item_of)
    for b, row in ((b, row) for b in range(2) for row in item_of):
        mine = rec[(rec[:, 0] == row) & (rec[:, 9] == b)]
        parts, of = mine[:, 8] & 0xffff, mine[:, 8] >> 16
        mine, of = mine[np.argsort(parts)], of[np.argsort(parts)]
        n, length = len(mine), int(hp.row_ptr[row + 1] - hp.row_ptr[row])
        assert sorted(parts.tolist()) == list(range(n)) and (of == n).all() and n <= 16
        ends = np.append(mine[:, 1], length)
        assert ends[0] == 0 and (ends[1:] - ends[:-1] == mine[:, 2]).all()
        assert n == 1 or (mine[:, 2] > 0).all()
        if max_blocks:
            assert n == max(1, min(16, -(-length // max_blocks)))
        assert (mine[:, 3] == hp.row_ptr[row] + mine[:, 1]).all()
        assert (mine[:, 4:6] == ([iv_ptr[row], iv_ptr[row + 1] - 1] if intervals else [0, 0])).all()
        w = item_of[row]
        assert (mine[:, 6:8] == [hp.fan_ptr[w], hp.fan_ptr[w + 1] - hp.fan_ptr[w]]).all()
        if n > 1:
            assert len(set(mine[:, 10])) == 1 and len(set(mine[:, 11])) == 1
            slots += range(mine[0, 10], mine[0, 10] + n)
            cut_rows.append(int(mine[0, 11]))
    assert sorted(slots) == list(range(split.n_slots))
    assert sorted(cut_rows) == list(range(split.n_rows))


def test_same_cuts_for_every_order_and_no_plan_for_long_calls(lib):
    mask, repeat = random_mask(5, 6, 40, 40, 0.5, 0.2, keep_diagonal=True)
    cuts = []
    for order in range(5):
        _, rec = _records(lib.compile_pattern(mask, repeat, 6, 40 * 128, 128, 128, order).plan_split(1))
        cuts.append(sorted(map(tuple, rec[:, [0, 1, 2, 8, 9]].tolist())))
    assert all(c == cuts[0] for c in cuts)
    hp = lib.compile_pattern(np.ones((8, 100, 100), np.uint8), None, 8, 100 * 128, 128, 128)
    assert hp.plan_split(1) is None  # 312 stages of work per workgroup that the device holds
    assert lib.compile_pattern(np.ones((6, 100, 100), np.uint8), None, 6, 100 * 128, 128, 128).plan_split(1) is not None


def test_workspace_and_refusals(lib):
    raw = lib.load_library()
    hp = lib.compile_pattern(np.ones((2, 10, 10), np.uint8), None, 2, 1280, 128, 128)
    split, _ = hp.plan_split(2, 4)
    assert (split.n_rows, split.n_slots) == (40, 120)
    assert raw.calibatt_split_workspace_bytes(C.byref(split), 128, 128) == 120 * (128 * 128 + 256 * 2) * 4
    for B, max_blocks, status in ((0, 0, -2), (1, -1, -2), (1, 4, -7)):
        c, out = binding._CPattern(), binding._CSplit()
        c.n_work, c.block_k, c.nnz, c.nbq = hp.n_work, 128, hp.nnz, 10
        c.row_ptr, c.work, c.fan_ptr = (a.ctypes.data for a in (hp.row_ptr, hp.work, hp.fan_ptr))
        buf = np.empty(12, np.int32)
        assert raw.calibatt_plan_split(C.byref(c), B, max_blocks, binding._ptr(buf, C.c_int32), 1, C.byref(out)) == status
    assert raw.calibatt_plan_split(None, 1, 0, None, 0, C.byref(out)) == -1


def test_plan_of_lists_that_are_views(lib):
    """Host lists that are strided views or of another integer type give the plan of their values."""
    import dataclasses

    mask, repeat = random_mask(6, 3, 20, 20, 0.5, 0.2, keep_diagonal=True)
    hp = lib.compile_pattern(mask, repeat, 3, 20 * 128, 128, 128)

    def view(a):  # every second entry of an array whose others are zero
        wide = np.full((a.size, 2), 0, np.int32)
        wide[:, 0] = a
        return wide[:, 0]

    lists = ("row_ptr", "col_idx", "work", "fan_ptr")
    want = hp.plan_split(1, 3)
    for change in (view, lambda a: a.astype(np.int64)):
        got = dataclasses.replace(hp, **{n: change(getattr(hp, n)) for n in lists}).plan_split(1, 3)
        assert (got[1] == want[1]).all() and got[0].n_slots == want[0].n_slots
    backwards = dataclasses.replace(hp, work=np.ascontiguousarray(hp.work[::-1])[::-1])
    assert (backwards.plan_split(1, 3)[1] == want[1]).all()


@pytest.mark.parametrize("intervals,head_map,persistent", [(False, None, True), (True, [5, 0, 2], True), (True, None, False)])
def test_a_small_pattern_is_one_copy(lib, monkeypatch, intervals, head_map, persistent):
    """Lists, plans and counters of a pattern go to the device in one copy, long lists in one of their own, with the values
    of the host."""
    import torch

    copies, plain = [], torch.from_numpy
    monkeypatch.setattr(torch, "from_numpy", lambda a: copies.append(a.size) or plain(a))
    for n, more in ((20, 0), (130, 0 if intervals else 1)):
        mask, repeat = random_mask(n, 3, n, n, 0.5, 0.2, keep_diagonal=True)
        mask[1, 3] = 0
        hp = lib.compile_pattern(mask, repeat, 3, n * 128, 128, 128)
        copies.clear()
        dp = hp.to_device("cpu", persistent=persistent, intervals=intervals, head_map=head_map)
        assert len(copies) == 1 + more + (n == 130 and persistent) * sum(p.n_parts * 12 > 1 << 14 for p, _ in dp._plans.values())
        want = {name: getattr(hp, name) for name in dp._NAMES if not (intervals and name == "col_idx")}
        if intervals:
            want["iv_ptr"], want["iv"] = hp.encode_intervals()
        if head_map:
            want["head_map"] = np.array(head_map, np.int32)
        assert sorted(dp.tensors) == sorted(want)
        for name, a in want.items():
            t = dp.tensors[name]
            assert t.dtype == torch.int32 and t.is_contiguous() and t.data_ptr() % 16 == 0
            assert getattr(dp.c, name) == t.data_ptr()
            assert (t.numpy().view(a.dtype) == a).all() if a.size else t.tolist() == [0]
        assert bool(dp._plans) == persistent
        for B, (split, parts) in dp._plans.items():
            host = hp.plan_split(B, 0, dp._iv_ptr)
            assert (parts.numpy() == host[1]).all() and parts.data_ptr() % 16 == 0 and split.n_rows == host[0].n_rows
        if persistent:
            words = [dp._own.words, *dp._spare]
            assert len(words) == 8 and all(len(w) == dp._words and not w.any() and w.data_ptr() % 128 == words[0].data_ptr() % 128
                                           for w in words)
            assert dp.c.work_counter == dp.counter.data_ptr() == words[0].data_ptr()
        else:
            assert dp.counter is None and dp.c.work_counter is None


def test_plan_bytes(lib):
    """What the plans take on the GPU is reported, for a pattern and for a dictionary whose keys share one."""
    from paper_2603_05503_amd.pipeline import CalibAttention

    mask, repeat = random_mask(3, 2, 64, 64, 0.4, 0.1, keep_diagonal=True)
    hp = lib.compile_pattern(mask, repeat, 2, 64 * 128, 128, 128)
    dp = hp.to_device("cpu", intervals=True)
    plans = [hp.plan_split(B) for B in (1, 2)]
    rows = max(p[0].n_rows for p in plans)
    assert rows > 0
    want = sum(p[1].nbytes for p in plans) + 8 * -(-rows // 32) * 32 * 4
    assert dp.plan_bytes == want and want > dp.index_bytes
    assert hp.to_device("cpu", persistent=False).plan_bytes == 0
    att = CalibAttention(2, 64 * 128, 128, device="cpu")
    att.add("a", mask, repeat=repeat)
    att.entries["b"] = att.entries["a"]
    assert att.plan_bytes == want and att.index_bytes == dp.index_bytes


@pytest.mark.parametrize("H,n,density", [(2, 128, 0.376), (2, 128, 0.25), (3, 95, 0.75), (2, 128, 0.46), (3, 90, 0.4)])
def test_no_round_for_a_few_parts(lib, H, n, density):
    """Rows of nearly one length are not cut into a few more parts than the 512 workgroups that the device holds."""
    for seed in range(3):
        mask, _ = random_mask(seed, H, n, n, density)
        plan = lib.compile_pattern(mask, None, H, n * 128, 128, 128).plan_split(1)
        n_parts = 0 if plan is None else len(_records(plan)[1])
        assert not 512 < n_parts < 600, n_parts


@pytest.mark.parametrize("H,n,density,bq", [(12, 85, 0.686, 128), (4, 128, 0.5, 128), (2, 512, 0.1, 64), (20, 60, 0.6, 128), (5, 77, 1.0, 64),
                                            (15, 17, 1.0, 128), (15, 17, 1.0, 64), (15, 30, 1.0, 128), (15, 40, 1.0, 64)])
@pytest.mark.parametrize("max_blocks", [0, 7, 1000])
@pytest.mark.parametrize("with_columns", [True, False])
def test_no_xcd_has_a_round_more(lib, H, n, density, bq, max_blocks, with_columns):
    """An XCD, with an eighth of the workgroups, gets no more parts than it takes in the rounds that all parts need, and
    where they fit at a time no more than its 32 CUs take by ones, twos and so on."""
    mask, _ = random_mask(n, H, n, n, density)
    mask[0] = np.tril(mask[0])  # uneven rows: shares of equal cost hold different numbers of parts
    if H == 15:
        mask = np.tril(mask)
    hp = lib.compile_pattern(mask, None, H, n * bq, bq, bq)
    if not with_columns:
        c = binding._CPattern()
        for f in ("H", "N", "block_q", "block_k", "nbq", "nbk", "n_work", "n_repeat", "order", "max_row", "nnz"):
            setattr(c, f, getattr(hp, f))
        c.row_ptr, c.work, c.fan_ptr = (a.ctypes.data for a in (hp.row_ptr, hp.work, hp.fan_ptr))
        split, buf = binding._CSplit(), np.empty((200000, 12), np.int32)
        assert binding.load_library().calibatt_plan_split(C.byref(c), 1, max_blocks, binding._ptr(buf, C.c_int32), len(buf),
                                                          C.byref(split)) == 0
        plan = (split, buf[:split.n_parts]) if split.n_parts else None
    else:
        plan = hp.plan_split(1, max_blocks)
    if plan is None:
        return
    slots = 512 if bq == 128 else 1024
    _, live = _records(plan)
    of_xcd = [int((plan[1][x::8, 0] >= 0).sum()) for x in range(8)]
    step = 256 if len(live) <= slots else slots
    assert max(of_xcd) <= step // 8 * -(-len(live) // step)
    # every row is there, once
    assert sorted(set(live[:, 0].tolist())) == sorted(hp.work.tolist())
    assert (np.bincount(live[:, 0], live[:, 2], minlength=H * n)[hp.work] == (hp.row_ptr[1:] - hp.row_ptr[:-1])[hp.work]).all()


@pytest.mark.parametrize("H,n,band", [(24, 8, 0.22), (28, 8, 0.24), (1, 64, 0.35), (3, 35, 0.31)])
def test_cuts_count_adding_up_and_shared_cus(lib, H, n, band):
    """Rows of one to four blocks are not cut to be added up for little, nor longer ones into a few more parts than there are
    CUs (256)."""
    for seed in range(3):
        if n == 8:  # a band and a few blocks beside it
            i = np.arange(n) / n
            mask = (np.abs(i[:, None] - i) < band / 2) | (np.random.default_rng(seed).random((H, n, n)) < band / 5)
            mask[:, np.arange(n), np.arange(n)] = 1
        else:
            mask, _ = random_mask(seed, H, n, n, band, keep_diagonal=True)
        split, live = _records(lib.compile_pattern(mask.astype(np.uint8), None, H, n * 128, 128, 128).plan_split(1))
        assert split.n_rows == 0 if n == 8 else len(live) <= 256, (split.n_rows, len(live))
