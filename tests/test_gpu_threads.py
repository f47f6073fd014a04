"""The forward called from several host threads at once, each on its own stream with its own
scheduler workspace, reproduces the bits of serial calls (the library keeps no state between calls
except per-device launch facts cached through atomics)."""
import threading

import numpy as np
import pytest

from tests.parity_utils import cut_rows, queues_ran, whole_rows
from tests.test_gpu_parity import _qkv
from workloads import random_mask, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,H", [("auto", 6), ("queues", 30), ("2wg", 30)])
def test_four_threads_four_streams(lib, kernel, H):
    import torch

    from paper_2603_05503_amd import binding

    print(f"threads kernel={kernel}", flush=True)
    which = binding.KERNEL_TWO_WORKGROUPS if kernel == "2wg" else binding.KERNEL_AUTO
    prepare = (lambda dp: cut_rows(dp, 4)) if kernel == "auto" else whole_rows
    B, N, D, blk = 1, 128 * 24 + 50, 128, 128
    nb = -(-N // blk)
    n_threads, rounds = 4, 6
    cases = []
    for i in range(n_threads):
        q, k, v = _qkv(700 + i, B, H, N, D, 2.0)
        mask, repeat = random_mask(800 + i, H, nb, nb, 0.3 + 0.1 * i, 0.2, tail_partial=True)
        hp = lib.compile_pattern(mask, repeat, H, N, blk, blk, 4)
        assert kernel == "auto" or hp.n_work > 512  # more rows than workgroups
        cases.append((to_dev(q), to_dev(k), to_dev(v), hp))
    # serial reference bits, each case with a workspace of its own
    want = []
    for tq, tk, tv, hp in cases:
        out = torch.empty_like(tq)
        lib.sparse_attn_fwd(tq, tk, tv, out, prepare(hp.to_device()), 0.09, kernel=which)
        torch.cuda.synchronize()
        want.append(out.view(torch.int16).clone())
    errors = []
    barrier = threading.Barrier(n_threads)

    def worker(i):
        try:
            tq, tk, tv, hp = cases[i]
            stream = torch.cuda.Stream()
            dp = prepare(hp.to_device())  # own index tensors and own work counters
            outs = [torch.empty_like(tq) for _ in range(rounds)]
            torch.cuda.synchronize()
            barrier.wait()
            for r in range(rounds):
                outs[r].view(torch.int16).fill_(0x7FC1)
                stream.wait_stream(torch.cuda.current_stream())
                lib.sparse_attn_fwd(tq, tk, tv, outs[r], dp, 0.09, stream=stream.cuda_stream, kernel=which)
            stream.synchronize()
            for r in range(rounds):
                if not torch.equal(outs[r].view(torch.int16), want[i]):
                    errors.append((i, r, "bits differ from the serial call"))
            if queues_ran(dp.counter) != (kernel != "auto"):
                errors.append((i, -1, "another launch than the one meant"))
        except Exception as e:  # noqa: BLE001
            errors.append((i, -1, repr(e)))

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(n_threads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors


@pytest.mark.parametrize("rows", ["queues", "cut"])
def test_first_calls_on_streams_do_not_wait_for_another(lib, rows):
    """A pattern that is in use gets cleared work counters and arrivals for every further stream, also while the stream
    that was current when the call was made is busy and its free memory holds other values."""
    import torch

    print(f"first calls on ten streams: {rows}", flush=True)
    B, H, N, D, blk = 2, 16, 3000, 128, 128
    nb = -(-N // blk)
    tq, tk, tv = (to_dev(x) for x in _qkv(900, B, H, N, D, 2.0))
    mask, repeat = random_mask(901, H, nb, nb, 0.3, 0.2, tail_partial=True)
    dp = lib.compile_pattern(mask, repeat, H, N, blk, blk, 3).to_device(persistent=True)
    dp = whole_rows(dp) if rows == "queues" else cut_rows(dp, 4)
    assert dp.host.n_work * B > 512  # more items than workgroups: whole rows use the counters
    want = lib.sparse_attn_fwd(tq, tk, tv, torch.empty_like(tq), dp, 0.09).view(torch.int16).clone()
    streams = [torch.cuda.Stream() for _ in range(10)]
    outs = [torch.full_like(tq, float("nan")) for _ in streams]
    for _ in range(64):
        torch.full((dp._words,), 1 << 24, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    torch.cuda._sleep(200_000_000)
    for out, s in zip(outs, streams):
        for _ in range(2):
            lib.sparse_attn_fwd(tq, tk, tv, out, dp, 0.09, stream=s.cuda_stream)
    for s in streams:
        s.synchronize()
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        assert torch.equal(out.view(torch.int16), want), i
    states = [dp._own, *dp._per_stream.values()]
    assert len(states) == 11 and not dp._spare
    assert all(queues_ran(s.words) == (rows == "queues") and not s.words[32:].any() for s in states)


def test_default_stream_by_its_handle(lib):
    """Handle 0 names the default stream also where another one is current: what a call allocates and clears lies there."""
    import torch

    from paper_2603_05503_amd import binding

    print("default stream by its handle", flush=True)
    H, N, D, blk = 4, 2000, 128, 128
    q, k, v = (to_dev(x) for x in _qkv(905, 1, H, N, D, 2.0))
    mask, repeat = random_mask(906, H, 16, 16, 0.6, 0.2, tail_partial=True)
    dp = cut_rows(lib.compile_pattern(mask, repeat, H, N, blk, blk).to_device(), 2)
    want = lib.sparse_attn_fwd(q, k, v, torch.empty_like(q), dp, 0.09).view(torch.int16).clone()
    cut_rows(dp, 2)._spare.clear()
    side, out = torch.cuda.Stream(), torch.empty_like(q)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        lib.sparse_attn_fwd(q, k, v, out, dp, 0.09)  # the pattern's own words go to the side stream
        side.synchronize()
        handle, other = binding._stream_of(0, q.device)
        assert handle == 0 and other.cuda_stream == 0
        for _ in range(2):
            lib.sparse_attn_fwd(q, k, v, out.zero_(), dp, 0.09, stream=side.cuda_stream)
            side.synchronize()
            lib.sparse_attn_fwd(q, k, v, out, dp, 0.09, stream=0)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), want)
    assert list(dp._per_stream) == [0]


def test_stream_objects_are_made_once(lib, monkeypatch):
    """A call on another than the current stream makes a torch stream of the handle the first time that it needs one
    (rows that are not cut need none), and leaves the current stream and device as they were, also when it is refused."""
    import torch

    from paper_2603_05503_amd import binding

    print("stream objects", flush=True)
    H, N, D, blk = 4, 2000, 128, 128
    q, k, v = (to_dev(x) for x in _qkv(907, 1, H, N, D, 2.0))
    mask, repeat = random_mask(908, H, 16, 16, 0.6, 0.2, tail_partial=True)
    hp = lib.compile_pattern(mask, repeat, H, N, blk, blk)
    made, plain = [], torch.cuda.ExternalStream
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda *a, **kw: made.append(a) or plain(*a, **kw))
    side, current, out = torch.cuda.Stream(), torch.cuda.current_stream(), torch.empty_like(q)
    for max_blocks, most in ((2, 1), (1000, 0)):
        dp = hp.to_device()
        dp._plan(True, max_blocks)
        assert (dp._plans[1][0].n_slots > 0) == (most > 0)
        made.clear()
        for _ in range(3):
            lib.sparse_attn_fwd(q, k, v, out, dp, 0.09, stream=side.cuda_stream)
            assert torch.cuda.current_stream() == current
        assert len(made) == most
        with pytest.raises(binding.CalibattError):
            lib.sparse_attn_fwd(q, k, v, out, dp, 0.09, block_k=7, stream=side.cuda_stream)
        assert torch.cuda.current_stream() == current and torch.cuda.current_device() == 0
    torch.cuda.synchronize()
