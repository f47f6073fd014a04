"""Kept for the tests' imports: the helpers live in workloads/device.py."""
from workloads.device import (  # noqa: F401
    MAX_ABS,
    MEAN_ABS,
    assert_parity,
    assert_repeats_bitwise,
    bits_to_f64,
    error_stats,
    from_dev,
    run_gpu,
    to_dev,
)


def whole_rows(dp):
    """The pattern without plans: its calls run whole rows, from the queues where there are more rows than workgroups."""
    dp._plan(True, None)
    assert not dp._plans
    return dp


def cut_rows(dp, max_blocks):
    """The pattern planned for parts of at most ``max_blocks`` key blocks, so that batches of one and two are cut."""
    dp._plan(True, max_blocks)
    assert sorted(dp._plans) == [1, 2] and all(p.n_slots > 0 for p, _ in dp._plans.values())
    return dp


def queues_ran(words):
    """Whether a persistent launch left its residency in a stream's scheduler words, and left the counters re-armed."""
    words = words[:16].cpu().tolist()
    assert words[:9] == [0] * 9 and words[12:] == [0] * 4
    return words[10] != 0 and words[11] != 0
