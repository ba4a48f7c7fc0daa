"""What the autotuner sweeps and writes, as far as it needs no GPU."""
import ctypes

import pytest

from paper_2003_01178_amd import autotune
from paper_2003_01178_amd import crystal as cx


def table(kind, keys, has_payload=True):
    """A table's description, without its memory."""
    desc = cx.HT()
    assert cx.load().crystal_ht_init(ctypes.byref(desc), kind, keys, 0, keys - 1, int(has_payload)) == cx.OK
    return desc


def slices(desc, with_payload=False):
    return cx.load().crystal_ht_probe_slices(ctypes.byref(desc), int(with_payload))


def test_swept_probe_tables_are_probed_by_the_tuned_kernel():
    for d in autotune.PROBE_KEYS:
        assert slices(table(cx.HT_LINEAR, d)) == 0, d


@pytest.mark.parametrize("kind,keys,has_payload,plain,with_payload", [
    (cx.HT_LINEAR, 1 << 18, True, 0, 0), (cx.HT_LINEAR, (1 << 18) + 1, True, 4, 4),
    (cx.HT_LINEAR, 1 << 20, True, 4, 4), (cx.HT_LINEAR, 1 << 21, True, 8, 4), (cx.HT_LINEAR, 1 << 22, True, 8, 0),
    (cx.HT_LINEAR, 1 << 23, True, 0, 0), (cx.HT_DIRECT, 1 << 20, True, 0, 0), (cx.HT_DIRECT, (1 << 20) + 1, True, 4, 4),
    (cx.HT_DIRECT, (1 << 21) + 1, True, 8, 4), (cx.HT_DIRECT, (1 << 23) + 1, True, 0, 0),
    (cx.HT_DIRECT, 1 << 23, False, 0, 0)])
def test_probe_slices_of_tables(kind, keys, has_payload, plain, with_payload):
    desc = table(kind, keys, has_payload)
    assert (slices(desc), slices(desc, True)) == (plain, with_payload)


def test_common_winner_of_several_sweeps():
    a = [(1.0, 256, 8, 1), (1.1, 512, 8, 1), (3.0, 1024, 16, 1)]
    b = [(10.0, 1024, 16, 1), (11.0, 512, 8, 1), (20.0, 256, 8, 1)]
    assert autotune.common_winner([a, b]) == (512, 8, 1)
    assert autotune.common_winner([a, b[:1] + b[2:]]) == (256, 8, 1)     # 512 x 8 was discarded in one
    assert autotune.common_winner([a]) == (256, 8, 1)


@pytest.fixture
def untuned():
    cx.tune_reset()
    yield
    cx.tune_reset()


def test_radix_entries_leave_shorter_inputs_untuned(untuned):
    """The built-in radix shapes follow the size; an entry measured at 2^28
    pairs governs inputs as long as that and no others."""
    sizes = (1000, 100_003, 1 << 20, 1 << 25, (1 << 28) - 1)
    before = [cx.tune_get(cx.K_RADIX, n) for n in sizes]
    autotune.assign(cx.K_RADIX, [(1 << 28, (512, 16, 1))], lowest=autotune.bucket(1 << 28))
    assert [cx.tune_get(cx.K_RADIX, n) for n in sizes] == before
    assert cx.tune_get(cx.K_RADIX, 1 << 28) == cx.tune_get(cx.K_RADIX, 1 << 31) == (512, 16, 1)


def test_entries_cover_all_sizes_of_a_kernel_measured_at_several(untuned):
    autotune.assign(cx.K_STAR, [(1 << 27, (512, 8, 8)), (1 << 22, (512, 4, 8))])
    assert cx.tune_get(cx.K_STAR, 1) == cx.tune_get(cx.K_STAR, (1 << 25) - 1) == (512, 4, 8)
    assert cx.tune_get(cx.K_STAR, 1 << 25) == cx.tune_get(cx.K_STAR, 1 << 40) == (512, 8, 8)
    autotune.assign(cx.K_SELECT, [])
    assert cx.tune_get(cx.K_SELECT, 1 << 29) == (512, 16, 0)


@pytest.mark.parametrize("winner,other,worth", [(0.97, 1.0, True), (0.99, 1.0, False), (0.5, 1.03, False)])
def test_an_entry_has_to_gain_and_not_to_slow_other_calls(untuned, monkeypatch, winner, other, worth):
    monkeypatch.setattr(autotune, "time_ms", lambda call, reps: call())
    rows = [(winner, 512, 8, 0), (2.0, 256, 8, 0)]
    assert autotune.improves(cx.K_SELECT, 1 << 29, rows, 1.0, [(lambda: other, 1.0)]) == worth


def test_shared_scans_are_swept_over_short_ranges_too(untuned):
    """The shipped table has other shapes for short ranges; a sweep of the
    long one alone would replace them."""
    autotune.assign(cx.K_SHARED_SCAN_SCALAR, [(m, (256 << i, 8, 0)) for i, m in enumerate(autotune.SCAN_ROWS)])
    shapes = {cx.tune_get(cx.K_SHARED_SCAN_SCALAR, n) for n in (10_000, 3_000_000, 75_000_000)}
    assert len(shapes) == 3
