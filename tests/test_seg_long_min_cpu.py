"""The long-segment threshold reserves scratch only for segments that can take the device-wide passes: those of
up to 4096 keys never do, whatever the threshold."""
from __future__ import annotations

import pytest

from paper_cs_0004013_amd import binding


@pytest.fixture
def long_min():
    saved = binding.ap_segmented_get_long_min()
    yield binding.ap_segmented_set_long_min
    binding.ap_segmented_set_long_min(saved)


def _bytes(n_total: int, nseg: int) -> int:
    return int(binding.lib().ap_segmented_workspace_bytes(n_total, nseg))


@pytest.mark.parametrize("low", [2, 100, 4096])
def test_low_threshold_reserves_as_the_lowest_that_matters(long_min, low):
    for n_total in (4096, 4097, 100_000, 1 << 24):
        long_min(4097)
        want = _bytes(n_total, 50)
        long_min(low)
        assert binding.ap_segmented_get_long_min() == low
        assert _bytes(n_total, 50) == want, n_total


def test_threshold_at_its_edges(long_min):
    long_min(0)
    never = _bytes(4097, 50)
    long_min(4097)
    assert _bytes(4097, 50) > never and _bytes(4096, 50) <= never
    long_min(5000)
    assert _bytes(4999, 50) <= _bytes(5000, 50) - 4096    # from 5000 keys on one long segment is possible
    with pytest.raises(binding.ApError):
        long_min(1)
