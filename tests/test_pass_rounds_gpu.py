"""Digit passes at the sizes where their tile changes (20K, 24K, 28K and 32K keys, by the rounds of tiles
that the device needs), with a ragged last tile, and in place."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, gpu_sort, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ipt", [20, 24, 28, 32])
def test_tile_bounds(ipt):
    torch = torch_cuda()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for n in (ipt * 1024 * cus, ipt * 1024 * cus + 1, 2 * ipt * 1024 * cus - 1, 3 * ipt * 1024 * cus + 77):
        rng = np.random.default_rng(n)
        keys = rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
        announce(f"pass rounds n={n}")
        out, spl = gpu_sort(keys, 64, inplace=bool(n & 1), pad_front=n % 3)
        want = np.sort(keys)
        assert np.array_equal(out, want), n
        assert np.array_equal(spl, oracle.splitters(want, 64)), n
