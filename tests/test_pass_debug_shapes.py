"""The perturbed digit pass covers every tile that the default pass runs: the kernels are built (seen in the
library's symbol names), and on the device each of the tiles used from 2^22 keys on sorts exactly under it."""
from __future__ import annotations

import os
import re

import numpy as np
import pytest

import oracle
from paper_cs_0004013_amd import build, inputs
from tests.gpu_util import announce, gpu_sort, torch_cuda

PERTURB = 1


def _built(kernel: bytes) -> set[int]:
    """Keys per lane of the 16-wave, 8-bit instances of a kernel in the library."""
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    with open(build.LIB, "rb") as f:
        names = f.read()
    return {int(x) for x in re.findall(kernel + rb"ILi8ELi16ELi(\d+)E", names)}


def test_every_tile_has_a_perturbed_kernel():
    tiles = _built(b"6k_pass")
    assert tiles == {4, 8, 16, 20, 24, 28, 32}
    assert _built(b"10k_pass_dbg") == tiles


@pytest.fixture
def debug_off():
    from paper_cs_0004013_amd import binding
    yield binding
    binding.ap_debug_pass(0)
    binding.ap_set_pass_shape(-1)


# the sizes at which the tile is the given one, whole rounds and one key into the next round's tile
@pytest.mark.gpu
@pytest.mark.parametrize("ipt", [20, 24, 28, 32])
@pytest.mark.parametrize("kind", ["uniform", "bands", "one_digit", "constant"])
def test_perturbed_tiles(debug_off, ipt, kind):
    torch = torch_cuda()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for n in (ipt * 1024 * cus, ipt * 1024 * cus - 4095):
        rng = np.random.default_rng(n)
        full = rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
        keys = {"uniform": full, "bands": inputs.dist_keys("e", n, rng),
                "one_digit": (full & np.uint32(0x00FF0000)) | np.uint32(0x12003456),
                "constant": np.full(n, 0x12345678, np.uint32)}[kind]
        debug_off.ap_debug_pass(PERTURB, n)
        announce(f"perturbed pass, {ipt} keys per lane, n={n} {kind}")
        out, spl = gpu_sort(keys, 64, inplace=bool(n & 1))
        want = np.sort(keys)
        assert np.array_equal(out, want), n
        assert np.array_equal(spl, oracle.splitters(want, 64)), n
