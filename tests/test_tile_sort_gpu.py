"""The sort of one tile in registers and LDS (short arrays and segments) at the edges of its
keys-per-lane steps, on keys whose varying bits start and end anywhere."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, gpu_sort, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

# workgroups of 4, 8 and 16 waves step at 256, 512 and 1024 keys times a power of two
EDGES = [1, 2, 64, 255, 256, 257, 512, 513, 1025, 2047, 2048, 2049, 4096, 4097, 8191, 8193, 16383, 16384]


def _keys(n: int, kind: str) -> np.ndarray:
    full = np.random.default_rng(n).integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
    return {"full": full,
            "top_bit": full & np.uint32(0x80000000),
            "one_window": (full & np.uint32(0x0001FE00)) | np.uint32(0xA00000F1),
            "split_windows": (full & np.uint32(0xC0000003)) | np.uint32(0x00FFFF00),
            "equal": np.full(n, 0xFFFFFFFF, np.uint32)}[kind]


@pytest.mark.parametrize("rank_mode", [0, 1])
@pytest.mark.parametrize("kind", ["full", "top_bit", "one_window", "split_windows", "equal"])
def test_tile_edges(kind, rank_mode):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    binding.ap_set_rank_mode(rank_mode)
    try:
        for n in EDGES:
            keys = _keys(n, kind)
            announce(f"tile sort n={n} {kind} rank {rank_mode}")
            out, spl = gpu_sort(keys, 64)
            want = oracle.sort_u32(keys)
            assert np.array_equal(out, want), n
            assert np.array_equal(spl, oracle.splitters(want, 64)), n
        # the same lengths as segments of one batch
        keys = np.concatenate([_keys(n, kind) for n in EDGES])
        off = np.concatenate([[0], np.cumsum(EDGES)]).astype(np.uint32)
        t, _ = to_dev(keys)
        binding.ap_sort_u32_segmented(t, torch.from_numpy(off.view(np.int32)).to("cuda"))
        torch.cuda.synchronize()
        assert np.array_equal(to_host(t), oracle.sort_segmented(keys, off.astype(np.uint64)))
    finally:
        binding.ap_set_rank_mode(0)


# the sort by shares of the ranks (4097 to 16384 keys, out of place): keys that put its share ends into
# one step, one value, the largest value, or past the last key
@pytest.mark.parametrize("rank_mode", [0, 1])
@pytest.mark.parametrize("kind", ["full", "bands", "long_tail", "few", "one_outlier", "ends", "half_one_value", "sorted"])
def test_rank_shares(kind, rank_mode):
    torch_cuda()
    from paper_cs_0004013_amd import binding
    binding.ap_set_rank_mode(rank_mode)
    try:
        for n in [4097, 8191, 8192, 8193, 12345, 16383, 16384]:
            rng = np.random.default_rng(n)
            full = rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
            keys = {"full": full,
                    "bands": ((full & np.uint32(0xF0000000)) | (full & np.uint32(0xFF))).astype(np.uint32),
                    "long_tail": np.exp(rng.normal(8, 4, n)).clip(0, 4e9).astype(np.uint32),
                    "few": np.array([5, 5, 5, 9, 0xFFFFFFFF], np.uint32)[full % np.uint32(5)],
                    "one_outlier": np.where(np.arange(n) == 77, np.uint32(0xFFFFFFFF), full & np.uint32(0xFFF)),
                    "ends": np.where(full & np.uint32(1), np.uint32(0xFFFFFFFF), np.uint32(0)),
                    "half_one_value": np.where(full & np.uint32(1), np.uint32(0x12345678), full),
                    "sorted": np.sort(full)}[kind].astype(np.uint32)
            announce(f"rank shares n={n} {kind} rank {rank_mode}")
            out, spl = gpu_sort(keys, 64, pad_front=n % 4)
            want = oracle.sort_u32(keys)
            assert np.array_equal(out, want), n
            assert np.array_equal(spl, oracle.splitters(want, 64)), n
        out, spl = gpu_sort(keys, 20000)                 # more cells than keys
        assert np.array_equal(out, want) and np.array_equal(spl, oracle.splitters(want, 20000))
    finally:
        binding.ap_set_rank_mode(0)


def test_rank_shares_splitters_into_the_input():
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    for n in [5000, 8192, 12345]:
        keys = _keys(n, "full")
        announce(f"splitters into the input, n={n}")
        for at in (0, n // 2, n - 63):
            t_in, _ = to_dev(keys)
            t_out = torch.empty(n, dtype=torch.int32, device="cuda")
            binding.ap_sort_u32(t_in, t_out, 64, t_in[at:at + 63])
            torch.cuda.synchronize()
            want = oracle.sort_u32(keys)
            assert np.array_equal(to_host(t_out), want), (n, at)
            assert np.array_equal(to_host(t_in[at:at + 63]), oracle.splitters(want, 64)), (n, at)



# a workgroup takes nseg / (24 per CU) segments, at most 64: below, between and above those bounds
@pytest.mark.parametrize("nseg,hi", [(12287, 700), (20000, 4200), (400_003, 40)])
def test_many_short_segments(nseg, hi):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    rng = np.random.default_rng(nseg)
    lens = rng.integers(0, hi + 1, size=nseg)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint32)
    keys = rng.integers(0, 1 << 32, size=int(off[-1]), dtype=np.uint64).astype(np.uint32)
    announce(f"short segments nseg={nseg} n={keys.size}")
    t, _ = to_dev(keys, 1)
    st = torch.full((1,), 99, dtype=torch.int32, device="cuda")
    binding.ap_sort_u32_segmented(t, torch.from_numpy(off.view(np.int32)).to("cuda"), st)
    torch.cuda.synchronize()
    assert int(st[0]) == 0
    assert np.array_equal(to_host(t), oracle.sort_segmented(keys, off.astype(np.uint64)))
