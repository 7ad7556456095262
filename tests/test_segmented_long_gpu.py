"""Long segments of a batch, one for every set of digits that vary (an odd number of sorting passes
needs the pass of a constant digit to copy), twice in a row through one control block, also after a call
with invalid offsets."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank_mode", [0, 1])
@pytest.mark.parametrize("stream", [False, True])
def test_varying_digits(rank_mode, stream):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    long_min = binding.ap_segmented_get_long_min()
    binding.ap_set_rank_mode(rank_mode)
    binding.ap_segmented_set_long_min(20_000)
    try:
        rng = np.random.default_rng(5)
        lens = [20_000 + 8191 * i + (i & 1) for i in range(16)]
        parts = []
        for i, n in enumerate(lens):
            mask = sum(0xFF << (8 * d) for d in range(4) if i >> d & 1)
            k = rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
            parts += [(k & np.uint32(mask)) | np.uint32(0x3C5A9617 & ~mask & 0xFFFFFFFF), k[:i * 700]]
        keys = np.concatenate(parts)
        off = np.concatenate([[0], np.cumsum([p.size for p in parts])]).astype(np.uint32)
        want = oracle.sort_segmented(keys, off.astype(np.uint64))
        wrong = off.copy()
        wrong[3], wrong[4] = off[4], off[3]
        t_off = torch.from_numpy(off.view(np.int32)).to("cuda")
        t_wrong = torch.from_numpy(wrong.view(np.int32)).to("cuda")
        announce(f"long segments, every set of varying digits, rank {rank_mode} stream {stream}")
        with torch.cuda.stream(torch.cuda.Stream() if stream else torch.cuda.current_stream()):
            for offsets, expect in ((t_off, want), (t_wrong, keys), (t_off, want)):
                t, _ = to_dev(keys)
                binding.ap_sort_u32_segmented(t, offsets)
                torch.cuda.synchronize()
                assert np.array_equal(to_host(t), expect)
    finally:
        binding.ap_segmented_set_long_min(long_min)
        binding.ap_set_rank_mode(0)


# below 2^20 keys in all the length groups run one after another, from there on side by side
@pytest.mark.parametrize("total", [(1 << 20) - 1, 1 << 20])
@pytest.mark.parametrize("stream", [False, True])
def test_groups_in_sequence_or_side_by_side(total, stream):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    rng = np.random.default_rng(total)
    lens = [4097, 8192, 8193, 16384, 16385, 100_000, 4096, 1024, 1, 0, 70_000] * 4
    lens.append(total - sum(lens))
    keys = rng.integers(0, 1 << 32, size=total, dtype=np.uint64).astype(np.uint32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint32)
    want = oracle.sort_segmented(keys, off.astype(np.uint64))
    t_off = torch.from_numpy(off.view(np.int32)).to("cuda")
    announce(f"groups, {total} keys, stream {stream}")
    t, _ = to_dev(keys)
    src = t.clone()
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream() if stream else torch.cuda.current_stream()):
        for _ in range(3):
            t.copy_(src)
            binding.ap_sort_u32_segmented(t, t_off)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(t), want)
