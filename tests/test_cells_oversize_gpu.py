"""Cells longer than a tile in the two-launch sort.  The sample that draws the cells takes its positions by a
scramble salted with the input's address: keys that avoid the unsalted positions must cost what any keys
cost, and keys that avoid the salted ones (all of them in one cell, sorted by digit sweeps) must still come
out sorted and stable."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

M64 = (1 << 64) - 1


def _salt(address: int) -> int:
    x = address
    x = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & M64
    x = ((x ^ (x >> 27)) * 0x94D049BB133111EB) & M64
    return x >> 32


def _sampled(n: int, salt: int) -> np.ndarray:
    """Mask of the positions that a sample of 1024, 2048 or 4096 keys takes."""
    hit = np.zeros(n, bool)
    for m in (1024, 2048, 4096):
        i = np.arange(m, dtype=np.uint64)
        h = (i * 0x9E3779B9 + np.uint64(salt)) & 0xFFFFFFFF
        h ^= h >> np.uint64(15)
        h = (h * 0x85EBCA6B) & 0xFFFFFFFF
        h ^= h >> np.uint64(13)
        hit[(i * (n // m) + ((h * (n // m)) >> np.uint64(32))).astype(np.int64)] = True
    return hit


def _off_sample(full: np.ndarray, salt: int, unseen: np.ndarray) -> np.ndarray:
    """`full` at the sampled positions, so that the sample is as of uniform keys, `unseen` elsewhere."""
    return np.where(_sampled(full.size, salt), full, unseen).astype(np.uint32)


def _full(n: int) -> np.ndarray:
    return np.random.default_rng(n).integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)


def _sorter(keys, pairs: bool):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    out = torch.empty_like(keys)
    if not pairs:
        return lambda: binding.ap_sort_u32(keys, out, 64, None)
    vals = torch.arange(keys.numel(), dtype=torch.int32, device="cuda")
    vout = torch.empty_like(vals)
    return lambda: binding.ap_sort_pairs_u32(keys, vals, out, vout, 64, None)


@pytest.mark.parametrize("n,pairs", [(100_003, False), (9 << 17, False), (5 << 17, True)])
def test_keys_off_the_known_positions_cost_no_more(n, pairs):
    """One array of a length is like another: 20 times is far above any spread (measured 1.7 at most)."""
    torch = torch_cuda()
    full = _full(n)
    cluster = np.uint32(0x70000000) + (full & np.uint32(0xFFFF))
    times = []
    for keys in (full, _off_sample(full, 0, cluster)):
        call = _sorter(to_dev(keys)[0], pairs)
        announce(f"time off the sample n={n} pairs={pairs}")
        call()
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            call()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    assert times[1] <= 20 * times[0], times


# what the unseen keys vary in: a cell of one value, two values, and one to four digits (odd and even
# numbers of sweeps), also with the type's largest key
def _unseen(full: np.ndarray, kind: str) -> np.ndarray:
    base = np.uint32(0x70000000)
    if kind == "value":
        return np.full(full.size, base + np.uint32(1), np.uint32)
    if kind == "two_values":
        return base + (full & np.uint32(1)) * np.uint32(0x10001)
    if kind == "wide":                                   # above every sampled key: the last cell
        return np.uint32(0x80000000) | full
    if kind == "largest":
        return np.uint32(0xFFFFFFFF) - (full & np.uint32(0x3FF))
    return base + (full & np.uint32({"digit": 0xFF, "digits": 0x3FFFF, "middle": 0xFF00}[kind]))


# cells near the tile of k_cells (10240 keys, 8192 pairs) and the sweeps' tile (6144), and the longest
@pytest.mark.parametrize("rank_mode", [0, 1])
@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("kind", ["value", "two_values", "digit", "digits", "middle", "largest", "wide"])
def test_off_the_salted_positions(kind, pairs, rank_mode):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    binding.ap_set_rank_mode(rank_mode)
    try:
        for n in ([9_300, 13_312, 13_313, 70_001, 5 << 17] if pairs else [16_385, 19_456, 19_457, 100_003, 9 << 17]):
            full = _full(n)
            t_in, _ = to_dev(full, n % 4)
            seen = full >> np.uint32(2) if kind == "wide" else full
            keys = _off_sample(seen, _salt(t_in.data_ptr()), _unseen(full, kind))
            t_in.copy_(torch.from_numpy(keys.view(np.int32)))
            inplace = bool(n & 1)
            t_out = t_in if inplace else torch.empty_like(t_in)
            announce(f"oversize cell n={n} {kind} pairs={pairs} rank {rank_mode}")
            for P in (64, 1000) if inplace else (64,):
                spl = torch.empty(P - 1, dtype=torch.int32, device="cuda")
                t_in.copy_(torch.from_numpy(keys.view(np.int32)))
                if pairs:
                    vals = torch.arange(n, dtype=torch.int32, device="cuda")
                    vout = vals if inplace else torch.empty_like(vals)
                    binding.ap_sort_pairs_u32(t_in, vals, t_out, vout, P, spl)
                else:
                    binding.ap_sort_u32(t_in, t_out, P, spl)
                torch.cuda.synchronize()
                want, perm = oracle.sort_pairs_u32(keys, np.arange(n, dtype=np.uint32))
                assert np.array_equal(to_host(t_out), want), n
                assert np.array_equal(to_host(spl), oracle.splitters(want, P)), n
                if pairs:
                    assert np.array_equal(to_host(vout), perm), n
    finally:
        binding.ap_set_rank_mode(0)
