"""The two-launch sort of middling arrays (split into cells, then one workgroup per cell) at the
edges of its shapes, on keys that make its cells uneven: few values, long runs of one value, narrow
bands, and keys that its sample does not see; and the one-launch sort of short pairs."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_cs_0004013_amd import inputs
from tests.gpu_util import announce, gpu_sort, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

# shape bounds (48K, 200000, 400000, 9 * 2^17 keys, 10 * 2^16 pairs), tile edges (2048, 4096, 8192), the one-launch
# limits (16384 keys, 8192 pairs)
SIZES = [16385, 2048 * 9, 2048 * 9 + 1, 49152, 49153, 200000, 200001, 400000, 400001, 8192 * 128 - 1, 9 << 17, (9 << 17) + 1]


def _sampled(n: int) -> np.ndarray:
    """Mask of the positions that a sample of 1024, 2048 or 4096 keys takes (sample_pos)."""
    hit = np.zeros(n, bool)
    for m in (1024, 2048, 4096):
        if n < m:
            continue
        i = np.arange(m, dtype=np.uint64)
        h = (i * 0x9E3779B9) & 0xFFFFFFFF
        h ^= h >> np.uint64(15)
        h = (h * 0x85EBCA6B) & 0xFFFFFFFF
        h ^= h >> np.uint64(13)
        hit[(i * (n // m) + ((h * (n // m)) >> np.uint64(32))).astype(np.int64)] = True
    return hit


def _keys(n: int, kind: str) -> np.ndarray:
    rng = np.random.default_rng(n)
    full = rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
    if kind == "full":
        return full
    if kind == "bands":
        return inputs.dist_keys("e", n, rng)
    if kind == "few":                                    # 5 values, one of them the largest key
        return np.array([0, 7, 1 << 20, 1 << 31, 0xFFFFFFFF], np.uint32)[rng.integers(0, 5, n)]
    if kind == "bytes":
        return (full & np.uint32(0xFF)) + np.uint32(1 << 16)
    if kind == "half_one_value":
        return np.where(rng.random(n) < 0.5, np.uint32(0x40000000), full)
    if kind == "sorted":
        return np.sort(full)
    if kind == "equal":
        return np.full(n, 123456789, np.uint32)
    hit = _sampled(n)                                    # what the sample misses
    if kind == "unseen_cluster":
        return np.where(hit, full, np.uint32(0x70000000) + (full & np.uint32(0xFFFF)))
    return np.where(hit, full, np.uint32(0x70000001))    # unseen_value


KINDS = ["full", "bands", "few", "bytes", "half_one_value", "sorted", "equal", "unseen_cluster", "unseen_value"]


@pytest.mark.parametrize("rank_mode", [0, 1])
@pytest.mark.parametrize("kind", KINDS)
def test_sizes_and_kinds(kind, rank_mode):
    torch_cuda()
    from paper_cs_0004013_amd import binding
    binding.ap_set_rank_mode(rank_mode)
    try:
        for n in SIZES:
            if kind.startswith("unseen") and n > 400001 and rank_mode:
                continue
            keys = _keys(n, kind)
            announce(f"cells n={n} {kind} rank {rank_mode}")
            out, spl = gpu_sort(keys, 64, inplace=bool(n & 1), pad_front=n % 4)
            want = oracle.sort_u32(keys)
            assert np.array_equal(out, want), n
            assert np.array_equal(spl, oracle.splitters(want, 64)), n
    finally:
        binding.ap_set_rank_mode(0)


@pytest.mark.parametrize("P", [1, 2, 1000, 20000, 20001, 30000])
def test_cell_counts(P):
    keys = _keys(20000, "full")
    out, spl = gpu_sort(keys, P)
    want = oracle.sort_u32(keys)
    assert np.array_equal(out, want) and np.array_equal(spl, oracle.splitters(want, P))


@pytest.mark.parametrize("kind", KINDS)
def test_pairs(kind):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    for n in [1, 255, 257, 2048, 2049, 4097, 8192, 8193, 49153, 200001, 400001, 10 << 16, (10 << 16) + 1]:
        keys = _keys(n, kind)
        vals = np.arange(n, dtype=np.uint32)
        announce(f"cells pairs n={n} {kind}")
        tk, tv = to_dev(keys, n % 3)[0], to_dev(vals)[0]
        ko, vo = (tk, tv) if n & 1 else (torch.empty_like(tk), torch.empty_like(tv))
        spl = torch.empty(63, dtype=torch.int32, device="cuda")
        binding.ap_sort_pairs_u32(tk, tv, ko, vo, 64, spl)
        torch.cuda.synchronize()
        wk, wv = oracle.sort_pairs_u32(keys, vals)
        assert np.array_equal(to_host(ko), wk) and np.array_equal(to_host(vo), wv), n
        assert np.array_equal(to_host(spl), oracle.splitters(wk, 64)), n
