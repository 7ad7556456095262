"""Every segmented kernel configuration through batches of the request server, which sorts requests of any
length with the length groups' kernels: requests of one tile (the tile sort at its keys-per-lane steps) and
of several, with the build of a group that also takes longer requests and with the one-tile build."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

N_CONFIGS = 12


def _batch(lens, seed: int) -> None:
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    rng = np.random.default_rng(seed)
    keys, ins, outs, spls = [], [], [], []
    for i, n in enumerate(lens):
        k = rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
        if i % 3 == 1:
            k &= np.uint32(0x00F0F000)
        if i % 7 == 2:
            k[:] = 9
        keys.append(k)
        ins.append(to_dev(k, i % 4)[0])
        outs.append(torch.empty(n, dtype=torch.int32, device="cuda"))
        spls.append(torch.empty(63, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    with binding.Server(hbm_budget_bytes=1 << 28, num_streams=1, max_batch=64, alone_min_keys=1 << 22) as srv:
        tickets = [srv.submit(a, o, 64, s) for a, o, s in zip(ins, outs, spls)]
        status = [srv.wait(t) for t in tickets]
        batches = srv.stats()["batches"]
    assert all(s == 0 for s in status)
    assert batches < len(lens)      # not one by one: those take the single-array sort
    for k, o, s in zip(keys, outs, spls):
        want = oracle.sort_u32(k)
        assert np.array_equal(to_host(o), want), k.size
        assert np.array_equal(to_host(s), oracle.splitters(want, 64)), k.size


@pytest.mark.parametrize("rank_mode", [0, 1])
@pytest.mark.parametrize("cfg", range(N_CONFIGS))
def test_every_config_in_batches(cfg, rank_mode):
    torch_cuda()
    from paper_cs_0004013_amd import binding
    _, waves, ipt = binding.ap_segmented_config_info(cfg)
    tile, cls = waves * 64 * ipt, (waves * 64 * ipt).bit_length() - 1
    steps = [tile // d + e for d in (1, 2, 4, 8) for e in (-1, 0, 1)]
    saved = binding.segmented_groups()
    binding.ap_set_rank_mode(rank_mode)
    try:
        binding.ap_segmented_set_config(cfg)
        announce(f"server batch, every group configuration {cfg}, rank {rank_mode}")
        _batch([1, 2, 3, 64, 65] + steps + [2 * tile, 3 * tile + 5] + [n for n in steps if n <= tile], cfg)
        other = 11 if cfg != 11 else 10
        binding.set_segmented_groups([(cls + 1, 31, other), (1, cls, cfg)])
        announce(f"server batch, one-tile group of configuration {cfg}, rank {rank_mode}")
        _batch([1, 2, 3, 64, 65] + [n for n in steps if n <= tile] * 2 + [tile + 1], cfg + 100)
    finally:
        binding.set_segmented_groups(saved)
        binding.ap_set_rank_mode(0)
