"""The device-wide digit passes at the sizes that the one- and two-launch sorts take over by default, reached
by a forced tile shape (ap_set_pass_shape), and captured into a graph at a size that takes them by itself."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_cs_0004013_amd import inputs
from tests.gpu_util import announce, gpu_sort, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture
def settings():
    """(shape, rank mode) for the process, restored afterwards."""
    from paper_cs_0004013_amd import binding

    def use(shape: int, rank_mode: int) -> None:
        binding.ap_set_pass_shape(shape)
        binding.ap_set_rank_mode(rank_mode)

    yield use
    binding.ap_set_pass_shape(-1)
    binding.ap_set_rank_mode(0)


def _keys(n: int, kind: str) -> np.ndarray:
    full = np.random.default_rng(n).integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32)
    return {"full": full, "three_digits": full >> np.uint32(8), "one_digit": full & np.uint32(0xFF00),
            "constant": np.full(n, 77, np.uint32), "bands": inputs.dist_keys("e", n, np.random.default_rng(n))}[kind]


def _check(keys: np.ndarray, P: int, **kw) -> None:
    out, spl = gpu_sort(keys, P, **kw)
    want = oracle.sort_u32(keys)
    assert np.array_equal(out, want), (keys.size, P, kw)
    assert np.array_equal(spl, oracle.splitters(want, P)), (keys.size, P, kw)


@pytest.mark.parametrize("rank_mode", [0, 1])
@pytest.mark.parametrize("shape", [0, 1, 2, 3])
@pytest.mark.parametrize("kind", ["full", "three_digits", "one_digit", "constant", "bands"])
def test_forced_passes(settings, kind, shape, rank_mode):
    """Tiny arrays, tile edges, in place with an odd number of passes (which ends with a copy), keys without a
    varying digit, more cells than keys."""
    torch_cuda()
    settings(shape, rank_mode)
    for n in [1, 2, 63, 1000, 4096, 4097, 12_345, 16_384, 65_537, 70_001, (1 << 19) + 3]:
        keys = _keys(n, kind)
        announce(f"forced passes shape {shape} rank {rank_mode} n={n} {kind}")
        _check(keys, 64, pad_front=n % 4)
        _check(keys, 5, inplace=True)
        if n <= 16_384:
            _check(keys, n + 1)


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("kind", ["full", "three_digits", "constant"])
def test_forced_passes_caller_workspace(settings, kind, pairs):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    settings(1, 0)
    sizes = (300_000, 5, 16_384, 8192)
    bytes_for = binding.ap_sort_pairs_workspace_bytes if pairs else binding.ap_sort_workspace_bytes
    ws = torch.empty(max(bytes_for(n) for n in sizes), dtype=torch.uint8, device="cuda")
    binding.ap_workspace_init(ws)
    for n in sizes:
        keys = _keys(n, kind)
        vals = np.arange(n, dtype=np.uint32)
        announce(f"forced passes, caller's workspace, n={n} {kind} pairs={pairs}")
        t_in, t_out = to_dev(keys)[0], to_dev(keys)[0]
        spl = torch.empty(63, dtype=torch.int32, device="cuda")
        if pairs:
            v_in, v_out = to_dev(vals)[0], to_dev(vals)[0]
            binding.ap_sort_pairs_u32_ws(t_in, v_in, t_out, v_out, 64, spl, ws)
        else:
            binding.ap_sort_u32_ws(t_in, t_out, 64, spl, ws)
        torch.cuda.synchronize()
        wk, wv = oracle.sort_pairs_u32(keys, vals)
        assert np.array_equal(to_host(t_out), wk) and np.array_equal(to_host(spl), oracle.splitters(wk, 64)), n
        assert not pairs or np.array_equal(to_host(v_out), wv), n


@pytest.mark.parametrize("kind", ["full", "three_digits", "constant"])
def test_forced_passes_noalloc(settings, kind):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    settings(0, 0)
    for n in [70_001, 9000, 3]:
        keys = _keys(n, kind)
        announce(f"forced passes, no allocation, n={n} {kind}")
        t, _ = to_dev(keys)
        spl = torch.empty(6, dtype=torch.int32, device="cuda")
        binding.ap_sort_u32_noalloc(t, t, 7, spl)
        torch.cuda.synchronize()
        want = oracle.sort_u32(keys)
        assert np.array_equal(to_host(t), want) and np.array_equal(to_host(spl), oracle.splitters(want, 7)), n


@pytest.mark.parametrize("pairs", [False, True])
def test_passes_captured_and_replayed(pairs):
    """The histogram's self-clearing counters and the passes' look-back words, over several replays with other
    keys and eager work in between."""
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    n = (9 << 17) + 333
    announce(f"digit passes captured, n={n} pairs={pairs}")
    nbytes = binding.ap_sort_pairs_workspace_bytes(n) if pairs else binding.ap_sort_workspace_bytes(n)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    binding.ap_workspace_init(ws)
    t_in = torch.zeros(n, dtype=torch.int32, device="cuda")
    v_in = torch.arange(n, dtype=torch.int32, device="cuda")
    t_out, v_out = torch.empty_like(t_in), torch.empty_like(v_in)
    spl = torch.empty(63, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        if pairs:
            binding.ap_sort_pairs_u32_ws(t_in, v_in, t_out, v_out, 64, spl, ws, stream=s)
        else:
            binding.ap_sort_u32_ws(t_in, t_out, 64, spl, ws, stream=s)
    for rep, kind in enumerate(["full", "bands", "constant", "three_digits", "full"]):
        keys = _keys(n, kind)
        t_in.copy_(to_dev(keys)[0])
        t_out.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        wk, wv = oracle.sort_pairs_u32(keys, np.arange(n, dtype=np.uint32))
        assert np.array_equal(to_host(t_out), wk), f"replay {rep}"
        assert np.array_equal(to_host(spl), oracle.splitters(wk, 64)), f"replay {rep}"
        assert not pairs or np.array_equal(to_host(v_out), wv), f"replay {rep}"
