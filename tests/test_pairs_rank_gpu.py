"""Short and middling pairs (one launch up to 8192, two up to 5 * 2^17) with the order-agnostic rank, whose
stability only the values show, and with more cells than keys under either rank."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, to_dev, to_host, torch_cuda
from tests.test_cells_gpu import KINDS, _keys

pytestmark = pytest.mark.gpu


def _check(keys: np.ndarray, P: int, inplace: bool) -> None:
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    n = keys.size
    vals = np.arange(n, dtype=np.uint32)
    tk, tv = to_dev(keys, n % 3)[0], to_dev(vals)[0]
    ko, vo = (tk, tv) if inplace else (torch.empty_like(tk), torch.empty_like(tv))
    spl = torch.full((P - 1,), 0x1111, dtype=torch.int32, device="cuda")
    binding.ap_sort_pairs_u32(tk, tv, ko, vo, P, spl)
    torch.cuda.synchronize()
    wk, wv = oracle.sort_pairs_u32(keys, vals)
    assert np.array_equal(to_host(ko), wk) and np.array_equal(to_host(vo), wv), n
    assert np.array_equal(to_host(spl), oracle.splitters(wk, P)), n


@pytest.fixture
def mask_rank():
    from paper_cs_0004013_amd import binding
    binding.ap_set_rank_mode(1)
    yield
    binding.ap_set_rank_mode(0)


# around the workgroups of the one launch (2048, 8192), the split's shapes (48K, 200000, 400000) and the end
@pytest.mark.parametrize("kind", KINDS)
def test_order_agnostic_rank(kind, mask_rank):
    for n in [1, 2, 255, 257, 2048, 2049, 8192, 8193, 49152, 49153, 200_000, 200_001, 400_000, 400_001, 5 << 17]:
        announce(f"pairs, order-agnostic rank, n={n} {kind}")
        _check(_keys(n, kind), 64, bool(n & 1))


@pytest.mark.parametrize("rank_mode", [0, 1])
def test_more_cells_than_keys(rank_mode):
    from paper_cs_0004013_amd import binding
    binding.ap_set_rank_mode(rank_mode)
    try:
        for n in [1, 63, 2000, 8192, 8193, 20_000]:
            for P in (n + 1, 2 * n + 77):
                announce(f"pairs n={n} P={P} rank {rank_mode}")
                _check(_keys(n, "full"), P, False)
    finally:
        binding.ap_set_rank_mode(0)
