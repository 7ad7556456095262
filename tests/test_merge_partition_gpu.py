"""Merge at the sizes where the tile boundaries per workgroup change (16, 32, 64) and where its last
workgroup holds one boundary, equal and lopsided runs."""
from __future__ import annotations

import pytest

from tests.gpu_util import announce, torch_cuda

pytestmark = pytest.mark.gpu

T = 8192


@pytest.mark.parametrize("n", [T - 1, 15 * T, 15 * T + 1, 16 * T, (1 << 26) - 1, 1 << 26, (1 << 28) - 1, 1 << 28])
@pytest.mark.parametrize("kind", ["even", "lopsided", "apart", "equal"])
def test_boundaries(n, kind):
    torch = torch_cuda()
    from paper_cs_0004013_amd import binding
    announce(f"merge partition n={n} {kind}")
    g = torch.Generator(device="cuda").manual_seed(n)
    na = {"even": n // 2, "lopsided": n - 777, "apart": n // 3, "equal": n // 2}[kind]
    keys = torch.randint(0, 1 << 31, (n,), dtype=torch.int64, device="cuda", generator=g).to(torch.int32)
    if kind == "apart":
        keys[:na] |= 1 << 30
        keys[na:] &= (1 << 30) - 1
    if kind == "equal":
        keys.fill_(5)
    a, b = keys[:na].sort().values, keys[na:].sort().values
    out = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    binding.ap_merge_u32(a, b, out)
    assert torch.equal(out, keys.sort().values)
