"""Performance cases of the sorting library: the calls that its users make, over the range of sizes,
distributions and forms that it is used at.

A case is a dict of plain values.  ``prepare`` makes what a program holds before the call (device
buffers filled from the seed, workspaces that the program would keep, the request server), ``run``
makes one pass through the public entry points and returns the whole output, ``work`` gives the
bytes that no implementation can avoid, and ``exact`` the expected output from torch alone.

Forms
  sort      ap_sort_u32: one array into another, 64 cells, 63 splitters
  pairs     ap_sort_pairs_u32: keys with the values 0..n-1 (the stable argsort)
  segments  ap_sort_u32_segmented: many independent arrays of one buffer, in place; the program
            keeps its unsorted keys, so the pass copies them into the buffer that is sorted
  merge     ap_merge_u32: two sorted runs of different lengths
  served    a burst of requests of mixed sizes handed to the request server, waited for

Key distributions (31-bit keys unless said otherwise): "a" uniform; "c" one value; "d" 32 Gaussians
(70%) over a uniform background; "e" 16 narrow bands; "f" uniform over all 32 bits; "m" segments
that draw one of a, c, d, e each.
"""
from __future__ import annotations

import math
import random

import torch

from paper_cs_0004013_amd import binding

CELLS = 64
KEY_END = 1 << 31


def listed():
    return [
        # the smallest requests that the server sees (2^10 keys): latency of one call
        {"name": "sort_1k", "form": "sort", "n": 1024, "dist": "a"},
        # a short array of clustered keys, ragged: still one workgroup's work
        {"name": "sort_12k", "form": "sort", "n": 12345, "dist": "d"},
        # the middle of the served sizes (log-uniform from 2^10 to 2^24): too long for one
        # workgroup, far too short to fill the device
        {"name": "sort_100k", "form": "sort", "n": 100003, "dist": "a"},
        # the plain 2^20-key sort
        {"name": "sort_1m", "form": "sort", "n": 1 << 20, "dist": "a"},
        # a served request near the upper end, keys in narrow bands (long runs of equal digits)
        {"name": "sort_6m_bands", "form": "sort", "n": 6000011, "dist": "e"},
        # the 64M-key sort of the contest, uniform keys
        {"name": "sort_64m", "form": "sort", "n": 1 << 26, "dist": "a"},
        # argsort of an ordinary, ragged array
        {"name": "pairs_300k", "form": "pairs", "n": 300007, "dist": "d"},
        # argsort of a large array
        {"name": "pairs_30m", "form": "pairs", "n": 30000001, "dist": "a"},
        # the 4096-array batch: lengths log-uniform from 64 to 2^18, a distribution each
        {"name": "segments_4096", "form": "segments", "nseg": 4096, "lo": 64, "hi": 1 << 18, "dist": "m"},
        # a batch of short arrays (rows of a sparse matrix, small buckets)
        {"name": "segments_short", "form": "segments", "nseg": 16384, "lo": 16, "hi": 4096, "dist": "f"},
        # two long sorted runs of different lengths into one
        {"name": "merge_60m", "form": "merge", "n": 36700163, "n2": 23068673, "dist": "a"},
        # requests that arrive together, sizes as in the serving loop
        {"name": "served_burst", "form": "served", "requests": 96, "lo": 1 << 10, "hi": 1 << 20, "dist": "a"},
    ]


def _log_size(rng: random.Random, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng: random.Random):
    form = rng.choice(["sort", "sort", "sort", "pairs", "pairs", "segments", "segments", "merge", "served"])
    if form == "sort":
        return {"form": form, "n": _log_size(rng, 1 << 10, 1 << 26), "dist": rng.choice("aacdef")}
    if form == "pairs":
        return {"form": form, "n": _log_size(rng, 1 << 10, 30000001), "dist": rng.choice("adef")}
    if form == "segments":
        lo = _log_size(rng, 1, 512)
        hi = _log_size(rng, 8 * lo, 1 << 18)
        # as many arrays as keep the batch below the listed one's keys
        most = min(32768, int(1.2e8 * math.log(hi / lo) / (hi - lo)))
        return {"form": form, "nseg": _log_size(rng, 64, max(64, most)), "lo": lo, "hi": hi,
                "dist": rng.choice("mmafe")}
    if form == "merge":
        return {"form": form, "n": _log_size(rng, 1 << 10, 36700163), "n2": _log_size(rng, 1 << 10, 23068673),
                "dist": rng.choice("ade")}
    return {"form": form, "requests": rng.randint(8, 96), "lo": 1 << 10, "hi": _log_size(rng, 1 << 14, 1 << 20),
            "dist": rng.choice("ade")}


# ---------------------------------------------------------------- sizes that follow from a case
# Lengths belong to the case, not to the seed: every seed's inputs have the same sizes, as the
# repeated calls of one program have.
def _segment_lengths(case) -> list[int]:
    rng = random.Random(case["nseg"] * 1000003 + case["lo"] * 31 + case["hi"])
    return [_log_size(rng, case["lo"], case["hi"]) for _ in range(case["nseg"])]


def _request_sizes(case) -> list[int]:
    rng = random.Random(case["requests"] * 7919 + case["hi"])
    return [_log_size(rng, case["lo"], case["hi"]) for _ in range(case["requests"])]


def _request_places(case) -> tuple[list[int], int]:
    """Where each request's output starts in the burst's output buffer (256-byte steps), and the
    buffer's size; the words between two outputs stay zero."""
    at, total = [], 0
    for n in _request_sizes(case):
        at.append(total)
        total += -(-n // 64) * 64
    return at, total


# ---------------------------------------------------------------- inputs
def _generator(seed: int) -> torch.Generator:
    return torch.Generator(device="cuda").manual_seed(seed)


def _keys(n: int, dist: str, g: torch.Generator) -> torch.Tensor:
    """n keys of a distribution as an int32 tensor of their bits."""
    dev = "cuda"
    if dist == "f":
        return torch.randint(-KEY_END, KEY_END, (n,), generator=g, device=dev, dtype=torch.int32)
    if dist == "c":
        return torch.randint(0, KEY_END, (1,), generator=g, device=dev, dtype=torch.int32).expand(n).contiguous()
    if dist == "d":
        centres = torch.randint(0, KEY_END, (32,), generator=g, device=dev)
        pick = torch.randint(0, 32, (n,), generator=g, device=dev)
        off = (torch.randn(n, generator=g, device=dev) * float(1 << 20)).long()
        near = (centres[pick] + off).clamp_(0, KEY_END - 1).to(torch.int32)
        uni = torch.randint(0, KEY_END, (n,), generator=g, device=dev, dtype=torch.int32)
        return torch.where(torch.rand(n, generator=g, device=dev) < 0.7, near, uni)
    if dist == "e":
        centres = torch.randint(128, KEY_END - 128, (16,), generator=g, device=dev)
        pick = torch.randint(0, 16, (n,), generator=g, device=dev)
        return (centres[pick] + torch.randint(-128, 128, (n,), generator=g, device=dev)).to(torch.int32)
    return torch.randint(0, KEY_END, (n,), generator=g, device=dev, dtype=torch.int32)


def _segment_keys(lengths: list[int], dist: str, g: torch.Generator) -> torch.Tensor:
    n = sum(lengths)
    if dist != "m":
        return _keys(n, dist, g)
    nseg = len(lengths)
    kind = torch.randint(0, 5, (nseg,), generator=g, device="cuda")
    seg = torch.repeat_interleave(torch.arange(nseg, device="cuda"), torch.tensor(lengths, device="cuda"))
    kind = kind[seg]                                  # 0, 1: uniform; 2: constant; 3: Gaussians; 4: bands
    centres = torch.randint(128, KEY_END - 128, (nseg, 32), generator=g, device="cuda").view(-1)
    pick = torch.randint(0, 32, (n,), generator=g, device="cuda")
    pick = torch.where(kind == 2, 0, torch.where(kind == 4, pick & 15, pick))
    base = centres[seg * 32 + pick]
    del seg, pick
    gauss = (torch.randn(n, generator=g, device="cuda") * float(1 << 20)).long()
    gauss = torch.where(kind == 3, gauss, 0)
    band = torch.where(kind == 4, torch.randint(-128, 128, (n,), generator=g, device="cuda"), 0)
    near = (base + gauss + band).clamp_(0, KEY_END - 1).to(torch.int32)
    del base, gauss, band
    uni = torch.randint(0, KEY_END, (n,), generator=g, device="cuda", dtype=torch.int32)
    mixed = (kind == 3) & (torch.rand(n, generator=g, device="cuda") >= 0.7)
    return torch.where((kind < 2) | mixed, uni, near)


def _unsigned(keys: torch.Tensor) -> torch.Tensor:
    return keys.to(torch.int64) & 0xFFFFFFFF


def _bits(values: torch.Tensor) -> torch.Tensor:
    """int64 values below 2^32 back to the int32 tensor with their bits."""
    return torch.where(values >= KEY_END, values - (1 << 32), values).to(torch.int32)


def _inputs(case, seed: int) -> dict:
    """The call's inputs alone, from the seed."""
    g = _generator(seed)
    form = case["form"]
    if form == "sort":
        return {"keys": _keys(case["n"], case["dist"], g)}
    if form == "pairs":
        return {"keys": _keys(case["n"], case["dist"], g),
                "vals": torch.arange(case["n"], dtype=torch.int32, device="cuda")}
    if form == "segments":
        lengths = _segment_lengths(case)
        off = torch.zeros(len(lengths) + 1, dtype=torch.int64)
        off[1:] = torch.cumsum(torch.tensor(lengths), 0)
        return {"keys": _segment_keys(lengths, case["dist"], g), "offsets": off.to(torch.int32).to("cuda")}
    if form == "merge":
        return {"a": _bits(torch.sort(_unsigned(_keys(case["n"], case["dist"], g))).values),
                "b": _bits(torch.sort(_unsigned(_keys(case["n2"], case["dist"], g))).values)}
    return {"reqs": [_keys(n, case["dist"], g) for n in _request_sizes(case)]}


def prepare(case, seed: int) -> dict:
    st = _inputs(case, seed)
    form = case["form"]
    st["form"] = form
    if form in ("sort", "pairs"):
        st["out"] = torch.empty_like(st["keys"])
        st["spl"] = torch.empty(CELLS - 1, dtype=torch.int32, device="cuda")
        if form == "pairs":
            st["vout"] = torch.empty_like(st["vals"])
    elif form == "segments":
        st["work"] = torch.empty_like(st["keys"])
        st["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    elif form == "merge":
        st["out"] = torch.empty(case["n"] + case["n2"], dtype=torch.int32, device="cuda")
    else:
        st["server"] = binding.Server(hbm_budget_bytes=1 << 28)
        at, total = _request_places(case)
        st["out"] = torch.zeros(total, dtype=torch.int32, device="cuda")
        st["outs"] = [st["out"][a:a + k.numel()] for a, k in zip(at, st["reqs"])]
        st["spl"] = torch.empty((len(at), CELLS - 1), dtype=torch.int32, device="cuda")
        st["spls"] = list(st["spl"])
    # the server works on streams of its own: its requests' keys have to be there
    torch.cuda.synchronize()
    return st


def run(st):
    form = st["form"]
    if form == "sort":
        binding.ap_sort_u32(st["keys"], st["out"], CELLS, st["spl"])
        return st["out"], st["spl"]
    if form == "pairs":
        binding.ap_sort_pairs_u32(st["keys"], st["vals"], st["out"], st["vout"], CELLS, st["spl"])
        return st["out"], st["vout"], st["spl"]
    if form == "segments":
        st["work"].copy_(st["keys"])
        binding.ap_sort_u32_segmented(st["work"], st["offsets"], st["status"])
        return st["work"], st["status"]
    if form == "merge":
        binding.ap_merge_u32(st["a"], st["b"], st["out"])
        return st["out"]
    server = st["server"]
    tickets = [server.submit(k, o, CELLS, s) for k, o, s in zip(st["reqs"], st["outs"], st["spls"])]
    for t in tickets:
        server.wait(t)
    return st["out"], st["spl"]


def work(case) -> dict:
    form = case["form"]
    if form == "sort":
        nbytes = 8 * case["n"]
    elif form == "pairs":
        nbytes = 16 * case["n"]
    elif form == "segments":
        # one read and one write for the copy of the unsorted keys, one of each for the sort
        nbytes = 16 * sum(_segment_lengths(case)) + 4 * case["nseg"]
    elif form == "merge":
        nbytes = 8 * (case["n"] + case["n2"])
    else:
        nbytes = 8 * sum(_request_sizes(case))
    return {"bytes": nbytes, "flops": 0}


def _splitters(sorted_keys: torch.Tensor) -> torch.Tensor:
    """First key of cells 1..63: n keys over 64 cells, lower cells taking one key more."""
    n = sorted_keys.numel()
    p = torch.arange(1, CELLS, device=sorted_keys.device)
    start = p * (n // CELLS) + torch.clamp(p, max=n % CELLS)
    return sorted_keys[start]


def exact(case, seed: int):
    x = _inputs(case, seed)
    form = case["form"]
    if form == "sort":
        out = torch.sort(_unsigned(x["keys"])).values
        return _bits(out), _bits(_splitters(out))
    if form == "pairs":
        out, perm = torch.sort(_unsigned(x["keys"]), stable=True)
        return _bits(out), x["vals"][perm], _bits(_splitters(out))
    if form == "segments":
        lengths = torch.tensor(_segment_lengths(case), device="cuda")
        seg = torch.repeat_interleave(torch.arange(lengths.numel(), device="cuda"), lengths)
        out = torch.sort((seg << 32) | _unsigned(x["keys"])).values & 0xFFFFFFFF
        return _bits(out), torch.zeros(1, dtype=torch.int32, device="cuda")
    if form == "merge":
        return _bits(torch.sort(torch.cat([_unsigned(x["a"]), _unsigned(x["b"])])).values)
    at, total = _request_places(case)
    out = torch.zeros(total, dtype=torch.int32, device="cuda")
    spl = torch.empty((len(at), CELLS - 1), dtype=torch.int32, device="cuda")
    for i, k in enumerate(x["reqs"]):
        s = torch.sort(_unsigned(k)).values
        out[at[i]:at[i] + s.numel()] = _bits(s)
        spl[i] = _bits(_splitters(s))
    return out, spl
