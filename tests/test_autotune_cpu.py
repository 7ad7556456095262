"""The tuner's descent over configurations, with made-up times: it finds the best configuration of every
group whose segments the tuning batches run through the group's kernel, and leaves the others alone."""
from __future__ import annotations

import random

from paper_cs_0004013_amd import autotune

NCFG = 12


def test_finds_the_best_of_the_measured_groups():
    best = [7, 3]

    def measure(choice):
        return 10.0 + sum(abs(c - b) for c, b in zip(choice, best))

    assert autotune.descend(measure, NCFG, rounds=2) == best + autotune.START[2:]


def test_noise_does_not_choose_for_groups_that_no_segment_runs():
    rng = random.Random(1)

    def measure(choice):          # 5% of noise, no effect of any choice
        return 10.0 * (1.0 + 0.05 * rng.random())

    for _ in range(20):
        chosen = autotune.descend(measure, NCFG, rounds=2)
        for (lo, hi), cfg, start in zip(autotune.GROUPS, chosen, autotune.START):
            if hi <= autotune.TILE_CLASS:
                assert cfg == start, (lo, hi)


def test_every_class_in_one_group():
    classes = sorted(c for lo, hi in autotune.GROUPS for c in range(lo, hi + 1))
    assert classes == list(range(1, 32))
    assert all((lo > autotune.TILE_CLASS) == (hi > autotune.TILE_CLASS) for lo, hi in autotune.GROUPS)
