"""Passes over the vocabulary at row lengths that are not a multiple of four and draft counts known / not known at compile time."""
import pytest

from paper_2601_20357_amd import synth

import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,n,policy,distance", [(1001, 1, 0, 0), (1002, 3, 0, 1), (1003, 5, 0, 0), (4099, 6, 0, 1), (2, 3, 0, 0), (3, 5, 0, 1),
                                                 (1025, 2, 2, 0), (4102, 2, 2, 1)])
def test_rounds_on_unaligned_rows(oracle, V, n, policy, distance):
    print(f"unaligned rows V={V} n={n} policy={policy} distance={distance}", flush=True)
    wl = synth.scaled(synth.WORKLOADS["serving"], V=V, d=64, n=n, B=5, gamma=3, h=4, cfg_id=160 + V % 9)
    tally = harness.run_rounds(oracle, wl, 4, synth.make_temperature(wl, "mixed07"), policy=policy, distance=distance)
    assert tally.flagged_divergences <= max(2, tally.decisions // 50)
