"""The launch-shape table and the shapes that the tuner tries (CPU only)."""
import json

import pytest

from paper_2602_15883_amd import tune

with open(tune.SHIPPED) as f:
    TABLE = json.load(f)


@pytest.mark.parametrize("key", sorted(TABLE))
def test_an_entry_is_the_fastest_of_its_trials(key):
    e = TABLE[key]
    best = min(e["trials"], key=lambda t: t["ms"])
    assert e["ms"] == best["ms"]
    assert {k: e[k] for k in best} == best


@pytest.mark.parametrize("width", [32, 64, 100, 200])
def test_the_tuner_tries_the_library_s_own_shape(width):
    """One item range per workgroup, whatever the number of workgroups per compute unit."""
    tried = {(c["blocks_per_cu"], c["ranges_per_wg"]) for c in tune.candidates(width)}
    assert {(1, 0), (2, 1), (3, 1), (4, 1)} <= tried


@pytest.mark.parametrize("key", sorted(TABLE))
def test_an_entry_was_chosen_among_them(key):
    tried = {(t["blocks_per_cu"], t["ranges_per_wg"]) for t in TABLE[key]["trials"]}
    assert (1, 0) in tried and (2, 1) in tried
