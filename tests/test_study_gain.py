"""Which run the accuracy study calls better, where a run has blown up (no GPU)."""
import math

import pytest

pytest.importorskip("torch")


def test_a_run_that_blew_up_is_not_better():
    from paper_2207_11571_amd import study
    base = {"e_max_momentum": [0.0, 1.0, 2.0, 3.0], "times": [0.0, 1.0, 2.0, 3.0], "mean_e_window": 1.0,
            "mean_e_beyond": 2.5}
    run = {"e_max_momentum": [0.0, 0.5, math.nan, math.nan], "mean_e_window": 0.5, "mean_e_beyond": math.nan}
    gain = study._gain(base, run)
    assert gain["better_than_uncorrected_until"] == 2.0
    assert math.isnan(gain["beyond_ratio"])
