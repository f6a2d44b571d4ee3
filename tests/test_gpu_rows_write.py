"""The rows engine's tall maps (four waves an environment) against the oracle where the voted
planes are dealt to the waves: fewer planes than waves up to four times as many, rows at and next
to 33 and 64, 4- and 8-byte rows, resets, launches of one step and of many; random rules, whose
steps share a match in which no rule fires."""
import numpy as np
import pytest

import oracle
from gpu_util import gpu_run, require_gpu, say
from paper_2407_04221_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [(33, 31, 4, 3, "dense"), (64, 64, 18, 24, "dense"), (63, 33, 12, 20, "planted"),
         (34, 9, 5, 9, "dense"), (48, 32, 8, 16, "planted"),
         (50, 30, 6, 24, "literal"), (64, 64, 8, 24, "literal")]


@pytest.mark.parametrize("H,W,C,R,variant", CASES)
def test_rows_four_waves_write_matches_oracle(H, W, C, R, variant):
    require_gpu()
    w = inputs.Workload(f"rows{H}", 500 + H, B=9, H=H, W=W, C=C, R=R,
                        shapes=((3, 3), (1, 2), (2, 1)), p_dc=0.7, per_env=False, T=24, L=7)
    say(f"[rows write] {H}x{W} C={C} R={R} {variant}")
    maps, rules, actions = inputs.make_all(w, 4, variant)
    want_m, want_r, want_d = oracle.run(w, maps, rules, actions, nthreads=8)
    for chunk in (w.T, 1):
        _, final, r, d, _ = gpu_run(w, maps, rules, actions, mode="step_n", chunk=chunk,
                                    engine="rows")
        np.testing.assert_array_equal(r, want_r)
        np.testing.assert_array_equal(d, want_d)
        np.testing.assert_array_equal(final, want_m[-1])
