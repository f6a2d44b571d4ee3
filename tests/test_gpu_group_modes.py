"""The one-wave kernel of the group engine and of the wave engine's sequential and controlled
batches against the oracle, at the sizes where its parts change: map rows at and next to 8, 16, 17
and 32 (one or two rows a lane, windows of 8 rows), rules at and next to 8 and 16 (probe windows),
pattern columns at and over 3 and 8, caps below and above the four maxima, batches on both sides
of two waves per SIMD, launches on both sides of 16 steps (lists in LDS or in memory)."""
import numpy as np
import pytest

import oracle
from ctl_util import random_control
from gpu_util import gpu_run, require_gpu, say
from paper_2407_04221_amd import inputs

pytestmark = pytest.mark.gpu


def wl(name, i, **kw):
    d = dict(B=19, C=5, p_dc=0.6, per_env=True, T=40, L=17)
    d.update(kw)
    return inputs.Workload(name, 300 + i, **d)


# (workload, variant)
CASES = [(wl(*c[:1], i, **c[1]), c[2]) for i, c in enumerate([
    ("h8", dict(H=8, W=32, R=8, shapes=((3, 3), (1, 2))), "planted"),
    ("h9", dict(H=9, W=5, R=9, shapes=((2, 2), (3, 1))), "dense"),
    ("h16", dict(H=16, W=16, R=16, shapes=((3, 3),)), "planted"),
    ("h17", dict(H=17, W=17, R=17, shapes=((1, 2), (2, 1), (3, 3))), "dense"),
    ("h32", dict(H=32, W=32, R=24, C=8, shapes=((3, 3), (1, 2)), T=20), "planted"),
    ("rare", dict(H=32, W=31, R=7, shapes=((3, 3),), p_dc=0.3), "literal"),
    ("one", dict(H=1, W=7, R=1, shapes=((1, 3),)), "dense"),
    ("none", dict(H=12, W=12, R=0, shapes=((1, 1),)), "literal"),
    ("wide", dict(H=20, W=32, R=9, shapes=((1, 16), (2, 9))), "dense"),
    ("tall", dict(H=32, W=10, R=8, shapes=((16, 1), (9, 1), (1, 1))), "dense"),
    ("five", dict(H=30, W=29, R=6, C=12, shapes=((5, 5), (4, 2)), p_dc=0.8), "planted"),
    ("many", dict(H=13, W=14, R=56, C=4, shapes=((2, 2), (1, 1)), T=20), "dense"),
    ("batch16", dict(H=16, W=11, R=6, B=2100, shapes=((3, 3), (2, 1)), T=18), "dense"),
    ("batch32", dict(H=27, W=32, R=10, B=2100, shapes=((3, 3), (1, 2)), T=18), "planted"),
])]
MODES = [("parallel", None), ("sequential", None), ("parallel", "rowmajor"),
         ("parallel", "random"), ("sequential", "random")]


@pytest.mark.parametrize("mode,order", MODES, ids=[f"{m}-{o}" for m, o in MODES])
@pytest.mark.parametrize("case", CASES, ids=[c[0].name for c in CASES])
def test_one_wave_kernel_matches_oracle(case, mode, order):
    require_gpu()
    w, variant = case
    if w.B > 100 and order == "rowmajor":
        pytest.skip("the large batches run one order")
    if order and not w.R:
        pytest.skip("no rule to control")
    say(f"[one-wave] {w.name} {mode} {order}")
    maps, rules, actions = inputs.make_all(w, 2, variant)
    control = None
    if order:
        limit, inhibit = random_control(np.random.default_rng(5), w.B, w.R, p_inh=0.1, kmax=9)
        control = (limit, inhibit, int(order == "random"), 77)
    want_m, want_r, want_d = oracle.run(w, maps, rules, actions, nthreads=8,
                                        rule_mode=int(mode == "sequential"), control=control)
    for chunk in (w.T, 3):                         # lists in LDS, lists in memory
        _, final, r, d, _ = gpu_run(w, maps, rules, actions, mode="step_n", chunk=chunk,
                                    rule_mode=mode, control=control)
        np.testing.assert_array_equal(r, want_r)
        np.testing.assert_array_equal(d, want_d)
        np.testing.assert_array_equal(final, want_m[-1])


@pytest.mark.parametrize("mode,order", MODES, ids=[f"{m}-{o}" for m, o in MODES])
@pytest.mark.parametrize("H,W,B,variant", [(16, 16, 19, "planted"), (16, 9, 19, "dense"),
                                           (32, 32, 19, "planted"), (32, 17, 19, "dense"),
                                           (31, 32, 19, "planted"), (16, 12, 2100, "planted"),
                                           (32, 11, 2100, "planted")])
def test_one_row_patterns_match_oracle(H, W, B, variant, mode, order):
    """Patterns of one row, where only the two-row built-in moves need a row above a match
    plane, on maps that fill the planes' 16 or 32 rows, with players moving on the last row."""
    require_gpu()
    if B > 100 and order == "rowmajor":
        pytest.skip("the large batches run one order")
    w = wl(f"row{H}", 40 + H + W, H=H, W=W, B=B, R=6, shapes=((1, 1), (1, 2), (1, 3)),
           T=30 if B < 100 else 18)
    say(f"[one-row patterns] {H}x{W} B={B} {variant} {mode} {order}")
    maps = inputs.make_maps(w, 3)
    g = np.random.default_rng(H * W)
    last = g.random((B, W)) < 0.3                      # more players, on the last row
    maps[:, :, H - 1] = np.where(last[:, None], np.arange(w.C)[:, None] == inputs.PLAYER,
                                 maps[:, :, H - 1])
    rules = inputs.make_rules(w, 3, variant, init_maps=maps)
    actions = inputs.make_actions(w, 3)
    control = None
    if order:
        limit, inhibit = random_control(np.random.default_rng(5), w.B, w.R, p_inh=0.1, kmax=9)
        control = (limit, inhibit, int(order == "random"), 77)
    want_m, want_r, want_d = oracle.run(w, maps, rules, actions, nthreads=8,
                                        rule_mode=int(mode == "sequential"), control=control)
    for chunk in (w.T, 3):
        _, final, r, d, _ = gpu_run(w, maps, rules, actions, mode="step_n", chunk=chunk,
                                    rule_mode=mode, control=control)
        np.testing.assert_array_equal(r, want_r)
        np.testing.assert_array_equal(d, want_d)
        np.testing.assert_array_equal(final, want_m[-1])
