"""Mutation operators on the GPU (paper Sec. 2.2.1, Fig. 2b caption) vs the oracle: map bit
flips, pattern-entry changes and reward redraws for populations of every workload's shape
(full size), ragged element counts, masks, in-place calls, extreme thresholds and reward
ranges; and one evolution step end to end (mutate on the GPU, load, step) against the same
step built from the oracle's mutation."""
import numpy as np
import pytest

import oracle
from gpu_util import first_mismatch, require_gpu, say
import paper_2407_04221_amd as av
from paper_2407_04221_amd import inputs

pytestmark = pytest.mark.gpu


def both(**kw):
    """The same parameters as the library's av_mutation and the oracle's Mutation."""
    base = dict(seed=11, generation=2, map_flip_p32=1 << 28, map_channels=0xFFFFFFFF,
                entry_p32=1 << 29, entry_channels=0xFFFFFFFF, reward_p32=1 << 30,
                reward_lo=-3, reward_hi=4)
    base.update(kw)
    a, o = av.av_mutation(), oracle.Mutation()
    for k, v in base.items():
        setattr(a, k, v)
        setattr(o, k, v)
    return a, o


MAP_SHAPES = [(1, 4, 1, 1), (3, 5, 7, 9), (7, 31, 3, 5), (2, 6, 16, 16), (5, 8, 32, 32),
              (2, 12, 64, 64), (1, 4, 64, 63)]


@pytest.mark.parametrize("shape", MAP_SHAPES, ids=["x".join(map(str, s)) for s in MAP_SHAPES])
def test_map_mutation_matches_oracle(shape):
    require_gpu()
    import torch
    say(f"[mutate maps] {shape}")
    g = np.random.default_rng(sum(shape))
    maps = ((g.random(shape) < 0.4) * g.integers(1, 5, shape)).astype(np.uint8)
    src = torch.from_numpy(maps).cuda()
    for kw in (dict(), dict(map_channels=0b10110, generation=5), dict(map_flip_p32=0xFFFFFFFF),
               dict(map_flip_p32=0)):
        a, o = both(**kw)
        dst = torch.empty_like(src)
        av.av_mutate_maps(src, dst, a)
        np.testing.assert_array_equal(dst.cpu().numpy(), oracle.mutate_maps(maps, o))
    # in place
    a, o = both()
    inplace = src.clone()
    av.av_mutate_maps(inplace, inplace, a)
    np.testing.assert_array_equal(inplace.cpu().numpy(), oracle.mutate_maps(maps, o))


@pytest.mark.parametrize("name", ["c1", "c2", "c3", "c4", "c5"])
def test_population_maps_full_size(name):
    require_gpu()
    import torch
    wl = inputs.WORKLOADS[name]
    say(f"[mutate maps full] {name} B={wl.B}")
    maps = inputs.make_maps(wl, 0)
    a, o = both(map_flip_p32=av.p32(0.01), map_channels=~(1 << 2) & 0xFFFFFFFF)
    src = torch.from_numpy(maps).cuda()
    dst = torch.empty_like(src)
    av.av_mutate_maps(src, dst, a)
    got = dst.cpu().numpy()
    want = oracle.mutate_maps(maps, o)
    assert first_mismatch(got, want) is None
    assert (got[:, 2] == maps[:, 2]).all()                 # the player channel was masked


RULE_CASES = ["c1", "c2", "c3", "c4", "c5"]


@pytest.mark.parametrize("name", RULE_CASES)
def test_rule_mutation_matches_oracle(name):
    require_gpu()
    import torch
    wl = inputs.WORKLOADS[name]
    say(f"[mutate rules] {name}")
    shape, ip, op, rw = inputs.make_rules(wl, 1, "literal")
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (shape, ip, op, rw)]
    for kw in (dict(), dict(entry_channels=0b1001101, generation=7, entry_p32=0xFFFFFFFF),
               dict(reward_lo=-(2**31), reward_hi=2**31 - 1, reward_p32=0xFFFFFFFF),
               dict(reward_lo=9, reward_hi=9), dict(entry_p32=0, reward_p32=0)):
        a, o = both(**kw)
        out = [torch.empty_like(x) for x in dev[1:]]
        av.av_mutate_rules(dev[0], dev[1], dev[2], dev[3], *out, a)
        want = oracle.mutate_rules(shape, ip, op, rw, o)
        for g_, w_ in zip(out, want):
            np.testing.assert_array_equal(g_.cpu().numpy(), w_)
    # in place
    a, o = both()
    av.av_mutate_rules(dev[0], dev[1], dev[2], dev[3], dev[1], dev[2], dev[3], a)
    want = oracle.mutate_rules(shape, ip, op, rw, o)
    for g_, w_ in zip(dev[1:], want):
        np.testing.assert_array_equal(g_.cpu().numpy(), w_)


def test_evolution_step_end_to_end():
    """Mutate a c2 population (per-environment rules and maps) on the GPU, load it and step
    it; the same with the oracle's mutation on the CPU gives the same trajectory."""
    require_gpu()
    import torch
    wl = inputs.WORKLOADS["c2"].with_(B=64, T=12, L=20)
    maps, (shape, ip, op, rw), actions = inputs.make_all(wl, 2, "planted")
    a, o = both(map_flip_p32=av.p32(0.02), map_channels=0b111011, entry_p32=av.p32(0.05),
                reward_p32=av.p32(0.2), reward_lo=-1, reward_hi=1)
    dmaps = torch.from_numpy(maps).cuda()
    av.av_mutate_maps(dmaps, dmaps, a)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (shape, ip, op, rw)]
    av.av_mutate_rules(*dev, dev[1], dev[2], dev[3], a)
    rules_gpu = (shape, dev[1].cpu().numpy(), dev[2].cpu().numpy(), dev[3].cpu().numpy())
    maps_o = oracle.mutate_maps(maps, o)
    rules_o = (shape,) + oracle.mutate_rules(shape, ip, op, rw, o)
    for x, y in zip(rules_gpu, rules_o):
        np.testing.assert_array_equal(x, y)
    want_m, want_r, want_d = oracle.run(wl, maps_o, rules_o, actions)
    b = av.Batch.for_workload(wl)
    try:
        b.load_rules(*rules_gpu)
        b.reset(dmaps)
        acts = torch.from_numpy(actions).cuda()
        for t in range(wl.T):
            r, d = b.step(acts[t])
            np.testing.assert_array_equal(b.maps().cpu().numpy(), want_m[t])
            np.testing.assert_array_equal(r.cpu().numpy(), want_r[t])
            np.testing.assert_array_equal(d.cpu().numpy(), want_d[t])
    finally:
        b.close()


@pytest.mark.parametrize("per", [1920, 2040, 2048, 2050, 4096])
@pytest.mark.parametrize("shift", [0, 3])
def test_map_mutation_rows_and_alignment(per, shift):
    """Individuals around whole workgroups of 256 blocks of eight cells (a grid row each, or
    packed), at addresses that are no multiple of eight."""
    require_gpu()
    import torch
    C = {1920: 4, 2040: 5, 2048: 4, 2050: 5, 4096: 4}[per]
    H, W = {1920: (20, 24), 2040: (12, 34), 2048: (16, 32), 2050: (10, 41), 4096: (32, 32)}[per]
    assert C * H * W == per
    n = 5
    maps = np.random.default_rng(per).integers(0, 3, (n, C, H, W)).astype(np.uint8)
    src = torch.zeros(n * per + shift, dtype=torch.uint8, device="cuda")[shift:].view(n, C, H, W)
    src.copy_(torch.from_numpy(maps))
    dst = torch.zeros(n * per + 8, dtype=torch.uint8, device="cuda")
    for kw in (dict(), dict(map_channels=0b0110)):
        a, o = both(**kw)
        av.av_mutate_maps(src, dst[shift:shift + n * per].view(n, C, H, W), a)
        np.testing.assert_array_equal(dst[shift:shift + n * per].cpu().numpy().reshape(maps.shape),
                                      oracle.mutate_maps(maps, o))
        assert not dst[:shift].any() and not dst[shift + n * per:].any()


@pytest.mark.parametrize("R,C,mh,mw", [(1, 4, 1, 1), (5, 4, 1, 3), (3, 6, 3, 1), (7, 31, 16, 16),
                                       (2, 4, 5, 5)])
def test_rule_mutation_pattern_shapes(R, C, mh, mw):
    """Patterns whose entries are not a multiple of four, down to a single cell, and the largest."""
    require_gpu()
    import torch
    g = np.random.default_rng(R * mh + mw)
    S = 3
    shape = np.stack([g.integers(1, mh + 1, (S, R)), g.integers(1, mw + 1, (S, R))], -1)
    shape = shape.astype(np.int32)
    ip, op = (g.integers(-1, 2, (S, R, C + 1, mh, mw)).astype(np.int8) for _ in range(2))
    rw = g.integers(-9, 9, (S, R)).astype(np.int32)
    dev = [torch.from_numpy(x).cuda() for x in (shape, ip, op, rw)]
    for kw in (dict(entry_p32=0xC0000000), dict(entry_channels=0b101, entry_p32=0xFFFFFFFF)):
        a, o = both(**kw)
        out = [torch.empty_like(x) for x in dev[1:]]
        av.av_mutate_rules(*dev, *out, a)
        for g_, w_ in zip(out, oracle.mutate_rules(shape, ip, op, rw, o)):
            np.testing.assert_array_equal(g_.cpu().numpy(), w_)
