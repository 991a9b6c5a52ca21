"""Observables do not depend on the order in which a step left the particles:
runs that differ in tiling, launches or a binning export in between hold the
same states in other slots, and return the same bits of P, E and T; the sums
are those of the returned state.
"""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

DEG = math.pi / 180.0


@pytest.fixture(scope="module")
def mpc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_15236_amd as m
    m.lib()
    return m


def boxes():
    out = []
    for k in range(12):
        out.append(dict(L=(15 + 2 * k, 14 + k, 12), h=0.1, alpha=130.0 * DEG, kT=0.7 + 0.13 * k,
                        mass=0.9 + 0.01 * k, density=10.0, seed=7 + k, mbs=True, walls=False,
                        g=(0.0, 0.0, 0.0)))
    return out


def bits(o):
    return [float(x).hex() for x in (*o["P"], o["E"], o["T"])]


@pytest.mark.parametrize("form", ["fp64", "fp32", "split"])
def test_same_bits_whatever_the_slots(mpc, form):
    """Twelve boxes of five values: sums of about 3000 to 100000 terms in slot
    order differ in the last bits of some of them from run to run."""
    bs = boxes()
    runs = {}
    print(f"case observables {form}", flush=True)
    for name in ("first", "again", "tiling", "binning", "retiled", "retiled again"):
        with mpc.Sim(bs, form=form, reorder_every=3, graph=name != "again") as sim:
            sim.init_state(5)
            if name == "tiling":
                sim.set_tiling(5, 0, 4, 1)
            sim.step(3)
            if name == "binning":
                sim.get_binning(2)
            sim.step(17)
            if name.startswith("retiled"):
                sim.set_tiling(6, 0, 8, 0)
            runs[name] = ([bits(sim.observables(k)) for k in range(len(bs))],
                          [sim.get_state(k) for k in range(len(bs))])
    for name in ("again", "tiling", "binning"):
        for k in range(len(bs)):
            for a, b in zip(runs[name][1][k], runs["first"][1][k]):
                np.testing.assert_array_equal(a, b)
        assert runs[name][0] == runs["first"][0], name
    assert runs["retiled again"][0] == runs["retiled"][0]
    if form != "fp64":
        assert runs["retiled"][0] == runs["first"][0]


def fsums(box, v):
    """P, E and T of velocities v[3][n] with every sum rounded once."""
    m, n = box["mass"], v.shape[1]
    P = np.array([math.fsum(m * v[k]) for k in range(3)])
    E = math.fsum(0.5 * m * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]))
    w = v - (P / (n * m))[:, None]
    return P, E, math.fsum(m * (w[0] * w[0] + w[1] * w[1] + w[2] * w[2])) / (3.0 * (n - 1))


@pytest.mark.parametrize("form", ["fp32", "split"])
def test_sums_are_rounded_once(mpc, form):
    """Bar: the digits cut off are below n 2^-80 of the largest term (n 2^-80 <
    2^-60 here), so a sum is its true value rounded to FP64, or beside a tie
    its neighbour: 2^-52."""
    for k, box in enumerate(boxes()[:3] + [dict(boxes()[0], L=(3, 2, 2), density=3.0)]):
        with mpc.Sim(box, form=form) as sim:
            sim.init_state(k)
            sim.step(5)
            o = sim.observables()
            _, v = sim.get_state()
        P, E, T = fsums(box, v)
        biggest = np.abs(v).max() * box["mass"]
        assert np.all(np.abs(o["P"] - P) <= 2.0**-52 * np.abs(P) + 2.0**-60 * biggest)
        assert abs(o["E"] - E) <= 2.0**-52 * E
        assert abs(o["T"] - T) <= 2.0**-51 * T  # and the division


@pytest.mark.parametrize("lo,hi", [(-60, 60), (-155, -140), (-3, 140), (100, 150)])
def test_relative_energy_over_wide_ranges(mpc, lo, hi):
    """Terms over hundreds of binary orders, the largest anywhere, down to
    squares that lose bits below the smallest normal number.  Bar as above with
    n = 3000, plus the smallest number's rounding of each term."""
    box = dict(boxes()[0], L=(10, 6, 5), mass=1.0)
    x, v = synth.box_state(box["L"], seed=3)
    rng = np.random.default_rng(hi - lo)
    v = v * 10.0 ** rng.uniform(lo, hi, size=v.shape)
    v[:, rng.integers(0, v.shape[1], size=50)] = 0.0
    with mpc.Sim(box) as sim:
        sim.set_state(x, v)
        o = sim.observables()
    n = v.shape[1]
    w = v - (o["P"] / n)[:, None]
    T = math.fsum(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]) / (3.0 * (n - 1))
    assert abs(o["T"] - T) <= 2.0**-51 * T + 2.0**-1074


def test_energy_beyond_the_range_is_refused(mpc):
    """A velocity whose square is infinite, alone in its cell."""
    box = dict(boxes()[0], L=(10, 10, 10), density=0.002, mbs=False)
    x = np.array([[2.5, 7.5], [2.5, 7.5], [2.5, 7.5]])
    for tiling in (None, (6, 0, 8, 0)):
        with mpc.Sim(box) as sim:
            sim.set_state(x, np.array([[1e200, 0.0], [0.0, 0.0], [0.0, 1.0]]))
            sim.step(1)
            if tiling:
                sim.set_tiling(*tiling)
            with pytest.raises(mpc.MPCError) as e:
                sim.observables()
            assert e.value.code == mpc.ESTATE


def test_more_tiles_than_one_launch_of_wavefronts(mpc):
    """2^26 rows of one cell: a wavefront each would be 2^32 threads, which one
    launch does not take."""
    box = dict(boxes()[0], L=(1, 8192, 8192), density=0.004, mbs=False)
    print("case observables of 2^26 rows", flush=True)
    with mpc.Sim(box) as sim:
        sim.init_state(3)
        o0 = sim.observables()
        sim.step(2)
        o1 = sim.observables()
        v = sim.get_state()[1]
    P, E, T = fsums(box, v)
    assert abs(o1["E"] - E) <= 2.0**-52 * E and abs(o1["T"] - T) <= 2.0**-51 * T
    # no thermostat: energy and momentum are kept, each by rounding of n terms
    n = v.shape[1]
    assert abs(o1["E"] - o0["E"]) < n * 2.0**-52 * E
    assert np.abs(o1["P"] - o0["P"]).max() < n * 2.0**-52 * np.abs(v).max()
