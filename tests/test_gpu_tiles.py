"""Tile run lists, tiles of several passes and the thermostat's attempt chains
against the oracle: multi-step runs at the sizes where these paths branch.

Bar: positions and velocities within 1e-11 of the oracle run, ten times the
one-step FP64 bar of 1e-12 for at most six steps.
"""
import math

import numpy as np
import pytest

import oracle as orc
import synth

DEG = math.pi / 180.0


def box_of(L, **kw):
    b = dict(L=tuple(L), h=0.1, alpha=130.0 * DEG, kT=1.0, mass=1.0, density=10.0, seed=7,
             mbs=True, walls=False, g=(0.0, 0.0, 0.0))
    b.update(kw)
    return b


def oparams(box):
    return orc.Params(**{k: v for k, v in box.items()})


@pytest.fixture(scope="module")
def mpc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_15236_amd as m
    m.lib()
    return m


CASES = {
    # few particles per cell: many first attempts of the gamma draw rejected
    "sparse": (box_of((18, 17, 16), density=2.5), 0, None),
    # cells of about 60: tiles of three or four cells, some of two passes
    "dense": (box_of((10, 9, 8), density=60.0), 2, None),
    # one cell per tile, of about 200 particles
    "one_cell_tiles": (box_of((5, 4, 4), density=200.0), 0, None),
    # tiles of 32 cells: every tile needs two passes
    "two_passes": (box_of((64, 6, 5)), 3, (32, 0, 0, 0)),
    # the shortest tiles, run tables shorter than the usual number of runs
    "short_tables": (box_of((61, 7, 5)), 0, (4, 0, 0, 1)),
    # several cells a step: hundreds of runs a tile (chains)
    "fast": (box_of((48, 14, 12), kT=225.0), 2, None),
    # sheared faces: particles far from their tile's rows share a destination
    "shear": (box_of((45, 8, 6), le_u=1.7), 0, None),
    "walls": (box_of((37, 6, 5), walls=True, g=(1e-3, 0.0, 0.0)), 0, None),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_steps_match_oracle(mpc, name):
    box, R, tiling = CASES[name]
    steps, t0 = 6, 11
    x, v = synth.box_state(box["L"], density=box["density"], kT=box["kT"], seed=3)
    print(f"case {name}", flush=True)
    with mpc.Sim(box, form="fp64", reorder_every=R) as sim:
        if tiling:
            sim.set_tiling(*tiling)
        sim.set_state(x, v)
        sim.set_step(t0)
        sim.step(steps)
        xg, vg = sim.get_state()
    p = oparams(box)
    xo, vo = x.copy(), v.copy()
    for t in range(t0, t0 + steps):
        xo, vo = orc.step(p, t, xo, vo, reorder=R > 0 and (t + 1) % R == 0)
    L = np.array(box["L"], dtype=float)[:, None]
    dx = np.abs(xg - xo)
    dx = np.minimum(dx, L - dx)
    e = np.linalg.norm(vg - vo, axis=0) / np.maximum(np.linalg.norm(vo, axis=0),
                                                     math.sqrt(box["kT"]))
    print(f"{name}: max |dx| = {dx.max():.2e}, max e = {e.max():.2e}")
    assert dx.max() < 1e-11 * max(1.0, math.sqrt(box["kT"])) and e.max() < 1e-11


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["fp64", "split"])
def test_binning_export_between_steps(mpc, form):
    """The export takes the run lists' memory; the run goes on unchanged."""
    box = box_of((23, 9, 8))
    x, v = synth.box_state(box["L"], seed=5)
    with mpc.Sim([box, box], form=form, reorder_every=4) as a, \
            mpc.Sim([box, box], form=form, reorder_every=4) as b:
        for sim in (a, b):
            for k in range(2):
                sim.set_state(x, v, k)
        a.step(7)
        b.step(3)
        first = [b.get_binning(k) for k in range(2)]
        again = [b.get_binning(k) for k in range(2)]
        b.step(4)
        for p, q in zip(first, again):
            for u, w in zip(p, q):
                np.testing.assert_array_equal(u, w)
        for k in range(2):
            for u, w in zip(a.get_state(k), b.get_state(k)):
                np.testing.assert_array_equal(u, w)
            for u, w in zip(a.get_binning(k), b.get_binning(k)):
                np.testing.assert_array_equal(u, w)


def test_gamma_acceptance_rises_with_the_particle_count():
    """What the attempt chains rest on: an attempt (z, log u) accepted for n
    particles is accepted for every larger n, in the kernels' arithmetic."""
    rng = np.random.default_rng(2)
    z = rng.normal(size=400_000)
    lu = np.log(rng.random(z.size))
    before = np.zeros(z.size, dtype=bool)
    for n in list(range(2, 48)) + [64, 100, 255, 383, 1024]:
        d = 1.5 * (n - 1) - 1.0 / 3.0
        vv = 1.0 + (1.0 / math.sqrt(9.0 * d)) * z
        ok = vv > 0.0
        vv = np.where(ok, vv, 1.0) ** 3
        ok &= lu < 0.5 * z * z + d - d * vv + d * np.log(vv)
        assert not np.any(before & ~ok), n
        before = ok
