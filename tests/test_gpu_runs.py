"""One step that gathers from run tables and chains, in every form and with
every feature: the state after some steps, then one more, against the oracle's
step from that state, and against the library's own step from the same state
set anew (a sort, one run a tile).

Bars, those of one step from a set state: FP64 positions, keys, permutation and
offsets bit-identical and velocities within 1e-12 (SRD+a: + 64 eps cond(I_c));
reduced forms: streaming within a few FP32 ulps (2e-6 cells, 4e-6 with particles
of several cells a step, in boxes of up to 16 cells; FP32 positions in proportion
to the box), binning bit-identical given the GPU's positions,
velocities within 2e-6 of the oracle's collision.  The step set anew: the same
bits.
"""
import math

import numpy as np
import pytest

import oracle as orc
import synth
from test_gpu_amc import EPS, cell_cond, frame, rel_err

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


def box_of(L, **kw):
    b = dict(L=tuple(L), h=0.1, alpha=130.0 * DEG, kT=1.0, mass=1.0, density=10.0, seed=7,
             mbs=True, walls=False, g=(0.0, 0.0, 0.0))
    b.update(kw)
    return b


def oparams(box):
    return orc.Params(**box)


# boxes, steps before the compared one, reorder interval, tiling
FEATURES = {
    "plain": ([box_of((33, 10, 9), mbs=False)], 4, 0, None),
    # attempt chains of the gamma draw in about 1700 of 64000 cells
    "dilute": ([box_of((40, 40, 40), density=2.2)], 3, 0, None),
    "fast": ([box_of((48, 14, 12), kT=225.0)], 4, 5, None),
    "very fast": ([box_of((30, 14, 12), kT=2500.0)], 3, 0, None),
    "fast short tables": ([box_of((61, 7, 9), kT=225.0)], 4, 0, (4, 0, 0, 1)),
    "fast two passes": ([box_of((64, 9, 8), kT=225.0)], 4, 2, (32, 0, 0, 0)),
    "amc": ([box_of((26, 10, 9), mbs=False, amc=True)], 4, 3, None),
    "amc mbs": ([box_of((26, 10, 9), amc=True)], 4, 5, None),
    "amc fast": ([box_of((40, 9, 10), amc=True, kT=225.0)], 4, 0, None),
    "amc two passes": ([box_of((32, 6, 7), amc=True, density=12.0)], 4, 3, (32, 0, 0, 0)),
    "amc slip": ([box_of((25, 8, 7), amc=True, walls=True, slip=True, g=(1e-3, 0.0, 0.0))], 4, 0,
                 None),
    "fixed": ([box_of((26, 10, 9), fixed=True)], 4, 3, None),
    "fixed fast": ([box_of((33, 10, 9), fixed=True, kT=225.0)], 4, 0, None),
    "amc fixed": ([box_of((26, 10, 9), amc=True, fixed=True)], 4, 0, None),
    "batch": ([box_of((17, 9, 8)), box_of((1, 1, 1), seed=2, kT=0.6), box_of((40, 5, 6), seed=3),
               box_of((3, 2, 9), seed=4, alpha=1.7, kT=1.8, density=20.0),
               box_of((50, 1, 1), seed=5, density=0.5)], 5, 3, None),
    "shear": ([box_of((45, 8, 6), le_u=1.7)], 4, 0, None),
    "amc shear": ([box_of((31, 8, 6), le_u=1.7, amc=True)], 4, 0, None),
    "channel": ([box_of((37, 6, 5), walls=True, g=(1e-3, 0.0, 0.0))], 4, 2, None),
    "couette fast": ([box_of((37, 6, 9), walls=True, uwall=0.4, kT=100.0)], 4, 0, None),
}


def two_states(mpc, form, name):
    """States before and after the compared step, its binning, and the state
    after the same step from the first one set anew."""
    boxes, steps, R, tiling = FEATURES[name]
    t0, nb = 11, range(len(boxes))
    print(f"case runs {form} {name}", flush=True)
    with mpc.Sim(boxes, form=form, reorder_every=R) as sim:
        if tiling:
            sim.set_tiling(*tiling)
        for k, b in enumerate(boxes):
            sim.set_state(*synth.box_state(b["L"], density=b["density"], kT=b["kT"], seed=3 + k), k)
        sim.set_step(t0)
        sim.step(steps)
        before = [sim.get_state(k) for k in nb]
        sim.step(1)
        after = [sim.get_state(k) for k in nb]
        binning = [sim.get_binning(k) for k in nb]
    with mpc.Sim(boxes, form=form, reorder_every=R) as sim:
        for k in nb:
            sim.set_state(*before[k], k)
        sim.set_step(t0 + steps)
        sim.step(1)
        anew = [sim.get_state(k) for k in nb]
    return boxes, t0 + steps, R, before, after, binning, anew


@pytest.mark.parametrize("form", ["fp64", "fp32", "split"])
@pytest.mark.parametrize("name", list(FEATURES))
def test_step_from_runs(mpc, form, name):
    boxes, t, R, before, after, binning, anew = two_states(mpc, form, name)
    for k, box in enumerate(boxes):
        for got, want in zip(after[k], anew[k]):
            np.testing.assert_array_equal(got, want)
        p, (x0, v0), (x1, v1), (kg, pg, og) = oparams(box), before[k], after[k], binning[k]
        gather = R > 0 and (t + 1) % R == 0
        if form == "fp64":
            xo, vo, ko, po, oo = orc.step(p, t, x0, v0, reorder=gather, binning=True)
            for got, want in ((kg, ko), (pg, po), (og, oo), (x1, xo)):
                np.testing.assert_array_equal(got, want)
            tol = 1e-12
            if box.get("amc") and not box.get("le_u"):
                xs, _, _ = orc.stream(p, x0, v0, t)
                cond = cell_cond(ko, oo, po, frame(p, t, xs))
                tol = tol + 64 * EPS * (cond[po] if gather else cond)
            elif box.get("amc"):
                continue  # image positions enter cond(I_c): the step set anew stands for it
            e = rel_err(v1, vo, box)
            print(f"{name} {box['L']}: max e = {e.max():.2e}")
            assert np.all(e <= tol)
        elif not (box["walls"] or box.get("le_u")):
            if gather:  # back to the order before the step
                x1, v1 = (np.empty_like(q) for q in after[k])
                x1[:, pg], v1[:, pg] = after[k]
            xs, _, _ = orc.stream(p, x0, v0, t)
            d = np.abs(x1 - xs)
            d = np.minimum(d, np.array(box["L"], dtype=float)[:, None] - d)
            # x + h v reaches further before the wrap at higher speeds: two ulps there
            far = 1.0 + np.abs(v0 * box["h"]).max() / max(box["L"])
            assert d.max() < (4e-6 if box["kT"] > 10.0 else 2e-6) * max(
                far, max(box["L"]) / 16.0 if form == "fp32" else 1.0)
            ko = orc.keys(p, t, x1)
            po, oo = orc.sort(ko, p.ncells)
            for got, want in ((kg, ko), (pg, po), (og, oo)):
                np.testing.assert_array_equal(got, want)
            vo = orc.collide(p, t, v0, po, oo, x=x1 if box.get("amc") else None)
            e = rel_err(v1, vo, box)
            print(f"{name} {box['L']} {form}: max e = {e.max():.2e}")
            assert e.max() <= 2e-6


@pytest.mark.parametrize("form", ["fp64", "split"])
def test_replayed_graphs_of_sixteen_steps(mpc, form):
    """Two replays of the default graph and a rest, with the program's own reads
    in between, against single launches and graphs of other lengths."""
    box = box_of((20, 11, 9))
    x, v = synth.box_state(box["L"], seed=3)
    res = []
    for graph, parts in ((1, (35, 16, 2)), (0, (35, 16, 2)), (1, (1,) * 53), (7, (50, 3)),
                         (1, (15, 38))):
        with mpc.Sim(box, form=form, reorder_every=5, graph=graph) as sim:
            sim.set_state(x, v)
            for n in parts:
                sim.step(n)
                sim.observables()
            res.append((sim.get_state(), sim.get_step(), sim.get_binning()))
    for state, step, binning in res[1:]:
        assert step == 53
        for a, b in zip(state + binning, res[0][0] + res[0][2]):
            np.testing.assert_array_equal(a, b)
