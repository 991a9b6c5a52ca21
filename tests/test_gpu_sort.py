"""The sort of a state by tile before its first step: from the caller's order,
from slots that a step left, from a mixture of both, between changes of the
tiling and binning exports.  Slots do not enter the results, so every run equals
the one that was not interrupted, bit for bit."""
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


def box_of(L, **kw):
    b = dict(L=tuple(L), h=0.1, alpha=130.0 * DEG, kT=1.0, mass=1.0, density=10.0, seed=7,
             mbs=True, walls=False, g=(0.0, 0.0, 0.0))
    b.update(kw)
    return b


def same(a, b):
    for u, w in zip(a, b):
        np.testing.assert_array_equal(u, w)


# (boxes: sizes of no whole blocks, one of a single particle block, empty tiles)
BOXES = {
    "periodic": [box_of((23, 11, 9)), box_of((5, 4, 3), seed=8), box_of((40, 3, 2), density=0.3)],
    "walls": [box_of((17, 9, 8), walls=True, g=(1e-3, 0.0, 0.0)),
              box_of((33, 5, 4), walls=True, seed=9)],
    # the binning export in the run lists' memory
    "larger": [box_of((44, 36, 9), mbs=False), box_of((9, 8, 7), mbs=False, seed=2)],
}


@pytest.mark.parametrize("form", ["fp64", "fp32", "split"])
@pytest.mark.parametrize("kind", list(BOXES))
def test_interrupted_runs(mpc, form, kind):
    boxes = BOXES[kind]
    if kind == "walls":
        boxes = [dict(b) for b in boxes]
    states = [synth.box_state(b["L"], density=b["density"], seed=3 + k)
              for k, b in enumerate(boxes)]
    print(f"case sort {form} {kind}", flush=True)

    def run(actions):
        with mpc.Sim(boxes, form=form, reorder_every=2) as sim:
            for k, (x, v) in enumerate(states):
                sim.set_state(x, v, k)
            for a in actions:
                a(sim)
            return [sim.get_state(k) for k in range(len(boxes))]

    def step(n):
        return lambda sim: sim.step(n)

    whole = run([step(7)])
    for between in (lambda s: s.set_tiling(6, 0, 4, 1), lambda s: s.get_binning(1),
                    lambda s: s.set_step(3), lambda s: s.autotune(1)):
        for k, got in enumerate(run([step(3), between, step(4)])):
            same(got, whole[k])


@pytest.mark.parametrize("form", ["fp64", "fp32", "split"])
def test_one_box_set_anew(mpc, form):
    """Box 1 in the caller's order, the others as the step left them."""
    boxes = BOXES["periodic"]
    states = [synth.box_state(b["L"], density=b["density"], seed=3 + k)
              for k, b in enumerate(boxes)]
    anew = synth.box_state(boxes[1]["L"], seed=77)
    print(f"case sort anew {form}", flush=True)
    with mpc.Sim(boxes, form=form, reorder_every=2) as a, \
            mpc.Sim(boxes, form=form, reorder_every=2) as b:
        for k, (x, v) in enumerate(states):
            a.set_state(x, v, k)
            b.set_state(*(anew if k == 1 else (x, v)), k)
        a.step(3)
        a.set_state(*anew, 1)
        same(a.get_state(1), b.get_state(1))
        a.step(4)
        with mpc.Sim(boxes, form=form, reorder_every=2) as c:
            for k, (x, v) in enumerate(states):
                c.set_state(x, v, k)
            c.step(7)
            for k in (0, 2):
                same(a.get_state(k), c.get_state(k))
        b.set_step(3)
        b.step(4)
        same(a.get_state(1), b.get_state(1))
