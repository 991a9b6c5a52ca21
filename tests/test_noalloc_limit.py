"""The allocation-free entry point takes every box within its documented limit,
256 MiB at 114 B per particle, 40 B per cell (88 B between walls) and 20 B per
tile of four cells: the workspace of such a box fits the static array, however
thin or sparse the box is."""
import numpy as np
import pytest

import synth

LIMIT, ARRAY = 256 << 20, 704 << 20  # as in include/mpc.h


def charge(L, density, walls):
    nlz = L[2] + 2 if walls else L[2]
    cells = -(-(L[0] * L[1] * nlz) // 4096) * 4096
    n = round(density * L[0] * L[1] * L[2])
    return 114 * n + (88 if walls else 40) * cells + 20 * L[1] * nlz * -(-L[0] // 4) + 65536


def edge_at_limit(l0, aspect, density, walls):
    """The largest box l0 x l1 x l2, l1 about aspect l2, within the limit."""
    def box(e):
        return (l0, max(1, int(e * aspect)), max(1, int(e / aspect)))
    lo, hi = 1.0, 1.0
    while charge(box(hi), density, walls) <= LIMIT:
        lo, hi = hi, 2 * hi
    while hi - lo > 1e-4 * hi:
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if charge(box(mid), density, walls) <= LIMIT else (lo, mid)
    return box(lo)


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("mbs", [False, True])
def test_workspace_of_every_accepted_box_fits(walls, mbs):
    import paper_2406_15236_amd as m
    worst = (0.0, None)
    for l0 in (1, 2, 3, 4, 5, 7, 8, 9, 16, 31, 33, 64, 100, 1000, 40000):
        for aspect in (1.0, 30.0, 0.02):
            for density in (1e-3, 0.01, 0.05, 0.09, 0.1, 0.101, 0.12, 0.2, 0.35, 0.5, 0.7, 1.0,
                            1.5, 2.5, 4.0, 7.0, 10.0, 20.0, 60.0, 215.0, 250.0):
                L = edge_at_limit(l0, aspect, density, walls)
                if round(density * L[0] * L[1] * L[2]) < 1 or charge(L, density, walls) > LIMIT:
                    continue
                p = m.make_params(dict(L=L, density=density, walls=walls, mbs=mbs))
                worst = max(worst, (m.workspace_bytes(p) / 2**20, (L, density)))
    print(f"largest workspace {worst[0]:.0f} MiB at {worst[1]}")
    assert worst[0] * 2**20 <= ARRAY


def test_thin_sparse_boxes_need_little_more_than_their_state():
    """Three times the charge, where tables of 32 runs a tile took 8 to 13."""
    import paper_2406_15236_amd as m
    for L, density in (((1, 1000, 1000), 0.5), ((1, 1400, 1400), 0.1), ((2, 1000, 1000), 0.2)):
        assert m.workspace_bytes(m.make_params(dict(L=L, density=density))) < 3 * charge(
            L, density, False)


@pytest.mark.gpu
@pytest.mark.parametrize("L,density,kw", [
    ((1, 1000, 1000), 0.5, {}), ((2, 1000, 1000), 0.2, {"mbs": True}),
    ((4, 800, 800), 0.1, {"walls": True}), ((1, 200, 150), 3.0, {"mbs": True})])
def test_thin_sparse_boxes_match_the_oracle(L, density, kw):
    """Bar: 1e-11 as for every run of a few steps against the oracle."""
    import math

    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as orc
    import paper_2406_15236_amd as m
    box = dict(L=L, h=0.1, alpha=2.2, kT=1.0, mass=1.0, density=density, seed=7, mbs=False,
               walls=False, g=(0.0, 0.0, 0.0))
    box.update(kw)
    x, v = synth.box_state(L, density=density, seed=5)
    print(f"case thin {L} {density} {kw}", flush=True)
    xd, vd = (torch.from_numpy(np.ascontiguousarray(q)).cuda() for q in (x, v))
    m.run_noalloc(m.make_params(box), xd.data_ptr(), vd.data_ptr(), x.shape[1], 3, 4,
                  torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    xo, vo = x, v
    for t in range(3, 7):
        xo, vo = orc.step(orc.Params(**box), t, xo, vo)
    d = np.abs(xd.cpu().numpy() - xo)
    d = np.minimum(d, np.array(L, dtype=float)[:, None] - d) if not kw.get("walls") else d
    if kw.get("walls"):
        d[:2] = np.minimum(d[:2], np.array(L[:2], dtype=float)[:, None] - d[:2])
    e = np.linalg.norm(vd.cpu().numpy() - vo, axis=0) / np.maximum(np.linalg.norm(vo, axis=0), 1.0)
    print(f"max |dx| = {d.max():.2e}, max e = {e.max():.2e}")
    assert d.max() < 1e-11 and e.max() < 1e-11
