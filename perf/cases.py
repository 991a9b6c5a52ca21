"""Workloads of the MPC-SRD library that its speed is judged on.

Each case is what a simulation program does between two looks at its system:
advance the particles by a number of time steps and read results back.  The
pass goes through the Python binding of the C ABI (`Sim`, `run_noalloc`) with
the library's default tiling; inputs are seeded fluid boxes as in the paper
(uniform positions, Maxwellian velocities, about Poisson cell counts).

Results are read the way the size allows: small boxes return their whole
state; boxes too large to copy to the host return every observable and the
state of some ten thousand tagged particles.

`exact` follows the method (arXiv:2406.15236, Sec. II) in 64-bit torch
operations, without the library.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2406_15236_amd as mpc

TAGGED = 32768         # tagged particles read back from a large box

# All keys of a case, with their defaults.
#   kind      sim: Sim handle; noalloc: run_noalloc on device arrays;
#             checkpoint: host state in, steps, host state out;
#             ensemble: many uneven boxes in one handle
#   whole     sim: the whole state is read back (else tagged particles)
DEFAULTS = dict(kind="sim", lx=16, ly=16, lz=16, density=10.0, alpha=130.0, kT=1.0, h=0.1,
                form="fp64", reorder=0, steps=10, graph=1, whole=False,
                mbs=False, amc=False, fixed=False, walls=False, slip=False,
                uwall=0.0, le_u=0.0, gx=0.0, boxes=1, lmin=16, lmax=64)


def listed():
    return [
        # The smallest system: one small box stepped in long runs, every step
        # bound by launches and by the latency of one tile.
        dict(DEFAULTS, name="cube16_fp64", steps=100, whole=True),
        # A caller that owns its arrays and may not allocate: in-place steps.
        dict(DEFAULTS, name="noalloc_24_fp64", kind="noalloc", lx=24, ly=24, lz=24, mbs=True,
             steps=10),
        # Sheared fluid (Lees-Edwards) in a small ragged FP32 box.
        dict(DEFAULTS, name="shear_ragged_fp32", form="fp32", lx=41, ly=33, lz=27, mbs=True,
             le_u=0.8, reorder=10, steps=20, whole=True),
        # Checkpoint and resume: host state in, a step, host state out.
        dict(DEFAULTS, name="checkpoint_64_split", kind="checkpoint", form="split", lx=64, ly=64,
             lz=64, mbs=True, reorder=1, steps=1),
        # Reproducible run with exact cell sums, medium ragged box.
        dict(DEFAULTS, name="fixed_ragged_fp64", lx=91, ly=75, lz=60, mbs=True, fixed=True,
             reorder=20, steps=20),
        # Dense fluid: 50 particles per cell.
        dict(DEFAULTS, name="dense50_fp64", lx=64, ly=64, lz=64, density=50.0, mbs=True, steps=10),
        # Angular-momentum-conserving collision with the thermostat, 100^3.
        dict(DEFAULTS, name="amc_100_fp64", lx=100, ly=100, lz=100, amc=True, mbs=True, reorder=20,
             steps=20),
        # Poiseuille channel: no-slip walls with phantoms, body force,
        # thermostat, split form, graphs of 50 steps.
        dict(DEFAULTS, name="channel_split", form="split", lx=256, ly=256, lz=64, walls=True,
             mbs=True, gx=1e-3, steps=50, graph=50),
        # Batched ensemble of 64 uneven boxes, each box's observables read
        # every 100 steps.
        dict(DEFAULTS, name="ensemble64_fp64", kind="ensemble", boxes=64, lmin=16, lmax=64,
             steps=100, graph=50),
        # The thermostatted 256^3 box with renumbering every 20 steps, in
        # double precision and in the split form.
        dict(DEFAULTS, name="thermo_256_fp64", lx=256, ly=256, lz=256, mbs=True, reorder=20,
             steps=20),
        dict(DEFAULTS, name="thermo_256_split", form="split", lx=256, ly=256, lz=256, mbs=True,
             reorder=20, steps=20),
        # Plain SRD at large scale (5.7e8 particles, 64 GB of device state).
        dict(DEFAULTS, name="plain_384_fp64", lx=384, ly=384, lz=384, steps=5),
    ]


def draw(rng):
    c = dict(DEFAULTS)
    c["kind"] = rng.choice(["sim"] * 7 + ["noalloc", "checkpoint", "ensemble"])
    c["kT"] = round(rng.uniform(0.5, 2.0), 3)
    c["alpha"] = round(rng.uniform(90.0, 150.0), 2)
    c["form"] = rng.choice(["fp64", "fp64", "split", "fp32"])
    c["reorder"] = rng.choice([0, 0, 1, 5, 20])
    if c["kind"] == "ensemble":
        c["boxes"] = rng.randint(2, 64)
        c["lmin"] = rng.randint(6, 20)
        c["lmax"] = rng.randint(24, 64)
        c["mbs"] = rng.random() < 0.5
        c["steps"] = rng.choice([10, 20, 50])
        c["graph"] = c["steps"]
        return c
    c["density"] = rng.choice([5.0, 10.0, 10.0, 20.0, 50.0,
                               round(math.exp(rng.uniform(math.log(3.0), math.log(60.0))), 2)])
    top = {"sim": 1.6e8, "noalloc": 1.2e6, "checkpoint": 3.0e6}[c["kind"]]
    n = math.exp(rng.uniform(math.log(4.0e3), math.log(top)))
    edge = (n / c["density"]) ** (1.0 / 3.0)
    fx, fy = rng.uniform(0.6, 1.6), rng.uniform(0.6, 1.6)
    c["lx"], c["ly"] = max(3, round(edge * fx)), max(3, round(edge * fy))
    c["lz"] = max(3, round(edge / (fx * fy)))
    option = rng.choice(["plain", "mbs", "mbs", "amc", "channel", "slip", "couette", "shear",
                         "fixed"])
    c["mbs"] = option != "plain"
    c["amc"] = option == "amc"
    c["fixed"] = option == "fixed"
    c["walls"] = option in ("channel", "slip", "couette")
    c["slip"] = option == "slip"
    c["gx"] = 1e-3 if option in ("channel", "slip") else 0.0
    c["uwall"] = 0.4 if option == "couette" else 0.0
    c["le_u"] = 0.6 if option == "shear" else 0.0
    if c["kind"] == "noalloc":
        c["form"], c["reorder"] = "fp64", 0
    cells = c["lx"] * c["ly"] * c["lz"]
    n = c["density"] * cells
    c["whole"] = c["kind"] == "sim" and n < 5e5
    c["steps"] = max(1, min(rng.choice([5, 10, 20, 50, 100]), int(2.0e9 / n)))
    if c["kind"] == "checkpoint":
        c["steps"] = rng.choice([1, 5])
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _box(case, seed):
    return dict(L=(case["lx"], case["ly"], case["lz"]), density=case["density"], h=case["h"],
                alpha=math.radians(case["alpha"]), kT=case["kT"], mass=1.0, seed=seed,
                mbs=case["mbs"], amc=case["amc"], fixed=case["fixed"], walls=case["walls"],
                slip=case["slip"], uwall=case["uwall"], le_u=case["le_u"],
                g=(case["gx"], 0.0, 0.0))


def _boxes(case, seed):
    """The boxes of an ensemble: edges, density, angle and temperature drawn
    from the case alone (they fix the sizes), random streams from the seed."""
    if case["kind"] != "ensemble":
        return [_box(case, seed)]
    rng = np.random.default_rng(4)
    out = []
    for b in range(case["boxes"]):
        lx, ly, lz = (int(v) for v in rng.integers(case["lmin"], case["lmax"] + 1, size=3))
        out.append(_box(dict(case, lx=lx, ly=ly, lz=lz,
                             density=float(rng.choice([5.0, 10.0, 20.0])),
                             alpha=float(rng.uniform(90.0, 150.0)),
                             kT=float(rng.uniform(0.5, 2.0))), 1000 * seed + b))
    return out


def _count(box):
    return int(round(box["density"] * box["L"][0] * box["L"][1] * box["L"][2]))


def _host_state(box, seed):
    rng = np.random.default_rng(seed)
    n = _count(box)
    x = np.empty((3, n))
    for k in range(3):
        x[k] = np.minimum(rng.random(n) * box["L"][k], np.nextafter(float(box["L"][k]), 0.0))
    v = rng.normal(0.0, math.sqrt(box["kT"] / box["mass"]), size=(3, n))
    v -= v.mean(axis=1, keepdims=True)
    return x, v


def _tagged(n):
    m = min(TAGGED, n)
    return (np.arange(m, dtype=np.int64) * n) // m


def prepare(case, seed):
    boxes = _boxes(case, seed)
    st = dict(case=case, boxes=boxes)
    if case["kind"] == "noalloc":
        x, v = _host_state(boxes[0], seed)
        st["params"] = mpc.make_params(boxes[0], "fp64", reorder_every=case["reorder"])
        st["x"], st["v"] = torch.from_numpy(x).cuda(), torch.from_numpy(v).cuda()
        st["t"] = 0
        return st
    sim = mpc.Sim(boxes, form=case["form"], reorder_every=case["reorder"], graph=case["graph"])
    st["sim"] = sim
    if case["kind"] == "checkpoint":
        st["x"], st["v"] = _host_state(boxes[0], seed)
    else:
        sim.init_state(seed)
        st["tagged"] = [_tagged(_count(b)) for b in boxes]
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "noalloc":
        stream = torch.cuda.current_stream().cuda_stream
        mpc.run_noalloc(st["params"], st["x"].data_ptr(), st["v"].data_ptr(), st["x"].shape[1],
                        st["t"], case["steps"], stream)
        st["t"] += case["steps"]
        return st["x"], st["v"]
    sim = st["sim"]
    if case["kind"] == "checkpoint":
        sim.set_state(st["x"], st["v"])
        sim.set_step(17)
        sim.step(case["steps"])
        return sim.get_state()
    sim.step(case["steps"])
    if case["kind"] == "ensemble":
        obs = [sim.observables(b) for b in range(len(st["boxes"]))]
        tag = [sim.get_particles(i, b) for b, i in enumerate(st["tagged"])]
        return (np.stack([o["P"] for o in obs]), np.array([o["E"] for o in obs]),
                np.array([o["T"] for o in obs]), np.concatenate([x for x, _ in tag], axis=1),
                np.concatenate([v for _, v in tag], axis=1))
    o = sim.observables()
    x, v = sim.get_state() if case["whole"] else sim.get_particles(st["tagged"][0])
    return o["P"], o["E"], o["T"], x, v


def work(case):
    """Every step reads and writes the state of each particle once (48, 24 or
    28 bytes); results are read once.  About 60 operations a particle-step
    (streaming 6, momentum 6, energy 9, rotation 33, binning 6)."""
    n = sum(_count(b) for b in _boxes(case, 1))
    state = {"fp64": 48, "fp32": 24, "split": 28}[case["form"]]
    per = 2 * state
    out = 48 * n if case["whole"] or case["kind"] in ("noalloc", "checkpoint") else 0
    if case["kind"] == "checkpoint":
        out *= 2
    return {"bytes": float(per * n * case["steps"] + out), "flops": 60.0 * n * case["steps"]}


# ---------------------------------------------------------------------------
# The method in 64-bit torch operations
# ---------------------------------------------------------------------------
_DEV = "cuda" if torch.cuda.is_available() else "cpu"
_MASK = 0xFFFFFFFF
SHIFT, AXIS, THERMO, PHANTOM, INIT_POS, INIT_VEL = 1, 2, 3, 4, 5, 6


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10; c0 and c1 tensors or numbers; four int64 tensors."""
    c0 = torch.as_tensor(c0, dtype=torch.int64, device=_DEV)
    c1 = torch.as_tensor(c1, dtype=torch.int64, device=_DEV)
    c0, c1 = torch.broadcast_tensors(c0, c1)
    c2, c3 = torch.full_like(c0, c2 & _MASK), torch.full_like(c0, c3)
    k0, k1 = seed & _MASK, (seed >> 32) & _MASK
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((b >> 32) & _MASK) ^ c1 ^ k0, b & _MASK,
                          ((a >> 32) & _MASK) ^ c3 ^ k1, a & _MASK)
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return c0, c1, c2, c3


def _u53(a, b):
    return ((a << 21) | (b >> 11)).double() * 2.0 ** -53


def _u53_open(a, b):
    return (2 * ((a << 20) | (b >> 12)) + 1).double() * 2.0 ** -53


def _u32_open(w):
    return (w.double() + 0.5) * 2.0 ** -32


def _angle(w):
    return 2.0 * math.pi * (w.double() * 2.0 ** -32)


def _initial(box, index, seed):
    """The library's device initialiser: uniform positions, normal velocities,
    mean velocity removed."""
    n = _count(box)
    x = torch.empty((3, n), dtype=torch.float64, device=_DEV)
    v = torch.empty_like(x)
    sd = math.sqrt(box["kT"] / box["mass"])
    for i0 in range(0, n, 1 << 25):
        i = torch.arange(i0, min(n, i0 + (1 << 25)), dtype=torch.int64, device=_DEV)
        s = slice(i0, i0 + i.numel())
        a, b = _philox(0, i, index, INIT_POS, seed), _philox(1, i, index, INIT_POS, seed)
        for k, u in enumerate((_u53(a[0], a[1]), _u53(a[2], a[3]), _u53(b[0], b[1]))):
            x[k, s] = (u * box["L"][k]).clamp_(max=np.nextafter(float(box["L"][k]), 0.0))
        c = _philox(0, i, index, INIT_VEL, seed)
        r0, r1 = (sd * torch.sqrt(-2.0 * torch.log(_u32_open(w))) for w in (c[0], c[2]))
        v[0, s], v[1, s] = r0 * torch.cos(_angle(c[1])), r0 * torch.sin(_angle(c[1]))
        v[2, s] = r1 * torch.cos(_angle(c[3]))
    return x, v - v.mean(dim=1, keepdim=True)


def _wrap(x, L):
    x = x - L * torch.floor(x / L)
    return torch.where((x >= L) | (x < 0.0), torch.zeros_like(x), x)


def _stream(box, x, v, d):
    L, h = box["L"], box["h"]
    e = x + h * v
    if box["walls"]:
        H = float(L[2])
        lo, hi = e[2] < 0.0, e[2] > H
        hit = lo | hi
        tr2 = torch.where(hit, 2.0 * (e[2] - hi.double() * H) / v[2], 0.0)
        ez = e[2] - tr2 * v[2]
        if not box["slip"]:
            u = (2.0 * hi.double() - 1.0) * box["uwall"]
            e[0] -= tr2 * (v[0] - u)
            e[1] -= tr2 * v[1]
            v[0] = torch.where(hit, 2.0 * u - v[0], v[0])
            v[1] = torch.where(hit, -v[1], v[1])
        e[2] = ez.clamp_(0.0, H)
        v[2] = torch.where(hit, -v[2], v[2])
    else:
        if box["le_u"]:
            side = (e[2] < 0.0).double() - (e[2] >= L[2]).double()
            e[0] += side * d
            v[0] += side * box["le_u"]
        e[2] = _wrap(e[2], L[2])
    e[0], e[1] = _wrap(e[0], L[0]), _wrap(e[1], L[1])
    return e, v


def _sum(key, ncell, *terms):
    return [torch.zeros(ncell, dtype=torch.float64, device=_DEV).index_add_(0, key, w)
            for w in terms]


def _gamma(cells, shape, t, seed):
    """Marsaglia-Tsang draws of Gamma(shape, 1) for `cells`."""
    out = torch.zeros_like(shape)
    left = torch.arange(cells.numel(), device=_DEV)
    for j in range(64):
        if left.numel() == 0:
            break
        d = shape[left] - 1.0 / 3.0
        w = _philox(j, cells[left], t, THERMO, seed)
        z = torch.sqrt(-2.0 * torch.log(_u32_open(w[0]))) * torch.cos(_angle(w[1]))
        c = (1.0 + z / torch.sqrt(9.0 * d)) ** 3
        ok = c > 0.0
        lhs = torch.log(_u53_open(w[2], w[3]))
        ok &= lhs < 0.5 * z * z + d - d * c + d * torch.log(torch.where(ok, c, 1.0))
        out[left[ok]] = (d * c)[ok]
        left = left[~ok]
    return out


def _phantoms(box, t, sz, nc):
    """Number, velocity sums and squared-speed sum of every cell's phantoms."""
    plane, H = box["L"][0] * box["L"][1], box["L"][2]
    sd = math.sqrt(box["kT"] / box["mass"])
    out = torch.zeros((5, nc), dtype=torch.float64, device=_DEV)
    cut = ((0, sz, -1.0), (H, 1.0 - sz, 1.0)) if sz >= 0.0 else ((-1, 1.0 + sz, -1.0),
                                                                (H - 1, -sz, 1.0))
    for cz, fw, top in cut:
        if fw <= 0.0:
            continue
        c = (cz + 1) * plane + torch.arange(plane, device=_DEV)
        w = _philox(0, c, t, PHANTOM, box["seed"])
        u, lam = _u53(w[0], w[1]), box["density"] * fw
        pk = math.exp(-lam)
        F, k = pk, torch.zeros(plane, dtype=torch.int64, device=_DEV)
        for m in range(1, 128):
            k += (u >= F).long()
            pk = pk * lam / m
            F = F + pk
        top_n = int(k.max())
        norm = torch.zeros((max(3 * top_n, 1), plane), dtype=torch.float64, device=_DEV)
        for m in range(3 * top_n):
            if m % 4 == 0:
                w = _philox(1 + m // 4, c, t, PHANTOM, box["seed"])
            p = (m % 4) // 2
            r = torch.sqrt(-2.0 * torch.log(_u32_open(w[2 * p])))
            a = _angle(w[2 * p + 1])
            norm[m] = sd * r * (torch.cos(a) if m % 2 == 0 else torch.sin(a))
        for q in range(top_n):
            on = (k > q).double()
            for a in range(3):
                vp = norm[3 * q + a] + (top * box["uwall"] if a == 0 else 0.0)
                out[a, c] += on * vp
                out[3, c] += on * vp * vp
        out[4, c] = k.double()
    return out


def _step(box, t, x, v, reorder):
    L, h, m, seed = box["L"], box["h"], box["mass"], box["seed"]
    walls, slip, le = box["walls"], box["slip"], box["le_u"]
    d = math.fmod(le * ((t + 1) * h), float(L[0])) if le else 0.0
    d = d + L[0] if d < 0.0 else d
    x, v = _stream(box, x, v, d)
    w = _philox(0, 0, t, SHIFT, seed)
    s = [float((q >> 8).double() * 2.0 ** -24 - 0.5) for q in w[:3]]
    cz = torch.floor(x[2] + s[2]).long()
    nlz = L[2] + 2 if walls else L[2]
    side = None
    xi = x[0]
    if le:
        side = (cz < 0).double() - (cz >= L[2]).double()
        xi = x[0] + side * d
    cx = torch.remainder(torch.floor(xi + s[0]).long(), L[0])
    cy = torch.remainder(torch.floor(x[1] + s[1]).long(), L[1])
    cz = cz + 1 if walls else torch.remainder(cz, L[2])
    key = (cz * L[1] + cy) * L[0] + cx
    del cx, cy, cz
    nc = L[0] * L[1] * nlz
    nf = torch.bincount(key, minlength=nc).double()
    if le:
        v[0] += torch.where(nf[key] >= 2.0, side * le, 0.0)
    ph = _phantoms(box, t, s[2], nc) if walls and not slip else None
    ntot = nf if ph is None else nf + torch.where(nf > 0, ph[4], 0.0)
    mom = _sum(key, nc, v[0], v[1], v[2])
    V = torch.stack([(q if ph is None else q + ph[k]) / ntot.clamp(min=1.0)
                     for k, q in enumerate(mom)])
    cells = torch.arange(nc, device=_DEV)
    w = _philox(0, cells, t, AXIS, seed)
    nz = 1.0 - 2.0 * _u53(w[0], w[1])
    nr, phi = torch.sqrt(1.0 - nz * nz), 2.0 * math.pi * _u53(w[2], w[3])
    n = torch.stack([nr * torch.cos(phi), nr * torch.sin(phi), nz])
    del w, nz, nr, phi
    ca, sa = math.cos(box["alpha"]), math.sin(box["alpha"])
    u = v - V[:, key]
    K = None
    if box["mbs"] and not box["amc"]:
        K = m * _sum(key, nc, (u * u).sum(0))[0]
        if ph is not None:
            K = K + m * (ph[3] - 2.0 * (ph[:3] * V).sum(0) + ph[4] * (V * V).sum(0))
    np_ = n[:, key]
    du = (ca * u + sa * torch.stack([np_[1] * u[2] - np_[2] * u[1], np_[2] * u[0] - np_[0] * u[2],
                                     np_[0] * u[1] - np_[1] * u[0]])
          + (1.0 - ca) * (np_ * u).sum(0) * np_)
    del np_
    if box["amc"]:
        r = torch.stack([x[0] if side is None else xi, x[1], x[2]])
        r = r + torch.tensor(s, dtype=torch.float64, device=_DEV)[:, None]
        r = r - torch.floor(r)
        r = r - torch.stack([q / nf.clamp(min=1.0) for q in _sum(key, nc, r[0], r[1], r[2])])[:, key]
        f = u - du
        dL = torch.stack(_sum(key, nc, r[1] * f[2] - r[2] * f[1], r[2] * f[0] - r[0] * f[2],
                              r[0] * f[1] - r[1] * f[0]))
        xx, yy, zz, xy, xz, yz = _sum(key, nc, r[0] * r[0], r[1] * r[1], r[2] * r[2], r[0] * r[1],
                                      r[0] * r[2], r[1] * r[2])
        I = [yy + zz, xx + zz, xx + yy]
        c00, c01, c02 = I[1] * I[2] - yz * yz, xz * yz + xy * I[2], xy * yz + I[1] * xz
        c11, c12, c22 = I[0] * I[2] - xz * xz, xy * xz + I[0] * yz, I[0] * I[1] - xy * xy
        det = I[0] * c00 - xy * c01 - xz * c02
        inv = torch.where((nf >= 3) & (det != 0.0), 1.0 / det, 0.0)
        om = torch.stack([c00 * dL[0] + c01 * dL[1] + c02 * dL[2],
                          c01 * dL[0] + c11 * dL[1] + c12 * dL[2],
                          c02 * dL[0] + c12 * dL[1] + c22 * dL[2]]) * inv
        half = 0.5 * (I[0] + I[1] + I[2])
        om = om + dL * torch.where((nf == 2) & (half > 0.0), 1.0 / half, 0.0)
        o = om[:, key]
        du = du + torch.stack([o[1] * r[2] - o[2] * r[1], o[2] * r[0] - o[0] * r[2],
                               o[0] * r[1] - o[1] * r[0]])
        if box["mbs"]:
            K = m * _sum(key, nc, (du * du).sum(0))[0]
    if box["mbs"]:
        live = torch.nonzero((nf > 0) & (ntot >= 2)).flatten()
        Ek = torch.zeros_like(nf)
        Ek[live] = box["kT"] * _gamma(live, 1.5 * (ntot[live] - 1.0), t, seed)
        kappa = torch.where((Ek > 0.0) & (K > 0.0), torch.sqrt(2.0 * Ek / K), 1.0)
        du = du * kappa[key]
    v = torch.where((ntot >= 2.0)[key], V[:, key] + du, v)
    if le:
        v[0] -= torch.where(nf[key] >= 2.0, side * le, 0.0)
    for k in range(3):
        if box["g"][k]:
            v[k] += box["g"][k] * h
    if reorder and (t + 1) % reorder == 0:
        order = torch.sort(key, stable=True)[1]
        x, v = x[:, order], v[:, order]
    return x, v


def exact(case, seed):
    """What `run` returns on new inputs.  No value (None) for the total momentum
    of a box without a body force, which is a sum of rounding errors, nor for
    single particles of a reduced form after more than one step: a particle
    that rounding puts into the next cell takes another path from there on."""
    boxes = _boxes(case, seed)
    paths = case["form"] == "fp64" or case["steps"] == 1
    if _DEV == "cpu" and sum(_count(b) for b in boxes) * case["steps"] > 5e6:
        return None
    out = []
    for b, box in enumerate(boxes):
        if case["kind"] in ("noalloc", "checkpoint"):
            x, v = (torch.from_numpy(q).to(_DEV) for q in _host_state(box, seed))
        else:
            x, v = _initial(box, b, seed)
        t0 = 17 if case["kind"] == "checkpoint" else 0
        for t in range(t0, t0 + case["steps"]):
            x, v = _step(box, t, x, v, case["reorder"])
        n = x.shape[1]
        if case["kind"] in ("noalloc", "checkpoint"):
            return (x, v) if paths else None
        P = box["mass"] * v.sum(1)
        E = 0.5 * box["mass"] * float((v * v).sum())
        dv = v - v.mean(dim=1, keepdim=True)
        T = box["mass"] * float((dv * dv).sum()) / (3.0 * (n - 1))
        i = torch.from_numpy(np.arange(n) if case["whole"] else _tagged(n)).to(_DEV)
        out.append((P.cpu().numpy(), E, T, x[:, i].cpu().numpy(), v[:, i].cpu().numpy()))
    if case["kind"] == "ensemble":
        P, E, T, x, v = zip(*out)
        return (None, np.array(E), np.array(T), np.concatenate(x, axis=1) if paths else None,
                np.concatenate(v, axis=1) if paths else None)
    P, E, T, x, v = out[0]
    return P if case["gx"] else None, E, T, x if paths else None, v if paths else None
