"""Timed cases of the library: the calls a user's program makes, over the sizes it makes them at.

`listed()` names them, `draw(rng)` gives more of the same ranges, `prepare` builds what such a program
has in hand (inputs on the GPU, the simulations it keeps), `run` is one pass through the public entry
points, `work` what a pass cannot do without, `exact` the same outputs in 64 bits from plain torch.

Every pass of a lattice case starts from its initial fields (`init_fields`, a run of a parameter
sweep), advances a number of coupled steps and reads the fields back into device memory, so a pass
gives the same outputs each time.  The simulations take the launch shape and layout that the
repository's autotuner names for their size, as its README shows.
"""

from __future__ import annotations

import ctypes as C
import math
import random

import numpy as np
import torch

from paper_2510_18688_amd import autotune, lbf, porous
from paper_2510_18688_amd import workloads as W
from paper_2510_18688_amd import workloads3 as W3

FIELDS2 = ["phi", "T", "fl", "fs", "ux", "uy", "p", "rhoH", "mu", "C", "chi", "rho", "phihat"]
FIELDS3 = ["phi", "T", "fl", "fs", "ux", "uy", "uz", "p", "rhoH", "mu", "C", "chi", "rho", "phihat"]


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the sessile drop of the parity runs: the smallest lattice in earnest use, a few microseconds of
        # work per step, where launches and latency count; its invariants are monitored as well
        {"name": "drop_128x96", "kind": "drop", "nx": 128, "ny": 96, "steps": 50, "reduce": True},
        # one lattice of the batch workload's range on its own, odd sides
        {"name": "drop_455x318", "kind": "drop", "nx": 455, "ny": 318, "steps": 30, "reduce": False},
        # the headline workload: drop on a held cold cylinder, state far larger than the caches
        {"name": "cylinder_2048x2048", "kind": "cylinder", "nx": 2048, "ny": 2048, "steps": 30, "mrt": False},
        # MRT collisions at a middling size with a ragged last strip
        {"name": "cylinder_mrt_1000x700", "kind": "cylinder", "nx": 1000, "ny": 700, "steps": 30, "mrt": True},
        # grains in a box walled on all sides, two Dirichlet walls: the largest 2D lattice
        {"name": "medium_4096x2048", "kind": "medium", "nx": 4096, "ny": 2048, "steps": 20},
        # 64 uneven drops stepped together (the batched workload)
        {"name": "batch_64", "kind": "batch", "count": 64, "lo": 64, "hi": 512, "pick": 4, "steps": 32},
        # gradient of a misfit through autograd, whole call (simulation and tape made on the way)
        {"name": "gradient_256x256", "kind": "gradient", "nx": 256, "ny": 256, "steps": 64},
        # the same run recorded and reversed with a kept tape on a lattice beyond the caches
        {"name": "tape_1024x1024", "kind": "tape", "nx": 1024, "ny": 1024, "steps": 16},
        # D3Q19: freezing between rough walls, and a drop in a periodic box
        {"name": "fracture_256x128x30", "kind": "fracture", "nx": 256, "ny": 128, "nz": 30, "steps": 24},
        {"name": "box_256x256x256", "kind": "box", "nx": 256, "ny": 256, "nz": 256, "steps": 10},
        # Cahn-Hilliard smoothing of a grain image, 2D with walls and 3D walled along x
        {"name": "smooth_4096x2048", "kind": "smooth2", "nx": 4096, "ny": 2048, "iterations": 100, "periodic": False},
        {"name": "smooth_256x256x256", "kind": "smooth3", "nx": 256, "ny": 256, "nz": 256, "iterations": 60,
         "periodic": True},
    ]


def _side(rng: random.Random, lo: int, hi: int) -> int:
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["drop", "drop", "cylinder", "cylinder", "medium", "batch", "gradient", "tape", "fracture",
                       "box", "smooth2", "smooth3"])
    s = lambda lo, hi: _side(rng, lo, hi)  # noqa: E731
    if kind == "drop":
        return {"kind": kind, "nx": s(64, 512), "ny": s(48, 400), "steps": rng.randint(10, 50),
                "reduce": rng.random() < 0.5}
    if kind == "cylinder":
        return {"kind": kind, "nx": s(200, 2048), "ny": s(200, 2048), "steps": rng.randint(8, 30),
                "mrt": rng.random() < 0.4}
    if kind == "medium":
        return {"kind": kind, "nx": s(320, 4096), "ny": s(320, 2048), "steps": rng.randint(6, 20)}
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(6, 64), "lo": 64, "hi": rng.choice([160, 300, 512]),
                "pick": rng.randint(5, 999), "steps": rng.randint(8, 40)}
    if kind == "gradient":
        return {"kind": kind, "nx": s(64, 256), "ny": s(64, 256), "steps": rng.randint(16, 64)}
    if kind == "tape":
        return {"kind": kind, "nx": s(256, 1024), "ny": s(256, 1024), "steps": rng.randint(6, 16)}
    if kind == "fracture":
        return {"kind": kind, "nx": s(64, 256), "ny": s(32, 128), "nz": rng.randint(24, 30),
                "steps": rng.randint(8, 24)}
    if kind == "box":
        return {"kind": kind, "nx": s(48, 256), "ny": s(48, 256), "nz": s(48, 256), "steps": rng.randint(4, 10)}
    if kind == "smooth2":
        return {"kind": kind, "nx": s(100, 4096), "ny": s(100, 2048), "iterations": rng.randint(20, 100),
                "periodic": rng.random() < 0.5}
    return {"kind": kind, "nx": s(40, 256), "ny": s(40, 256), "nz": s(40, 256), "iterations": rng.randint(10, 60),
            "periodic": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs
def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _axes(shape):
    """Coordinates (x, y[, z]) of every node, shape (ny, nx) or (nz, ny, nx), FP64."""
    ax = [torch.arange(n, dtype=torch.float64, device=_dev()) for n in shape]
    return tuple(reversed(torch.meshgrid(*ax, indexing="ij")))


def _tanh(d, eps=4.0):
    return torch.tanh(2.0 * d / eps)


def _profile(n, r, modes=4):
    """A smooth periodic profile of n points with max |s| = 1."""
    x = torch.arange(n, dtype=torch.float64, device=_dev())
    s = torch.zeros_like(x)
    for _ in range(modes):
        k, a, ph = r.randint(1, 5), r.gauss(0.0, 1.0), r.uniform(0.0, 2.0 * math.pi)
        s = s + a * torch.cos(2.0 * math.pi * k * x / n + ph)
    return s / s.abs().max().clamp_min(1e-12)


def _inputs(case, seed, nx=None, ny=None):
    """Fields of one 2D lattice as a dict: phi0, cos_theta, phi, T (FP32 on the device, [ny, nx]), wall
    temperatures (bottom, top, left, right; FP32 vectors), and the options of the step."""
    r = random.Random(1000003 * int(seed) + 17)
    kind = case["kind"]
    nx, ny = nx or case["nx"], ny or case["ny"]
    x, y = _axes((ny, nx))
    d = {"px": True, "py": False, "tbc": [0, 0, 0, 0], "fixed": False, "Tsub": -1.0, "mrt": False,
         "mdot": kind in ("gradient", "tape")}
    one = torch.ones_like(x)
    walls = [torch.zeros(nx if w < 2 else ny, dtype=torch.float64, device=_dev()) for w in range(4)]
    if kind in ("drop", "batch", "gradient", "tape"):
        # a drop on a diffuse slab over a cold wall (the smallest stands on the bare wall), wettability and
        # wall temperature varying along the wall
        h_s = 0.0 if kind == "drop" and nx * ny < 20000 else 4.0 if d["mdot"] else 10.0
        rad = r.uniform(0.27, 0.33) * min(nx, ny)
        phi0 = 0.5 + 0.5 * _tanh(h_s - y) if h_s > 0 else 0.0 * one
        phi = (1.0 - phi0) * _tanh(rad - torch.hypot(x - nx * r.uniform(0.45, 0.55), y - h_s + 0.5))
        theta = r.uniform(60.0, 120.0) + 12.0 * _profile(nx, r)
        cth = torch.cos(torch.deg2rad(theta))[None, :] * one
        walls[0] = r.uniform(-1.6, -0.8) + 0.2 * _profile(nx, r)
        T = 0.0 * one
        d["tbc"] = [1, 0, 0, 0]
    elif kind == "cylinder":
        n = min(nx, ny)
        R_s, R_0 = 0.195 * n, r.uniform(0.13, 0.15) * n
        cx, cy = nx * r.uniform(0.47, 0.53), 0.25 * ny
        phi0 = 0.5 + 0.5 * _tanh(R_s - torch.hypot(x - cx, y - cy))
        phi = (1.0 - phi0) * _tanh(R_0 - torch.hypot(x - cx, y - cy - R_s))
        cth = math.cos(math.radians(r.uniform(50.0, 80.0))) * one
        d["Tsub"] = r.uniform(-1.2, -0.8)
        T = torch.where(phi0 >= 0.5, d["Tsub"] * one, 0.0 * one)
        d["fixed"], d["mrt"] = True, bool(case["mrt"])
    else:   # medium: one grain per cell of a coarse grid, left half liquid, cold left wall
        cell = 104
        gx, gy = -(-nx // cell), -(-ny // cell)
        g = torch.Generator().manual_seed(int(seed) + 5)
        rad = (20.0 + 26.0 * torch.rand(gy, gx, generator=g, dtype=torch.float64)).to(_dev())
        u = torch.rand(2, gy, gx, generator=g, dtype=torch.float64).to(_dev())
        ix, iy = (x // cell).long(), (y // cell).long()
        rr = rad[iy, ix]
        room = cell / 2.0 - 4.0 - rr
        gxc = (ix + 0.5) * cell + (2.0 * u[0][iy, ix] - 1.0) * room
        gyc = (iy + 0.5) * cell + (2.0 * u[1][iy, ix] - 1.0) * room
        phi0 = 0.5 + 0.5 * _tanh(rr - torch.hypot(x - gxc, y - gyc))
        phi = (1.0 - phi0) * _tanh(nx * r.uniform(0.45, 0.55) - x)
        cth = math.cos(math.radians(r.uniform(35.0, 55.0))) * one
        T = 0.0 * one
        d["px"], d["tbc"] = False, [0, 0, 1, 1]
        walls[2] = r.uniform(-1.2, -0.8) + 0.0 * walls[2]
    d.update(nx=nx, ny=ny, phi0=phi0.float(), cos_theta=cth.float().contiguous(), phi=phi.float(), T=T.float(),
             walls=[w.float() for w in walls])
    return d


def _material(d):
    m = W.Material(phi_src_mdot=int(d["mdot"]))
    if d["mrt"]:
        m.mrt, m.s_b, m.s_q, m.s_g = 1, 1.5, 1.2, 1.4
    return m


def _case2(d, name, host=False):
    f = (lambda t: t.cpu().numpy()) if host else (lambda t: t)
    return W.Case(name, d["nx"], d["ny"], d["px"], d["py"], list(d["tbc"]),
                  {w: d["walls"][w].double().cpu().numpy() for w in range(4)},
                  f(d["phi0"]), f(d["cos_theta"]), f(d["phi"]), f(d["T"]), _material(d),
                  substrate_fixed=d["fixed"], T_substrate=d["Tsub"])


def _inputs3(case, seed):
    """Fields of one 3D lattice (FP32, [nz, ny, nx]) and its boundary settings."""
    r = random.Random(1000003 * int(seed) + 29)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    x, y, z = _axes((nz, ny, nx))
    one = torch.ones_like(x)
    if case["kind"] == "fracture":
        ys = torch.arange(ny, dtype=torch.float64, device=_dev())
        xs = torch.arange(nx, dtype=torch.float64, device=_dev())

        def rough(amp, modes):
            h = torch.zeros(ny, nx, dtype=torch.float64, device=_dev())
            for _ in range(modes):
                ky = 2.0 * math.pi * r.randint(0, 4) / ny
                kx = 2.0 * math.pi * r.uniform(0.5, 6.0) / nx
                h = h + torch.cos(kx * xs[None, :] + ky * ys[:, None] + r.uniform(0.0, 2.0 * math.pi))
            return amp * h / max(1.0, math.sqrt(modes / 2.0))

        zc, both = (nz - 1) / 2.0, rough(1.2, 6)
        lo = zc - 7.0 + both + rough(0.8, 6)
        hi = zc + 7.0 + both + rough(0.8, 6)
        phi0 = 0.5 + 0.5 * _tanh(torch.maximum(lo[None] - z, z - hi[None]))
        liquid = _tanh(0.75 * nx - x)
        for (bx, by), rad in (((0.25, 0.25), 0.075), ((0.5, 0.5), 0.05)):
            rr = torch.sqrt((x - bx * nx) ** 2 + (y - by * ny) ** 2 + (z - 0.5 * nz) ** 2)
            liquid = torch.minimum(liquid, _tanh(rr - rad * nx))
        phi = (1.0 - phi0) * liquid
        cth = torch.cos(torch.deg2rad(90.0 + rough(15.0, 5).clamp(-30.0, 30.0)))[None] * one
        T, per, tbc, Tw = 0.0 * one, (False, True, True), [1, 0, 0, 0, 0, 0], [r.uniform(-1.2, -0.8)] + [0.0] * 5
    else:
        c = [(n - 1) / 2.0 + r.uniform(-2.0, 2.0) for n in (nx, ny, nz)]
        rad = r.uniform(0.22, 0.28) * min(nx, ny, nz)
        rr = torch.sqrt((x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2)
        phi0, cth, phi, T = 0.0 * one, 0.0 * one, _tanh(rad - rr), one
        per, tbc, Tw = (True, True, True), [0] * 6, [0.0] * 6
    # FP32 values from here on (the face temperature too, which the step holds in FP32)
    return {"phi0": phi0.float(), "cos_theta": cth.float().contiguous(), "phi": phi.float(), "T": T.float(), "per": per,
            "tbc": tbc, "Tw": [float(np.float32(v)) for v in Tw]}


def _image(case, seed):
    """A poorly sorted grain pack (uint8, 1 = solid): one disk or sphere per cell of a jittered grid, radii
    log-normal about 6 (2D) or 9 (3D) nodes, overlapping their neighbours."""
    shape = (case["ny"], case["nx"]) if case["kind"] == "smooth2" else (case["nz"], case["ny"], case["nx"])
    cell = 15
    median = 6.2 if len(shape) == 2 else 8.6
    g = torch.Generator().manual_seed(int(seed) + 11)
    cells = [-(-n // cell) + 2 for n in shape]
    rad = median * torch.exp(0.35 * torch.randn(*cells, generator=g)).clamp(0.3, 1.8).to(_dev())
    jit = torch.rand(len(shape), *cells, generator=g).to(_dev())
    pos = torch.meshgrid(*[torch.arange(n, device=_dev()) for n in shape], indexing="ij")
    img = torch.zeros(shape, dtype=torch.bool, device=_dev())
    for k in range(3 ** len(shape)):
        idx, rem = [], k
        for p in pos:
            idx.append(p // cell + rem % 3)
            rem //= 3
        d2 = torch.zeros(shape, device=_dev())
        for a, p in enumerate(pos):
            d2 += (p - (idx[a] - 1) * cell - cell * jit[a][tuple(idx)]) ** 2
        img |= d2 <= rad[tuple(idx)] ** 2
    return img.to(torch.uint8)


def _smooth_axes(case):
    p = bool(case["periodic"])
    return (p, p) if case["kind"] == "smooth2" else (False, p, p)


def _batch_sizes(case):
    """Sides log-uniform in [lo, hi], the longer one along x."""
    r = random.Random(case["pick"])
    out = []
    for _ in range(case["count"]):
        a, b = _side(r, case["lo"], case["hi"]), _side(r, case["lo"], case["hi"])
        out.append((max(a, b), min(a, b)))
    return out


def _target(case, seed):
    """A target liquid fraction near the initial one, [ny, nx], for the misfit."""
    r = random.Random(int(seed) + 3)
    x, y = _axes((case["ny"], case["nx"]))
    front = 9.0 + 3.0 * _profile(case["nx"], r)[None, :]
    return (0.75 + 0.25 * _tanh(y - front)).float()


# ------------------------------------------------------------------ a user's program
def _sim(d, name, row_block=None):
    if row_block is None:
        row_block, pad = autotune.lookup_layout(d["nx"], d["ny"])
    else:
        pad = 0
    return lbf.Sim(_case2(d, name), tile=autotune.lookup(d["nx"], d["ny"]), row_block=row_block, plane_pad=pad)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("drop", "cylinder", "medium"):
        d = _inputs(case, seed)
        s.update(sim=_sim(d, kind), phi=d["phi"], T=d["T"],
                 out=torch.empty((13, d["ny"], d["nx"]), dtype=torch.float32, device="cuda"))
    elif kind == "batch":
        ds = [_inputs(case, 100 * seed + i, nx, ny) for i, (nx, ny) in enumerate(_batch_sizes(case))]
        sims = [_sim(d, kind) for d in ds]
        tile = autotune.lookup_batch(64, 0) or (128, 32)
        s.update(sims=sims, batch=lbf.Batch(sims, tile=tile), init=[(d["phi"], d["T"]) for d in ds],
                 outs=[torch.empty((13, d["ny"], d["nx"]), dtype=torch.float32, device="cuda") for d in ds])
    elif kind == "gradient":
        d = _inputs(case, seed)
        s.update(model=_case2(d, kind, host=True), target=_target(case, seed),
                 cos_theta=d["cos_theta"].clone().requires_grad_(True),
                 wall_T=torch.cat(d["walls"]).requires_grad_(True))
    elif kind == "tape":
        d = _inputs(case, seed)
        sim = _sim(d, kind, row_block=0)
        s.update(sim=sim, tape=lbf.Tape(sim, case["steps"]), phi=d["phi"], T=d["T"], target=_target(case, seed),
                 fs=torch.empty((d["ny"], d["nx"]), dtype=torch.float32, device="cuda"))
    elif kind in ("fracture", "box"):
        d = _inputs3(case, seed)
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        host = {k: d[k].cpu().numpy() for k in ("phi0", "cos_theta", "phi", "T")}
        c3 = W3.Case3(kind, nx, ny, nz, d["per"], d["tbc"], d["Tw"], host["phi0"], host["cos_theta"], host["phi"],
                      host["T"], W.Material())
        rb, pad = autotune.lookup_layout3(nx, ny, nz)
        sim = lbf.Sim3(c3, plane_pad=pad, row_block=rb)
        sim.set_strip(autotune.lookup_strip3(nx, ny, nz))
        s.update(sim=sim, lib=lbf.load(), phi=d["phi"], T=d["T"],
                 out=torch.empty((14, nz, ny, nx), dtype=torch.float32, device="cuda"))
    else:
        img = _image(case, seed)
        need = 2 * ((img.numel() * 4 + 255) // 256 * 256)
        s.update(img=img, ws=torch.empty(need, dtype=torch.uint8, device="cuda"))
    return s


def _read2(sim, out):
    """Every read-out field of the current state into device memory (one call of the C ABI)."""
    lbf.check(lbf.load().lbf_read_fields(sim.h, C.c_void_p(out.data_ptr()), 1))
    return {k: out[i] for i, k in enumerate(FIELDS2)}


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("drop", "cylinder", "medium"):
        sim = s["sim"]
        sim.init_fields(s["phi"], s["T"])
        sim.step(case["steps"])
        got = _read2(sim, s["out"])
        if case.get("reduce"):
            red = sim.reduce()
            got["sums"] = [red[k] for k in ("sum_g", "sum_h", "sum_fs", "sum_liq", "umax")]
        return got
    if kind == "batch":
        for sim, (phi, T) in zip(s["sims"], s["init"]):
            sim.init_fields(phi, T)
        s["batch"].step(case["steps"])
        # the fields of a few of them (the driver of a sweep looks at some in passing)
        return [_read2(s["sims"][i], s["outs"][i]) for i in range(min(4, len(s["sims"])))]
    if kind == "gradient":
        ct, wt = s["cos_theta"], s["wall_T"]
        ct.grad = wt.grad = None
        phi, T, fs = lbf.freeze_fields(ct, wt, s["model"], case["steps"])
        loss = 0.5 * ((1.0 - fs - s["target"]) ** 2).sum() + 0.01 * (phi * T).sum()
        loss.backward()
        return {"phi": phi.detach(), "T": T.detach(), "fs": fs.detach(), "cos_theta": ct.grad, "wall_T": wt.grad}
    if kind == "tape":
        sim = s["sim"]
        sim.init_fields(s["phi"], s["T"])
        s["tape"].forward()
        fs = sim.field("fs", s["fs"])
        gc, gw = s["tape"].backward(seed_fs=(s["target"] - 1.0 + fs))
        return {"fs": fs, "cos_theta": gc, "wall_T": gw}
    if kind in ("fracture", "box"):
        sim, L = s["sim"], s["lib"]
        lbf.check(L.lbf3_init_fields(sim.h, C.c_void_p(s["phi"].data_ptr()), C.c_void_p(s["T"].data_ptr()), 1))
        sim.step(case["steps"])
        lbf.check(L.lbf3_read_fields(sim.h, C.c_void_p(s["out"].data_ptr()), 1))
        return {k: s["out"][i] for i, k in enumerate(FIELDS3)}
    return porous.ch_smooth(s["img"], _smooth_axes(case), case["iterations"], workspace=s["ws"])


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Bytes: a step reads and writes its state once (27 distributions and 6 lagged fields in 2D, 57 and 11 in
    3D, FP32) and reads its static fields; a reversed step reads the state and reads and writes the adjoint
    state; a smoothing step reads and writes its one plane.  Flops: the update rule's own operations."""
    kind = case["kind"]
    if kind == "batch":
        n = sum(a * b for a, b in _batch_sizes(case))
    else:
        n = case["nx"] * case["ny"] * case.get("nz", 1)
    k = case.get("steps", case.get("iterations"))
    if kind == "smooth2":
        return {"bytes": n * (8 * k + 5), "flops": n * k * 40}
    if kind == "smooth3":
        return {"bytes": n * (8 * k + 5), "flops": n * k * 80}
    if kind in ("fracture", "box"):
        return {"bytes": n * (k * 556 + 14 * 4 + 8), "flops": n * k * 1700}
    if kind in ("gradient", "tape"):
        # forward, recomputation, reverse (state read, adjoint of 27 + 5 planes read and written)
        return {"bytes": n * k * (2 * 268 + 132 + 256), "flops": n * k * 4000}
    return {"bytes": n * (k * 276 + 13 * 4 + 8), "flops": n * k * 800}


# ------------------------------------------------------------------ the method in 64 bits
# Velocity sets of Sec. 3.1 (order free: the outputs are fields, not populations).
_D2 = [(0, 0)] + [c for c in ((1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1))]
_D3 = [(x, y, z) for x in (0, 1, -1) for y in (0, 1, -1) for z in (0, 1, -1) if abs(x) + abs(y) + abs(z) <= 2]


def _weight(c):
    k = sum(abs(v) for v in c)
    return (4 / 9, 1 / 9, 1 / 36)[k] if len(c) == 2 else (1 / 3, 1 / 18, 1 / 36)[k]


class _Model:
    """The coupled update on a whole lattice with torch operations in FP64; axis a of a field is x, y[, z]."""

    def __init__(self, mat, per, phi0, cth, face_T, fixed=False, Tsub=0.0):
        self.m, self.per, self.phi0, self.cth = mat, per, phi0, cth
        self.face_T = face_T      # face 2 a + side: None (adiabatic) or the temperature on that face
        self.fixed, self.Tsub = fixed, Tsub
        self.dim = phi0.dim()
        self.c = _D2 if self.dim == 2 else _D3
        self.w = [_weight(c) for c in self.c]
        self.opp = [self.c.index(tuple(-v for v in c)) for c in self.c]
        self.Eref = mat.rho_ref * 2.0 * mat.cp_s * mat.cp_l / (mat.cp_s + mat.cp_l)
        self.lap0 = self.lap(phi0)

    def at(self, X, c):
        """X(x + c): wrapped, or the first node repeated beyond a wall."""
        for a, v in enumerate(c):
            if v:
                t = self.dim - 1 - a
                n = X.shape[t]
                if self.per[a]:
                    X = torch.roll(X, -v, t)
                elif v > 0:
                    X = torch.cat([X.narrow(t, 1, n - 1), X.narrow(t, n - 1, 1)], t)
                else:
                    X = torch.cat([X.narrow(t, 0, 1), X.narrow(t, 0, n - 1)], t)
        return X

    def grad(self, X, axes=None):
        out = [None] * self.dim
        for c, w in zip(self.c, self.w):
            if any(c):
                v = self.at(X, c)
                for a in range(self.dim):
                    if c[a]:
                        t = 3.0 * w * c[a] * v
                        out[a] = t if out[a] is None else out[a] + t
        return out

    def lap(self, X):
        s = 0.0
        for c, w in zip(self.c, self.w):
            if any(c):
                s = s + 6.0 * w * (self.at(X, c) - X)
        return s

    @staticmethod
    def zeta(s, Cw, zs, zl, zg):
        return s * zs + (1.0 - s) * (Cw * zl + (1.0 - Cw) * zg)

    def kcap(self, s, Cw):
        m = self.m
        return self.zeta(s, Cw, m.rho_s, m.rho_l, m.rho_g) * self.zeta(s, Cw, m.cp_s, m.cp_l, m.cp_g)

    def potential(self, phi, lphi, fs, lfs):
        m, p0, ct = self.m, self.phi0, self.cth
        a, k = 3.0 * m.sigma / m.eps, 3.0 * m.eps * m.sigma / 8.0
        mu = a * phi * (phi * phi - 1.0) - k * lphi
        mu = mu + 3.0 * a * p0 * p0 * phi + a * ct * p0 * (3.0 * phi * phi + p0 * p0 - 1.0) - k * ct * self.lap0
        return mu + 3.0 * a * fs * fs * phi + a * m.cos_psi * fs * (3.0 * phi * phi + fs * fs - 1.0) \
            - k * m.cos_psi * lfs

    def fraction(self, phihat):
        Cw = torch.clamp(0.5 * (1.0 - self.phi0 + phihat), 0.0, 1.0)
        return Cw, torch.clamp((Cw - self.m.pcm_floor) / (1.0 - self.m.pcm_floor), 0.0, 1.0)

    def start(self, phi, T):
        m, zero = self.m, torch.zeros_like(phi)
        mu = self.potential(phi, self.lap(phi), zero, zero)
        Cw, chi = self.fraction(phi)
        chi = torch.minimum(chi, 1.0 - self.phi0)
        K = self.kcap(self.phi0, Cw)
        rhoH = K * (T - m.T_m) + K * m.T_m + chi * m.rho_l * m.latent
        ET = self.Eref * T
        f = [torch.zeros_like(phi) for _ in self.c]
        g = [w * mu if any(c) else phi + (w - 1.0) * mu for c, w in zip(self.c, self.w)]
        h = [w * ET if any(c) else rhoH - ET + w * ET for c, w in zip(self.c, self.w)]
        lag = {k: torch.zeros_like(phi) for k in ("fs", "Q", "p")}
        lag["j"] = [torch.zeros_like(phi) for _ in range(self.dim)]
        lag["u"] = [torch.zeros_like(phi) for _ in range(self.dim)]
        return f, g, h, lag

    def moments(self, g, h, lag):
        m, p0 = self.m, self.phi0
        phihat, rhoH = sum(g), sum(h) + 0.5 * lag["Q"]
        Cw, chi = self.fraction(phihat)
        chi = torch.maximum(chi, lag["fs"]) if m.latch_fs else chi
        hi = 1.0 - p0
        chi = torch.where(chi < 0.0, torch.zeros_like(chi), torch.where(chi > hi, hi, chi))
        Kl, Ks = self.kcap(p0, Cw), self.kcap(torch.clamp(p0 + chi, max=1.0), Cw)
        Es, El = Ks * m.T_m, Kl * m.T_m + chi * m.rho_l * m.latent
        sol = rhoH < Es
        liq = (~sol) & (rhoH > El)
        span = El - Es
        flm = torch.where(span > 0, (rhoH - Es) / torch.where(span > 0, span, torch.ones_like(span)),
                          torch.ones_like(span))
        fl = torch.where(sol, torch.zeros_like(flm), torch.where(liq, torch.ones_like(flm), flm))
        T = torch.where(sol, rhoH / Ks, torch.where(liq, m.T_m + (rhoH - El) / Kl, torch.full_like(rhoH, m.T_m)))
        fs = chi * (1.0 - fl)
        mdot = (1.0 - m.rho_s / m.rho_l) * (fs - lag["fs"])
        if m.phi_src_mdot:
            divu = mdot
        else:
            divu = sum(self.grad(lag["u"][a])[a] for a in range(self.dim))
        fstot = torch.clamp(p0 + fs, max=1.0)
        return {"phihat": phihat, "rhoH": rhoH, "C": Cw, "chi": chi, "T": T, "fs": fs, "fstot": fstot, "mdot": mdot,
                "divu": divu, "phi": phihat / (1.0 - 0.5 * divu), "Ks": Ks, "Kl": Kl,
                "rho": self.zeta(fstot, Cw, m.rho_s, m.rho_l, m.rho_g)}

    def step(self, state, collide=True):
        m, D = self.m, range(self.dim)
        f, g, h, lag = state
        M = self.moments(g, h, lag)
        phi, rho, Cw, fs, st, mdot, T = (M[k] for k in ("phi", "rho", "C", "fs", "fstot", "mdot", "T"))
        tau = 3.0 * self.zeta(st, Cw, m.mu_s, m.mu_l, m.mu_g) / rho + 0.5
        ta = 3.0 * self.zeta(st, Cw, m.lam_s, m.lam_l, m.lam_g) / self.Eref + 0.5
        ts = 1.0 / (2.0 - 1.0 / ta)
        tg = 3.0 * m.mobility + 0.5
        gph, gr, gp = self.grad(phi), self.grad(rho), self.grad(lag["p"])
        mu = self.potential(phi, self.lap(phi), fs, self.lap(fs))
        F = [mu * gph[a] for a in D]
        mom = [sum(c[a] * fi for c, fi in zip(self.c, f) if c[a]) for a in D]
        us = [(mom[a] + 0.5 * F[a]) / rho for a in D]
        fd = [-st * us[a] for a in D]
        u = [us[a] + 0.5 * fd[a] for a in D]
        S = rho * mdot + sum(u[a] * gr[a] for a in D)
        Ft = [F[a] - gp[a] + gr[a] / 3.0 for a in D]
        uu, uFt = sum(v * v for v in u), sum(u[a] * Ft[a] for a in D)
        w0 = self.w[0]
        mrt = bool(m.mrt)
        t0 = 1.0 / m.s_b if mrt and m.s_b > 0 else tau
        p = (1.0 / 3.0) / (1.0 - w0) * (sum(fi for c, fi in zip(self.c, f) if any(c)) + 0.5 * S
                                        + (t0 - 0.5) * w0 * (S - 3.0 * uFt) - 1.5 * w0 * rho * uu)
        M.update(u=u, p=p, mu=mu)
        if not collide:
            return M
        j = [phi * u[a] for a in D]
        rhocp = rho * self.zeta(st, Cw, m.cp_s, m.cp_l, m.cp_g)
        Q, ET, cT = rhocp * T * mdot, self.Eref * T, rhocp * T
        src = ta if m.h_src_tau_a else ts
        nf, ng, heq = [], [], []
        for c, w, fi, gi in zip(self.c, self.w, f, g):
            dot = lambda v: sum((c[a] * v[a] for a in D if c[a]), torch.zeros_like(phi))  # noqa: E731
            cu, rest = dot(u), not any(c)
            P = 3.0 * cu + 4.5 * cu * cu - 1.5 * uu
            feq = 3.0 * p * (w - float(rest)) + rho * w * P
            Fi = w * (S + 3.0 * dot([F[a] + rho * fd[a] for a in D]) + 9.0 * cu * dot(Ft) - 3.0 * uFt)
            geq = (phi + (w - 1.0) * mu if rest else w * mu) + 3.0 * w * dot(j)
            Gi = w * (3.0 * dot([j[a] - lag["j"][a] for a in D]) + phi * M["divu"])
            nf.append((fi, fi - feq + 0.5 * Fi, Fi))
            ng.append((gi, gi - geq + 0.5 * Gi, Gi))
            heq.append(M["rhoH"] - ET + w * (ET - 1.5 * cT * uu) if rest else w * (ET + cT * P))
        f = [a - b / tau + s for a, b, s in nf]
        g = [a - b / tg + s for a, b, s in ng]
        if mrt:
            f = self.relax(f, [b for _, b, _ in nf], [("rho", m.s_b), ("e", m.s_b), ("eps", m.s_b), ("qx", m.s_q),
                                                      ("qy", m.s_q)], 1.0 / tau)
            g = self.relax(g, [b for _, b, _ in ng], [(k, m.s_g) for k in ("e", "eps", "qx", "qy", "pxx", "pxy")],
                           1.0 / tg)
        hn = []
        for i, o in enumerate(self.opp):
            a, e = h[i] - h[o] - heq[i] + heq[o], h[i] + h[o] - heq[i] - heq[o]
            hn.append(h[i] - 0.5 * a / ta - 0.5 * e / ts + (1.0 - 0.5 / src) * self.w[i] * Q)
        if self.fixed:
            Tw, held = self.Tsub, self.phi0 >= 0.5
            rH = M["Ks"] * Tw if Tw <= m.T_m else M["Kl"] * Tw + M["chi"] * m.rho_l * m.latent
            EW = self.Eref * Tw
            hn = [torch.where(held, torch.full_like(v, w * EW) if any(c) else rH - EW + w * EW, v)
                  for c, w, v in zip(self.c, self.w, hn)]
        return self.pull(f), self.pull(g), self.pull(hn, True), {"fs": fs, "Q": Q, "p": p, "j": j, "u": u}

    def relax(self, f, neq, moments, s0):
        """Moments that relax at a rate of their own, in the orthogonal D2Q9 basis."""
        poly = {"rho": lambda x, y, q: 1.0, "e": lambda x, y, q: 3.0 * q - 4.0,
                "eps": lambda x, y, q: 4.0 - 10.5 * q + 4.5 * q * q, "qx": lambda x, y, q: (3.0 * q - 5.0) * x,
                "qy": lambda x, y, q: (3.0 * q - 5.0) * y, "pxx": lambda x, y, q: x * x - y * y,
                "pxy": lambda x, y, q: x * y}
        for name, s in moments:
            if s > 0:
                r = [float(poly[name](c[0], c[1], c[0] ** 2 + c[1] ** 2)) for c in self.c]
                d = sum(a * b for a, b in zip(r, neq)) * ((s - s0) / sum(a * a for a in r))
                f = [v - a * d for a, v in zip(r, f)]
        return f

    def pull(self, X, heat=False):
        """Populations after streaming: half-way bounce-back at walls, anti-bounce-back of h at a Dirichlet wall;
        a link through several walls takes the last axis."""
        out = []
        for i, c in enumerate(self.c):
            v = self.at(X[i], tuple(-k for k in c))
            own = X[self.opp[i]]
            for a in range(self.dim):
                if c[a] and not self.per[a]:
                    t = self.dim - 1 - a
                    n, side = v.shape[t], 0 if c[a] > 0 else 1
                    s = own.narrow(t, 0 if side == 0 else n - 1, 1)
                    Tw = self.face_T[2 * a + side] if heat else None
                    if Tw is not None:
                        s = 2.0 * self.w[i] * self.Eref * (Tw.unsqueeze(t) if torch.is_tensor(Tw) else Tw) - s
                    v = torch.cat([s, v.narrow(t, 1, n - 1)] if side == 0 else [v.narrow(t, 0, n - 1), s], t)
            out.append(v)
        return out


def _model2(d, cth=None, walls=None):
    walls = [w.double() for w in d["walls"]] if walls is None else walls
    faces = [walls[w] if d["tbc"][w] else None for w in (2, 3, 0, 1)]   # left, right, bottom, top
    return _Model(_material(d), (d["px"], d["py"]), d["phi0"].double(),
                  d["cos_theta"].double() if cth is None else cth, faces, d["fixed"], float(np.float32(d["Tsub"])))


def _named(M, names):
    v = dict(M, fl=1.0 - M["fs"], **{"u" + a: t for a, t in zip("xyz", M["u"])})
    return {k: v[k] for k in names}


def _advance(model, phi, T, steps):
    state = model.start(phi, T)
    for _ in range(steps):
        state = model.step(state)
    return state


def _exact2(d, case):
    model = _model2(d)
    state = _advance(model, d["phi"].double(), d["T"].double(), case["steps"])
    M = model.step(state, collide=False)
    got = _named(M, FIELDS2)
    if case.get("reduce"):
        sums = [M["phihat"], sum(state[2]), M["fs"], M["chi"] - M["fs"]]
        got["sums"] = [float(v.sum()) for v in sums] + [float(torch.sqrt(M["u"][0] ** 2 + M["u"][1] ** 2).max())]
    return got


def _exact_gradient(case, seed):
    from torch.utils.checkpoint import checkpoint
    d = _inputs(case, seed)
    nx, ny = case["nx"], case["ny"]
    cth = d["cos_theta"].double().requires_grad_(True)
    wall = torch.cat(d["walls"]).double().requires_grad_(True)

    def model(c, w):
        return _model2(d, c, list(torch.split(w, [nx, nx, ny, ny])))

    def pack(s):
        return [*s[0], *s[1], *s[2], s[3]["fs"], s[3]["Q"], s[3]["p"], *s[3]["j"], *s[3]["u"]]

    def unpack(v):
        return list(v[:9]), list(v[9:18]), list(v[18:27]), {"fs": v[27], "Q": v[28], "p": v[29], "j": list(v[30:32]),
                                                            "u": list(v[32:34])}

    flat = pack(model(cth, wall).start(d["phi"].double(), d["T"].double()))
    for _ in range(case["steps"]):
        flat = checkpoint(lambda c, w, *v: tuple(pack(model(c, w).step(unpack(v)))), cth, wall, *flat,
                          use_reentrant=False)
    s = unpack(flat)
    M = model(cth, wall).moments(s[1], s[2], s[3])
    target = _target(case, seed).double()
    loss = 0.5 * ((1.0 - M["fs"] - target) ** 2).sum()
    if case["kind"] == "gradient":
        loss = loss + 0.01 * (M["phi"] * M["T"]).sum()
    loss.backward()
    got = {"fs": M["fs"].detach(), "cos_theta": cth.grad, "wall_T": wall.grad}
    if case["kind"] == "gradient":
        got.update(phi=M["phi"].detach(), T=M["T"].detach())
    return got


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gradient", "tape"):
        return _exact_gradient(case, seed)
    with torch.no_grad():
        if kind in ("drop", "cylinder", "medium"):
            return _exact2(_inputs(case, seed), case)
        if kind == "batch":
            sizes = _batch_sizes(case)
            return [_exact2(_inputs(case, 100 * seed + i, *sizes[i]), case) for i in range(min(4, len(sizes)))]
        if kind in ("fracture", "box"):
            d = _inputs3(case, seed)
            faces = [d["Tw"][f] if d["tbc"][f] else None for f in range(6)]
            model = _Model(W.Material(), d["per"], d["phi0"].double(), d["cos_theta"].double(), faces)
            state = _advance(model, d["phi"].double(), d["T"].double(), case["steps"])
            return _named(model.step(state, collide=False), FIELDS3)
        img = _image(case, seed)
        lat = _Model(W.Material(), _smooth_axes(case), torch.zeros(img.shape, dtype=torch.float64, device=img.device),
                     None, [])
        c = 2.0 * img.double() - 1.0
        for _ in range(case["iterations"]):
            c = c + 0.02 * lat.lap(c ** 3 - c - 2.0 * lat.lap(c))
        return torch.clamp(0.5 * (1.0 + c), 0.0, 1.0)
