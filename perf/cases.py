"""Measured work of the library: what its users have it do, over the range of
sizes, precisions and boxes that the workload presets, the benchmark and the
served form use.

Four kinds of case, each through the public entry points:
  sum       the stand-alone non-local Biot-Savart sum (vlb_biot_savart), or its
            far-field approximation (FarField.run), on filaments resident on
            the GPU: post-processing of a tangle, other integrators;
  velocity  the line velocity and mutual-friction force of a run's filaments
            (Run.eval_line_velocity): one Runge-Kutta stage on its own;
  fluid     the normal fluid alone (Run.step without filaments) and its
            populations afterwards (Run.read_state);
  steps     coupled steps from a checkpoint (write_state, seed, step or
            step_graph) and the state they lead to.

A run of FP32 or FP16 precision computes in single precision (FP16: the
populations are stored as halves); its results, which the library hands out
as doubles, are kept here in the precision they carry.
"""

import ctypes
import math

import numpy as np
import torch

import paper_2108_04435_amd as vlb

KAPPA = 0.1
TAU = 0.8
# coupling parameters of every workload preset
VORTEX = dict(kappa=KAPPA, core_a=1e-3, core_c=0.5, alpha=0.2, alpha_p=0.01,
              rho_s_over_rho_n=1.35, dxi_min=0.70, dxi_max=0.95, reconnect_dist=0.95,
              min_loop_pts=5)
STORE = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}
BYTES = {"f64": 8, "f32": 4, "f16": 2}


def listed():
    return [
        # one small ring of 64 points in a 32^3 box, the plain path: the
        # smallest run, where launches and latency are the time
        dict(name="ring_steps_f64", kind="steps", nx=32, ny=32, nz=32, walls=0, precision="f64",
             points=64, steps=20, graph=10, reconnect=False, balance=False, flow=0.01),
        # counterflow channel: walls on x and y, about 9.4e3 points, reconnection
        # and mass balance, captured chunks of steps
        dict(name="channel_steps_f32", kind="steps", nx=64, ny=64, nz=256, walls=3,
             precision="f32", points=9400, steps=10, graph=10, reconnect=True, balance=True,
             flow=0.02),
        # a served request of the largest lattice with few filaments: the
        # lattice part is the larger one
        dict(name="served_steps_f32", kind="steps", nx=128, ny=128, nz=256, walls=3,
             precision="f32", points=2000, steps=10, graph=0, reconnect=True, balance=True,
             flow=0.03),
        # the 256^3 tangle of the benchmark, halves stored
        dict(name="tangle_steps_f16", kind="steps", nx=256, ny=256, nz=256, walls=0,
             precision="f16", points=100000, steps=2, graph=0, reconnect=False, balance=True,
             flow=0.02),
        # line velocity in a box closed along z with the superfluid wall
        # images, the plain path
        dict(name="velocity_images_f64", kind="velocity", nx=48, ny=48, nz=128, walls=4,
             precision="f64", points=700, images=True, flow=0.01),
        # stand-alone sums: a thousand points; the plain path in a channel; a tangle
        dict(name="sum_1e3_f32", kind="sum", nx=64, ny=64, nz=64, walls=0, precision="f32",
             points=1000, cell=0),
        dict(name="sum_2e4_f64", kind="sum", nx=64, ny=64, nz=256, walls=3, precision="f64",
             points=20000, cell=0),
        dict(name="sum_1e5_f32", kind="sum", nx=256, ny=256, nz=256, walls=0, precision="f32",
             points=100000, cell=0),
        # the same tangle by the far-field approximation, two levels of cells
        dict(name="farfield_1e5", kind="sum", nx=256, ny=256, nz=256, walls=0, precision="f32",
             points=100000, cell=16),
        # the normal fluid alone: the 256^3 box, halves stored; the heater
        # channel (walls and velocity planes) in single precision; a ragged
        # closed box on the plain path
        dict(name="fluid_256_f16", kind="fluid", nx=256, ny=256, nz=256, walls=0,
             precision="f16", planes=False, steps=10),
        dict(name="fluid_heater_f32", kind="fluid", nx=128, ny=128, nz=512, walls=3,
             precision="f32", planes=True, steps=10),
        dict(name="fluid_ragged_f64", kind="fluid", nx=61, ny=67, nz=129, walls=7,
             precision="f64", planes=False, steps=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sum", "sum", "fluid", "fluid", "velocity", "steps", "steps"])
    if kind == "sum" and rng.random() < 0.3:
        # far field: a periodic box of whole cells
        cell = rng.choice([8, 16])
        n = [2 * cell * rng.randint(3, 128 // cell) for _ in range(3)]
        pts = min(_log(rng, 3000, 100000), n[0] * n[1] * n[2] // 60)
        return dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], walls=0, precision="f32", points=pts,
                    cell=cell)
    if kind == "sum":
        n = [_log(rng, 48, 256) for _ in range(3)]
        p = rng.choice(["f32", "f32", "f64"])
        pts = min(_log(rng, 64, 100000), n[0] * n[1] * n[2] // 60)
        return dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], walls=rng.choice([0, 0, 3, 4, 7]),
                    precision=p, points=pts, cell=0)
    if kind == "fluid":
        n = [_log(rng, 24, 288) for _ in range(3)]
        if rng.random() < 0.5:
            n = [rng.choice([32, 64, 96, 128, 192, 256]) for _ in range(3)]
        walls = rng.choice([0, 0, 3, 4, 7])
        return dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], walls=walls,
                    precision=rng.choice(["f64", "f32", "f16"]), steps=rng.randint(3, 10),
                    planes=bool(walls < 4 and rng.random() < 0.4))
    n = [_log(rng, 32, 160) for _ in range(3)]
    if rng.random() < 0.5:
        n = [rng.choice([32, 64, 128]), rng.choice([32, 64, 128]), rng.choice([64, 128, 256])]
    pts = min(_log(rng, 64, 20000), n[0] * n[1] * n[2] // 60)
    prec = rng.choice(["f64", "f32", "f16"])
    if kind == "velocity":
        return dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], walls=rng.choice([0, 3, 4]),
                    precision=prec, points=min(pts, 6000), images=rng.random() < 0.5, flow=0.01)
    return dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], walls=rng.choice([0, 0, 3]),
                precision=prec, points=pts, steps=2 * rng.randint(1, 4), graph=rng.choice([0, 2]),
                reconnect=rng.random() < 0.6, balance=rng.random() < 0.7, flow=0.02)


# ------------------------------------------------------------------- inputs

def _dims(case):
    return (case["nx"], case["ny"], case["nz"])


def _walls(case):
    return tuple(bool((case["walls"] >> a) & 1) for a in range(3))


def _clash(pts, ids, sub, L, walls, sep):
    """Of the points ``sub``, the rings (ids) that come within sep of a point
    of a ring of smaller id."""
    bad = torch.zeros(int(ids.max()) + 1, dtype=torch.bool, device=pts.device)
    p32 = pts.float()
    for c in range(0, sub.numel(), 1024):
        s = sub[c:c + 1024]
        d2 = torch.zeros(s.numel(), pts.shape[0], device=pts.device)
        for a in range(3):
            d = p32[s, a][:, None] - p32[None, :, a]
            if not walls[a]:
                d -= L[a] * torch.round(d / L[a])
            d2 += d * d
        hit = (d2 < sep * sep) & (ids[None, :] < ids[s][:, None])
        bad[ids[s][hit.any(dim=1)]] = True
    return bad


def _rings(case, seed, spacing=0.95, sep=1.5):
    """About case["points"] points of rings with radii in [4, 12] (smaller in
    small boxes), uniform centres and directions, at least sep apart where
    the box has room; links of each ring.  numpy arrays."""
    dims, walls = _dims(case), _walls(case)
    rng = np.random.default_rng(seed)
    r_hi = min(12.0, min(dims) / 4.0)
    r_lo = min(4.0, 0.5 * r_hi)
    if case["points"] < 400:   # a single ring of that many points, where it fits
        r_hi = r_lo = min(r_hi, max(1.5, 0.9 * case["points"] / (2 * math.pi)))
    # the rings' sizes are the case's, their places the seed's: every seed
    # has the same number of points
    size = np.random.default_rng(case["points"])
    radii = []
    left = case["points"]
    while left > 0:
        R = size.uniform(r_lo, r_hi)
        m = max(8, int(math.ceil(2 * math.pi * R / spacing)))
        radii.append((R, m))
        left -= m

    def place(R, m):
        c = np.empty(3)
        for a in range(3):
            lo, hi = (R + 0.5, dims[a] - 1.5 - R) if walls[a] else (0.0, dims[a])
            c[a] = rng.uniform(lo, hi)
        n = rng.normal(size=3)
        n /= np.linalg.norm(n)
        e1 = np.cross(n, np.eye(3)[int(np.argmin(np.abs(n)))])
        e1 /= np.linalg.norm(e1)
        e2 = np.cross(n, e1)
        th = 2 * np.pi * (np.arange(m) + rng.uniform()) / m
        p = c + R * (np.cos(th)[:, None] * e1 + np.sin(th)[:, None] * e2)
        for a in range(3):
            if not walls[a]:
                p[:, a] = np.mod(p[:, a], dims[a])
                p[p[:, a] >= dims[a], a] = 0.0
        return p

    rings = [place(R, m) for R, m in radii]
    todo = np.arange(len(rings))
    for _ in range(40):
        sizes = np.array([r.shape[0] for r in rings])
        ids = np.repeat(np.arange(len(rings)), sizes)
        pts = torch.as_tensor(np.concatenate(rings)).cuda()
        ids_t = torch.as_tensor(ids).cuda()
        sub = torch.as_tensor(np.nonzero(np.isin(ids, todo))[0]).cuda()
        # rings placed again come last, so that they give way to the others
        bad = _clash(pts, ids_t, sub, dims, walls, sep).cpu().numpy()
        keep = [rings[i] for i in range(len(rings)) if not bad[i]]
        clash = [i for i in range(len(rings)) if bad[i]]
        if not clash:
            break
        again = [place(*radii[i]) for i in clash]
        radii = [radii[i] for i in range(len(rings)) if not bad[i]] + [radii[i] for i in clash]
        todo = np.arange(len(keep), len(keep) + len(again))
        rings = keep + again
    pos = np.concatenate(rings)
    nxt, off = [], 0
    for r in rings:
        m = r.shape[0]
        nxt.append(off + (np.arange(m) + 1) % m)
        off += m
    return np.ascontiguousarray(pos), np.concatenate(nxt).astype(np.int32)


def _velocity(case, seed, flow):
    """u = flow along z plus noise of 1e-4, on the GPU, (3, nz, ny, nx)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    nx, ny, nz = _dims(case)
    u = 1e-4 * torch.randn((3, nz, ny, nx), generator=g, device="cuda", dtype=torch.float64)
    u[2] += flow
    return u


def _lattice(case):
    walls = _walls(case)
    body = (0.0, 0.0, 0.0)
    if walls[0] and walls[1] and not walls[2] and not case.get("planes"):
        # duct flow of mean velocity 0.02 (laminar square-duct relation)
        body = (0.0, 0.0, 28.45 * 0.1 * 0.02 / (case["nx"] * case["ny"]))
    planes = bool(case.get("planes"))
    return dict(nx=case["nx"], ny=case["ny"], nz=case["nz"], tau=TAU, walls=walls,
                plane_lo=planes, plane_hi=planes, plane_u=(0.0, 0.0, 0.03 if planes else 0.0),
                body_force=body, precision=case["precision"])


def _start(case, seed, vortex, n_cap):
    """A run on a stream of its own with the initial normal fluid written."""
    u = _velocity(case, seed, case.get("flow", 0.02))
    rho = torch.ones(u.shape[1:], device="cuda", dtype=torch.float64)
    torch.cuda.synchronize()
    run = vlb.Run(_lattice(case), vortex, n_cap, recon_cap=1 << 16, stream=torch.cuda.Stream())
    run._check(run.lib.vlb_write_fields(run.h, run._ptr(rho), run._ptr(u)))
    return run


def prepare(case, seed):
    kind = case["kind"]
    if kind == "fluid":
        return dict(case=case, run=_start(case, seed, dict(VORTEX), 1))
    pos, nxt = _rings(case, seed)
    n = pos.shape[0]
    if kind == "sum":
        p = torch.as_tensor(pos).cuda()
        q = torch.as_tensor(nxt).cuda()
        v = torch.empty((n, 3), dtype=torch.float64, device="cuda")
        st = dict(case=case, p=p, q=q, v=v)
        if case["cell"]:
            st["ff"] = vlb.FarField(_dims(case), n, case["cell"], 0.25, KAPPA, levels=2)
        else:
            lib = vlb.load_library()
            d = vlb.bs_desc(_dims(case), _walls(case), KAPPA, case["precision"])
            nb = ctypes.c_uint64(0)
            vlb._raise(lib, lib.vlb_biot_savart_workspace(ctypes.byref(d), n, ctypes.byref(nb)))
            ws = torch.empty(int(nb.value) + 256, dtype=torch.uint8, device="cuda")
            st.update(lib=lib, desc=d, ws=ws, base=(ws.data_ptr() + 255) // 256 * 256,
                      ws_bytes=int(nb.value))
        if case["precision"] != "f64":
            st["out"] = torch.empty((n, 3), dtype=torch.float32, device="cuda")
        return st
    if kind == "velocity":
        vor = dict(VORTEX, wall_images=case["images"], mass_balance=False)
        run = _start(case, seed, vor, int(1.4 * n) + 256)
        run.seed(pos, nxt)
        return dict(case=case, run=run)
    vor = dict(VORTEX, reconnect=case["reconnect"], mass_balance=case["balance"])
    run = _start(case, seed, vor, int(1.4 * n) + 256)
    run.seed(pos, nxt)
    saved, _ = run.read_state()
    # host buffers for the filaments, of the run's capacity
    return dict(case=case, run=run, saved=saved, pos=pos, nxt=nxt,
                xyz=np.zeros((run.n_cap, 3)), links=np.zeros(run.n_cap, dtype=np.int32))


# --------------------------------------------------------------------- work

def run(state):
    case = state["case"]
    kind = case["kind"]
    single = case["precision"] != "f64"
    if kind == "sum":
        n = state["p"].shape[0]
        if case["cell"]:
            state["ff"].run(state["p"], state["q"], state["v"])
        else:
            vp = ctypes.c_void_p
            vlb._raise(state["lib"], state["lib"].vlb_biot_savart(
                ctypes.byref(state["desc"]), n, vp(state["p"].data_ptr()),
                vp(state["q"].data_ptr()), vp(state["v"].data_ptr()), vp(state["base"]),
                ctypes.c_uint64(state["ws_bytes"]), vp(torch.cuda.current_stream().cuda_stream)))
        return state["out"].copy_(state["v"]) if single else state["v"]
    r = state["run"]
    if kind == "velocity":
        out = r.eval_line_velocity()
        return {k: v.astype(np.float32) for k, v in out.items()} if single else out
    if kind == "fluid":
        r.step(case["steps"])
        buf, _ = r.read_state()
        return buf.view(STORE[case["precision"]])
    # from the checkpoint, so that every pass is the same work
    r.write_state(state["saved"], 0)
    r.seed(state["pos"], state["nxt"])
    if case["graph"]:
        for _ in range(case["steps"] // case["graph"]):
            r.step_graph(case["graph"])
    else:
        r.step(case["steps"])
    xyz, links, n = state["xyz"], state["links"], ctypes.c_int64(0)
    r._check(r.lib.vlb_read_filaments(r.h, r.n_cap, xyz.ctypes.data_as(ctypes.c_void_p),
                                      links.ctypes.data_as(ctypes.c_void_p), ctypes.byref(n)))
    xyz[n.value:] = 0.0
    links[n.value:] = 0
    buf, _ = r.read_state()
    return dict(points=int(n.value), positions=xyz.astype(np.float32) if single else xyz,
                links=links, fluid=buf.view(STORE[case["precision"]]))


def work(case):
    """Arithmetic: 35 operations per (target, segment) pair of the closed form
    of the straight-segment integral (the far field counts its cells as
    such pairs), 200 per node update.  Bytes: positions and links in, the
    velocities out; every population read and written once per update."""
    nx, ny, nz = _dims(case)
    cells, kind = nx * ny * nz, case["kind"]
    b = BYTES[case["precision"]]
    n = case.get("points", 0)
    if kind == "sum":
        m = n if not case["cell"] else min(n, cells // case["cell"] ** 3)
        return {"bytes": 28.0 * n + (24.0 if b == 8 else 12.0) * n, "flops": 35.0 * n * m}
    if kind == "fluid":
        k = case["steps"]
        return {"bytes": 38.0 * b * cells * k, "flops": 200.0 * cells * k}
    fb = 8 if b == 8 else 4
    if kind == "velocity":
        walled = bin(case["walls"]).count("1") if case["images"] else 0
        return {"bytes": (19.0 * b + 3 * fb) * cells + 130.0 * n,
                "flops": 35.0 * n * n * 3 ** walled + 50.0 * cells}
    k = case["steps"]
    return {"bytes": k * ((57.0 * b + 6 * fb) * cells + 800.0 * n),
            "flops": k * (4 * 35.0 * n * n + 250.0 * cells)}


# ------------------------------------------------- the same in 64 bits, plain

C19 = ([0, 0, 0], [1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1],
       [1, 1, 0], [-1, -1, 0], [1, -1, 0], [-1, 1, 0], [1, 0, 1], [-1, 0, -1], [1, 0, -1],
       [-1, 0, 1], [0, 1, 1], [0, -1, -1], [0, 1, -1], [0, -1, 1])
W19 = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
OPP = [0] + [i + 1 if i % 2 else i - 1 for i in range(1, 19)]


def _exact_sum(pos, nxt, dims, walls, images=False):
    """Non-local velocity: every segment at the nearest periodic image of its
    start (decided on the 32-bit position grid) but the two that touch the
    target; with images also every reflection in the closed axes' walls."""
    n = pos.shape[0]
    nl = nxt.long()
    prv = torch.empty_like(nl)
    prv[nl] = torch.arange(n, device=pos.device)
    L = [float(d) for d in dims]
    seg = pos[nl] - pos
    for a in range(3):
        if not walls[a]:
            seg[:, a] -= L[a] * (seg[:, a] > 0.5 * L[a]).double()
            seg[:, a] += L[a] * (seg[:, a] < -0.5 * L[a]).double()
    copies = [([0, 0, 0], 1.0)]
    if images:
        copies = []
        opts = [(0, 1, 2) if walls[a] else (0,) for a in range(3)]
        for cz in opts[2]:
            for cy in opts[1]:
                for cx in opts[0]:
                    c = [cx, cy, cz]
                    copies.append((c, (-1.0) ** sum(1 for x in c if x)))
    out = torch.zeros_like(pos)
    step = max(1, (1 << 24) // n)
    for refl, sign in copies:
        src, sg = pos.clone(), seg.clone()
        for a in range(3):
            if refl[a]:
                src[:, a] = 2.0 * (-0.5 if refl[a] == 1 else L[a] - 0.5) - src[:, a]
                sg[:, a] = -sg[:, a]
        for c in range(0, n, step):
            t = torch.arange(c, min(n, c + step), device=pos.device)
            R1 = []
            for a in range(3):
                r = src[None, :, a] - pos[t, a][:, None]
                if not walls[a]:
                    q = 4294967296.0 / L[a]
                    raw = (torch.floor(src[:, a] * q).long()[None, :]
                           - torch.floor(pos[t, a] * q).long()[:, None])
                    r -= L[a] * torch.div(raw + (1 << 31), 1 << 32, rounding_mode="floor").double()
                R1.append(r)
            R2 = [R1[a] + sg[None, :, a] for a in range(3)]
            n1 = (R1[0] ** 2 + R1[1] ** 2 + R1[2] ** 2).sqrt()
            n2 = (R2[0] ** 2 + R2[1] ** 2 + R2[2] ** 2).sqrt()
            p = n1 * n2
            f = (n1 + n2) / (p * (p + R1[0] * R2[0] + R1[1] * R2[1] + R1[2] * R2[2]))
            if not any(refl):
                f[t - c, t] = 0.0
                f[t - c, prv[t]] = 0.0
            f *= sign
            out[t, 0] += (f * (R1[1] * R2[2] - R1[2] * R2[1])).sum(1)
            out[t, 1] += (f * (R1[2] * R2[0] - R1[0] * R2[2])).sum(1)
            out[t, 2] += (f * (R1[0] * R2[1] - R1[1] * R2[0])).sum(1)
    return out * (KAPPA / (4 * math.pi))


def _exact_velocity(case, seed):
    """Line velocity and force: non-local sum and the local term, the normal
    fluid interpolated from the 8 nodes around a point (zero beyond a wall),
    the equation of motion and the reaction."""
    dims, walls = _dims(case), _walls(case)
    posn, nxtn = _rings(case, seed)
    pos, nl = torch.as_tensor(posn).cuda(), torch.as_tensor(nxtn).cuda().long()
    vs = _exact_sum(pos, nl, dims, walls, case["images"])
    prv = torch.empty_like(nl)
    prv[nl] = torch.arange(nl.numel(), device=nl.device)
    dp, dm = pos[nl] - pos, pos - pos[prv]
    for d in (dp, dm):
        for a in range(3):
            if not walls[a]:
                d[:, a] -= dims[a] * torch.round(d[:, a] / dims[a])
    lp, lm = dp.norm(dim=1, keepdim=True), dm.norm(dim=1, keepdim=True)
    den = lp * lm * (lp + lm)
    sp = (lm ** 2 * dp + lp ** 2 * dm) / den
    sp = sp / sp.norm(dim=1, keepdim=True)
    spp = 2 * (lm * dp - lp * dm) / den
    beta = KAPPA / (4 * math.pi) * torch.log(
        2 * torch.sqrt(lp * lm) / (math.exp(VORTEX["core_c"]) * VORTEX["core_a"]))
    vs = vs + beta * torch.cross(sp, spp, dim=1)
    u = _velocity(case, seed, case["flow"])
    base = torch.floor(pos).long()
    fr = pos - base
    vn = torch.zeros_like(pos)
    for o in range(8):
        w = torch.ones(pos.shape[0], device=pos.device, dtype=torch.float64)
        node = []
        for a in range(3):
            k = (o >> a) & 1
            w = w * (fr[:, a] if k else 1 - fr[:, a])
            c = base[:, a] + k
            if walls[a]:
                w = w * ((c >= 0) & (c < dims[a])).double()
                c = c.clamp(0, dims[a] - 1)
            node.append(c % dims[a])
        vn += w[:, None] * u[:, node[2], node[1], node[0]].T
    rel = vn - vs
    sxw = torch.cross(sp, rel, dim=1)
    sdot = vs + VORTEX["alpha"] * sxw - VORTEX["alpha_p"] * torch.cross(sp, sxw, dim=1)
    force = VORTEX["rho_s_over_rho_n"] * KAPPA * torch.cross(sp, sdot - vs, dim=1) * (0.5 * (lp + lm))
    return {k: v.cpu().numpy() for k, v in
            dict(vs=vs, vn=vn, sdot=sdot, force=force).items()}


def _exact_fluid(case, seed):
    """Forced BGK collision and streaming of the whole distributions."""
    lat = _lattice(case)
    dims, walls = _dims(case), lat["walls"]
    om = 1.0 / TAU
    pref = 1.0 - 0.5 * om
    g = lat["body_force"]

    def dot(i, v):
        return sum(C19[i][a] * v[a] for a in range(3) if C19[i][a])

    def feq(i, drho, v, uu):
        # equilibrium less the weight
        cu = dot(i, v) if i else 0.0
        return W19[i] * (drho + (1 + drho) * (3 * cu + 4.5 * cu * cu - 1.5 * uu))

    u = _velocity(case, seed, 0.02)
    uu = (u * u).sum(0)
    d = torch.stack([feq(i, torch.zeros_like(uu), u, uu) for i in range(19)])
    del u, uu
    for _ in range(case["steps"]):
        for z, on in ((0, lat["plane_lo"]), (dims[2] - 1, lat["plane_hi"])):
            if on:
                pu = lat["plane_u"]
                puu = sum(x * x for x in pu)
                for i in range(19):
                    d[i, z] = feq(i, 0.0, pu, puu)
        drho = d.sum(0)
        v = []
        for a in range(3):
            j = sum(C19[i][a] * d[i] for i in range(19) if C19[i][a])
            v.append((j + 0.5 * g[a]) / (1 + drho))
        uu = v[0] ** 2 + v[1] ** 2 + v[2] ** 2
        ug = sum(v[a] * g[a] for a in range(3))
        for i in range(19):
            cu, cg = (dot(i, v), dot(i, g)) if i else (0.0, 0.0)
            force = W19[i] * pref * (3 * (cg - ug) + 9 * cu * cg)
            d[i] += om * (feq(i, drho, v, uu) - d[i]) + force
        new = torch.empty_like(d)
        for i in range(19):
            c = C19[i]
            new[i] = torch.roll(d[i], shifts=(c[2], c[1], c[0]), dims=(0, 1, 2))
            for a in range(3):
                if walls[a] and c[a]:
                    # the node next to the wall that the population leaves
                    sl = [slice(None)] * 3
                    sl[2 - a] = 0 if c[a] > 0 else dims[a] - 1
                    new[i][tuple(sl)] = d[OPP[i]][tuple(sl)]
        d = new
        del new
    return d.reshape(-1) * (1024.0 if case["precision"] == "f16" else 1.0)


def exact(case, seed):
    if case["kind"] == "sum":
        pos, nxt = _rings(case, seed)
        return _exact_sum(torch.as_tensor(pos).cuda(), torch.as_tensor(nxt).cuda(), _dims(case),
                          _walls(case))
    if case["kind"] == "velocity":
        return _exact_velocity(case, seed)
    if case["kind"] == "fluid":
        return _exact_fluid(case, seed)
    return None   # a whole coupled step has no short plain form
