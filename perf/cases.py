"""The work that users of this library have it do, as cases that can be timed.

A case is one pass through the public Python entry points
(``paper_2008_06134_amd.vi``), on inputs made on the GPU from a seed:

open     a volume that has just been loaded is laid out for rendering
         (quads or bricks, empty-space map, occupancy bits): what a viewer
         does for a new scan, and per time step of a 4D one
build    the light has moved: the attenuation stack is built again
render   the camera has moved: one frame from a resident stack
frame    both have moved: the stack, then one frame from it
serve    a burst of requests of several sessions to the request server

Volumes are CT-like phantoms (nested ellipsoids, a dense shell, inserts,
vessel-like tubes, scanner noise) or a noisy sphere; most of a volume is
empty, as a scan is.  Every buffer a program would keep (volume, transfer
function, stack, image) is made in ``prepare``.

``exact`` computes the same outputs in 64 bits with plain torch.
"""
from __future__ import annotations

import math
import random

import torch
import torch.nn.functional as F

from paper_2008_06134_amd import vi

DEV = "cuda"
TF_ENTRIES = 256

# what every case holds unless it says otherwise
DEFAULTS = {
    "content": "phantom",     # sphere | phantom (with vessels)
    "edge": 256, "voxels": "u16", "layout": "quads", "cell": 16, "bits": True, "entries": TF_ENTRIES,
    "slabs": 256, "res": 512, "stack": "f32", "rows": True, "darken": 0.0, "point": False,
    "width": 1024, "height": 1024, "camera": "persp", "mode": "shell", "grid": 0, "shells": 1, "step": 0.5,
}


def _case(name, kind, **over):
    c = {"name": name, "kind": kind, **DEFAULTS, **over}
    return c


def listed():
    return [
        # a thumbnail or a preview while the light is dragged: 64^3 u8, a few
        # workgroups of work, so launches and latency are what it costs
        _case("small frame", "frame", content="sphere", edge=64, voxels="u8", slabs=32, res=64, width=256, height=256,
              camera="ortho"),
        # the calls with their default arguments (linear volume, no map,
        # tiled stack) at the sizes of the paper's figures: 256^3, 128 slices
        # of 256^2, a 512^2 viewport
        _case("default frame", "frame", layout="linear", cell=0, bits=False, slabs=128, res=256, rows=False,
              width=512, height=512),
        # an ordinary scan: 256^3, 256 slices of 512^2, 1024^2 image
        _case("medium build", "build"),
        # the same scan under the 5 x 5 cone lattice, the richest gather
        _case("medium lattice", "render", mode="cone", grid=5),
        # the benchmark's configuration: 512^3, 512 slices of 1024^2, full HD
        _case("large build", "build", edge=512, slabs=512, res=1024),
        _case("large shell", "render", edge=512, slabs=512, res=1024, width=1920, height=1080),
        _case("large cone", "render", edge=512, slabs=512, res=1024, width=1920, height=1080, mode="cone"),
        # the largest volume in the precision form: 1024^3 half voxels in
        # bricks, bfloat16 optical depth
        _case("precision frame", "frame", edge=1024, voxels="f16", layout="bricks", cell=32, slabs=512, res=1024,
              stack="bf16", width=1920, height=1080, mode="cone"),
        # a lamp near the object: point light, ragged sizes, half stack
        _case("point frame", "frame", edge=301, voxels="u8", slabs=300, res=601, stack="f16", point=True,
              width=1283, height=717, mode="cone"),
        # local Phong shading, the paper's comparison mode: no stack
        _case("phong frame", "render", edge=384, slabs=256, res=512, width=1280, height=720, mode="phong"),
        # a new 512^3 scan is laid out
        _case("open volume", "open", edge=512),
        # eight frames of four viewers' sessions (128^3 to 320^3), cameras
        # orbiting, each light moving every third burst
        _case("serve burst", "serve", edge=320, width=1280, height=720),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: edges 40 to 512, any voxel and stack
    type, layout, light and gather, images from 64^2 to full HD."""
    kind = rng.choice(["build", "build", "render", "render", "render", "frame", "frame", "open", "serve"])
    edge = _log_int(rng, 40, 512)
    c = {"kind": kind, **DEFAULTS, "edge": edge, "content": rng.choice(["phantom", "phantom", "sphere"]),
         "voxels": rng.choice(["u8", "u16", "u16", "f16", "f32"]),
         "layout": rng.choice(["linear", "bricks", "quads", "quads"]),
         "cell": rng.choice([0, 8, 16, 16, 32]), "entries": rng.choice([64, 256, 256, 1024])}
    c["bits"] = c["cell"] > 0 and rng.random() < 0.8
    c["slabs"] = max(8, min(512, int(edge * rng.uniform(0.4, 1.2))))
    c["res"] = max(24, min(1024, int(edge * rng.uniform(0.8, 2.2))))
    c["rows"] = rng.random() < 0.75
    c["stack"] = rng.choice(["f32", "f32", "bf16", "f16"] if c["rows"] else ["f32", "f32", "bf16"])
    c["darken"] = rng.choice([0.0, 0.0, 0.0, 1.0])
    c["point"] = rng.random() < 0.25
    c["width"], c["height"] = _log_int(rng, 64, 1920), _log_int(rng, 64, 1080)
    c["camera"] = rng.choice(["persp", "persp", "persp", "ortho"])
    c["mode"] = rng.choice(["none", "shadow", "shell", "shell", "cone", "cone", "phong"])
    c["grid"] = rng.choice([0, 0, 3, 5]) if c["mode"] == "cone" else 0
    c["shells"] = rng.choice([1, 1, 2]) if c["mode"] == "shell" else 1
    c["step"] = rng.choice([0.5, 0.5, 1.0])
    if kind == "open":
        c["layout"], c["cell"], c["bits"] = rng.choice(["bricks", "quads"]), rng.choice([8, 16, 16, 32]), True
    if kind == "serve":
        c["edge"], c["width"], c["height"] = max(96, edge * 5 // 8), min(c["width"], 1280), min(c["height"], 720)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _tf_table(case):
    """Opacity 0 below 0.20 of the value range, then skin, soft tissue and bone
    (a ramp for the sphere); float32, K x 4, on the host."""
    K = case["entries"]
    v = torch.arange(K, dtype=torch.float64) / (K - 1)
    if case["content"] == "sphere":
        return torch.stack([v, 1.0 - v, torch.full_like(v, 0.5), v], 1).float()
    pts = [(0.00, (0.0, 0.0, 0.0, 0.0)), (0.20, (0.8, 0.5, 0.4, 0.0)), (0.25, (0.8, 0.5, 0.4, 0.02)),
           (0.35, (0.9, 0.6, 0.5, 0.05)), (0.60, (1.0, 0.9, 0.8, 0.30)), (0.75, (1.0, 1.0, 1.0, 0.90)),
           (1.00, (1.0, 1.0, 1.0, 1.00))]
    out = torch.zeros(K, 4, dtype=torch.float64)
    for (x0, a), (x1, b) in zip(pts[:-1], pts[1:]):
        m = (v >= x0) & (v <= x1)
        t = ((v[m] - x0) / (x1 - x0))[:, None]
        out[m] = torch.tensor(a, dtype=torch.float64) * (1 - t) + torch.tensor(b, dtype=torch.float64) * t
    return out.float()


def _noise(N, gen, spacing=32.0, octaves=3):
    """Value noise in [0, 1]: random lattices, the spacing halving per octave."""
    out, total = torch.zeros(N, N, N, device=DEV), 0.0
    for o in range(octaves):
        G = int(math.ceil(N / (spacing / 2 ** o))) + 1
        lat = torch.rand(1, 1, G, G, G, generator=gen, device=DEV)
        out += 0.5 ** o * F.interpolate(lat, size=(N, N, N), mode="trilinear", align_corners=False)[0, 0]
        total += 0.5 ** o
    return out.div_(total)


def _voxels(case, seed):
    """The volume as loaded: raw[z][y][x] on the GPU (12-bit values in int16 for
    u16; scaled to 0..255 for u8; normalised for f16 and f32)."""
    N, r = case["edge"], random.Random(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    x = (torch.arange(N, device=DEV, dtype=torch.float32) + 0.5) / N
    if case["content"] == "sphere":
        c, rad = x - 0.5, 0.375 * r.uniform(0.95, 1.05)
        inside = c[:, None, None] ** 2 + c[None, :, None] ** 2 + c[None, None, :] ** 2 <= rad * rad
        val = (200 + torch.randint(-20, 21, (N, N, N), generator=gen, device=DEV)) * (4095.0 / 255.0)
        val = val * inside
    else:
        n1, n2 = _noise(N, gen), _noise(N, gen)
        c = [0.5 + r.uniform(-0.01, 0.01) for _ in range(3)]
        body = [a * r.uniform(0.97, 1.03) for a in (0.40, 0.34, 0.42)]
        shell = [0.86 * a for a in body]
        ells = [(c, body, 1000.0 + r.uniform(-30, 30)), (c, shell, 3000.0 + r.uniform(-100, 100)),
                (c, [a - 6.0 / 256.0 for a in shell], 1100.0 + r.uniform(-30, 30))]
        for _ in range(3):
            ells.append(([a + r.uniform(-0.4, 0.4) * s for a, s in zip(c, shell)],
                         [r.uniform(0.04, 0.10) for _ in range(3)], r.uniform(1500.0, 4000.0)))
        val = torch.zeros(N, N, N, device=DEV)
        inside = None
        for cen, ax, v in ells:
            q = [((x - cen[k]) / ax[k]) ** 2 for k in range(3)]
            cov = (q[2][:, None, None] + q[1][None, :, None] + q[0][None, None, :]).sqrt_()
            cov = cov.sub_(1.0).mul_(-min(ax) * N).add_(0.5).clamp_(0.0, 1.0)
            val.lerp_(torch.full((), v, device=DEV), cov)
            inside = cov if inside is None else inside
        tube = ((0.035 - (n1 - 0.5).abs()) / 0.015).clamp_(0, 1) * ((0.035 - (n2 - 0.5).abs()) / 0.015).clamp_(0, 1)
        val.lerp_(torch.full((), 3500.0, device=DEV), tube.mul_(inside))
        del n1, n2, tube, inside, cov
        val += 30.0 * torch.randn(N, N, N, generator=gen, device=DEV)
    raw = val.round_().clamp_(0, 4095)
    if case["voxels"] == "u8":
        return (raw * (255.0 / 4095.0)).round_().to(torch.uint8)
    if case["voxels"] == "u16":
        return raw.to(torch.int16)
    return (raw.double() / 4095.0).to(torch.float16 if case["voxels"] == "f16" else torch.float32)


def _on_sphere(az, el):
    return [math.cos(el) * math.cos(az), math.cos(el) * math.sin(az), math.sin(el)]


def _light(case, r):
    """(direction, position): a lamp 25 to 45 degrees above the object; for a
    point light 1.2 to 2.5 edges from its centre."""
    d = _on_sphere(r.uniform(0, 2 * math.pi), math.radians(r.uniform(25.0, 45.0)))
    if case["point"]:
        dist = r.uniform(1.2, 2.5)
        return None, [0.5 + dist * a for a in d]
    return [-a for a in d], None


def _camera(case, az, width, height):
    if case["camera"] == "ortho":
        d = _on_sphere(az, 0.0)
        return {"kind": "ortho", "eye": [0.5 + 1.5 * a for a in d], "target": [0.5] * 3, "up": [0.0, 0.0, 1.0],
                "fovy_deg": 0.0, "ortho_half_h": 0.75, "width": width, "height": height}
    d = _on_sphere(az, math.radians(20.0))
    return {"kind": "persp", "eye": [0.5 + 2.0 * a for a in d], "target": [0.5] * 3, "up": [0.0, 0.0, 1.0],
            "fovy_deg": 40.0, "ortho_half_h": 0.0, "width": width, "height": height}


def _opts(case):
    o = {}
    if case["mode"] == "cone" and case["grid"]:
        o["cone_grid"] = case["grid"]
    if case["mode"] == "shell" and case["shells"] > 1:
        o["shell_count"], o["shell_w"] = case["shells"], [1.0, 0.5]
    return o


def _stack_args(case):
    return ({"f32": vi.VI_F32, "bf16": vi.VI_BF16, "f16": vi.VI_F16}[case["stack"]],
            vi.VI_STACK_ROWS if case["rows"] else vi.VI_STACK_TILED)


def _laid_out(case, vol, tf):
    if case["layout"] == "quads":
        vol = vol.to_quads()
    elif case["layout"] == "bricks":
        vol = vol.to_bricks()
    if case["cell"]:
        vol = vol.with_minmax(case["cell"])
        if case["bits"]:
            vol = vol.with_occupancy(tf)
    return vol


def _sessions(case, seed):
    """The serve case's viewers: (volume case, light angles, camera angle)."""
    out = []
    for s, f in enumerate((0.4, 0.6, 0.8, 1.0)):
        e = max(48, int(case["edge"] * f))
        r = random.Random(seed * 16 + s)
        vc = {**case, "edge": e, "content": "phantom", "voxels": "u16", "layout": "quads", "cell": 16, "bits": True,
              "entries": TF_ENTRIES, "slabs": e, "res": min(2 * e, 1024), "stack": "f32", "rows": True, "point": False,
              "darken": 0.0, "camera": "persp", "grid": 0, "shells": 1, "step": 0.5}
        out.append((vc, [_light(vc, r)[0] for _ in range(4)], r.uniform(0, 2 * math.pi)))
    return out


def _burst(case, sessions, b):
    """The requests of burst b: two frames of each session, the camera turning
    two degrees a frame, the light moving every third burst."""
    out = []
    for k in range(2):
        for s, (vc, lights, az) in enumerate(sessions):
            w, h = (case["width"], case["height"]) if (s + k) % 2 else (max(16, case["width"] * 2 // 5),
                                                                       max(16, case["height"] * 2 // 3))
            out.append({"session": s, "light": lights[((b + s) // 3) % 4], "mode": "cone" if (s + k) % 2 else "shell",
                        "cam": _camera(vc, az + math.radians(2.0) * (2 * b + k), w, h)})
    return out


def _inputs(case, seed):
    """The plain values both prepare and exact start from."""
    r = random.Random(seed + 7)
    light, position = _light(case, r)
    return light, position, _camera(case, r.uniform(0, 2 * math.pi), case["width"], case["height"])


def prepare(case, seed):
    if case["kind"] == "serve":
        sessions, vols = _sessions(case, seed), []
        for s, (vc, _, _) in enumerate(sessions):
            tf = vi.TF(_tf_table(vc).to(DEV))
            vols.append((_laid_out(vc, vi.Volume(_voxels(vc, seed * 16 + s)), tf), tf))
        # room for one and a half stacks a session: lights that come back
        # after others find theirs gone
        need = sum(vi.slices_bytes(vc["slabs"], vc["res"], vi.VI_F32, vi.VI_STACK_ROWS) for vc, _, _ in sessions)
        srv = vi.Server(need + need // 2)
        outs = [torch.zeros(q["cam"]["height"], q["cam"]["width"], 4, device=DEV) for q in _burst(case, sessions, 0)]
        torch.cuda.synchronize()  # the server renders on streams of its own
        return {"case": case, "sessions": sessions, "vols": vols, "server": srv, "burst": 0, "outs": outs,
                "ids": [srv.register(v, t) for v, t in vols]}
    light, position, cam = _inputs(case, seed)
    tf = vi.TF(_tf_table(case).to(DEV))
    vol = vi.Volume(_voxels(case, seed))
    st = {"case": case, "tf": tf, "light": light, "position": position, "cam": cam, "opts": _opts(case)}
    if case["kind"] == "open":
        st["vol"] = vol
        return st
    st["vol"] = vol = _laid_out(case, vol, tf)
    dtype, layout = _stack_args(case)
    if case["mode"] == "phong" and case["kind"] == "render":
        st["stack"] = vi.light_frame(light, case["slabs"], case["res"], position=position)
    elif case["mode"] != "none" or case["kind"] != "render":
        st["buffer"] = vi.stack_buffer(case["slabs"], case["res"], dtype, DEV, layout)
        st["buffer"].zero_()
        if case["kind"] == "render":
            st["stack"] = vi.build_attenuation(vol, tf, light, case["slabs"], case["res"], dtype, st["buffer"],
                                               layout=layout, darken=case["darken"], position=position)
    if case["kind"] != "build":
        st["image"] = torch.zeros(case["height"], case["width"], 4, device=DEV)
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "open":
        vol = state["vol"].to_quads() if case["layout"] == "quads" else state["vol"].to_bricks()
        vol = vol.with_minmax(case["cell"]).with_occupancy(state["tf"])
        return {"voxels": vol.data, "map": vol.minmax, "bits": vol.occ}
    if case["kind"] == "serve":
        srv, sessions, tickets = state["server"], state["sessions"], []
        for q, out in zip(_burst(case, sessions, state["burst"]), state["outs"]):
            vc = sessions[q["session"]][0]
            tickets.append(srv.submit(state["ids"][q["session"]], q["light"], vc["slabs"], vc["res"], q["cam"],
                                      q["mode"], vc["step"], out=out, layout=vi.VI_STACK_ROWS)[0])
        state["burst"] += 1
        for t in tickets:
            if srv.wait(t) != 0:
                raise RuntimeError("a request failed")
        return list(state["outs"])
    vol, tf = state["vol"], state["tf"]
    stack, out = state.get("stack"), {}
    if case["kind"] != "render":
        dtype, layout = _stack_args(case)
        stack = vi.build_attenuation(vol, tf, state["light"], case["slabs"], case["res"], dtype, state["buffer"],
                                     layout=layout, darken=case["darken"], position=state["position"])
        out["stack"] = stack.dense() if case["rows"] else stack.data
    if case["kind"] != "build":
        out["image"] = vi.render(vol, tf, stack, state["cam"], case["mode"], case["step"], state["opts"],
                                 state["image"])
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

_VOXEL_BYTES = {"u8": 1, "u16": 2, "f16": 2, "f32": 4}
# operations per composited segment: position, fetch, transfer function,
# opacity and compositing, plus the gather's taps
_SEGMENT_FLOPS = {"none": 83, "shadow": 113, "shell": 245, "cone": 354, "phong": 297}


def _stack_bytes(case):
    return case["slabs"] * case["res"] ** 2 * (4 if case["stack"] == "f32" else 2)


def work(case):
    """Bytes: the volume and the stack once, the outputs once.  Operations: a
    build's slabs inside the cube (a fifth of the light's box) and a frame's
    composited segments (about 16 a pixel on these phantoms: most rays end in
    the shell or miss), each with its arithmetic."""
    if case["kind"] == "serve":
        b = f = 0
        sessions = _sessions(case, 0)
        for vc, _, _ in sessions:
            b += vc["edge"] ** 3 * 2 + _stack_bytes(vc)
        for q in _burst(case, sessions, 0):
            px = q["cam"]["width"] * q["cam"]["height"]
            b += px * 16
            f += px * 16 * _SEGMENT_FLOPS[q["mode"]]
        return {"bytes": b, "flops": f}
    vb = case["edge"] ** 3 * _VOXEL_BYTES[case["voxels"]]
    if case["kind"] == "open":
        cells = math.ceil(case["edge"] / case["cell"]) ** 3
        return {"bytes": vb + vb * (4 if case["layout"] == "quads" else 1) + 8 * cells, "flops": 2 * case["edge"] ** 3}
    b, f = vb, 0
    if case["kind"] != "render":
        b += _stack_bytes(case)
        f += 0.2 * case["slabs"] * case["res"] ** 2 * 60
    elif case["mode"] not in ("none", "phong"):
        b += _stack_bytes(case)
    if case["kind"] != "build":
        px = case["width"] * case["height"]
        b += px * 16
        per = _SEGMENT_FLOPS[case["mode"]]
        if case["grid"]:
            per = 115 + 30 * case["grid"] ** 2
        elif case["shells"] > 1:
            per += 156 * (case["shells"] - 1)
        f += px * 8 * per / case["step"]
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------

_SCALE = {"u8": 1.0 / 255.0, "u16": 1.0 / 4095.0, "f16": 1.0, "f32": 1.0}


def _dot(a, b):
    return sum(x * y for x, y in zip(a, b))


def _cross(a, b):
    return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]


def _unit(a):
    n = math.sqrt(_dot(a, a))
    return [x / n for x in a]


class _Light:
    """The light's frame: axis L, plane basis U, V, depth range, half width R."""

    def __init__(self, light, position, n, res):
        self.P, self.n, self.res = position, n, res
        self.L = L = _unit(light if position is None else [0.5 - a for a in position])
        j = min(range(3), key=lambda a: (abs(L[a]), a))
        self.U = _unit([(1.0 if a == j else 0.0) - L[j] * L[a] for a in range(3)])
        self.V = _cross(L, self.U)
        corners = [[(v >> a) & 1 for a in range(3)] for v in range(8)]
        if position is None:
            d = [_dot(L, c) for c in corners]
            self.R = math.sqrt(3.0) / 2.0
        else:
            rel = [[c[a] - position[a] for a in range(3)] for c in corners]
            d = [_dot(L, c) for c in rel]
            self.R = max(max(abs(_dot(self.U, c)), abs(_dot(self.V, c))) / x for c, x in zip(rel, d))
        self.dmin, self.dmax = min(d), max(d)
        self.ds = (self.dmax - self.dmin) / n

    def grid(self, p):
        """(depth index less one, column, row, ahead of the light) of points p."""
        if self.P is None:
            d, u, v = _dot(self.L, p), _dot(self.U, [a - 0.5 for a in p]), _dot(self.V, [a - 0.5 for a in p])
            ahead = None
        else:
            r = [a - b for a, b in zip(p, self.P)]
            d = _dot(self.L, r)
            ahead = d > 0
            safe = torch.where(ahead, d, torch.ones_like(d))
            u, v = _dot(self.U, r) / safe, _dot(self.V, r) / safe
        k = self.res / (2.0 * self.R)
        return self.n * (d - self.dmin) / (self.dmax - self.dmin) - 1.0, (u + self.R) * k - 0.5, (v + self.R) * k - 0.5, ahead


class _Scene:
    def __init__(self, case, raw, table):
        self.N, self.scale = case["edge"], _SCALE[case["voxels"]]
        self.raw, self.tab = raw.reshape(-1), table.double().to(DEV)

    def value(self, p):
        """Trilinear value at world points p (three tensors), clamped to the edge."""
        N, acc = self.N, 0.0
        ax = []
        for a in p:
            g = a * N - 0.5
            f = g.floor()
            i = f.long()
            ax.append((g - f, i.clamp(0, N - 1), (i + 1).clamp(0, N - 1)))
        for dz in (0, 1):
            for dy in (0, 1):
                for dx in (0, 1):
                    at = (ax[2][1 + dz] * N + ax[1][1 + dy]) * N + ax[0][1 + dx]
                    w = 1.0
                    for (t, _, _), d in zip(ax, (dx, dy, dz)):
                        w = w * (t if d else 1.0 - t)
                    acc = acc + w * (self.raw[at].double() * self.scale).clamp(0.0, 1.0)
        return acc

    def colour(self, v, channels):
        K = self.tab.shape[0]
        x = v * (K - 1)
        i = x.floor().long().clamp(0, K - 2)
        w = x - i
        return [(1.0 - w) * self.tab[i, c] + w * self.tab[i + 1, c] for c in channels]


def _exact_stack(case, scene, lt):
    """n x res x res transmittance, or optical depth in base 2 where the stack
    holds it (each slab adds at most 64 / ln 2, as the library documents)."""
    n, res, N = lt.n, lt.res, scene.N
    t = -lt.R + (torch.arange(res, device=DEV, dtype=torch.float64) + 0.5) * (2.0 * lt.R / res)
    u, v = t[None, :].expand(res, res), t[:, None].expand(res, res)
    D = [lt.L[a] + u * lt.U[a] + v * lt.V[a] for a in range(3)]
    seg = lt.ds if lt.P is None else lt.ds * torch.sqrt(D[0] ** 2 + D[1] ** 2 + D[2] ** 2)
    out = torch.empty(n, res, res, device=DEV, dtype=torch.float64)
    T, tau = torch.ones(res, res, device=DEV, dtype=torch.float64), 0.0
    Lc = _dot(lt.L, [0.5] * 3)
    for k in range(n):
        d = lt.dmin + (k + 0.5) * lt.ds
        if lt.P is None:
            p = [0.5 + u * lt.U[a] + v * lt.V[a] + (d - Lc) * lt.L[a] for a in range(3)]
        else:
            p = [lt.P[a] + d * D[a] for a in range(3)]
        inside = torch.ones(res, res, device=DEV, dtype=torch.bool)
        for a in range(3):
            inside &= (p[a] >= 0.0) & (p[a] <= 1.0)
        a = scene.colour(scene.value(p), (3,))[0]
        f = torch.pow(1.0 - a, seg * N)
        if case["darken"]:
            f = (f * torch.pow(2.0 - f, case["darken"])).clamp(max=1.0)
        T = torch.where(inside, T * f, T)
        if case["stack"] == "bf16":
            tau = tau + torch.where(inside, -torch.log2(f), torch.zeros_like(f)).clamp(0.0, 64.0 / math.log(2.0))
        out[k] = tau if case["stack"] == "bf16" else T
    return out


def _lookup(stack, lt, p):
    z, x, y, ahead = lt.grid(p)
    n, res = lt.n, lt.res
    z = z.clamp(-1.0, n - 1.0)
    zf, xf, yf = z.floor(), x.floor(), y.floor()
    wz, wx, wy = z - zf, x - xf, y - yf
    k0, i0, j0 = zf.long(), xf.clamp(-2, res).long(), yf.clamp(-2, res).long()
    flat, acc = stack.reshape(-1), 0.0
    for dk in (0, 1):
        k = (k0 + dk).clamp(max=n - 1)
        for dj in (0, 1):
            for di in (0, 1):
                i, j = i0 + di, j0 + dj
                ok = (k >= 0) & (i >= 0) & (j >= 0) & (i < res) & (j < res)
                at = (k.clamp(min=0) * res + j.clamp(0, res - 1)) * res + i.clamp(0, res - 1)
                w = (wz if dk else 1 - wz) * (wy if dj else 1 - wy) * (wx if di else 1 - wx)
                acc = acc + w * torch.where(ok, flat[at], 1.0)
    return acc if ahead is None else torch.where(ahead, acc, torch.ones_like(acc))


def _coefficient(case, scene, stack, lt, p, d):
    mode = case["mode"]
    if mode == "shadow":
        return _lookup(stack, lt, p)
    if mode == "shell":
        num = tot = 0.0
        for r, w in zip(range(1, case["shells"] + 1), (1.0, 0.5)):
            for a in range(3):
                for s in (-1, 1):
                    num = num + w / 6.0 * _lookup(stack, lt, [q + (s * r / scene.N if b == a else 0.0)
                                                              for b, q in enumerate(p)])
            tot += w
        return num / tot
    one = torch.ones_like(p[0])
    if lt.P is None:
        Ls, step = [one * a for a in lt.L], lt.ds
    else:
        r = [a - b for a, b in zip(p, lt.P)]
        nr = torch.sqrt(_dot(r, r))
        Ls = [a / nr for a in r]
        step = lt.ds / _dot(lt.L, Ls)
    wl = -_dot(d, Ls)
    B = [-a - wl * l for a, l in zip(d, Ls)]
    nb = torch.sqrt(_dot(B, B))
    B = [a / nb for a in B]
    X = _cross(Ls, B)
    acc, taps = 0.0, 0
    if case["grid"]:
        G = case["grid"]
        for ia in range(G):
            for ib in range(G):
                a, b = (ia - (G - 1) / 2.0) * step / 2.0, (ib - (G - 1) / 2.0) * step / 2.0
                acc = acc + _lookup(stack, lt, [q - step * l + a * e + b * x for q, l, e, x in zip(p, Ls, B, X)])
                taps += 1
    else:
        for m in (1, 2):
            for q4 in range(4):
                c, s = math.cos(math.pi * q4 / 2.0), math.sin(math.pi * q4 / 2.0)
                acc = acc + _lookup(stack, lt, [q - m * step * l + m * step * (c * e + s * x)
                                                for q, l, e, x in zip(p, Ls, B, X)])
                taps += 1
    return acc / taps


def _exact_image(case, scene, stack, lt, cam):
    N, W, H, dt = scene.N, cam["width"], cam["height"], case["step"] / case["edge"]
    fwd = _unit([t - e for t, e in zip(cam["target"], cam["eye"])])
    right = _unit(_cross(fwd, cam["up"]))
    up = _cross(right, fwd)
    xn = (2.0 * (torch.arange(W, device=DEV, dtype=torch.float64) + 0.5) / W - 1.0)[None, :].expand(H, W).reshape(-1)
    yn = (1.0 - 2.0 * (torch.arange(H, device=DEV, dtype=torch.float64) + 0.5) / H)[:, None].expand(H, W).reshape(-1)
    one = torch.ones_like(xn)
    if cam["kind"] == "persp":
        th = math.tan(0.5 * math.radians(cam["fovy_deg"]))
        o = [one * e for e in cam["eye"]]
        d = [fwd[a] + xn * (th * W / H) * right[a] + yn * th * up[a] for a in range(3)]
        nd = torch.sqrt(_dot(d, d))
        d = [a / nd for a in d]
    else:
        h = cam["ortho_half_h"]
        o = [cam["eye"][a] + xn * (h * W / H) * right[a] + yn * h * up[a] for a in range(3)]
        d = [one * a for a in fwd]
    tn, tf, hit = torch.zeros_like(xn), torch.full_like(xn, 1e300), torch.ones_like(xn, dtype=torch.bool)
    for a in range(3):
        flat = d[a] == 0
        hit &= ~(flat & ((o[a] < 0) | (o[a] > 1)))
        q = torch.where(flat, one, d[a])
        t1, t2 = -o[a] / q, (1.0 - o[a]) / q
        tn = torch.where(flat, tn, torch.maximum(tn, torch.minimum(t1, t2)))
        tf = torch.where(flat, tf, torch.minimum(tf, torch.maximum(t1, t2)))
    ids = torch.nonzero(hit & (tf > tn))[:, 0]
    image = torch.zeros(H * W, 4, device=DEV, dtype=torch.float64)
    S = 8
    for part in ids.split(1 << 19):
        po, pd = [a[part][:, None] for a in o], [a[part][:, None] for a in d]
        ti, te = tn[part][:, None], tf[part][:, None]
        K = torch.ceil((te - ti) / dt)
        rgb = torch.zeros(len(part), 3, device=DEV, dtype=torch.float64)
        T = torch.ones(len(part), 1, device=DEV, dtype=torch.float64)
        live = torch.ones(len(part), 1, device=DEV, dtype=torch.bool)
        for k0 in range(0, int(K.max()), S):
            if k0 % 64 == 0 and not bool(live.any()):
                break
            k = k0 + torch.arange(S, device=DEV, dtype=torch.float64)[None, :]
            t0, t1 = ti + k * dt, torch.minimum(ti + (k + 1) * dt, te)
            ln, tm = (t1 - t0).clamp(min=0.0), 0.5 * (t0 + t1)
            p = [a + tm * b for a, b in zip(po, pd)]
            val = scene.value(p)
            om = torch.pow(1.0 - scene.colour(val, (3,))[0], ln * N)
            om = torch.where((k < K) & live, om, torch.ones_like(om))
            incl = T * torch.cumprod(om, 1)
            excl = torch.cat([T, incl[:, :-1]], 1)
            done = incl <= 2.0 ** -15
            before = torch.cat([torch.zeros_like(done[:, :1]), torch.cummax(done.long(), 1)[0][:, :-1] > 0], 1)
            w = torch.where(before, torch.zeros_like(excl), excl) * (1.0 - om)
            at = torch.nonzero(w > 0)
            if len(at):
                sel = (at[:, 0], at[:, 1])
                ps, ds = [a[sel] for a in p], [a.expand(-1, S)[sel] for a in pd]
                c = torch.stack(scene.colour(val[sel], (0, 1, 2)), 1)
                spec = 0.0
                if case["mode"] == "phong":
                    g = []
                    for a in range(3):
                        hi, lo = ([q + (s / N if b == a else 0.0) for b, q in enumerate(ps)] for s in (1, -1))
                        g.append(0.5 * (scene.value(hi) - scene.value(lo)))
                    den = torch.sqrt(_dot(g, g)).clamp(min=0.02)
                    nrm = [-a / den for a in g]
                    if lt.P is None:
                        l = [-a for a in lt.L]
                    else:
                        l = [b - a for a, b in zip(ps, lt.P)]
                        nl = torch.sqrt(_dot(l, l))
                        l = [a / nl for a in l]
                    nl, nn = _dot(nrm, l), _dot(nrm, nrm)
                    rv = -_dot([2.0 * nl * a - nn * b for a, b in zip(nrm, l)], ds)
                    A = 0.1 + 0.9 * nl.clamp(min=0.0)
                    spec = (0.4 * rv.clamp(min=0.0) ** 20)[:, None]
                elif case["mode"] == "none":
                    A = torch.ones_like(ps[0])
                else:
                    A = _coefficient(case, scene, stack, lt, ps, ds)
                rgb.index_add_(0, at[:, 0], w[sel][:, None] * (A[:, None] * c + spec))
            # past the terminating segment the ray's transmittance stays
            T = torch.where(before, torch.full_like(incl, 2.0), incl).amin(1, keepdim=True)
            live = live & ~(T <= 2.0 ** -15)
        image[part, :3], image[part, 3:] = rgb, 1.0 - T
    return image.reshape(H, W, 4)


def _exact_scene(case, seed):
    return _Scene(case, _voxels(case, seed), _tf_table(case))


def exact(case, seed):
    if case["kind"] == "serve":
        sessions, out, scenes, stacks = _sessions(case, seed), [], {}, {}
        for q in _burst(case, sessions, 0):
            s = q["session"]
            vc = {**sessions[s][0], "mode": q["mode"]}
            lt = _Light(q["light"], None, vc["slabs"], vc["res"])
            if s not in scenes:
                scenes[s] = _exact_scene(vc, seed * 16 + s)
                stacks[s] = _exact_stack(vc, scenes[s], lt)
            out.append(_exact_image(vc, scenes[s], stacks[s], lt, q["cam"]))
        return out
    scene = _exact_scene(case, seed)
    if case["kind"] == "open":
        N, B = case["edge"], case["cell"]
        v = (scene.raw.reshape(1, 1, N, N, N).float() if case["voxels"] != "f32" else
             scene.raw.reshape(1, 1, N, N, N))
        ends = []
        for s in (1.0, -1.0):
            # a cell's voxels and the next one along each axis (the pooling
            # takes exact values; the normalisation follows it in 64 bits)
            pad = F.pad(s * v, (0, -N % B + 1) * 3, value=-math.inf)
            ends.append(s * F.max_pool3d(pad, B + 1, B)[0, 0].double())
        mm = torch.stack([ends[1], ends[0]], -1) * scene.scale
        return {"voxels": None, "map": mm.clamp(0.0, 1.0).reshape(-1), "bits": None}
    light, position, cam = _inputs(case, seed)
    lt = _Light(light, position, case["slabs"], case["res"])
    reads = case["kind"] != "render" or case["mode"] not in ("none", "phong")
    stack, out = (_exact_stack(case, scene, lt) if reads else None), {}
    if case["kind"] != "build":
        T = torch.exp2(-stack) if reads and case["stack"] == "bf16" else stack
        out["image"] = _exact_image(case, scene, T, lt, cam)
    if case["kind"] != "render":
        T = stack
        if not case["rows"]:
            n, res, r8, r4 = lt.n, lt.res, -lt.res % 8, -lt.res % 4
            T = F.pad(T, (0, r8, 0, r4))
            T = T.reshape(n, (res + r4) // 4, 4, (res + r8) // 8, 8).permute(0, 1, 3, 2, 4)
        out["stack"] = T
    return out
