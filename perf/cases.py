"""Workloads of the ray tracer, called through its public entry points.

``listed()`` names them, ``draw(rng)`` gives more of the same ranges,
``prepare(case, seed)`` makes what a user's program holds before the call (on
the GPU), ``run(state)`` is one pass, ``work(case)`` the bytes and operations a
pass cannot do without, and ``exact(case, seed)`` the outputs in 64 bits where
plain numpy or torch can give them in seconds.

Kinds of case:

* ``trace``  trace a problem and take its channel: read back whole
  (``configs`` 0: E_env and H on the host) or summed for ``configs`` RIS
  configurations into the field and power maps E and P; ``rebuild`` also
  builds the scene (BVH and tables) from the device-resident mesh first.
* ``sum``    the coherent sum of a channel that is already there over
  ``configs`` configurations (a served query, or a codebook search).
* ``cir``    the delay-binned impulse response of a traced channel.
"""
import math

import numpy as np
import torch

from paper_2402_13034_amd import risrt, synth

ETA0 = 120.0 * math.pi
PRECISIONS = ("valu", "bf16x2", "bf16x3", "f16x2")   # risrt.PREC_* in order

_ctx = None


def context():
    """The program's one library context."""
    global _ctx
    if _ctx is None:
        _ctx = risrt.Context(0)
    return _ctx


def _trace(name, scene, order, n_rays, nx, ny, ris, **kw):
    c = dict(name=name, kind="trace", scene=scene, tris=0, order=order, n_rays=n_rays, nx=nx, ny=ny, ris=ris,
             fresnel=0, incoming=False, rebuild=False, configs=1, real=False, precision="valu")
    c.update(kw)
    return c


def _sum(name, rx, elems, configs, precision, real, want_E, want_P):
    return dict(name=name, kind="sum", rx=rx, elems=elems, configs=configs, precision=precision, real=real,
                want_E=want_E, want_P=want_P)


def listed():
    return [
        # the smallest trace: a box, a 7 x 7 RIS, receivers on a line, order 1; the channel read back whole
        _trace("trace_tiny_box", "box", 1, 10_000, 64, 1, "sq7", configs=0),
        # the paper's reflective scenario: the 1 cm power map of one configuration (metal walls, TE Fresnel
        # coefficients, monopole receivers, order 2)
        _trace("map_paper_1cm", "paper", 2, 100_000, 61, 91, "hex6", fresnel=1),
        # the benchmark's step: a changed lab room is rebuilt, traced at order 3 and summed for one configuration
        _trace("step_lab_room", "lab", 3, 1_000_000, 64, 64, "hex6", tris=3, rebuild=True),
        # an ordinary trace with every reflection modelled (incoming ones too, TM Fresnel), odd sizes; the channel
        # read back whole
        _trace("trace_lab_incoming_tm", "lab", 2, 200_000, 37, 53, "hex5", tris=5, fresnel=2, incoming=True,
               configs=0),
        # a serving miss: a furnished room is traced, then the query's 24 configurations are summed
        _trace("serve_miss_50k", "room", 2, 100_000, 64, 64, "hex10", tris=50_000, configs=24, precision="bf16x2"),
        # a changed room of 200 000 triangles rebuilt for a small query (the BVH build dominates)
        _trace("rebuild_200k", "room", 1, 10_000, 16, 16, "hex3", tris=200_000, rebuild=True, configs=1),
        # the large configuration: the office floor (1.08 million triangles, order 5, 64 x 64 RIS, 256 x 256
        # receivers), summed for 16 on/off-type configurations
        _trace("office_floor", "office", 5, 10_000_000, 256, 256, "sq64", configs=16, real=True,
               precision="bf16x2"),
        # the smallest sum: one configuration at a few receivers (a controller probing a setting)
        _sum("sum_one_config", 256, 37, 1, "valu", False, True, True),
        # a served query on a cached channel: some tens of 2-bit configurations, power only
        _sum("sum_query_c37", 4096, 127, 37, "bf16x2", False, False, True),
        # a codebook of odd sizes at fp16-split accuracy, field and power
        _sum("sum_codebook_f16", 3000, 331, 333, "f16x2", False, True, True),
        # the many-configuration search: 4096 +-1 configurations of a 32 x 32 RIS over a 128 x 128 map
        _sum("sum_many_configs", 16384, 1024, 4096, "bf16x2", True, False, True),
        # the impulse response of the lab room's traced channel, 0.25 ns x 400 bins
        dict(name="cir_lab_room", kind="cir", scene="lab", tris=3, order=3, n_rays=200_000, nx=64, ny=64, ris="hex6",
             fresnel=0, incoming=False, bin_ns=0.25, bins=400),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("trace", "trace", "trace", "trace", "sum", "sum", "sum", "cir"))
    if kind == "sum":
        while True:
            R, M, C = _log_int(rng, 64, 20_000), _log_int(rng, 37, 2_000), _log_int(rng, 1, 4_096)
            if R * M * C <= 16384 * 1024 * 4096 and R * M <= 1 << 25 and R * C <= 1 << 26:
                break
        what = rng.choice((1, 2, 3))
        return dict(kind="sum", rx=R, elems=M, configs=C, precision=rng.choice(PRECISIONS),
                    real=rng.random() < 0.4, want_E=bool(what & 1), want_P=bool(what & 2))
    ris = rng.choice(("hex%d" % rng.randint(3, 18), "sq%d" % rng.randint(5, 40)))
    if kind == "cir":
        n = _log_int(rng, 16, 72)
        return dict(kind="cir", scene="lab", tris=rng.randint(2, 6), order=rng.randint(1, 3),
                    n_rays=_log_int(rng, 20_000, 400_000), nx=n, ny=rng.randint(max(1, n // 2), n),
                    ris="hex%d" % rng.randint(3, 9), fresnel=rng.randint(0, 2), incoming=False,
                    bin_ns=rng.choice((0.1, 0.25, 0.5, 1.0)), bins=_log_int(rng, 50, 3_000))
    scene = rng.choice(("box", "paper", "lab", "lab", "room", "room", "office"))
    n = _log_int(rng, 8, 128)
    c = dict(kind="trace", scene=scene, tris=0, order=rng.randint(1, 3), n_rays=_log_int(rng, 5_000, 1_000_000),
             nx=n, ny=rng.randint(max(1, n // 2), n), ris=ris, fresnel=0, incoming=rng.random() < 0.25,
             rebuild=rng.random() < 0.4, configs=rng.choice((0, 1, _log_int(rng, 2, 256))), real=rng.random() < 0.4)
    c["precision"] = "valu" if c["configs"] < 2 else rng.choice(PRECISIONS)
    if scene == "lab":
        c["tris"] = rng.randint(1, 9)            # face subdivision: 212 to 17 000 triangles
        c["fresnel"] = rng.randint(0, 2)
    elif scene == "room":
        c["tris"] = _log_int(rng, 1_000, 100_000)
    elif scene == "paper":
        c.update(ris="hex6", order=2, fresnel=1)
    elif scene == "office":
        c["tris"] = rng.randint(2, 8)            # rooms along x (half as many along y)
        c["order"] = rng.randint(2, 5)
    # a channel of at most 64 MB, or 16 MB where it is read back whole
    while _elements(c["ris"]) * c["nx"] * c["ny"] > (1 << 23 if c["configs"] else 1 << 21):
        c["nx"], c["ny"] = max(1, c["nx"] // 2), max(1, c["ny"] // 2)
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _elements(ris):
    return synth.hex_count(int(ris[3:])) if ris.startswith("hex") else int(ris[2:]) ** 2


def _ris(ris, lam, centre, normal):
    n = int(ris[3:]) if ris.startswith("hex") else int(ris[2:])
    e = synth.hex_ris(n, lam / 2, centre, normal) if ris.startswith("hex") else \
        synth.square_ris(n, n, lam / 2, centre, normal)
    return synth.Ris(e, normal, centre, lam / 2, lam / 2, math.pi, 3.0)


def _problem(case, seed):
    """The synthetic problem of a traced case: geometry, antennas, RIS, receivers."""
    rng = np.random.default_rng(7919 * (seed + 1))
    lam = synth.C0 / 28e9
    nx, ny, normal = case["nx"], case["ny"], np.array([-1.0, 0.0, 0.0])
    iso = synth.Antenna(np.array([0.0, 0.0, 1.0]), 1.0, synth.PAT_ISO, 0.0)
    name = case["scene"]
    if name == "paper":
        p = synth.paper_room(True, "target", n_rays=case["n_rays"])
        p.rx_pos = synth.rx_grid(0.92, 1.52, nx, 0.02, 0.92, ny, 0.114, 1e-4, rng)
        return p
    if name == "office":
        if case["tris"]:
            rooms = case["tris"]
            p = synth.office_floor(seed=synth.BASE_SEED + seed, n_rays=case["n_rays"], order=case["order"], n_rx=1,
                                   n_side=2, nx=rooms, ny=max(1, rooms // 2))
            room = (rooms // 2, rooms // 4)       # the RIS on the far wall of a middle room
            centre = np.array([2.0 * room[0] + 1.949, 2.0 * room[1] + 1.0, 1.5])
            tx = np.array([2.0 * room[0] + 0.35, 2.0 * room[1] + 0.35, 2.5])
            p.rx_pos = synth.rx_grid(0.15, 2.0 * rooms - 0.15, nx, 0.15, 2.0 * max(1, rooms // 2) - 0.15, ny, 1.2,
                                     3e-4, rng)
            p.ris, p.tx_pos = _ris(case["ris"], lam, centre, normal), tx
            p.tx_ant = synth.Antenna(synth.unit(centre - tx), 18.0, synth.PAT_COSPOW, 8.0)
            return p
        return synth.office_floor(seed=synth.BASE_SEED + seed, n_rays=case["n_rays"], order=case["order"], n_rx=nx,
                                  n_side=int(case["ris"][2:]))
    if name == "box":
        size = (5.0, 4.0, 3.0)
        scene = synth.box_room(size, 0.5 + 0j)
        tx = np.array([1.0, 1.0, 1.5]) + rng.uniform(-0.2, 0.2, 3)
        rx = synth.rx_line((0.5, 3.3, 1.5), (4.5, 2.7, 1.5), nx, 1e-3, rng) if ny == 1 else \
            synth.rx_grid(0.25, 4.75, nx, 0.25, 3.75, ny, 1.5, 3e-4, rng)
        ant = (1.0, synth.PAT_ISO, 0.0)
    elif name == "lab":
        size = (6.0, 5.0, 3.0)
        scene = synth.lab_room_scene(rng, sub=case["tris"])
        tx = np.array([0.5, 0.5, 2.5])
        rx = synth.rx_grid(0.3, 5.7, nx, 0.3, 4.7, ny, 1.2, 5e-4, rng)
        ant = (18.0, synth.PAT_COSPOW, 8.0)
    else:
        scene, size = synth.random_box_room(rng, case["tris"])
        tx = np.array([0.3, 0.3, 2.5])
        rx = synth.rx_grid(0.4, size[0] - 0.4, nx, 0.4, size[1] - 0.4, ny, 1.2, 3e-4, rng)
        ant = (18.0, synth.PAT_COSPOW, 8.0)
    centre = np.array([size[0] - 0.001, size[1] / 2, 1.5])
    p = synth.Problem(name, scene, 28e9, tx, 0.01, synth.Antenna(synth.unit(centre - tx), *ant),
                      _ris(case["ris"], lam, centre, normal), rx, iso, case["order"], case["n_rays"], seed)
    return synth.with_materials(p, case["fresnel"], seed=seed) if case["fresnel"] else p


def _gamma(M, C, real, seed):
    """Random RIS configurations: 0.9 (+-1) or the 2-bit phases 0.9 j^b."""
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    if real:
        return torch.complex(torch.randint(0, 2, (M, C), generator=g, device="cuda").float() * 1.8 - 0.9,
                             torch.zeros(M, C, device="cuda"))
    b = torch.randint(0, 4, (M, C), generator=g, device="cuda")
    table = torch.tensor([0.9, 0.9j, -0.9, -0.9j], dtype=torch.complex64, device="cuda")
    return table[b]


def _fields(case, seed):
    """E_env and H of a channel made elsewhere: phases uniform, magnitudes
    spread over receivers by some 20 dB and, within a receiver, by fading."""
    g = torch.Generator(device="cuda").manual_seed(1000 + seed)
    R, M = case["rx"], case["elems"]

    def cn(*shape):
        return torch.complex(torch.randn(*shape, generator=g, device="cuda"),
                             torch.randn(*shape, generator=g, device="cuda"))
    level = 1e-5 * torch.exp(torch.randn(R, 1, generator=g, device="cuda"))
    H = cn(R, M) * level
    E = cn(R) * (3.0 * math.sqrt(M) * level[:, 0])
    return E, H


class State:
    """What the program holds between calls; its handles go with it."""

    def __init__(self, case):
        self.case, self.handles = case, []

    def __del__(self):
        try:
            for h in reversed(self.handles):
                context().destroy(h)
        except Exception:
            pass


def _up(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a, dtype)).cuda()


def prepare(case, seed):
    ctx, s = context(), State(case)
    if case["kind"] == "sum":
        E, H = _fields(case, seed)
        s.channel = ctx.channel_create(E.cpu().numpy(), H.cpu().numpy())
        s.handles.append(s.channel)
        s.gamma = _gamma(case["elems"], case["configs"], case["real"], seed)
        return s
    p = s.prob = _problem(case, seed)
    s.rx = _up(p.rx_pos, np.float64)
    sc = p.scene
    s.mesh = (_up(sc.V, np.float32), _up(sc.T, np.int32), _up(sc.surf, np.int32), _up(sc.refl_re, np.float32),
              _up(sc.refl_im, np.float32))
    s.mat = (_up(p.mat_eps_r, np.float32), _up(p.mat_sigma, np.float32)) if p.mat_eps_r is not None else None
    r = p.ris
    s.ris = ctx.ris_create(r.elems, r.centre, r.normal, r.dy, r.dz, r.gain, r.q)
    s.handles.append(s.ris)
    if case.get("rebuild"):
        s.scene = 0
    else:
        s.scene = _scene(s)
        s.handles.append(s.scene)
    s.flags = risrt.FLAG_RIS_INCOMING if case["incoming"] else 0
    if case["kind"] == "cir":
        s.channel, _ = risrt.trace_problem(ctx, p, s.scene, s.ris, flags=risrt.FLAG_KEEP_CIR, rx=s.rx)
        s.handles.append(s.channel)
        s.gamma = _gamma(r.elems.shape[0], 1, False, seed)[:, 0].contiguous()
    elif case["configs"]:
        s.gamma = _gamma(r.elems.shape[0], case["configs"], case["real"], seed)
    return s


def _scene(s):
    scene = context().scene_create(*s.mesh)
    if s.mat is not None:
        context().scene_set_materials(scene, *s.mat)
    return scene


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(state):
    s, case, ctx = state, state.case, context()
    if case["kind"] == "sum":
        E, P = ctx.ris_sum(s.channel, s.gamma, gamma_is_real=case["real"],
                           precision=PRECISIONS.index(case["precision"]), want_E=case["want_E"],
                           want_P=case["want_P"])
        return {"E": E, "P": P}
    if case["kind"] == "cir":
        return {"cir": ctx.cir(s.channel, s.gamma, case["bin_ns"] * 1e-9, case["bins"])}
    scene = _scene(s) if case["rebuild"] else s.scene
    ch, st = risrt.trace_problem(ctx, s.prob, scene, s.ris, flags=s.flags, rx=s.rx)
    out = {k: st[k] for k in ("n_cand_tx", "n_cand_u", "n_env_paths", "n_u_paths", "n_ris_slots", "n_in_seq",
                              "n_in_paths", "discovery_segments", "leg_segments")}
    if case["configs"]:
        out["E"], out["P"] = ctx.ris_sum(ch, s.gamma, gamma_is_real=case["real"],
                                         precision=PRECISIONS.index(case["precision"]), want_E=True)
    else:
        out["E_env"], out["H"] = ctx.channel_read(ch)
    ctx.destroy(ch)
    if case["rebuild"]:
        ctx.destroy(scene)
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    if case["kind"] == "sum":
        R, M, C = case["rx"], case["elems"], case["configs"]
        out = R * C * (8 * case["want_E"] + 4 * case["want_P"])
        return {"bytes": 8 * R * M + 8 * M * C + 8 * R + out, "flops": (4 if case["real"] else 8) * R * M * C}
    M, R = _elements(case["ris"]), case["nx"] * case["ny"]
    if case["kind"] == "cir":   # the kept direct element paths (16 B each), the bins out
        return {"bytes": 16 * R * M + 8 * M + 8 * R * case["bins"], "flops": 10 * R * M}
    n_tri = {"box": 12, "paper": 18, "lab": 212 * case["tris"] ** 2, "room": case["tris"],
             "office": 5400 * (case["tris"] * max(1, case["tris"] // 2) if case["tris"] else 200)}[case["scene"]]
    # mesh and receivers in; E_env and H out, or the maps
    C = case["configs"]
    b = n_tri * 72 + 24 * R + (12 * R * C + 8 * M * C if C else 8 * R * (M + 1))
    # every discovery segment descends the tree once (two 40-flop node tests a level of a binary tree, one
    # triangle); every (receiver, element) direct path costs at least the 150 flops of its geometry and field
    # and one descent for its leg
    walk = 40.0 * max(1.0, math.log2(n_tri)) + 40.0
    f = 2.0 * case["n_rays"] * case["order"] * walk + R * M * (150.0 + walk) + 8.0 * R * M * C
    return {"bytes": float(b), "flops": f}


# --------------------------------------------------------------------------
# the outputs in 64 bits
# --------------------------------------------------------------------------
def exact(case, seed):
    if case["kind"] == "sum":
        R, M, C = case["rx"], case["elems"], case["configs"]
        E0, H = _fields(case, seed)
        G = _gamma(M, C, case["real"], seed)
        E = torch.empty(R, C, dtype=torch.complex128, device="cuda")
        step = max(1, (1 << 24) // max(M, C))
        Gr, Gi = G.real.double().contiguous(), G.imag.double().contiguous()
        for a in range(0, R, step):
            hr, hi = H[a:a + step].real.double().contiguous(), H[a:a + step].imag.double().contiguous()
            E[a:a + step] = torch.complex(hr @ Gr - hi @ Gi, hr @ Gi + hi @ Gr) + E0[a:a + step, None].to(E.dtype)
        P = (E.real ** 2 + E.imag ** 2) / (2.0 * ETA0)
        return {"E": E if case["want_E"] else None, "P": P if case["want_P"] else None}
    if case["kind"] == "trace" and case["scene"] == "box" and case["order"] == 1 and not case["incoming"]:
        E0, H = _box_channel(_problem(case, seed))
        out = {k: None for k in ("n_cand_tx", "n_cand_u", "n_env_paths", "n_u_paths", "n_ris_slots", "n_in_seq",
                                 "n_in_paths", "discovery_segments", "leg_segments")}
        if not case["configs"]:
            return dict(out, E_env=E0, H=H)
        G = _gamma(H.shape[1], case["configs"], case["real"], seed).cpu().numpy().astype(np.complex128)
        E = E0[:, None] + H @ G
        return dict(out, E=E, P=np.abs(E) ** 2 / (2.0 * ETA0))
    return None


def _box_channel(p):
    """E_env and H of an empty box at order 1 from its image sources: the
    direct path and one mirror path per wall (for the RIS, the walls in front
    of its plane), 1 / length spreading, coefficient 0.5 per bounce."""
    lam, lo, hi = p.wavelength, p.scene.V.min(0).astype(np.float64), p.scene.V.max(0).astype(np.float64)
    a0 = math.sqrt(2.0 * ETA0 * p.tx_power_w * p.tx_ant.gain)
    coef = complex(p.scene.refl_re[0], p.scene.refl_im[0])

    def images(src):
        yield src, 1.0
        for k in range(3):
            for w in (lo[k], hi[k]):
                m = src.copy()
                m[..., k] = 2.0 * w - m[..., k]
                yield m, coef

    def wave(d):
        return np.exp(-2j * np.pi * ((d / lam) % 1.0))

    E = np.zeros(p.rx_pos.shape[0], np.complex128)
    for im, c in images(p.tx_pos):
        d = np.linalg.norm(p.rx_pos - im, axis=1)
        E += c * a0 * lam / (4.0 * np.pi * d) * wave(d)
    r = p.ris
    back = p.tx_pos - r.elems
    dt = np.linalg.norm(back, axis=1)
    f_in = np.maximum(back @ r.normal / dt, 0.0) ** r.q
    T = a0 * np.sqrt(r.gain * f_in * r.dy * r.dz / (4.0 * np.pi)) / dt * wave(dt)
    H = np.zeros((p.rx_pos.shape[0], r.elems.shape[0]), np.complex128)
    for im, c in images(r.elems):
        v = p.rx_pos[:, None, :] - im[None]
        d = np.linalg.norm(v, axis=2)
        # the leaving direction is the arriving one mirrored back: its component along the RIS normal keeps
        # its value unless the mirror wall is parallel to the RIS
        flip = -1.0 if abs(im[0, 0] - r.elems[0, 0]) > 1e-9 else 1.0
        cos = flip * (v @ r.normal) / d
        H += np.where(cos > 0, c * lam / (4.0 * np.pi * d) * np.maximum(cos, 0.0) ** (r.q / 2) * wave(d), 0.0)
    return E, H * T[None, :]
