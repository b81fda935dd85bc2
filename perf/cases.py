"""The work that users of the library have it do, as measurable cases.

Each case is one call sequence through the public entry points: tracing a
scene, summing a path list into an FMCW or stepped-frequency cube, imaging,
the learned proposal's network, a batched launch, a frame of a moving hand,
and the smallest whole call, where latency counts.  Sizes are those of the
repository's own workloads (`scenegen`) and bench legs, or of the ranges that
`scenegen.workload_batch` spans.

The path lists of the synthesis cases are drawn here from a seed with the
distribution that traces of the street and the hand have: of the street's
paths 96 to 99.9 % are single bounces off the static ground within a metre or
two of the array, the rest come from poles and moving cars up to 60 m away;
the hand's all lie on its surface.  So their cubes can be checked against a
plain FP64 sum.
"""
import math

import numpy as np
import torch

import scenegen as sg
import paper_2307_15412_amd as rr

DEV = "cuda:0"
C0 = 299792458.0
DEG = math.pi / 180.0


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest whole call: one frame of the tiny scene (1 x 4 array,
        # 64 samples x 16 chirps), traced and summed, as a real-time loop does
        dict(name="frame_tiny", kind="frame", scene="tiny", rays=100_000, T=1, R=4, M=16, K=64),
        # a small trace by a caller that wants the path list itself (`keep`: at
        # most this many paths, as the large-MIMO workload caps its list)
        dict(name="trace_tiny", kind="trace", scene="tiny", rays=100_000, T=1, R=4, sampler="uniform", keep=2_000),
        # the street configuration's launch: 5.1e5 triangles, 12 x 16 elements
        dict(name="trace_street", kind="trace", scene="street", scale=1.0, rays=10_000_000, T=12, R=16,
             sampler="uniform", keep=100_000),
        # the street configuration's cube: per-element launch, exact model
        dict(name="synth_street", kind="synth", model="exact", geom="street", mode="per_tx", T=12, R=16,
             M=128, K=256, P=263_000, moving=0.002),
        # the paper's stepped-frequency cube of a hand: 94 x 94 channels
        dict(name="synth_hand", kind="synth", model="exact", geom="hand", mode="shared", T=94, R=94,
             M=1, K=128, P=496_000, moving=0.0),
        # the large-MIMO cube: 3 072 channels, separable model (the bench's step)
        dict(name="synth_mimo", kind="synth", model="separable", geom="street", mode="shared", T=48, R=64,
             M=256, K=512, P=100_000, moving=0.0016),
        # the paper's image: 3.3e6 voxels of 1 mm and its projection
        dict(name="image_hand", kind="image", T=94, R=94, K=128, nx=81, ny=201, nz=201, step=1e-3),
        # a quick look with a thinned array and a coarse, ragged grid
        dict(name="image_preview", kind="image", T=30, R=37, K=33, nx=17, ny=41, nz=39, step=5e-3),
        # one step of the proposal network's training batch
        dict(name="proposal_step", kind="mlp_step", scenes=16),
        # logits of every direction bin for a large set of scenes
        dict(name="proposal_eval", kind="mlp_eval", scenes=128),
        # a batched launch of uneven streets, exact model
        dict(name="batch_8", kind="batch", scenes=8, seed0=2000, rays=300_000, tri_hi=100_000, ch_hi=1024),
        # one frame of a moving hand: refit, trace, cube
        dict(name="motion_frame", kind="motion", rays=1_000_000, T=94, R=94, K=128),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["frame", "trace", "synth", "synth", "synth", "image", "image", "mlp_step",
                       "mlp_eval", "batch", "motion"])
    if kind == "frame":
        return dict(kind="frame", scene=rng.choice(["tiny", "box"]), rays=int(_log(rng, 2e4, 2e6)),
                    T=rng.randint(1, 4), R=rng.randint(2, 9), M=rng.randint(1, 48), K=rng.randint(16, 300))
    if kind == "trace":
        scene = rng.choice(["tiny", "street", "hand"])
        if scene == "hand":
            g = rng.randint(1, 9)
            return dict(kind="trace", scene="hand", rays=g * g, T=24, R=31, sampler="per_triangle",
                        keep=1_000 * g * g)
        rays = int(_log(rng, 1e4, 5e6))
        return dict(kind="trace", scene=scene, scale=round(_log(rng, 0.02, 0.4), 3), rays=rays,
                    T=rng.randint(1, 13), R=rng.randint(1, 16), sampler="uniform", keep=rays // 200)
    if kind == "synth":
        model = rng.choice(["exact", "exact", "separable"])
        geom = rng.choice(["street", "street", "hand"])
        mode = "shared" if geom == "hand" else rng.choice(["shared", "per_tx"])
        while True:
            ch = _log(rng, 4, 3072 if mode == "shared" else 400)
            R = max(1, min(96, int(round(math.sqrt(ch) * _log(rng, 0.7, 1.5)))))
            T = max(1, min(96, int(math.ceil(ch / R))))
            M = 1 if geom == "hand" else rng.randint(1, 256)
            K = rng.randint(16, 512)
            P = int(_log(rng, 200, 300_000))
            per = P // T if mode == "per_tx" else P
            if T * R * M * K <= 1.5e8 and per * float(T * R * M * K) <= 6e12:
                break
        return dict(kind="synth", model=model, geom=geom, mode=mode, T=T, R=R, M=M, K=K, P=P,
                    moving=0.0 if geom == "hand" else round(_log(rng, 5e-4, 5e-2), 5))
    if kind == "image":
        while True:
            T, R, K = rng.randint(4, 96), rng.randint(4, 96), rng.randint(16, 160)
            n = _log(rng, 8, 120)
            nx, ny, nz = (max(3, int(round(n * f))) for f in (0.5, rng.uniform(0.8, 1.2), rng.uniform(0.8, 1.2)))
            if float(nx * ny * nz) * T * R * K <= 1e12:
                break
        return dict(kind="image", T=T, R=R, K=K, nx=nx, ny=ny, nz=nz, step=round(0.2 / max(ny, nz), 6))
    if kind in ("mlp_step", "mlp_eval"):
        return dict(kind=kind, scenes=int(round(_log(rng, 1, 128 if kind == "mlp_eval" else 64))))
    if kind == "batch":
        return dict(kind="batch", scenes=rng.randint(2, 6), seed0=rng.randint(1, 10**6),
                    rays=int(_log(rng, 5e4, 3e5)), tri_hi=int(_log(rng, 2e4, 1e5)), ch_hi=rng.randint(16, 600))
    return dict(kind="motion", rays=int(_log(rng, 1e5, 2e6)), T=rng.randint(16, 96), R=rng.randint(16, 96),
                K=rng.randint(16, 128))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1_000_003 + salt) & 0x7FFFFFFF)


def _scene(case, seed):
    s = int(seed) % 10_007
    if case["scene"] == "tiny":
        return sg.scene_c1(s)
    if case["scene"] == "box":
        return sg.scene_box_family(s)
    if case["scene"] == "hand":
        return sg.scene_hand_proxy(s)
    big = case["scale"] > 0.05
    return sg.scene_street(s, scale=case["scale"], n_cars=20 if big else 5, n_poles=40 if big else 10)


def _array(case):
    if case.get("geom") == "hand" or case["kind"] in ("image", "motion") or case.get("scene") == "hand":
        full = sg.array_square(48)
        pick = lambda n: np.linspace(0, 95, n).round().astype(int)
        return sg.Array(full.tx[pick(case["T"])], full.rx[pick(case["R"])], 0.07, sg.MODE_SHARED).checked()
    if case["kind"] == "synth" and case["mode"] == "shared":
        return sg.array_sparse_grid(case["T"], case["R"], 17)
    if (case["T"], case["R"]) == (1, 4):
        return sg.array_c1()
    return sg.array_ula(case["T"], case["R"])


def _chirp(case):
    if case.get("geom") == "hand" or case["kind"] in ("image", "motion"):
        return sg.chirp_sfcw(n_steps=case["K"])
    return sg.Chirp(n_samples=case["K"], n_chirps=case["M"])


def _path_list(case, seed):
    """A path list as tensors on the GPU (see the module's docstring)."""
    g = _gen(seed, 1)
    n, T = case["P"], case["T"]
    U = lambda lo, hi: lo + (hi - lo) * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    p = torch.zeros((12, n), device=DEV, dtype=torch.float64)
    vid = torch.full((4, n), -1, device=DEV, dtype=torch.int32)
    K = torch.ones(n, device=DEV, dtype=torch.int32)
    vid[0] = 0
    if case["geom"] == "hand":
        p[0], p[1], p[2] = 0.3 + 0.002 * (U(0, 1) < 0.4), U(-0.04, 0.095), U(-0.05, 0.10)
        vel = np.zeros((1, 3))
    else:
        rho = (0.3 * torch.exp(0.9 * torch.randn(n, generator=g, device=DEV, dtype=torch.float64))).clamp(1e-3, 30)
        az = U(-math.pi / 2, math.pi / 2)
        p[0], p[1] = rho * torch.cos(az), rho * torch.sin(az)
        who = U(0, 1)
        far, car = who < 0.006, who > 1 - case["moving"]
        fx, fy, fz = U(2, 60), U(-8, 8), U(0.2, 1.7)
        pole = 21 + (U(0, 40)).to(torch.int32)
        cars = 1 + (U(0, 20)).to(torch.int32)
        away = far | car
        for a, v in ((0, fx), (1, fy), (2, fz)):
            p[a] = torch.where(away, v, p[a])
        vid[0] = torch.where(car, cars, torch.where(far, pole, vid[0]))
        two = U(0, 1) < 0.01                     # a second bounce off the ground near by
        K = torch.where(two, 2, 1).to(torch.int32)
        p[3] = torch.where(two, p[0] + U(-0.4, 0.4), p[3])
        p[4] = torch.where(two, p[1] + U(-0.4, 0.4), p[4])
        vid[1] = torch.where(two, 0, vid[1])
        rng = np.random.default_rng(int(seed) % 65_537)
        vel = np.zeros((61, 3))
        vel[1:21, 0] = rng.uniform(-15, 15, 20)
    if case["mode"] == "shared":
        src = torch.full((n,), -1, device=DEV, dtype=torch.int32)
    else:
        src = torch.sort(torch.randint(0, T, (n,), generator=g, device=DEV, dtype=torch.int32)).values
    amp = torch.full((n,), 1.0 / n, device=DEV, dtype=torch.float64)
    return dict(src=src, K=K, vid=vid, p=p, amp=amp), vel


def _velocity_scene(vel):
    """A mesh with one face per object: synthesis reads only the velocities."""
    n = len(vel)
    v = np.array([[1e3, 0, 0], [1e3, 1, 0], [1e3, 0, 1]], np.float32)
    return sg.Scene(v, np.tile([[0, 1, 2]], (n, 1)), np.arange(n), np.full(n, 0.5, np.float32), vel).checked()


def _grid(case):
    st, nx, ny, nz = case["step"], case["nx"], case["ny"], case["nz"]
    return (0.26, -st * (ny - 1) / 2, -st * (nz - 1) / 2), st, (nx, ny, nz)


def _image_cube(case, seed):
    """A sweep of 48 point scatterers on a hand-sized surface, FP64 summed."""
    g = _gen(seed, 2)
    U = lambda lo, hi: lo + (hi - lo) * torch.rand(48, generator=g, device=DEV, dtype=torch.float64)
    pts = torch.stack([U(0.28, 0.32), U(-0.05, 0.09), U(-0.05, 0.09)], 1)
    amp = U(0.2, 1.0)
    a, ch = _array(case), _chirp(case)
    tx, rx = (torch.as_tensor(x, device=DEV) for x in (a.tx, a.rx))
    dT, dR = torch.cdist(tx, pts), torch.cdist(rx, pts)
    out = torch.empty((a.n_tx * a.n_rx, 1, case["K"]), dtype=torch.complex64, device=DEV)
    for k in range(case["K"]):
        w = -2 * math.pi * (ch.f0 + ch.bandwidth * k / ch.n_samples) / C0
        out[:, 0, k] = (torch.polar(amp.expand_as(dT).contiguous(), w * dT)
                        @ torch.polar(torch.ones_like(dR), w * dR).T.contiguous()).reshape(-1)
    return out


def _mlp_inputs(case, seed):
    g = _gen(seed, 3)
    n = case["scenes"]
    sizes = [(64, 18), (64,), (64, 64), (64,), (64, 64), (64,), (1, 64), (1,)]
    parts = []
    for s in sizes:
        w = torch.randn(int(np.prod(s)), generator=g, device=DEV)
        parts.append(w * (math.sqrt(2.0 / s[1]) if len(s) == 2 else 0.02))
    codes = torch.rand((n, 16), generator=g, device=DEV) * (torch.rand((n, 16), generator=g, device=DEV) < 0.3)
    hists = torch.rand((n, 8192), generator=g, device=DEV) ** 4
    return torch.cat(parts), codes, hists


def prepare(case, seed):
    kind = case["kind"]
    ctx = rr.Context(0)
    st = dict(case=dict(case), ctx=ctx)
    if kind in ("frame", "trace"):
        a = _array(case)
        ctx.upload(_scene(case, seed))
        ctx.set_array(a.tx, a.rx, a.rx_radius, a.mode)
        st["seed"] = int(seed) & 0xFFFFFFFF
        if kind == "frame":
            ch = _chirp(case)
            ctx.set_chirp(ch.f0, ch.bandwidth, ch.t_chirp, ch.t_rep, ch.n_samples, ch.n_chirps)
            st["out"] = torch.empty((a.n_ch, case["M"], case["K"]), dtype=torch.complex64, device=DEV)
        fov = 25 * DEG if case["scene"] == "hand" else math.pi / 2
        st["args"] = dict(n_rays=case["rays"], path_cap=case.get("keep", 0), max_bounces=3 if case["scene"] == "street" else 2,
                          az_min=-fov, az_max=fov, el_min=-fov, el_max=fov, record_hits=False,
                          sampler=rr.PER_TRIANGLE if case.get("sampler") == "per_triangle" else rr.UNIFORM)
    elif kind == "synth":
        a, ch = _array(case), _chirp(case)
        paths, vel = _path_list(case, seed)
        ctx.upload(_velocity_scene(vel))
        ctx.set_array(a.tx, a.rx, a.rx_radius, sg.MODE_SHARED if case["mode"] == "shared" else sg.MODE_PER_TX)
        ctx.set_chirp(ch.f0, ch.bandwidth, ch.t_chirp, ch.t_rep, ch.n_samples, ch.n_chirps)
        ctx.set_paths(paths)
        st["model"] = rr.EXACT if case["model"] == "exact" else rr.SEPARABLE
        st["out"] = torch.empty((a.n_ch, case["M"], case["K"]), dtype=torch.complex64, device=DEV)
    elif kind == "image":
        a, ch = _array(case), _chirp(case)
        ctx.set_array(a.tx, a.rx, a.rx_radius, a.mode)
        ctx.set_chirp(ch.f0, ch.bandwidth, ch.t_chirp, ch.t_rep, ch.n_samples, ch.n_chirps)
        st.update(cube=_image_cube(case, seed), grid=_grid(case))
    elif kind in ("mlp_step", "mlp_eval"):
        params, st["codes"], st["hists"] = _mlp_inputs(case, seed)
        ctx.mlp_set_params(params.cpu().numpy())
    elif kind == "batch":
        s0 = (case["seed0"] + 97 * int(seed)) % 1_000_000_007
        ws = sg.workload_batch(n_scenes=case["scenes"], seed0=s0, rays=case["rays"], tri_hi=case["tri_hi"],
                               ch_hi=case["ch_hi"])
        # channels, samples and chirps are the case's, scenes and arrays the seed's
        for w, v in zip(ws, _batch_shapes(case)):
            w.array = sg.array_sparse_grid(v[0], v[1], s0 % 1000 + 17, mode=sg.MODE_SHARED)
            w.chirp = sg.Chirp(n_samples=v[3], n_chirps=v[2])
        st["batch"] = rr.Batch(ctx, len(ws))
        for i, w in enumerate(ws):
            st["batch"].set_workload(i, w)
        st["cubes"] = st["batch"].alloc_cubes()
    else:
        a, ch = _array(case), _chirp(case)
        scene, frames = sg.hand_motion(int(seed) % 10_007, n_frames=8)
        ctx.upload(scene)
        ctx.set_array(a.tx, a.rx, a.rx_radius, a.mode)
        ctx.set_chirp(ch.f0, ch.bandwidth, ch.t_chirp, ch.t_rep, ch.n_samples, ch.n_chirps)
        st["verts"] = frames[3]
        st["out"] = torch.empty((a.n_ch, 1, case["K"]), dtype=torch.complex64, device=DEV)
        st["args"] = dict(n_rays=case["rays"], max_bounces=2, az_min=-25 * DEG, az_max=25 * DEG,
                          el_min=-25 * DEG, el_max=25 * DEG, record_hits=False)
        st["seed"] = int(seed) & 0xFFFFFFFF
    return st


def _batch_shapes(case):
    """(T, R, M, K) per slot, as `scenegen.workload_batch` spreads them."""
    out = []
    for i in range(case["scenes"]):
        rng = np.random.default_rng(case["seed0"] + i)
        ch = math.exp(rng.uniform(math.log(4), math.log(case["ch_hi"])))
        R = min(64, int(math.ceil(math.sqrt(ch))))
        T = max(1, int(math.ceil(ch / R)))
        out.append((T, R, int(rng.choice([64, 128, 256])), int(rng.choice([128, 256, 512]))))
    return out


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "frame":
        n = ctx.trace(seed=st["seed"], **st["args"])
        return {"paths": n, "cube": ctx.synthesize(model=rr.EXACT, out=st["out"])}
    if kind == "trace":
        ctx.trace(seed=st["seed"], **st["args"])
        p = ctx.paths()
        # hit slots past a path's count hold nothing; every path has one hit
        return {k: (v[0] if k in ("tri", "vid") else v[:3] if k == "p" else v) for k, v in p.items()}
    if kind == "synth":
        return ctx.synthesize(model=st["model"], out=st["out"])
    if kind == "image":
        img = ctx.backproject(st["cube"], st["grid"])
        return {"image": img, "projection": ctx.max_projection(img, st["grid"])}
    if kind == "mlp_step":
        # the last, small steps of a training schedule
        loss, grad = ctx.mlp_train_step(st["codes"], st["hists"], 1e-5, want_grad=True)
        return {"loss": loss, "grad": grad}
    if kind == "mlp_eval":
        return ctx.mlp_forward(st["codes"])
    if kind == "batch":
        counts = st["batch"].launch(st["cubes"])
        return {"counts": counts, "cubes": list(st["cubes"])}
    ctx.update_vertices(st["verts"])
    n = ctx.trace(seed=st["seed"], **st["args"])
    return {"paths": n, "cube": ctx.synthesize(model=rr.EXACT, out=st["out"])}


# ---------------------------------------------------------------------------
# what a pass cannot do without: each input read and each output written once,
# and one operation per ray, path entry, voxel entry or network weight
# ---------------------------------------------------------------------------

TRIS = {"tiny": 14, "box": 14, "hand": 21_176, "street": 509_360}
RETURNED = {"tiny": 0.024, "box": 0.024, "hand": 0.05, "street": 0.0264}


def work(case):
    kind = case["kind"]
    if kind in ("frame", "trace", "motion"):
        scene = case.get("scene", "hand")
        tris = TRIS[scene] * (case["scale"] if scene == "street" else 1)
        rays = case["rays"] * (tris if case.get("sampler") == "per_triangle" else 1)
        paths = case.get("keep") or rays * RETURNED[scene]
        cube = case["T"] * case["R"] * case.get("M", 1) * case["K"] * 8 if kind != "trace" else 0
        return {"bytes": tris * 48 + rays + paths * 100 + cube, "flops": rays * 200.0 + paths * 50.0}
    if kind == "synth":
        cube = case["T"] * case["R"] * case["M"] * case["K"] * 8.0
        return {"bytes": cube + case["P"] * 130.0, "flops": cube + 50.0 * case["P"]}
    if kind == "image":
        vox = float(case["nx"]) * case["ny"] * case["nz"]
        cube = case["T"] * case["R"] * case["K"] * 8.0
        return {"bytes": vox * 8 + cube, "flops": vox * 30.0 * (case["T"] + case["R"]) + cube}
    if kind in ("mlp_step", "mlp_eval"):
        rows = case["scenes"] * 8192.0
        step = kind == "mlp_step"
        return {"bytes": rows * 4 + 9601 * (16 if step else 4), "flops": rows * 2 * 9408 * (3 if step else 1)}
    cubes = sum(8.0 * t * r * m * k for t, r, m, k in _batch_shapes(case))
    rays = case["scenes"] * case["rays"]
    return {"bytes": cubes + rays, "flops": rays * 200.0 + cubes}


# ---------------------------------------------------------------------------
# the same in 64 bits, as plain torch gives it
# ---------------------------------------------------------------------------

def _cis(u):
    """exp(-j 2 pi u), u in cycles."""
    return torch.polar(torch.ones_like(u), (-2 * math.pi) * (u - torch.floor(u)))


def _hits_at(paths, vel, tau):
    """First and last hit points at time tau and the length between them."""
    p, vid, K = paths["p"], paths["vid"].long(), paths["K"]
    v = torch.as_tensor(vel, device=DEV)
    q = lambda j: p[3 * j:3 * j + 3].T + v[vid[j].clamp(min=0)] * tau
    first = last = q(0)
    inner = torch.zeros_like(p[0])
    for j in (1, 2, 3):
        m = K > j
        if bool(m.any()):
            nxt = q(j)
            inner = inner + torch.where(m, (nxt - last).norm(dim=1), 0.0)
            last = torch.where(m[:, None], nxt, last)
    return first, last, inner


def _exact_chirp(case, ch, sub, vel, w, et, rx, oT, oR, m):
    """Samples of chirp m, [channels of et x rx][K], from the paths `sub`."""
    K, nt, R, n = case["K"], et.shape[0], rx.shape[0], w.numel()
    fk = torch.tensor([(ch.f0 + ch.bandwidth * k / K) / C0 for k in range(K)], device=DEV, dtype=torch.float64)
    dist = lambda e, q: (e[:, None, :] - q[None, :, :]).norm(dim=2)
    q1, qk, inner = _hits_at(sub, vel, m * ch.t_rep)
    o = torch.empty((nt * R, K), dtype=torch.complex128, device=DEV)
    if case["model"] == "separable":
        p1, pk, _ = _hits_at(sub, vel, 0.0)
        dT = dist(et, p1) - (p1 - oT).norm(dim=1)
        dR = dist(rx, pk) - (pk - oR).norm(dim=1)
        A = ((_cis(dT * fk[0]) * w)[:, None, :] * _cis(dR * fk[0])[None]).reshape(nt * R, n)
        D = (q1 - oT).norm(dim=1) + inner + (qk - oR).norm(dim=1)
        step = max(1, 100_000_000 // n)
        for k in range(0, K, step):
            o[:, k:k + step] = A @ _cis(D[:, None] * fk[None, k:k + step])
        return o
    dX, dY = dist(et, q1) + inner, dist(rx, qk)
    step = max(1, 50_000_000 // (n * (nt + R)))
    for k in range(0, K, step):
        f = fk[k:k + step, None, None]
        X, Y = _cis(dX[None] * f) * w, _cis(dY.T.contiguous()[None] * f)
        o[:, k:k + step] = torch.bmm(X, Y).reshape(-1, nt * R).T
    return o


def _exact_synth(case, seed):
    T, R, M, K, P = (case[k] for k in ("T", "R", "M", "K", "P"))
    per = P / T if case["mode"] == "per_tx" else P
    if per * float(T * R * M * K) > 6e13:
        return None
    a, ch = _array(case), _chirp(case)
    paths, vel = _path_list(case, seed)
    tx, rx = (torch.as_tensor(x, device=DEV) for x in (a.tx, a.rx))
    oT, oR = tx.mean(0), rx.mean(0)
    out = torch.empty((T * R, M, K), dtype=torch.complex128, device=DEV)
    amp = paths["amp"].to(torch.complex128)
    if case["mode"] == "shared":
        groups = [(slice(0, P), range(T))]
    else:
        at = torch.searchsorted(paths["src"], torch.arange(T + 1, device=DEV, dtype=torch.int32)).tolist()
        groups = [(slice(at[t], at[t + 1]), range(t, t + 1)) for t in range(T)]
    moves = (torch.as_tensor(vel, device=DEV)[paths["vid"].long().clamp(min=0)] != 0).any(2) & (paths["vid"] >= 0)
    moves = moves.any(0)
    out.zero_()
    for sl, ts in groups:
        for moving in (False, True):             # a path at rest adds the same to every chirp
            sel = torch.arange(P, device=DEV)[sl]
            sel = sel[moves[sl] == moving]
            if sel.numel() == 0:
                continue
            sub = {k: v[..., sel] for k, v in paths.items()}
            o = out[ts[0] * R:(ts[-1] + 1) * R]
            for m in range(M if moving else 1):
                part = _exact_chirp(case, ch, sub, vel, amp[sel], tx[ts[0]:ts[-1] + 1], rx,
                                    oT if case["mode"] == "shared" else tx[ts[0]], oR, m)
                if moving:
                    o[:, m] += part
                else:
                    o += part[:, None, :]
    return out


def _exact_image(case, seed):
    a, ch = _array(case), _chirp(case)
    cube = _image_cube(case, seed).to(torch.complex128)[:, 0].reshape(case["T"], case["R"], case["K"])
    (x0, y0, z0), st, (nx, ny, nz) = _grid(case)
    ax = [o + st * torch.arange(n, device=DEV, dtype=torch.float64) for o, n in ((x0, nx), (y0, ny), (z0, nz))]
    vox = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
    tx, rx = (torch.as_tensor(x, device=DEV) for x in (a.tx, a.rx))
    img = torch.zeros(vox.shape[0], dtype=torch.complex128, device=DEV)
    for v0 in range(0, vox.shape[0], 1 << 18):
        v = vox[v0:v0 + (1 << 18)]
        dT, dR = ((e[:, None, :] - v[None]).norm(dim=2) for e in (tx, rx))
        acc = torch.zeros(v.shape[0], dtype=torch.complex128, device=DEV)
        for k in range(case["K"]):
            fk = -(ch.f0 + ch.bandwidth * k / ch.n_samples) / C0
            acc += (_cis(dT * fk) * (cube[:, :, k].contiguous() @ _cis(dR * fk))).sum(0)
        img[v0:v0 + (1 << 18)] = acc
    mag = img.abs().reshape(nx, ny * nz).max(0).values
    db = (20 * torch.log10(mag / mag.max())).clamp(min=-15.0).reshape(ny, nz)
    return {"image": img.reshape(nx, ny, nz), "projection": db}


def _exact_mlp(case, seed):
    params, codes, hists = (x.double() for x in _mlp_inputs(case, seed))
    params.requires_grad_(case["kind"] == "mlp_step")
    b = torch.arange(8192, device=DEV)
    ua, ue = 2 * (b % 128 + 0.5) / 128 - 1, 2 * (b // 128 + 0.5) / 64 - 1
    at, h = 0, None
    n = case["scenes"]
    x = torch.cat([torch.stack([ua, ue], 1).double().expand(n, -1, -1), codes[:, None, :].expand(-1, 8192, -1)], 2)
    for rows, cols in ((64, 18), (64, 64), (64, 64), (1, 64)):
        W, bias = params[at:at + rows * cols].reshape(rows, cols), params[at + rows * cols:at + rows * cols + rows]
        at += rows * cols + rows
        x = x @ W.T + bias
        x = torch.relu(x) if rows > 1 else x[:, :, 0]
    if case["kind"] == "mlp_eval":
        return x
    loss = -(hists * torch.log_softmax(x, 1)).sum(1).div(hists.sum(1)).mean()
    loss.backward()
    return {"loss": float(loss), "grad": params.grad}


def exact(case, seed):
    if case["kind"] == "synth":
        return _exact_synth(case, seed)
    if case["kind"] == "image":
        return _exact_image(case, seed)
    if case["kind"] in ("mlp_step", "mlp_eval"):
        return _exact_mlp(case, seed)
    return None
