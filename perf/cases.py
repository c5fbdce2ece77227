"""The work a user of this package has it do, as a fixed set of timed cases.

listed() names the cases and draw() gives more of the same ranges; prepare()
makes the inputs and the handles a program keeps between calls, run() is one
pass through the public entry points, work() the bytes and operations a pass
cannot do without, and exact() the same results in FP64 from plain torch.

Two kinds of work:

* the lattice Boltzmann solver (lbm.Solver, lbm.BatchSolver): a run of time
  steps, eager or as HIP-graph replays, and the read-out that follows it
  (density fields on the device, the observables' record);
* the surrogate network (surrogate.UNet and its layer calls): inference,
  a training step, and one convolution layer forward and backward.
"""
import math
import os

import numpy as np
import torch

from paper_2111_08666_amd import inputs as I
from paper_2111_08666_amd import lbm
from paper_2111_08666_amd import surrogate as S

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(S.__file__)), "weights", "unet_drainage256.npz")
LEVELS = (32, 64, 128, 256)
IN_CH = 8
SRT, MRT, TRT = 0, 1, 2


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed():
    return [
        # A trial domain stepped eagerly, as in an interactive session or a
        # test: launches and latency are all there is.
        dict(name="eager_127x37", kind="drain2d", nx=127, ny=37, coll=TRT, math=0, storage=0, G=3.5,
             eager=1, steps=20, reps=1, record=0),
        # A drainage at the size of the small workload, watched: graph replays
        # between two looks at the observables.
        dict(name="watched_128x64", kind="drain2d", nx=128, ny=64, coll=MRT, math=0, storage=0, G=3.5,
             eager=0, steps=100, reps=2, record=1),
        # The large drainage workload of the pressure protocol.
        dict(name="drain_1024x512", kind="drain2d", nx=1024, ny=512, coll=MRT, math=0, storage=0, G=3.5,
             eager=0, steps=50, reps=2, record=0),
        # A study medium of ragged size in FP64 node arithmetic.
        dict(name="drain_401x203_f64", kind="drain2d", nx=401, ny=203, coll=MRT, math=1, storage=0, G=3.5,
             eager=0, steps=50, reps=2, record=0),
        # A calibration sweep: periodic droplets of one size in one batch.
        dict(name="droplets_9x192", kind="droplets", k=9, n=192, coll=SRT, math=0, steps=50, reps=2),
        # A production sweep: uneven drainage instances in one batch, larger
        # than the last-level cache, watched.
        dict(name="sweep_24", kind="sweep", k=24, lo=4, hi=14, coll=MRT, storage=0, steps=20, reps=2),
        # 3D drainage in a sphere pack, resident in HBM.
        dict(name="pack_192", kind="pack3d", nx=192, ny=192, nz=192, coll=TRT, math=0, storage=0, steps=10, reps=1),
        # A smaller ragged pack held in BF16 deviations.
        dict(name="pack_130x97x101_bf16", kind="pack3d", nx=130, ny=97, nz=101, coll=SRT, math=0, storage=1,
             steps=10, reps=1),
        # A 3D droplet in a periodic box: every node fluid.
        dict(name="box_96", kind="box3d", n=96, coll=TRT, steps=20, reps=1),
        # One field's warm start: the trained network on a single medium.
        dict(name="unet_infer_1x256", kind="infer", n=1, h=256, w=256),
        # A training step at the batch the network was trained with.
        dict(name="unet_train_16x256", kind="train", n=16, h=256, w=256),
        # One 3x3 layer with its ReLU, forward and backward.
        dict(name="conv_64to64_16x128", kind="conv", n=16, h=128, w=128, cin=64, cout=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["drain2d", "drain2d", "droplets", "sweep", "pack3d", "box3d", "infer", "train", "conv", "conv"])
    if kind == "drain2d":
        nx = _log(rng, 96, 1100)
        ny = max(37, min(560, int(nx * rng.uniform(0.35, 0.7))))
        eager = int(rng.random() < 0.2)
        steps = 2 * rng.randint(5, 30)
        record = int(rng.random() < 0.3)  # a watched run has to stay finite over many passes: MRT
        return dict(kind=kind, nx=nx, ny=ny, coll=MRT if record else rng.choice([SRT, MRT, TRT]),
                    math=int(rng.random() < 0.2), storage=int(rng.random() < 0.15), G=3.5, eager=eager, steps=steps,
                    reps=1 if eager else rng.randint(1, 3), record=record)
    if kind == "droplets":
        return dict(kind=kind, k=rng.randint(2, 15), n=rng.randint(96, 200), coll=rng.choice([SRT, MRT, TRT]),
                    math=int(rng.random() < 0.2), steps=2 * rng.randint(5, 25), reps=rng.randint(1, 2))
    if kind == "sweep":
        lo = rng.randint(4, 6)
        return dict(kind=kind, k=rng.randint(4, 24), lo=lo, hi=rng.randint(lo, 12), coll=MRT,
                    storage=int(rng.random() < 0.2), steps=2 * rng.randint(3, 10), reps=rng.randint(1, 2))
    if kind == "pack3d":
        nx, ny, nz = (_log(rng, 48, 176) for _ in range(3))
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, coll=rng.choice([SRT, TRT, TRT]), math=int(rng.random() < 0.2),
                    storage=int(rng.random() < 0.25), steps=2 * rng.randint(2, 5), reps=1)
    if kind == "box3d":
        return dict(kind=kind, n=rng.randint(40, 110), coll=rng.choice([SRT, TRT]), steps=2 * rng.randint(3, 8), reps=1)
    if kind == "infer":
        if rng.random() < 0.5:  # the fields the network was trained on
            return dict(kind=kind, n=rng.randint(1, 16), h=256, w=256)
        return dict(kind=kind, n=rng.randint(1, 8), h=8 * rng.randint(8, 32), w=8 * rng.randint(8, 50))
    if kind == "train":
        s = rng.choice([128, 256])
        return dict(kind=kind, n=rng.randint(2, 15), h=s, w=s)
    c = rng.choice([(8, 32), (32, 32), (32, 64), (64, 64), (64, 32), (64, 128), (128, 64), (128, 128), (128, 256),
                    (256, 256), (256, 128)])
    if rng.random() < 0.6:  # a level of the network
        s = {8: 256, 32: 256, 64: 128, 128: 64, 256: 32}[max(c) if c[0] != 8 else 8]
        return dict(kind=kind, n=rng.randint(1, 16), h=s, w=s, cin=c[0], cout=c[1])
    return dict(kind=kind, n=rng.randint(1, 4), h=rng.randint(16, 120), w=rng.randint(16, 200), cin=c[0], cout=c[1])


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _discs(nx, ny, rmin, rmax, porosity, rng, reservoir=8, gap=1.0):
    """Non-overlapping random discs between two walls, `reservoir` columns free
    at both ends, as in the package's 2D media; candidates are tested against
    all placed discs at once, so that a medium takes milliseconds."""
    m = np.zeros((ny, nx), np.uint8)
    m[0] = m[-1] = 1
    x0, x1 = reservoir, nx - reservoir
    target = (1.0 - porosity) * (x1 - x0) * (ny - 2)
    cx, cy, cr = np.empty(0), np.empty(0), np.empty(0)
    area = 0.0
    for _ in range(60):
        r = rng.uniform(rmin, rmax, 512)
        x, y = rng.uniform(x0, x1, 512), rng.uniform(1, ny - 1, 512)
        ok = (x - r >= x0) & (x + r <= x1 - 1) & (y - r >= 1 + gap) & (y + r <= ny - 2 - gap)
        if cx.size:
            d2 = (x[:, None] - cx) ** 2 + (y[:, None] - cy) ** 2
            ok &= (d2 >= (r[:, None] + cr + gap) ** 2).all(axis=1)
        n0 = cx.size
        for k in np.flatnonzero(ok):
            if np.any((cx[n0:] - x[k]) ** 2 + (cy[n0:] - y[k]) ** 2 < (cr[n0:] + r[k] + gap) ** 2):
                continue
            cx, cy, cr = np.append(cx, x[k]), np.append(cy, y[k]), np.append(cr, r[k])
            area += math.pi * r[k] * r[k]
            if area >= target:
                break
        if area >= target:
            break
    for x, y, r in zip(cx, cy, cr):
        a, b = int(x - r), int(x + r) + 2
        c, d = int(y - r), int(y + r) + 2
        yy, xx = np.ogrid[c:d, a:b]
        m[c:d, a:b][((xx - x) ** 2 + (yy - y) ** 2 <= r * r)[:m[c:d, a:b].shape[0], :m[c:d, a:b].shape[1]]] = 1
    return m


def _spheres(nx, ny, nz, rmin, rmax, porosity, rng, reservoir=8):
    """Overlapping random spheres between walls in y and z (Boolean medium)."""
    m = np.zeros((nz, ny, nx), np.uint8)
    m[:, 0] = m[:, -1] = m[0] = m[-1] = 1
    lo, hi = reservoir, nx - reservoir
    mean = math.pi / 3 * (rmax + rmin) * (rmax ** 2 + rmin ** 2)  # of 4/3 pi r^3
    count = int(-math.log(porosity) * (hi - lo) * (ny - 2) * (nz - 2) / mean)
    r = rng.uniform(rmin, rmax, count)
    c = np.stack([rng.uniform(lo, hi, count), rng.uniform(1, ny - 1, count), rng.uniform(1, nz - 1, count)], 1)
    for (x, y, z), s in zip(c, r):
        a, b = max(lo, math.floor(x - s)), min(hi, math.ceil(x + s) + 1)
        e, f = max(1, math.floor(y - s)), min(ny - 1, math.ceil(y + s) + 1)
        g, h = max(1, math.floor(z - s)), min(nz - 1, math.ceil(z + s) + 1)
        zz, yy, xx = np.ogrid[g:h, e:f, a:b]
        m[g:h, e:f, a:b][(xx - x) ** 2 + (yy - y) ** 2 + (zz - z) ** 2 <= s * s] = 1
    return m


def _front(mask, minor, reservoir=8):
    """Component 1 in the inlet reservoir, component 2 in the medium."""
    rho = np.empty((2,) + mask.shape)
    rho[0], rho[1] = minor, 1.0
    rho[0][..., :reservoir], rho[1][..., :reservoir] = 1.0, minor
    rho[:, mask != 0] = 0.0
    return rho


def _droplet(shape, r0, shift, width=5.0, minor=0.027):
    g = np.meshgrid(*[np.arange(n) for n in shape], indexing="ij")
    d2 = sum((a - n / 2 - s) ** 2 for a, n, s in zip(g, shape, shift))
    t = np.tanh(2.0 * (np.sqrt(d2) - r0) / width)
    return np.stack([0.5 * (1 + minor) - 0.5 * (1 - minor) * t, 0.5 * (1 + minor) + 0.5 * (1 - minor) * t])


TAU_M10 = (1.7, 0.62)


def _problems(case, seed):
    """The instances of a solver case, as plain dicts of the solver's inputs."""
    rng = np.random.default_rng([seed, 7])
    kind = case["kind"]
    out = []
    if kind == "drain2d":
        small = case["nx"] < 300
        r = (3.0, 8.0) if small else (4.0, 20.0)
        m = _discs(case["nx"], case["ny"], *r, 0.65, rng)
        out.append(dict(q=9, mask=m, rho0=_front(m, 0.027), open_x=1, periodic=0,
                        tau=(1.0, 1.0) if case["coll"] == SRT else TAU_M10, G=case["G"], xi=-0.4,
                        rho_in1=1.0 + 3 * 10 ** rng.uniform(-3.5, -2.3)))
    elif kind == "droplets":
        for i in range(case["k"]):
            m = np.zeros((case["n"], case["n"]), np.uint8)
            out.append(dict(q=9, mask=m, rho0=_droplet(m.shape, case["n"] * rng.uniform(0.12, 0.25), rng.uniform(-3, 3, 2)),
                            open_x=0, periodic=3, tau=((1.0, 1.0), (1.7, 0.62), (0.62, 1.0))[i % 3], G=3.5, xi=0.0,
                            rho_in1=1.0))
    elif kind == "sweep":
        for i in range(case["k"]):
            nx = 64 * int(np.random.default_rng([i, case["k"]]).integers(case["lo"], case["hi"] + 1))
            m = _discs(nx, nx // 2, 4.0, 20.0, 0.62, rng)
            out.append(dict(q=9, mask=m, rho0=_front(m, 0.027), open_x=1, periodic=0, tau=TAU_M10, G=3.5,
                            xi=rng.uniform(-0.5, 0.5), rho_in1=1.0 + 3 * 10 ** rng.uniform(-4, -2.3)))
    elif kind == "pack3d":
        m = _spheres(case["nx"], case["ny"], case["nz"], 6.0, 14.0, 0.42, rng)
        out.append(dict(q=19, mask=m, rho0=_front(m, 0.027), open_x=1, periodic=0,
                        tau=(1.0, 1.0) if case["coll"] == SRT else TAU_M10, G=3.5, xi=-0.3, rho_in1=1.015))
    else:  # box3d
        n = case["n"]
        m = np.zeros((n, n, n), np.uint8)
        out.append(dict(q=19, mask=m, rho0=_droplet(m.shape, n * rng.uniform(0.2, 0.3), rng.uniform(-2, 2, 3)),
                        open_x=0, periodic=7, tau=(1.0, 1.0), G=3.5, xi=0.0, rho_in1=1.0))
    for p in out:
        p["coll"] = case["coll"]
    return out


def _problem(p):
    nx = p["mask"].shape[-1]
    return I.Problem(q=p["q"], mask=p["mask"], rho0=p["rho0"], periodic=p["periodic"], open_x=p["open_x"],
                     porous_x0=8 if p["open_x"] else 0, porous_x1=nx - 8 if p["open_x"] else 0, collision=p["coll"],
                     tau=p["tau"], G=p["G"], xi=p["xi"], rho_in1=p["rho_in1"], rho_out2=1.0)


def _bf16(a):
    """Rounded to BF16 values."""
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).bfloat16().float().numpy()


def _specs():
    specs, prev = [], IN_CH
    for k, ch in enumerate(LEVELS):
        specs += [(f"enc{k}a", 3, prev, ch), (f"enc{k}b", 3, ch, ch)]
        prev = ch
    for k in range(len(LEVELS) - 2, -1, -1):
        specs += [(f"up{k}", 2, LEVELS[k + 1], LEVELS[k]), (f"dec{k}a", 3, 2 * LEVELS[k], LEVELS[k]),
                  (f"dec{k}b", 3, LEVELS[k], LEVELS[k])]
    return specs


def _params(case, seed):
    """Weights of a network case: the trained ones for inference, a fresh
    draw for training (BF16 values, as the kernels hold them)."""
    p = {}
    if case["kind"] == "infer":
        with np.load(WEIGHTS, allow_pickle=False) as z:
            for k in z.files:
                if k != "levels":
                    a = z[k]
                    p[k] = (a.astype(np.uint32) << 16).view(np.float32) if a.dtype == np.uint16 else a
        return p
    rng = np.random.default_rng([seed, 3])
    for name, t, ci, co in _specs():
        p[name + ".w"] = _bf16(rng.normal(0.0, math.sqrt(2.0 / (t * t * ci)), (co, t, t, ci)))
        p[name + ".b"] = rng.normal(0.0, 0.02, co).astype(np.float32)
    p["head.w"] = rng.normal(0.0, math.sqrt(1.0 / LEVELS[0]), LEVELS[0]).astype(np.float32)
    p["head.b"] = np.zeros(1, np.float32)
    return p


def _fields(case, seed):
    """Network input planes (solid map, contact angle, pressure step), target
    and fluid mask: smooth random blobs for the solid and the saturation."""
    g = torch.Generator(device="cpu").manual_seed(seed)
    n, h, w = case["n"], case["h"], case["w"]

    def blobs(share):
        c = torch.rand(n, 1, max(2, h // 12), max(2, w // 12), generator=g)
        f = torch.nn.functional.interpolate(c, size=(h, w), mode="bicubic", align_corners=False)[:, 0]
        return f > torch.quantile(f[:, ::4, ::4].reshape(-1)[:100000], 1 - share)

    x = torch.zeros(n, h, w, IN_CH)
    solid = blobs(0.45)
    x[..., 0] = solid.float()
    x[..., 1] = (torch.rand(n, 1, 1, generator=g) * 2 - 1)
    x[..., 2] = (torch.rand(n, 1, 1, generator=g) * 2 - 1)
    return x.bfloat16(), (blobs(0.3) & ~solid).float(), (~solid).to(torch.uint8)


def _layer(case, seed):
    """Operands of one convolution layer: activations after a ReLU, weights,
    bias and the gradient from above, BF16."""
    g = torch.Generator(device="cpu").manual_seed(seed)
    n, h, w, ci, co = (case[k] for k in ("n", "h", "w", "cin", "cout"))
    x = torch.randn(n, h, w, ci, generator=g).clamp_(min=0).bfloat16()
    wt = (torch.randn(co, 3, 3, ci, generator=g) * math.sqrt(2.0 / (9 * ci))).bfloat16()
    b = torch.randn(co, generator=g) * 0.05
    dy = (torch.randn(n, h, w, co, generator=g) * 1e-3).bfloat16()
    return x, wt, b, dy


# --------------------------------------------------------------------------
# prepare and run
# --------------------------------------------------------------------------
SOLVER = ("drain2d", "droplets", "sweep", "pack3d", "box3d")


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case)
    if kind in SOLVER:
        probs = [_problem(p) for p in _problems(case, seed)]
        opt = dict(math=case.get("math", 0), storage=case.get("storage", 0))
        if kind in ("droplets", "sweep"):
            st["s"] = lbm.BatchSolver(probs, **opt)
        else:
            st["s"] = lbm.Solver(probs[0], **opt)
        st["out"] = [torch.empty((2,) + p.mask.shape, dtype=torch.float32, device="cuda") for p in probs]
    elif kind in ("infer", "train"):
        net = S.UNet(levels=LEVELS, seed=0)
        net.set_params(_params(case, seed))
        x, t, m = _fields(case, seed)
        st.update(net=net, x=x.cuda().view(torch.int16), t=t.cuda(), m=m.cuda(), count=int(m.sum()))
    else:
        x, wt, b, dy = _layer(case, seed)
        n, h, w, ci, co = (case[k] for k in ("n", "h", "w", "cin", "cout"))
        e = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda")  # noqa: E731
        f = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")  # noqa: E731
        st.update(x=x.cuda(), wt=wt.cuda(), b=b.cuda(), dy=dy.cuda(), y=e(n, h, w, co), g=e(n, h, w, co),
                  flip=e(ci, 3, 3, co), dx=e(n, h, w, ci), dw=f(co, 3, 3, ci), db=f(co),
                  part=f(S.lib().unet_wgrad_scratch_floats(n, h, w, ci, co, 9)))
    return st


RECORD = ("sum_rho_w", "sum_rho", "s_w_weighted", "p_in", "p_out", "pc")


def _advance(st):
    s = st["s"]
    if st.get("eager"):
        s.step(st["steps"])
    else:
        s.step_graph(st["steps"], st["reps"])


def run(st):
    kind = st["kind"]
    if kind in SOLVER:
        s, out = st["s"], st["out"]
        _advance(st)
        if kind in ("droplets", "sweep"):
            obs = s.observables()
            for i, o in enumerate(out):
                lbm.lib().lbm_batch_get_density(s._h, i, o.data_ptr(), 1)
        else:
            obs = [s.observables()] if st.get("record") else []
            s.density_device(out[0])
        rec = [[*o["mass"], *(o[k] for k in RECORD)] for o in obs]
        return {"density": out, "record": np.array(rec, np.float32)}
    if kind == "infer":
        return st["net"].forward(st["x"])
    if kind == "train":
        net = st["net"]
        loss = net.train_step(st["x"], st["t"], st["m"], lr=1e-4, count=st["count"])
        return {"loss": loss, "grad": net.g, "params": net.p, "sat": net.sat}
    n, h, w, ci, co = (st[k] for k in ("n", "h", "w", "cin", "cout"))
    p, call = S.ptr, S.call
    s = torch.cuda.current_stream().cuda_stream
    call("unet_conv3x3_fwd", p(st["x"]), n, h, w, ci, ci, 0, p(st["wt"]), p(st["b"]), co, p(st["y"]), co, 0, 1, s)
    st["g"].copy_(st["dy"])
    call("unet_relu_bwd", p(st["y"]), n * h * w, co, co, 0, p(st["g"]), co, 0, s)
    call("unet_conv3x3_wgrad", p(st["x"]), n, h, w, ci, ci, 0, p(st["g"]), co, co, 0, p(st["dw"]), p(st["db"]),
         p(st["part"]), 0, s)
    call("unet_conv3x3_flip", p(st["wt"]), co, ci, p(st["flip"]), s)
    call("unet_conv3x3_fwd", p(st["g"]), n, h, w, co, co, 0, p(st["flip"]), None, ci, p(st["dx"]), ci, 0, 0, s)
    return {"y": st["y"], "dx": st["dx"], "dw": st["dw"], "db": st["db"]}


# --------------------------------------------------------------------------
# work
# --------------------------------------------------------------------------
# bytes per fluid node and step: every population read once and written once
NODE_BYTES = {(9, 0): 144, (9, 1): 80, (19, 0): 304, (19, 1): 160}
NODE_FLOPS = {9: 500, 19: 1100}


def work(case):
    kind = case["kind"]
    if kind in SOLVER:
        steps = case["steps"] * case["reps"]
        q = 19 if kind in ("pack3d", "box3d") else 9
        if kind == "drain2d":
            nodes = 0.65 * case["nx"] * case["ny"]
            dense = case["nx"] * case["ny"]
        elif kind == "droplets":
            nodes = dense = case["k"] * case["n"] ** 2
        elif kind == "sweep":
            dense = sum((64 * int(np.random.default_rng([i, case["k"]]).integers(case["lo"], case["hi"] + 1))) ** 2 // 2
                        for i in range(case["k"]))
            nodes = 0.62 * dense
        elif kind == "pack3d":
            dense = case["nx"] * case["ny"] * case["nz"]
            nodes = 0.42 * dense
        else:
            nodes = dense = case["n"] ** 3
        return dict(bytes=nodes * steps * NODE_BYTES[q, case.get("storage", 0)] + 8 * dense,
                    flops=nodes * steps * NODE_FLOPS[q])
    n, h, w = case["n"], case["h"], case["w"]
    if kind == "conv":
        ci, co = case["cin"], case["cout"]
        px = n * h * w
        return dict(bytes=2 * px * (2 * ci + 2 * co + co) + 4 * 9 * ci * co + 2 * 2 * 9 * ci * co,
                    flops=3 * 2 * px * 9 * ci * co)
    nbytes, flops = 0, 0
    for name, t, ci, co in _specs():
        lv = int(name[3]) if t == 3 else int(name[2:])
        px = n * (h >> lv) * (w >> lv)
        flops += 2 * px * (9 if t == 3 else 1) * ci * co
        nbytes += 2 * (px * co + (px if t == 3 else px // 4) * ci) + 2 * t * t * ci * co
    return dict(bytes=nbytes if kind == "infer" else 3 * nbytes, flops=flops if kind == "infer" else 3 * flops)


# --------------------------------------------------------------------------
# the same in FP64, from plain torch
# --------------------------------------------------------------------------
E9 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
E19 = [(0, 0, 0)] + [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)
                     if 0 < abs(x) + abs(y) + abs(z) < 3]


def _lattice(q):
    e = E9 if q == 9 else E19
    w0 = {9: (4 / 9, 1 / 9, 1 / 36), 19: (1 / 3, 1 / 18, 1 / 36)}[q]
    w = [w0[sum(abs(c) for c in v)] for v in e]
    opp = [e.index(tuple(-c for c in v)) for v in e]
    return e, w, opp


def _moments9():
    """Rows of the D2Q9 moment basis rho, e, eps, jx, qx, jy, qy, pxx, pxy."""
    rows = []
    for ex, ey, _ in E9:
        s = ex * ex + ey * ey
        rows.append((1, -4 + 3 * s, 4 - 10.5 * s + 4.5 * s * s, ex, (-5 + 3 * s) * ex, ey, (-5 + 3 * s) * ey,
                     ex * ex - ey * ey, ex * ey))
    return torch.tensor(rows, dtype=torch.float64).T.contiguous()


def _exact_density(p, steps, dev):
    q = p["q"]
    e, w, opp = _lattice(q)
    f64 = dict(dtype=torch.float64, device=dev)
    shape = p["mask"].shape
    three = shape if len(shape) == 3 else (1,) + shape
    solid = torch.from_numpy(p["mask"]).to(dev).bool().reshape(three)
    fluid = (~solid).to(torch.float64)
    rho0 = torch.from_numpy(p["rho0"]).to(**f64).reshape((2,) + three)
    fs = torch.stack([wi * rho0 for wi in w], 1)
    nx = three[2]
    open_x = p["open_x"]
    lam, s_e, s_eps = 3.0 / 16.0, 1.0, 1.0  # the problem description's defaults
    tau1, tau2 = p["tau"]

    def at(a, v):  # a at x - v
        return torch.roll(a, (v[2], v[1], v[0]), (-3, -2, -1))

    def inside(a, v):  # zero where x - v left an open x face
        if open_x and v[0]:
            a = a.clone()
            a[..., 0 if v[0] > 0 else nx - 1] = 0
        return a

    neg = [tuple(-c for c in v) for v in e]
    from_solid = [at(solid, v) for v in e]
    weight = sum(wi * inside(at(fluid, v), v) for wi, v in list(zip(w, neg))[1:])
    weight = torch.where(weight > 0, weight, torch.ones_like(weight))
    M = _moments9().to(dev) if q == 9 else None

    def pull():
        f = torch.empty_like(fs)
        for i, v in enumerate(e):
            f[:, i] = torch.where(from_solid[i], fs[:, opp[i]], at(fs[:, i], v))
        if not open_x:
            return f
        for x, normal, zc, rho_b, other in ((0, 1, 0, p["rho_in1"], 1), (nx - 1, -1, 1, 1.0, 0)):
            g = f[..., x]
            for i, v in enumerate(e):  # the other component's missing links
                if v[0] == normal:
                    g[other, i] = fs[other, i, ..., x] if normal > 0 else w[i] * rho0[0, ..., x]
            par = sum(g[zc, i] for i, v in enumerate(e) if v[0] == 0)
            out = sum(g[zc, i] for i, v in enumerate(e) if v[0] == -normal)
            ty = 0.5 * sum(v[1] * g[zc, i] for i, v in enumerate(e) if v[0] == 0)
            tz = 0.5 * sum(v[2] * g[zc, i] for i, v in enumerate(e) if v[0] == 0)
            m = rho_b - par - 2 * out
            for i, v in enumerate(e):
                if v[0] == normal:
                    g[zc, i] = g[zc, opp[i]] + 6 * w[i] * m - v[1] * ty - v[2] * tz
        return f

    for _ in range(steps):
        f = pull()
        rho = f.sum(1) * fluid
        psi = rho.clone()
        for c, chi in ((0, 1 + p["xi"]), (1, 1 - p["xi"])):
            virt = chi * sum(wi * inside(at(rho[c], v), v) for wi, v in list(zip(w, neg))[1:]) / weight
            psi[c] = torch.where(solid, virt, rho[c])
        F = torch.zeros((2, 3) + three, **f64)
        for c in range(2):
            for i, v in enumerate(e):
                if not i:
                    continue
                b = at(psi[1 - c], neg[i])
                if open_x and v[0]:  # mirrored pairs cancel at an open face
                    b = b.clone()
                    b[..., 0] = b[..., nx - 1] = 0
                for d in range(3):
                    if v[d]:
                        F[c, d] -= p["G"] * w[i] * v[d] * b
            F[c] *= rho[c]
        tot = rho[0] + rho[1]
        tot = torch.where(solid, torch.ones_like(tot), tot)
        u = [(sum(v[d] * (f[0, i] + f[1, i]) for i, v in enumerate(e) if v[d]) + 0.5 * (F[0, d] + F[1, d])) / tot
             if any(v[d] for v in e) else torch.zeros_like(tot) for d in range(3)]
        tau = (rho[0] * tau1 + rho[1] * tau2) / tot
        tau = torch.where(solid, torch.ones_like(tau), tau)
        s_nu = 1 / tau
        s_q = 1 / (0.5 + lam / (tau - 0.5))
        s_j = torch.minimum(s_nu, s_q)
        usq = u[0] ** 2 + u[1] ** 2 + u[2] ** 2
        for c in range(2):
            dep, src = [], []
            uF = u[0] * F[c, 0] + u[1] * F[c, 1] + u[2] * F[c, 2]
            for i, v in enumerate(e):
                eu = sum(v[d] * u[d] for d in range(3)) if i else torch.zeros_like(tot)
                eF = sum(v[d] * F[c, d] for d in range(3)) if i else torch.zeros_like(tot)
                dep.append(w[i] * rho[c] * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * usq) - f[c, i])
                src.append(w[i] * (3 * (eF - uF) + 9 * eu * eF))
            if p["coll"] == SRT:
                df = [s_nu * a + (1 - 0.5 * s_nu) * b for a, b in zip(dep, src)]
            elif p["coll"] == TRT:
                df = [0.5 * (s_nu * (dep[i] + dep[opp[i]]) + s_q * (dep[i] - dep[opp[i]])
                             + (1 - 0.5 * s_nu) * (src[i] + src[opp[i]]) + (1 - 0.5 * s_q) * (src[i] - src[opp[i]]))
                      for i in range(q)]
            else:
                rate = [torch.ones_like(tau), s_e * torch.ones_like(tau), s_eps * torch.ones_like(tau), s_j, s_q, s_j,
                        s_q, s_nu, s_nu]
                mom = [r * sum(M[k, i] * dep[i] for i in range(9)) + (1 - 0.5 * r) * sum(M[k, i] * src[i] for i in range(9))
                       for k, r in enumerate(rate)]
                norm = (M * M).sum(1)
                df = [sum(M[k, i] / norm[k] * mom[k] for k in range(9)) for i in range(9)]
            for i in range(q):
                fs[c, i] = (f[c, i] + df[i]) * fluid
    return (pull().sum(1) * fluid).reshape((2,) + shape)


def _conv(x, w, b):
    n, h, wd, ci = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b.expand(n * h * wd, -1) if b is not None else 0
    for ky in range(3):
        for kx in range(3):
            y = y + xp[:, ky:ky + h, kx:kx + wd].reshape(-1, ci) @ w[:, ky, kx].T.contiguous()
    return y.reshape(n, h, wd, -1)


def _up(x, w, b):
    n, h, wd, ci = x.shape
    co = w.shape[0]
    y = x.reshape(-1, ci) @ w.reshape(co * 4, ci).T.contiguous()
    y = y.reshape(n, h, wd, co, 2, 2).permute(0, 1, 4, 2, 5, 3).reshape(n, 2 * h, 2 * wd, co)
    return y + b


def _logits(p, x):
    skips, top = [], len(LEVELS) - 1
    for k in range(len(LEVELS)):
        x = _conv(x, p[f"enc{k}a.w"], p[f"enc{k}a.b"]).relu()
        x = _conv(x, p[f"enc{k}b.w"], p[f"enc{k}b.b"]).relu()
        if k < top:
            skips.append(x)
            x = torch.nn.functional.max_pool2d(x.permute(0, 3, 1, 2), 2).permute(0, 2, 3, 1)
    for k in range(top - 1, -1, -1):
        x = torch.cat([skips[k], _up(x, p[f"up{k}.w"], p[f"up{k}.b"])], 3)
        x = _conv(x, p[f"dec{k}a.w"], p[f"dec{k}a.b"]).relu()
        x = _conv(x, p[f"dec{k}b.w"], p[f"dec{k}b.b"]).relu()
    return x @ p["head.w"] + p["head.b"]


def _flat(d, names):
    """Tensors one after another, each on a 64-element boundary."""
    out = []
    for k in names:
        a = d[k].reshape(-1)
        out += [a, a.new_zeros(-a.numel() % 64)]
    return torch.cat(out)


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    kind = case["kind"]
    if kind in SOLVER:
        steps = case["steps"] * case["reps"]
        return {"density": [_exact_density(p, steps, dev) for p in _problems(case, seed)], "record": None}
    if kind == "conv":
        x, wt, b, dy = (a.to(dev).double() for a in _layer(case, seed))
        y = _conv(x, wt, b).relu()
        g = dy * (y > 0)
        xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        n, h, w, ci, co = (case[k] for k in ("n", "h", "w", "cin", "cout"))
        gt = g.reshape(-1, co).T.contiguous()
        dw = torch.stack([gt @ xp[:, ky:ky + h, kx:kx + w].reshape(-1, ci) for ky in range(3) for kx in range(3)], 1)
        dx = _conv(g, wt.flip(1, 2).permute(3, 1, 2, 0).contiguous(), None)
        return {"y": y, "dx": dx, "dw": dw.reshape(co, 3, 3, ci), "db": g.sum((0, 1, 2))}
    p = {k: torch.from_numpy(np.asarray(v, np.float64)).to(dev) for k, v in _params(case, seed).items()}
    x, t, m = (a.to(dev) for a in _fields(case, seed))
    if kind == "infer":
        return torch.cat([torch.sigmoid(_logits(p, x[i:i + 1].double())) for i in range(case["n"])])
    for v in p.values():
        v.requires_grad_(True)
    count, loss, sat = int(m.sum()), 0.0, []
    for i in range(case["n"]):  # image by image, gradients summed
        z = _logits(p, x[i:i + 1].double())
        l = ((torch.nn.functional.softplus(z) - t[i:i + 1] * z) * m[i:i + 1]).sum() / count
        l.backward()
        loss += float(l.detach())
        sat.append(torch.sigmoid(z.detach()))
    names = [n + s for n, *_ in _specs() for s in (".w", ".b")] + ["head.w", "head.b"]
    g = _flat({k: p[k].grad for k in names}, names)
    old = _flat({k: p[k].detach() for k in names}, names)
    return {"loss": torch.tensor([loss], dtype=torch.float64), "grad": g,
            "params": old - 1e-4 * g / (g.abs() + 1e-8), "sat": torch.cat(sat)}
