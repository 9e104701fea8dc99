"""Performance cases: the work a user of the simulator has it do, each through
the public entry points of the package.

Six kinds of work, over the range of sizes that the benchmark, the training
driver and the tests use:

  frames  sg_simulate: frames of a list of environments, described anew on
          every call (a tool that shows one pose; a script that renders a set)
  batch   a plan stepped in a simulation loop: new poses, one step
  recon   one episode of the bone-surface task: poses, step, surface update
          per step, then the voxel observation
  infer   audited surrogate inference of one frame per environment
  train   a few surrogate training steps (targets rendered on the way) without
          waiting for each, then the losses and the gradient
  conv    one conv layer: forward, data gradient and weight gradient

The phantoms are painted on the GPU: blocks with ellipsoids of fat and bone,
and a body with a fat layer and a chain of vertebra-like ellipsoids.  exact()
computes the same outputs with plain torch in 64 bits.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2507_01152_amd import sonosim as sg
from paper_2507_01152_amd.session import Session

DEV = "cuda"
M64 = (1 << 64) - 1

# per label (air, soft tissue, fat, bone): Z [MRayl], alpha [Np/cm/MHz], mu0, sigma0, mu1
TABLE = np.array([[0.0, 0.0, 0.0, 0.0, -np.inf], [1.63, 0.062, 0.05, 0.02, 0.0], [1.38, 0.055, 0.03, 0.015, -0.5],
                  [7.8, 2.3, 0.08, 0.03, 0.5]], dtype=np.float32)
HU_MEAN = (-1000.0, 40.0, -100.0, 700.0)

# fields of a case of the first five kinds, with their usual values
BASE = dict(envs=1, w=128, w_to=0, h=256, h_to=0, pixel_mm=0.5, planes=1, phantom="spine", volumes=1, edge=256,
            edge_to=0, ct=False, scales=1, tuned=False, steps=1)


def _case(name, kind, **over):
    c = dict(BASE, kind=kind, **over)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one small frame of one block phantom, nothing planned (interactive use, smoke test)
        _case("one frame", "frames", w=64, h=128, phantom="ellipsoid", edge=64),
        # one call that renders 64 poses on one patient's CT (impedance from HU)
        _case("CT frames", "frames", envs=64, ct=True),
        # the benchmark's step: 256 environments on 8 volumes of uneven size, images of uneven size
        _case("uneven batch", "batch", envs=256, volumes=8, edge=160, edge_to=256, w=64, w_to=256, h=128, h_to=512,
              tuned=True),
        # the same with three scales of speckle noise
        _case("uneven batch, 3 scales", "batch", envs=256, volumes=8, edge=160, edge_to=256, w=64, w_to=256, h=128,
              h_to=512, scales=3, tuned=True),
        # the surgery task's probe: 50 x 37 x 5 volumes at 2 x 2 x 10 mm
        _case("volumetric probe", "batch", envs=256, volumes=8, edge=160, edge_to=256, w=37, h=50, pixel_mm=2.0,
              planes=5, tuned=True),
        # an episode of the bone-surface task with 100 environments at the paper's image size, as the plan comes
        _case("bone surface episode", "recon", envs=100, volumes=4, edge=192, edge_to=256, w=150, h=200, steps=4),
        # serving: 1024 environments, 1/16 of them audited
        _case("inference, 1024 envs", "infer", envs=1024, pixel_mm=0.25, phantom="ellipsoid", volumes=32, edge=64),
        # the learned simulator in an RL loop of 128 environments, CT input
        _case("CT inference, 128 envs", "infer", envs=128, volumes=2, ct=True),
        # the training driver's batch
        _case("training, 64 pairs", "train", envs=64, pixel_mm=0.25, phantom="ellipsoid", volumes=32, edge=64, steps=3),
        # training with the adversarial term on CT input
        _case("CT training, 32 pairs", "train", envs=32, volumes=2, ct=True, steps=3),
        # a decoder layer by itself: 128 channels read upsampled to 64, as in a training step of 64 pairs
        dict(name="decoder layer", kind="conv", n=64, h=32, w=16, c=128, co=64, k=3, stride=1, up=1),
        # a layer of odd sizes and channel counts
        dict(name="odd layer", kind="conv", n=5, h=53, w=37, c=40, co=72, k=3, stride=1, up=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frames", "frames", "batch", "batch", "recon", "infer", "train", "conv", "conv"])
    if kind == "conv":
        k, stride = rng.choice([(3, 1), (3, 1), (3, 2), (1, 1)])
        up = rng.choice([0, 1]) if (k, stride) == (3, 1) else 0
        c, co = (8 * rng.choice([1, 2, 3, 4, 5, 8, 12, 16, 32]) for _ in range(2))
        h, w = rng.randint(7, 128), rng.randint(7, 128)
        most = max(1, min(64, int(6e7 // (h * w * (4 if up else 1) * max(c, co)))))
        return dict(kind=kind, n=_log(rng, 1, most), h=h, w=w, c=c, co=co, k=k, stride=stride, up=up)
    phantom = rng.choice(["spine", "ellipsoid"])
    ct = phantom == "spine" and rng.random() < 0.4
    over = dict(phantom=phantom, ct=ct, edge=64 if phantom == "ellipsoid" else rng.randint(150, 256),
                pixel_mm=0.25 if phantom == "ellipsoid" else 0.5, volumes=rng.randint(1, 4))
    if kind in ("infer", "train"):
        over.update(w=16 * rng.randint(4, 16), h=16 * rng.randint(4, 20))
        if kind == "infer":
            over["envs"] = _log(rng, 4, max(4, min(1024, 20000000 // (over["w"] * over["h"]))))
        else:
            over.update(envs=_log(rng, 2, max(2, min(64, 1500000 // (over["w"] * over["h"])))), steps=rng.randint(2, 3))
        return _case(None, kind, **over)
    over["scales"] = rng.choice([1, 1, 1, 2, 3])
    if kind == "batch" and rng.random() < 0.2:
        over.update(envs=_log(rng, 8, 256), w=rng.randint(20, 50), h=rng.randint(30, 70), pixel_mm=2.0,
                    planes=rng.randint(2, 6))
    else:
        over.update(envs=_log(rng, 1, 64 if kind == "frames" else 256), w=rng.randint(32, 200), h=rng.randint(64, 400))
        if kind == "batch":
            over.update(w_to=min(256, over["w"] + rng.randint(0, 100)), h_to=min(512, over["h"] + rng.randint(0, 200)))
    over["tuned"] = kind == "batch" and rng.random() < 0.5
    if kind == "recon":
        over["steps"] = rng.randint(2, 6)
    return _case(None, kind, **over)


# ---------------------------------------------------------------------------
# inputs

def _rotations(q):
    """Rotation matrices [n, 3, 3] of quaternions [n, 4]."""
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    return np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                     1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                     1 - 2 * (x * x + y * y)], axis=1).reshape(-1, 3, 3)


def _axis_quat(axis, ang):
    q = np.zeros((len(ang), 4))
    q[:, 0], q[:, 1 + axis] = np.cos(ang / 2), np.sin(ang / 2)
    return q


def _paint(lab, centre, semi, R, value):
    """Label `value` inside the rotated ellipsoid (x, y, z in voxels)."""
    lo = [max(0, int(math.floor(c - max(semi) - 1))) for c in centre]
    hi = [min(n, int(math.ceil(c + max(semi) + 1)) + 1) for c, n in zip(centre, lab.shape[::-1])]
    if any(b <= a for a, b in zip(lo, hi)):
        return
    z, y, x = torch.meshgrid(*[torch.arange(lo[i], hi[i], device=DEV, dtype=torch.float32) for i in (2, 1, 0)],
                             indexing="ij")
    d = [x - centre[0], y - centre[1], z - centre[2]]
    q = sum(((d[0] * float(R[0, j]) + d[1] * float(R[1, j]) + d[2] * float(R[2, j])) / semi[j]) ** 2 for j in range(3))
    sub = lab[lo[2]:hi[2], lo[1]:hi[1], lo[0]:hi[0]]
    sub.masked_fill_(q <= 1.0, value)


def _volume(case, v, rng):
    """(labels uint8 [nz][ny][nx] on the GPU, body (centre x, centre z, semi-axes) or None)."""
    if case["phantom"] == "ellipsoid":
        n = case["edge"]
        lab = torch.ones((n, n, n), dtype=torch.uint8, device=DEV)
        for _ in range(6):
            _paint(lab, rng.uniform(0.19 * n, 0.81 * n, 3), rng.uniform(0.05 * n, 0.19 * n, 3),
                   _rotations(rng.normal(size=(1, 4)))[0], int(rng.integers(2, 4)))
        return lab, None
    lo, to = case["edge"], case["edge_to"] or case["edge"]
    f = v / max(1, case["volumes"] - 1)
    top = (1.25 * to, to, 1.5 * to) if case["edge_to"] else (to, to, to)
    nx, ny, nz = (int(round(lo + (t - lo) * f)) for t in top)
    cx, cz, ax, az = nx / 2.0, nz / 2.0, 0.43 * nx, 0.31 * nz
    x = torch.arange(nx, device=DEV, dtype=torch.float32)[None, :] - cx
    z = torch.arange(nz, device=DEV, dtype=torch.float32)[:, None] - cz
    outer, inner = (x / ax) ** 2 + (z / az) ** 2, (x / (ax - 10.0)) ** 2 + (z / (az - 10.0)) ** 2
    sl = torch.zeros((nz, nx), dtype=torch.uint8, device=DEV)
    sl[outer <= 1.0] = 1
    sl[(outer <= 1.0) & (inner > 1.0) & (z > 0)] = 2
    lab = sl[:, None, :].expand(nz, ny, nx).contiguous()
    for i in range(5):
        R = _rotations(_axis_quat(0, rng.uniform(-0.2, 0.2, 1)))[0]
        _paint(lab, (cx + rng.uniform(-3, 3), ny / 2 + (i - 2) * 35.0 * ny / 256 + rng.uniform(-3, 3),
                     cz + az - 60.0 + rng.uniform(-3, 3)), rng.uniform(0.9, 1.1, 3) * (20.0, 12.0, 15.0), R, 3)
    return lab, (cx, cz, ax, az)


def _inputs(case, seed):
    """Volumes, probes and poses of a case, from the seed alone."""
    rng = np.random.default_rng((int(seed), 77))
    gen = torch.Generator(device=DEV).manual_seed(int(seed) + 13)
    vols, bodies = [], []
    for v in range(case["volumes"]):
        lab, body = _volume(case, v, rng)
        ct = None
        if case["ct"]:
            mean = torch.tensor(HU_MEAN, device=DEV)[lab.long()]
            ct = (mean + 30.0 * torch.randn(lab.shape, device=DEV, generator=gen)).round_().clamp_(-1024, 3071).short()
        vols.append(SimpleNamespace(labels=lab, ct=ct, seed=int(rng.integers(0, 1 << 62)), scales=case["scales"]))
        bodies.append(body)
    n = case["envs"]
    vid = np.arange(n) % case["volumes"]
    # the image sizes belong to the case: a plan's probes stay as its volumes and poses change
    sizes = np.random.default_rng((n, case["w"], case["w_to"], case["h"], case["h_to"]))
    W = sizes.integers(case["w"], max(case["w"], case["w_to"]) + 1, n)
    H = sizes.integers(case["h"], max(case["h"], case["h_to"]) + 1, n)
    p = case["pixel_mm"]
    probes = [SimpleNamespace(W=int(a), H=int(b), dx=p, dy=p, f=5.0, E0=1.0, psf=0.01, dr=60.0,
                              n_elev=case["planes"], elev=10.0 if case["planes"] > 1 else 0.0) for a, b in zip(W, H)]

    def poses():
        """Probe on the back skin, beam into the body, or anywhere in a block phantom."""
        P = np.zeros((n, 3, 4))
        if case["phantom"] == "ellipsoid":
            P[:, :, :3] = _rotations(rng.normal(size=(n, 4)))
            P[:, :, 3] = rng.uniform(0.25, 0.75, (n, 3)) * case["edge"]
        else:
            cx, cz, ax, az = (np.array([bodies[v][i] for v in vid]) for i in range(4))
            x0 = cx + rng.uniform(-30, 30, n)
            R = np.diag([1.0, -1.0, -1.0]) @ _rotations(_axis_quat(2, rng.uniform(0, 2 * math.pi, n)))
            for axis in (0, 1):
                R = R @ _rotations(_axis_quat(axis, rng.uniform(-0.35, 0.35, n)))
            P[:, :, :3] = R
            P[:, 0, 3] = x0
            P[:, 1, 3] = np.array([vols[v].labels.shape[1] for v in vid]) / 2 + rng.uniform(-30, 30, n)
            P[:, 2, 3] = cz + az * np.sqrt(1 - np.clip((x0 - cx) / ax, -1, 1) ** 2) - 3.0
        return P.reshape(n, 12)

    size = np.array([q.W * q.H * case["planes"] for q in probes], dtype=np.int64)
    return SimpleNamespace(vols=vols, vid=vid, probes=probes, offs=np.concatenate([[0], np.cumsum(size)[:-1]]),
                           total=int(size.sum()), poses=[poses() for _ in range(case["steps"])], rng=rng, draw=poses)


def _params(rng, layers, extra):
    """He-normal conv weights with zero biases, then the extra tensors, as one vector."""
    parts = []
    for ci, co in layers:
        parts += [rng.normal(0, math.sqrt(2 / (9 * ci)), co * 9 * ci), np.zeros(co)]
    return np.concatenate(parts + extra).astype(np.float32)


# 3x3 convs of the network: name, input, skip, input channels, output channels, stride, upsampled input
NET = [("T1", "X", "", 8, 16, 1, 0), ("E0", "T1", "", 16, 16, 1, 0), ("T2", "E0", "", 16, 32, 2, 0),
       ("E1", "T2", "", 32, 32, 1, 0), ("T3", "E1", "", 32, 64, 2, 0), ("E2", "T3", "", 64, 64, 1, 0),
       ("T4", "E2", "", 64, 128, 2, 0), ("E3", "T4", "", 128, 128, 1, 0), ("T5", "E3", "", 128, 256, 2, 0),
       ("B4", "T5", "", 256, 256, 1, 0), ("U3", "B4", "E3", 256, 128, 1, 1), ("D3", "U3", "", 128, 128, 1, 0),
       ("U2", "D3", "E2", 128, 64, 1, 1), ("D2", "U2", "", 64, 64, 1, 0), ("U1", "D2", "E1", 64, 32, 1, 1),
       ("D1", "U1", "", 32, 32, 1, 0), ("U0", "D1", "E0", 32, 16, 1, 1), ("D0", "U0", "", 24, 16, 1, 0)]
DISC = [(8, 32, 2), (32, 64, 2), (64, 128, 2), (128, 128, 1), (128, 8, 1)]
ADV, LR = 0.01, 1e-5   # weight of the adversarial term; learning rate late in the schedule


def _net_params(rng):
    # a head small enough for frames inside [0, 1], as a trained one gives them
    return _params(rng, [(l[3], l[4]) for l in NET],
                   [rng.normal(0, 0.25, 128), np.zeros(8), rng.normal(0, 0.02, 16), [0.4]])


def _disc_params(rng):
    p = _params(rng, [d[:2] for d in DISC], [])
    p[-8 * 9 * 128 - 8 + 9 * 128:] = 0.0   # the last conv's channels after the first stay zero
    return p


class State:
    """What a user's program keeps between calls; closes its session when it goes."""

    def __init__(self, case):
        self.case, self.sess = case, Session(0)
        self.ctx = self.sess.ctx

    def __del__(self):
        self.sess.close()


def _conv_desc(case):
    return sg.conv_desc(case["n"], case["h"], case["w"], case["c"], case["co"], case["k"], case["stride"], case["k"] // 2,
                        case["up"])


def _conv_out(case):
    u = 2 if case["up"] else 1
    return tuple((u * case[d] - 1) // case["stride"] + 1 for d in ("h", "w"))


def _conv_inputs(case, seed):
    g = torch.Generator(device=DEV).manual_seed(int(seed) + 29)
    n, c, co, k = case["n"], case["c"], case["co"], case["k"]
    ho, wo = _conv_out(case)

    def rnd(*shape):
        return torch.randn(shape, device=DEV, generator=g)

    return SimpleNamespace(x=rnd(n, case["h"], case["w"], c).relu_().bfloat16(), bias=0.1 * rnd(co),
                           wt=(rnd(co, k, k, c) * math.sqrt(2 / (k * k * c))).bfloat16(),
                           dy=(rnd(n, ho, wo, co) * 1e-3).bfloat16())


def prepare(case, seed):
    s = State(case)
    if case["kind"] == "conv":
        i = s.i = _conv_inputs(case, seed)
        s.desc = _conv_desc(case)
        s.y = torch.empty_like(i.dy)
        s.dx, s.dw = torch.empty(i.x.shape, device=DEV), torch.empty(i.wt.shape, device=DEV)
        s.db = torch.empty(case["co"], device=DEV)
        return s
    i = s.i = _inputs(case, seed)
    ids = [sg.sg_volume_register(s.ctx, v.labels, (1.0, 1.0, 1.0), v.ct, v.seed, v.scales) for v in i.vols]
    s.vids = np.array([ids[v] for v in i.vid], dtype=np.int32)
    sg.sg_tissue_table_set(s.ctx, TABLE)
    s.probes = sg.probes_array(i.probes)
    if case["kind"] in ("frames", "batch", "recon"):
        s.out = torch.empty(i.total, dtype=torch.float32, device=DEV)
    if case["kind"] in ("batch", "recon"):
        s.plan = sg.sg_batch_plan_create(s.ctx, s.vids, s.probes, i.offs)
        sg.sg_batch_set_poses(s.ctx, s.plan, i.poses[0])
        if case["tuned"]:
            sg.sg_autotune(s.ctx, s.plan, None)
    if case["kind"] == "recon":
        s.recon = sg.sg_recon_create(s.ctx, s.plan, 4096, seed=int(seed) & M64)
        s.grids = torch.empty(case["envs"] * 40 ** 3, dtype=torch.uint8, device=DEV)
    if case["kind"] in ("infer", "train"):
        train = case["kind"] == "train"
        i.params = _net_params(i.rng)
        if case["ct"]:
            s.sid = sg.sg_surr_create_ct(s.ctx, case["h"], case["w"], 1, ADV if train else 0.0)
            sg.sg_surr_set_ct_reference(s.ctx, s.sid, s.vids, s.probes, i.draw())
        else:
            s.sid = sg.sg_surr_create(s.ctx, case["h"], case["w"], 1)
        sg.sg_surr_set_params(s.ctx, s.sid, i.params)
        if case["ct"] and train:
            sg.sg_surr_disc_set_params(s.ctx, s.sid, _disc_params(i.rng))
        if not train:
            s.out = torch.empty(i.total, dtype=torch.bfloat16, device=DEV)
            s.audit = np.arange(0, case["envs"], 16, dtype=np.int32)
    return s


def run(s):
    case, i, ctx = s.case, s.i, s.ctx
    if case["kind"] == "frames":
        sg.sg_simulate(ctx, s.vids, s.probes, i.poses[0], s.out, i.offs)
        return s.out
    if case["kind"] == "batch":
        sg.sg_batch_set_poses(ctx, s.plan, i.poses[0])
        sg.sg_batch_step(ctx, s.plan, s.out)
        return s.out
    if case["kind"] == "recon":
        sg.sg_recon_reset(ctx, s.recon)
        for k in range(case["steps"]):
            sg.sg_batch_set_poses(ctx, s.plan, i.poses[k])
            sg.sg_batch_step(ctx, s.plan, s.out)
            sg.sg_recon_update(ctx, s.recon, k)
        sg.sg_recon_observe(ctx, s.recon, s.grids)
        return {"frames": s.out, "grids": s.grids}
    if case["kind"] == "infer":
        psnr, _ = sg.sg_surr_infer_bf16(ctx, s.sid, s.vids, s.probes, i.poses[0], s.out, s.audit, -np.inf, 1.0)
        return {"frames": s.out, "psnr": psnr}
    if case["kind"] == "train":
        first = sg.sg_surr_step_count(ctx, s.sid) + 1
        for k in range(case["steps"]):
            sg.sg_surr_train_step_async(ctx, s.sid, s.vids, s.probes, i.poses[k], LR)
        return {"losses": sg.sg_surr_loss_history(ctx, s.sid, first, case["steps"]),
                "grad": sg.sg_surr_get_grads(ctx, s.sid)}
    sg.sg_conv_forward(ctx, s.desc, i.x, i.wt, i.bias, True, y=s.y)
    sg.sg_conv_backward_data(ctx, s.desc, i.dy, i.wt, s.dx)
    sg.sg_conv_backward_weight(ctx, s.desc, i.x, i.dy, s.dw, s.db if case["co"] <= 256 else None)
    return {"y": s.y, "dx": s.dx, "dw": s.dw, "db": s.db if case["co"] <= 256 else None}


def _pixel_flops(H, W, case):
    """Arithmetic of one physics pixel: position 12, noise 10 rounds of 8 and Box-Muller 12 per scale,
    interface and energy 20, separable PSF of two fields, composition and display 8, CT 40."""
    ra, rl = (max(1, math.ceil(0.03 * v)) for v in (H, W))
    return 40 + 92 * case["scales"] + 4 * (2 * ra + 1 + 2 * rl + 1) + (40 if case["ct"] else 0)


def work(case):
    if case["kind"] == "conv":
        ho, wo = _conv_out(case)
        x = case["n"] * case["h"] * case["w"] * case["c"]
        y = case["n"] * ho * wo * case["co"]
        wts = case["co"] * case["k"] ** 2 * case["c"]
        # x, weights, dy once; y, dx (FP32), dw (FP32) once
        return {"bytes": 2.0 * (x + wts + y) + 2.0 * y + 4.0 * x + 4.0 * wts, "flops": 6.0 * y * case["k"] ** 2 * case["c"]}
    W, H = ((case[d] + max(case[d], case[d + "_to"])) / 2 for d in ("w", "h"))
    px = case["envs"] * case["planes"] * W * H
    image = px * (3 if case["ct"] else 1)              # label (and HU) of each pixel
    phys = px * _pixel_flops(H, W, case)
    if case["kind"] in ("frames", "batch"):
        return {"bytes": image + 4.0 * px, "flops": phys}
    if case["kind"] == "recon":
        return {"bytes": case["steps"] * (image + 4.0 * px) + 64000.0 * case["envs"], "flops": case["steps"] * phys}
    level = {"X": 0}
    flops = 300.0 * px
    for name, src, _, ci, co, stride, up in NET:
        level[name] = level[src] + (stride == 2) - up
        flops += 18.0 * ci * co * px / 4 ** level[name]
    if case["kind"] == "infer":
        return {"bytes": image + 2.0 * px, "flops": flops + 92.0 * px + phys / 16}
    if case["ct"]:
        flops += 2 * sum(18.0 * ci * co * px / 4 ** (k + 1 if k < 3 else 3) for k, (ci, co, _) in enumerate(DISC))
    # per step: the image, the target, weights and moments read and written, the gradient; the activations
    # that the backward needs again are not counted
    return {"bytes": case["steps"] * (image + 1768793 * 28.0), "flops": case["steps"] * (3 * flops + 92.0 * px + phys)}


# ---------------------------------------------------------------------------
# the same in 64 bits, with plain torch

def _philox(c0, c2, key):
    """Philox4x32-10 of the counters (c0, 0, c2, 0): four words as int64 tensors."""
    m = 0xFFFFFFFF
    k0, k1 = key & m, key >> 32
    c = [c0, torch.zeros_like(c0), torch.full_like(c0, c2), torch.zeros_like(c0)]
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57   # modulo 2^64
        c = [((p1 >> 32) & m) ^ c[1] ^ k0, p1 & m, ((p0 >> 32) & m) ^ c[3] ^ k1, p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c


def _normal(w0, w1):
    u0, u1 = ((2.0 * (w >> 9).double() + 1.0) * 2.0 ** -24 for w in (w0, w1))
    return torch.sqrt(-2.0 * torch.log(u0)) * torch.cos(2.0 * math.pi * u1)


def _quantiles():
    p = (torch.arange(4096, dtype=torch.float64) + 0.5) / 4096
    return torch.round(torch.special.ndtri(p) * 2 ** 20).long().to(DEV)


class Slice:
    """Positions, labels and noise of one image plane."""

    def __init__(self, vol, probe, pose, plane):
        self.vol, self.probe = vol, probe
        pose = pose.reshape(3, 4)
        nz, ny, nx = vol.labels.shape
        self.dims = (nx, ny, nz)
        b = 0.0 if probe.n_elev <= 1 else (plane - 0.5 * (probe.n_elev - 1)) * probe.elev
        self.P0, self.DX, self.DY = [], [], []
        for c in range(3):
            u = pose[c, 3] + pose[c, 0] * (-0.5 * (probe.W - 1) * probe.dx)
            self.P0.append(int(np.rint((u + pose[c, 1] * b) * 65536.0)))
            self.DX.append(int(np.rint(pose[c, 0] * probe.dx * 65536.0)))
            self.DY.append(int(np.rint(pose[c, 2] * probe.dy * 65536.0)))
        x, y = torch.arange(probe.W, device=DEV)[None, :], torch.arange(probe.H, device=DEV)[:, None]
        self.Q = [p + x * dx + y * dy for p, dx, dy in zip(self.P0, self.DX, self.DY)]
        self.I = [(q + 32768) >> 16 for q in self.Q]
        self.inside = self._in(self.I)
        self.vox = torch.where(self.inside, (self.I[2] * ny + self.I[1]) * nx + self.I[0], 0)
        self.lab = torch.where(self.inside, vol.labels.reshape(-1)[self.vox], 0).long()

    def _in(self, I):
        ok = torch.ones_like(I[0], dtype=torch.bool)
        for i, n in zip(I, self.dims):
            ok &= (i >= 0) & (i < n)
        return ok

    def hu(self, I):
        ok = self._in(I)
        at = torch.where(ok, (I[2] * self.dims[1] + I[1]) * self.dims[0] + I[0], 0)
        return torch.where(ok, self.vol.ct.reshape(-1)[at].double(), -1000.0)

    def impedance(self):
        if self.vol.ct is None:
            return torch.tensor(TABLE[:, 0], device=DEV).double()[self.lab]
        base, w = [q >> 16 for q in self.Q], [(q & 0xFFFF).double() / 65536 for q in self.Q]
        v = [[[self.hu([base[0] + i, base[1] + j, base[2] + k]) for i in (0, 1)] for j in (0, 1)] for k in (0, 1)]
        v = [[a[0] + w[0] * (a[1] - a[0]) for a in b] for b in v]
        v = [b[0] + w[1] * (b[1] - b[0]) for b in v]
        return (v[0] + w[2] * (v[1] - v[0]) + 1000.0).clamp_min(0.0)

    def scatterer(self):
        """(N0, gate) of every pixel; the gate is false outside the volume."""
        S = self.vol.scales
        w = _philox(self.vox, 0, self.vol.seed)
        mu1 = [float(m) for m in TABLE[:, 4]]
        if S <= 1:
            thr = [int(math.floor(0.5 * math.erfc(-m / math.sqrt(2.0)) * 2.0 ** 32)) for m in mu1]
            return _normal(w[0], w[1]), self.inside & (w[2] < torch.tensor(thr, device=DEV)[self.lab])
        q = _quantiles()
        n0, n1 = _normal(w[0], w[1]), q[w[2] >> 20]
        for s in range(1, S):
            mx, my = ((self.dims[c] + (1 << s) - 1) >> s for c in (0, 1))
            I = [torch.where(self.inside, i, 0) >> s for i in self.I]
            w = _philox((I[2] * my + I[1]) * mx + I[0], s, self.vol.seed)
            n0, n1 = n0 + _normal(w[0], w[1]), n1 + q[w[2] >> 20]
        thr = [-(1 << 31) if m == -math.inf else int(math.floor(math.sqrt(S) * m * 2 ** 20)) for m in mu1]
        return n0 / math.sqrt(S), self.inside & (n1 <= torch.tensor(thr, device=DEV)[self.lab])


def _psf(f, size, axis, frac):
    """f filtered along an axis with the sampled Gaussian of `frac` of the size, zeros outside."""
    sigma = frac * size
    r = max(1, math.ceil(3.0 * sigma))
    k = [math.exp(-i * i / (2 * sigma * sigma)) for i in range(-r, r + 1)]
    pad = torch.nn.functional.pad(f, (0, 0, r, r) if axis == 0 else (r, r))
    return sum(k[i] / sum(k) * pad.narrow(axis, i, f.shape[axis]) for i in range(2 * r + 1))


def _frame(vol, probe, pose, plane):
    """Display frame [H][W] of one image plane."""
    s = Slice(vol, probe, pose, plane)
    lab, (H, W) = s.lab, s.lab.shape
    Z = s.impedance()
    Z1 = torch.cat([Z[1:], Z[-1:]])
    G = torch.cat([lab[1:] != lab[:-1], torch.zeros((1, W), dtype=torch.bool, device=DEV)]) if H > 1 else lab < 0
    live, total = G & (Z != Z1), (Z == 0) | (Z1 == 0)
    sm = torch.where(Z + Z1 > 0, Z + Z1, 1.0)
    r = torch.where(live, torch.where(total, 1.0, ((Z1 - Z) / sm).abs()), 0.0)
    t = torch.where(live, torch.where(total, 0.0, (2 * Z / sm) * (2 * Z1 / sm)), 1.0)
    alpha = torch.tensor(TABLE[:, 1], device=DEV).double()[lab]
    one = torch.ones((1, W), dtype=torch.float64, device=DEV)
    E = probe.E0 * torch.cat([one, torch.cumprod(t, 0)[:-1]]) * torch.exp(
        -probe.f * probe.dy / 10 * torch.cat([0 * one, torch.cumsum(alpha, 0)[:-1]]))
    y, x = (torch.arange(-1, n + 1, device=DEV).clamp(0, n - 1) for n in (H, W))
    pad = lab[y][:, x]
    b = {(j, i): (pad[1 + j:1 + j + H, 1 + i:1 + i + W] != lab).double() for j in (-1, 0, 1) for i in (-1, 0, 1)}
    gx = ((b[-1, 1] - b[-1, -1]) + 2 * (b[0, 1] - b[0, -1]) + (b[1, 1] - b[1, -1])) / probe.dx
    gy = ((b[1, -1] - b[-1, -1]) + 2 * (b[1, 0] - b[-1, 0]) + (b[1, 1] - b[-1, 1])) / probe.dy
    h = torch.sqrt(gx * gx + gy * gy)
    cos = torch.where(h == 0, 1.0, gy.abs() / torch.where(h == 0, 1.0, h))
    n0, gate = s.scatterer()
    mu, sd = (torch.tensor(TABLE[:, c], device=DEV).double()[lab] for c in (2, 3))
    T = torch.where(gate, n0 * sd + mu, 0.0)
    R, T = (_psf(_psf(f, H, 0, probe.psf), W, 1, probe.psf) for f in (torch.where(G, E * cos * r, 0.0), T))
    I = (R + E * T).clamp_min(0.0) / probe.E0
    return torch.where(I > 0, 1 + 20 / probe.dr * torch.log10(torch.where(I > 0, I, 1.0)), 0.0).clamp(0, 1)


def _frames(i, poses):
    return torch.cat([_frame(i.vols[v], p, q, j).reshape(-1) for v, p, q in zip(i.vid, i.probes, poses)
                      for j in range(p.n_elev)])


def _bf16(x):
    return x.float().bfloat16().double()


def _histogram(s):
    return torch.bincount((torch.where(s.inside, s.hu(s.I), -1000.0).long() + 1024).clamp(0, 4095).reshape(-1), minlength=4096)


def _encode(i, poses, ref):
    """The network's input [n][H][W][8], rounded to bf16 as it is stored."""
    out = []
    q = _quantiles()
    for v, p, pose in zip(i.vid, i.probes, poses):
        s = Slice(i.vols[v], p, pose, 0)
        depth = ((torch.arange(p.H, device=DEV).double()[:, None] + 0.5) / p.H).expand(p.H, p.W)
        zero = torch.zeros_like(depth)
        if ref is None:
            n0, gate = s.scatterer()
            ch = [(s.lab == k).double() for k in range(4)] + [torch.where(gate, n0, 0.0), depth, zero, zero]
        else:
            hist = _histogram(s)
            lut = torch.searchsorted(ref.cumsum(0) * hist.sum(), hist.cumsum(0) * ref.sum())
            bins = (torch.where(s.inside, s.hu(s.I), -1000.0).long() + 1024).clamp(0, 4095)
            w = _philox(s.vox, 0, s.vol.seed)
            ch = [(lut[bins] - 1024).double() / 1000, torch.where(s.inside, _normal(w[0], w[1]), 0.0),
                  torch.where(s.inside, q[w[2] >> 20].double() * 2.0 ** -20, 0.0), depth] + [zero] * 4
        out.append(_bf16(torch.stack(ch, -1)))
    return torch.stack(out)


def _conv64(x, w, b, stride=1, up=0):
    """k x k conv (pad k // 2) of NHWC x with w [co][k][k][ci]."""
    if up:
        x = x.repeat_interleave(2, 1).repeat_interleave(2, 2)
    k = w.shape[1]
    n, h, wd, _ = x.shape
    ho, wo = (h - 1) // stride + 1, (wd - 1) // stride + 1
    x = torch.nn.functional.pad(x, (0, 0, k // 2, k // 2, k // 2, k // 2))
    acc = 0
    for r in range(k):
        for c in range(k):
            v = x[:, r:r + stride * (ho - 1) + 1:stride, c:c + stride * (wo - 1) + 1:stride]
            acc = acc + v.reshape(-1, v.shape[-1]) @ w[:, r, c].t()
    return (acc if b is None else acc + b).reshape(n, ho, wo, -1)


def _split(p, layers):
    """(weight [co][3][3][ci], bias) of each conv and what is left of the vector."""
    out, at = [], 0
    for ci, co in layers:
        n = co * 9 * ci
        out.append((p[at:at + n].reshape(co, 3, 3, ci), p[at + n:at + n + co]))
        at += n + co
    return out, p[at:]


def _held(w):
    return w + (_bf16(w.detach()) - w.detach())   # the bf16 copy that the convs read


def _net(p, x):
    """Network output [n][H][W]."""
    convs, rest = _split(p, [(l[3], l[4]) for l in NET])
    pw, pb, hw, hb = rest[:128].reshape(8, 16), rest[128:136], rest[136:152], rest[152]
    t = {"X": x}
    for (name, src, skip, _, _, stride, up), (w, b) in zip(NET, convs):
        y = torch.relu(_conv64(t[src], _held(w), b, stride, up))
        if skip:
            y = y + t[skip]
        if name == "U0":
            m = (t["E0"].reshape(-1, 16) @ _held(pw).t() + pb).reshape(*y.shape[:3], 8)
            y = torch.cat([y, (torch.cumsum(m, 1) - m) / 16], -1)
        t[name] = y
    return (t["D0"].reshape(-1, 16) @ _held(hw) + hb).reshape(x.shape[:3])


def _disc(p, x, image):
    convs, _ = _split(p, [d[:2] for d in DISC])
    z = torch.cat([x[..., :4], image[..., None], torch.zeros_like(x[..., :3])], -1)
    for k, ((_, _, stride), (w, b)) in enumerate(zip(DISC, convs)):
        z = _conv64(z, _held(w), b, stride)
        if k + 1 < len(DISC):
            z = torch.nn.functional.leaky_relu(z, 0.2)
    return z[..., 0]


class _Adam:
    def __init__(self, p):
        self.p, self.m, self.v, self.t = torch.tensor(p, device=DEV).double(), 0.0, 0.0, 0

    def step(self, g):
        self.t += 1
        self.m, self.v = 0.9 * self.m + 0.1 * g, 0.999 * self.v + 0.001 * g * g
        self.p = self.p - LR * (self.m / (1 - 0.9 ** self.t)) / (torch.sqrt(self.v / (1 - 0.999 ** self.t)) + 1e-8)


def _grad(p, parts):
    """Sum of the losses and of their gradients over functions of the parameters."""
    loss, g = 0.0, 0.0
    for f in parts:
        q = p.detach().requires_grad_(True)
        v = f(q)
        g = g + torch.autograd.grad(v, q)[0]
        loss += float(v)
    return loss, g


def _train64(case, i, ref, disc):
    net, dis = _Adam(i.params), _Adam(disc) if disc is not None else None
    sp, losses, grad = torch.nn.functional.softplus, [], None
    n, H, W = case["envs"], case["h"], case["w"]
    cells, patches = n * H * W, n * (H // 8) * (W // 8)
    for k in range(case["steps"]):
        X, Y = _encode(i, i.poses[k], ref), _frames(i, i.poses[k]).reshape(n, H, W)
        parts = [slice(a, min(n, a + 8)) for a in range(0, n, 8)]
        row = [0.0, 0.0, 0.0]
        if dis is not None:
            with torch.no_grad():
                fake = torch.cat([_net(net.p, X[c]) for c in parts])
            row[1], g = _grad(dis.p, [lambda q, c=c: (sp(-_disc(q, X[c], Y[c])).sum() + sp(_disc(q, X[c], fake[c])).sum())
                                      / (2 * patches) for c in parts])
            dis.step(g)

        def loss(q, c):
            out = _net(q, X[c])
            l1 = (out - Y[c]).abs().sum() / cells
            row[0] += float(l1)
            if dis is None:
                return l1
            adv = sp(-_disc(dis.p, X[c], out)).sum() / patches
            row[2] += float(adv)
            return l1 + ADV * adv

        _, grad = _grad(net.p, [lambda q, c=c: loss(q, c) for c in parts])
        net.step(grad)
        losses.append(row)
    return {"losses": torch.tensor(losses, dtype=torch.float64), "grad": grad}


def exact(case, seed):
    if case["kind"] == "conv":
        i = _conv_inputs(case, seed)
        x, w = i.x.double().requires_grad_(True), i.wt.double().requires_grad_(True)
        v = _conv64(x, w, None, case["stride"], case["up"])
        dx, dw = torch.autograd.grad(v, (x, w), i.dy.double())
        db = i.dy.double().sum((0, 1, 2)) if case["co"] <= 256 else None
        return {"y": torch.relu(v.detach() + i.bias.double()), "dx": dx, "dw": dw, "db": db}
    i = _inputs(case, seed)
    if case["kind"] in ("frames", "batch"):
        return _frames(i, i.poses[0])
    if case["kind"] == "recon":
        return {"frames": _frames(i, i.poses[-1]), "grids": None}
    i.params, ref, disc = _net_params(i.rng), None, None
    if case["ct"]:
        # the order of prepare(): parameters, reference poses, discriminator
        ref = sum(_histogram(Slice(i.vols[v], p, q, 0)) for v, p, q in zip(i.vid, i.probes, i.draw()))
        disc = _disc_params(i.rng) if case["kind"] == "train" else None
    if case["kind"] == "train":
        return _train64(case, i, ref, disc)
    p, out, psnr = torch.tensor(i.params, device=DEV).double(), [], []
    poses, n = i.poses[0], case["envs"]
    with torch.no_grad():
        for a in range(0, n, 32):
            part = SimpleNamespace(vols=i.vols, vid=i.vid[a:a + 32], probes=i.probes[a:a + 32])
            out.append(_net(p, _encode(part, poses[a:a + 32], ref)).clamp(0, 1))
        out = torch.cat(out)
        for e in range(0, n, 16):
            mse = (out[e] - _frame(i.vols[i.vid[e]], i.probes[e], poses[e], 0)).square().mean()
            psnr.append(-10 * math.log10(float(mse)))
    return {"frames": out.reshape(-1), "psnr": torch.tensor(psnr, dtype=torch.float64)}
