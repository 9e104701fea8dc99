#!/usr/bin/env python3
"""Benchmark: simulated B-mode frames/s at 256 batched environments.

Workload: 256 environments over 8 seeded label volumes of uneven size
(160^3 ... 320x256x384 uint8), per-env images of 64..256 scanlines x
128..512 depth samples at 0.5 mm, random probe poses on a spine phantom,
stepped by two persistent kernels per step.  Inputs
(volumes, poses) are resident in device memory before timing starts.

Prints one JSON line (see the keys below).  Only one GPU is used; --gpus
above 1 is refused.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0
# MI355X's FP32 vector peak (157.3 TFLOP/s, an FMA counted as 2 flops) is
# 256 CUs x 4 SIMDs x 32 lanes x 2.4 GHz non-packed 32-bit VALU lane-ops:
# 78.6 T lane-ops/s.  Two-operand encodings approach it, three-operand ones
# issue at about half of it and the 32x32->64 multiply-add at a quarter
# (weighted 4 below); the probe's measurements go into the roofline line.
PEAK_VALU_TOPS = 256 * 4 * 32 * 2.4e9 / 1e12


def psf_radius(size: int, frac: float = 0.01) -> int:
    return max(1, math.ceil(3.0 * frac * size))


def ray_ops_per_pixel(W: int, H: int) -> int:
    """Algorithmic 32-bit VALU lane-op count of one pixel in the ray kernel
    (quarter-rate ops -- 32-bit integer multiplies, transcendentals -- count 4)."""
    sample = 20          # Q16 position, rounding, bounds, voxel index, label gather
    interface = 4        # boundary indicator and reflection/transmission select
    scans = 18           # 6-step wave scans: FP32 product and sum
    energy = 10          # exp and products
    philox = 10 * 20     # 10 rounds: two 32x32->64 products (4 quarter-rate ops) + xors
    scatter = 22         # Box-Muller (log, sqrt, cos) + gate + amplitude
    axial = 2 * (2 * psf_radius(H) + 1)   # axial PSF FMAs, two fields
    return sample + interface + scans + energy + philox + scatter + axial


def psf_ops_per_pixel(W: int, H: int) -> int:
    """Same count for the PSF kernel: lateral FMAs of two fields + display."""
    return 2 * (2 * psf_radius(W) + 1) + 18


# surrogate network: (Ci, Co, level, stride) of each 3x3 conv (output level for
# the FLOP count) -- five levels 16/32/64/128/256, decoders read x2 upsampled
SURR_CONVS = [(8, 16, 0), (16, 16, 0), (16, 32, 1), (32, 32, 1), (32, 64, 2), (64, 64, 2), (64, 128, 3),
              (128, 128, 3), (128, 256, 4), (256, 256, 4), (256, 128, 3), (128, 128, 3), (128, 64, 2),
              (64, 64, 2), (64, 32, 1), (32, 32, 1), (32, 16, 0), (24, 16, 0)]


def surrogate_flops_per_frame(H: int, W: int) -> float:
    """Forward FLOPs (2 per multiply-add) of the convolutions, the 1x1 depth
    map (16 -> 8) with its running sum, and the head."""
    f = sum(2.0 * 9 * ci * co * (H >> lv) * (W >> lv) for ci, co, lv in SURR_CONVS)
    return f + (2.0 * 16 * 8 + 8) * H * W + 2.0 * 16 * H * W


# algorithmic HBM bytes of the inference forward: (channels, level) of every tensor read and written once
# per consumer in bf16 (2 B), plus the encoder's label gather (1 B/px) and the FP32 head output and clamp
SURR_FWD_TENSORS = [
    # (reads, writes): lists of (channels, level)
    ([], [(8, 0)]),                                   # encoder -> X
    ([(8, 0)], [(16, 0)]), ([(16, 0)], [(16, 0)]),    # T1, E0
    ([(16, 0)], [(8, 0)]),                            # depth map + running sum -> A0
    ([(16, 0)], [(32, 1)]), ([(32, 1)], [(32, 1)]),   # T2, E1
    ([(32, 1)], [(64, 2)]), ([(64, 2)], [(64, 2)]),   # T3, E2
    ([(64, 2)], [(128, 3)]), ([(128, 3)], [(128, 3)]),   # T4, E3
    ([(128, 3)], [(256, 4)]), ([(256, 4)], [(256, 4)]),  # T5, B4
    ([(256, 4), (128, 3)], [(128, 3)]), ([(128, 3)], [(128, 3)]),   # U3 + E3 -> S3, D3
    ([(128, 3), (64, 2)], [(64, 2)]), ([(64, 2)], [(64, 2)]),       # U2 + E2 -> S2, D2
    ([(64, 2), (32, 1)], [(32, 1)]), ([(32, 1)], [(32, 1)]),        # U1 + E1 -> S1, D1
    ([(32, 1), (16, 0), (8, 0)], [(24, 0)]),          # U0 + E0 + A0 -> S0
    ([(24, 0)], []),                                  # D0 with the fused head (output below)
]


def surrogate_bytes_per_frame(H: int, W: int) -> float:
    """Algorithmic HBM bytes of one frame's inference forward."""
    b = 0.0
    for reads, writes in SURR_FWD_TENSORS:
        for c, lv in reads + writes:
            b += 2.0 * c * (H >> lv) * (W >> lv)
    # label gather, FP32 head output, clamp (read + write), BF16 frame (FP32 read + BF16 write)
    return b + (1.0 + 4.0 + 8.0 + 6.0) * H * W


RAY_TRAFFIC_SUMMARY = os.path.join(ROOT, "profiles", "k_ray_hbm_traffic_256env.md")
RAY_SOURCES = [os.path.join(ROOT, "paper_2507_01152_amd", "csrc", f) for f in ("physics.hip", "sg_internal.h")]


def cpu_model() -> str:
    """The host CPU's model name (first 'model name' line of /proc/cpuinfo)."""
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def traffic_split():
    """(ray fetch, ray write, PSF fetch, PSF write) bytes per launch from the
    committed counter summary, or None (missing or other kernel sources)."""
    try:
        with open(RAY_TRAFFIC_SUMMARY) as fh:
            text = fh.read()
    except OSError:
        return None
    d = re.search(r"^kernel_sources_sha256:\s*([0-9a-f]{64})", text, re.M)
    if not d or d.group(1) != ray_kernel_digest():
        return None
    vals = []
    for key in ("ray_fetch_bytes", "ray_write_bytes", "psf_fetch_bytes", "psf_write_bytes"):
        m = re.search(r"^" + key + r":\s*(\d+)", text, re.M)
        if not m:
            return None
        vals.append(int(m.group(1)))
    return vals


def ray_kernel_digest() -> str:
    h = hashlib.sha256()
    for f in RAY_SOURCES:
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def ray_traffic_bytes(key="traffic_bytes_per_launch"):
    """HBM bytes per ray-kernel (or, with key psf_traffic_bytes_per_launch,
    PSF-kernel) launch from the committed counter summary (FETCH_SIZE +
    WRITE_SIZE, scaled by a plain copy's reading), or None when the summary
    is missing or was taken on other kernel sources."""
    try:
        with open(RAY_TRAFFIC_SUMMARY) as fh:
            text = fh.read()
    except OSError:
        return None
    b = re.search(r"^" + key + r":\s*(\d+)", text, re.M)
    d = re.search(r"^kernel_sources_sha256:\s*([0-9a-f]{64})", text, re.M)
    if not b or not d or d.group(1) != ray_kernel_digest():
        return None
    return int(b.group(1))


def ct_surrogate_leg(train_steps: int, n_envs: int = 256, batch: int = 32, audit_frac: int = 16,
                     psnr_min: float = 30.0):
    """CT-conditioned surrogate with histogram matching and the adversarial
    term (weight 0.01): train on spine CT phantom pairs, then audited
    inference of n_envs frames on held-out phantoms beside physics."""
    import numpy as np
    import torch

    from paper_2507_01152_amd import sonosim as sg
    from paper_2507_01152_amd.train_surrogate import CT_FRAME_H, CT_FRAME_W, CtPairSource, train_ct

    sess, sid, _src, step_s, last = train_ct(train_steps, batch, 1e-3, adv_weight=0.01, log=lambda s: None)
    test_src = CtPairSource(sess, 4, seed0=9000)     # held-out phantoms
    rng = np.random.default_rng(77)
    vids, probes, poses = test_src.batch(n_envs, rng)
    audit = np.sort(np.random.Generator(np.random.Philox(key=9)).choice(n_envs, n_envs // audit_frac,
                                                                         replace=False)).astype(np.int32)
    HW = CT_FRAME_W * CT_FRAME_H
    out = torch.empty(n_envs * HW, dtype=torch.float32, device=sess.device)
    out16 = torch.empty(n_envs * HW, dtype=torch.bfloat16, device=sess.device)   # the served BF16 frames
    # a serving loop's probes are fixed per env: marshalled once, as the physics plan takes them once
    vids = np.ascontiguousarray(vids, dtype=np.int32)
    probes = sg.probes_array(probes)
    sg.sg_surr_infer_bf16(sess.ctx, sid, vids, probes, poses, out16, audit, psnr_min, 0.25)   # warm-up
    reps = 5
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(reps):
        psnr, n_fb = sg.sg_surr_infer_bf16(sess.ctx, sid, vids, probes, poses, out16, audit, psnr_min, 0.25)
    surr_s = (time.perf_counter() - t) / reps
    all_psnr, _ = sg.sg_surr_infer(sess.ctx, sid, vids[:64], probes[:64], poses[:64], out, list(range(64)),
                                   -np.inf, 1.0)
    offs = np.arange(n_envs, dtype=np.int64) * HW
    plan = sg.sg_batch_plan_create(sess.ctx, vids, probes, offs)
    sg.sg_batch_set_poses(sess.ctx, plan, poses)
    for _ in range(3):
        sg.sg_batch_step(sess.ctx, plan, out)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(20):
        sg.sg_batch_step(sess.ctx, plan, out)
    torch.cuda.synchronize()
    phys_s = (time.perf_counter() - t) / 20
    sess.close()
    return {
        "workload": f"{n_envs} envs, {CT_FRAME_W}x{CT_FRAME_H} frames at 0.5 mm on held-out 256^3 spine CT "
                    f"phantoms, histogram-matched CT input, BF16 frames, 1/{audit_frac} seeded physics audit at "
                    f"PSNR >= {psnr_min} dB",
        "frame_dtype": "bf16",
        "frames_per_s": round(n_envs / surr_s, 1),
        "physics_frames_per_s_same_workload": round(n_envs / phys_s, 1),
        "psnr_audit_mean_db": round(float(np.mean(psnr)), 2),
        "psnr_held_out_64_mean_db": round(float(np.mean(all_psnr)), 2),
        "frames_from_physics": int(n_fb),
        "train": {"steps": train_steps, "batch": batch, "pairs": train_steps * batch, "adv_weight": 0.01,
                  "ms_per_step": round(step_s * 1e3, 2), "pairs_per_s": round(batch / step_s, 1), "last": last},
    }


def train_step_timing(sess, sid_src, n: int = 64, steps: int = 40):
    """Wall and device time per training step on a fixed batch of n pairs
    (the last batch sid_src trained on), enqueued without loss readbacks, with
    the step replayed from its HIP graph and kernel by kernel; a fresh network
    of the same shape, so the trained one is left as it is."""
    import torch

    from paper_2507_01152_amd import sonosim as sg
    from paper_2507_01152_amd.train_surrogate import FRAME_H, FRAME_W
    xin, tgt = sg.sg_surr_get_batch(sess.ctx, sid_src, n, FRAME_H, FRAME_W)
    xin = torch.from_numpy(xin.view("int16")).to(sess.device)
    tgt = torch.from_numpy(tgt).to(sess.device)
    res = {"pairs": n, "steps": steps}
    for mode in ("graph", "eager"):
        sid = sg.sg_surr_create(sess.ctx, FRAME_H, FRAME_W, seed=1)
        sg.sg_surr_set_graph(sess.ctx, sid, mode == "graph")
        for _ in range(3):   # eager sizing step, capture, one replay
            sg.sg_surr_train_pairs(sess.ctx, sid, xin, tgt, 1e-3)
        st = torch.cuda.current_stream()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        t = time.perf_counter()
        a.record(st)
        for _ in range(steps):
            sg.sg_surr_train_pairs_async(sess.ctx, sid, xin, tgt, 1e-3)
        b.record(st)
        torch.cuda.synchronize()
        wall = (time.perf_counter() - t) / steps
        first = sg.sg_surr_step_count(sess.ctx, sid) - steps + 1
        last = sg.sg_surr_loss_history(sess.ctx, sid, first, steps)[-1, 0]
        res[mode] = {"wall_ms": round(wall * 1e3, 3), "device_ms": round(a.elapsed_time(b) / steps, 3),
                     "last_loss": round(float(last), 5)}
        sg.sg_surr_destroy(sess.ctx, sid)
    return res


def surrogate_leg(train_steps: int, n_envs: int = 1024, audit_frac: int = 16, psnr_min: float = 30.0):
    """Train the surrogate on physics pairs for a fixed budget, then time
    audited inference of n_envs 128 x 256 frames beside the physics path on
    the same workload."""
    import numpy as np
    import torch

    import synth
    from paper_2507_01152_amd import sonosim as sg
    from paper_2507_01152_amd.train_surrogate import FRAME_H, FRAME_W, PairSource, train

    t0 = time.perf_counter()
    sess, sid, _train_src, _ev, hist = train(train_steps, 64, 1e-3, seed=0, eval_every=max(1, train_steps),
                                             log=lambda s: None)
    train_s = time.perf_counter() - t0
    step_timing = train_step_timing(sess, sid)
    test_src = PairSource(sess, 64, seed0=200000)     # held-out phantoms
    rng = np.random.default_rng(2024)
    vids, probes, poses = test_src.batch(n_envs, rng)
    audit = np.sort(np.random.Generator(np.random.Philox(key=7)).choice(n_envs, n_envs // audit_frac,
                                                                         replace=False)).astype(np.int32)
    HW = FRAME_W * FRAME_H
    out = torch.empty(n_envs * HW, dtype=torch.float32, device=sess.device)
    out16 = torch.empty(n_envs * HW, dtype=torch.bfloat16, device=sess.device)   # the served BF16 frames
    # a serving loop's probes are fixed per env: marshalled once, as the physics plan takes them once
    vids = np.ascontiguousarray(vids, dtype=np.int32)
    probes = sg.probes_array(probes)
    sg.sg_surr_infer_bf16(sess.ctx, sid, vids, probes, poses, out16, audit, psnr_min, 0.25)   # warm-up
    reps = 5
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(reps):
        psnr, n_fb = sg.sg_surr_infer_bf16(sess.ctx, sid, vids, probes, poses, out16, audit, psnr_min, 0.25)
    surr_s = (time.perf_counter() - t) / reps
    # network alone (no audit), for the MFMA roofline
    t = time.perf_counter()
    for _ in range(reps):
        sg.sg_surr_infer_bf16(sess.ctx, sid, vids, probes, poses, out16, [], psnr_min, 0.25)
    net_s = (time.perf_counter() - t) / reps
    # physics on the same workload: batched plan, steps enqueued back to back
    offs = np.arange(n_envs, dtype=np.int64) * HW
    plan = sg.sg_batch_plan_create(sess.ctx, vids, probes, offs)
    sg.sg_batch_set_poses(sess.ctx, plan, poses)
    for _ in range(3):
        sg.sg_batch_step(sess.ctx, plan, out)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(20):
        sg.sg_batch_step(sess.ctx, plan, out)
    torch.cuda.synchronize()
    phys_s = (time.perf_counter() - t) / 20
    mse = 10.0 ** (-np.asarray(psnr, dtype=np.float64) / 10.0)
    flops = surrogate_flops_per_frame(FRAME_H, FRAME_W) * n_envs
    nbytes = surrogate_bytes_per_frame(FRAME_H, FRAME_W) * n_envs
    res = {
        "workload": f"{n_envs} envs, {FRAME_W}x{FRAME_H} BF16 frames on held-out 64^3 ellipsoid phantoms, "
                    f"1/{audit_frac} seeded physics audit at PSNR >= {psnr_min} dB",
        "frame_dtype": "bf16",
        "frames_per_s": round(n_envs / surr_s, 1),
        "physics_frames_per_s_same_workload": round(n_envs / phys_s, 1),
        "surrogate_vs_physics": round(phys_s / surr_s, 4),
        "psnr_audit_mean_db": round(float(np.mean(psnr)), 2),
        "psnr_audit_pooled_db": round(float(-10 * np.log10(mse.mean())), 2),
        "frames_from_physics": int(n_fb),
        "train": {"steps": train_steps, "pairs": train_steps * 64, "seconds": round(train_s, 1),
                  "last_eval": hist[-1] if hist else None, "step_timing": step_timing},
        "roofline": {"bound": "mfma", "kernel": "network forward (encode + 18 convs + depth integral + head)",
                     "achieved": round(flops / net_s / 1e12, 2), "peak": 2500.0, "unit": "TFLOP/s",
                     "frac": round(flops / net_s / 1e12 / 2500.0, 4), "flops_per_launch": flops,
                     "ms": round(net_s * 1e3, 3),
                     "hbm_view": {"algorithmic_bytes": nbytes, "achieved_GBps": round(nbytes / net_s / 1e9, 1),
                                  "frac_of_8TBps": round(nbytes / net_s / 8e12, 4)}},
    }
    sess.close()
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-tune", action="store_true", help="skip the launch-shape autotuner")
    ap.add_argument("--launch-shape", default=None, metavar="SPW,TX,CHUNKS",
                    help="fixed launch shape of the physics step instead of the autotuner's")
    ap.add_argument("--profile-launches", type=int, default=20)
    ap.add_argument("--ct-surrogate-steps", type=int, default=4500,
                    help="training steps (batch 32) of the CT-conditioned surrogate with the adversarial term; "
                         "0 skips it")
    ap.add_argument("--surrogate-steps", type=int, default=3125,
                    help="training steps (batch 64; 3125 = 200k pairs) before timing surrogate inference; "
                         "0 skips the surrogate")
    ap.add_argument("--noise-scales", type=int, default=3,
                    help="also time the workload with this many noise scales (<= 1 skips it)")
    ap.add_argument("--no-volumetric", dest="volumetric", action="store_false",
                    help="skip the volumetric-probe leg")
    ap.add_argument("--no-recon", dest="recon", action="store_false",
                    help="skip the reconstruction-observation leg")
    ap.add_argument("--cpu-seconds", type=float, default=10.0,
                    help="minimum CPU time of the oracle baseline sample (whole steps, at most 200)")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="MIB",
                    help="also run one plain device copy of MIB MiB (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (asked for {args.gpus}); the environments shard "
              "across GPUs without communication, see the design notes", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import synth
    from paper_2507_01152_amd import sonosim as sg
    from paper_2507_01152_amd.session import Session

    wl = synth.batched_workload(seed=0)
    n = wl.n_envs
    offs, total = wl.out_offsets()
    sess = Session(0)
    vids = sess.load(wl)
    plan = sg.sg_batch_plan_create(sess.ctx, vids, wl.probes, offs)
    sg.sg_batch_set_poses(sess.ctx, plan, wl.poses)
    out = torch.empty(total, dtype=torch.float32, device=sess.device)
    if args.launch_shape:
        sg.sg_batch_set_config(sess.ctx, plan, *(int(v) for v in args.launch_shape.split(",")))
    elif not args.no_tune:
        sg.sg_autotune(sess.ctx, plan, os.environ.get("SG_TUNE_CACHE", "/tmp/sonosim_tune.jsonl"))
    spw, tx, ty, chunks = sg.sg_batch_config(sess.ctx, plan)

    for _ in range(args.warmup):
        sg.sg_batch_step(sess.ctx, plan, out)
    torch.cuda.synchronize()
    assert sg.sg_batch_status(sess.ctx, plan) == 0

    stream = torch.cuda.current_stream()
    t0 = torch.cuda.Event(enable_timing=True)
    t1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    wall0 = time.perf_counter()
    t0.record(stream)
    for _ in range(args.steps):
        sg.sg_batch_step(sess.ctx, plan, out)
    t1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - wall0
    ms = t0.elapsed_time(t1)
    ms_per_step = ms / args.steps
    fps = n * args.steps / (ms / 1e3)
    assert sg.sg_batch_status(sess.ctx, plan) == 0

    # the two persistent kernels, timed with events on the stream they run on
    prof = np.array([sg.sg_batch_step_profiled(sess.ctx, plan, out) for _ in range(args.profile_launches)])
    ray_ms, psf_ms = float(prof[:, 0].mean()), float(prof[:, 1].mean())
    pixels = sum(p.W * p.H for p in wl.probes)
    ray_ops = sum(ray_ops_per_pixel(p.W, p.H) * p.W * p.H for p in wl.probes)
    psf_ops = sum(psf_ops_per_pixel(p.W, p.H) * p.W * p.H for p in wl.probes)
    achieved_tops = ray_ops / (ray_ms / 1e3) / 1e12
    fma_r, int_r, mad_r, fma3_r = sg.sg_valu_probe(sess.ctx)
    probe = {"what": "measured VALU rates of independent instruction chains, Top/s (sg_valu_probe)",
             "fma_vop2": round(fma_r / 1e12, 2), "xor_add_vop2": round(int_r / 1e12, 2),
             "mad_u64": round(mad_r / 1e12, 2), "fma_vop3": round(fma3_r / 1e12, 2)}
    # achievable HBM bandwidth: a 1 GiB device copy (read + written bytes per second)
    cp_src = torch.ones(1 << 28, dtype=torch.float32, device=sess.device)
    cp_dst = torch.empty_like(cp_src)
    copy_gbs = sg.sg_hbm_probe(sess.ctx, cp_src, cp_dst) / 1e9
    c0, c1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    c0.record(stream)
    for _ in range(3):
        cp_dst.copy_(cp_src)
    c1.record(stream)
    torch.cuda.synchronize()
    torch_copy_gbs = 3 * 2 * cp_src.numel() * 4 / (c0.elapsed_time(c1) * 1e-3) / 1e9
    achievable_gbs = max(copy_gbs, torch_copy_gbs)   # the better of the two copies
    del cp_src, cp_dst
    psf_traffic = ray_traffic_bytes("psf_traffic_bytes_per_launch")
    # whole step on algorithmic bytes: 1 B label gather + 4 B FP32 frame per pixel
    alg_bytes = 5 * pixels
    achieved_gbs = alg_bytes / (ms_per_step / 1e3) / 1e9
    split = traffic_split()
    hbm_target = {
        "target": "physics at >= 50 % of achievable HBM bandwidth",
        "met": achieved_gbs / achievable_gbs >= 0.5,
        "why_not": "the step is bound by the ray kernel's VALU work (per-pixel Philox, scans, PSF taps), not by "
                   "bytes: its algorithmic 5 B/px move in a few microseconds at HBM speed",
    }
    if split:
        rf, rw, pf, pw = split
        hbm_target["measured_traffic_per_step"] = {
            "field_round_trip_bytes": rw + pf,
            "what": "three FP32 fields per pixel written by the ray kernel and read back (with the lateral halo) "
                    "by the PSF kernel",
            "other_bytes": rf + pw, "other_what": "label gathers (ray kernel) and frame stores (PSF kernel)",
            "total_bytes": rf + rw + pf + pw,
            "total_GBps": round((rf + rw + pf + pw) / (ms_per_step / 1e3) / 1e9, 1),
        }

    res = {
        "metric": "simulated B-mode frames/sec at 256 envs (physics vs surrogate @ stated PSNR)",
        "value": round(fps, 1),
        "unit": "frames/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": "batched physics, 256 envs over 8 uneven label volumes 160^3..320x256x384, "
                        "W 64-256 x H 128-512 at 0.5 mm, two persistent kernels per step",
            "n_envs": n,
            "pixels_per_step": pixels,
            "launch_shape": {"scanlines_per_item": spw, "tile_x": tx, "tile_y": ty, "chunks": chunks},
        },
        "roofline": {
            "bound": "alu",
            "kernel": "k_ray (sampling, scans, speckle, axial PSF)",
            "achieved": round(achieved_tops, 3),
            "peak": round(PEAK_VALU_TOPS, 2),
            "peak_probe": probe,
            "unit": "Top/s",
            "frac": round(achieved_tops / PEAK_VALU_TOPS, 4),
            "ops_per_launch": ray_ops,
            "kernel_ms": round(ray_ms, 4),
            "traffic": ray_traffic_bytes(),
            "psf_kernel": {"kernel_ms": round(psf_ms, 4), "ops_per_launch": psf_ops,
                           "achieved_Tops": round(psf_ops / (psf_ms / 1e3) / 1e12, 3),
                           "traffic": psf_traffic,
                           "traffic_GBps": (round(psf_traffic / (psf_ms / 1e3) / 1e9, 1)
                                            if psf_traffic else None),
                           "traffic_frac_of_achievable": (round(psf_traffic / (psf_ms / 1e3) / 1e9
                                                                / achievable_gbs, 4) if psf_traffic else None)},
            "hbm_achievable": {"what": "1 GiB device copies, read + written GB/s; the better one is the achievable",
                               "sg_hbm_probe": round(copy_gbs, 1), "torch_copy": round(torch_copy_gbs, 1)},
            "hbm_view_whole_step": {"algorithmic_bytes": alg_bytes, "achieved_GBps": round(achieved_gbs, 1),
                                    "frac_of_8TBps": round(achieved_gbs / PEAK_HBM_GBS, 4),
                                    "frac_of_achievable": round(achieved_gbs / achievable_gbs, 4),
                                    "hbm_target": hbm_target},
        },
        "wall_s_timed": round(wall, 3),
    }

    if args.noise_scales > 1:
        # the same workload with a multi-scale noise field (coarser N0 / N1 scales)
        import dataclasses
        ms = dataclasses.replace(wl, volumes=[dataclasses.replace(v, noise_scales=args.noise_scales)
                                              for v in wl.volumes])
        vids_ms = sess.load(ms)
        plan_ms = sg.sg_batch_plan_create(sess.ctx, vids_ms, ms.probes, offs)
        sg.sg_batch_set_poses(sess.ctx, plan_ms, ms.poses)
        sg.sg_batch_set_config(sess.ctx, plan_ms, spw, tx, chunks)
        for _ in range(args.warmup):
            sg.sg_batch_step(sess.ctx, plan_ms, out)
        torch.cuda.synchronize()
        t0.record(stream)
        for _ in range(args.steps):
            sg.sg_batch_step(sess.ctx, plan_ms, out)
        t1.record(stream)
        torch.cuda.synchronize()
        ms_ms = t0.elapsed_time(t1) / args.steps
        assert sg.sg_batch_status(sess.ctx, plan_ms) == 0
        res["multiscale_noise"] = {"noise_scales": args.noise_scales, "ms_per_step": round(ms_ms, 4),
                                   "frames_per_s": round(n / (ms_ms / 1e3), 1),
                                   "vs_one_scale": round(ms_per_step / ms_ms, 3)}
    if args.recon:
        # bone-surface reconstruction observation after each physics step (256 envs)
        rid = sg.sg_recon_create(sess.ctx, plan, 65536, None, 0.2, seed=1)
        grids = torch.zeros(n * 40 ** 3, dtype=torch.uint8, device=sess.device)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        upd, obs = [], []
        for st in range(20):
            ev[0].record(stream)
            sg.sg_recon_update(sess.ctx, rid, st)
            ev[1].record(stream)
            sg.sg_recon_observe(sess.ctx, rid, grids)
            ev[2].record(stream)
            torch.cuda.synchronize()
            upd.append(ev[0].elapsed_time(ev[1]))
            obs.append(ev[1].elapsed_time(ev[2]))
        stored, over = sg.sg_recon_counts(sess.ctx, rid, n)
        res["recon_observation"] = {
            "workload": "256 envs of the benchmark batch, 20 updates at one pose each, 40^3 grids at 3 mm",
            "update_ms": round(float(np.median(upd)), 4), "observe_ms": round(float(np.median(obs)), 4),
            "points_stored": int(stored.sum()), "points_overflow": int(over.sum()),
            "occupied_cells": int(grids.sum().item())}
        sg.sg_recon_destroy(sess.ctx, rid)
    if args.volumetric:
        # the surgery task's volumetric probe (50 x 37 x 5 at 2 x 2 x 10 mm) on the same volumes and poses
        vw = synth.volumetric_workload(seed=0)
        voffs, vtotal = vw.out_offsets()
        vout = torch.empty(vtotal, dtype=torch.float32, device=sess.device)
        plan_v = sg.sg_batch_plan_create(sess.ctx, vids, vw.probes, voffs)
        sg.sg_batch_set_poses(sess.ctx, plan_v, vw.poses)
        if not args.no_tune:
            sg.sg_autotune(sess.ctx, plan_v, os.environ.get("SG_TUNE_CACHE", "/tmp/sonosim_tune.jsonl"))
        for _ in range(args.warmup):
            sg.sg_batch_step(sess.ctx, plan_v, vout)
        torch.cuda.synchronize()
        t0.record(stream)
        for _ in range(args.steps):
            sg.sg_batch_step(sess.ctx, plan_v, vout)
        t1.record(stream)
        torch.cuda.synchronize()
        v_ms = t0.elapsed_time(t1) / args.steps
        assert sg.sg_batch_status(sess.ctx, plan_v) == 0
        res["volumetric_probe"] = {"workload": "256 envs, 50 x 37 x 5 volumes at 2 x 2 x 10 mm, same volumes/poses",
                                   "ms_per_step": round(v_ms, 4), "volumes_per_s": round(n / (v_ms / 1e3), 1),
                                   "planes_per_s": round(5 * n / (v_ms / 1e3), 1),
                                   "launch_shape": list(sg.sg_batch_config(sess.ctx, plan_v))}
    if not args.no_cpu:
        import oracle
        reps, dt = 0, 0.0
        while reps < 200 and (reps == 0 or dt < args.cpu_seconds):
            t = time.perf_counter()
            _frames, used = oracle.simulate_batch(wl, n_threads=0)
            dt += time.perf_counter() - t
            reps += 1
        # one core: the first 64 envs once, scaled by their share of the step's pixels
        sub = list(range(min(64, n)))
        sub_px = sum(wl.probes[e].W * wl.probes[e].H for e in sub)
        t = time.perf_counter()
        _frames, used1 = oracle.simulate_batch(wl, env_ids=sub, n_threads=1)
        dt1 = time.perf_counter() - t
        res["cpu_baseline"] = {
            "value": round(reps * n / dt, 2),
            "unit": "frames/s",
            "cores": used,
            "cpu_model": cpu_model(),
            "kind": "oracle",
            "sample": f"{reps} full steps of the same workload ({n} envs, {pixels} px each), FP64, "
                      f"OpenMP over envs, {dt:.1f} s wall",
            "single_core": {"value": round(n * sub_px / pixels / dt1, 2), "unit": "frames/s", "cores": used1,
                            "sample": f"envs 0..{len(sub) - 1} of the step once ({sub_px} px), {dt1:.2f} s, "
                                      f"as frames of the step's mean size"},
        }
        res["gpu_vs_cpu"] = round(fps / res["cpu_baseline"]["value"], 1)
    if args.surrogate_steps > 0:
        sess.close()
        res["surrogate"] = surrogate_leg(args.surrogate_steps)
    if args.ct_surrogate_steps > 0:
        if sess.ctx is not None:
            sess.close()
        res["ct_surrogate"] = ct_surrogate_leg(args.ct_surrogate_steps)
    if args.copy_probe:
        src = torch.ones(args.copy_probe << 18, dtype=torch.float32, device=sess.device)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        res["copy_probe_bytes"] = src.numel() * 4
    if sess.ctx is not None:
        sess.close()
    print(json.dumps(res))


if __name__ == "__main__":
    main()
