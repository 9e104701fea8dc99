"""Batched steps that follow each other without waiting, and plans and calls
large enough for every launch shape (GPU).  Frames are compared bit for bit
with single calls of few frames."""
import numpy as np
import pytest

import synth
from synth import Probe, Volume, Workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sess():
    from paper_2507_01152_amd.session import Session
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s = Session(0)
    yield s
    s.close()


def _workload(n, sizes, seed=4):
    """n envs on two phantoms; image sizes taken from `sizes` in turn."""
    rng = np.random.default_rng(seed)
    vols = [Volume(labels=synth.ellipsoid_volume(seed + i, n=32), seed=60 + i) for i in range(2)]
    probes = [Probe(W=w, H=h) for w, h in (sizes[i % len(sizes)] for i in range(n))]
    return Workload(vols, (np.arange(n) % 2).astype(np.int32), probes, _poses(n, rng))


def _poses(n, rng):
    return np.stack([synth.pose_from(synth.random_rotation(rng), rng.uniform(8, 24, 3)).reshape(-1) for _ in range(n)])


def _few_at_a_time(sess, wl, vids, poses, k=16):
    """The frames by calls of k frames each."""
    from paper_2507_01152_amd import sonosim as sg
    offs, total = wl.out_offsets()
    out = torch.full((total,), -1.0, device="cuda")
    for i in range(0, wl.n_envs, k):
        s = slice(i, min(i + k, wl.n_envs))
        sg.sg_simulate(sess.ctx, vids[s], wl.probes[s], poses[s], out, offs[s])
    return out


# the chunked pipeline with more ray items than fit at once, so that its PSF kernels run on the second stream
@pytest.mark.parametrize("chunks", [2, 3, 4])
def test_chunked_pipeline_of_a_large_plan(sess, chunks):
    from paper_2507_01152_amd import sonosim as sg
    wl = _workload(700, [(20, 70), (9, 40), (33, 65)])
    vids = sess.load(wl)
    offs, total = wl.out_offsets()
    plan = sg.sg_batch_plan_create(sess.ctx, vids, wl.probes, offs)
    sg.sg_batch_set_config(sess.ctx, plan, 4, 32, chunks)
    rng = np.random.default_rng(chunks)
    poses = [_poses(wl.n_envs, rng) for _ in range(3)]
    outs = [torch.full((total,), -1.0, device="cuda") for _ in poses]
    for p, o in zip(poses, outs):
        sg.sg_batch_set_poses(sess.ctx, plan, p)
        sg.sg_batch_step(sess.ctx, plan, o)
    for p, o in zip(poses, outs):
        assert torch.equal(o, _few_at_a_time(sess, wl, vids, p))
    sg.sg_batch_plan_destroy(sess.ctx, plan)


# pose uploads past the by-value limit (32 envs) through the ring of pinned slots: more sets than slots, none waited
# for, each step's frames those of its own poses
@pytest.mark.parametrize("n", [33, 200])
def test_pose_sets_in_flight(sess, n):
    from paper_2507_01152_amd import sonosim as sg
    wl = _workload(n, [(24, 60), (7, 33)])
    vids = sess.load(wl)
    offs, total = wl.out_offsets()
    plan = sg.sg_batch_plan_create(sess.ctx, vids, wl.probes, offs)
    rng = np.random.default_rng(n)
    poses = [_poses(n, rng) for _ in range(11)]
    outs = [torch.full((total,), -1.0, device="cuda") for _ in poses]
    buf = np.empty_like(poses[0])
    for p, o in zip(poses, outs):
        buf[:] = p   # the caller's buffer may be reused at once
        sg.sg_batch_set_poses(sess.ctx, plan, buf)
        sg.sg_batch_step(sess.ctx, plan, o)
        buf[:] = np.nan
    for p, o in zip(poses, outs):
        assert torch.equal(o, _few_at_a_time(sess, wl, vids, p))
    # single calls stage their parameters the same way
    outs = [torch.full((total,), -1.0, device="cuda") for _ in poses]
    for p, o in zip(poses, outs):
        sg.sg_simulate(sess.ctx, vids, wl.probes, p, o, offs)
    for p, o in zip(poses, outs):
        assert torch.equal(o, _few_at_a_time(sess, wl, vids, p))
    sg.sg_batch_plan_destroy(sess.ctx, plan)


# a plan's steps take up a new output buffer, another stream and a volume registered in between
def test_steps_after_changes(sess):
    from paper_2507_01152_amd import sonosim as sg
    wl = _workload(40, [(24, 60)])
    vids = sess.load(wl)
    offs, total = wl.out_offsets()
    plan = sg.sg_batch_plan_create(sess.ctx, vids, wl.probes, offs)
    sg.sg_batch_set_poses(sess.ctx, plan, wl.poses)
    ref = _few_at_a_time(sess, wl, vids, wl.poses)
    a, b = (torch.full((total,), -1.0, device="cuda") for _ in range(2))
    sg.sg_batch_step(sess.ctx, plan, a)
    sg.sg_batch_step(sess.ctx, plan, b)
    assert torch.equal(a, ref) and torch.equal(b, ref)
    for k in range(40):   # the device's volume table grows
        sess.register(Volume(labels=synth.ellipsoid_volume(50 + k, n=8), seed=k))
    a.fill_(-1.0)
    sg.sg_batch_step(sess.ctx, plan, a)
    assert torch.equal(a, ref)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    b.fill_(-1.0)
    torch.cuda.synchronize()
    sg.sg_set_stream(sess.ctx, side)
    try:
        sg.sg_batch_set_poses(sess.ctx, plan, wl.poses)
        sg.sg_batch_step(sess.ctx, plan, b)
        sg.sg_synchronize(sess.ctx)
    finally:
        sg.sg_set_stream(sess.ctx, None)
    assert torch.equal(b, ref)
    sg.sg_batch_plan_destroy(sess.ctx, plan)


# two and four scanlines a wave by the rule (past 12,288 and 36,864 scanlines), ragged widths, both tile widths
@pytest.mark.parametrize("n,sizes,items,tile", [(300, [(61, 40), (30, 66), (33, 9)], 8, 64), (1200, [(61, 20), (35, 12), (3, 30)], 16, 64),
                                               (2400, [(17, 12), (31, 70), (5, 3)], 16, 32)])
def test_default_shapes_of_large_calls(sess, n, sizes, items, tile):
    from paper_2507_01152_amd import sonosim as sg
    wl = _workload(n, sizes)
    vids = sess.load(wl)
    offs, total = wl.out_offsets()
    ref = _few_at_a_time(sess, wl, vids, wl.poses)
    plan = sg.sg_batch_plan_create(sess.ctx, vids, wl.probes, offs)
    assert sg.sg_batch_config(sess.ctx, plan) == (items, tile, 64, 1)
    sg.sg_batch_set_poses(sess.ctx, plan, wl.poses)
    for call in (lambda o: sg.sg_batch_step(sess.ctx, plan, o),
                 lambda o: sg.sg_simulate(sess.ctx, vids, wl.probes, wl.poses, o, offs)):
        out = torch.full((total,), -1.0, device="cuda")
        call(out)
        assert torch.equal(out, ref)
    sg.sg_batch_plan_destroy(sess.ctx, plan)


# the entry point without allocation builds its own work lists: two and four scanlines a wave, narrow frames
@pytest.mark.parametrize("n,sizes", [(256, [(61, 40), (30, 66), (65, 9)]), (250, [(170, 9), (149, 5)]), (256, [(8, 256)])])
def test_noalloc_launch_shapes(sess, n, sizes):
    from paper_2507_01152_amd import sonosim as sg
    wl = _workload(n, sizes)
    vids = sess.load(wl)
    offs, total = wl.out_offsets()
    out = torch.full((total,), -1.0, device="cuda")
    sg.sg_simulate_noalloc(sess.ctx, vids, wl.probes, wl.poses, out, offs)
    assert torch.equal(out, _few_at_a_time(sess, wl, vids, wl.poses))
