"""Edges of the physics launches (GPU): work items around the number of work
counters and of resident blocks, and uploads on both sides of the by-value
limit.  All frames of a plan come from one frame's inputs, so each has to be
that frame bit for bit, on every step (the counters are cleared in between).
"""
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


# one item per env (4 scanlines): below, at and past the 64 counters; past the resident blocks (at most 8 per
# compute unit of 256); 32 poses are the last by-value upload (3072 bytes), 33 the first pinned one
@pytest.mark.parametrize("n", [1, 32, 33, 63, 64, 65, 130, 2049, 4200])
def test_every_item_is_taken_once(sess, n):
    from paper_2507_01152_amd import sonosim as sg
    vol = Volume(labels=synth.ellipsoid_volume(3, n=32), seed=77)
    wl = synth.ellipsoid_workload(seed=3, n_envs=1, n=32)
    probe, pose = Probe(W=4, H=70), wl.poses[0]
    one = Workload([vol], np.zeros(1, np.int32), [probe], pose[None])
    vid = sess.load(one)
    ref, _, _ = sess.simulate(one, vid)
    ref = ref.cpu().numpy()
    assert ref.max() > 0
    many = Workload([vol], np.zeros(n, np.int32), [probe] * n, np.repeat(pose[None], n, 0))
    offs, total = many.out_offsets()
    plan = sg.sg_batch_plan_create(sess.ctx, np.repeat(vid, n), many.probes, offs)
    for _ in range(3):
        out = torch.full((total,), -1.0, device="cuda")
        sg.sg_batch_set_poses(sess.ctx, plan, many.poses)
        sg.sg_batch_step(sess.ctx, plan, out)
        assert np.array_equal(out.cpu().numpy().reshape(n, -1), np.broadcast_to(ref, (n, ref.size)))
    single = torch.full((total,), -1.0, device="cuda")
    for _ in range(2):
        sg.sg_simulate(sess.ctx, np.repeat(vid, n), many.probes, many.poses, single, offs)
    assert np.array_equal(single.cpu().numpy().reshape(n, -1), np.broadcast_to(ref, (n, ref.size)))
    sg.sg_batch_plan_destroy(sess.ctx, plan)


# 16 scanlines a block, four a wave, 64 rows a step; with air among the bone labels the rows outside the volume
# are surface points too
@pytest.mark.parametrize("bone", [(2, 3), (0, 3)])
@pytest.mark.parametrize("H", [1, 64, 65, 130])
def test_surface_points_of_ragged_frames(sess, H, bone):
    import oracle
    from paper_2507_01152_amd import sonosim as sg
    widths = [1, 3, 15, 16, 17, 33]
    wl = synth.ellipsoid_workload(seed=9, n_envs=len(widths), n=32)
    wl.probes = [Probe(W=w, H=H, dx=0.7, dy=0.7) for w in widths]
    wl.probes[3] = Probe(W=16, H=H, dx=0.7, dy=0.7, n_elev=3, elev=4.0)
    vids = sess.load(wl)
    offs, total = wl.out_offsets()
    plan = sg.sg_batch_plan_create(sess.ctx, vids, wl.probes, offs)
    sg.sg_batch_set_poses(sess.ctx, plan, wl.poses)
    sg.sg_batch_step(sess.ctx, plan, torch.empty(total, device="cuda"))
    rid = sg.sg_recon_create(sess.ctx, plan, 64, bone, 0.2, seed=5)
    sg.sg_recon_update(sess.ctx, rid, 1)
    stored, over = sg.sg_recon_counts(sess.ctx, rid, wl.n_envs)
    for e in range(wl.n_envs):
        ref = oracle.recon_points(wl.volumes[e], wl.probes[e], wl.poses[e], e, 1, 5, 0.2, bone)
        got = sg.sg_recon_points(sess.ctx, rid, e, 64)
        key = lambda a: a[np.lexsort(a.T[::-1])]
        assert stored[e] == len(ref) and over[e] == 0
        assert np.array_equal(key(got), key(ref)), e
    sg.sg_recon_destroy(sess.ctx, rid)
    sg.sg_batch_plan_destroy(sess.ctx, plan)
