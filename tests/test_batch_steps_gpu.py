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
