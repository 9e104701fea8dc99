"""Frames that fail their audit (GPU): some of the audited ones, none, and all,
against the physics frames and the frames of an inference without audit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# one replaced frame, an odd number past the by-value index upload (384 frames), audits out of order; frames of one
# and of several blocks
@pytest.mark.parametrize("n,h,w,audited", [(1, 16, 16, 1), (7, 32, 48, 5), (5, 112, 80, 5), (801, 16, 16, 801)])
def test_failing_frames_become_physics_frames(n, h, w, audited):
    from paper_2507_01152_amd import sonosim as sg
    from paper_2507_01152_amd.session import Session
    from synth import Workload
    from test_surrogate_gpu import _pairs
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    with Session(0) as sess:
        few = _pairs(min(n, 8), h, w, seed=n)
        k = np.arange(n) % few.n_envs
        poses = few.poses.reshape(-1, 3, 4)[k].copy()
        poses[:, :, 3] += np.random.default_rng(3).uniform(-2.0, 2.0, (n, 3))
        wl = Workload(few.volumes, k.astype(np.int32), [few.probes[i] for i in k], poses.reshape(n, 12))
        vids = sess.load(wl)
        sid = sg.sg_surr_create(sess.ctx, h, w, seed=5)
        physics = sess.simulate(wl, vids)[0].reshape(n, h, w)
        out, net = (torch.empty((n, h, w), device="cuda") for _ in range(2))
        out16 = torch.empty((n, h, w), dtype=torch.bfloat16, device="cuda")
        audit = np.random.default_rng(n).permutation(n)[:audited].astype(np.int32)
        psnr, nf = sg.sg_surr_infer(sess.ctx, sid, vids, wl.probes, wl.poses, net, audit, -np.inf, 1.0)
        assert nf == 0
        for bar in (float(np.median(psnr)), np.inf):
            fails = psnr < bar
            want = net.clone()
            at = torch.from_numpy(audit[fails].astype(np.int64)).cuda()
            want[at] = physics[at]
            for call, o, ref in ((sg.sg_surr_infer, out, want), (sg.sg_surr_infer_bf16, out16, want.bfloat16())):
                o.fill_(-1.0)
                got, nf = call(sess.ctx, sid, vids, wl.probes, wl.poses, o, audit, bar, 1.0)
                assert nf == int(fails.sum()) and np.array_equal(got, psnr)
                assert torch.equal(o, ref)
        sg.sg_surr_destroy(sess.ctx, sid)
