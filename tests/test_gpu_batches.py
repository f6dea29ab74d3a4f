"""A batched application with two lanes: bit for bit the results, recurrent state included, of one with a single lane (an odd
queue depth), for batches that come alone and for batches in flight together."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,nw,nh,depth,annotate", [
    (2, 1100, 560, 2, False),
    (3, 854, 480, 4, False),      # the 64 -> 128-channel layer's tiles of consecutive pixels
    (5, 680, 360, 2, True),       # stage 3 in launches of its own
    (12, 854, 480, 2, False),     # that layer as a walk over its tiles
    (16, 300, 256, 4, False),
])
def test_two_lanes_are_one_lane(hs, batch, nw, nh, depth, annotate):
    from paper_2402_04466_amd.harness import AppStream
    fw, fh, runs = 640, 360, [1, depth, 1, 1]
    blob = si.he_normal_blob(si.RESNET18_CONVLSTM_LAYERS, 8)
    ctx = hs.hs_init(0)
    two, one = (AppStream(ctx, net=hs.HS_NET_RESNET18_CONVLSTM, frame_w=fw, frame_h=fh, net_w=nw, net_h=nh, blob=blob,
                              palette=si.DEFAULT_PALETTE, queue_depth=d, batch=batch,
                              glyphs=si.DEFAULT_GLYPHS if annotate else None) for d in (depth, 1))
    try:
        frames = list(si.uniform_frames(3, fh, fw, 11))
        d_frames = [two.upload_frame(f) for f in frames]
        outs = {a: [[a.new_output() for _ in range(batch)] for _ in range(sum(runs))] for a in (two, one)}
        t = 0
        for n in runs:
            print(f"[batches] batch {batch} of {nw}x{nh}, depth {depth}: {n} steps from {t}", flush=True)
            src = [[d_frames[(k + j) % 3] for j in range(batch)] for k in range(t, t + n)]
            for i in range(n):
                assert two.submit_batch(src[i], outs[two][t + i], t + i) == hs.HS_OK
            got = [two.wait_batch() for _ in range(n)]
            for i in range(n):
                assert one.submit_batch(src[i], outs[one][t + i], t + i) == hs.HS_OK
                ref = one.wait_batch()
                for j in range(batch):
                    r = got[i][j]
                    assert r.t_submit_ns <= r.t_pre_done_ns < r.t_infer_done_ns < r.t_post_done_ns <= r.t_overlay_done_ns
                    a, b = two.fetch(r, outs[two][t + i][j]), one.fetch(ref[j], outs[one][t + i][j])
                    for key in (a if n == 1 or i == n - 1 else ["overlay"]):   # a slot's maps are the next frame's by then
                        assert np.array_equal(a[key], b[key]), (t + i, j, key)
            for j in range(batch):
                for a, b in zip(two.state(got[-1][j], stream=j), one.state(ref[j], stream=j)):
                    assert np.array_equal(a, b), (t, j, "state")
            t += n
    finally:
        two.close()
        one.close()
        hs.hs_shutdown(ctx)
