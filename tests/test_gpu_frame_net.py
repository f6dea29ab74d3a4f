"""Stage 1 inside the small network's launch: bit for bit what the two launches of graph mode leave (network input in both
types, logits, maps, overlay), at tiles that hang over the image on every side, frames of odd widths and
pitches, enlarged and much reduced ones, batches, and the first size beyond its range."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fw,fh,pad,nw,nh,batch,fp32", [
    (320, 240, 0, 128, 128, 1, True),      # whole tiles
    (322, 241, 32, 96, 72, 2, True),       # ragged rows, padding behind them
    (17, 5, 0, 33, 31, 1, True),           # enlarged; one tile and one pixel more each way
    (1, 1, 0, 8, 8, 3, True),
    (64, 48, 0, 200, 150, 1, False),
    (1921, 333, 16, 67, 129, 3, True),     # reduced by 29; source rows far apart
    (640, 360, 0, 512, 512, 1, False),     # 256 tiles
    (640, 360, 0, 513, 512, 1, False),     # 272: two launches
])
def test_stage_one_in_the_networks_launch(hs, fw, fh, pad, nw, nh, batch, fp32):
    from paper_2402_04466_amd.harness import AppStream
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=fw, frame_h=fh, net_w=nw, net_h=nh, batch=batch, queue_depth=2,
                  blob=si.he_normal_blob(si.TINY4_LAYERS, 5), palette=si.DEFAULT_PALETTE, net_fp32_input=fp32,
                  frame_pitch=(3 * fw + 15) // 16 * 16 + pad)
    try:
        frames = list(si.uniform_frames(2 * batch, fh, fw, 21))
        got = {}
        for mode in (hs.HS_LAUNCH_GRAPH, hs.HS_LAUNCH_EAGER):
            hs.hs_set_launch_mode(s.app, mode)
            for t in range(2):             # both slots; the second mode overwrites the first one's images
                print(f"[frame-net] {fw}x{fh} to {nw}x{nh} batch {batch} mode {mode} step {t}", flush=True)
                d_in = [s.upload_frame(f) for f in frames[t * batch:(t + 1) * batch]]
                d_out = [s.new_output() for _ in d_in]
                assert s.submit_batch(d_in, d_out, t) == hs.HS_OK
                got[mode, t] = [s.fetch(r, o) for r, o in zip(s.wait_batch(), d_out)]
        for t in range(2):
            for a, b in zip(got[hs.HS_LAUNCH_GRAPH, t], got[hs.HS_LAUNCH_EAGER, t]):
                for key in a:
                    assert np.array_equal(a[key], b[key]), (t, key)
    finally:
        s.close()
        hs.hs_shutdown(ctx)
