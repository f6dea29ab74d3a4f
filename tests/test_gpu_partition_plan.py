"""Under a partition the convolutions are planned for the CUs that it keeps busy, in other tile forms (one of them taken
nowhere else): the results are the whole device's bit for bit, and again once the partition is released."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,nw,nh,cus", [
    (2, 854, 480, 80),       # 512 channels in tiles of 32 channels x 128 pixels
    (3, 641, 361, 128),
    (1, 288, 160, 16),       # two of the four shader engines
])
def test_partition_plans_give_the_same_results(hs, batch, nw, nh, cus):
    from paper_2402_04466_amd.harness import AppStream
    fw, fh = 640, 360
    blob = si.he_normal_blob(si.RESNET18_CONVLSTM_LAYERS, 8)
    ctx = hs.hs_init(0)
    part, free = (AppStream(ctx, net=hs.HS_NET_RESNET18_CONVLSTM, frame_w=fw, frame_h=fh, net_w=nw, net_h=nh, blob=blob,
                            palette=si.DEFAULT_PALETTE, queue_depth=2, batch=batch) for _ in range(2))
    try:
        frames = list(si.uniform_frames(2, fh, fw, 31))
        d_frames = [part.upload_frame(f) for f in frames]
        for t, mask in enumerate((hs.cu_mask_words(range(cus)),) * 2 + (None,)):
            print(f"[partition plan] batch {batch} of {nw}x{nh} on {cus} CUs, step {t}", flush=True)
            hs.hs_set_partition(part.app, mask, mask)
            got = []
            for s in (part, free):
                outs = [s.new_output() for _ in range(batch)]
                assert s.submit_batch([d_frames[(t + j) % 2] for j in range(batch)], outs, t) == hs.HS_OK
                rs = s.wait_batch()
                got.append([(s.fetch(r, o), s.state(r, stream=j)) for j, (r, o) in enumerate(zip(rs, outs))])
            for j, ((a, sa), (b, sb)) in enumerate(zip(*got)):
                for key in a:
                    assert np.array_equal(a[key], b[key]), (t, j, key)
                assert np.array_equal(sa[0], sb[0]) and np.array_equal(sa[1], sb[1]), (t, j, "state")
    finally:
        part.close()
        free.close()
        hs.hs_shutdown(ctx)
