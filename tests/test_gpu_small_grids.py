"""The convolution kernels against the CPU oracle, at maps smaller than one tile, one tile plus a
remainder, and many ragged tiles: every form of k_conv3x3_run and k_conv3x3s2_run, the walking stride-2
kernel (a test of the host's planning holds that these sizes take them all), k_tiny_net and
k_conv_direct (the small network).  The recurrent cell is checked alone on the GPU's own inputs."""
import numpy as np
import pytest

import oracle
import synth_inputs as si
from gpu_common import TOL_CELL, TOL_STATE_RMS, check_frame, make_oracles, rel_err, rms_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw,nh,batch", [
    (8, 8, 1),        # the smallest input: maps of 2 x 2 and 1 x 1 pixels, the last stage's the largest tensor
    (8, 8, 3),        # the same, several images in every tensor
    (96, 64, 1),      # maps of 8 x 12, 4 x 6 and 2 x 3 pixels: tiles of 32 channels x 32 pixels, and those for tiny maps
    (130, 66, 6),     # the former alone, grids beyond one round of workgroups
    (130, 66, 16),    # runs that span several images
    (288, 160, 5),    # four K splits at every layer but the first at stride 2
    (288, 160, 12),   # tiles of 32 and 64 channels x 64 pixels, of 64 x 96; maps of 20 x 36, 10 x 18 and 5 x 9
])
def test_small_grid_convolutions_match_the_oracle(hs, nw, nh, batch):
    from paper_2402_04466_amd.harness import AppStream
    fw, fh, frames = 320, 180, 2
    blob = si.he_normal_blob(si.RESNET18_CONVLSTM_LAYERS, 8)
    w16 = [w.astype(np.float16).astype(np.float32)
           for w in oracle.split_blob(blob, oracle.ResNet18ConvLSTMNet.shapes())[-2:]]
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_RESNET18_CONVLSTM, frame_w=fw, frame_h=fh, net_w=nw, net_h=nh,
                  blob=blob, palette=si.DEFAULT_PALETTE, queue_depth=2, batch=batch)
    try:
        host = {j: list(si.tool_scene_frames(frames, fh, fw, 70 + j)) for j in range(batch)}
        sampled = sorted({0, batch - 1})
        oracles = {j: make_oracles("resnet18_convlstm", blob, nw, nh, True, si.DEFAULT_PALETTE)[0]
                   for j in sampled}
        prev = {}
        for t in range(frames):
            print(f"[small-grid] {nw}x{nh} batch {batch} frame {t}", flush=True)
            d_in = [s.upload_frame(host[j][t]) for j in range(batch)]
            d_out = [s.new_output() for _ in range(batch)]
            assert s.submit_batch(d_in, d_out, t) == hs.HS_OK
            rs = s.wait_batch()
            for j in sampled:
                g, o = s.fetch(rs[j], d_out[j]), oracles[j].process(host[j][t])
                check_frame(g, host[j][t], o, None, threshold=0.5, alpha=0.5,
                            palette=si.DEFAULT_PALETTE, fp32_input=False,
                            tag=f"small-grid/{nw}x{nh}x{batch}/stream{j}/frame{t}")
                h, c = s.state(rs[j], stream=j)
                h0, c0 = prev.get(j, (np.zeros_like(h), np.zeros_like(c)))
                oh, oc = oracle.convlstm_step(s.features(rs[j], stream=j), h0, c0, w16[0])
                head = oracle.conv2d(h, w16[1], 1, 0)
                assert max(rel_err(h, oh), rel_err(c, oc), rel_err(g["logits"], head)) <= TOL_CELL
                assert rms_rel(h, o["h"]) <= TOL_STATE_RMS and rms_rel(c, o["c"]) <= TOL_STATE_RMS
                prev[j] = (h, c)
    finally:
        s.close()
        hs.hs_shutdown(ctx)


@pytest.mark.parametrize("nw,nh,batch", [
    (40, 520, 2),     # maps of 2 x 17 pixels and wider: strips of a few columns, tiles over several images
    (300, 170, 16),   # tiles of 32 channels x 32 pixels, of 32 and 64 x 64, on several rounds of workgroups
    (430, 250, 16),   # tiles of 64 channels x 64 and 128 pixels
    (860, 500, 11),   # of 64 channels x 128 and 160 pixels, 96 at stride 2, maps no multiple of any strip; walking workgroups
])
def test_tiles_of_consecutive_pixels_match_the_oracle(hs, nw, nh, batch):
    test_small_grid_convolutions_match_the_oracle(hs, nw, nh, batch)


@pytest.mark.parametrize("nw,nh,batch", [
    (8, 8, 1),        # a 2 x 2 map: one pixel tile, mostly beyond the layer's end
    (33, 17, 3),      # ragged maps, images that end inside a pixel tile, two K splits
    (250, 190, 5),    # 240 tiles: nearly a round
])
def test_small_network_layers_match_the_oracle(hs, nw, nh, batch):
    from paper_2402_04466_amd.harness import AppStream
    fw, fh = 64, 48
    blob = si.he_normal_blob(si.TINY4_LAYERS, 9)
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=fw, frame_h=fh, net_w=nw, net_h=nh, blob=blob,
                  palette=si.DEFAULT_PALETTE, queue_depth=2, batch=batch)
    try:
        host = [si.uniform_frames(1, fh, fw, 90 + j)[0] for j in range(batch)]
        print(f"[small-network] {nw}x{nh} batch {batch}", flush=True)
        d_in, d_out = [s.upload_frame(f) for f in host], [s.new_output() for _ in host]
        assert s.submit_batch(d_in, d_out, 0) == hs.HS_OK
        for j, r in enumerate(s.wait_batch()):
            o32, o16 = make_oracles("tiny4", blob, nw, nh, True, si.DEFAULT_PALETTE)
            check_frame(s.fetch(r, d_out[j]), host[j], o32.process(host[j]), o16.process(host[j]),
                        threshold=0.5, alpha=0.5, palette=si.DEFAULT_PALETTE, fp32_input=False,
                        tag=f"small-network/{nw}x{nh}/stream{j}")
    finally:
        s.close()
        hs.hs_shutdown(ctx)


@pytest.mark.parametrize("nw,nh,batch", [
    (8, 8, 1),        # one tile, mostly beyond the map
    (33, 17, 3),      # 9 x 5 logits: tiles of one column and of five rows
    (130, 122, 2),    # several ragged tiles
])
def test_small_network_in_one_launch_equals_its_layers(hs, nw, nh, batch):
    from paper_2402_04466_amd.harness import AppStream
    fw, fh = 64, 48
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=fw, frame_h=fh, net_w=nw, net_h=nh,
                  blob=si.he_normal_blob(si.TINY4_LAYERS, 10), palette=si.DEFAULT_PALETTE, queue_depth=2, batch=batch)
    try:
        print(f"[small-network] one launch against layers {nw}x{nh} batch {batch}", flush=True)
        host = [si.uniform_frames(1, fh, fw, 40 + j)[0] for j in range(batch)]
        d_in = [s.upload_frame(f) for f in host]
        got = []
        for timed in (False, True):          # layer by layer, behind the one launch, while kernels are being timed
            hs.hs_set_kernel_timing(s.app, timed)
            d_out = [s.new_output() for _ in host]
            assert s.submit_batch(d_in, d_out, 0) == hs.HS_OK
            got.append([s.fetch(r, o) for r, o in zip(s.wait_batch(), d_out)])
        for a, b in zip(*got):
            for key in ("logits", "heat", "mask", "overlay"):
                assert np.array_equal(a[key], b[key]), key
    finally:
        s.close()
        hs.hs_shutdown(ctx)


def test_small_network_of_many_tiles_matches_the_oracle(hs):
    from paper_2402_04466_amd.harness import AppStream
    nw, nh, batch, fw, fh = 522, 402, 16, 64, 48       # 131 x 101 logits: 17 x 13 x 16 tiles
    blob = si.he_normal_blob(si.TINY4_LAYERS, 11)
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=fw, frame_h=fh, net_w=nw, net_h=nh, blob=blob,
                  palette=si.DEFAULT_PALETTE, queue_depth=2, batch=batch)
    try:
        print(f"[small-network] {nw}x{nh} batch {batch}", flush=True)
        host = [si.uniform_frames(1, fh, fw, 60 + j)[0] for j in range(batch)]
        d_in, d_out = [s.upload_frame(f) for f in host], [s.new_output() for _ in host]
        assert s.submit_batch(d_in, d_out, 0) == hs.HS_OK
        rs = s.wait_batch()
        for j in (0, batch - 1):
            o32, o16 = make_oracles("tiny4", blob, nw, nh, True, si.DEFAULT_PALETTE)
            check_frame(s.fetch(rs[j], d_out[j]), host[j], o32.process(host[j]), o16.process(host[j]),
                        threshold=0.5, alpha=0.5, palette=si.DEFAULT_PALETTE, fp32_input=False,
                        tag=f"small-network/{nw}x{nh}/stream{j}")
    finally:
        s.close()
        hs.hs_shutdown(ctx)


@pytest.mark.parametrize("frame_w,frame_h,net_w,net_h,batch", [
    (64, 48, 130, 128, 8),       # 1024 rows: the longest launch of one round
    (64, 48, 130, 129, 8),       # beyond it: 256 threads
    (1367, 40, 300, 80, 13),     # rows of 257 vectors
    (5466, 40, 70, 80, 13),      # 1025 vectors: more than four for each of 256 threads, 320 are taken
])
def test_resize_of_many_rows_matches_the_oracle(hs, frame_w, frame_h, net_w, net_h, batch):
    from paper_2402_04466_amd.harness import AppStream
    blob = si.he_normal_blob(si.TINY4_LAYERS, 12)
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=frame_w, frame_h=frame_h, net_w=net_w, net_h=net_h, blob=blob,
                  palette=si.DEFAULT_PALETTE, queue_depth=2, batch=batch)
    try:
        print(f"[resize-rows] {frame_w}x{frame_h} -> {net_w}x{net_h} batch {batch}", flush=True)
        host = [si.uniform_frames(1, frame_h, frame_w, 80 + j)[0] for j in range(batch)]
        d_in, d_out = [s.upload_frame(f) for f in host], [s.new_output() for _ in host]
        assert s.submit_batch(d_in, d_out, 0) == hs.HS_OK
        rs = s.wait_batch()
        lut = oracle.normalize_lut(0.5, 0.25, fp16=True)
        for j in (0, batch - 1):
            o32, _ = make_oracles("tiny4", blob, net_w, net_h, True, si.DEFAULT_PALETTE)
            got = s.fetch(rs[j], d_out[j])["net_input"].astype(np.float32)
            assert np.array_equal(got[..., :3], lut[o32.process(host[j])["resized"]]), j
            assert np.all(got[..., 3] == 0), j
    finally:
        s.close()
        hs.hs_shutdown(ctx)
