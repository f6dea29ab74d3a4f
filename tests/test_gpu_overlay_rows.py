"""Stage 4 where a frame row does not end on a group of 16 pixels: rows shorter than a group, one
pixel short of and past a group's end, wavefronts that cross row ends, rows with padding behind
them.  Bit-exact against the oracle's overlay of the GPU's own mask (and its annotations); the
output's padding bytes stay untouched."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fw,fh,extra_pitch,net,annotate", [
    (1, 1, 0, "tiny4", False),
    (15, 9, 0, "tiny4", True),
    (16, 70, 16, "tiny4", False),
    (17, 5, 32, "tiny4", False),
    (335, 33, 0, "tiny4", True),
    (337, 200, 48, "resnet18_convlstm", False),
    (1279, 31, 0, "resnet18_convlstm", True),
])
def test_overlay_row_ends(hs, fw, fh, extra_pitch, net, annotate):
    from paper_2402_04466_amd.harness import AppStream
    tiny = net == "tiny4"
    pitch = (3 * fw + 15) // 16 * 16 + extra_pitch
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4 if tiny else hs.HS_NET_RESNET18_CONVLSTM, frame_w=fw,
                  frame_h=fh, net_w=96 if not tiny else 40, net_h=64 if not tiny else 24,
                  blob=si.he_normal_blob(si.TINY4_LAYERS if tiny else si.RESNET18_CONVLSTM_LAYERS, 11),
                  palette=si.DEFAULT_PALETTE, frame_pitch=pitch, alpha=0.37,
                  glyphs=si.DEFAULT_GLYPHS if annotate else None, marker_arm=5, marker_half=1,
                  glyph_scale=1)
    try:
        for i, f in enumerate(si.uniform_frames(2, fh, fw, 12)):
            print(f"[overlay-rows] {fw}x{fh} pitch {pitch} {net} frame {i}", flush=True)
            d_in, d_out = s.upload_frame(f), s.new_output()
            d_out.fill_(0xA5)
            torch.cuda.synchronize()
            assert s.submit(d_in, d_out, i) == hs.HS_OK
            g = s.fetch(s.wait(), d_out)
            want = oracle.overlay(f, g["mask"], si.DEFAULT_PALETTE, 0.37)
            if annotate:
                want = oracle.annotate(want, g["argmax_idx"], g["present"], g["mask"].shape[2],
                                       g["mask"].shape[1], si.DEFAULT_PALETTE, si.DEFAULT_GLYPHS, 5, 1, 1)
            assert np.array_equal(g["overlay"], want)
            p = oracle.postprocess(g["logits"], 0.5)
            for key in ("mask", "argmax_idx", "present"):
                assert np.array_equal(g[key], p[key]), key
            assert np.abs(g["heat"] - p["heat"]).max() <= 1e-6
            assert np.abs(g["peak"] - p["peak"]).max() <= 1e-6
            assert bool((d_out[:, 3 * fw:] == 0xA5).all()), "row padding was written"
    finally:
        s.close()
        hs.hs_shutdown(ctx)


@pytest.mark.parametrize("arm,half,scale", [
    (0, 0, 1),      # a single pixel and its label
    (0, 3, 1),      # bars thicker than long: the vertical bar is the wider one
    (3, 8, 2),
    (4, 4, 1),
    (64, 8, 8),     # the largest
])
def test_marker_shapes(hs, arm, half, scale):
    """Cross-hair and label of every accepted shape, bit-exact against the oracle's, in rows that end
    inside a group of 16 pixels."""
    from paper_2402_04466_amd.harness import AppStream
    fw, fh = 335, 201
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=fw, frame_h=fh, net_w=40, net_h=24,
                  blob=si.he_normal_blob(si.TINY4_LAYERS, 11), palette=si.DEFAULT_PALETTE, alpha=0.37,
                  glyphs=si.DEFAULT_GLYPHS, marker_arm=arm, marker_half=half, glyph_scale=scale)
    try:
        for i, f in enumerate(si.uniform_frames(2, fh, fw, 13)):
            print(f"[marker-shapes] arm {arm} half {half} scale {scale} frame {i}", flush=True)
            d_in, d_out = s.upload_frame(f), s.new_output()
            assert s.submit(d_in, d_out, i) == hs.HS_OK
            g = s.fetch(s.wait(), d_out)
            assert g["present"].any()
            want = oracle.annotate(oracle.overlay(f, g["mask"], si.DEFAULT_PALETTE, 0.37), g["argmax_idx"],
                                   g["present"], g["mask"].shape[2], g["mask"].shape[1], si.DEFAULT_PALETTE,
                                   si.DEFAULT_GLYPHS, arm, half, scale)
            assert np.array_equal(g["overlay"], want)
    finally:
        s.close()
        hs.hs_shutdown(ctx)


@pytest.mark.parametrize("fw,fh,extra_pitch,net_w,net_h,batch,annotate", [
    (1023, 767, 0, 96, 64, 1, True),      # 49 088 groups of 16 pixels: quads
    (1023, 768, 0, 96, 64, 1, True),      # 49 152: groups of 16
    (1030, 378, 16, 64, 64, 2, True),     # 49 140, padded rows that end inside a word
    (1021, 385, 16, 64, 64, 2, True),     # 49 280
    (360, 67, 0, 96, 64, 1, False),       # 24 cells of 15 pixels
    (359, 67, 0, 96, 64, 1, False),       # cells of less than 15: quads on any frame
    (359, 460, 32, 96, 64, 5, True),
    (361, 460, 32, 96, 64, 5, True),
    (13, 7, 0, 96, 64, 2, False),         # more cells than pixels
])
def test_overlay_forms(hs, fw, fh, extra_pitch, net_w, net_h, batch, annotate):
    """Both sides of the lines between the overlay's two forms, several images per launch; bit-exact as above."""
    from paper_2402_04466_amd.harness import AppStream
    pitch = (3 * fw + 15) // 16 * 16 + extra_pitch
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=fw, frame_h=fh, net_w=net_w, net_h=net_h, batch=batch,
                  blob=si.he_normal_blob(si.TINY4_LAYERS, 11), palette=si.DEFAULT_PALETTE, frame_pitch=pitch, alpha=0.61,
                  glyphs=si.DEFAULT_GLYPHS if annotate else None, marker_arm=9, marker_half=1, glyph_scale=3)
    try:
        frames = list(si.uniform_frames(batch, fh, fw, 21))
        print(f"[overlay-forms] {fw}x{fh} pitch {pitch} batch {batch}", flush=True)
        d_in, d_out = [s.upload_frame(f) for f in frames], [s.new_output() for _ in frames]
        for o in d_out:
            o.fill_(0xA5)
        torch.cuda.synchronize()
        assert s.submit_batch(d_in, d_out, 0) == hs.HS_OK
        for f, r, o in zip(frames, s.wait_batch(), d_out):
            g = s.fetch(r, o)
            want = oracle.overlay(f, g["mask"], si.DEFAULT_PALETTE, 0.61)
            if annotate:
                want = oracle.annotate(want, g["argmax_idx"], g["present"], g["mask"].shape[2],
                                       g["mask"].shape[1], si.DEFAULT_PALETTE, si.DEFAULT_GLYPHS, 9, 1, 3)
            assert np.array_equal(g["overlay"], want)
            assert bool((o[:, 3 * fw:] == 0xA5).all()), "row padding was written"
    finally:
        s.close()
        hs.hs_shutdown(ctx)
