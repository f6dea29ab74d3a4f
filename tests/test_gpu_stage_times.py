"""The time stamps of a frame's stages on the GPU: stage 3 ends after stage 2 and no later than the
overlay, also where its channel maxima have no launch of their own (on a small frame the drawing may be
done before them: both stages then end together)."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

_LAYERS = {"tiny4": si.TINY4_LAYERS, "resnet18_convlstm": si.RESNET18_CONVLSTM_LAYERS}


def _app(hs, ctx, net, **kw):
    from paper_2402_04466_amd.harness import AppStream
    return AppStream(ctx, net=hs.HS_NET_TINY4 if net == "tiny4" else hs.HS_NET_RESNET18_CONVLSTM, frame_w=640,
                     frame_h=360, net_w=128, net_h=96, blob=si.he_normal_blob(_LAYERS[net], 5),
                     palette=si.DEFAULT_PALETTE, **kw)


def _check(results):
    for r in results:
        assert r.t_submit_ns <= r.t_pre_done_ns < r.t_infer_done_ns < r.t_post_done_ns <= r.t_overlay_done_ns, \
            [r.t_pre_done_ns - r.t_submit_ns, r.t_infer_done_ns - r.t_pre_done_ns,
             r.t_post_done_ns - r.t_infer_done_ns, r.t_overlay_done_ns - r.t_post_done_ns]


@pytest.mark.parametrize("net,batch,depth,mode,annotate,timing", [
    ("tiny4", 1, 2, "eager", False, False),
    ("resnet18_convlstm", 1, 2, "eager", False, False),
    ("resnet18_convlstm", 3, 3, "eager", False, False),   # an odd depth: the overlay has a stream of its own
    ("resnet18_convlstm", 1, 2, "graph", False, False),
    ("tiny4", 1, 2, "eager", True, False),                # maxima in a launch of their own
    ("tiny4", 1, 2, "eager", False, True),
])
def test_stage_three_ends_between_its_neighbours(hs, net, batch, depth, mode, annotate, timing):
    ctx = hs.hs_init(0)
    s = _app(hs, ctx, net, batch=batch, queue_depth=depth, glyphs=si.DEFAULT_GLYPHS if annotate else None)
    try:
        hs.hs_set_launch_mode(s.app, hs.HS_LAUNCH_GRAPH if mode == "graph" else hs.HS_LAUNCH_EAGER)
        if timing:
            hs.hs_set_kernel_timing(s.app, True)
        frames = list(si.uniform_frames(batch, 360, 640, 3))
        d_in, d_out = [s.upload_frame(f) for f in frames], [s.new_output() for _ in frames]
        for i in range(4):
            print(f"[stage-times] {net} batch {batch} depth {depth} {mode} frame {i}", flush=True)
            assert s.submit_batch(d_in, d_out, i) == hs.HS_OK
            _check(s.wait_batch())
    finally:
        s.close()
        hs.hs_shutdown(ctx)


@pytest.mark.parametrize("timed", [None, 0, 1])
def test_stage_three_of_a_group(hs, timed):
    """One overlay launch finds every member's maxima; also while one member's kernels are timed."""
    from paper_2402_04466_amd.harness import GroupStream
    ctx = hs.hs_init(0)
    members = [_app(hs, ctx, net, queue_depth=2) for net in ("tiny4", "resnet18_convlstm")]
    grp = GroupStream(ctx, members)
    try:
        if timed is not None:
            hs.hs_set_kernel_timing(members[timed].app, True)
        d_in, d_out = members[0].upload_frame(next(iter(si.uniform_frames(1, 360, 640, 4)))), members[0].new_output()
        for i in range(3):
            print(f"[stage-times] group, timed member {timed}, frame {i}", flush=True)
            assert grp.submit(d_in, d_out, i) == hs.HS_OK
            _check(grp.wait_batch())
    finally:
        grp.close()
        hs.hs_shutdown(ctx)


@pytest.mark.parametrize("net,depth", [("tiny4", 2), ("resnet18_convlstm", 2), ("resnet18_convlstm", 3),
                                       ("resnet18_convlstm", 4)])
def test_frames_alone_and_in_flight(hs, net, depth):
    """A frame that comes alone leaves the next one, in another lane, another event to wait for than a frame in flight
    does: mixed, the stages end in order and the frames are those of a stream whose every frame comes alone."""
    ctx = hs.hs_init(0)
    mixed, alone = _app(hs, ctx, net, queue_depth=depth), _app(hs, ctx, net, queue_depth=depth)
    runs = [1, 2, 1, min(3, depth), depth, 1, 2]
    try:
        frames = list(si.uniform_frames(sum(runs), 360, 640, 9))
        d_in = [mixed.upload_frame(f) for f in frames]
        got, want = [mixed.new_output() for _ in frames], [alone.new_output() for _ in frames]
        for i, out in enumerate(want):
            assert alone.submit_batch([d_in[i]], [out], i) == hs.HS_OK
            alone.wait_batch()
        i = 0
        for n in runs:
            print(f"[stage-times] {net} depth {depth}: {n} frames from {i}", flush=True)
            for j in range(i, i + n):
                assert mixed.submit_batch([d_in[j]], [got[j]], j) == hs.HS_OK
            for _ in range(n):
                _check(mixed.wait_batch())
            i += n
        for i, (a, b) in enumerate(zip(got, want)):
            assert (a == b).all(), i
    finally:
        mixed.close()
        alone.close()
        hs.hs_shutdown(ctx)
