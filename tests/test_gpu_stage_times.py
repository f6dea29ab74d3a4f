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


@pytest.mark.parametrize("frame_w,frame_h,net_w,net_h", [(1920, 1080, 640, 360), (1920, 1080, 480, 270)])   # drawn in quads, in groups of 16
def test_the_last_stage_waits_for_the_maxima(hs, frame_w, frame_h, net_w, net_h):
    """On a large map the search for the channels' maxima, in the overlay's launch, takes longer than the drawing, as long as it does in
    a launch of its own while kernels are timed.  Allowed: a fifth of that, and 2 us for the stamps and that launch's boundary."""
    from paper_2402_04466_amd.harness import AppStream
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=frame_w, frame_h=frame_h, net_w=net_w, net_h=net_h, queue_depth=2,
                  blob=si.he_normal_blob(si.TINY4_LAYERS, 5), palette=si.DEFAULT_PALETTE)
    try:
        d_in, d_out = s.upload_frame(next(iter(si.uniform_frames(1, frame_h, frame_w, 6)))), s.new_output()

        def steps(n):
            after = []
            for i in range(n):
                assert s.submit(d_in, d_out, i) == hs.HS_OK
                r = s.wait()
                _check([r])
                after.append((r.t_overlay_done_ns - r.t_infer_done_ns) / 1e3)
            return sorted(after)[n // 2]
        steps(4)
        hs.hs_set_kernel_timing(s.app, True)
        steps(8)
        times = {k["name"]: 1e3 * k["total_ms"] / 8 for k in hs.hs_get_kernel_times(s.app)}
        hs.hs_set_kernel_timing(s.app, False)
        after = steps(9)
        print(f"[stage-times] {frame_w}x{frame_h}, net {net_w}x{net_h}: kernels {times}, stage 2 ends {after:.1f} us before the frame", flush=True)
        assert after >= 0.8 * max(times["overlay"], times["postprocess"]) - 2
    finally:
        s.close()
        hs.hs_shutdown(ctx)


@pytest.mark.parametrize("frame_w,frame_h,batch,depth,mode,annotate", [
    (1920, 1080, 1, 2, "eager", False),    # drawn by workgroups that are all there at once
    (1920, 1080, 2, 2, "eager", False),
    (1920, 1080, 1, 2, "eager", True),
    (320, 240, 1, 2, "eager", True),       # a few workgroups, of which those that paint take far longer
    (7680, 4320, 1, 2, "eager", False),    # and in many rounds
    (7680, 4320, 1, 2, "eager", True),
    (7680, 4320, 1, 3, "eager", False),    # the overlay on a stream of its own
    (3840, 2160, 4, 2, "eager", True),
    (7680, 4320, 1, 2, "graph", True),
])
def test_the_last_stage_is_as_long_as_the_drawing(hs, frame_w, frame_h, batch, depth, mode, annotate):
    """What lies between the ends of the stages before the overlay and the frame's end is the overlay kernel, as kernel
    timing measures it.  Allowed: a fifth of it (clocks and bandwidth differ from run to run), 2 us for the stamps and, above
    it, 12 us for the gaps between launches and events."""
    from paper_2402_04466_amd.harness import AppStream
    ctx = hs.hs_init(0)
    s = AppStream(ctx, net=hs.HS_NET_TINY4, frame_w=frame_w, frame_h=frame_h, net_w=128, net_h=96, batch=batch,
                  queue_depth=depth, blob=si.he_normal_blob(si.TINY4_LAYERS, 5), palette=si.DEFAULT_PALETTE,
                  glyphs=si.DEFAULT_GLYPHS if annotate else None)
    try:
        hs.hs_set_launch_mode(s.app, hs.HS_LAUNCH_GRAPH if mode == "graph" else hs.HS_LAUNCH_EAGER)
        frames = list(si.uniform_frames(batch, frame_h, frame_w, 6))
        d_in, d_out = [s.upload_frame(f) for f in frames], [s.new_output() for _ in frames]

        def step(i):
            assert s.submit_batch(d_in, d_out, i) == hs.HS_OK
            return s.wait_batch()
        for i in range(4):
            step(i)
        hs.hs_set_kernel_timing(s.app, True)
        for i in range(8):
            step(4 + i)
        times = {k["name"]: 1e3 * k["total_ms"] / 8 for k in hs.hs_get_kernel_times(s.app)}
        hs.hs_set_kernel_timing(s.app, False)
        draw = times["overlay"]
        after = {"pre": [], "infer": [], "post": []}
        for i in range(9):
            r = step(12 + i)[0]
            _check([r])
            for k, t in (("pre", r.t_pre_done_ns), ("infer", r.t_infer_done_ns), ("post", r.t_post_done_ns)):
                after[k].append((r.t_overlay_done_ns - t) / 1e3)
        after = {k: sorted(v)[4] for k, v in after.items()}
        print(f"[stage-times] {frame_w}x{frame_h} {mode} batch {batch} depth {depth} annotate {annotate}: overlay kernel "
              f"{draw:.1f} us, ends before the frame's {after}, kernels {times}", flush=True)
        assert 0.8 * draw - 2 <= after["infer"] <= 1.2 * draw + times["postprocess"] + 12
        assert after["pre"] - after["infer"] <= 1.2 * times["conv_mfma"] + 12
        if annotate:                                      # stage 3 has a launch of its own, the drawing follows it
            assert 0.8 * draw - 2 <= after["post"] <= 1.2 * draw + 12
        elif draw > 25:                                   # the maxima are found by the launch's first workgroups
            assert after["post"] >= 0.3 * draw
    finally:
        s.close()
        hs.hs_shutdown(ctx)
