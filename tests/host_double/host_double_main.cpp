// Host code of the library against the stand-in runtime: `host_double_main <check>` exits 0 when the
// check holds, prints what does not and exits 1 otherwise.
#include <math.h>
#include <sched.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>
#include <unistd.h>

#include <string>
#include <vector>

#include "fake_hip.h"
#include "hs.h"

#define CHECK(cond)                                                                \
  do {                                                                             \
    if (!(cond)) {                                                                 \
      printf("line %d: %s does not hold (%s)\n", __LINE__, #cond, hs_last_error()); \
      exit(1);                                                                     \
    }                                                                              \
  } while (0)

struct Program {   // what a program has in hand before it creates an application
  hs_ctx* ctx = nullptr;
  hs_app_desc d;
  std::vector<float> weights;
  void* workspace = nullptr;
  std::vector<uint8_t> frame, out;
  explicit Program(int net, int batch = 1, int net_w = 40, int net_h = 24) : frame(64 * 48 * 3 + 16), out(64 * 48 * 3 + 16) {
    CHECK(hs_init(0, &ctx) == HS_OK);
    memset(&d, 0, sizeof(d));
    d.frame_w = 64; d.frame_h = 48; d.frame_pitch = 192;
    d.net_w = net_w; d.net_h = net_h; d.net = net;
    d.mean = 0.5f; d.std = 0.25f; d.threshold = 0.5f; d.alpha = 0.5f;
    d.queue_depth = 2; d.batch = batch; d.glyph_scale = 1;
    size_t need = 0;
    CHECK(hs_query_workspace(&d, &need) == HS_OK);
    workspace = aligned_alloc(256, (need + 255) / 256 * 256);
    d.d_workspace = workspace; d.workspace_bytes = need;
    weights.assign(net == HS_NET_TINY4 ? 16 * 27 + 32 * 144 + 32 * 288 + 8 * 288 : 18246848, 0.01f);
    d.weights = weights.data(); d.weight_floats = weights.size();
  }
  const uint8_t* src() { return (const uint8_t*)(((uintptr_t)frame.data() + 15) & ~(uintptr_t)15); }
  uint8_t* dst() { return (uint8_t*)(((uintptr_t)out.data() + 15) & ~(uintptr_t)15); }
  ~Program() {
    CHECK(hs_shutdown(ctx) == HS_OK);
    free(workspace);
  }
};

// A packing thread whose own state cannot be allocated, or that the system refuses to start: the
// threads that there are do the work.
static void packing_threads() {
  Program p(HS_NET_RESNET18_CONVLSTM);
  hs_app* app = nullptr;
  fake::fail_block_after_thread_start = true;
  CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
  CHECK(hs_destroy_app(app) == HS_OK);
  fake::reset_failures();
  fake::threads_until_failure = 2;
  CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
  CHECK(hs_destroy_app(app) == HS_OK);
}

// Every allocation of a create call fails once, then every thread start: an error code, and nothing
// of the half-made application is left.
static void create_failures() {
  for (int threads = 0; threads < 2; ++threads) {
    Program p(HS_NET_TINY4);
    hs_app* first = nullptr;        // the context's list of applications has its storage from here on
    CHECK(hs_create_app(p.ctx, &p.d, &first) == HS_OK && hs_destroy_app(first) == HS_OK);
    const long objects = fake::live_objects, blocks = fake::live_blocks;
    for (long n = 0;; ++n) {
      hs_app* app = nullptr;
      (threads ? fake::threads_until_failure : fake::blocks_until_failure) = n;
      const hs_status st = hs_create_app(p.ctx, &p.d, &app);
      const bool reached = (threads ? fake::threads_until_failure : fake::blocks_until_failure) < 0;
      fake::reset_failures();
      if (!reached) {               // the call needs no more than n
        CHECK(st == HS_OK && n > 0);
        CHECK(hs_destroy_app(app) == HS_OK);
        break;
      }
      CHECK(st == HS_E_NOMEM || st == HS_E_DEVICE);
      CHECK(app == nullptr);
      CHECK(fake::live_objects == objects);
      CHECK(fake::live_blocks == blocks);
    }
  }
}

// The same for a group of three: no thread and no memory of it is left, and its members are free.
static void group_failures() {
  Program p(HS_NET_TINY4);
  Program p2(HS_NET_TINY4), p3(HS_NET_TINY4);
  hs_app* m[3];
  CHECK(hs_create_app(p.ctx, &p.d, &m[0]) == HS_OK);
  CHECK(hs_create_app(p.ctx, &p2.d, &m[1]) == HS_OK);
  CHECK(hs_create_app(p.ctx, &p3.d, &m[2]) == HS_OK);
  const long blocks = fake::live_blocks, running = fake::live_threads;
  for (int threads = 0; threads < 2; ++threads)
    for (long n = 0;; ++n) {
      hs_group* g = nullptr;
      (threads ? fake::threads_until_failure : fake::blocks_until_failure) = n;
      const hs_status st = hs_create_group(p.ctx, m, 3, &g);
      const bool reached = (threads ? fake::threads_until_failure : fake::blocks_until_failure) < 0;
      fake::reset_failures();
      if (!reached) {
        CHECK(st == HS_OK && n > 0);
        CHECK(hs_destroy_group(g) == HS_OK);
        break;
      }
      CHECK(st == HS_E_NOMEM || st == HS_E_DEVICE);
      CHECK(fake::live_blocks == blocks);
      CHECK(fake::live_threads == running);
    }
  for (hs_app* a : m) CHECK(hs_destroy_app(a) == HS_OK);
}

// A source whose thread cannot be started: the sources that run are seen to their end, the call
// reports it, and the applications can be used and destroyed.
static void feed_failures() {
  Program p(HS_NET_TINY4), p2(HS_NET_TINY4), p3(HS_NET_TINY4);
  Program* all[3] = {&p, &p2, &p3};
  hs_feed feeds[3];
  memset(feeds, 0, sizeof(feeds));
  const uint8_t* src[3];
  uint8_t* dst[3];
  hs_result out[3][4];
  hs_result* results[3];
  for (int i = 0; i < 3; ++i) {
    CHECK(hs_create_app(p.ctx, &all[i]->d, &feeds[i].app) == HS_OK);
    src[i] = all[i]->src(); dst[i] = all[i]->dst();
    feeds[i].d_frames = &src[i]; feeds[i].d_outs = &dst[i];
    feeds[i].n_frames = feeds[i].n_outs = feeds[i].batch = feeds[i].results_per_frame = 1;
    feeds[i].cpu = -1;
    results[i] = out[i];
  }
  for (long n = 0; n < 3; ++n) {
    fake::threads_until_failure = n;
    CHECK(hs_run_feeds(feeds, 3, 0.0, 4, results, nullptr, nullptr, nullptr) == HS_E_NOMEM);
    fake::reset_failures();
  }
  fake::fail_block_after_thread_start = true;
  CHECK(hs_run_feeds(feeds, 3, 0.0, 4, results, nullptr, nullptr, nullptr) == HS_E_NOMEM);
  fake::reset_failures();
  CHECK(hs_run_feeds(feeds, 3, 0.0, 4, results, nullptr, nullptr, nullptr) == HS_OK);
  for (hs_feed& f : feeds) CHECK(hs_destroy_app(f.app) == HS_OK);
}

// A feed that the caller's own thread drives leaves that thread as it was: its current device, and what its last failure was.
static void callers_thread() {
  Program p(HS_NET_TINY4);
  hs_feed feed;
  memset(&feed, 0, sizeof(feed));
  const uint8_t* src = p.src();
  uint8_t* dst = p.dst();
  hs_result out[4], *results = out;
  CHECK(hs_create_app(p.ctx, &p.d, &feed.app) == HS_OK);
  feed.d_frames = &src; feed.d_outs = &dst;
  feed.n_frames = feed.n_outs = feed.batch = feed.results_per_frame = 1;
  feed.cpu = -1;
  CHECK(hs_get_state(nullptr, 0, nullptr, nullptr) == HS_E_INVAL);
  const std::string before = hs_last_error();
  fake::device = 3;
  CHECK(hs_run_feeds(&feed, 1, 0.0, 4, &results, nullptr, nullptr, nullptr) == HS_OK);
  CHECK(before == hs_last_error() && fake::device == 3);
  feed.batch = 2;                            // more than the application takes: its submits fail
  const uint8_t* two[2] = {nullptr, nullptr};
  feed.d_frames = two;
  CHECK(hs_run_feeds(&feed, 1, 0.0, 4, &results, nullptr, nullptr, nullptr) == HS_E_INVAL);
  CHECK(strstr(hs_last_error(), "feed 0: hs_submit_batch: NULL frame pointer") && fake::device == 3);
  CHECK(hs_destroy_app(feed.app) == HS_OK);
}

// Every other call that allocates: a refused allocation is an error code.  A submit that fails after
// work has been handed over leaves an application that says so.
static void call_failures() {
  hs_ctx* ctx = nullptr;
  fake::blocks_until_failure = 0;
  CHECK(hs_init(0, &ctx) == HS_E_NOMEM && ctx == nullptr);
  fake::reset_failures();
  const double x[3] = {1, 2, 3};
  hs_latency_metrics lm;
  hs_mwu u;
  fake::blocks_until_failure = 0;
  CHECK(hs_latency_metrics_compute(x, 3, 0, &lm) == HS_E_NOMEM);
  fake::blocks_until_failure = 0;
  CHECK(hs_mann_whitney_u(x, 3, x, 3, &u) == HS_E_NOMEM);
  fake::reset_failures();

  Program p(HS_NET_RESNET18_CONVLSTM), p2(HS_NET_TINY4);
  hs_app *a = nullptr, *b = nullptr;
  hs_result r[2];
  CHECK(hs_create_app(p.ctx, &p.d, &a) == HS_OK && hs_create_app(p.ctx, &p2.d, &b) == HS_OK);
  CHECK(hs_submit_frame(a, p.src(), p.dst(), 0) == HS_OK && hs_wait_result(a, r, 1000000000) == HS_OK);
  std::vector<float> map((size_t)512 * r->map_w * r->map_h);
  fake::blocks_until_failure = 0;
  CHECK(hs_get_features(a, 0, map.data()) == HS_E_NOMEM);
  fake::blocks_until_failure = 0;
  CHECK(hs_get_state(a, 0, map.data(), nullptr) == HS_E_NOMEM);
  fake::blocks_until_failure = 0;
  CHECK(hs_get_state(a, 0, nullptr, map.data()) == HS_E_NOMEM);
  fake::reset_failures();
  CHECK(hs_set_kernel_timing(b, 1) == HS_OK);
  fake::blocks_until_failure = 1;
  CHECK(hs_submit_frame(b, p2.src(), p2.dst(), 0) == HS_E_NOMEM);
  fake::reset_failures();
  CHECK(hs_submit_frame(b, p2.src(), p2.dst(), 1) == HS_E_DEVICE);
  CHECK(strstr(hs_last_error(), "destroy the application"));
  CHECK(hs_destroy_app(b) == HS_OK && hs_destroy_app(a) == HS_OK);
}

// Every allocation of a call that sets or releases a partition fails once: nothing has changed then, neither claims nor the plan
// of any layer.
static void partition_failures() {
  Program p(HS_NET_RESNET18_CONVLSTM, 2, 427, 240), p2(HS_NET_TINY4);
  p.d.queue_depth = 2;
  hs_app *a = nullptr, *b = nullptr;
  CHECK(hs_create_app(p.ctx, &p.d, &a) == HS_OK && hs_create_app(p.ctx, &p2.d, &b) == HS_OK);
  uint32_t mask[8] = {0xffffffffu, 0xffffffffu, 0xffffu};     // 80 CUs
  const uint8_t* src[2] = {p.src(), p.src()};
  uint8_t* dst[2] = {p.dst(), p.dst()};
  hs_result r[2];
  auto plan = [&] {                          // of the launches of one batch in each lane
    fake::n_conv_launches = 0;
    for (int i = 0; i < 2; ++i) CHECK(hs_submit_batch(a, src, dst, 1) == HS_OK && hs_wait_batch(a, r, 1000000000) == HS_OK);
    std::vector<int> v;
    for (int i = 0; i < fake::n_conv_launches; ++i) {
      const hs::ConvParams& c = fake::conv_launches[i];
      for (int x : {c.run_form, c.tiles_m, c.tiles_n, c.tiles_per_xcd, c.n_block, c.run_nb_shift, (int)c.run_by_blk}) v.push_back(x);
    }
    return v;
  };
  const std::vector<int> whole = plan();
  std::vector<int> part;
  for (int release = 0; release < 2; ++release)
    for (long n = 0;; ++n) {
      fake::blocks_until_failure = n;
      const hs_status st = release ? hs_set_partition(a, nullptr, nullptr, 0) : hs_set_partition(a, mask, mask, 8);
      const bool reached = fake::blocks_until_failure < 0;
      fake::reset_failures();
      if (!reached) {
        CHECK(st == HS_OK && n > 10);
        break;
      }
      CHECK(st == HS_E_NOMEM && plan() == (release ? part : whole));
      CHECK(hs_set_partition(b, mask, mask, 8) == (release ? HS_E_OVERSUBSCRIBED : HS_OK));
      CHECK(hs_set_partition(b, nullptr, nullptr, 0) == HS_OK);
      if (!release && n == 0) {
        CHECK(hs_set_partition(a, mask, mask, 8) == HS_OK);
        part = plan();
        CHECK(part != whole && hs_set_partition(a, nullptr, nullptr, 0) == HS_OK && plan() == whole);
      }
    }
  CHECK(plan() == whole);
  CHECK(hs_destroy_app(b) == HS_OK && hs_destroy_app(a) == HS_OK);
}

// A mux whose allocations are refused, one after the other: a frame that is not taken can be handed
// over again, a result that cannot be fetched is still there at the next call, and every stream gets
// its own ids, in order.
static void mux_failures() {
  Program p(HS_NET_TINY4);
  p.d.batch = 2;
  size_t need = 0;
  CHECK(hs_query_workspace(&p.d, &need) == HS_OK);
  void* workspace = aligned_alloc(256, (need + 255) / 256 * 256);
  p.d.d_workspace = workspace; p.d.workspace_bytes = need;
  hs_app* app = nullptr;
  CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
  fake::event_wait_ns = 200000;
  for (int waiting = 0; waiting < 2; ++waiting)
    for (long n = 0; n < 40; ++n) {
      hs_mux* mux = nullptr;
      CHECK(hs_create_mux(app, 2, &mux) == HS_OK);
      hs_result r;
      bool refused = false;
      // calls f until it no longer lacks memory; its n-th allocation over the frames is refused
      auto insist = [&](auto f) {
        hs_status st;
        while ((st = f()) == HS_E_NOMEM) { CHECK(!refused); refused = true; }
        return st;
      };
      fake::blocks_until_failure = n;
      for (uint64_t k = 0; k < 3; ++k) {
        CHECK(insist([&] { return hs_mux_submit(mux, 0, p.src(), p.dst(), 100 + k); }) == HS_OK);
        CHECK(insist([&] { return hs_mux_submit(mux, 1, p.src(), p.dst(), 200 + k); }) == HS_OK);
        for (int stream = 0; stream < 2; ++stream) {
          hs_status st;
          do {
            st = insist([&] {
              return waiting ? hs_mux_wait(mux, stream, &r, 1000000000) : hs_mux_poll(mux, stream, &r);
            });
          } while (!waiting && st == HS_E_NOT_READY);
          CHECK(st == HS_OK && r.frame_id == (stream ? 200 : 100) + k);
        }
      }
      fake::reset_failures();
      CHECK(hs_destroy_mux(mux) == HS_OK);
    }
  fake::event_wait_ns = 0;
  CHECK(hs_destroy_app(app) == HS_OK);
  free(workspace);
}

// A thread confined to one core sleeps in hs_wait_* and hs_wait_group: the completion thread may be
// pinned to that core.
static void pinned_wait() {
  Program p(HS_NET_TINY4);
  hs_app* app = nullptr;
  CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
  cpu_set_t all, one;
  CHECK(sched_getaffinity(0, sizeof(all), &all) == 0);
  int cpu = 0;
  while (!CPU_ISSET(cpu, &all)) ++cpu;
  CPU_ZERO(&one);
  CPU_SET(cpu, &one);
  CHECK(sched_setaffinity(0, sizeof(one), &one) == 0);
  fake::event_wait_ns = 900000;
  auto clock_ns = [](clockid_t c) {
    timespec t;
    clock_gettime(c, &t);
    return t.tv_sec * 1000000000ll + t.tv_nsec;
  };
  hs_group* group = nullptr;
  for (int grouped = 0; grouped < 2; ++grouped) {
    if (grouped) CHECK(hs_create_group(p.ctx, &app, 1, &group) == HS_OK);
    const long long wall = clock_ns(CLOCK_MONOTONIC), busy = clock_ns(CLOCK_THREAD_CPUTIME_ID);
    hs_result r;
    for (uint64_t k = 0; k < 40; ++k) {
      if (grouped) {
        CHECK(hs_submit_group(group, p.src(), p.dst(), k) == HS_OK);
        CHECK(hs_wait_group(group, &r, 1000000000) == HS_OK);
      } else {
        CHECK(hs_submit_frame(app, p.src(), p.dst(), k) == HS_OK);
        CHECK(hs_wait_result(app, &r, 1000000000) == HS_OK);
      }
    }
    // 36 ms of waiting at least
    CHECK(4 * (clock_ns(CLOCK_THREAD_CPUTIME_ID) - busy) < clock_ns(CLOCK_MONOTONIC) - wall);
  }
  fake::event_wait_ns = 0;
  CHECK(hs_destroy_group(group) == HS_OK);
  CHECK(hs_destroy_app(app) == HS_OK);
}

// A result that is there already is delivered without a system call, a later frame in flight or not.
static void ready_result() {
  Program p(HS_NET_TINY4);
  hs_app* app = nullptr;
  CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
  hs_result r;
  for (uint64_t k = 0; k < 5; ++k) {
    fake::event_wait_ns = 0;
    CHECK(hs_submit_frame(app, p.src(), p.dst(), 2 * k) == HS_OK);
    usleep(50000);                       // its completion has been noted
    fake::event_wait_ns = 50000000;
    CHECK(hs_submit_frame(app, p.src(), p.dst(), 2 * k + 1) == HS_OK);
    const long queries = fake::mask_queries;
    CHECK(hs_wait_result(app, &r, 1000000000) == HS_OK && r.frame_id == 2 * k);
    CHECK(fake::mask_queries == queries);
    CHECK(hs_wait_result(app, &r, 1000000000) == HS_OK && r.frame_id == 2 * k + 1);
  }
  fake::event_wait_ns = 0;
  CHECK(hs_destroy_app(app) == HS_OK);
}

// A time-out as long as its type allows is no time-out of the past.
static void endless_wait() {
  Program p(HS_NET_TINY4);
  hs_app* app = nullptr;
  CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
  fake::event_wait_ns = 5000000;
  hs_result r;
  for (uint64_t timeout : {UINT64_MAX, UINT64_MAX / 2, UINT64_MAX / 2 + 1}) {
    CHECK(hs_submit_frame(app, p.src(), p.dst(), 1) == HS_OK);
    CHECK(hs_wait_result(app, &r, timeout) == HS_OK);
    hs_mux* mux = nullptr;
    CHECK(hs_create_mux(app, 1, &mux) == HS_OK);
    CHECK(hs_mux_submit(mux, 0, p.src(), p.dst(), 1) == HS_OK);
    CHECK(hs_mux_wait(mux, 0, &r, timeout) == HS_OK);
    CHECK(hs_destroy_mux(mux) == HS_OK);
    hs_group* group = nullptr;
    CHECK(hs_create_group(p.ctx, &app, 1, &group) == HS_OK);
    CHECK(hs_submit_group(group, p.src(), p.dst(), 1) == HS_OK);
    CHECK(hs_wait_group(group, &r, timeout) == HS_OK);
    CHECK(hs_destroy_group(group) == HS_OK);
  }
  CHECK(hs_wait_result(app, &r, 1000000) == HS_E_NOT_READY);
  CHECK(hs_wait_result(app, &r, 0) == HS_E_NOT_READY);
  fake::event_wait_ns = 0;
  CHECK(hs_destroy_app(app) == HS_OK);
}

// A kernel is told to prefetch the next layer's weights only if it does so (k_conv3x3_run, k_conv3x3s2_run), and then
// exactly those that the layer has.
static void prefetched_weights() {
  for (int net : {(int)HS_NET_TINY4, (int)HS_NET_RESNET18_CONVLSTM}) {
    Program p(net, 2);
    hs_app* app = nullptr;
    CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
    fake::n_conv_launches = 0;
    const uint8_t* src[2] = {p.src(), p.src()};
    uint8_t* dst[2] = {p.dst(), p.dst()};
    hs_result r[2];
    CHECK(hs_submit_batch(app, src, dst, 1) == HS_OK && hs_wait_batch(app, r, 1000000000) == HS_OK);
    const int n = fake::n_conv_launches;
    CHECK(n > 0 && n < fake::kMaxConvLaunches);
    int told = 0;
    for (int i = 0; i < n; ++i) {
      const hs::ConvParams& a = fake::conv_launches[i];
      if (a.next_lines == 0) continue;
      ++told;
      CHECK(a.variant == hs::CONV_KW && i + 1 < n);
      const hs::ConvParams& b = fake::conv_launches[i + 1];
      CHECK(a.next_wt == b.wt_frag);
      CHECK((size_t)a.next_lines * 128 ==
            (size_t)(b.variant == hs::CONV_DIRECT ? 32 : b.cout_pad) * b.ktot * sizeof(hs::f16));
    }
    CHECK((told > 0) == (net != HS_NET_TINY4));
    CHECK(hs_destroy_app(app) == HS_OK);
  }
}

// A frame or batch that finds its application idle is one launch per layer, all in one stream, whatever its size: its tensors
// share their buffers from stage to stage, and a second queue of this process would slow down other processes' on the device.
static void one_queue_alone() {
  const struct { int w, h, batch; bool annotate; } sizes[] = {{854, 480, 1, false}, {854, 480, 3, false}, {820, 300, 5, true}, {300, 256, 16, false}};
  for (const auto& z : sizes) {
    Program p(HS_NET_RESNET18_CONVLSTM, z.batch, z.w, z.h);
    p.d.annotate = z.annotate;
    size_t need = 0;
    CHECK(hs_query_workspace(&p.d, &need) == HS_OK);
    free(p.workspace);
    p.workspace = aligned_alloc(256, (need + 255) / 256 * 256);
    p.d.d_workspace = p.workspace; p.d.workspace_bytes = need;
    hs_app* app = nullptr;
    CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
    std::vector<const uint8_t*> src((size_t)z.batch, p.src());
    std::vector<uint8_t*> dst((size_t)z.batch, p.dst());
    std::vector<hs_result> r((size_t)z.batch);
    for (int i = 0; i < 3; ++i) {
      fake::n_launches = 0;
      CHECK(hs_submit_batch(app, src.data(), dst.data(), 1) == HS_OK && hs_wait_batch(app, r.data(), 1000000000) == HS_OK);
      CHECK(fake::n_launches == (z.annotate ? 20 : 19));
      for (int k = 1; k < fake::n_launches; ++k) CHECK(fake::launch_streams[k] == fake::launch_streams[0]);
    }
    CHECK(hs_destroy_app(app) == HS_OK);
  }
}

// Of the grid of a layer in tiles of consecutive pixels every tile is one workgroup's, and what the surplus workgroups load
// lies inside the layer's tensors as well.
static void tile_grids() {
  const int sizes[][3] = {{8, 8, 1}, {40, 24, 1}, {130, 66, 6}, {96, 64, 1}, {288, 160, 5}, {300, 170, 16}, {40, 520, 2}};
  long surplus = 0;
  for (const auto& z : sizes) {
    Program p(HS_NET_RESNET18_CONVLSTM, z[2], z[0], z[1]);
    hs_app* app = nullptr;
    CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
    fake::n_conv_launches = 0;
    std::vector<const uint8_t*> src((size_t)z[2], p.src());
    std::vector<uint8_t*> dst((size_t)z[2], p.dst());
    std::vector<hs_result> r((size_t)z[2]);
    CHECK(hs_submit_batch(app, src.data(), dst.data(), 1) == HS_OK && hs_wait_batch(app, r.data(), 1000000000) == HS_OK);
    int run = 0;
    for (int i = 0; i < fake::n_conv_launches; ++i) {
      const hs::ConvParams& c = fake::conv_launches[i];
      if (c.variant != hs::CONV_KW) continue;
      ++run;
      std::vector<int> seen((size_t)(c.tiles_m * c.tiles_n));
      const int channels = c.cout / c.tiles_n;
      CHECK(8 * c.tiles_per_xcd >= c.tiles_m * c.tiles_n);
      for (uint32_t t = 0; t < 8u * (uint32_t)c.tiles_per_xcd; ++t) {
        const hs::RunTile at = hs::run_tile(t, c.tiles_m, c.tiles_n, c.n_block, c.run_nb_shift, c.run_by_blk);
        CHECK(at.run < (uint32_t)c.tiles_m && at.channels < (uint32_t)c.tiles_n);
        // the last byte of the tile's weights: chunks x 36 KB per 32 channels, and 4 KB of the projection's
        const uint64_t groups = (uint64_t)(at.channels + 1) * (uint64_t)channels / 32;
        CHECK(groups * (uint64_t)c.chunks_per_tap * 36 * 1024 <= c.run_w_bytes);
        CHECK(groups * (uint64_t)c.chunks_per_tap * 4 * 1024 <= c.run_w_bytes / 9);
        if (t < seen.size()) ++seen[(size_t)(at.run * (uint32_t)c.tiles_n + at.channels)];
        else ++surplus;
      }
      for (int n : seen) CHECK(n == 1);
    }
    CHECK(run > 10);
    CHECK(hs_destroy_app(app) == HS_OK);
  }
  CHECK(surplus > 0);
}

// The small network runs in one launch where that is the faster form, measured at these sizes, and else layer by layer.
static void small_network_forms() {
  const struct { int w, h, batch; bool one; } sizes[] = {
      {128, 128, 1, true},   {320, 320, 8, true},   {320, 320, 16, true},  {1280, 720, 1, true}, {4000, 16, 4, true},
      {300, 200, 16, false}, {640, 360, 8, false},  {4000, 16, 8, false},  {16, 4000, 16, false}, {1448, 1448, 1, false}};
  for (const auto& z : sizes) {
    Program p(HS_NET_TINY4, z.batch, z.w, z.h);
    hs_app* app = nullptr;
    CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
    fake::n_conv_launches = 0;
    std::vector<const uint8_t*> src((size_t)z.batch, p.src());
    std::vector<uint8_t*> dst((size_t)z.batch, p.dst());
    std::vector<hs_result> r((size_t)z.batch);
    CHECK(hs_submit_batch(app, src.data(), dst.data(), 1) == HS_OK && hs_wait_batch(app, r.data(), 1000000000) == HS_OK);
    CHECK(fake::n_conv_launches == (z.one ? 1 : 4));
    CHECK(fake::conv_launches[0].variant == (z.one ? hs::CONV_TINY_NET : hs::CONV_DIRECT));
    CHECK(hs_destroy_app(app) == HS_OK);
  }
}

// A frame that comes alone ends with the drawing or, on a large map, with the last channel maximum: whichever is later.
static void end_of_a_frame() {
  Program p(HS_NET_TINY4);
  hs_app* app = nullptr;
  CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK);
  const struct { uint64_t drawn; int32_t maxima; double infer_us, post_us; } ends[] = {{500, 300, 6, 3}, {500, 2000, 20, 0}, {500, 550, 6, 0.5}};
  for (const auto& z : ends) {
    fake::overlay_drawn = z.drawn; fake::overlay_maxima = z.maxima;
    hs_result r;
    CHECK(hs_submit_frame(app, p.src(), p.dst(), 1) == HS_OK && hs_wait_result(app, &r, 1000000000) == HS_OK);
    auto from_end = [&](uint64_t t) { return 1e-3 * (double)(r.t_overlay_done_ns - t); };
    CHECK(fabs(from_end(r.t_infer_done_ns) - z.infer_us) < 0.1 && fabs(from_end(r.t_post_done_ns) - z.post_us) < 0.1);
    CHECK(fabs(from_end(r.t_pre_done_ns) - from_end(r.t_infer_done_ns) - 1000) < 0.1);
  }
  CHECK(hs_destroy_app(app) == HS_OK);
}

// While kernels are timed, the launches that every other frame makes of the small network are timed, too: with stage 1, where
// that is the faster form, and without.
static void timed_small_network() {
  Program p(HS_NET_TINY4);
  hs_app* app = nullptr;
  CHECK(hs_create_app(p.ctx, &p.d, &app) == HS_OK && hs_set_kernel_timing(app, 1) == HS_OK);
  hs_result r;
  for (int i = 0; i < 2; ++i)
    CHECK(hs_submit_frame(app, p.src(), p.dst(), (uint64_t)i) == HS_OK && hs_wait_result(app, &r, 1000000000) == HS_OK);
  hs_kernel_time t[16];
  int n = 0, net = 0, layers = 0, frame_net = 0;
  CHECK(hs_get_kernel_times(app, t, 16, &n) == HS_OK && n <= 16);
  for (int i = 0; i < n; ++i) {
    if (!strcmp(t[i].name, "tiny_net_mfma")) net = (int)t[i].launches;
    if (!strcmp(t[i].name, "conv_mfma")) layers = (int)t[i].launches;
    if (!strcmp(t[i].name, "frame_net_mfma")) {
      frame_net = (int)t[i].launches;
      CHECK(t[i].flops > 0 && t[i].bytes > 0);
    }
  }
  CHECK(net == 2 && layers == 8 && frame_net == 2);
  CHECK(hs_destroy_app(app) == HS_OK);
}

int main(int argc, char** argv) {
  const std::string check = argc > 1 ? argv[1] : "";
  if (check == "packing_threads") packing_threads();
  else if (check == "create_failures") create_failures();
  else if (check == "group_failures") group_failures();
  else if (check == "feed_failures") feed_failures();
  else if (check == "call_failures") call_failures();
  else if (check == "mux_failures") mux_failures();
  else if (check == "pinned_wait") pinned_wait();
  else if (check == "ready_result") ready_result();
  else if (check == "endless_wait") endless_wait();
  else if (check == "prefetched_weights") prefetched_weights();
  else if (check == "tile_grids") tile_grids();
  else if (check == "one_queue_alone") one_queue_alone();
  else if (check == "end_of_a_frame") end_of_a_frame();
  else if (check == "partition_failures") partition_failures();
  else if (check == "callers_thread") callers_thread();
  else if (check == "small_network_forms") small_network_forms();
  else if (check == "timed_small_network") timed_small_network();
  else { printf("no check named '%s'\n", check.c_str()); return 2; }
  return 0;
}
