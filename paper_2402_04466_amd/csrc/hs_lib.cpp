// libhs host runtime: contexts, applications, the per-frame launch plan, CU-masked stream
// partitions with admission control, per-frame time stamps and the completion thread.
// Paper: Section III-A (application and its four stages), Section II-C (time stamps at the
// first and last stage), Section IV-A (exclusive partitions, admission control).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <exception>
#include <functional>
#include <memory>
#include <mutex>
#include <new>
#include <stdexcept>
#include <thread>
#include <pthread.h>
#include <sched.h>
#include <time.h>
#include <unistd.h>
#include <vector>

#include "hs.h"
#include "hs_internal.h"
#include "hs_kernels.h"

namespace hs {

#define HS_HIP(call)                                                                   \
  do {                                                                                 \
    hipError_t e_ = (call);                                                            \
    if (e_ != hipSuccess) {                                                            \
      set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), __FILE__, __LINE__); \
      return HS_E_DEVICE;                                                              \
    }                                                                                  \
  } while (0)

// ---- kernel families (for timing) ----------------------------------------------------------
enum Family { F_RESIZE, F_CONV, F_LSTM, F_STEM, F_POST, F_OVERLAY, F_NET, F_FRAME_NET, F_COUNT };   // F_NET: the small network in one launch,
// F_FRAME_NET: with stage 1
static const char* kFamilyName[F_COUNT] = {"resize_norm", "conv_mfma", "lstm_head",
                                           "stem_pool_mfma", "postprocess", "overlay", "tiny_net_mfma", "frame_net_mfma"};

struct Op {
  Family fam;
  double flops = 0, bytes = 0;
  size_t wt_halves = 0;    // F_CONV: what conv.wt_frag holds
  ResizeParams resize;
  ConvParams conv;
  LstmEpilogueParams lstm;
  StemPoolParams stem;
  PostParams post;
  OverlayParams overlay;
  TinyFrameParams frame_net;
};

static KernelDesc op_desc(const Op& op) {
  switch (op.fam) {
    case F_RESIZE: return describe(op.resize);
    case F_CONV: case F_NET: return describe(op.conv);
    case F_LSTM: return describe(op.lstm);
    case F_STEM: return describe(op.stem);
    case F_POST: return describe(op.post);
    case F_FRAME_NET: return describe(op.frame_net);
    default: return describe(op.overlay);
  }
}

static void* op_params(Op& op) {
  switch (op.fam) {
    case F_RESIZE: return &op.resize;
    case F_CONV: case F_NET: return &op.conv;
    case F_LSTM: return &op.lstm;
    case F_STEM: return &op.stem;
    case F_POST: return &op.post;
    case F_FRAME_NET: return &op.frame_net;
    default: return &op.overlay;
  }
}

// done != NULL: the event completes with the kernel.  It is attached to the dispatch itself: an
// event recorded behind the kernel is a packet of its own in the queue (3.8 us per record between
// back-to-back kernels, against 1.5 us for the attached one) and its waiters see it 2.5 us later.
static hipError_t launch_op(Op& op, hipStream_t s, hipEvent_t done) {
  const KernelDesc d = op_desc(op);
  void* args[1] = {op_params(op)};
  if (done) return hipExtLaunchKernel(d.func, d.grid, d.block, args, d.shmem, s, nullptr, done, 0);
  return hipLaunchKernel(d.func, d.grid, d.block, args, d.shmem, s);
}

// ---- workspace carving -----------------------------------------------------------------------
struct Carver {
  uint8_t* base;   // may be NULL for a dry run
  size_t off = 0;
  explicit Carver(void* b) : base((uint8_t*)b) {}
  template <typename T>
  T* take(size_t count) {
    off = (off + 255) & ~(size_t)255;
    T* p = base ? (T*)(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

struct Tensor {
  f16* p = nullptr;
  int h = 0, w = 0, c = 0, pitch = 0;
  size_t cap = 0;   // halves its buffer holds (known in a sizing walk too, where p is NULL)
};

enum SlotState { SLOT_FREE = 0, SLOT_INFLIGHT = 1, SLOT_DONE = 2 };
// Two lanes: with more frames in flight the submitting host thread is the limit, not the GPU.  A 1080p frame
// back to back takes 106 us, of which the host spends 80 handing over its 19 launches.  (Four lanes were
// measured with one graph launch per frame, about 75 us: no gain.)
constexpr int kMaxLanes = 2;

struct Slot {
  std::vector<Op> pre;     // stage 1: one launch, blockIdx.y = stream of the batch
  std::vector<Op> infer;   // stage 2: the network over the whole batch
  std::vector<Op> frame_net;      // stages 1 and 2 of the small network in one launch (empty: two are the better form)
  std::vector<Op> infer_layers;   // the small network layer by layer; all its forms are run while kernels are being timed
  std::vector<Op> infer_static;   // the same with the gate scratch in the library's fixed
                                  // device array (empty when the scratch needed exceeds it)
  std::vector<Op> post;    // stage 3: the channel maxima
  bool maxima_with_overlay = false;   // they may ride in the overlay's launch instead,
  bool maxima_rode = false;           // and did so for the slot's frame
  std::vector<Op> overlay; // stage 4: one launch, blockIdx.y = stream of the batch
  hipEvent_t ev_pre = nullptr, ev_infer = nullptr, ev_post = nullptr, ev_overlay = nullptr;
  // the event that the overlay waits for: behind stage 3 where it has a launch of its own, else
  // behind stage 2
  hipEvent_t ev_stage3 = nullptr;
  // Frames launched kernel by kernel take the stages' ends from `stamps`.  Their ev_infer / ev_stage3 order streams, and
  // are there only where another stream waits for them at submit or is likely to later (order_behind).  What ties the
  // device's clock to the frame's end is a stamp of the overlay's last workgroup (end_stamped), or else ev_stage3 (has_event).
  bool stamped = false, end_stamped = false, has_event = true;
  hipStream_t stream = nullptr;       // the frame's, up to stage 3
  // the event that says the frame has left the last stage: ev_overlay, or, for a member of a
  // group, the first member's (one overlay launch serves them all)
  hipEvent_t ev_done = nullptr;
  // Consecutive frames rotate over the lanes (activation sets + streams) and overlap;
  // the recurrent cell is the only thing that chains them: its gate convolution (op wait_idx)
  // waits for the previous frame's state update, the last kernel of stage 2 (ev_infer).
  // -1: the network has no recurrent state.
  int lane = 0, wait_idx = -1;
  // stages 1-3 as one HIP graph (kernel nodes chained in order, event-record nodes at the
  // stage boundaries); only the frame pointer of the first node changes from frame to frame
  hipGraph_t graph = nullptr;
  hipGraphExec_t graph_exec = nullptr;
  std::vector<hipGraphNode_t> resize_nodes;
  StageStamps* stamps = nullptr; // pinned host memory, written by the overlay's kernel
  PostRecord* rec = nullptr;   // [batch], pinned host memory, written by the stage-3 kernel
  f16* d_netin = nullptr;      // [batch] padded images
  float* d_netin_f32 = nullptr;
  float* d_logits = nullptr;   // [batch][8][n]
  float* d_heat = nullptr;
  uint8_t* d_mask = nullptr;
  int state = SLOT_FREE;
  std::vector<hs_result> results;   // one per stream of the batch
};

struct TimedLaunch {
  Family fam;
  double flops, bytes;
  hipEvent_t e0, e1;
};

}  // namespace hs

using namespace hs;

struct hs_ctx {
  int device = 0;
  int n_cus = 0;
  int wall_clock_khz = 0;             // rate of the clock that kernels stamp with
  void* d_static_scratch = nullptr;   // the library's fixed scratch array on this device
  size_t static_scratch_bytes = 0;
  std::mutex mu;
  std::vector<hs_app*> apps;
  unsigned n_created = 0;             // applications created so far
  // Idle streams created with the context.  The runtime deals streams out to its four hardware
  // queues strictly in turn only once each queue exists: of the first four streams of a process whose
  // default stream has been used, two share a queue, and an application created first would have
  // both of its lanes on it (12 frames back to back: 1.51 ms instead of 1.29).
  hipStream_t queue_openers[4] = {nullptr};
};

struct hs_app {
  hs_ctx* ctx = nullptr;
  hs_app_desc desc;
  int map_w = 0, map_h = 0;
  int batch = 1;
  int netin_w = 0, netin_h = 0, netin_pad = 0;   // padded stage-1 output geometry
  bool stateful = false;
  // recurrent state
  float* d_c = nullptr;
  f16* d_concat[kMaxLanes] = {nullptr};   // per lane: [x_t ; h_{t-1}] of the frames that run there
  int concat_pitch = 0, hid = 0, x_ch = 0;
  int lanes = 1;
  hipStream_t lane_last_stream[kMaxLanes] = {nullptr};   // stream each lane's latest frame used
  // streams / partition: s_lane[i] carries lane i (all equal to s_lane[0] when partitioned, so
  // that a partition keeps to one hardware queue); s_overlay is NULL when the overlay follows
  // its frame's lane stream
  hipStream_t s_lane[kMaxLanes] = {nullptr};
  hipStream_t s_overlay = nullptr;
  // Lane whose stream carries the frames that find the application idle.  The runtime deals
  // streams out to four hardware queues in turn, so applications i and i + 2 own the same pair of
  // them: of each two such applications one is at home on its first stream and the other on its
  // second, and up to four applications (or members of a group) with one frame in flight each run
  // on four queues instead of two (three networks per frame: 375 -> 320 us).
  int home_lane = 0, last_stream = 0;
  bool partitioned = false;
  uint32_t claim[HS_MAX_CU_WORDS] = {0};
  // ring
  std::vector<Slot> slots;
  int depth = 0;
  uint64_t n_submitted = 0, n_completed = 0, n_delivered = 0;
  std::mutex mu;
  std::condition_variable cv_work, cv_done;
  std::atomic<uint64_t> completed_pub{0};   // n_completed for waiters that spin without the lock
  std::thread completer;
  bool stop = false;
  Message completer_error;
  int launch_mode = HS_LAUNCH_EAGER;
  // kernel timing
  bool timing = false;
  std::vector<TimedLaunch> timed;
  double acc_ms[F_COUNT] = {0}, acc_flops[F_COUNT] = {0}, acc_bytes[F_COUNT] = {0};
  uint64_t acc_n[F_COUNT] = {0};
  void* pinned = nullptr;
  hs_group* group = nullptr;   // set while the application is a member of a multi-network group
  size_t partial_bytes = 0;    // gate scratch (pre-activations, fp32) one frame needs
};

// A multi-network application: the members run stages 1-3 on the same frame side by side, one
// overlay launch of the group draws all their layers.
// The paper's inference operator launches the parallel inferences from one CPU thread each
// (Section III-B); likewise every member but the first has a thread that enqueues its stages
// 1-3 while the caller's thread enqueues the first member's, so the host launch costs overlap.
struct GroupWorker {
  std::thread th;
  std::mutex mu;
  std::condition_variable cv;
  bool has_job = false, done = false, stop = false;
  // the job: one frame for member `app`
  hs_app* app = nullptr;
  const uint8_t* d_frame = nullptr;
  uint8_t* d_out = nullptr;
  uint64_t frame_id = 0, t_submit = 0;
  // its outcome
  hs_status status = HS_OK;
  Message error;
  Slot* slot = nullptr;
  hipStream_t tail = nullptr;

  ~GroupWorker() {   // ends the thread, once its job is done
    {
      std::lock_guard<std::mutex> lk(mu);
      stop = true;
    }
    cv.notify_all();
    if (th.joinable()) th.join();
  }
};

struct hs_group {
  hs_ctx* ctx = nullptr;
  std::vector<hs_app*> members;
  std::vector<Op> overlay;   // one op; its layers are refilled from the members' slots per frame
  std::vector<std::unique_ptr<GroupWorker>> workers;   // workers[i] serves members[i + 1]
};

namespace hs {

// ---- weight packing ----------------------------------------------------------------------------
// The blob is converted to fp16 once, then every layer is rearranged by tasks of 32 output channels
// that run on a few host threads (create time: 18 M weights; converting and scattering them one by
// one took 130 ms).
#if !defined(__HIP_DEVICE_COMPILE__) && (defined(__x86_64__) || defined(__i386__))
__attribute__((target("f16c"))) static void to_half_f16c(const float* src, f16* dst, size_t n) {
  for (size_t i = 0; i < n; ++i) dst[i] = (f16)src[i];
}
static bool has_f16c() { return __builtin_cpu_supports("f16c"); }
#else
static void to_half_f16c(const float*, f16*, size_t) {}
static bool has_f16c() { return false; }
#endif
static void to_half(const float* src, f16* dst, size_t n) {
  if (has_f16c()) return to_half_f16c(src, dst, n);
  for (size_t i = 0; i < n; ++i) dst[i] = (f16)src[i];
}

// Generic layer: packed[n][(ky*k + kx)*cin + c] = w[n][c][ky][kx], taps = k * k.
static void pack_generic(const f16* w, int cout, int cin, int taps, f16* dst) {
  const size_t ktot = (size_t)taps * cin;
  for (int n = 0; n < cout; ++n) {
    f16* row = dst + (size_t)n * ktot;
    const f16* src = w + (size_t)n * ktot;
    for (int t = 0; t < taps; ++t)
      for (int c = 0; c < cin; ++c) row[(size_t)t * cin + c] = src[(size_t)c * taps + t];
  }
}

// The same layer in MFMA fragment order for the kernels that read their weight operand straight
// from memory (3x3, cin % 64 == 0), channel group g = rows 32*g .. +31: dst[(((g*chunks + cc)*taps +
// tap)*4 + ks)*64 + lane][j] = w[32*g + r][64*cc + 16*ks + 8*h + j][tap], lane = r + 32*h; channels above
// cout are zero.  taps = 9 (3x3) or 1 (the 1x1 projection fused into a stride-2 layer).
static void pack_frag(const f16* w, int cout, int cin, int taps, int g, f16* dst) {
  const int chunks = cin / 64;
  f16* out = dst + (size_t)g * chunks * taps * 4 * 512;
  for (int cc = 0; cc < chunks; ++cc)
    for (int r = 0; r < 32; ++r) {
      const int n = 32 * g + r;
      for (int oct = 0; oct < 8; ++oct) {               // channels 64*cc + 8*oct .. +7: ks = oct / 2, h = oct % 2
        const f16* src = w + ((size_t)std::min(n, cout - 1) * cin + 64 * cc + 8 * oct) * taps;
        for (int tap = 0; tap < taps; ++tap) {
          f16* o = out + (((size_t)cc * taps + tap) * 4 + oct / 2) * 512 + (size_t)(r + 32 * (oct % 2)) * 8;
          for (int j = 0; j < 8; ++j) o[j] = n < cout ? src[(size_t)j * taps + tap] : (f16)0.0f;
        }
      }
    }
}

// A layer of the small network in fragment order: dst[(q*ksteps + ks)*64 + lane][j] = weight of
// channel r (zero from cout on) at k = 16*ks + 8*h + j of chunk q, lane = r + 32*h.  `rows`: the packed
// rows [cout][nchunks * kc].
static void pack_direct(const f16* rows, int cout, int nchunks, int kc, f16* dst) {
  for (int q = 0; q < nchunks; ++q)
    for (int ks = 0; ks < kc / 16; ++ks)
      for (int lane = 0; lane < 64; ++lane) {
        const int r = lane & 31, h = lane >> 5;
        f16* out = dst + ((size_t)(q * (kc / 16) + ks) * 64 + lane) * 8;
        for (int j = 0; j < 8; ++j)
          out[j] = r < cout ? rows[(size_t)r * nchunks * kc + (size_t)q * kc + 16 * ks + 8 * h + j] : (f16)0.0f;
      }
}

// First layer on the padded 4-channel image: one chunk per kernel row, covering chunk_px
// adjacent pixels of 4 channels; packed[n][ky][px][ch] = w[n][ch][ky][px] (px < k, ch < 3).
static void pack_rowtap(const f16* w, int cout, int k, int chunk_px, int cout_pad, f16* dst) {
  const size_t ktot = (size_t)k * chunk_px * 4;
  std::memset(dst, 0, (size_t)cout_pad * ktot * sizeof(f16));
  for (int n = 0; n < cout; ++n)
    for (int ch = 0; ch < 3; ++ch)
      for (int ky = 0; ky < k; ++ky)
        for (int px = 0; px < k; ++px)
          dst[(size_t)n * ktot + ((size_t)ky * chunk_px + px) * 4 + ch] =
              w[(((size_t)n * 3 + ch) * k + ky) * k + px];
}

// The 7x7 stem's weights in MFMA fragment order for k_stem_pool: block ((wn * 7 + ky) * 2 + s) of
// 64 lanes x 8 halves; lane (h, r) holds channel 32 * wn + r, k = ky * 32 + s * 16 + h * 8 .. + 7 of
// the row-tap layout (k = (ky * 8 + px) * 4 + ch, zero where px == 7 or ch == 3).
static void pack_stem_frag(const f16* w, f16* dst) {
  std::vector<f16> rows((size_t)64 * 224);
  pack_rowtap(w, 64, 7, 8, 64, rows.data());
  for (int wn = 0; wn < 2; ++wn)
    for (int ky = 0; ky < 7; ++ky)
      for (int s = 0; s < 2; ++s)
        for (int lane = 0; lane < 64; ++lane) {
          const int h = lane >> 5, r = lane & 31;
          const f16* src = rows.data() + (size_t)(32 * wn + r) * 224 + ky * 32 + s * 16 + h * 8;
          f16* out = dst + ((size_t)((wn * 7 + ky) * 2 + s) * 64 + lane) * 8;
          for (int e = 0; e < 8; ++e) out[e] = src[e];
        }
}

// ---- plan builder ------------------------------------------------------------------------------
static inline int conv_out(int n, int k, int s, int p) { return (n + 2 * p - k) / s + 1; }
static inline int round_up(int v, int m) { return (v + m - 1) / m * m; }
static inline size_t round_up_sz(size_t v, size_t m) { return (v + m - 1) / m * m; }

// Walks the layers of a network in blob order.  Used twice: a sizing walk (no pointers, no
// packing) that yields the packed-weight and gate scratch sizes, then the real walk.
struct Builder {
  const hs_app_desc& d;
  Carver carve;
  bool pack;                      // pack weights on the host (create only)
  bool carve_acts;                // hand out activation storage (second walk)
  std::vector<f16> host_w;        // packed weights staged on the host
  std::vector<f16> half_blob;     // the blob in fp16 (pack only)
  std::vector<std::function<void()>> pack_tasks;   // run by run_pack() once host_w has its size
  f16* d_w = nullptr;             // device weights base
  size_t w_halves = 0;            // packed weights consumed so far
  const float* blob;
  size_t blob_off = 0;
  size_t partial_floats = 0;
  float* d_partial = nullptr;     // gate scratch of this lane inside the workspace
  std::vector<Op> ops;            // stage-2 ops; slot-dependent pointers are patched per slot
  std::vector<Op> layer_ops;      // the small network: its layers as launches of their own
  int first_conv_op = -1;         // op whose conv.in is the slot's padded net input
  int logits_op = -1;             // op that writes the slot's logits
  int lstm_conv_op = -1;          // gate convolution of the recurrent cell (-1: none)
  int map_h = 0, map_w = 0;
  bool stateful = false;
  float* d_c = nullptr;
  f16* d_concat = nullptr;

  Builder(const hs_app_desc& desc, void* base, bool do_pack, bool do_carve)
      : d(desc), carve(base), pack(do_pack), carve_acts(do_carve), blob(desc.weights) {}

  template <typename T>
  T* acts(size_t count) { return carve_acts ? carve.take<T>(count) : nullptr; }

  // A buffer for activations.
  Tensor act(size_t halves) {
    Tensor t;
    t.p = acts<f16>(halves);
    t.cap = halves;
    return t;
  }
  // A plan whose layer writes past its output's buffer is refused here, on the host.
  static void check_room(const Tensor& t, int pixels) {
    if ((size_t)pixels * t.pitch > t.cap) throw std::logic_error("a layer's output exceeds its buffer");
  }

  // Reserve room for n packed halves; returns the offset. Regions start 256-byte aligned.
  size_t reserve_w(size_t n) {
    const size_t off = w_halves;
    w_halves = round_up_sz(off + n, 128);
    return off;
  }

  // Packing tasks of a layer whose weights start at blob offset `at`, into region `off`.
  void pack_frag_at(size_t at, int cout, int cin, int taps, int cout_pad, size_t off) {
    if (!pack) return;
    for (int g = 0; g < cout_pad / 32; ++g)
      pack_tasks.push_back([=] { pack_frag(half_blob.data() + at, cout, cin, taps, g, host_w.data() + off); });
  }
  // Converts the blob and runs the packing tasks, on up to eight host threads.
  void run_pack() {
    host_w.assign(w_halves, (f16)0.0f);
    half_blob.resize(d.weight_floats);
    std::vector<std::function<void()>> convert;
    constexpr size_t kPiece = (size_t)1 << 20;
    for (size_t i = 0; i < d.weight_floats; i += kPiece)
      convert.push_back([=] { to_half(blob + i, half_blob.data() + i, std::min(kPiece, d.weight_floats - i)); });
    run_tasks(convert);
    run_tasks(pack_tasks);
    pack_tasks.clear();
    half_blob = std::vector<f16>();
  }
  static void run_tasks(const std::vector<std::function<void()>>& tasks) {
    std::atomic<size_t> next{0};
    std::mutex mu;
    std::exception_ptr failed;           // a task's exception reaches the caller, not the thread's end
    auto work = [&] {
      try {
        for (size_t i = next++; i < tasks.size(); i = next++) tasks[i]();
      } catch (...) {
        std::lock_guard<std::mutex> lk(mu);
        failed = std::current_exception();
      }
    };
    // (a thread costs about as much as one task: few tasks run on the caller's)
    const size_t n = tasks.size() < 16 ? 1 : std::min<size_t>(8, std::max(1u, std::thread::hardware_concurrency()));
    std::vector<std::thread> threads;
    threads.reserve(n);
    try {
      for (size_t i = 1; i < n; ++i) threads.emplace_back(work);
    } catch (...) {
      // no more threads to be had (system_error), or no memory for one's state (bad_alloc): those that
      // there are do the work
    }
    work();
    for (std::thread& x : threads) x.join();
    if (failed) std::rethrow_exception(failed);
  }

  // k_conv3x3_run with a form of kRunForms.  False: the layer is out of the form's range.
  static bool plan_run(ConvParams& c, int form) {
    const RunForm& f = kRunForms[form];
    const double in_bytes = 2.0 * c.batch * c.hin * c.win * c.cin_pitch, w_bytes = 2.0 * c.cout_pad * c.ktot;
    if (c.chunks_per_tap % 2 != 0 || c.cout % f.ch != 0 || in_bytes >= 2147483648.0 || w_bytes >= 2147483648.0) return false;
    c.variant = CONV_KW;
    c.run_form = form;
    c.run_in_bytes = (uint32_t)in_bytes; c.run_w_bytes = (uint32_t)w_bytes;
    c.tiles_m = run_plan(c.hout, c.wout, c.batch, f.px, f.passes, f.lds, c.run);
    c.tiles_n = c.cout / f.ch;
    return c.tiles_m > 0 && (double)c.tiles_m * c.tiles_n * c.tiles_m * c.tiles_n < 2147483648.0;   // run_div31
  }

  // k_conv3x3s2_run with a form of kRun2Forms.  (Its items are chunks with four K splits, half chunks with two, and it takes
  // them in pairs, or a single one.)
  static bool plan_run2(ConvParams& c, int form) {
    const Run2Form& f = kRun2Forms[form];
    if (f.splits() == 4 && c.chunks_per_tap % 2 != 0 && c.chunks_per_tap != 1) return false;
    const double in_bytes = 2.0 * c.batch * c.hin * c.win * c.cin_pitch, w_bytes = 2.0 * c.cout_pad * c.ktot;
    if (c.cout % f.ch != 0 || in_bytes >= 2147483648.0 || w_bytes >= 2147483648.0) return false;
    c.variant = CONV_KW;
    c.run_form = form;
    c.run_in_bytes = (uint32_t)in_bytes; c.run_w_bytes = (uint32_t)w_bytes;
    c.tiles_m = run2_plan(c.hin, c.win, c.batch, f.px, f.passes, f.lds, f.step, f.units, c.run);
    c.tiles_n = c.cout / f.ch;
    return c.tiles_m > 0 && (double)c.tiles_m * c.tiles_n * c.tiles_m * c.tiles_n < 2147483648.0;   // run_div31
  }

  // The form of k_conv3x3_run or k_conv3x3s2_run for a layer.  A tile's time is a fixed part and one per Cin chunk
  // (kRunForms, kRun2Forms, fitted to twelve 854 x 480 frames, where every CU works on several tiles); the launch lasts as
  // long as its busiest CU, which has ceil(tiles / 256) of them.  A CU with a single tile hides nothing of its latencies
  // behind another one: 1 us more.  Over eleven sizes from one 192 x 110 to twelve 854 x 480 frames, all layers, the form with
  // the smallest sum is the fastest one or within 8 % of it (four 641 x 361 frames, 512 channels at stride 1: 8.0 us, the
  // other forms 10.5 to 17.3).
  // splits: only forms with that many K splits, whose sums are the same bit for bit (0: any).
  // cus: the CUs that a round of tiles has, fewer in a partition (effective_cus), where wider forms then take fewer rounds.  Over 24
  // layers on 40, 64, 80 and 128 CUs the form chosen is 1 % slower than the best one with as many K splits on average, at
  // most 16 %.  (80 CUs, two 854 x 480 frames, us per layer, planned for 256 CUs / for their own: 512 channels 16.4 / 14.2, gates 37.0 / 31.6.)
  static constexpr int kAllCus = 256;
  template <class Form, class Plan>
  static void choose_form(ConvParams& c, const Form* forms, int n_forms, int any_map, int splits, int cus, Plan plan) {
    double best = 0;
    int form = -1;
    for (int i = 0; i < n_forms; ++i) {
      if ((i == any_map && form >= 0) || (i > any_map && cus >= kAllCus)) continue;
      ConvParams t = c;
      if ((splits && forms[i].splits() != splits) || !plan(t, i)) continue;
      const int rounds = (t.tiles_m * t.tiles_n + cus - 1) / cus;
      const double tile = forms[i].cost + forms[i].chunk_cost * c.chunks_per_tap;
      const double cost = rounds * tile + (rounds == 1 ? 1.0 : 0.0);
      if (form < 0 || cost < best) { best = cost; form = i; }
    }
    if (form < 0) throw std::logic_error("no tile form for a layer of this network");
    plan(c, form);
  }

  // Picks the kernel variant, the tile grid and the split along K.  like: the plan that the layer has for other CUs, whose sums
  // this one's are to be, bit for bit.
  static void choose_split(ConvParams& c, const ConvParams* like = nullptr, int cus = kAllCus) {
    // the shared-patch kernels address the input with 32-bit offsets (in halves)
    const bool fits32 = (double)c.batch * c.hin * c.win * c.cin_pitch < 2147483648.0;
    const bool s3x3 = c.ntaps == 9 && c.kw == 3 && c.pad == 1 && c.kc == 64 && c.cout % 128 == 0 && fits32;
    c.tiles_per_wg = 1;
    if (s3x3 && c.stride == 2) {
      const int n = c.batch * ((c.hout + 7) / 8) * ((c.wout + 7) / 8) * (c.cout / 128);   // tiles of 8 x 8 x 128
      if (c.chunks_per_tap == 1 && n > 1024) {
        // One chunk, more tiles than two rounds of workgroups: k_conv3x3s2_dira walks them, the next tile's patch fetched
        // during the current one's products (two workgroups per CU are resident, so walk in one round), in steps of 10 us
        // per 512 tiles; k_conv3x3s2_run goes by rounds of its own tiles.  Us at 854 x 480, the latter first: eight frames (896
        // tiles) 23.7, 25.1, nine (1008) 27.0, 26.0, ten (1120) 28.7, 30.8, eleven (1232) 28.9, 30.0, twelve (1344) 33.1,
        // 30.3, sixteen (1792) 43.3, 39.1; six 1280 x 720 (1440) 36.2, 31.5; sixteen 416 x 240 (448) 16.0, 17.3.
        c.variant = CONV_S2_DIRA;
        c.tiles_x = (c.wout + 7) / 8;
        c.tiles_m = c.batch * ((c.hout + 7) / 8) * c.tiles_x;
        c.tiles_n = c.cout / 128;
        c.tiles_per_wg = (n + 511) / 512;
      } else {
        choose_form(c, kRun2Forms, kRun2FormCount, kRun2FormAnyMap, like ? kRun2Forms[like->run_form].splits() : 0, cus, plan_run2);
      }
    } else if (s3x3 && c.stride == 1 && c.chunks_per_tap >= 2) {
      choose_form(c, kRunForms, kRunFormCount, kRunFormAnyMap, like ? kRunForms[like->run_form].splits() : 0, cus, plan_run);
    } else if (c.cout <= 32 && c.kc <= 32 && c.chunks_per_tap == 1 && c.ntaps <= 9) {
      // two K splits, of at most five taps each, while tiles of 64 pixels would be fewer than 192
      c.variant = CONV_DIRECT;
      const int ns = (c.m + 63) / 64 < 192 && c.nchunks >= 8 ? 2 : 1;
      c.kw_splits = ns;
      c.chunks_per_split = (c.nchunks + ns - 1) / ns;
      c.tiles_x = 0;
      c.tiles_m = ((c.m + 31) / 32 + 4 / ns - 1) / (4 / ns);
      c.tiles_n = 1;
    } else {
      throw std::logic_error("no convolution kernel for a layer of this network");
    }
    const int groups_m = (c.tiles_m + c.tiles_per_wg - 1) / c.tiles_per_wg;
    c.tiles_per_xcd = (groups_m * c.tiles_n + 7) / 8;
    // Tile order: every XCD (own L2) takes a run of tiles_per_xcd consecutive tiles.  For every
    // block size, count what the eight L2s fetch (each its own spatial groups' input slices and
    // its own channel tiles' weight slices, once) and keep the cheapest.
    c.n_block = 1;
    if (c.tiles_n > 1) {
      const double in_unit = 2.0 * c.batch * c.hin * c.win * (c.chunks_per_tap * 64.0) / (double)groups_m;
      const double w_unit = 2.0 * c.cout_pad * c.ktot / (double)c.tiles_n;
      const int total = groups_m * c.tiles_n;
      double best = 0;
      for (int nb = 1; nb <= c.tiles_n; nb *= 2) {
        if (c.tiles_n % nb) continue;
        double bytes = 0;
        std::vector<char> seen_in((size_t)groups_m), seen_w((size_t)c.tiles_n);
        for (int x = 0; x < 8; ++x) {
          std::fill(seen_in.begin(), seen_in.end(), 0);
          std::fill(seen_w.begin(), seen_w.end(), 0);
          for (int t = x * c.tiles_per_xcd; t < std::min(total, (x + 1) * c.tiles_per_xcd); ++t) {
            const int blk = groups_m * nb, in_blk = t % blk;
            char& si = seen_in[(size_t)(in_blk / nb)];
            char& sw = seen_w[(size_t)((t / blk) * nb + in_blk % nb)];
            if (!si) { si = 1; bytes += in_unit; }
            if (!sw) { sw = 1; bytes += w_unit; }
          }
        }
        if (nb == 1 || bytes < 0.9 * best) { best = bytes; c.n_block = nb; }
      }
    }
    if (c.variant == CONV_KW) {
      c.run_nb_shift = 0;
      while ((1 << c.run_nb_shift) < c.n_block) ++c.run_nb_shift;
      const uint64_t blk = (uint64_t)c.tiles_m * c.n_block;
      c.run_by_blk = (uint32_t)((((uint64_t)1 << 31) + blk - 1) / blk);
    }
  }

  // Appends the convolution.
  // keep_partial: leave the partial sums in the scratch buffer for a later kernel (ConvLSTM).
  // Returns the index of the convolution op.
  // wf_off: offset of the weights in fragment order.  wf2_off / out2: fragment-ordered weights and
  // output of a 1x1 stride-2 projection fused into a 3x3 stride-2 layer (out2 == NULL: none).
  static constexpr size_t kNoWeights = (size_t)-1;
  int add_conv(ConvParams c, size_t wf_off, const Tensor* res, const Tensor* out, bool relu,
               bool want_f32, bool keep_partial, double flops, size_t wf2_off = kNoWeights, const Tensor* out2 = nullptr) {
    Op op;
    op.fam = F_CONV;
    op.flops = flops;
    auto at = [&](size_t off) { return d_w && off != kNoWeights ? d_w + off : nullptr; };
    c.wt_frag = at(wf_off); c.wt2_frag = at(wf2_off);
    choose_split(c);
    if (!describe(c).func) throw std::logic_error("no instantiation of the planned convolution kernel");
    c.use_partial = keep_partial ? 1 : 0;
    c.partial = nullptr;   // patched when the scratch buffer is carved
    c.out = nullptr; c.out_pitch = 0; c.res = nullptr; c.res_pitch = 0; c.relu = 0;
    c.out_f32 = nullptr;   // the slot's, for the layer that writes the logits
    c.out2 = nullptr; c.out2_pitch = 0;
    if (out2) { c.out2 = out2->p; c.out2_pitch = out2->pitch; }
    if (keep_partial) {
      partial_floats = std::max(partial_floats, (size_t)c.m * c.cout_pad);
    } else {
      if (out) { c.out = out->p; c.out_pitch = out->pitch; }
      if (res) { c.res = res->p; c.res_pitch = res->pitch; }
      c.relu = relu ? 1 : 0;
    }
    op.conv = c;
    ops.push_back(op);
    if (want_f32) logits_op = (int)ops.size() - 1;
    return (int)ops.size() - 1;
  }

  // Generic convolution on a pixel-major tensor; weights are the next cout*cin*k*k floats of the
  // blob starting at blob_at. Fills out->h/w/c.
  // proj_at / proj_out: blob offset and output of the block's 1x1 stride-2 projection, fused into
  // this 3x3 stride-2 layer (none: NULL).
  int conv_layer(const Tensor& in, size_t blob_at, int cout, int k, int stride, int pad, bool relu,
                 const Tensor* res, Tensor* out, bool want_f32, bool keep_partial,
                 size_t proj_at = 0, Tensor* proj_out = nullptr) {
    const int cin = in.c;
    ConvParams g;
    std::memset(&g, 0, sizeof(g));
    g.in = in.p; g.hin = in.h; g.win = in.w; g.cin_pitch = in.pitch;
    g.hout = conv_out(in.h, k, stride, pad); g.wout = conv_out(in.w, k, stride, pad);
    g.batch = d.batch; g.img_m = g.hout * g.wout; g.m = g.batch * g.img_m;
    g.cout = cout; g.cout_pad = round_up(cout, 64);
    g.kc = (cin % 64 == 0) ? 64 : (cin % 32 == 0 ? 32 : 16);
    g.ntaps = k * k; g.kw = k; g.chunks_per_tap = cin / g.kc;
    g.nchunks = g.ntaps * g.chunks_per_tap; g.ktot = g.nchunks * g.kc;
    g.stride = stride; g.pad = pad;
    out->h = g.hout; out->w = g.wout; out->c = cout;
    if (!want_f32 && !keep_partial) check_room(*out, g.m);
    // The kernel variant is a function of the shapes alone.
    ConvParams probe = g;
    choose_split(probe);
    const bool direct = probe.variant == CONV_DIRECT, fuse = proj_out != nullptr;
    if (probe.variant == CONV_KW && stride == 2 && !fuse) throw std::logic_error("k_conv3x3s2_run computes a projection too");
    const size_t wf_halves = (size_t)(direct ? 32 : g.cout_pad) * g.ktot, wf_off = reserve_w(wf_halves);
    size_t wf2_off = kNoWeights;
    if (!direct) {
      pack_frag_at(blob_at, cout, cin, 9, g.cout_pad, wf_off);
    } else if (pack) {
      pack_tasks.push_back([=] {
        std::vector<f16> rows((size_t)cout * g.ktot);
        pack_generic(half_blob.data() + blob_at, cout, cin, k * k, rows.data());
        pack_direct(rows.data(), cout, g.nchunks, g.kc, host_w.data() + wf_off);
      });
    }
    if (fuse) {
      proj_out->h = g.hout; proj_out->w = g.wout; proj_out->c = cout;
      check_room(*proj_out, g.m);
      wf2_off = reserve_w((size_t)g.cout_pad * cin);
      pack_frag_at(proj_at, cout, cin, 1, g.cout_pad, wf2_off);
    }
    const int idx = add_conv(g, wf_off, res, out, relu, want_f32, keep_partial,
                             2.0 * g.m * (double)cout * cin * (k * k + (fuse ? 1 : 0)), wf2_off,
                             fuse ? proj_out : nullptr);
    ops[(size_t)idx].wt_halves = wf_halves;
    return idx;
  }

  // A 64 -> 64 -> 64 channel BasicBlock without projection as ONE launch (k_block64_fused):
  // out = ReLU(conv_b(ReLU(conv_a(in))) + in).  Weights are reserved in blob order (conv a, conv b).
  void block64_layer(const Tensor& in, size_t at_a, size_t at_b, Tensor* out) {
    ConvParams g;
    std::memset(&g, 0, sizeof(g));
    g.in = in.p; g.hin = in.h; g.win = in.w; g.cin_pitch = in.pitch;
    g.hout = in.h; g.wout = in.w;
    g.batch = d.batch; g.img_m = g.hout * g.wout; g.m = g.batch * g.img_m;
    g.cout = 64; g.cout_pad = 64; g.kc = 64;
    g.ntaps = 9; g.kw = 3; g.chunks_per_tap = 1; g.nchunks = 9; g.ktot = 576;
    g.stride = 1; g.pad = 1;
    const size_t wa_off = reserve_w((size_t)64 * 576);
    pack_frag_at(at_a, 64, 64, 9, 64, wa_off);
    const size_t wb_off = reserve_w((size_t)64 * 576);
    pack_frag_at(at_b, 64, 64, 9, 64, wb_off);
    out->h = g.hout; out->w = g.wout; out->c = 64;
    check_room(*out, g.m);
    g.variant = CONV_BLOCK64;
    g.tiles_x = (g.wout + 15) / 16;
    g.tiles_m = g.batch * ((g.hout + 7) / 8) * g.tiles_x;
    g.tiles_n = 1; g.chunks_per_split = 1; g.tiles_per_wg = 1; g.n_block = 1;
    g.tiles_per_xcd = (g.tiles_m + 7) / 8;
    g.tiles_img = (uint32_t)(g.tiles_m / g.batch);
    auto by = [](uint64_t d) { return (uint32_t)((((uint64_t)1 << 31) + d - 1) / d); };
    g.by_tiles_img = by(g.tiles_img); g.by_tiles_x = by((uint64_t)g.tiles_x);
    g.run_in_bytes = (uint32_t)(g.batch * g.hin * g.win * 128);
    g.wt_frag = d_w ? d_w + wa_off : nullptr;
    g.wt2_frag = d_w ? d_w + wb_off : nullptr;
    g.out = out->p; g.out_pitch = out->pitch;
    g.res = in.p; g.res_pitch = in.pitch;
    g.relu = 1;
    Op op;
    op.fam = F_CONV;
    op.flops = 2.0 * (2.0 * g.m * 64.0 * 64.0 * 9.0);
    op.wt_halves = (size_t)64 * 576;
    op.conv = g;
    ops.push_back(op);
  }

  // First layer: 3 input channels on the padded 4-channel image, k x k, stride 2, ReLU.
  void first_layer(size_t blob_at, int pad_img_h, int pad_img_w, int cout, int k, Tensor* out) {
    const int pad = k / 2;
    const int chunk_px = (k <= 4) ? 4 : 8;
    ConvParams g;
    std::memset(&g, 0, sizeof(g));
    g.in = nullptr;   // per slot
    g.hin = pad_img_h; g.win = pad_img_w; g.cin_pitch = 4;
    g.hout = conv_out(d.net_h, k, 2, pad); g.wout = conv_out(d.net_w, k, 2, pad);
    g.batch = d.batch; g.img_m = g.hout * g.wout; g.m = g.batch * g.img_m;
    g.cout = cout; g.cout_pad = round_up(cout, 64);
    g.kc = chunk_px * 4;
    g.ntaps = k; g.kw = 1; g.chunks_per_tap = 1; g.nchunks = k; g.ktot = k * g.kc;
    g.stride = 2; g.pad = 0;
    const size_t wf_halves = (size_t)32 * g.ktot, wf_off = reserve_w(wf_halves);
    if (pack)
      pack_tasks.push_back([=] {
        std::vector<f16> rows((size_t)cout * g.ktot);
        pack_rowtap(half_blob.data() + blob_at, cout, k, chunk_px, cout, rows.data());
        pack_direct(rows.data(), cout, g.nchunks, g.kc, host_w.data() + wf_off);
      });
    out->h = g.hout; out->w = g.wout; out->c = cout;
    check_room(*out, g.m);
    first_conv_op = add_conv(g, wf_off, nullptr, out, true, false, false, 2.0 * g.m * (double)cout * 3 * k * k);
    ops[(size_t)first_conv_op].wt_halves = wf_halves;
  }

  void walk_tiny(int ph, int pw) {
    const int h1 = conv_out(d.net_h, 3, 2, 1), w1 = conv_out(d.net_w, 3, 2, 1);
    const int h2 = conv_out(h1, 3, 2, 1), w2 = conv_out(w1, 3, 2, 1);
    const size_t nb = (size_t)d.batch;
    Tensor t1 = act(nb * h1 * w1 * 16), t2 = act(nb * h2 * w2 * 32), t3 = act(nb * h2 * w2 * 32), lg;
    t1.pitch = 16; t2.pitch = 32; t3.pitch = 32;
    size_t at = 0;
    first_layer(at, ph, pw, 16, 3, &t1);                                 at += 16 * 3 * 9;
    conv_layer(t1, at, 32, 3, 2, 1, true, nullptr, &t2, false, false);   at += 32 * 16 * 9;
    conv_layer(t2, at, 32, 3, 1, 1, true, nullptr, &t3, false, false);   at += 32 * 32 * 9;
    conv_layer(t3, at, 8, 3, 1, 1, false, nullptr, &lg, true, false);    at += 8 * 32 * 9;
    blob_off = at;
    map_h = lg.h; map_w = lg.w; stateful = false;
    // One launch for all layers (and, while kernels are being timed, the layers one after the other behind it), unless the halos
    // that k_tiny_net computes again, and its tiles beyond the map's edges, cost more than the launches and tensors it saves.  It
    // takes a round of 256 tiles at a time, the layers go by pixels: times in us, fitted to 35 sizes from one 128 x 128 frame
    // to one of 1448 x 1448, thin ones among them.  Measured, layers / one launch: one 128 x 128 frame 15.6 / 6.8, eight 320 x 320
    // 26.2 / 23.4, sixteen (1600 tiles) 41.5 / 39.9; sixteen 300 x 200 (1120 tiles, 84 % full) 27.6 / 28.9, eight 640 x 360
    // (1920 tiles) 43.6 / 45.2, sixteen 4000 x 16 (2000 tiles, half full) 28.6 / 44.4.
    const double pixels = (double)d.batch * map_h * map_w;
    const int rounds = (d.batch * ((map_h + 7) / 8) * ((map_w + 7) / 8) + 255) / 256;
    if (2.0 + 5.3 * rounds > std::max(15.6, 10.3 + 0.288e-3 * pixels)) return;
    layer_ops = ops;
    Op net;
    net.fam = F_NET;
    net.conv = layer_ops[0].conv;
    const ConvParams& last = layer_ops[3].conv;
    net.conv.variant = CONV_TINY_NET;
    net.conv.mid_h = h1; net.conv.mid_w = w1;
    net.conv.hout = last.hout; net.conv.wout = last.wout;
    net.conv.m = last.m; net.conv.img_m = last.img_m;
    for (const Op& op : layer_ops) { net.flops += op.flops; net.wt_halves += op.wt_halves; }
    // k_tiny_net takes the four layers' weights as one run
    size_t end = 0;
    for (const Op& op : layer_ops) {
      if (d_w && op.conv.wt_frag != d_w + end) throw std::logic_error("the small network's weights are not one run");
      end += op.wt_halves;
    }
    ops = {net};
    first_conv_op = logits_op = 0;
  }

  void walk_resnet(int ph, int pw) {
    const int hs_ = conv_out(d.net_h, 7, 2, 3), ws_ = conv_out(d.net_w, 7, 2, 3);
    const int hp = conv_out(hs_, 3, 2, 1), wp = conv_out(ws_, 3, 2, 1);
    const int widths[4] = {64, 128, 256, 512};
    int hf = hp, wf = wp;
    // The four buffers rotate through all stages.  A stage halves the map and doubles the width: the first
    // stage is the largest but on maps of a few pixels, whose halves round up.
    size_t act_img = (size_t)hp * wp * 64;
    for (int s = 1; s < 4; ++s) {
      hf = conv_out(hf, 3, 2, 1); wf = conv_out(wf, 3, 2, 1);
      act_img = std::max(act_img, (size_t)hf * wf * widths[s]);
    }
    const size_t nb = (size_t)d.batch;
    const int mf = (int)nb * hf * wf;                    // feature-map pixels over the batch
    Tensor buf[4];
    for (Tensor& t : buf) t = act(nb * act_img);
    const Tensor concat_buf = act((size_t)mf * 768);
    f16* const concat = concat_buf.p;
    float* cstate = acts<float>((size_t)mf * 256);

    size_t at = 0;
    {
      // stem convolution and max-pool in one kernel; weights packed as MFMA fragments of row
      // taps of 8 pixels
      const size_t w_off = reserve_w((size_t)64 * 224);
      if (pack) pack_tasks.push_back([=] { pack_stem_frag(half_blob.data() + at, host_w.data() + w_off); });
      Op op;
      op.fam = F_STEM;
      StemPoolParams& sp = op.stem;
      std::memset(&sp, 0, sizeof(sp));
      sp.in = nullptr;   // per slot
      sp.wt = d_w ? d_w + w_off : nullptr;
      sp.out = buf[0].p;
      sp.hin = ph; sp.win = pw; sp.hc = hs_; sp.wc = ws_; sp.hp = hp; sp.wp = wp;
      sp.batch = d.batch;
      sp.tiles_x = (wp + 14) / 15; sp.tiles_y = (hp + 7) / 8;
      sp.tiles_per_xcd = (sp.batch * sp.tiles_x * sp.tiles_y + 7) / 8;
      op.flops = 2.0 * nb * hs_ * ws_ * 64.0 * 3 * 49;
      op.bytes = nb * ((double)d.net_h * d.net_w * 8 + (double)hp * wp * 64 * 2);
      ops.push_back(op);
      first_conv_op = (int)ops.size() - 1;
    }
    at += 64 * 3 * 49;
    int cur = 0;
    buf[0].h = hp; buf[0].w = wp; buf[0].c = 64; buf[0].pitch = 64;
    check_room(buf[0], (int)nb * hp * wp);
    int cin = 64;
    for (int s = 0; s < 4; ++s) {
      for (int blk = 0; blk < 2; ++blk) {
        const int width = widths[s];
        const bool proj = blk == 0 && cin != width;
        const int bc_in = blk == 0 ? cin : width;
        const Tensor a = buf[cur];
        Tensor& t = buf[(cur + 1) % 4];
        Tensor& sc = buf[(cur + 2) % 4];
        Tensor& o = buf[(cur + 3) % 4];
        // blob order within a block: conv a, conv b, projection
        const size_t at_a = at, at_b = at_a + (size_t)width * bc_in * 9,
                     at_p = at_b + (size_t)width * width * 9;
        at = at_p + (proj ? (size_t)width * bc_in : 0);
        t.pitch = width;
        const Tensor* shortcut = &a;
        if (proj) {
          // the projection reads the centre-tap pixels of conv a: one kernel computes both
          sc.pitch = width;
          conv_layer(a, at_a, width, 3, 2, 1, true, nullptr, &t, false, false, at_p, &sc);
          shortcut = &sc;
        } else if (width == 64) {
          // the whole block in one launch; the intermediate tensor t is never written
          o.pitch = width;
          block64_layer(a, at_a, at_b, &o);
          cur = (cur + 3) % 4;
          cin = width;
          continue;
        } else {
          conv_layer(a, at_a, width, 3, 1, 1, true, nullptr, &t, false, false);
        }
        const bool last = s == 3 && blk == 1;
        if (last) o = concat_buf;
        o.pitch = last ? 768 : width;
        conv_layer(t, at_b, width, 3, 1, 1, true, shortcut, &o, false, false);
        cur = (cur + 3) % 4;
        cin = width;
      }
    }
    Tensor cat;
    cat.p = concat; cat.h = hf; cat.w = wf; cat.c = 768; cat.pitch = 768;
    Tensor gates;
    const int lstm_conv = conv_layer(cat, at, 1024, 3, 1, 1, false, nullptr, &gates, false, true);
    lstm_conv_op = lstm_conv;
    at += (size_t)1024 * 768 * 9;
    // head weights: 8 x 256 fp16, plain [k][c]; the head runs inside the ConvLSTM epilogue
    const size_t w_off = reserve_w(2048);
    if (pack)
      pack_tasks.push_back([=] { std::copy_n(half_blob.data() + at, 2048, host_w.data() + w_off); });
    at += 2048;
    {
      Op op;
      op.fam = F_LSTM;
      op.lstm = LstmEpilogueParams{nullptr, mf, 256, cstate,
                                   concat ? concat + 512 : nullptr, 768,
                                   d_w ? d_w + w_off : nullptr, nullptr, hf * wf, 0.0f, nullptr, nullptr,
                                   nullptr, nullptr};
      op.bytes = (double)mf * 1024 * 4.0 + (double)mf * 256 * 10.0;
      op.flops = 2.0 * mf * 8 * 256;
      ops.push_back(op);
      logits_op = (int)ops.size() - 1;
    }
    blob_off = at;
    map_h = hf; map_w = wf; stateful = true;
    d_c = cstate; d_concat = concat;
  }

  void walk(int ph, int pw) {
    if (d.net == HS_NET_TINY4) walk_tiny(ph, pw); else walk_resnet(ph, pw);
    // With several frames per launch the layers that k_conv3x3_run and k_conv3x3s2_run compute prefetch the next layer's
    // weights (not its projection's): a pass then touches more than the last-level cache holds and finds
    // the weights in HBM (four frames 641 x 361: 363 -> 337 us, sixteen frames 416 x 240: 375 -> 358).  The 36 MB of a one-frame
    // application stay cached, and the prefetch would only cost (168 -> 172 us).
    ConvParams* prev = nullptr;
    for (Op& op : ops) {
      if (op.fam != F_CONV) continue;
      if (prev && prev->variant == CONV_KW && op.conv.wt_frag && d.batch > 1) {
        prev->next_wt = op.conv.wt_frag;
        prev->next_lines = (int)(op.wt_halves * sizeof(f16) / 128);
      }
      prev = &op.conv;
    }
  }
};

static void padded_input_geometry(int net_w, int net_h, int k, int* pw, int* ph, int* pad) {
  const int p = k / 2, chunk_px = (k <= 4) ? 4 : 8;
  const int wout = conv_out(net_w, k, 2, p);
  *pad = p;
  *ph = net_h + 2 * p;
  *pw = round_up(std::max(net_w + 2 * p, 2 * (wout - 1) + chunk_px), 2);
}

static size_t expected_weight_floats(int net) {
  if (net == HS_NET_TINY4) return 16 * 3 * 9 + 32 * 16 * 9 + 32 * 32 * 9 + 8 * 32 * 9;
  size_t n = 64 * 3 * 49;
  int cin = 64;
  const int widths[4] = {64, 128, 256, 512};
  for (int s = 0; s < 4; ++s) {
    const int w = widths[s];
    n += (size_t)w * cin * 9 + (size_t)w * w * 9 * 3;
    if (cin != w) n += (size_t)w * cin;
    cin = w;
  }
  n += (size_t)1024 * 768 * 9 + 8 * 256;
  return n;
}

static hs_status validate_desc(const hs_app_desc* d) {
  if (!d) { set_error("NULL description"); return HS_E_INVAL; }
  if (d->frame_w < 1 || d->frame_h < 1 || d->net_w < 8 || d->net_h < 8 || d->frame_w > 10922 ||
      d->frame_h > 65535 || d->net_w > 16384 || d->net_h > 16384) {
    set_error("bad frame or network size");
    return HS_E_INVAL;
  }
  if (d->frame_pitch < (size_t)3 * d->frame_w || d->frame_pitch % 16 != 0) {
    set_error("frame_pitch must be >= 3*frame_w and a multiple of 16");
    return HS_E_INVAL;
  }
  // exact 32-bit integer resize: 255*D + D/2 with D = 4*net_w*net_h must stay below 2^31
  if ((double)d->net_w * d->net_h * 4.0 * 255.5 >= 2147483648.0 ||
      (2.0 * d->net_w + 1.0) * d->frame_w >= 2147483648.0 ||
      (2.0 * d->net_h + 1.0) * d->frame_h >= 2147483648.0) {
    set_error("resize dimensions exceed the exact 32-bit range");
    return HS_E_INVAL;
  }
  if (d->net != HS_NET_TINY4 && d->net != HS_NET_RESNET18_CONVLSTM) {
    set_error("unknown network kind %d", d->net);
    return HS_E_INVAL;
  }
  if (!std::isfinite(d->mean) || !(d->std > 0.0f) || !std::isfinite(d->std) ||
      !(d->threshold > 0.0f && d->threshold < 1.0f) || !(d->alpha >= 0.0f && d->alpha <= 1.0f)) {
    set_error("mean must be finite, std finite and > 0, threshold in (0,1), alpha in [0,1]");
    return HS_E_INVAL;
  }
  if (d->annotate && (d->marker_arm < 0 || d->marker_arm > 64 || d->marker_half < 0 ||
                      d->marker_half > 8 || d->glyph_scale < 1 || d->glyph_scale > 8)) {
    set_error("annotation: marker_arm 0..64, marker_half 0..8, glyph_scale 1..8");
    return HS_E_INVAL;
  }
  if (d->batch < 1 || d->batch > 16) {
    set_error("batch must be 1..16");
    return HS_E_INVAL;
  }
  if (d->queue_depth < 1 || d->queue_depth > 64) {
    set_error("queue_depth must be 1..64");
    return HS_E_INVAL;
  }
  return HS_OK;
}

// Whether stage 1 is part of the small network's launch: where that is one round of workgroups, 256 tiles.  A workgroup that
// resizes 2.6 times its pixels takes 2 us longer, a launch of its own 4, and back to back the host waits for each launch.  Us, two
// launches / one: 128 x 128 (16 tiles) 29.3 / 28.6, sixteen (256) 47 / 46.5; 320 x 320 (100) 35.2 / 34.5, three (300) 45 / 47,
// sixteen 89 / 102; sixteen frames back to back 322 x 241 to 96 x 72 300 / 238, 1920 x 1080 to 320 x 200 340 / 270; four batches of
// twelve 300 x 300 (1200) 250 / 292.  Frames that are large beside the network's input gain back to back only: 3840 x 2160 to 128 x 128
// alone 39.0 / 40.6, twelve 260 / 221; fifteen 1920 x 1080 to 128 x 128 in a batch 81.1 / 82.2, twelve batches 767 / 680.
static bool frame_net_pays(const hs_app_desc& d, int map_h, int map_w) {
  return (double)d.frame_pitch * d.frame_h < 2147483648.0 &&             // 32-bit offsets
         d.batch * ((map_h + 7) / 8) * ((map_w + 7) / 8) <= 256;
}

// Builds the whole plan into `app`, or only sizes the workspace when app == NULL.
static hs_status build_plan(const hs_app_desc* d, hs_app* app, size_t* bytes_out) {
  const bool create = app != nullptr;
  const int depth = d->queue_depth;
  const int k1 = d->net == HS_NET_TINY4 ? 3 : 7;
  int pw, ph, pad;
  padded_input_geometry(d->net_w, d->net_h, k1, &pw, &ph, &pad);

  // sizing walk: packed-weight size
  Builder sizing(*d, nullptr, false, false);
  sizing.walk(ph, pw);
  if (sizing.blob_off != expected_weight_floats(d->net)) {
    set_error("internal: layer walk consumed %zu floats, expected %zu", sizing.blob_off,
              expected_weight_floats(d->net));
    return HS_E_INVAL;
  }

  // real walk: workspace = [weights][activations, state][gate scratch][tables][slots]
  Builder b(*d, create ? d->d_workspace : nullptr, create, true);
  b.d_w = b.carve.take<f16>(sizing.w_halves);
  b.walk(ph, pw);
  auto bind_partial = [](Builder& bb) {
    float* d_partial = bb.carve.take<float>(bb.partial_floats);
    bb.d_partial = d_partial;
    for (Op& op : bb.ops) {
      if (op.fam == F_CONV && op.conv.use_partial) op.conv.partial = d_partial;
      if (op.fam == F_LSTM) op.lstm.partial = d_partial;
    }
  };
  bind_partial(b);
  // Further lanes: the same plan over their own activations and scratch (weights shared), so
  // that consecutive frames can overlap.  Slot i runs in lane i % lanes and frames must rotate
  // strictly, hence lanes divides the queue depth.  The cell state c is shared; a lane's state
  // update writes h where the NEXT lane's gate convolution reads it.
  const int lanes = depth % kMaxLanes == 0 ? kMaxLanes : 1;
  std::vector<std::unique_ptr<Builder>> extra;
  std::vector<Builder*> lane_b{&b};
  for (int l = 1; l < lanes; ++l) {
    extra.push_back(std::make_unique<Builder>(*d, create ? d->d_workspace : nullptr, false, true));
    Builder& bl = *extra.back();
    bl.carve.off = lane_b.back()->carve.off;
    bl.d_w = b.d_w;
    bl.walk(ph, pw);
    bind_partial(bl);
    lane_b.push_back(&bl);
  }
  if (lanes > 1) {
    b.carve.off = lane_b.back()->carve.off;
    if (b.stateful) {
      std::vector<f16*> own_h(lanes);
      for (int l = 0; l < lanes; ++l) own_h[l] = lane_b[l]->ops[b.logits_op].lstm.h_out;
      for (int l = 0; l < lanes; ++l) {
        LstmEpilogueParams& ll = lane_b[l]->ops[b.logits_op].lstm;
        ll.c = b.ops[b.logits_op].lstm.c;
        ll.h_out = own_h[(l + 1) % lanes];
      }
    }
  }
  float* d_lut32 = b.carve.take<float>(256);
  f16* d_lut16 = b.carve.take<f16>(256);
  const int mh = b.map_h, mw = b.map_w;
  const size_t n_map = (size_t)mh * mw;
  const int B = d->batch;
  struct SlotBuf { f16* netin; float* netin32; float* logits; float* heat; uint8_t* mask;
                   uint8_t* kmap; int* marks; uint64_t* t_stages; };
  std::vector<SlotBuf> sb(depth);
  for (int i = 0; i < depth; ++i) {
    sb[i].netin = b.carve.take<f16>((size_t)B * ph * pw * 4);
    sb[i].netin32 = d->net_fp32_input ? b.carve.take<float>((size_t)B * 3 * d->net_h * d->net_w)
                                      : nullptr;
    sb[i].logits = b.carve.take<float>(B * 8 * n_map);
    sb[i].heat = b.carve.take<float>(B * 8 * n_map);
    sb[i].mask = b.carve.take<uint8_t>(B * 8 * n_map);
    sb[i].kmap = b.carve.take<uint8_t>(B * n_map);
    sb[i].marks = d->annotate ? b.carve.take<int>((size_t)B * 16) : nullptr;
    sb[i].t_stages = b.carve.take<uint64_t>(3);
  }
  const size_t total = round_up_sz(b.carve.off, 256);
  if (bytes_out) *bytes_out = total;
  if (!create) return HS_OK;

  if (d->workspace_bytes < total) {
    set_error("workspace too small: %zu bytes given, %zu needed", d->workspace_bytes, total);
    return HS_E_NOMEM;
  }
  app->map_h = mh; app->map_w = mw; app->stateful = b.stateful; app->batch = B;
  app->d_c = b.d_c; app->concat_pitch = 768; app->hid = 256;
  for (int l = 0; l < lanes; ++l) app->d_concat[l] = lane_b[l]->d_concat;
  app->lanes = lanes;
  app->x_ch = 512;

  // upload weights and tables, zero the recurrent state and the padded borders
  b.run_pack();
  HS_HIP(hipMemcpy(b.d_w, b.host_w.data(), b.host_w.size() * sizeof(f16), hipMemcpyHostToDevice));
  {
    float lut32[256];
    f16 lut16[256];
    for (int v = 0; v < 256; ++v) {
      lut32[v] = (float)(((double)v / 255.0 - (double)d->mean) / (double)d->std);
      lut16[v] = (f16)lut32[v];
    }
    HS_HIP(hipMemcpy(d_lut32, lut32, sizeof(lut32), hipMemcpyHostToDevice));
    HS_HIP(hipMemcpy(d_lut16, lut16, sizeof(lut16), hipMemcpyHostToDevice));
  }
  for (int i = 0; i < depth; ++i)
    HS_HIP(hipMemset(sb[i].netin, 0, (size_t)B * ph * pw * 4 * sizeof(f16)));
  if (app->stateful) {
    HS_HIP(hipMemset(app->d_c, 0, B * n_map * 256 * sizeof(float)));
    for (int l = 0; l < lanes; ++l)
      HS_HIP(hipMemset(app->d_concat[l], 0, B * n_map * 768 * sizeof(f16)));
  }
  HS_HIP(hipDeviceSynchronize());

  // per-slot launch plans
  app->netin_w = pw; app->netin_h = ph; app->netin_pad = pad;
  const double theta_d = std::log((double)d->threshold / (1.0 - (double)d->threshold));
  int a_q8 = (int)lrint(256.0 * (double)d->alpha);
  a_q8 = std::max(0, std::min(256, a_q8));
  const size_t pinned_bytes = (sizeof(PostRecord) * B + sizeof(StageStamps)) * depth;
  HS_HIP(hipHostMalloc(&app->pinned, pinned_bytes, hipHostMallocDefault));
  std::memset(app->pinned, 0, pinned_bytes);
  app->slots.resize(depth);
  for (int i = 0; i < depth; ++i) {
    Slot& s = app->slots[i];
    s.d_netin = sb[i].netin; s.d_netin_f32 = sb[i].netin32;
    s.d_logits = sb[i].logits; s.d_heat = sb[i].heat; s.d_mask = sb[i].mask;
    s.rec = (PostRecord*)app->pinned + (size_t)i * B;
    s.stamps = (StageStamps*)((PostRecord*)app->pinned + (size_t)depth * B) + i;
    s.results.resize(B);
    {
      Op r;
      r.fam = F_RESIZE;
      ResizeParams& rp = r.resize;
      std::memset(&rp, 0, sizeof(rp));
      rp.batch = B; rp.src_pitch = d->frame_pitch;
      rp.dst_img_stride = (size_t)ph * pw * 4;
      rp.dst32_img_stride = (size_t)3 * d->net_h * d->net_w;
      rp.wi = d->frame_w; rp.hi = d->frame_h; rp.wo = d->net_w; rp.ho = d->net_h;
      rp.dst = s.d_netin; rp.dst_w = pw; rp.pad_l = pad; rp.pad_t = pad;
      rp.t_end = sb[i].t_stages;
      rp.dst_f32 = s.d_netin_f32; rp.lut32 = d_lut32; rp.lut16 = d_lut16;
      rp.rcp_dx = 1.0f / (2.0f * d->net_w); rp.rcp_dy = 1.0f / (2.0f * d->net_h);
      {
        // D = 4*wo*ho; l = ceil(log2 D); magic = ceil(2^(31+l) / D) < 2^32.  The error term
        // magic*D - 2^(31+l) is below D <= 2^l, so floor(n/D) = (n*magic) >> (31+l) for n < 2^31.
        const uint64_t D = 4ull * (uint64_t)d->net_w * (uint64_t)d->net_h;
        int l = 0;
        while ((1ull << l) < D) ++l;
        const unsigned __int128 num = (unsigned __int128)1 << (31 + l);
        rp.d_magic = (uint32_t)((num + D - 1) / D);
        rp.d_shift = (uint32_t)(l - 1);
      }
      // algorithmic bytes: the frame read once, three fp16 channels written per pixel (the
      // fourth, zero channel of the padded layout is this implementation's, not the method's)
      r.bytes = B * (3.0 * d->frame_w * d->frame_h + 6.0 * d->net_w * d->net_h +
                     (d->net_fp32_input ? 12.0 * d->net_w * d->net_h : 0.0));
      s.pre.push_back(r);
    }
    s.lane = i % lanes;
    s.infer = lane_b[s.lane]->ops;
    s.infer_layers = lane_b[s.lane]->layer_ops;
    if (b.stateful) s.wait_idx = b.lstm_conv_op;
    if (s.infer[b.first_conv_op].fam == F_STEM) s.infer[b.first_conv_op].stem.in = s.d_netin;
    else s.infer[b.first_conv_op].conv.in = s.d_netin;
    auto bind_logits = [&](auto& w, float*& logits) {
      logits = s.d_logits;
      w.theta = (float)theta_d;
      w.heat = s.d_heat; w.mask = s.d_mask; w.kmap = sb[i].kmap;
      w.t_end = sb[i].t_stages + 1;
    };
    Op& lo = s.infer[b.logits_op];
    if (lo.fam == F_CONV || lo.fam == F_NET) bind_logits(lo.conv, lo.conv.out_f32);
    else bind_logits(lo.lstm, lo.lstm.logits);
    if (!s.infer_layers.empty()) {
      s.infer_layers.front().conv.in = s.d_netin;
      bind_logits(s.infer_layers.back().conv, s.infer_layers.back().conv.out_f32);
    }
    if (lo.fam == F_NET && frame_net_pays(*d, mh, mw)) {
      Op o;
      o.fam = F_FRAME_NET;
      o.flops = lo.flops; o.bytes = s.pre[0].bytes;
      TinyFrameParams& f = o.frame_net;
      const ConvParams& c = lo.conv;
      std::memset(&f, 0, sizeof(f));
      f.r = s.pre[0].resize;
      f.wt_frag = c.wt_frag;
      f.out_f32 = c.out_f32; f.heat = c.heat; f.mask = c.mask; f.kmap = c.kmap; f.t_end = c.t_end; f.theta = c.theta;
      f.mid_h = c.mid_h; f.mid_w = c.mid_w; f.hout = c.hout; f.wout = c.wout; f.m = c.m; f.img_m = c.img_m;
      s.frame_net.push_back(o);
    }
    app->partial_bytes = b.partial_floats * sizeof(float);
    if (app->partial_bytes <= app->ctx->static_scratch_bytes && app->ctx->d_static_scratch) {
      // the same launches with every scratch pointer moved from the lane's scratch in the
      // workspace to the same offset inside the library's fixed array
      float* const from = lane_b[s.lane]->d_partial;
      float* const to = (float*)app->ctx->d_static_scratch;
      auto move = [&](auto*& ptr) {
        if (ptr) ptr = to + (ptr - from);
      };
      s.infer_static = s.infer;
      for (Op& op : s.infer_static) {
        if (op.fam == F_CONV) move(op.conv.partial);
        if (op.fam == F_LSTM) move(op.lstm.partial);
      }
    }
    {
      // Stage 3 behind the kernel that writes the logits (and, with them, the per-cell outputs) is the
      // channel maxima alone.  Only the annotation layer waits for them; without it they are found
      // in the overlay's launch, one launch (4 us) less, unless the kernels are being timed.
      Op p;
      p.fam = F_POST;
      p.post = PostParams{s.d_logits, (int)n_map, (float)theta_d, s.rec, B, sb[i].marks, mw, mh,
                          d->frame_w, d->frame_h, sb[i].t_stages + 2};
      p.bytes = B * 8.0 * n_map * 4;
      s.post.push_back(p);
      s.maxima_with_overlay = !d->annotate;
    }
    {
      Op o;
      o.fam = F_OVERLAY;
      OverlayParams& op = o.overlay;
      std::memset(&op, 0, sizeof(op));
      op.batch = B; op.pitch = d->frame_pitch;
      op.wf = d->frame_w; op.hf = d->frame_h;
      op.rcp_gpr = 1.0f / (float)((d->frame_w + 15) / 16); op.rcp_qpr = 1.0f / (float)((d->frame_w + 3) / 4);
      op.rcp_hf = 1.0f / (float)d->frame_h; op.rcp_wf = 1.0f / (float)d->frame_w;
      op.n_layers = 1;
      OverlayLayer& L = op.layer[0];
      L.kmap = sb[i].kmap; L.wm = mw; L.hm = mh;
      L.logits = s.d_logits; L.theta = (float)theta_d; L.t_stages = sb[i].t_stages;   // rec, stamps and n_max: per frame
      L.rcp_wm = 1.0f / (float)mw;
      L.a = a_q8;
      L.marks = sb[i].marks;
      L.arm = d->marker_arm; L.half = d->marker_half; L.scale = d->glyph_scale;
      for (int g = 0; g < 9; ++g) {
        uint64_t bits = 0;
        for (int r = 0; r < 7; ++r)
          for (int c = 0; c < 5; ++c)
            if ((d->glyphs[g][r] >> (4 - c)) & 1) bits |= 1ull << (5 * r + c);
        L.glyph[g] = bits;
      }
      for (int k = 0; k < 8; ++k)
        L.pal[k] = (uint32_t)d->palette[k][0] | ((uint32_t)d->palette[k][1] << 8) |
                   ((uint32_t)d->palette[k][2] << 16);
      o.bytes = B * (6.0 * d->frame_w * d->frame_h + 1.0 * n_map);
      s.overlay.push_back(o);
    }
    HS_HIP(hipEventCreate(&s.ev_pre));
    HS_HIP(hipEventCreate(&s.ev_infer));
    HS_HIP(hipEventCreate(&s.ev_post));
    HS_HIP(hipEventCreate(&s.ev_overlay));
    s.ev_done = s.ev_overlay;
    s.ev_stage3 = s.ev_post;
  }
  return HS_OK;
}

// ---- completion thread ---------------------------------------------------------------------------
// From the end of stage 2 until the last channel maximum of the frame (batch) was found, where that
// happened in the overlay's launch.  Stamped by the kernels themselves: an event for the start of that
// launch is a packet of its own in the queue (one 1080p frame 160 -> 167 us, twelve back to back 1189 -> 1256).
static float stage3_ms(const Slot& s, int khz) {
  int32_t ticks = 0;
  for (size_t j = 0; j < s.results.size(); ++j) ticks = std::max(ticks, *std::max_element(s.rec[j].ticks, s.rec[j].ticks + 8));
  return (float)ticks / (float)khz;
}

// From a stage's stamp, in the workgroup that ends last, until the event on that launch: events see a launch 0.8 to 1.0 us
// longer, at both ends together, than its workgroups' stamps do.
constexpr float kStampToEventMs = 0.0005f;
// From StageStamps::drawn until the overlay's end, unless the search for a channel's maximum, one workgroup's on a map of any size, takes
// longer: a frame ends with the later of the two.  Against the event behind stage 2, in plain frames of 64 x 48 to 4000 x 1000
// pixels and batches of 4 to 16, groups and quads, both networks: medians of -0.4 to 2.5 us after drawn, or -0.4 to 0.4 after the maxima
// where they are the later ones (1920 x 1080 pixels, a map of 160 x 90: 13.8 us after drawn).
constexpr float kDrawnToEndMs = 0.001f;

static void completer_main(hs_app* app) {
  (void)hipSetDevice(app->ctx->device);
  for (;;) {
    Slot* s = nullptr;
    {
      std::unique_lock<std::mutex> lk(app->mu);
      app->cv_work.wait(lk, [&] { return app->stop || app->n_completed < app->n_submitted; });
      if (app->n_completed >= app->n_submitted) return;   // stop requested and nothing pending
      s = &app->slots[app->n_completed % app->depth];
    }
    hipError_t e = hipEventSynchronize(s->ev_done);
    const uint64_t t_done = now_ns();
    float ms_pre = 0, ms_inf = 0, ms_post = 0;
    if (s->stamped) {
      const StageStamps& t = *s->stamps;
      auto span = [&](uint64_t from, uint64_t to) { return (float)(int64_t)(to - from) / (float)app->ctx->wall_clock_khz; };
      float ms = 0;                      // from the stamp of ev_stage3's stage on
      if (!s->end_stamped && e == hipSuccess) e = hipEventElapsedTime(&ms, s->ev_stage3, s->ev_done);
      const float maxima_ms = s->maxima_rode ? stage3_ms(*s, app->ctx->wall_clock_khz) : 0.0f;
      ms = s->end_stamped ? std::max(span(t.infer, t.drawn) + kDrawnToEndMs, maxima_ms) : ms + kStampToEventMs;
      ms_post = s->maxima_rode ? std::max(0.0f, ms - maxima_ms) : ms;
      ms_inf = s->maxima_rode ? ms : ms + span(t.infer, t.post);
      ms_pre = ms_inf + span(t.pre, t.infer);
    } else {
      if (e == hipSuccess) e = hipEventElapsedTime(&ms_pre, s->ev_pre, s->ev_done);
      if (e == hipSuccess) e = hipEventElapsedTime(&ms_inf, s->ev_infer, s->ev_done);
      if (s->maxima_rode) ms_post = std::max(0.0f, ms_inf - stage3_ms(*s, app->ctx->wall_clock_khz));
      else if (e == hipSuccess) e = hipEventElapsedTime(&ms_post, s->ev_stage3, s->ev_done);
    }
    auto back = [&](float ms) {
      const double ns = (double)ms * 1e6;
      return t_done - (uint64_t)std::max(0.0, ns);
    };
    for (size_t j = 0; j < s->results.size(); ++j) {
      hs_result& r = s->results[j];
      r.t_overlay_done_ns = t_done;
      r.t_pre_done_ns = back(ms_pre);
      r.t_infer_done_ns = back(ms_inf);
      r.t_post_done_ns = back(ms_post);
      std::memcpy(r.argmax_idx, s->rec[j].argmax_idx, sizeof(r.argmax_idx));
      std::memcpy(r.peak, s->rec[j].peak, sizeof(r.peak));
      std::memcpy(r.present, s->rec[j].present, sizeof(r.present));
    }
    {
      std::lock_guard<std::mutex> lk(app->mu);
      if (e != hipSuccess && app->completer_error.empty())
        app->completer_error.set(hipGetErrorString(e));
      s->state = SLOT_DONE;
      app->n_completed++;
      app->completed_pub.store(app->n_completed, std::memory_order_release);
    }
    app->cv_done.notify_all();
  }
}

static void destroy_streams(hs_app* app) {
  if (app->s_overlay && app->s_overlay != app->s_lane[0]) (void)hipStreamDestroy(app->s_overlay);
  for (int l = kMaxLanes - 1; l >= 0; --l)
    if (app->s_lane[l] && (l == 0 || app->s_lane[l] != app->s_lane[0]))
      (void)hipStreamDestroy(app->s_lane[l]);
  for (int l = 0; l < kMaxLanes; ++l) app->s_lane[l] = nullptr;
  app->s_overlay = nullptr;
}

static hs_status make_streams(hs_app* app, const uint32_t* mi, const uint32_t* mo, int n_words) {
  hipStream_t sl[kMaxLanes] = {nullptr};
  hipStream_t so = nullptr;
  hipError_t e = hipSuccess;
  if (mi && std::memcmp(mi, mo, sizeof(uint32_t) * (size_t)n_words) == 0) {
    // equal masks: one stream, i.e. one hardware queue, carries all four stages of every lane
    e = hipExtStreamCreateWithCUMask(&sl[0], (uint32_t)n_words, mi);
    so = sl[0];
  } else if (mi) {
    e = hipExtStreamCreateWithCUMask(&sl[0], (uint32_t)n_words, mi);
    if (e == hipSuccess) e = hipExtStreamCreateWithCUMask(&so, (uint32_t)n_words, mo);
  } else if (app->lanes > 1) {
    // the overlay follows its frame's stream (the lanes already overlap one frame's overlay
    // with the next frame's first stages): lanes streams per application, no more
    for (int l = 0; l < app->lanes && e == hipSuccess; ++l)
      e = hipStreamCreateWithFlags(&sl[l], hipStreamNonBlocking);
  } else {
    e = hipStreamCreateWithFlags(&sl[0], hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&so, hipStreamNonBlocking);
  }
  if (e != hipSuccess) {
    for (int l = 0; l < kMaxLanes; ++l)
      if (sl[l]) (void)hipStreamDestroy(sl[l]);
    if (so && so != sl[0]) (void)hipStreamDestroy(so);
    set_error("creating the application's streams failed: %s", hipGetErrorString(e));
    return HS_E_DEVICE;
  }
  for (int l = 1; l < kMaxLanes; ++l)
    if (!sl[l]) sl[l] = sl[0];   // partitioned, or fewer lanes: in one queue, in order
  destroy_streams(app);
  for (int l = 0; l < kMaxLanes; ++l) {
    app->s_lane[l] = sl[l];
    app->lane_last_stream[l] = nullptr;   // no frame is in flight here
  }
  app->s_overlay = so;
  return HS_OK;
}

static void close_queue_openers(hs_ctx* ctx) {
  for (hipStream_t& st : ctx->queue_openers) {
    if (st) (void)hipStreamDestroy(st);
    st = nullptr;
  }
}

static bool frames_in_flight(hs_app* app) {
  std::lock_guard<std::mutex> lk(app->mu);
  return app->n_completed < app->n_submitted;
}

static void collect_timing(hs_app* app) {
  for (TimedLaunch& t : app->timed) {
    float ms = 0;
    if (t.e1 && hipEventSynchronize(t.e1) == hipSuccess && hipEventElapsedTime(&ms, t.e0, t.e1) == hipSuccess) {
      app->acc_ms[t.fam] += ms;
      app->acc_flops[t.fam] += t.flops;
      app->acc_bytes[t.fam] += t.bytes;
      app->acc_n[t.fam] += 1;
    }
    if (t.e0) (void)hipEventDestroy(t.e0);
    if (t.e1) (void)hipEventDestroy(t.e1);
  }
  app->timed.clear();
}

// Waits for the application's frames and gives back everything it holds; one that is only half made
// holds less.
static void release_app(hs_app* app) {
  (void)hipSetDevice(app->ctx->device);
  {
    std::lock_guard<std::mutex> lk(app->mu);
    app->stop = true;
  }
  app->cv_work.notify_all();
  if (app->completer.joinable()) app->completer.join();   // drains pending frames first
  for (int l = 0; l < kMaxLanes; ++l)
    if (app->s_lane[l]) (void)hipStreamSynchronize(app->s_lane[l]);
  if (app->s_overlay) (void)hipStreamSynchronize(app->s_overlay);
  collect_timing(app);
  for (Slot& s : app->slots) {
    if (s.graph_exec) (void)hipGraphExecDestroy(s.graph_exec);
    if (s.graph) (void)hipGraphDestroy(s.graph);
    for (hipEvent_t ev : {s.ev_pre, s.ev_infer, s.ev_post, s.ev_overlay})
      if (ev) (void)hipEventDestroy(ev);
  }
  destroy_streams(app);
  if (app->pinned) (void)hipHostFree(app->pinned);
  {
    std::lock_guard<std::mutex> lk(app->ctx->mu);
    auto& v = app->ctx->apps;
    v.erase(std::remove(v.begin(), v.end(), app), v.end());
  }
  delete app;
}

// done: event that completes with the last of the launched ops.
static hs_status run_ops(hs_app* app, std::vector<Op>& ops, hipStream_t st, hipEvent_t done,
                         size_t first = 0, size_t last = (size_t)-1) {
  last = std::min(last, ops.size());
  for (size_t i = first; i < last; ++i) {
    Op& op = ops[i];
    if (app->timing) {
      app->timed.push_back(TimedLaunch{op.fam, op.flops, op.bytes, nullptr, nullptr});
      TimedLaunch& t = app->timed.back();
      HS_HIP(hipEventCreate(&t.e0));
      HS_HIP(hipEventCreate(&t.e1));
      // events attached to the dispatch itself: elapsed = the kernel's own begin -> end
      // time stamps, without the gap between consecutive dispatches
      const KernelDesc d = op_desc(op);
      void* args[1] = {op_params(op)};
      HS_HIP(hipExtLaunchKernel(d.func, d.grid, d.block, args, d.shmem, st, t.e0, t.e1, 0));
    } else {
      HS_HIP(launch_op(op, st, i + 1 == last ? done : nullptr));
    }
  }
  if (app->timing && done) HS_HIP(hipEventRecord(done, st));   // the dispatch carries e1 already
  return HS_OK;
}

static hipKernelNodeParams node_params(Op& op, void** args) {
  const KernelDesc d = op_desc(op);
  hipKernelNodeParams kp;
  std::memset(&kp, 0, sizeof(kp));
  kp.func = const_cast<void*>(d.func);
  kp.gridDim = d.grid;
  kp.blockDim = d.block;
  kp.sharedMemBytes = d.shmem;
  args[0] = op_params(op);
  kp.kernelParams = args;
  kp.extra = nullptr;
  return kp;
}

// Stages 1-3 of one queue slot as a linear HIP graph: resize, [event], network kernels,
// [event], postprocess.  Built once; per frame only the resize node's source pointer changes.
// wait_ev: the previous slot's ev_infer (the frame before this slot's frame ran there).
static hs_status build_slot_graph(Slot& s, hipEvent_t wait_ev) {
  HS_HIP(hipGraphCreate(&s.graph, 0));
  hipGraphNode_t prev = nullptr;
  auto add_kernel = [&](Op& op, hipGraphNode_t* out) -> hipError_t {
    void* args[1];
    hipKernelNodeParams kp = node_params(op, args);
    hipGraphNode_t n = nullptr;
    hipError_t e = hipGraphAddKernelNode(&n, s.graph, prev ? &prev : nullptr, prev ? 1 : 0, &kp);
    prev = n;
    if (out) *out = n;
    return e;
  };
  auto add_event = [&](hipEvent_t ev) -> hipError_t {
    hipGraphNode_t n = nullptr;
    hipError_t e = hipGraphAddEventRecordNode(&n, s.graph, &prev, 1, ev);
    prev = n;
    return e;
  };
  s.resize_nodes.resize(s.pre.size());
  for (size_t j = 0; j < s.pre.size(); ++j) HS_HIP(add_kernel(s.pre[j], &s.resize_nodes[j]));
  HS_HIP(add_event(s.ev_pre));
  for (size_t j = 0; j < s.infer.size(); ++j) {
    if ((int)j == s.wait_idx && wait_ev) {
      hipGraphNode_t n = nullptr;
      HS_HIP(hipGraphAddEventWaitNode(&n, s.graph, &prev, 1, wait_ev));
      prev = n;
    }
    HS_HIP(add_kernel(s.infer[j], nullptr));
  }
  HS_HIP(add_event(s.ev_infer));
  if (!s.maxima_with_overlay)
    for (Op& op : s.post) HS_HIP(add_kernel(op, nullptr));
  HS_HIP(hipGraphInstantiate(&s.graph_exec, s.graph, nullptr, nullptr, 0));
  return HS_OK;
}

}  // namespace hs

// ================================================================================================
int hs_internal_app_batch(const hs_app* app) { return app->batch; }
int hs_internal_app_grouped(const hs_app* app) { return app->group != nullptr; }
int hs_internal_current_device() {
  int device = -1;
  return hipGetDevice(&device) == hipSuccess ? device : -1;
}
void hs_internal_use_device(int device) {
  if (device >= 0) (void)hipSetDevice(device);
}

extern "C" {

hs_status hs_init(int device, hs_ctx** out) {
  return guarded("hs_init", [&]() -> hs_status {
  if (!out) { set_error("hs_init: NULL out"); return HS_E_INVAL; }
  *out = nullptr;
  int n = 0;
  hipError_t e = hipGetDeviceCount(&n);
  if (e != hipSuccess || device < 0 || device >= n) {
    set_error("hs_init: no HIP device %d (%s)", device,
              e == hipSuccess ? "out of range" : hipGetErrorString(e));
    return HS_E_DEVICE;
  }
  HS_HIP(hipSetDevice(device));
  hipDeviceProp_t prop;
  HS_HIP(hipGetDeviceProperties(&prop, device));
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
    set_error("hs_init: device %d is %s; this library contains gfx950 code only", device,
              prop.gcnArchName);
    return HS_E_DEVICE;
  }
  int clock_khz = 0;
  HS_HIP(hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, device));
  if (clock_khz <= 0) { set_error("hs_init: device %d has no constant-rate clock", device); return HS_E_DEVICE; }
  // the fixed scratch array of this device (for hs_submit_frame_static_scratch)
  void* d_scratch = nullptr;
  size_t scratch_bytes = 0;
  HS_HIP(static_scratch_address(&d_scratch, &scratch_bytes));
  hs_ctx* c = new hs_ctx();
  c->device = device;
  c->n_cus = prop.multiProcessorCount;
  c->wall_clock_khz = clock_khz;
  c->d_static_scratch = d_scratch;
  c->static_scratch_bytes = scratch_bytes;
  for (hipStream_t& st : c->queue_openers) {
    const hipError_t es = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
    if (es != hipSuccess) {
      close_queue_openers(c);
      delete c;
      set_error("hs_init: creating a stream failed: %s", hipGetErrorString(es));
      return HS_E_DEVICE;
    }
  }
  *out = c;
  return HS_OK;
  });
}

hs_status hs_shutdown(hs_ctx* ctx) {
  if (!ctx) { set_error("hs_shutdown: NULL"); return HS_E_INVAL; }
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    if (!ctx->apps.empty()) {
      set_error("hs_shutdown: %zu applications still exist", ctx->apps.size());
      return HS_E_STATE;
    }
  }
  close_queue_openers(ctx);
  delete ctx;
  return HS_OK;
}

hs_status hs_device_cus(hs_ctx* ctx, int* n_cus) {
  if (!ctx || !n_cus) { set_error("hs_device_cus: NULL"); return HS_E_INVAL; }
  *n_cus = ctx->n_cus;
  return HS_OK;
}

hs_status hs_device_copy(hs_ctx* ctx, void* d_dst, const void* d_src, size_t bytes) {
  if (!ctx || !d_dst || !d_src || bytes % 16 != 0 || ((uintptr_t)d_dst & 15) || ((uintptr_t)d_src & 15)) {
    set_error("hs_device_copy: NULL, misaligned pointer or size not a multiple of 16");
    return HS_E_INVAL;
  }
  HS_HIP(hipSetDevice(ctx->device));
  launch_copy(d_dst, d_src, bytes, nullptr);
  HS_HIP(hipGetLastError());
  HS_HIP(hipStreamSynchronize(nullptr));
  return HS_OK;
}

hs_status hs_partition_copy(hs_app* app, void* d_dst, const void* d_src, size_t bytes,
                            int repeats, double* seconds_per_copy) {
  if (!app || !d_dst || !d_src || !seconds_per_copy || repeats < 1 || bytes == 0 ||
      bytes % 16 != 0 || ((uintptr_t)d_dst & 15) || ((uintptr_t)d_src & 15)) {
    set_error("hs_partition_copy: NULL, misaligned pointer, size not a multiple of 16 or repeats < 1");
    return HS_E_INVAL;
  }
  if (frames_in_flight(app)) { set_error("hs_partition_copy: frames in flight"); return HS_E_STATE; }
  HS_HIP(hipSetDevice(app->ctx->device));
  hipStream_t st = app->s_overlay ? app->s_overlay : app->s_lane[0];
  hipEvent_t e0 = nullptr, e1 = nullptr;
  HS_HIP(hipEventCreate(&e0));
  hipError_t e = hipEventCreate(&e1);
  if (e == hipSuccess) {
    launch_copy(d_dst, d_src, bytes, st);   // untimed: first touch of the buffers
    e = hipEventRecord(e0, st);
  }
  for (int i = 0; i < repeats && e == hipSuccess; ++i) {
    launch_copy(d_dst, d_src, bytes, st);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipEventRecord(e1, st);
  if (e == hipSuccess) e = hipEventSynchronize(e1);
  float ms = 0;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
  (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (e != hipSuccess) {
    set_error("hs_partition_copy: %s", hipGetErrorString(e));
    return HS_E_DEVICE;
  }
  *seconds_per_copy = (double)ms * 1e-3 / repeats;
  return HS_OK;
}

hs_status hs_query_workspace(const hs_app_desc* desc, size_t* bytes) {
  return guarded("hs_query_workspace", [&]() -> hs_status {
  if (!bytes) { set_error("hs_query_workspace: NULL bytes"); return HS_E_INVAL; }
  hs_status st = validate_desc(desc);
  if (st != HS_OK) return st;
  return build_plan(desc, nullptr, bytes);
  });
}

hs_status hs_create_app(hs_ctx* ctx, const hs_app_desc* desc, hs_app** out) {
  return guarded("hs_create_app", [&]() -> hs_status {
  if (!ctx || !out) { set_error("hs_create_app: NULL argument"); return HS_E_INVAL; }
  *out = nullptr;
  hs_status st = validate_desc(desc);
  if (st != HS_OK) return st;
  if (!desc->weights || desc->weight_floats != expected_weight_floats(desc->net)) {
    set_error("weight blob has %zu floats, network needs %zu", desc->weights ? desc->weight_floats : 0,
              expected_weight_floats(desc->net));
    return HS_E_INVAL;
  }
  if (!desc->d_workspace || ((uintptr_t)desc->d_workspace & 255) != 0) {
    set_error("d_workspace must be a 256-byte aligned device pointer");
    return HS_E_INVAL;
  }
  HS_HIP(hipSetDevice(ctx->device));
  // whatever ends this call early, an exception included, gives back what has been made so far
  std::unique_ptr<hs_app, void (*)(hs_app*)> app(new hs_app(), release_app);
  app->ctx = ctx;
  app->desc = *desc;
  app->desc.weights = nullptr;   // not retained
  app->depth = desc->queue_depth;
  size_t need = 0;
  st = build_plan(desc, app.get(), &need);
  for (size_t i = 0; st == HS_OK && i < app->slots.size(); ++i) {
    const size_t n_slots = app->slots.size();
    st = build_slot_graph(app->slots[i],
                          n_slots > 1 ? app->slots[(i + n_slots - 1) % n_slots].ev_infer : nullptr);
  }
  if (st == HS_OK) st = make_streams(app.get(), nullptr, nullptr, 0);
  if (st != HS_OK) return st;
  app->completer = std::thread(completer_main, app.get());
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    ctx->apps.push_back(app.get());
    app->home_lane = (int)(ctx->n_created++ / 2 % (unsigned)app->lanes);
  }
  *out = app.release();
  return HS_OK;
  });
}

hs_status hs_destroy_app(hs_app* app) {
  if (!app) { set_error("hs_destroy_app: NULL"); return HS_E_INVAL; }
  if (app->group) { set_error("hs_destroy_app: destroy the application's group first"); return HS_E_STATE; }
  release_app(app);
  return HS_OK;
}

// Lane the most recently submitted frame ran in (0 before the first frame).
static int last_frame_lane(hs_app* app) {
  std::lock_guard<std::mutex> lk(app->mu);
  if (app->n_submitted == 0) return app->lanes - 1;   // so that the "next" lane is lane 0
  return app->slots[(app->n_submitted - 1) % app->depth].lane;
}

hs_status hs_reset_state(hs_app* app) {
  if (!app) { set_error("hs_reset_state: NULL"); return HS_E_INVAL; }
  if (frames_in_flight(app)) { set_error("hs_reset_state: frames in flight"); return HS_E_STATE; }
  if (!app->stateful) return HS_OK;
  HS_HIP(hipSetDevice(app->ctx->device));
  const size_t n = (size_t)app->map_w * app->map_h * app->batch;
  launch_fill_zero(app->d_c, n * app->hid * sizeof(float), app->s_lane[0]);
  for (int l = 0; l < app->lanes; ++l)
    launch_fill_zero(app->d_concat[l], n * app->concat_pitch * sizeof(f16), app->s_lane[0]);
  HS_HIP(hipGetLastError());
  HS_HIP(hipStreamSynchronize(app->s_lane[0]));
  return HS_OK;
}

hs_status hs_get_state(hs_app* app, int stream, float* h_out, float* c_out) {
  return guarded("hs_get_state", [&]() -> hs_status {
  if (!app) { set_error("hs_get_state: NULL"); return HS_E_INVAL; }
  if (!app->stateful) { set_error("hs_get_state: network has no recurrent state"); return HS_E_INVAL; }
  if (stream < 0 || stream >= app->batch) { set_error("hs_get_state: no stream %d", stream); return HS_E_INVAL; }
  if (frames_in_flight(app)) { set_error("hs_get_state: frames in flight"); return HS_E_STATE; }
  HS_HIP(hipSetDevice(app->ctx->device));
  const size_t n = (size_t)app->map_w * app->map_h;
  const int hid = app->hid;
  if (c_out) {
    std::vector<float> tmp(n * hid);
    HS_HIP(hipMemcpy(tmp.data(), app->d_c + (size_t)stream * n * hid, tmp.size() * sizeof(float),
                     hipMemcpyDeviceToHost));
    for (size_t m = 0; m < n; ++m)
      for (int j = 0; j < hid; ++j) c_out[(size_t)j * n + m] = tmp[m * hid + j];
  }
  if (h_out) {
    // h of the last frame sits where the NEXT frame's gate convolution will read it
    const f16* cat = app->d_concat[(last_frame_lane(app) + 1) % app->lanes];
    std::vector<f16> tmp(n * app->concat_pitch);
    HS_HIP(hipMemcpy(tmp.data(), cat + (size_t)stream * n * app->concat_pitch,
                     tmp.size() * sizeof(f16), hipMemcpyDeviceToHost));
    for (size_t m = 0; m < n; ++m)
      for (int j = 0; j < hid; ++j)
        h_out[(size_t)j * n + m] = (float)tmp[m * app->concat_pitch + app->x_ch + j];
  }
  return HS_OK;
  });
}

hs_status hs_get_features(hs_app* app, int stream, float* x_out) {
  return guarded("hs_get_features", [&]() -> hs_status {
  if (!app || !x_out) { set_error("hs_get_features: NULL"); return HS_E_INVAL; }
  if (!app->stateful) { set_error("hs_get_features: network has no recurrent cell"); return HS_E_INVAL; }
  if (stream < 0 || stream >= app->batch) { set_error("hs_get_features: no stream %d", stream); return HS_E_INVAL; }
  if (frames_in_flight(app)) { set_error("hs_get_features: frames in flight"); return HS_E_STATE; }
  HS_HIP(hipSetDevice(app->ctx->device));
  const size_t n = (size_t)app->map_w * app->map_h;
  std::vector<f16> tmp(n * app->concat_pitch);
  const f16* cat = app->d_concat[last_frame_lane(app)];
  HS_HIP(hipMemcpy(tmp.data(), cat + (size_t)stream * n * app->concat_pitch,
                   tmp.size() * sizeof(f16), hipMemcpyDeviceToHost));
  for (size_t m = 0; m < n; ++m)
    for (int j = 0; j < app->x_ch; ++j)
      x_out[(size_t)j * n + m] = (float)tmp[m * app->concat_pitch + j];
  return HS_OK;
  });
}

// CUs that a launch under the mask keeps busy.  Bit i is a CU of XCD i mod 8, in its shader engine i / 8 mod 4, and workgroups
// are dealt out evenly to the engines that have CUs: the one with the fewest sets the pace.  (Every layer timed on 80 CUs, two or
// three per engine, takes as long as on 64: gates of two 854 x 480 frames 31.6 and 31.4 us; on 40 as on 32.)
static int effective_cus(const uint32_t* mask, int n_words, int device_cus) {
  const int xcds = xcd_count(device_cus);
  constexpr int kEngines = 4;
  std::vector<int> n((size_t)xcds * kEngines, 0);
  for (int i = 0; i < device_cus && i < 32 * n_words; ++i)
    if (mask[i / 32] >> (i % 32) & 1u) ++n[(size_t)(i % xcds * kEngines + i / xcds % kEngines)];
  int engines = 0, fewest = device_cus;
  for (int k : n)
    if (k) { ++engines; fewest = std::min(fewest, k); }
  return engines ? engines * fewest : device_cus;
}

// The plans of the network's layers for that many CUs (of those that k_conv3x3_run and k_conv3x3s2_run compute).  Made before
// anything changes: planning allocates.
static std::vector<ConvParams> plans_for_cus(const hs_app* app, int cus) {
  std::vector<ConvParams> plans;
  for (const Op& op : app->slots[0].infer)
    if (op.fam == F_CONV && op.conv.variant == CONV_KW) {
      plans.push_back(op.conv);
      Builder::choose_split(plans.back(), &op.conv, cus);
    }
  return plans;
}
// Every slot's launches take them, each with its own buffers.  (A slot's graph keeps the forms that it was built with.)
static void take_plans(hs_app* app, const std::vector<ConvParams>& plans) {
  for (Slot& s : app->slots)
    for (std::vector<Op>* ops : {&s.infer, &s.infer_static}) {
      size_t n = 0;
      for (Op& op : *ops) {
        if (op.fam != F_CONV || op.conv.variant != CONV_KW) continue;
        const ConvParams own = op.conv;
        op.conv = plans[n++];
        op.conv.in = own.in; op.conv.out = own.out; op.conv.out2 = own.out2; op.conv.res = own.res; op.conv.partial = own.partial;
      }
    }
}

hs_status hs_set_partition(hs_app* app, const uint32_t* cu_mask_infer,
                           const uint32_t* cu_mask_overlay, int n_words) {
  return guarded("hs_set_partition", [&]() -> hs_status {
  if (!app) { set_error("hs_set_partition: NULL app"); return HS_E_INVAL; }
  if ((cu_mask_infer == nullptr) != (cu_mask_overlay == nullptr)) {
    set_error("hs_set_partition: give both masks or neither");
    return HS_E_INVAL;
  }
  if (frames_in_flight(app)) { set_error("hs_set_partition: frames in flight"); return HS_E_STATE; }
  hs_ctx* ctx = app->ctx;
  HS_HIP(hipSetDevice(ctx->device));
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (!cu_mask_infer) {
    const std::vector<ConvParams> plans = plans_for_cus(app, Builder::kAllCus);
    hs_status st = make_streams(app, nullptr, nullptr, 0);
    if (st != HS_OK) return st;
    std::memset(app->claim, 0, sizeof(app->claim));
    app->partitioned = false;
    take_plans(app, plans);
    return HS_OK;
  }
  uint32_t others[HS_MAX_CU_WORDS] = {0};
  for (hs_app* o : ctx->apps)
    if (o != app)
      for (int w = 0; w < HS_MAX_CU_WORDS; ++w) others[w] |= o->claim[w];
  hs_status st = admission_check(others, cu_mask_infer, cu_mask_overlay, n_words, ctx->n_cus);
  if (st != HS_OK) return st;
  const std::vector<ConvParams> plans = plans_for_cus(app, effective_cus(cu_mask_infer, n_words, ctx->n_cus));
  st = make_streams(app, cu_mask_infer, cu_mask_overlay, n_words);
  if (st != HS_OK) return st;
  std::memset(app->claim, 0, sizeof(app->claim));
  for (int w = 0; w < n_words; ++w) app->claim[w] = cu_mask_infer[w] | cu_mask_overlay[w];
  app->partitioned = true;
  take_plans(app, plans);
  return HS_OK;
  });
}

// Marks the slot as in flight and wakes the completion thread (the last step of a submit).
static void finish_submit(hs_app* app, Slot* s) {
  const uint64_t t_enq = now_ns();
  for (hs_result& r : s->results) r.t_enqueued_ns = t_enq;
  {
    std::lock_guard<std::mutex> lk(app->mu);
    s->state = SLOT_INFLIGHT;
    app->n_submitted++;
  }
  app->cv_work.notify_one();
}

// Enqueues stages 1-3 of one batch and, with own_overlay, stage 4 as well.  Without it the
// caller draws the overlay (a group), records s->ev_overlay and calls finish_submit; *slot_out
// and *stream_out then name the slot taken and the stream whose tail is ev_stage3.
static hs_status enqueue_stages(hs_app* app, Slot* s, bool idle, const uint8_t* const* d_frames,
                                uint8_t* const* d_overlay_outs, uint64_t frame_id,
                                uint64_t t_submit, bool own_overlay, Slot** slot_out,
                                hipStream_t* stream_out, hipEvent_t frames_ready,
                                bool static_scratch);

// A submit that fails after part of a frame has been handed to the GPU leaves the recurrent
// state advanced by a frame that is never delivered: the application is unusable from then on.
// Every later submit returns HS_E_DEVICE with this message.
static void poison(hs_app* app, const char* what) {
  std::lock_guard<std::mutex> lk(app->mu);
  if (app->completer_error.empty())
    app->completer_error.set("a submit failed after work had been enqueued (", what, "); destroy the application");
}

static hs_status submit_stages(hs_app* app, const uint8_t* const* d_frames,
                               uint8_t* const* d_overlay_outs, uint64_t frame_id,
                               uint64_t t_submit, bool own_overlay, Slot** slot_out,
                               hipStream_t* stream_out, hipEvent_t frames_ready = nullptr,
                               bool static_scratch = false) {
  if (!app || !d_frames || !d_overlay_outs) { set_error("hs_submit_batch: NULL argument"); return HS_E_INVAL; }
  const int B = app->batch;
  for (int j = 0; j < B; ++j) {
    if (!d_frames[j] || !d_overlay_outs[j]) { set_error("hs_submit_batch: NULL frame pointer"); return HS_E_INVAL; }
    if (((uintptr_t)d_frames[j] & 15) || ((uintptr_t)d_overlay_outs[j] & 15)) {
      set_error("hs_submit_batch: frame pointers must be 16-byte aligned");
      return HS_E_INVAL;
    }
    if (d_frames[j] == d_overlay_outs[j]) { set_error("hs_submit_batch: output aliases input"); return HS_E_INVAL; }
  }
  Slot* s = nullptr;
  bool idle = false;   // nothing in flight: this frame cannot overlap with an earlier one
  {
    std::lock_guard<std::mutex> lk(app->mu);
    if (!app->completer_error.empty()) {
      set_error("device error in an earlier frame: %s", app->completer_error.text);
      return HS_E_DEVICE;
    }
    if (app->n_submitted - app->n_delivered >= (uint64_t)app->depth) {
      set_error("hs_submit_batch: queue full (%d slots)", app->depth);
      return HS_E_QUEUE_FULL;
    }
    s = &app->slots[app->n_submitted % app->depth];
    idle = app->n_completed == app->n_submitted;
    if (static_scratch && !idle) {
      // one scratch array serves every frame that uses it: no second frame beside it
      set_error("hs_submit_frame_static_scratch: a frame of this application is still in flight");
      return HS_E_STATE;
    }
  }
  const hs_status st = guarded("hs_submit_batch", [&] {    // timed launches are noted in a list that grows
    return enqueue_stages(app, s, idle, d_frames, d_overlay_outs, frame_id, t_submit, own_overlay,
                          slot_out, stream_out, frames_ready, static_scratch);
  });
  if (st != HS_OK) poison(app, hs_last_error());
  return st;
}

// `stream` goes on behind `event` (ev_stage3, or at a recurrent cell ev_infer) of frame `before`, which may be in flight;
// where that frame has no such event, behind its overlay.
static hs_status order_behind(hipStream_t stream, const Slot& before, hipEvent_t Slot::*event) {
  if (before.stream == stream) return HS_OK;             // one queue: in order
  HS_HIP(hipStreamWaitEvent(stream, before.has_event ? before.*event : before.ev_overlay, 0));
  return HS_OK;
}

static hs_status enqueue_stages(hs_app* app, Slot* s, bool idle, const uint8_t* const* d_frames,
                                uint8_t* const* d_overlay_outs, uint64_t frame_id,
                                uint64_t t_submit, bool own_overlay, Slot** slot_out,
                                hipStream_t* stream_out, hipEvent_t frames_ready,
                                bool static_scratch) {
  HS_HIP(hipSetDevice(app->ctx->device));
  std::vector<Op>& infer = static_scratch ? s->infer_static : s->infer;
  const int B = app->batch;
  const size_t n_map = (size_t)app->map_w * app->map_h;
  const size_t netin_img = (size_t)app->netin_h * app->netin_w * 4;
  for (int j = 0; j < B; ++j) {
    hs_result& r = s->results[j];
    std::memset(&r, 0, sizeof(r));
    r.frame_id = frame_id;
    r.t_submit_ns = t_submit;
    r.map_w = app->map_w; r.map_h = app->map_h;
    r.net_input_pitch_bytes = (size_t)app->netin_w * 4 * sizeof(f16);
    r.d_overlay = d_overlay_outs[j];
    r.d_mask = s->d_mask + j * 8 * n_map;
    r.d_heat = s->d_heat + j * 8 * n_map;
    r.d_logits = s->d_logits + j * 8 * n_map;
    r.d_net_input = s->d_netin + j * netin_img +
                    ((size_t)app->netin_pad * app->netin_w + app->netin_pad) * 4;
    r.d_net_input_f32 = s->d_netin_f32
                            ? s->d_netin_f32 + (size_t)j * 3 * app->desc.net_h * app->desc.net_w
                            : nullptr;
    s->pre[0].resize.src[j] = d_frames[j];
    s->overlay[0].overlay.src[j] = d_frames[j];
    s->overlay[0].overlay.dst[j] = d_overlay_outs[j];
  }

  hs_status st = HS_OK;
  // A frame that finds the application idle runs on the home lane's stream whatever its lane (paced
  // streams then use one queue, like a single-lane application); otherwise on the stream after
  // the previous frame's, behind its lane's previous frame if that one ran elsewhere (they share
  // activation buffers).
  app->last_stream = idle ? app->home_lane : (app->last_stream + 1) % app->lanes;
  hipStream_t lane_stream = app->s_lane[app->last_stream];
  const bool graph = app->launch_mode == HS_LAUNCH_GRAPH && !app->timing && !static_scratch;
  const bool maxima_here = s->maxima_with_overlay && !app->timing;
  s->overlay[0].overlay.layer[0].rec = maxima_here ? s->rec : nullptr;
  s->overlay[0].overlay.n_max = maxima_here ? 8 : 0;
  hipStream_t ov_stream = app->s_overlay ? app->s_overlay : lane_stream;
  s->stamped = !graph && !app->timing;
  s->overlay[0].overlay.layer[0].stamps = s->stamped ? s->stamps : nullptr;
  // An event on a stage's last kernel costs 4.6 us of its queue.  Whoever waits for this frame's stage 2 or 3: the overlay
  // on another stream, a group's overlay, or the next frame in another lane if it comes while this one is in flight: at
  // its recurrent cell, or where it follows a frame of its own lane in this stream.  A frame that comes alone has events
  // for a recurrent cell only: for the next frame to wait for its overlay instead measured 2 to 4 % on twelve full-HD
  // frames back to back, and an event recorded when that frame comes (4 us of host) 1.5 % on five applications.
  const bool two_queues = app->lanes > 1 && app->s_lane[0] != app->s_lane[1];
  const bool others_wait = !own_overlay || ov_stream != lane_stream || (two_queues && (!idle || s->wait_idx >= 0));
  // What the overlay's last workgroup sees of the frame's end (kDrawnToEndMs) serves to tie the stages' stamps to it while
  // the workgroups run side by side, not held up by another frame, and take equally long: up to 1024 of 4096 pixels, or four times as
  // many of a quarter of the work.  With more of them it is up to 7 us early (a plain 7680 x 4320 frame), with annotations up to 11 (320 x 240).  Such frames have the
  // event behind stage 3 for it, and the completion thread spends 1 us (35 at an application's first frame) on its time.
  s->end_stamped = s->stamped && idle && !app->desc.annotate && !app->partitioned &&
                   (double)B * app->desc.frame_w * app->desc.frame_h <= 1024 * 4096.0;
  s->has_event = !s->stamped || others_wait || !s->end_stamped;
  s->overlay[0].overlay.stamp_end = s->end_stamped;
  s->stream = lane_stream;
  auto event = [&](hipEvent_t e, bool wanted) { return !s->stamped || wanted ? e : nullptr; };
  if (!idle && app->lane_last_stream[s->lane] && app->lane_last_stream[s->lane] != lane_stream &&
      app->depth >= app->lanes) {
    Slot& same_lane =
        app->slots[(size_t)((s - app->slots.data()) + app->depth - app->lanes) % app->depth];
    st = order_behind(lane_stream, same_lane, &Slot::ev_stage3);
    if (st != HS_OK) return st;
  }
  app->lane_last_stream[s->lane] = lane_stream;
  // the caller's producer (another stream) may still be writing the frames
  if (frames_ready) HS_HIP(hipStreamWaitEvent(lane_stream, frames_ready, 0));
  if (graph) {
    void* args[1];
    hipKernelNodeParams kp = node_params(s->pre[0], args);
    HS_HIP(hipGraphExecKernelNodeSetParams(s->graph_exec, s->resize_nodes[0], &kp));
    HS_HIP(hipGraphLaunch(s->graph_exec, lane_stream));
  } else {
    const bool frame_net = s->stamped && !static_scratch && !s->frame_net.empty();
    if (frame_net) std::copy_n(s->pre[0].resize.src, B, s->frame_net[0].frame_net.r.src);
    else st = run_ops(app, s->pre, lane_stream, event(s->ev_pre, false));
    if (st != HS_OK) return st;
    if (frame_net) {
      st = run_ops(app, s->frame_net, lane_stream, event(s->ev_infer, maxima_here ? s->has_event : others_wait));
    } else if (s->wait_idx >= 0 && app->depth > 1 && !idle) {
      // the recurrent cell waits for the previous frame's state update (other lane)
      Slot& before = app->slots[(size_t)((s - app->slots.data()) + app->depth - 1) % app->depth];
      st = run_ops(app, infer, lane_stream, nullptr, 0, (size_t)s->wait_idx);
      if (st != HS_OK) return st;
      st = order_behind(lane_stream, before, &Slot::ev_infer);
      if (st != HS_OK) return st;
      st = run_ops(app, infer, lane_stream, event(s->ev_infer, maxima_here ? s->has_event : others_wait), (size_t)s->wait_idx);
    } else {
      st = run_ops(app, infer, lane_stream, event(s->ev_infer, maxima_here ? s->has_event : others_wait));
    }
    if (st != HS_OK) return st;
    // (to time them; what they leave is the same up to the order of fp32 sums)
    if (app->timing && !s->frame_net.empty()) {
      std::copy_n(s->pre[0].resize.src, B, s->frame_net[0].frame_net.r.src);
      st = run_ops(app, s->frame_net, lane_stream, nullptr);
      if (st != HS_OK) return st;
    }
    if (app->timing && !s->infer_layers.empty()) st = run_ops(app, s->infer_layers, lane_stream, s->ev_infer);
    if (st != HS_OK) return st;
    if (!maxima_here) st = run_ops(app, s->post, lane_stream, event(s->ev_post, s->has_event));
    if (st != HS_OK) return st;
  }
  if (graph) HS_HIP(hipEventRecord(s->ev_post, lane_stream));
  s->ev_stage3 = !graph && maxima_here ? s->ev_infer : s->ev_post;
  s->maxima_rode = maxima_here;
  s->ev_done = s->ev_overlay;
  if (!own_overlay) {
    *slot_out = s;
    *stream_out = lane_stream;
    return HS_OK;
  }
  if (ov_stream != lane_stream) HS_HIP(hipStreamWaitEvent(ov_stream, s->ev_stage3, 0));
  st = run_ops(app, s->overlay, ov_stream, s->ev_overlay);
  if (st != HS_OK) return st;
  finish_submit(app, s);
  return HS_OK;
}

static hs_status refuse_grouped(hs_app* app, const char* fn) {
  if (app && app->group) {
    set_error("%s: the application is a member of a group; use the hs_*_group calls", fn);
    return HS_E_STATE;
  }
  return HS_OK;
}

hs_status hs_submit_batch(hs_app* app, const uint8_t* const* d_frames,
                          uint8_t* const* d_overlay_outs, uint64_t frame_id) {
  const uint64_t t_submit = now_ns();
  if (refuse_grouped(app, "hs_submit_batch") != HS_OK) return HS_E_STATE;
  return submit_stages(app, d_frames, d_overlay_outs, frame_id, t_submit, true, nullptr, nullptr);
}

hs_status hs_submit_batch_after(hs_app* app, const uint8_t* const* d_frames,
                                uint8_t* const* d_overlay_outs, uint64_t frame_id,
                                void* hip_event_frames_ready) {
  const uint64_t t_submit = now_ns();
  if (refuse_grouped(app, "hs_submit_batch_after") != HS_OK) return HS_E_STATE;
  return submit_stages(app, d_frames, d_overlay_outs, frame_id, t_submit, true, nullptr, nullptr,
                       (hipEvent_t)hip_event_frames_ready);
}

hs_status hs_submit_frame(hs_app* app, const uint8_t* d_frame, uint8_t* d_overlay_out,
                          uint64_t frame_id) {
  if (!app) { set_error("hs_submit_frame: NULL argument"); return HS_E_INVAL; }
  if (app->batch != 1) {
    set_error("hs_submit_frame: the application batches %d streams; use hs_submit_batch", app->batch);
    return HS_E_STATE;
  }
  return hs_submit_batch(app, &d_frame, &d_overlay_out, frame_id);
}

hs_status hs_submit_frame_static_scratch(hs_app* app, const uint8_t* d_frame,
                                         uint8_t* d_overlay_out, uint64_t frame_id) {
  const uint64_t t_submit = now_ns();
  if (!app) { set_error("hs_submit_frame_static_scratch: NULL argument"); return HS_E_INVAL; }
  if (refuse_grouped(app, "hs_submit_frame_static_scratch") != HS_OK) return HS_E_STATE;
  if (app->batch != 1) {
    set_error("hs_submit_frame_static_scratch: the application batches %d streams", app->batch);
    return HS_E_STATE;
  }
  if (app->timing) {   // per-kernel timing creates events, i.e. allocates
    set_error("hs_submit_frame_static_scratch: kernel timing is on");
    return HS_E_STATE;
  }
  if (app->slots[0].infer_static.empty()) {
    set_error("hs_submit_frame_static_scratch: a frame of this application needs %zu bytes of "
              "scratch for the gate pre-activations, the library's fixed array holds %zu", app->partial_bytes,
              app->ctx->static_scratch_bytes);
    return HS_E_NOMEM;
  }
  return submit_stages(app, &d_frame, &d_overlay_out, frame_id, t_submit, true, nullptr, nullptr,
                       nullptr, true);
}

// Copies the oldest finished batch's results (one per stream) out and frees its slot.
static hs_status deliver_locked(hs_app* app, hs_result* out) {
  Slot& s = app->slots[app->n_delivered % app->depth];
  const uint64_t t_obs = now_ns();
  for (size_t j = 0; j < s.results.size(); ++j) {
    out[j] = s.results[j];
    out[j].t_observed_ns = t_obs;
  }
  s.state = SLOT_FREE;
  app->n_delivered++;
  if (!app->completer_error.empty()) {
    set_error("device error: %s", app->completer_error.text);
    return HS_E_DEVICE;
  }
  return HS_OK;
}

hs_status hs_poll_batch(hs_app* app, hs_result* out) {
  if (!app || !out) { set_error("hs_poll_batch: NULL argument"); return HS_E_INVAL; }
  if (refuse_grouped(app, "hs_poll_batch") != HS_OK) return HS_E_STATE;
  std::lock_guard<std::mutex> lk(app->mu);
  if (app->n_delivered >= app->n_completed) {
    set_error("hs_poll_batch: no finished frame");
    return HS_E_NOT_READY;
  }
  return deliver_locked(app, out);
}

// Spins until the application has completed more than n_delivered frames, at most as long as a
// frame takes in practice (1 ms) and never past `deadline_ns` (now_ns clock); the caller then takes
// the lock and sleeps if need be.  A thread that sleeps on the condition variable sees a finished
// frame 7 us (one frame in flight) to 14 us (after 0.6 ms of sleep, its core idle) late.
// Only a thread that may run on four cores or more spins: one that is pinned, as the completion thread
// may be to the same core, or confined to a few would hold off the threads it waits for.  For the same
// reason it offers its core every 10 us (with every look, a third of a microsecond apart, the system
// call is where it spends its time: twelve 1080p frames back to back 1204 -> 1227 us).
static void spin_for_completion(hs_app* app, uint64_t n_delivered, uint64_t deadline_ns) {
  cpu_set_t cores;
  if (sched_getaffinity(0, sizeof(cores), &cores) != 0 || CPU_COUNT(&cores) < 4) return;
  uint64_t now = now_ns(), offer = now + 10000ull;
  const uint64_t until = std::min<uint64_t>(now + 1000000ull, deadline_ns);
  do {
    for (int i = 0; i < 32; ++i) {
      if (app->completed_pub.load(std::memory_order_acquire) > n_delivered) return;
      __builtin_ia32_pause();
    }
    now = now_ns();
    if (now >= offer) {
      (void)sched_yield();
      offer = now + 10000ull;
    }
  } while (now < until);
}

hs_status hs_wait_batch(hs_app* app, hs_result* out, uint64_t timeout_ns) {
  if (!app || !out) { set_error("hs_wait_batch: NULL argument"); return HS_E_INVAL; }
  if (refuse_grouped(app, "hs_wait_batch") != HS_OK) return HS_E_STATE;
  uint64_t delivered;
  bool running;            // nothing to deliver yet, and a frame in flight
  {
    std::lock_guard<std::mutex> lk(app->mu);
    delivered = app->n_delivered;
    running = app->n_delivered >= app->n_completed && app->n_completed < app->n_submitted;
  }
  const uint64_t deadline_ns = deadline_after(timeout_ns);
  if (running) spin_for_completion(app, delivered, deadline_ns);
  std::unique_lock<std::mutex> lk(app->mu);
  const bool ok = app->cv_done.wait_until(lk, clock_time(deadline_ns), [&] {
    return app->n_delivered < app->n_completed;
  });
  if (!ok) {
    set_error("hs_wait_batch: timed out");
    return HS_E_NOT_READY;
  }
  return deliver_locked(app, out);
}

hs_status hs_poll_result(hs_app* app, hs_result* out) {
  if (app && app->batch != 1) {
    set_error("hs_poll_result: the application batches %d streams; use hs_poll_batch", app->batch);
    return HS_E_STATE;
  }
  return hs_poll_batch(app, out);
}

hs_status hs_wait_result(hs_app* app, hs_result* out, uint64_t timeout_ns) {
  if (app && app->batch != 1) {
    set_error("hs_wait_result: the application batches %d streams; use hs_wait_batch", app->batch);
    return HS_E_STATE;
  }
  return hs_wait_batch(app, out, timeout_ns);
}

// ---- multi-network applications ---------------------------------------------------------------
static_assert(HS_MAX_GROUP == kMaxLayers, "one overlay layer per group member");

static void group_worker_main(GroupWorker* w, int device) {
  (void)hipSetDevice(device);
  for (;;) {
    {
      std::unique_lock<std::mutex> lk(w->mu);
      w->cv.wait(lk, [&] { return w->has_job || w->stop; });
      if (!w->has_job) return;
      w->has_job = false;
    }
    const hs_status st = submit_stages(w->app, &w->d_frame, &w->d_out, w->frame_id, w->t_submit,
                                       false, &w->slot, &w->tail);
    {
      std::lock_guard<std::mutex> lk(w->mu);
      w->status = st;
      if (st != HS_OK) w->error.set(hs_last_error());
      w->done = true;
    }
    w->cv.notify_all();
  }
}

hs_status hs_create_group(hs_ctx* ctx, hs_app* const* members, int n_members, hs_group** out) {
  return guarded("hs_create_group", [&]() -> hs_status {
  if (!ctx || !members || !out) { set_error("hs_create_group: NULL argument"); return HS_E_INVAL; }
  if (n_members < 1 || n_members > kMaxLayers) {
    set_error("hs_create_group: %d members, 1..%d allowed", n_members, kMaxLayers);
    return HS_E_INVAL;
  }
  for (int i = 0; i < n_members; ++i) {
    hs_app* a = members[i];
    if (!a || a->ctx != ctx) { set_error("hs_create_group: member %d is NULL or of another context", i); return HS_E_INVAL; }
    for (int j = 0; j < i; ++j)
      if (members[j] == a) { set_error("hs_create_group: member %d listed twice", i); return HS_E_INVAL; }
    if (a->batch != 1) { set_error("hs_create_group: member %d batches %d streams", i, a->batch); return HS_E_INVAL; }
    const hs_app_desc &d = a->desc, &d0 = members[0]->desc;
    if (d.frame_w != d0.frame_w || d.frame_h != d0.frame_h || d.frame_pitch != d0.frame_pitch) {
      set_error("hs_create_group: member %d takes another frame geometry than member 0", i);
      return HS_E_INVAL;
    }
    if (a->group) { set_error("hs_create_group: member %d already belongs to a group", i); return HS_E_STATE; }
    std::lock_guard<std::mutex> lk(a->mu);
    if (a->n_delivered != a->n_submitted) {
      set_error("hs_create_group: member %d has frames in flight or unpolled", i);
      return HS_E_STATE;
    }
  }
  std::unique_ptr<hs_group> g(new hs_group());
  g->ctx = ctx;
  g->members.assign(members, members + n_members);
  // the frame-level fields of the overlay launch come from member 0; layers are set per frame
  Op o = members[0]->slots[0].overlay[0];
  o.overlay.n_layers = n_members;
  double map_bytes = 0;
  for (hs_app* a : g->members) map_bytes += (double)a->map_w * a->map_h;
  o.bytes = 6.0 * members[0]->desc.frame_w * members[0]->desc.frame_h + map_bytes;
  g->overlay.push_back(o);
  for (int i = 1; i < n_members; ++i) {
    g->workers.push_back(std::make_unique<GroupWorker>());
    GroupWorker* w = g->workers.back().get();
    w->app = members[i];
    w->th = std::thread(group_worker_main, w, ctx->device);
  }
  for (hs_app* a : g->members) a->group = g.get();
  *out = g.release();
  return HS_OK;
  });
}

hs_status hs_destroy_group(hs_group* group) {
  if (!group) { set_error("hs_destroy_group: NULL"); return HS_E_INVAL; }
  for (hs_app* a : group->members) {   // frames in flight still need the group's bookkeeping
    std::unique_lock<std::mutex> lk(a->mu);
    a->cv_done.wait(lk, [&] { return a->n_completed == a->n_submitted; });
  }
  group->workers.clear();              // ends their threads
  for (hs_app* a : group->members) a->group = nullptr;
  delete group;
  return HS_OK;
}

hs_status hs_submit_group(hs_group* group, const uint8_t* d_frame, uint8_t* d_overlay_out,
                          uint64_t frame_id) {
  const uint64_t t_submit = now_ns();
  if (!group || !d_frame || !d_overlay_out) { set_error("hs_submit_group: NULL argument"); return HS_E_INVAL; }
  const size_t n = group->members.size();
  // nothing is enqueued unless every member can take the frame
  for (size_t i = 0; i < n; ++i) {
    hs_app* a = group->members[i];
    std::lock_guard<std::mutex> lk(a->mu);
    if (!a->completer_error.empty()) {
      set_error("device error in an earlier frame: %s", a->completer_error.text);
      return HS_E_DEVICE;
    }
    if (a->n_submitted - a->n_delivered >= (uint64_t)a->depth) {
      set_error("hs_submit_group: queue of member %d full (%d slots)", (int)i, a->depth);
      return HS_E_QUEUE_FULL;
    }
  }
  Slot* slot[kMaxLayers];
  hipStream_t tail[kMaxLayers];
  OverlayParams& op = group->overlay[0].overlay;
  for (auto& w : group->workers) {   // members 1.. on their own threads
    {
      std::lock_guard<std::mutex> lk(w->mu);
      w->d_frame = d_frame; w->d_out = d_overlay_out;
      w->frame_id = frame_id; w->t_submit = t_submit;
      w->done = false;
      w->has_job = true;
    }
    w->cv.notify_all();
  }
  hs_status st0 = submit_stages(group->members[0], &d_frame, &d_overlay_out, frame_id, t_submit,
                                false, &slot[0], &tail[0]);
  Message err0;
  if (st0 != HS_OK) err0.set(hs_last_error());
  for (size_t i = 1; i < n; ++i) {   // always collect every worker, also after a failure
    GroupWorker* w = group->workers[i - 1].get();
    std::unique_lock<std::mutex> lk(w->mu);
    w->cv.wait(lk, [&] { return w->done; });
    slot[i] = w->slot; tail[i] = w->tail;
    if (st0 == HS_OK && w->status != HS_OK) { st0 = w->status; err0 = w->error; }
  }
  // From here on a failure leaves some members a frame ahead of the others (their cells have
  // been updated by a frame that will never be delivered): the whole group is poisoned.
  auto fail_all = [&](hs_status st) {
    Message why;
    why.set(hs_last_error());
    for (hs_app* a : group->members) poison(a, why.text);
    set_error("%s", why.text);
    return st;
  };
  if (st0 != HS_OK) { set_error("%s", err0.text); return fail_all(st0); }
  op.n_max = 0;
  bool even = true;        // no member's annotations are drawn, and its maxima take as long to find as the others'
  for (const hs_app* a : group->members)
    even = even && !a->desc.annotate && !a->partitioned && a->map_w * a->map_h == group->members[0]->map_w * group->members[0]->map_h;
  op.stamp_end = 0;
  for (size_t i = 0; i < n; ++i) {
    slot[i]->end_stamped = slot[i]->end_stamped && even;       // (else its event: a member's stage 3 has one)
    if (slot[i]->end_stamped) op.stamp_end = 1;
    op.layer[i] = slot[i]->overlay[0].overlay.layer[0];
    if (op.layer[i].rec) op.n_max = 8 * (int)n;
  }
  op.src[0] = d_frame;
  op.dst[0] = d_overlay_out;
  // one launch draws every member's layer, on member 0's overlay stream, after all stage 3s
  hs_app* a0 = group->members[0];
  hipStream_t ov_stream = a0->s_overlay ? a0->s_overlay : tail[0];
  auto overlay_all = [&]() -> hs_status {
    for (size_t i = 0; i < n; ++i)
      if (tail[i] != ov_stream) HS_HIP(hipStreamWaitEvent(ov_stream, slot[i]->ev_stage3, 0));
    for (size_t i = 1; i < n; ++i) slot[i]->ev_done = slot[0]->ev_overlay;
    return run_ops(a0, group->overlay, ov_stream, slot[0]->ev_overlay);
  };
  const hs_status st = guarded("hs_submit_group", overlay_all);
  if (st != HS_OK) return fail_all(st);
  for (size_t i = 0; i < n; ++i) finish_submit(group->members[i], slot[i]);
  return HS_OK;
}

// Delivers one frame's results of all members if every member has finished it.
static hs_status deliver_group(hs_group* group, hs_result* out) {
  for (hs_app* a : group->members) {
    std::lock_guard<std::mutex> lk(a->mu);
    if (a->n_delivered >= a->n_completed) {
      set_error("hs_poll_group: no finished frame");
      return HS_E_NOT_READY;
    }
  }
  hs_status worst = HS_OK;
  for (size_t i = 0; i < group->members.size(); ++i) {
    hs_app* a = group->members[i];
    std::lock_guard<std::mutex> lk(a->mu);
    const hs_status st = deliver_locked(a, out + i);
    if (st != HS_OK) worst = st;
  }
  return worst;
}

hs_status hs_poll_group(hs_group* group, hs_result* out) {
  if (!group || !out) { set_error("hs_poll_group: NULL argument"); return HS_E_INVAL; }
  return deliver_group(group, out);
}

hs_status hs_wait_group(hs_group* group, hs_result* out, uint64_t timeout_ns) {
  if (!group || !out) { set_error("hs_wait_group: NULL argument"); return HS_E_INVAL; }
  const uint64_t deadline_ns = deadline_after(timeout_ns);
  for (hs_app* a : group->members) {
    std::unique_lock<std::mutex> lk(a->mu);
    if (a->n_delivered >= a->n_completed && a->n_completed < a->n_submitted) {
      const uint64_t delivered = a->n_delivered;
      lk.unlock();
      spin_for_completion(a, delivered, deadline_ns);
      lk.lock();
    }
    if (!a->cv_done.wait_until(lk, clock_time(deadline_ns), [&] { return a->n_delivered < a->n_completed; })) {
      set_error("hs_wait_group: timed out");
      return HS_E_NOT_READY;
    }
  }
  return deliver_group(group, out);
}

hs_status hs_set_launch_mode(hs_app* app, int mode) {
  if (!app) { set_error("hs_set_launch_mode: NULL"); return HS_E_INVAL; }
  if (mode != HS_LAUNCH_GRAPH && mode != HS_LAUNCH_EAGER) {
    set_error("hs_set_launch_mode: unknown mode %d", mode);
    return HS_E_INVAL;
  }
  if (frames_in_flight(app)) { set_error("hs_set_launch_mode: frames in flight"); return HS_E_STATE; }
  app->launch_mode = mode;
  return HS_OK;
}

hs_status hs_set_cpu_affinity(hs_app* app, int cpu) {
  if (!app) { set_error("hs_set_cpu_affinity: NULL"); return HS_E_INVAL; }
  cpu_set_t set;
  CPU_ZERO(&set);
  if (cpu < 0) {
    const long n = sysconf(_SC_NPROCESSORS_CONF);
    for (long c = 0; c < n && c < CPU_SETSIZE; ++c) CPU_SET((int)c, &set);
  } else {
    if (cpu >= CPU_SETSIZE) { set_error("hs_set_cpu_affinity: no such core %d", cpu); return HS_E_INVAL; }
    CPU_SET(cpu, &set);
  }
  int rc = pthread_setaffinity_np(app->completer.native_handle(), sizeof(set), &set);
  if (rc == 0 && app->group) {   // a group member's submitting thread follows its completion thread
    const auto& m = app->group->members;
    const size_t i = (size_t)(std::find(m.begin(), m.end(), app) - m.begin());
    if (i >= 1 && i < m.size())
      rc = pthread_setaffinity_np(app->group->workers[i - 1]->th.native_handle(), sizeof(set), &set);
  }
  if (rc != 0) {
    set_error("hs_set_cpu_affinity: core %d refused (%s)", cpu, strerror(rc));
    return HS_E_INVAL;
  }
  return HS_OK;
}

hs_status hs_set_kernel_timing(hs_app* app, int enable) {
  if (!app) { set_error("hs_set_kernel_timing: NULL"); return HS_E_INVAL; }
  if (frames_in_flight(app)) { set_error("hs_set_kernel_timing: frames in flight"); return HS_E_STATE; }
  (void)hipSetDevice(app->ctx->device);
  collect_timing(app);
  for (int f = 0; f < F_COUNT; ++f) {
    app->acc_ms[f] = app->acc_flops[f] = app->acc_bytes[f] = 0;
    app->acc_n[f] = 0;
  }
  app->timing = enable != 0;
  return HS_OK;
}

hs_status hs_get_kernel_times(hs_app* app, hs_kernel_time* entries, int max_entries,
                              int* n_entries) {
  if (!app || !n_entries) { set_error("hs_get_kernel_times: NULL"); return HS_E_INVAL; }
  if (frames_in_flight(app)) { set_error("hs_get_kernel_times: frames in flight"); return HS_E_STATE; }
  (void)hipSetDevice(app->ctx->device);
  collect_timing(app);
  int n = 0;
  for (int f = 0; f < F_COUNT; ++f) {
    if (!app->acc_n[f]) continue;
    if (entries && n < max_entries) {
      hs_kernel_time& k = entries[n];
      std::memset(&k, 0, sizeof(k));
      std::strncpy(k.name, kFamilyName[f], sizeof(k.name) - 1);
      k.launches = app->acc_n[f];
      k.total_ms = app->acc_ms[f];
      k.flops = app->acc_flops[f];
      k.bytes = app->acc_bytes[f];
    }
    ++n;
  }
  *n_entries = n;
  return HS_OK;
}

}  // extern "C"
