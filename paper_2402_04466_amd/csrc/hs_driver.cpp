// Native stream driver: feeds several applications concurrently, one submitting thread each,
// the way the paper runs one process per application instance (Section V-B), at a fixed frame
// rate with absolute deadlines or back to back.  It sits on top of the public calls only
// (hs_submit_* / hs_poll_* / hs_wait_*), so what it measures is what any caller of the library
// gets -- without an interpreter between the frames.  Also here, on the same footing: the
// per-stream front of a batched application (hs_mux).
#include <pthread.h>
#include <sched.h>
#include <sys/prctl.h>
#include <time.h>

#include <cerrno>
#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <cstring>
#include <deque>
#include <list>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "hs.h"
#include "hs_internal.h"

using hs::now_ns;

// ---- per-stream front of a batched application --------------------------------------------------
// The streams of the batch hand over their frames one by one, each with its own arrival stamp;
// the batch is submitted when its last frame arrives, and every stream collects its own result.
struct hs_mux {
  hs_app* app = nullptr;
  int batch = 0;
  std::mutex mu;
  std::condition_variable cv;
  // the batch being assembled
  std::vector<const uint8_t*> frames;
  std::vector<uint8_t*> outs;
  std::vector<uint64_t> ids, t_submit;
  std::vector<char> have;
  int n_have = 0;
  uint64_t n_batches = 0;
  // per submitted batch, in submit order: what to restore in its results
  struct Rec { std::vector<uint64_t> ids, t_submit; };
  std::deque<Rec> in_flight;
  // finished batches not yet collected by every stream, oldest first, and room for further ones: a
  // batch is delivered into room that is there already, so that filing it cannot fail
  struct Done { std::vector<hs_result> r; std::vector<char> taken; int n_taken = 0; };
  std::list<Done> done, room;
  bool draining = false;   // a thread is blocked in hs_wait_batch on behalf of all
};

// Room for one batch (mux lock held).
static std::list<hs_mux::Done> mux_room(hs_mux* m) {
  std::list<hs_mux::Done> one;
  if (m->room.empty()) {
    one.emplace_back();
    one.front().r.resize((size_t)m->batch);
    one.front().taken.resize((size_t)m->batch);
  } else {
    one.splice(one.end(), m->room, m->room.begin());
  }
  std::fill(one.front().taken.begin(), one.front().taken.end(), 0);
  one.front().n_taken = 0;
  return one;
}

// Files the batch the application has just delivered into `one` (mux lock held).
static void mux_file(hs_mux* m, std::list<hs_mux::Done>& one) {
  if (!m->in_flight.empty()) {
    const hs_mux::Rec& rec = m->in_flight.front();
    for (int j = 0; j < m->batch; ++j) {
      hs_result& r = one.front().r[(size_t)j];
      r.frame_id = rec.ids[(size_t)j];
      r.t_submit_ns = rec.t_submit[(size_t)j];   // the stream's own arrival
    }
    m->in_flight.pop_front();
  }
  m->done.splice(m->done.end(), one);
}

// Oldest finished result of `stream`, if any (mux lock held).
static bool mux_take(hs_mux* m, int stream, hs_result* out) {
  for (hs_mux::Done& d : m->done) {
    if (d.taken[(size_t)stream]) continue;
    *out = d.r[(size_t)stream];
    out->t_observed_ns = now_ns();
    d.taken[(size_t)stream] = 1;
    ++d.n_taken;
    while (!m->done.empty() && m->done.front().n_taken == m->batch)
      m->room.splice(m->room.end(), m->done, m->done.begin());
    return true;
  }
  return false;
}

extern "C" hs_status hs_create_mux(hs_app* app, int batch, hs_mux** out) {
  using hs::set_error;
  if (!app || !out || batch < 1 || batch > 16) { set_error("hs_create_mux: bad argument"); return HS_E_INVAL; }
  // the batch buffers below are handed to hs_submit_batch / hs_poll_batch, which move exactly
  // the application's batch of entries
  if (batch != hs_internal_app_batch(app)) {
    set_error("hs_create_mux: batch %d given, the application batches %d streams", batch,
              hs_internal_app_batch(app));
    return HS_E_INVAL;
  }
  if (hs_internal_app_grouped(app)) {
    set_error("hs_create_mux: the application is a member of a group");
    return HS_E_STATE;
  }
  try {
    hs_mux* m = new hs_mux();
    m->app = app;
    m->batch = batch;
    m->frames.assign((size_t)batch, nullptr);
    m->outs.assign((size_t)batch, nullptr);
    m->ids.assign((size_t)batch, 0);
    m->t_submit.assign((size_t)batch, 0);
    m->have.assign((size_t)batch, 0);
    *out = m;
    return HS_OK;
  } catch (const std::exception& e) {
    set_error("hs_create_mux: %s", e.what());
    return HS_E_NOMEM;
  }
}

extern "C" hs_status hs_destroy_mux(hs_mux* mux) {
  if (!mux) { hs::set_error("hs_destroy_mux: NULL"); return HS_E_INVAL; }
  delete mux;
  return HS_OK;
}

extern "C" hs_status hs_mux_submit(hs_mux* m, int stream, const uint8_t* d_frame,
                                   uint8_t* d_overlay_out, uint64_t frame_id) {
  using hs::set_error;
  const uint64_t t_arrival = now_ns();
  if (!m || stream < 0 || stream >= m->batch || !d_frame || !d_overlay_out) {
    set_error("hs_mux_submit: bad argument");
    return HS_E_INVAL;
  }
  try {
    std::lock_guard<std::mutex> lk(m->mu);
    const size_t j = (size_t)stream;
    if (m->have[j]) {
      set_error("hs_mux_submit: stream %d already has a frame waiting for its batch", stream);
      return HS_E_QUEUE_FULL;
    }
    m->frames[j] = d_frame; m->outs[j] = d_overlay_out; m->ids[j] = frame_id;
    m->t_submit[j] = t_arrival;
    if (m->n_have + 1 < m->batch) {
      m->have[j] = 1;
      ++m->n_have;
      return HS_OK;
    }
    // the last frame of the batch: hand the batch to the application.  It is noted first: once it has
    // been handed over nothing may fail
    m->in_flight.push_back(hs_mux::Rec{m->ids, m->t_submit});
    const hs_status st = hs_submit_batch(m->app, m->frames.data(), m->outs.data(), m->n_batches);
    if (st != HS_OK) {   // this frame was not taken; the others keep waiting
      m->in_flight.pop_back();
      return st;
    }
    ++m->n_batches;
    std::fill(m->have.begin(), m->have.end(), 0);
    m->n_have = 0;
    return HS_OK;
  } catch (const std::exception& e) {
    set_error("hs_mux_submit: %s", e.what());
    return HS_E_NOMEM;
  }
}

extern "C" hs_status hs_mux_poll(hs_mux* m, int stream, hs_result* out) {
  using hs::set_error;
  if (!m || !out || stream < 0 || stream >= m->batch) { set_error("hs_mux_poll: bad argument"); return HS_E_INVAL; }
  try {
    std::lock_guard<std::mutex> lk(m->mu);
    for (;;) {
      if (mux_take(m, stream, out)) return HS_OK;
      if (m->draining) break;   // another thread is fetching: it will file what it gets
      auto one = mux_room(m);
      const hs_status st = hs_poll_batch(m->app, one.front().r.data());
      if (st == HS_OK) { mux_file(m, one); continue; }
      m->room.splice(m->room.end(), one);
      if (st == HS_E_NOT_READY) break;
      return st;
    }
    set_error("hs_mux_poll: no finished frame for stream %d", stream);
    return HS_E_NOT_READY;
  } catch (const std::exception& e) {
    set_error("hs_mux_poll: %s", e.what());
    return HS_E_NOMEM;
  }
}

extern "C" hs_status hs_mux_wait(hs_mux* m, int stream, hs_result* out, uint64_t timeout_ns) {
  using hs::set_error;
  if (!m || !out || stream < 0 || stream >= m->batch) { set_error("hs_mux_wait: bad argument"); return HS_E_INVAL; }
  try {
    const uint64_t deadline = hs::deadline_after(timeout_ns);
    std::unique_lock<std::mutex> lk(m->mu);
    for (;;) {
      if (mux_take(m, stream, out)) return HS_OK;
      const int64_t left = (int64_t)deadline - (int64_t)now_ns();
      if (left <= 0) { set_error("hs_mux_wait: timed out"); return HS_E_NOT_READY; }
      if (m->draining) {   // another thread is fetching the next batch for everybody
        m->cv.wait_for(lk, std::chrono::nanoseconds(std::min<int64_t>(left, 20000000)));
        continue;
      }
      // fetch the next finished batch on behalf of every stream; one thread at a time talks to
      // the application, so batches are filed in the order they are delivered
      auto one = mux_room(m);
      hs_status st = hs_poll_batch(m->app, one.front().r.data());
      if (st == HS_E_NOT_READY) {
        m->draining = true;
        lk.unlock();
        st = hs_wait_batch(m->app, one.front().r.data(), (uint64_t)std::min<int64_t>(left, 20000000));
        lk.lock();
        m->draining = false;
        m->cv.notify_all();
      }
      if (st == HS_OK) mux_file(m, one);
      else m->room.splice(m->room.end(), one);
      if (st != HS_OK && st != HS_E_NOT_READY) return st;
    }
  } catch (const std::exception& e) {
    set_error("hs_mux_wait: %s", e.what());
    return HS_E_NOMEM;
  }
}

namespace {

struct Worker {
  const hs_feed* feed = nullptr;
  int per_frame = 1;              // results per frame (batch streams or group members)
  hs_result* results = nullptr;   // [n_frames][per_frame]
  int64_t* lateness = nullptr;    // [n_frames] or NULL
  int n_frames = 0;
  uint64_t t0 = 0, period = 0;    // period 0: back to back
  int dropped = 0;
  hs_status status = HS_OK;
  hs::Message error;
};

hs_status feed_submit(const hs_feed* f, int k) {
  const uint8_t* const* fr = f->d_frames + (size_t)(k % f->n_frames) * f->batch;
  uint8_t* const* ou = f->d_outs + (size_t)(k % f->n_outs) * f->batch;
  if (f->mux) return hs_mux_submit(f->mux, f->mux_stream, fr[0], ou[0], (uint64_t)k);
  if (f->group) return hs_submit_group(f->group, fr[0], ou[0], (uint64_t)k);
  return hs_submit_batch(f->app, fr, ou, (uint64_t)k);
}

hs_status feed_poll(const hs_feed* f, hs_result* out) {
  if (f->mux) return hs_mux_poll(f->mux, f->mux_stream, out);
  return f->group ? hs_poll_group(f->group, out) : hs_poll_batch(f->app, out);
}

hs_status feed_wait(const hs_feed* f, hs_result* out) {
  const uint64_t ten_s = 10000000000ull;
  if (f->mux) return hs_mux_wait(f->mux, f->mux_stream, out, ten_s);
  return f->group ? hs_wait_group(f->group, out, ten_s) : hs_wait_batch(f->app, out, ten_s);
}

void worker_main(Worker* w) {
  const hs_feed* f = w->feed;
  if (f->cpu >= 0) {   // paper Section IV-C: the application's thread on a core of its own
    cpu_set_t set;
    CPU_ZERO(&set);
    CPU_SET(f->cpu, &set);
    (void)pthread_setaffinity_np(pthread_self(), sizeof(set), &set);
  }
  if (w->period) (void)prctl(PR_SET_TIMERSLACK, 1000UL);   // wake within 1 us of a deadline, not 50
  int got = 0;   // frames whose results have been collected, in order
  auto fail = [&](hs_status st) {
    w->status = st;
    w->error.set(hs_last_error());
  };
  auto slot = [&](int i) { return w->results + (size_t)i * w->per_frame; };
  for (int k = 0; k < w->n_frames; ++k) {
    for (;;) {   // collect whatever has finished
      const hs_status st = feed_poll(f, slot(got));
      if (st == HS_E_NOT_READY) break;
      if (st != HS_OK) return fail(st);
      ++got;
    }
    if (w->period) {
      const uint64_t deadline = w->t0 + (uint64_t)k * w->period;
      timespec ts;
      ts.tv_sec = (time_t)(deadline / 1000000000ull);
      ts.tv_nsec = (long)(deadline % 1000000000ull);
      while (clock_nanosleep(CLOCK_MONOTONIC, TIMER_ABSTIME, &ts, nullptr) == EINTR) {}
      if (w->lateness) w->lateness[k] = (int64_t)(now_ns() - deadline);
    }
    for (;;) {
      const hs_status st = feed_submit(f, k);
      if (st == HS_OK) break;
      if (st != HS_E_QUEUE_FULL) return fail(st);
      if (w->period) {   // a paced source does not wait: the frame is lost
        ++w->dropped;
        break;
      }
      const hs_status sw = feed_wait(f, slot(got));   // back to back: make room, try again
      if (sw != HS_OK) return fail(sw);
      ++got;
    }
  }
  while (got + w->dropped < w->n_frames) {
    const hs_status st = feed_wait(f, slot(got));
    if (st != HS_OK) return fail(st);
    ++got;
  }
}

}  // namespace

extern "C" hs_status hs_run_feeds(const hs_feed* feeds, int n_feeds, double fps, int n_frames,
                                  hs_result* const* results, int* dropped,
                                  int64_t* const* lateness_ns, double* elapsed_s) {
  using hs::set_error;
  if (!feeds || !results || n_feeds < 1 || n_frames < 1 || !(fps >= 0.0)) {
    set_error("hs_run_feeds: bad argument");
    return HS_E_INVAL;
  }
  for (int i = 0; i < n_feeds; ++i) {
    const hs_feed& f = feeds[i];
    if ((!f.app && !f.group && !f.mux) || ((f.group || f.mux) && f.batch != 1) || !f.d_frames || !f.d_outs || f.n_frames < 1 || f.n_outs < 1 ||
        f.batch < 1 || f.results_per_frame < 1 || !results[i]) {
      set_error("hs_run_feeds: feed %d is incomplete", i);
      return HS_E_INVAL;
    }
  }
  try {
    std::vector<Worker> workers((size_t)n_feeds);
    std::vector<std::thread> threads;
    const uint64_t t0 = now_ns() + 20000000ull;   // first deadline 20 ms from now
    for (int i = 0; i < n_feeds; ++i) {
      Worker& w = workers[(size_t)i];
      w.feed = &feeds[i];
      w.per_frame = feeds[i].results_per_frame;
      w.results = results[i];
      w.lateness = lateness_ns ? lateness_ns[i] : nullptr;
      w.n_frames = n_frames;
      w.t0 = t0;
      w.period = fps > 0.0 ? (uint64_t)(1e9 / fps) : 0;
    }
    const uint64_t t_begin = now_ns();
    // A single feed runs on the caller's thread, which would only wait, unless the feed sets its thread's core or timer: a thread
    // started and joined costs 40 to 60 us (sixteen annotated 322 x 241 frames 434 -> 392 us, twelve 1920 x 1080 1047 -> 998, four batches of twelve 2065 -> 2000).
    const bool here = n_feeds == 1 && fps == 0.0 && feeds[0].cpu < 0;
    const size_t n_threads = here ? 0 : (size_t)n_feeds;
    threads.reserve(n_threads);
    hs::Message not_started;     // a source whose thread cannot be had; those that run are seen to their end
    try {
      for (size_t i = 0; i < n_threads; ++i) threads.emplace_back(worker_main, &workers[i]);
    } catch (const std::exception& e) {
      not_started.set(e.what());
    }
    if (here) {                  // and leaves no trace there: current device, last failure
      const int device = hs_internal_current_device();
      hs::Message last;
      last.set(hs_last_error());
      worker_main(&workers[0]);
      hs_internal_use_device(device);
      set_error("%s", last.text);
    }
    for (std::thread& t : threads) t.join();
    if (threads.size() < n_threads) {
      set_error("hs_run_feeds: no thread for feed %zu: %s", threads.size(), not_started.text);
      return HS_E_NOMEM;
    }
    if (elapsed_s) *elapsed_s = (double)(now_ns() - t_begin) * 1e-9;
    hs_status st = HS_OK;
    for (int i = 0; i < n_feeds; ++i) {
      if (dropped) dropped[i] = workers[(size_t)i].dropped;
      if (st == HS_OK && workers[(size_t)i].status != HS_OK) {
        st = workers[(size_t)i].status;
        set_error("hs_run_feeds: feed %d: %s", i, workers[(size_t)i].error.text);
      }
    }
    return st;
  } catch (const std::exception& e) {
    set_error("hs_run_feeds: %s", e.what());
    return HS_E_NOMEM;
  }
}
