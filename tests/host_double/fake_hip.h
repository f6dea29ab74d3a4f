// What a test can set and read of the stand-in (fake_hip.cpp).
#pragma once
#include <atomic>

#include "hs_kernels.h"

namespace fake {
extern std::atomic<long> live_objects;     // events, streams, graphs, pinned blocks
extern std::atomic<long> live_blocks;      // operator new
extern std::atomic<long> live_threads;     // started and not ended
extern std::atomic<long> event_wait_ns;    // how long hipEventSynchronize sleeps
extern std::atomic<long> mask_queries;     // calls of sched_getaffinity
extern std::atomic<long> blocks_until_failure, threads_until_failure;   // that many succeed, one fails; -1: never
extern std::atomic<bool> fail_block_after_thread_start;   // the thread's starter fails to allocate once, right after
// the convolutions described so far with their weights in place: planned, or launched
constexpr int kMaxConvLaunches = 128;
extern hs::ConvParams conv_launches[kMaxConvLaunches];
extern std::atomic<int> n_conv_launches;
// kernels launched so far, and the streams that the first of them went to
constexpr int kMaxLaunches = 256;
extern void* launch_streams[kMaxLaunches];
extern std::atomic<int> n_launches;
// what an overlay's launch leaves in the stamps and records that it is given, in ticks of 10 ns
extern uint64_t overlay_drawn;             // from the end of stage 2 to StageStamps::drawn
extern int32_t overlay_maxima;             // to the last channel maximum
extern thread_local int device;            // the calling thread's current device
void reset_failures();
}  // namespace fake
