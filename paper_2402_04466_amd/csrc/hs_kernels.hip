// HIP kernels (gfx950 / CDNA4 only) of the per-frame tool-tracking hot path:
// paper Section III-A stages format conversion -> inference -> postprocess -> overlay.
#include "hs_kernels.h"

#include <algorithm>
#include <mutex>

namespace hs {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // plain 16-byte register value
typedef uint32_t u32x3 __attribute__((ext_vector_type(3), aligned(4)));   // 12 bytes in memory, at any word

// floor(num / d) for num, d < 2^31 where the quotient is < 2^22: float estimate, exact fix-up.
__device__ __forceinline__ uint32_t udiv_est(uint32_t num, uint32_t d, float rcp_d) {
  uint32_t q = (uint32_t)((float)num * rcp_d);
  int32_t r = (int32_t)(num - q * d);
  if (r < 0) { q -= 1; r += (int32_t)d; }
  if (r >= (int32_t)d) { q += 1; }
  return q;
}

// A buffer of `bytes` bytes (below 2^31) for loads with a scalar and a per-lane offset: no address arithmetic per
// load, and a lane whose offset lies behind the buffer reads zeros (kOutside: always).
typedef __amdgpu_buffer_rsrc_t BufferRsrc;
constexpr int kOutside = (int)0x80000000u;
// (Both arguments are the same for the whole wavefront; unless told so the compiler may keep the descriptor in vector
// registers, and then every load is a loop over the lanes' values.)
__device__ __forceinline__ BufferRsrc buffer_of(const void* base, uint32_t bytes) {
  const uint64_t b = (uint64_t)base;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00027000);
}
__device__ __forceinline__ u32x4 load16(BufferRsrc buf, int lane_offset, int offset) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, lane_offset, offset, 0));
}

// =============================================================================================
// Stage 1: one workgroup per output row.  The two source rows the row needs are staged in
// LDS with 16-byte loads; every output pixel is the exact integer 4-tap sum, rounded once.
// =============================================================================================
// a * b (+ c) on the low 24 bits of a and b, low 32 bits of the result: the full-rate integer
// multiplier (the 32 x 32-bit one runs at a quarter of its rate).  Written as instructions
// because the compiler turns __umul24 back into a 32-bit multiply when it knows one factor
// to be small.
__device__ __forceinline__ uint32_t mul24(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t mad24(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Block size: 256..512 threads, chosen by the host so that a source row is at most kResizeVecs 16-byte vectors per
// thread.  A launch of one round of workgroups takes the size whose passes over the output row are as full as possible
// (two 854 x 480 frames of 3840 x 2160: two passes of 448 threads 6.9 us, four of 256 7.4).  A longer one takes the smallest:
// what counts there is how many rows a CU has under way while each waits for its source (sixteen 416 x 240 frames: 256
// threads 8.5 us, 448 10.1; eight 5.4, 6.6; six 854 x 480 11.5, 12.3; twelve of 192 and 128 threads 27 to 29).  Over 24
// launches of 128 to 5760 rows that is the fastest of 256 to 512 threads or within 5 % of it.  The row loads are the first
// thing a workgroup issues: the lookup tables and the row arithmetic are set up behind them.
constexpr int kResizeVecs = 4;
// The bilinear sum of the two source pixels that start in bytes 0 .. 5 of a (upper row) and c (lower row), rounded, per channel.
__device__ __forceinline__ void resize_sum(const ResizeParams& p, uint32_t d, const uint32_t (&a)[2], const uint32_t (&c)[2], uint32_t wx0,
                                           uint32_t wx1, uint32_t wy0, uint32_t wy1, uint32_t (&q)[3]) {
  const uint64_t r0 = (uint64_t)a[1] << 32 | a[0], r1 = (uint64_t)c[1] << 32 | c[0];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint32_t p00 = (uint32_t)(r0 >> (8 * i)) & 0xffu, p01 = (uint32_t)(r0 >> (8 * i + 24)) & 0xffu;
    const uint32_t p10 = (uint32_t)(r1 >> (8 * i)) & 0xffu, p11 = (uint32_t)(r1 >> (8 * i + 24)) & 0xffu;
    // every factor is below 2^24 (weights <= 2*wo, 2*ho <= 2^15; a row sum <= 2*wo*255 < 2^24) and
    // the sum below 2^31: 24-bit multiplies are exact here and run at four times the rate of
    // the 32-bit ones
    const uint32_t acc = mad24(wy0, mad24(wx0, p00, mul24(wx1, p01)),
                               mul24(wy1, mad24(wx0, p10, mul24(wx1, p11))));
    // floor((acc + d/2) / d) by multiplication: exact for numerators below 2^31
    q[i] = __umulhi(acc + (d >> 1), p.d_magic) >> p.d_shift;
  }
}
// First of the two source columns (rows) of output column (row) i of `out`, and the second one's weight out of 2 * out.
__device__ __forceinline__ uint32_t resize_source(int i, int in, int out, float rcp, uint32_t& weight) {
  const uint32_t span = 2u * (uint32_t)out;
  const int n = max(0, min((2 * i + 1) * in - out, (in - 1) * (int)span));
  const uint32_t first = udiv_est((uint32_t)n, span, rcp);
  weight = (uint32_t)n - first * span;
  return first;
}
template <int NV>   // 16-byte vectors per thread and source row: 1, 2 or 4
__global__ __launch_bounds__(512) void k_resize_norm(ResizeParams p) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ float s_lut32[256];
  __shared__ f16 s_lut16[256];
  const int tid = threadIdx.x, T = blockDim.x;
  const int Y = blockIdx.x;
  const uint8_t* const src = p.src[blockIdx.y];          // stream blockIdx.y of the batch
  f16* const dst = p.dst + blockIdx.y * p.dst_img_stride;
  float* const dst_f32 = p.dst_f32 ? p.dst_f32 + blockIdx.y * p.dst32_img_stride : nullptr;
  const uint32_t dy = 2u * (uint32_t)p.ho, dx = 2u * (uint32_t)p.wo;
  uint32_t fy;
  const uint32_t y0 = resize_source(Y, p.hi, p.ho, p.rcp_dy, fy);
  const uint32_t y1 = min(y0 + 1u, (uint32_t)(p.hi - 1));

  // the two source rows: 16-byte loads into named registers (as arrays they end up in scratch
  // memory), addresses clamped to the row so that every load is unconditional
  const int row_vecs = (3 * p.wi + 15) >> 4;          // 16-byte vectors per source row
  const uint4* const row0 = reinterpret_cast<const uint4*>(src + (size_t)y0 * p.src_pitch);
  const uint4* const row1 = reinterpret_cast<const uint4*>(src + (size_t)y1 * p.src_pitch);
  uint4 st0_0, st0_1, st0_2, st0_3, st1_0, st1_1, st1_2, st1_3;
#define HS_FETCH_VEC(I_)                                                                       \
  if constexpr (NV > I_) {                                                                     \
    const int v_ = min(tid + I_ * T, row_vecs - 1);                                            \
    st0_##I_ = row0[v_];                                                                       \
    st1_##I_ = row1[v_];                                                                       \
  }
#define HS_HAND_VEC(I_)                                                                        \
  if constexpr (NV > I_) {                                                                     \
    if (tid + I_ * T < row_vecs) {                                                             \
      l0[tid + I_ * T] = st0_##I_;                                                             \
      l1[tid + I_ * T] = st1_##I_;                                                             \
    }                                                                                          \
  }
  HS_FETCH_VEC(0) HS_FETCH_VEC(1) HS_FETCH_VEC(2) HS_FETCH_VEC(3)
  if (tid < 256) {
    s_lut32[tid] = p.lut32[tid];
    s_lut16[tid] = p.lut16[tid];
  }
  uint4* const l0 = reinterpret_cast<uint4*>(lds);
  uint4* const l1 = l0 + row_vecs;
  const uint32_t* const p0 = reinterpret_cast<const uint32_t*>(lds);
  const uint32_t* const p1 = reinterpret_cast<const uint32_t*>(lds + (size_t)row_vecs * 16);
  const uint32_t d = dx * dy;

  HS_HAND_VEC(0) HS_HAND_VEC(1) HS_HAND_VEC(2) HS_HAND_VEC(3)
  __syncthreads();
  const uint32_t wy1 = fy, wy0 = dy - fy;
  for (int X = tid; X < p.wo; X += T) {
    uint32_t fx;
    const uint32_t x0 = resize_source(X, p.wi, p.wo, p.rcp_dx, fx);
    const uint32_t wx1 = fx, wx0 = dx - fx;
    // The two source pixels x0, x0+1 are 6 consecutive bytes inside three aligned words: fetch
    // the words from each row and funnel-shift the bytes into place (v_alignbyte).  At the
    // right edge x0 + 1 is past the row, its weight fx is 0 there and the bytes read are the
    // next row or the padding behind the rows.
    const uint32_t b0 = 3u * x0, wi0 = b0 >> 2, sh = b0 & 3u;
    const uint32_t a[2] = {__builtin_amdgcn_alignbyte(p0[wi0 + 1], p0[wi0], sh),        // bytes 0..3
                           __builtin_amdgcn_alignbyte(p0[wi0 + 2], p0[wi0 + 1], sh)};   // bytes 4..7
    const uint32_t c[2] = {__builtin_amdgcn_alignbyte(p1[wi0 + 1], p1[wi0], sh),
                           __builtin_amdgcn_alignbyte(p1[wi0 + 2], p1[wi0 + 1], sh)};
    uint32_t q[3];
    resize_sum(p, d, a, c, wx0, wx1, wy0, wy1, q);
    half4 px;
    px[0] = s_lut16[q[0]];
    px[1] = s_lut16[q[1]];
    px[2] = s_lut16[q[2]];
    px[3] = (f16)0.0f;
    *reinterpret_cast<half4*>(dst + ((size_t)(Y + p.pad_t) * p.dst_w + (X + p.pad_l)) * 4) = px;
    if (dst_f32) {
      const size_t plane = (size_t)p.ho * p.wo;
      float* o = dst_f32 + (size_t)Y * p.wo + X;
      o[0] = s_lut32[q[0]];
      o[plane] = s_lut32[q[1]];
      o[2 * plane] = s_lut32[q[2]];
    }
  }
#undef HS_HAND_VEC
#undef HS_FETCH_VEC
  if (tid == 0 && blockIdx.x == gridDim.x - 1 && blockIdx.y == gridDim.y - 1) *p.t_end = wall_clock64();
}

static unsigned resize_block(const ResizeParams& p) {
  const unsigned row_vecs = (unsigned)((3 * p.wi + 15) >> 4);
  const unsigned t_min = std::max(256u, (row_vecs + kResizeVecs - 1) / kResizeVecs);
  const bool one_round = (unsigned)p.ho * (unsigned)p.batch <= 4 * 256;   // four workgroups of 448 threads on every CU
  unsigned best = 0;
  for (unsigned t = 256; t <= 512; t += 64) {
    if (t < t_min) continue;
    if (!one_round) return t;
    if (!best || (p.wo + t - 1) / t * t < (p.wo + best - 1) / best * best) best = t;
  }
  return best ? best : 512;
}

KernelDesc describe(const ResizeParams& p) {
  const unsigned lds = (unsigned)((3 * p.wi + 15) >> 4) * 16 * 2 + 16;   // + padding read at the edge
  const unsigned t = resize_block(p);
  const unsigned nv = ((unsigned)((3 * p.wi + 15) >> 4) + t - 1) / t;
  const void* f = nv <= 1   ? (const void*)k_resize_norm<1>
                  : nv == 2 ? (const void*)k_resize_norm<2>
                            : (const void*)k_resize_norm<kResizeVecs>;
  return KernelDesc{f, dim3(p.ho, p.batch), dim3(t), lds};
}

// =============================================================================================
// Stage 2: implicit-GEMM convolution on v_mfma_f32_32x32x16_f16.  The MFMA "A" operand is the weight
// tile and the "B" operand the pixel tile, so a lane ends up holding 4 consecutive output channels
// of one pixel per accumulator quad of the pixel-major output.
// =============================================================================================
__device__ __forceinline__ float sigmoid_f(float x) { return 1.0f / (1.0f + __expf(-x)); }
// stage 3's heat value of a logit
__device__ __forceinline__ float heat_of(float x) { return 1.0f / (1.0f + expf(-x)); }

// Pairs q[i] = fp16 channels cbase + 8i + 4h .. +3 of the lane's pixel: the exchange and the store.
__device__ __forceinline__ void store_quads_to(f16* out, int pitch, bool valid, int m, int cbase, int h,
                                               uint32_t (&q)[4][2]) {
#pragma unroll
  for (int pr = 0; pr < 2; ++pr)
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const auto sw = __builtin_amdgcn_permlane32_swap(q[2 * pr][w], q[2 * pr + 1][w], false, false);
      q[2 * pr][w] = sw[0];
      q[2 * pr + 1][w] = sw[1];
    }
  if (valid) {
    f16* dst = out + (size_t)m * pitch + cbase + h * 8;
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
      const u32x4 o = {q[2 * pr][0], q[2 * pr][1], q[2 * pr + 1][0], q[2 * pr + 1][1]};
      *reinterpret_cast<u32x4*>(dst + 16 * pr) = o;
    }
  }
}

// Epilogue of the 32 channels of one pixel that a lane pair (r, r + 32) holds as accumulator
// quads: lane half h has channels cbase + 4h + 8i .. +3 in acc[4i .. 4i+3], i = 0..3.  Residual,
// ReLU and rounding to fp16; then the two lanes swap one quad of every pair
// (v_permlane32_swap: lanes 32..63 of the first operand <-> lanes 0..31 of the second), so that
// each holds 8 consecutive channels per pair and stores 16 bytes at a time instead of 8.
// For fp16 outputs whose channel count is a multiple of 32.  Every lane of the wavefront must
// call it (the swap needs both lanes of a pair); `valid` gates the store.  out / pitch / relu:
// the destination tensor (the layer's output, or the projection's).
__device__ __forceinline__ void store_octets_to(f16* out, int pitch, bool relu, bool valid, int m,
                                                int cbase, int h, const floatx16& acc,
                                                const half4 (&res)[4], bool has_res) {
  uint32_t q[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float v[4] = {acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]};
    if (has_res) {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] += (float)res[i][j];
    }
    half4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (f16)v[j];
    if (relu) o = __builtin_elementwise_max(o, half4{});   // ReLU and rounding commute: two values at once
    const uint2 w = __builtin_bit_cast(uint2, o);
    q[i][0] = w.x;
    q[i][1] = w.y;
  }
  store_quads_to(out, pitch, valid, m, cbase, h, q);
}
__device__ __forceinline__ void store_octets(const ConvParams& p, bool valid, int m, int cbase,
                                             int h, const floatx16& acc, const half4 (&res)[4],
                                             bool has_res) {
  store_octets_to(p.out, p.out_pitch, p.relu != 0, valid, m, cbase, h, acc, res, has_res);
}
// The residual of a pixel's 32 channels, fetched the way store_octets stores them: lane half h
// loads channels cbase + 8h .. +7 and cbase + 16 + 8h .. +7 (two 16-byte loads, o[0] and o[1],
// from pixel_base + cbase + 8 * h and 16 halves further); the same lane exchange (it is its own
// inverse) turns them into the quads res[i] = channels cbase + 4h + 8i .. +3 that the
// accumulators are laid out in.  Every lane of the wavefront must call it.
__device__ __forceinline__ void res_octets_to_quads(const u32x4 (&o)[2], half4 (&res)[4]) {
  uint32_t q[4][2] = {{o[0][0], o[0][1]}, {o[0][2], o[0][3]}, {o[1][0], o[1][1]}, {o[1][2], o[1][3]}};
#pragma unroll
  for (int pr = 0; pr < 2; ++pr)
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const auto sw = __builtin_amdgcn_permlane32_swap(q[2 * pr][w], q[2 * pr + 1][w], false, false);
      q[2 * pr][w] = sw[0];
      q[2 * pr + 1][w] = sw[1];
    }
#pragma unroll
  for (int i = 0; i < 4; ++i) res[i] = __builtin_bit_cast(half4, make_uint2(q[i][0], q[i][1]));
}

// The same for one half of them, 16 channels from cbase on: v0 = channels cbase + 4h .. + 3, v1 = 8 further;
// res: the lane's 16 bytes of the residual (channels cbase + 8h .. + 7).  m < 0: nothing is stored.
__device__ __forceinline__ void store_half(f16* out, int pitch, bool relu, int m, int cbase, int h, const float4& v0,
                                           const float4& v1, const u32x4& res, bool has_res) {
  float v[2][4] = {{v0.x, v0.y, v0.z, v0.w}, {v1.x, v1.y, v1.z, v1.w}};
  if (has_res) {
    const auto s0 = __builtin_amdgcn_permlane32_swap(res[0], res[2], false, false);
    const auto s1 = __builtin_amdgcn_permlane32_swap(res[1], res[3], false, false);
    const half4 r0 = __builtin_bit_cast(half4, make_uint2(s0[0], s1[0]));
    const half4 r1 = __builtin_bit_cast(half4, make_uint2(s0[1], s1[1]));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[0][j] += (float)r0[j];
      v[1][j] += (float)r1[j];
    }
  }
  uint2 w[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    half4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (f16)v[i][j];
    if (relu) o = __builtin_elementwise_max(o, half4{});
    w[i] = __builtin_bit_cast(uint2, o);
  }
  const auto s0 = __builtin_amdgcn_permlane32_swap(w[0].x, w[1].x, false, false);
  const auto s1 = __builtin_amdgcn_permlane32_swap(w[0].y, w[1].y, false, false);
  if (m >= 0) {
    const u32x4 o = {s0[0], s1[0], s0[1], s1[1]};
    *reinterpret_cast<u32x4*>(out + (size_t)m * pitch + cbase + 8 * h) = o;
  }
}
// And for one quad, channels cbase + 4h .. + 3; res: the lane's 8 bytes of the residual.
__device__ __forceinline__ void store_quad(const RunParams& p, int m, int cbase, int h, const float4& v0, const u32x4& res) {
  float v[4] = {v0.x, v0.y, v0.z, v0.w};
  const half4 rq = __builtin_bit_cast(half4, make_uint2(res[0], res[1]));
  half4 o;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (p.res) v[j] += (float)rq[j];
    o[j] = (f16)v[j];
  }
  if (p.relu) o = __builtin_elementwise_max(o, half4{});
  if (m >= 0) *reinterpret_cast<half4*>(p.out + (size_t)m * p.out_pitch + cbase + 4 * h) = o;
}

// The small network's last layer: logits of pixel ml of an image, eight channels, planar per image, and stage 3's per-cell
// outputs (see PostParams).  Lane half h holds four of a pixel's channels; every lane of the wavefront must call it.
template <class P>   // ConvParams or TinyFrameParams
__device__ __forceinline__ void store_logits(const P& p, bool valid, int img, int ml, int h, const floatx16& acc) {
  uint32_t set_channels = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float x = acc[j];
    const bool set = x > p.theta;
    set_channels |= set ? 1u << (4 * h + j) : 0u;
    if (valid) {
      const size_t at = ((size_t)img * 8 + 4 * h + j) * p.img_m + ml;
      p.out_f32[at] = x;
      p.heat[at] = heat_of(x);
      p.mask[at] = set ? 1 : 0;
    }
  }
  set_channels |= (uint32_t)__shfl_xor((int)set_channels, 32, 64);
  const int m = img * p.img_m + ml;
  if (valid && h == 0) p.kmap[m] = set_channels ? (uint8_t)__builtin_ctz(set_channels) : 0xff;
  if (valid && m == p.m - 1 && h == 0) *p.t_end = wall_clock64();
}

// =============================================================================================
// The small network's layers: at most 32 output channels, 16 or 32 input channels (or four
// 4-channel pixels of the first layer) per tap, at most nine taps.  A layer is one launch and one
// memory round trip: a wavefront owns 32 consecutive pixels x 32 channels of one K split, gathers
// every tap's pixel vectors and weight fragments (wt_frag) straight from memory, all before its
// first MFMA, and the two wavefronts of a split pair meet in LDS.  (Tiles of 64 pixels x 64 channels
// staged through LDS computed two to eight times the channels there are, and split K over workgroups
// whose sums a further launch added: 128 x 128 input, 38 us of launches per frame -> 25.)
// Per output: chunks in order within a split, then the splits in order.
// The layer that computes the logits also finishes stage 3's per-cell outputs (see PostParams).
// KSTEPS: MFMA K-steps of 16 per chunk.  NS: K splits, 1 or 2.
// =============================================================================================
template <int KSTEPS, int NS>
__global__ __launch_bounds__(256) void k_conv_direct(ConvParams p) {
  constexpr int MAXC = NS == 2 ? 5 : 9;                // chunks of a split
  constexpr int TILES = 4 / NS;                        // pixel tiles per workgroup
  __shared__ float4 s_part[NS == 2 ? TILES : 1][4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31, h = lane >> 5;
  const int split = wave % NS, pt = wave / NS;
  const int tile = (int)(blockIdx.x & 7u) * p.tiles_per_xcd + (int)(blockIdx.x >> 3);
  const int m = (tile * TILES + pt) * 32 + r;
  const bool valid = m < p.m;
  const int mc = min(m, p.m - 1), img = mc / p.img_m, ml = mc - img * p.img_m;
  const int oy = ml / p.wout, ox = ml - oy * p.wout;
  const int iy0 = oy * p.stride - p.pad, ix0 = ox * p.stride - p.pad;
  const int q0 = split * p.chunks_per_split, q1 = min(p.nchunks, q0 + p.chunks_per_split);
  const f16* const base = p.in + (((long)img * p.hin + iy0) * p.win + ix0) * p.cin_pitch + h * 8;
  const u32x4* const wf = reinterpret_cast<const u32x4*>(p.wt_frag) + lane;

  u32x4 xb[MAXC][KSTEPS], wa[MAXC][KSTEPS];
#pragma unroll
  for (int c = 0; c < MAXC; ++c) {
    const int q = min(q0 + c, q1 - 1), ky = q / p.kw, kx = q - ky * p.kw;
    const int iy = iy0 + ky, ix = ix0 + kx;
    const bool inb = iy >= 0 && iy < p.hin && ix >= 0 && ix < p.win;
    const f16* src = inb ? base + ((long)ky * p.win + kx) * p.cin_pitch : p.in;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      wa[c][ks] = wf[(q * KSTEPS + ks) * 64];
      const u32x4 v = *reinterpret_cast<const u32x4*>(src + ks * 16);
      const u32x4 zero = {0u, 0u, 0u, 0u};
      xb[c][ks] = inb ? v : zero;
    }
  }
  floatx16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll
  for (int c = 0; c < MAXC; ++c)
    if (c < q1 - q0) {
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, wa[c][ks]),
                                                    __builtin_bit_cast(half8, xb[c][ks]), acc, 0, 0, 0);
    }
  if (NS == 2) {
    if (split == 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        s_part[pt][i][lane] = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
    }
    __syncthreads();
    if (split == 1) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 b = s_part[pt][i][lane];
      const float v[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[4 * i + j] = (0.0f + acc[4 * i + j]) + v[j];
    }
  }
  // accumulator quad i: channels 8 * i + 4 * h .. + 3 of pixel m
  if (p.out_f32 == nullptr) {
    if (!valid) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int n = 8 * i + 4 * h;
      if (n >= p.cout) continue;
      half4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = (f16)(p.relu ? fmaxf(acc[4 * i + j], 0.0f) : acc[4 * i + j]);
      *reinterpret_cast<half4*>(p.out + (size_t)m * p.out_pitch + n) = o;
    }
    return;
  }
  store_logits(p, valid, img, ml, h, acc);
}

// =============================================================================================
// The whole small network in one launch: a workgroup takes 8 x 8 logits through all four layers.  The layers' halos
// (10 x 10, 12 x 12 and 25 x 25 pixels of the layers before) are computed again by the neighbouring workgroups -- up to
// 2.4 times the products, of which there are few -- and the intermediate tensors stay in LDS: as launches of their own
// the layers take 3.7 to 5.9 us each for one 128 x 128 input, almost all of it launch, memory round trip and set-up.
// Eight wavefronts of 32 pixels x 32 channels (20 such groups in the first layer, then 5, 4 and 2).  The first layer's
// pixels come straight from the 4-channel image (see k_conv_direct), all layers' weights straight from memory, asked for
// before the first product by the wavefronts that need them.  LDS pixels are padded to 48 and 80 bytes against bank
// conflicts.  Sums as in k_conv_direct with two K splits (first layer: one).
// p.wt_frag: the four layers' weights in k_conv_direct's order, one after the other.
//
// FRAME: stage 1 is part of the launch.  The workgroup computes the 51 x 52 pixels of the network's input under its tile from
// the frame (2.6 times as many as there are, with k_resize_norm's arithmetic), keeps them in LDS and stores its own 32 x 32.
// What it saves is a launch, which is what bounds the host back to back, and a trip of the image through memory: sixteen annotated
// 322 x 241 frames to 96 x 72 381 -> 316 us, one 320 x 240 frame to 128 x 128 29.3 -> 28.6.
// =============================================================================================
template <bool FRAME> struct TinyNetArgs { typedef ConvParams type; };
template <> struct TinyNetArgs<true> { typedef TinyFrameParams type; };
template <bool FRAME>
__global__ __launch_bounds__(512, 2) void k_tiny_net(typename TinyNetArgs<FRAME>::type p) {
  constexpr int N1 = 25, N2 = 12, N3 = 10, N4 = 8;                 // pixels per side of the layers' tiles
  constexpr int P1 = 24, P2 = 40;                                  // halves per LDS pixel of 16 and 32 channels
  constexpr int W2 = 3 * 1024, W3 = W2 + 9 * 1024, W4 = W3 + 18 * 1024, W_BYTES = W4 + 18 * 1024;
  constexpr int H0 = 2 * N1 + 1, W0 = 2 * N1 + 2, NP = (H0 * W0 + 511) / 512;   // FRAME: rows and pixels per row of the input, per thread
  __shared__ __align__(16) f16 s1[N1 * N1 * P1], s2[N2 * N2 * P2], s3[N3 * N3 * P2], s0[FRAME ? H0 * W0 * 4 : 8];

  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int x0 = N4 * (int)blockIdx.x, y0 = N4 * (int)blockIdx.y, img = (int)blockIdx.z;
  const BufferRsrc w_buf = buffer_of(p.wt_frag, W_BYTES);
  const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // ---- operands: first layer's pixels (groups wave, wave + 8, wave + 16), then the weights
  u32x4 xb[3][3], w1[3], w2[9], w34[18];
  u32x3 upper[NP], lower[NP];
  f16 lut16 = (f16)0.0f;
  float lut32 = 0.0f;
  if constexpr (FRAME) {
    lut16 = p.r.lut16[threadIdx.x & 255];
    lut32 = p.r.lut32[threadIdx.x & 255];
    // (rows are read in whole 16-byte vectors, no further: what lies behind the last one reads as zeros)
    const BufferRsrc frame = buffer_of(p.r.src[img], (uint32_t)p.r.src_pitch * (uint32_t)(p.r.hi - 1) + (uint32_t)(3 * p.r.wi + 15) / 16 * 16);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int q = min((int)threadIdx.x + 512 * i, H0 * W0 - 1), Y = 4 * y0 - 11 + q / W0, X = 4 * x0 - 11 + q % W0;
      uint32_t fx, fy;
      const uint32_t sx = resize_source(X, p.r.wi, p.r.wo, p.r.rcp_dx, fx), sy = resize_source(Y, p.r.hi, p.r.ho, p.r.rcp_dy, fy);
      const uint32_t at = sy * (uint32_t)p.r.src_pitch + (3 * sx & ~3u);
      upper[i] = __builtin_bit_cast(u32x3, __builtin_amdgcn_raw_buffer_load_b96(frame, (int)at, 0, 0));
      lower[i] = __builtin_bit_cast(u32x3, __builtin_amdgcn_raw_buffer_load_b96(
          frame, (int)(at + (sy + 1 < (uint32_t)p.r.hi ? (uint32_t)p.r.src_pitch : 0u)), 0, 0));
    }
  } else {
    const BufferRsrc in_buf = buffer_of(p.in, (uint32_t)(p.batch * p.hin * p.win * 8));
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int q = 32 * (wave + 8 * i) + r, ry = q / N1, rx = q - ry * N1, y = 2 * y0 - 5 + ry, x = 2 * x0 - 5 + rx;
      const bool in = q < N1 * N1 && y >= 0 && y < p.mid_h && x >= 0 && x < p.mid_w;
      const int off = in ? ((img * p.hin + 2 * y) * p.win + 2 * x + 2 * h) * 8 : kOutside;
#pragma unroll
      for (int ky = 0; ky < 3; ++ky) xb[i][ky] = load16(in_buf, off, ky * p.win * 8);
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) w1[q] = load16(w_buf, lane * 16, q * 1024);
  // wavefronts 0-4 compute the second layer, 0-3 the third, 4 and 5 the last one (the others fetch nothing: 64 bytes a clock come in)
  const int lane2 = wave < 5 ? lane * 16 : kOutside, lane34 = wave < 6 ? lane * 16 : kOutside;
#pragma unroll
  for (int q = 0; q < 9; ++q) w2[q] = load16(w_buf, lane2, W2 + q * 1024);
#pragma unroll
  for (int q = 0; q < 18; ++q) w34[q] = load16(w_buf, lane34, (wave < 4 ? W3 : W4) + q * 1024);

  if constexpr (FRAME) {
    // ---- stage 1: the image's pixels, zero outside it
    __shared__ float s_lut32[256];
    __shared__ f16 s_lut16[256];
    if (threadIdx.x < 256) {
      s_lut16[threadIdx.x] = lut16;
      s_lut32[threadIdx.x] = lut32;
    }
    __syncthreads();
    const uint32_t dx = 2u * (uint32_t)p.r.wo, dy = 2u * (uint32_t)p.r.ho;
    f16* const dst = p.r.dst + (size_t)img * p.r.dst_img_stride;
    float* const dst_f32 = p.r.dst_f32 ? p.r.dst_f32 + (size_t)img * p.r.dst32_img_stride : nullptr;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int q = (int)threadIdx.x + 512 * i, row = q / W0, col = q % W0, Y = 4 * y0 - 11 + row, X = 4 * x0 - 11 + col;
      uint32_t fx, fy, v[3];
      const uint32_t sh = 3 * resize_source(X, p.r.wi, p.r.wo, p.r.rcp_dx, fx) & 3u;
      (void)resize_source(Y, p.r.hi, p.r.ho, p.r.rcp_dy, fy);
      const uint32_t a[2] = {__builtin_amdgcn_alignbyte(upper[i][1], upper[i][0], sh), __builtin_amdgcn_alignbyte(upper[i][2], upper[i][1], sh)};
      const uint32_t c[2] = {__builtin_amdgcn_alignbyte(lower[i][1], lower[i][0], sh), __builtin_amdgcn_alignbyte(lower[i][2], lower[i][1], sh)};
      resize_sum(p.r, dx * dy, a, c, dx - fx, fx, dy - fy, fy, v);
      const bool in = Y >= 0 && Y < p.r.ho && X >= 0 && X < p.r.wo;
      half4 px = {s_lut16[v[0]], s_lut16[v[1]], s_lut16[v[2]], (f16)0.0f};
      if (!in) px = half4{};
      if (q < H0 * W0) *reinterpret_cast<half4*>(&s0[q * 4]) = px;
      if (in && row >= 11 && row < 43 && col >= 11 && col < 43) {
        *reinterpret_cast<half4*>(dst + ((size_t)(Y + p.r.pad_t) * p.r.dst_w + X + p.r.pad_l) * 4) = px;
        if (dst_f32) {
          const size_t plane = (size_t)p.r.ho * p.r.wo;
          float* const o = dst_f32 + (size_t)Y * p.r.wo + X;
          o[0] = s_lut32[v[0]];
          o[plane] = s_lut32[v[1]];
          o[2 * plane] = s_lut32[v[2]];
        }
      }
    }
    __syncthreads();
    if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1 && blockIdx.y == gridDim.y - 1 && blockIdx.z == gridDim.z - 1)
      *p.r.t_end = wall_clock64();
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int q = 32 * (wave + 8 * i) + r, ry = q / N1, rx = q - ry * N1, y = 2 * y0 - 5 + ry, x = 2 * x0 - 5 + rx;
      const bool in = q < N1 * N1 && y >= 0 && y < p.mid_h && x >= 0 && x < p.mid_w;
#pragma unroll
      for (int ky = 0; ky < 3; ++ky) {
        xb[i][ky] = u32x4{};
        if (in) xb[i][ky] = *reinterpret_cast<const u32x4*>(&s0[((2 * ry + ky) * W0 + 2 * rx + 2 * h) * 4]);
      }
    }
  }
  // ---- first layer: 3 -> 16 channels, stride 2.  Zero outside the layer's map, the next layer's padding
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (wave + 8 * i >= (N1 * N1 + 31) / 32) break;
    floatx16 acc = zero16;
#pragma unroll
    for (int ky = 0; ky < 3; ++ky)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, w1[ky]), __builtin_bit_cast(half8, xb[i][ky]),
                                                  acc, 0, 0, 0);
    const int q = 32 * (wave + 8 * i) + r;
    if (q < N1 * N1) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {                                // (out of the map the pixels were zeros, and so is acc)
        half4 o = {(f16)acc[4 * j], (f16)acc[4 * j + 1], (f16)acc[4 * j + 2], (f16)acc[4 * j + 3]};
        *reinterpret_cast<half4*>(&s1[q * P1 + 8 * j + 4 * h]) = __builtin_elementwise_max(o, half4{});
      }
    }
  }
  __syncthreads();
  // One group of a further layer: pixel `at` (LDS halves of its first tap, channel 8 * h) of a source with `row` pixels per
  // row and PITCH_ halves per pixel, KS_ K-steps per tap; taps 0-4 and 5-8 are summed apart
#define HS_LAYER(ACC_, SRC_, AT_, ROW_, PITCH_, KS_, W_)                                       \
  floatx16 ACC_ = zero16;                                                                      \
  {                                                                                            \
    floatx16 acc_b = zero16;                                                                   \
    _Pragma("unroll") for (int t = 0; t < 9; ++t)                                              \
      _Pragma("unroll") for (int k = 0; k < KS_; ++k) {                                        \
        const half8 b_ = *reinterpret_cast<const half8*>(&SRC_[(AT_) + ((t / 3) * ROW_ + t % 3) * PITCH_ + 16 * k]); \
        floatx16& a_ = t < 5 ? ACC_ : acc_b;                                                   \
        a_ = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, W_[t * KS_ + k]), b_, a_, 0, 0, 0); \
      }                                                                                        \
    _Pragma("unroll") for (int i = 0; i < 16; ++i) ACC_[i] = (0.0f + ACC_[i]) + acc_b[i];      \
  }
  // ---- second layer: 16 -> 32 channels, stride 2
  if (wave < (N2 * N2 + 31) / 32) {
    const int q = 32 * wave + r, qc = min(q, N2 * N2 - 1), ry = qc / N2, rx = qc - ry * N2;
    HS_LAYER(acc, s1, (2 * ry * N1 + 2 * rx) * P1 + 8 * h, N1, P1, 1, w2)
    const int y = y0 - 2 + ry, x = x0 - 2 + rx;
    const bool in = y >= 0 && y < p.hout && x >= 0 && x < p.wout;
    if (q < N2 * N2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        half4 o = {(f16)acc[4 * j], (f16)acc[4 * j + 1], (f16)acc[4 * j + 2], (f16)acc[4 * j + 3]};
        *reinterpret_cast<half4*>(&s2[q * P2 + 8 * j + 4 * h]) = in ? __builtin_elementwise_max(o, half4{}) : half4{};
      }
    }
  }
  __syncthreads();
  // ---- third layer: 32 -> 32 channels
  if (wave < 4) {
    const int q = 32 * wave + r, qc = min(q, N3 * N3 - 1), ry = qc / N3, rx = qc - ry * N3;
    HS_LAYER(acc, s2, (ry * N2 + rx) * P2 + 8 * h, N2, P2, 2, w34)
    const int y = y0 - 1 + ry, x = x0 - 1 + rx;
    const bool in = y >= 0 && y < p.hout && x >= 0 && x < p.wout;
    if (q < N3 * N3) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        half4 o = {(f16)acc[4 * j], (f16)acc[4 * j + 1], (f16)acc[4 * j + 2], (f16)acc[4 * j + 3]};
        *reinterpret_cast<half4*>(&s3[q * P2 + 8 * j + 4 * h]) = in ? __builtin_elementwise_max(o, half4{}) : half4{};
      }
    }
  }
  __syncthreads();
  // ---- last layer: 32 -> 8 channels, the logits, and stage 3's per-cell outputs
  if (wave == 4 || wave == 5) {
    const int q = 32 * (wave - 4) + r, ry = q / N4, rx = q % N4, y = y0 + ry, x = x0 + rx;
    HS_LAYER(acc, s3, (ry * N3 + rx) * P2 + 8 * h, N3, P2, 2, w34)
    store_logits(p, y < p.hout && x < p.wout, img, y * p.wout + x, h, acc);
  }
#undef HS_LAYER
}

// =============================================================================================
// Stage 2, 3x3 layers (all of the big network's convolutions but the stem): a workgroup's output
// tile is a SPATIAL block or a run of pixels, so that the nine taps read one shared input
// patch in LDS.  Patch pixels are padded to 144 bytes: the 16
// lanes of one ds_read_b128 pass then fall into 16 different 16-byte bank
// groups (two rows of 8 pixels: with patch rows of 128 mod 256 bytes).
//
// Tile order of all of them: workgroup id mod 8 selects the XCD, and each XCD (own L2) takes a run
// of consecutive tiles.  Tiles are ordered in blocks of n_block channel tiles; inside a block the
// channel tile varies fastest, then the spatial tile.  n_block == 1: the workgroups of one L2 share
// a weight slice and every L2 that holds a channel tile fetches the input; n_block == tiles_n: they
// share input patches and every L2 fetches all the weights.  The host picks the block size that
// brings the fewest bytes into the eight L2s.
// =============================================================================================

// =============================================================================================
// A whole 64-channel BasicBlock in one launch: out = ReLU(conv_b(ReLU(conv_a(x))) + x), both
// convolutions 3x3 stride 1 pad 1, 64 -> 64 channels (one workgroup owns every channel of its
// tile, so the intermediate tensor need not leave the CU).  On small grids that saves a kernel
// boundary and a cold start, on large ones the intermediate's trip through memory (80 MB per block
// at twelve 854x480 frames).
//
// Output tile 8 x 16.  conv_b needs the intermediate on 10 x 18 pixels, conv_a therefore the
// input on 12 x 20.  Phase A: the 180 intermediate pixels in row-major order form six groups of
// 32 (the last 12 lanes idle); wavefront (wm, wn) computes groups wm, wm + 2, wm + 4 for
// channels 32*wn .. +31 and writes them -- ReLU, rounded to fp16 exactly as a layer of its own
// would store them, zero outside the image (conv_b's padding) -- into LDS over the input patch.
// Phase B: conv_b on that patch, wavefront (wm, wn) rows 4*wm .. +3.
// The 72 weight fragments of a wavefront stream from memory through one ring of FR register sets
// that runs on from conv_a into conv_b: no weight tile in LDS, and three barriers in all.  (Staged
// through LDS tap by tap they cost 18 barriers and a fragment read per K-step: one 854x480 frame
// 11.3 -> 9.4 us, four 641x361 20.6 -> 18.1, sixteen 416x240 29.2 -> 24.5; twelve 854x480 frames as
// two launches with the weights resident in LDS and registers 61.4 -> 58.9, which was the last
// grid where two launches had been the faster form.)
// FR and BD are the largest that leave three workgroups per CU (146 registers): with BD = 3 and two
// workgroups 64 us at twelve frames; FR = 9 is equal, FR = 18 (two workgroups) 64.
// Every output accumulates tap-major with four K-steps of 16 per tap, as in the other stride-1
// kernels.
// p.wt_frag / p.wt2_frag: weights of conv_a / conv_b in fragment order; p.res = p.in (the shortcut).
// =============================================================================================
__global__ __launch_bounds__(256, 3) void k_block64_fused(ConvParams p) {
  constexpr int TH = 8, TW = 16, YH = TH + 2, YW = TW + 2, XH = TH + 4, XW = TW + 4;
  constexpr int PITCH = 64 + 8;
  constexpr int RPY = (YW * PITCH * 2 + ((128 - (YW * PITCH * 2) % 256 + 256) % 256)) / 2;
  // input rows: the 18 pixels of an intermediate row end where, 16 bank groups of 16 bytes round, the next row's begin
  constexpr int RPX = XW * PITCH + 8 * (((YW - XW) * 9 % 16 + 32) % 16);
  static_assert((RPY * 2) % 256 == 128, "row pitch must be 128 mod 256 bytes");
  static_assert(RPX / 8 % 16 == YW * 9 % 16 && RPX >= XW * PITCH, "phase A's lanes must not meet in a bank group");
  static_assert(XH * RPX >= YH * RPY, "the intermediate patch is written over the input patch");
  constexpr int NPY = YH * YW;                         // 180 intermediate pixels
  constexpr int XV = XH * XW * 8, XL = (XV + 255) / 256;   // input patch vectors, per thread
  constexpr int FR = 12, BD = 2;        // weight fragments and pixel K-steps in flight
  __shared__ __align__(16) f16 s_xy[XH * RPX];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 31, h = lane >> 5;
  const uint32_t tm = (blockIdx.x & 7u) * (uint32_t)p.tiles_per_xcd + (blockIdx.x >> 3);
  const uint32_t img_u = run_div31(tm, p.by_tiles_img), ts = tm - img_u * p.tiles_img, ty = run_div31(ts, p.by_tiles_x);
  const int img = (int)img_u, y0 = (int)ty * TH, x0 = (int)(ts - ty * (uint32_t)p.tiles_x) * TW;
  const int wm = wave & 1, wn = wave >> 1;

  // ---- input patch: pixel (y0 - 2 + py, x0 - 2 + px), zeros outside the image
  const BufferRsrc in_buf = buffer_of(p.in, p.run_in_bytes), wa_buf = buffer_of(p.wt_frag, 72 * 1024),
                   wb_buf = buffer_of(p.wt2_frag, 72 * 1024);
  u32x4 st_x[XL];
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int v = tid + 256 * i;
    const int pix = v >> 3, py = pix / XW, px = pix - py * XW;
    const int iy = y0 - 2 + py, ix = x0 - 2 + px;
    const bool in = v < XV && iy >= 0 && iy < p.hin && ix >= 0 && ix < p.win;
    st_x[i] = load16(in_buf, in ? (((img * p.hin + iy) * p.win + ix) * p.cin_pitch + (tid & 7) * 8) * 2 : kOutside, 0);
  }
  // ---- weight fragments of this wavefront's 32 channels: 36 of conv_a, then 36 of conv_b
  const int w0 = wn * 36 * 1024;
  u32x4 fa[FR];
#pragma unroll
  for (int q = 0; q < FR; ++q) fa[q] = load16(wa_buf, lane * 16, w0 + q * 1024);
  // (only here: see k_conv3x3_run; a surplus workgroup's pixels lie behind the buffer, and the weights are every tile's)
  if (tm >= (uint32_t)p.tiles_m) return;
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int v = tid + 256 * i;
    if (v < XV) {
      const int pix = v >> 3, py = pix / XW, px = pix - py * XW;
      *reinterpret_cast<u32x4*>(&s_xy[py * RPX + px * PITCH + (v & 7) * 8]) = st_x[i];
    }
  }

  const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // ---- phase A: intermediate pixel q = 32*(wm + 2k) + r of the 10 x 18 patch, k = 0..2
  int a_py[3], a_px[3], a_off[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int q = min(32 * (wm + 2 * k) + r, NPY - 1);
    a_py[k] = q / YW;
    a_px[k] = q - a_py[k] * YW;
    a_off[k] = a_py[k] * RPX + a_px[k] * PITCH + h * 8;
  }
  floatx16 acc_a[3] = {zero16, zero16, zero16};
  half8 bf[BD + 1][3];
  // K-step Q_ of a convolution: tap Q_ / 4, K-step Q_ % 4 of it
#define HS_READ_A(Q_)                                                                          \
  _Pragma("unroll") for (int k = 0; k < 3; ++k)                                                \
    bf[(Q_) % (BD + 1)][k] = *reinterpret_cast<const half8*>(                                  \
        &s_xy[a_off[k] + ((Q_) / 12) * RPX + (((Q_) / 4) % 3) * PITCH + ((Q_) % 4) * 16]);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < BD; ++q) HS_READ_A(q)
#pragma unroll
  for (int q = 0; q < 36; ++q) {
    if (q + BD < 36) HS_READ_A(q + BD)
    const half8 a = __builtin_bit_cast(half8, fa[q % FR]);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      acc_a[k] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bf[q % (BD + 1)][k], acc_a[k], 0, 0, 0);
    fa[q % FR] = q + FR < 36 ? load16(wa_buf, lane * 16, w0 + (q + FR) * 1024) : load16(wb_buf, lane * 16, w0 + (q + FR - 36) * 1024);
    __builtin_amdgcn_sched_barrier(0);
  }
#undef HS_READ_A
  __syncthreads();          // every wavefront is done with the input patch
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int q = 32 * (wm + 2 * k) + r;
    const int iy = y0 - 1 + a_py[k], ix = x0 - 1 + a_px[k];
    const bool inside = iy >= 0 && iy < p.hin && ix >= 0 && ix < p.win;
    if (q < NPY) {
      f16* dst = &s_xy[a_py[k] * RPY + a_px[k] * PITCH + wn * 32 + h * 4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        half4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = (f16)acc_a[k][4 * i + j];
        o = inside ? __builtin_elementwise_max(o, half4{}) : half4{};
        *reinterpret_cast<half4*>(dst + 8 * i) = o;
      }
    }
  }

  // ---- residual of this tile (the block's input), fetched now, used after phase B: two 16-byte
  // pieces per pixel (res_octets_to_quads)
  const int oy = y0 + 4 * wm + (r >> 3);
  u32x4 res_raw[2][2];
  {
    const int oy_c = min(oy, p.hout - 1);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int ox_c = min(x0 + 8 * g + (r & 7), p.wout - 1);
      const f16* rp = p.res + (size_t)(img * p.img_m + oy_c * p.wout + ox_c) * p.res_pitch + wn * 32 + h * 8;
      res_raw[g][0] = *reinterpret_cast<const u32x4*>(rp);
      res_raw[g][1] = *reinterpret_cast<const u32x4*>(rp + 16);
    }
  }
  __syncthreads();          // the intermediate patch is complete

  // ---- phase B: conv_b on the intermediate patch
  const int fp_off = (4 * wm + (r >> 3)) * RPY + (r & 7) * PITCH + h * 8;
  floatx16 acc_b[2] = {zero16, zero16};
#define HS_READ_B(Q_)                                                                          \
  _Pragma("unroll") for (int g = 0; g < 2; ++g)                                                \
    bf[(Q_) % (BD + 1)][g] = *reinterpret_cast<const half8*>(                                  \
        &s_xy[fp_off + ((Q_) / 12) * RPY + (((Q_) / 4) % 3) * PITCH + g * 8 * PITCH + ((Q_) % 4) * 16]);
#pragma unroll
  for (int q = 0; q < BD; ++q) HS_READ_B(q)
#pragma unroll
  for (int q = 0; q < 36; ++q) {
    if (q + BD < 36) HS_READ_B(q + BD)
    const half8 a = __builtin_bit_cast(half8, fa[q % FR]);
#pragma unroll
    for (int g = 0; g < 2; ++g)
      acc_b[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bf[q % (BD + 1)][g], acc_b[g], 0, 0, 0);
    if (q + FR < 36) fa[q % FR] = load16(wb_buf, lane * 16, w0 + (q + FR) * 1024);
    __builtin_amdgcn_sched_barrier(0);
  }
#undef HS_READ_B
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int ox = x0 + 8 * g + (r & 7);
    half4 res_q[4];
    res_octets_to_quads(res_raw[g], res_q);
    store_octets(p, oy < p.hout && ox < p.wout, img * p.img_m + oy * p.wout + ox, wn * 32, h,
                 acc_b[g], res_q, true);
  }
}

// =============================================================================================
// 3x3 stride-2 pad-1 layers (with the block's 1x1 stride-2 projection riding along) of one Cin chunk
// on grids beyond two rounds of workgroups (the others: k_conv3x3s2_run).  Output tile 8 x 8
// pixels x 128 channels; wavefront w = all 64 pixels (two groups of four rows), channels
// 32*w .. +31: a weight fragment is fetched by one wavefront only and serves two MFMAs, and
// the patch -- the heavy operand of a stride-2 tile -- serves 128 channels.
// A stride-2 tile needs four input pixels per output pixel (17 x 17 of them), and with the
// weight tile in LDS and a barrier per tap a wavefront got four MFMAs per barrier: those layers
// ran the matrix pipe at 16-23 %.  Here
//   - the weights come as MFMA fragments straight from memory (p.wt_frag, and p.wt2_frag for the
//     projection), three taps ahead: no weight tile, no per-tap barrier;
//   - the patch is cut into half chunks of 32 input channels (one "item" = one half chunk of
//     one tile: nine taps + the projection, two K-steps of 16 each), stored as four parity
//     planes of 9 x 9 pixels (pixel (py, px) in plane (py & 1, px & 1) at (py / 2, px / 2), so that
//     the lanes of a tap read neighbouring plane pixels) with 64 bytes per pixel and no padding:
//     the four 16-byte vectors of a pixel are permuted by its plane row and column
//     (v ^ ((col >> 2) & 1 | (row & 1) << 1)), which makes every fragment read conflict free.
//     Two buffers of 20 KB: the next item's patch streams in during the taps of the current
//     one (four vectors per thread in flight), one barrier per item, two workgroups per CU
//     (four accumulators per wavefront with the projection's);
//   - a workgroup walks tiles_per_wg consecutive spatial tiles in one pipeline (the next tile's
//     first patch and weights are fetched during the last taps of the current tile), so the
//     short K loops of the 64-channel layer do not pay a cold start per tile.
// Per output the K order is chunk, half chunk, tap, K-step.
// =============================================================================================
__global__ __launch_bounds__(256, 2) void k_conv3x3s2_dira(ConvParams p) {
  constexpr int TH = 8, TW = 8, IPW = 2 * TW + 1, NPIX = IPW * IPW;   // 17 x 17 input pixels
  constexpr int PLW = TW + 1, PLANE = PLW * PLW;                      // 9 x 9 pixels per parity plane
  constexpr int PV = NPIX * 4, PL = (PV + 255) / 256;                 // 16-byte vectors, per thread
  static_assert(PL == 5, "the patch pipeline below is written out for five vectors per thread");
  __shared__ __align__(16) f16 s_patch[2][4 * PLANE * 32];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 31, h = lane >> 5;
  const int tile = (int)(blockIdx.x & 7u) * p.tiles_per_xcd + (int)(blockIdx.x >> 3);
  const int groups_m = (p.tiles_m + p.tiles_per_wg - 1) / p.tiles_per_wg;
  if (tile >= groups_m * p.tiles_n) return;
  const int blk = groups_m * p.n_block, in_blk = tile % blk;       // tile order: see above
  const int tm_begin = (in_blk / p.n_block) * p.tiles_per_wg;
  const int tm_end = min(p.tiles_m, tm_begin + p.tiles_per_wg);
  const int tile_n = (tile / blk) * p.n_block + in_blk % p.n_block;
  const int tiles_img = p.tiles_m / p.batch;
  const int n0 = tile_n * 128;
  const int n_halves = 2 * p.chunks_per_tap;                      // items per tile
  const int n_items = (tm_end - tm_begin) * n_halves;
  const bool has_proj = p.wt2_frag != nullptr;

  // ---- patch loader: the LDS slot of every vector is fixed, its source depends on the tile
  int l_plds[PL], l_pyx[PL], l_poff[PL];
#pragma unroll
  for (int i = 0; i < PL; ++i) {
    const int vec = tid + 256 * i, pix = min(vec >> 2, NPIX - 1), v = vec & 3;
    const int py = pix / IPW, px = pix - py * IPW, prow = py >> 1, pcol = px >> 1;
    const int sw = ((pcol >> 2) & 1) | ((prow & 1) << 1);
    l_pyx[i] = py | (px << 8);
    l_plds[i] = vec >= PV ? -1
                          : ((((py & 1) * 2 + (px & 1)) * PLANE + prow * PLW + pcol) * 4 + (v ^ sw)) * 8;
  }
  // source offsets (halves from p.in, channel 8 * (tid & 3) of the pixel; -1: padding) of tile TM_
#define HS_TILE_SETUP(TM_, IMG_, Y0_, X0_)                                                     \
  {                                                                                            \
    IMG_ = (TM_) / tiles_img;                                                                  \
    const int ts_ = (TM_) - IMG_ * tiles_img, ty_ = ts_ / p.tiles_x;                           \
    Y0_ = ty_ * TH;                                                                            \
    X0_ = (ts_ - ty_ * p.tiles_x) * TW;                                                        \
    _Pragma("unroll") for (int i = 0; i < PL; ++i) {                                           \
      const int iy_ = 2 * Y0_ + (l_pyx[i] & 0xff) - 1, ix_ = 2 * X0_ + (l_pyx[i] >> 8) - 1;    \
      const bool inb_ = l_plds[i] >= 0 && iy_ >= 0 && iy_ < p.hin && ix_ >= 0 && ix_ < p.win;  \
      l_poff[i] = inb_ ? ((IMG_ * p.hin + iy_) * p.win + ix_) * p.cin_pitch + (tid & 3) * 8 : -1; \
    }                                                                                          \
  }
  u32x4 st_p[4];
#define HS_LOAD_P(I_) \
  st_p[(I_) & 3] = *reinterpret_cast<const u32x4*>(p.in + (l_poff[I_] >= 0 ? l_poff[I_] + ch_n : 0));
#define HS_HAND_P(I_, PB_)                                                                     \
  if (l_plds[I_] >= 0) {                                                                       \
    const u32x4 zero_ = {0u, 0u, 0u, 0u};                                                      \
    *reinterpret_cast<u32x4*>(&s_patch[PB_][l_plds[I_]]) = l_poff[I_] >= 0 ? st_p[(I_) & 3] : zero_; \
  }

  // ---- pixel fragments: lane (r, h) reads output pixels (4*g + r/8, r%8), g = 0, 1; tap (ky, kx)
  // reads plane (ky & 1, kx & 1) at (+ky/2, +kx/2); K-step j of the item is vector 2*j + h of the
  // pixel.  Group 1 lies four plane rows below group 0 (same row parity, same permutation).
  constexpr int GOFF = 4 * PLW * 32;
  const int oy_l = r >> 3, ox_l = r & 7;
  int fb[2][2][2];    // [ky / 2][kx / 2][j]: halves offset inside a plane
#pragma unroll
  for (int dy = 0; dy < 2; ++dy)
#pragma unroll
    for (int dx = 0; dx < 2; ++dx) {
      const int prow = oy_l + dy, pcol = ox_l + dx;
      const int sw = ((pcol >> 2) & 1) | ((prow & 1) << 1);
#pragma unroll
      for (int j = 0; j < 2; ++j) fb[dy][dx][j] = ((prow * PLW + pcol) * 4 + ((2 * j + h) ^ sw)) * 8;
    }

  // ---- weight fragments of this wavefront's 32 channels: blocks of 64 lanes x 16 bytes,
  // [chunk][tap][K-step of 16] for the 3x3 taps, [chunk][K-step] for the projection
  const u32x4* const wf0 = reinterpret_cast<const u32x4*>(p.wt_frag) +
                           (size_t)(n0 / 32 + wave) * p.chunks_per_tap * (9 * 4 * 64) + lane;
  const u32x4* const wp0 = has_proj ? reinterpret_cast<const u32x4*>(p.wt2_frag) +
                                          (size_t)(n0 / 32 + wave) * p.chunks_per_tap * (4 * 64) + lane
                                    : wf0;
  // half chunk HF_ (0 .. n_halves - 1): chunk HF_ / 2, K-steps 2 * (HF_ & 1) ..
#define HS_WBASE(HF_) (wf0 + ((size_t)((HF_) >> 1) * 36 + 2 * ((HF_) & 1)) * 64)
#define HS_PBASE(HF_) (wp0 + ((size_t)((HF_) >> 1) * 4 + 2 * ((HF_) & 1)) * 64)
  u32x4 fa[3][2], fp2[2];
#define HS_LOAD_A(S_, BASE_, T_)                                                               \
  {                                                                                            \
    fa[S_][0] = (BASE_)[(T_) * 4 * 64];                                                        \
    fa[S_][1] = (BASE_)[(T_) * 4 * 64 + 64];                                                   \
  }

  const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  floatx16 acc[2] = {zero16, zero16}, acc2[2] = {zero16, zero16};

  // K-step Q_ (literal) of the current item: Q_ / 2 = tap (9: the projection, on the centre
  // tap's pixels), Q_ & 1 = which 16 of the item's 32 channels.  Pixel fragments are read BD
  // steps ahead (ring of BD + 1); weight stage tap % 3 is refilled behind its last use with
  // the tap three ahead, from the next item's block once that runs past this item's ninth tap.
  constexpr int BD = 3;
  half8 bf[BD + 1][2];
#define HS_TAPQ(Q_) ((Q_) / 2 == 9 ? 4 : (Q_) / 2)     /* the projection reads the centre tap */
#define HS_READ_B(Q_)                                                                          \
  {                                                                                            \
    const f16* fp_ = &s_patch[pb][((((HS_TAPQ(Q_) / 3) & 1) * 2 + ((HS_TAPQ(Q_) % 3) & 1)) * PLANE) * 32 + \
                                  fb[(HS_TAPQ(Q_) / 3) >> 1][(HS_TAPQ(Q_) % 3) >> 1][(Q_) & 1]]; \
    bf[(Q_) % (BD + 1)][0] = *reinterpret_cast<const half8*>(fp_);                             \
    bf[(Q_) % (BD + 1)][1] = *reinterpret_cast<const half8*>(fp_ + GOFF);                      \
  }
#define HS_KSTEP(Q_)                                                                           \
  {                                                                                            \
    if ((Q_) + BD < 20) { if ((Q_) + BD < 18 || has_proj) HS_READ_B((Q_) + BD) }               \
    if (((Q_) & 1) == 0 && more) {                                                             \
      if ((Q_) / 2 >= 3 && (Q_) / 2 - 3 < PL) HS_HAND_P((Q_) / 2 - 3, pb ^ 1)                  \
      if ((Q_) / 2 < PL) HS_LOAD_P((Q_) / 2)                                                   \
    }                                                                                          \
    if ((Q_) < 18) {                                                                           \
      const half8 a_ = __builtin_bit_cast(half8, fa[((Q_) / 2) % 3][(Q_) & 1]);                \
      _Pragma("unroll") for (int g = 0; g < 2; ++g)                                            \
        acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_, bf[(Q_) % (BD + 1)][g], acc[g], 0, 0, 0); \
      if ((Q_) & 1) {                                                                          \
        if ((Q_) / 2 + 3 < 9) HS_LOAD_A(((Q_) / 2) % 3, w_cur, (Q_) / 2 + 3)                   \
        else HS_LOAD_A(((Q_) / 2) % 3, w_nxt, (Q_) / 2 + 3 - 9)                                \
      }                                                                                        \
    } else if (has_proj) {                                                                     \
      const half8 a_ = __builtin_bit_cast(half8, fp2[(Q_) & 1]);                               \
      _Pragma("unroll") for (int g = 0; g < 2; ++g)                                            \
        acc2[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_, bf[(Q_) % (BD + 1)][g], acc2[g], 0, 0, 0); \
    }                                                                                          \
    __builtin_amdgcn_sched_barrier(0);                                                         \
  }

  // ---- prologue: first item's patch into buffer 0, its first three taps of weights
  int img, y0, x0;
  HS_TILE_SETUP(tm_begin, img, y0, x0)
  int pb = 0;
  {
    u32x4 first[PL];
#pragma unroll
    for (int i = 0; i < PL; ++i)
      first[i] = *reinterpret_cast<const u32x4*>(p.in + (l_poff[i] >= 0 ? l_poff[i] : 0));
    const u32x4* w0 = HS_WBASE(0);
    HS_LOAD_A(0, w0, 0) HS_LOAD_A(1, w0, 1) HS_LOAD_A(2, w0, 2)
#pragma unroll
    for (int i = 0; i < PL; ++i)
      if (l_plds[i] >= 0) {
        const u32x4 zero = {0u, 0u, 0u, 0u};
        *reinterpret_cast<u32x4*>(&s_patch[0][l_plds[i]]) = l_poff[i] >= 0 ? first[i] : zero;
      }
  }
  __syncthreads();

  int tm = tm_begin, hf = 0;
  for (int item = 0; item < n_items; ++item) {
    // the item after this one: next half chunk of the tile, or the first of the next tile
    const bool more = item + 1 < n_items;
    const bool cross = hf + 1 == n_halves;
    const int hf_n = more ? (cross ? 0 : hf + 1) : hf;
    const int s_img = img, s_y0 = y0, s_x0 = x0;      // this item's tile (for the store below)
    if (more && cross) HS_TILE_SETUP(tm + 1, img, y0, x0)   // l_poff now describes the next tile
    const int ch_n = (hf_n >> 1) * 64 + (hf_n & 1) * 32;
    const u32x4* const w_cur = HS_WBASE(hf);
    const u32x4* const w_nxt = HS_WBASE(hf_n);
    if (has_proj) {
      const u32x4* pbase = HS_PBASE(hf);
      fp2[0] = pbase[0];
      fp2[1] = pbase[64];
    }
    HS_READ_B(0) HS_READ_B(1) HS_READ_B(2)
    HS_KSTEP(0) HS_KSTEP(1) HS_KSTEP(2) HS_KSTEP(3) HS_KSTEP(4) HS_KSTEP(5) HS_KSTEP(6)
    HS_KSTEP(7) HS_KSTEP(8) HS_KSTEP(9) HS_KSTEP(10) HS_KSTEP(11) HS_KSTEP(12) HS_KSTEP(13)
    HS_KSTEP(14) HS_KSTEP(15) HS_KSTEP(16) HS_KSTEP(17) HS_KSTEP(18) HS_KSTEP(19)
    if (cross) {
      // ---- the tile is complete: group g = pixel (4*g + r/8, r%8) of the tile
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int oy = s_y0 + 4 * g + oy_l, ox = s_x0 + ox_l;
        const bool valid = oy < p.hout && ox < p.wout;
        const int m = s_img * p.img_m + oy * p.wout + ox;
        // fp16 outputs with whole 128-channel tiles (the host selects this kernel only then)
        const half4 none[4] = {};
        store_octets(p, valid, m, n0 + wave * 32, h, acc[g], none, false);
        if (has_proj)                            // projection: no residual, no ReLU
          store_octets_to(p.out2, p.out2_pitch, false, valid, m, n0 + wave * 32, h, acc2[g], none,
                          false);
      }
      acc[0] = acc[1] = zero16;
      acc2[0] = acc2[1] = zero16;
      ++tm;
    }
    hf = hf_n;
    __syncthreads();      // the next patch is complete, and every wavefront is done with this one
    pb ^= 1;
  }
#undef HS_KSTEP
#undef HS_READ_B
#undef HS_TAPQ
#undef HS_LOAD_A
#undef HS_PBASE
#undef HS_WBASE
#undef HS_HAND_P
#undef HS_LOAD_P
#undef HS_TILE_SETUP
}

// Touches this workgroup's share of the next layer's weights (one 4-byte load per 128-byte line),
// so that they are on their way into the last-level cache when that layer starts: streamed from
// HBM by the layer itself, every ring of fragments in flight costs a full memory latency.  Called
// behind the K loop; the loads complete during the epilogue (the values are consumed at its end).
// At most four lines per thread, all in flight at once: a grid of few workgroups leaves the rest to the next layer (sixteen
// 8 x 8 inputs, up to 27 lines per thread one after the other 150 us a pass, so 128; two 192 x 108 123, 114).
constexpr int kTouched = 4;
__device__ __forceinline__ void prefetch_next(const RunParams& p, int block, int n_blocks, uint32_t (&x)[kTouched]) {
  const BufferRsrc buf = buffer_of(p.next_wt, (uint32_t)p.next_lines * 128);
  const uint32_t stride = (uint32_t)n_blocks * blockDim.x, first = (uint32_t)block * blockDim.x + threadIdx.x;
#pragma unroll
  for (int k = 0; k < kTouched; ++k) {
    const uint32_t i = first + k * stride;
    x[k] = __builtin_amdgcn_raw_buffer_load_b32(buf, i < (uint32_t)p.next_lines ? (int)(i * 128) : kOutside, 0, 0);
  }
}

// =============================================================================================
// 3x3 stride-1 pad-1 layers with several Cin chunks (stages 2-4 and the ConvLSTM gates), at every size.
// A tile is 32 * CW channels x a RUN of 32 * PG consecutive pixels: the map is cut into strips of strip_w columns, and
// the pixels of all strips of all images of the launch, row by row, are one list that the runs are cut from.  So no
// tile but the last is partly empty, whatever the map (tiles of 8 x 16 pixels are to 79 % full on a 27 x 15 map), and
// the host can pick the tile whose count fills the CUs (Builder::choose_form).
//   - The patch under a run, the border columns and a row of zeros between the images included, goes through LDS one
//     chunk of 64 input channels at a time, double buffered: a chunk's loads are issued two chunks ahead, one barrier
//     per chunk.  Rows are padded so that the pixel behind a row's last one lies in the bank group it would lie in
//     without the border pixels between them: the lanes of a run never meet (gates, twelve 854 x 480 frames, without:
//     a fifth of the cycles).
//   - The KS K splits are wavefronts of the workgroup: of the four K-steps of every tap a wavefront takes 4 / KS.  Each
//     weight fragment is fetched by one wavefront only, straight from memory through a ring of FR register sets, and
//     serves PG MFMAs: what bounds these layers is the 64 bytes per clock a CU takes in, and with the splits inside the
//     tile a tile's weights come in once (two wavefronts that share a channel group fetch them twice).
//   - All loads have scalar offsets into buffers of known size: no address arithmetic in the loop, and padding reads
//     as zeros (flat pointers and selects instead: 4 to 10 % of a launch).
//   - The partial sums meet in LDS and are added in pairs; every wavefront finishes its share of the channels.
// Per output and K split: chunk, tap, K-step; then the splits in pairs.
// PL: 16-byte vectors of a patch per thread; LDS: bytes of a patch buffer (128 of them taken by vectors beyond the
// patch); FR, BD: weight and pixel fragments in flight; OCC: workgroups per CU.  The values are the fastest of those
// tried on eleven sizes from 192 x 110 x 1 to 854 x 480 x 12 frames.  (A wavefront with 64 channels x 64 to 160 pixels
// and four K splits moves the fewest bytes, but its registers leave one workgroup per CU or too few fragments in
// flight: 2 to 10 % slower.)
// Against the kernels it replaced (8 x 16-pixel tiles x 64 channels, or 32 to 64-pixel tiles with the K splits
// chunk by chunk), mean us per layer of 128 / 256 / 512 channels and gates: one 288 x 160 frame 6.4 / 6.3 / 7.0 / 8.9
// -> 4.5 / 5.1 / 6.6 / 8.3, one 854 x 480 frame 7.5 / 7.5 / 7.4 / 15.2 -> 6.2 / 6.2 / 6.9 / 11.2, four 641 x 361
// frames 12.7 / 12.5 / 16.4 / 27.0 -> 8.5 / 8.5 / 9.6 / 17.5, sixteen 416 x 240 frames 15.1 / 14.5 / 18.7 / 31.5 ->
// 12.9 / 12.0 / 12.2 / 27.2, twelve 854 x 480 frames 32.7 / 32.4 / 35.1 / 81 -> 29.6 / 25.8 / 26.3 / 62.
// =============================================================================================
template <int PG, int KS, int CW, int FR, int BD, int PL, int LDS, int OCC>
__global__ __launch_bounds__(64 * KS * CW, OCC) void k_conv3x3_run(RunParams p) {
  constexpr int NW = KS * CW, C = 32 * CW, PITCH = kRunPitch;
  constexpr int KK = 4 / KS, SPC = 9 * KK;        // K-steps of a tap, of a chunk, that a wavefront takes
  static_assert(2 * SPC % FR == 0, "the fragment ring must divide the K-steps of two chunks");
  // accumulators are finished in pieces of 16 channels x 32 pixels (QU = 2 quads per lane), or 8 where there are fewer
  // such pieces than K splits
  constexpr int QU = 2 * PG < KS ? 1 : 2, UNITS = 4 / QU * PG, UB = QU * 1024;
  constexpr int UN = UNITS / KS;                                   // pieces a wavefront finishes
  static_assert(UNITS % KS == 0, "every K split finishes the same number of pieces");
  constexpr int RED = UNITS * NW * UB, SHM = RED > 2 * LDS ? RED : 2 * LDS;
  static_assert(RED <= 2 * LDS || RED <= 65536, "the partial sums take no more LDS than the patches, or 64 KB");
  __shared__ __align__(16) unsigned char s_raw[SHM];
  f16* const s_patch = reinterpret_cast<f16*>(s_raw);

  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave % KS, cw = wave / KS;
  // the parameters of the prologue, all in one round trip
  asm volatile("" ::"s"(p.in), "s"(p.wt_frag), "s"(p.run_in_bytes), "s"(p.run_w_bytes), "s"(p.cin_pitch), "s"(p.chunks_per_tap),
               "s"(p.tiles_per_xcd), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.n_block), "s"(p.run_by_blk), "s"(p.run_nb_shift),
               "s"(p.run.strip_w), "s"(p.run.rows), "s"(p.run.h), "s"(p.run.w), "s"(p.run.by_strip_w), "s"(p.run.by_h),
               "s"(p.run.by_batch), "s"(p.run.by23_row));
  const uint32_t tile = (blockIdx.x & 7u) * (uint32_t)p.tiles_per_xcd + (blockIdx.x >> 3);
  const RunTile rt = run_tile(tile, p.tiles_m, p.tiles_n, p.n_block, p.run_nb_shift, p.run_by_blk);   // tile order: see above
  const int n0 = (int)rt.channels * C;
  const RunOrigin org = run_origin(p.run, rt.run);
  const int rw = p.run.strip_w + 2, rp = run_row_pitch(p.run.strip_w);   // patch pixels, LDS halves per row

  const BufferRsrc in_buf = buffer_of(p.in, p.run_in_bytes), w_buf = buffer_of(p.wt_frag, p.run_w_bytes);
  u32x4 first[PL];
  // ---- patch loader: pixel (tid + threads * i) / 8 of the patch: source offset in bytes (padding: reads as
  // zeros), LDS slot (beyond the patch: 128 bytes that nothing reads)
  int l_poff[PL], l_lds[PL];
  {
    const uint32_t pix = (uint32_t)tid >> 3;
    uint32_t prow = run_div23(pix, p.run.by23_row), pcol = pix - prow * (uint32_t)rw;
#pragma unroll
    for (int i = 0; i < PL; ++i) {
      int m;
      const bool fits = prow < (uint32_t)p.run.rows, in = run_patch_pixel(p.run, org, prow, pcol, m) && fits;
      l_poff[i] = in ? (m * p.cin_pitch + (tid & 7) * 8) * 2 : kOutside;
      l_lds[i] = fits ? (int)prow * rp + (int)pcol * PITCH + (tid & 7) * 8 : LDS / 2 - 64 + (tid & 7) * 8;
      first[i] = load16(in_buf, l_poff[i], 0);
      prow += (uint32_t)p.run.step_q;
      pcol += (uint32_t)p.run.step_r;
      if (pcol >= (uint32_t)rw) { pcol -= (uint32_t)rw; ++prow; }
    }
  }
  u32x4 st_p[PL];
#define HS_LOAD_P(I_, CC_) st_p[I_] = load16(in_buf, l_poff[I_], (CC_) * 128);
#define HS_HAND_P(V_, I_, B_) *reinterpret_cast<u32x4*>(&s_patch[(B_) * (LDS / 2) + l_lds[I_]]) = (V_);

  // ---- prologue: loads of the first patch (and the second), of the weight ring, in the order of the loop below,
  // whose waits count the loads issued since
  const int n_cc = p.chunks_per_tap;                               // even
#pragma unroll
  for (int i = 0; i < PL; ++i) HS_LOAD_P(i, 1)
  int wf = ((n0 / 32 + cw) * n_cc * 36 + ks * KK) * 1024;          // bytes from wt_frag on
  // K-step S_ (literal, counted from an even chunk) of this wavefront
#define HS_WOFF(S_) ((((S_) / SPC) * 36 + (((S_) % SPC) / KK) * 4 + (S_) % KK) * 1024)
  u32x4 fa[FR];
#pragma unroll
  for (int s = 0; s < FR; ++s) fa[s] = load16(w_buf, lane * 16, wf + HS_WOFF(s));
  // ---- pixels of this wavefront: LDS offset of a pixel's first tap, output pixel (-1: none)
  auto pixel = [&](int g, int& lds, int& m) {
    uint32_t row, col;
    run_pixel(p.run, org, 32 * g + r, row, col, m);
    lds = (int)row * rp + (int)col * PITCH + h * 8 + ks * KK * 16;
  };
  int fpo[PG], o_m[PG];
#pragma unroll
  for (int g = 0; g < PG; ++g) pixel(g, fpo[g], o_m[g]);
  // (Only here: an exit further up would split the loads of the parameters into several round trips.  Beyond the last tile all
  // of the above is the last tile's.)
  if (tile >= (uint32_t)(p.tiles_m * p.tiles_n)) return;
#pragma unroll
  for (int i = 0; i < PL; ++i) HS_HAND_P(first[i], i, 0)
  __syncthreads();

  const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  floatx16 acc[PG];
#pragma unroll
  for (int g = 0; g < PG; ++g) acc[g] = zero16;
  // Pixel fragment F_ = K-step * PG + group of a chunk, read BD fragments ahead of its MFMAs
  half8 bf[BD + 1];
#define HS_READ_B(U_, F_)                                                                      \
  bf[(F_) % (BD + 1)] = *reinterpret_cast<const half8*>(                                       \
      &s_patch[(U_) * (LDS / 2) + fpo[(F_) % PG] + ((F_) / PG / KK / 3) * rp +                 \
               (((F_) / PG / KK) % 3) * PITCH + (((F_) / PG) % KK) * 16]);
  // Chunk cc + U_ (U_ literal: its parity).  The next chunk's patch, fetched a chunk ago, goes to the other buffer
  // spread over the K-steps, and its registers are refilled with the chunk behind that.
#define HS_CHUNK(U_, LAST_)                                                                    \
  {                                                                                            \
    _Pragma("unroll") for (int f = 0; f < BD; ++f) HS_READ_B(U_, f)                            \
    _Pragma("unroll") for (int s = 0; s < SPC; ++s) {                                          \
      _Pragma("unroll") for (int i = 0; i < PL; ++i)                                           \
        if ((2 * i + 1) * SPC / (2 * PL) == s && (!(LAST_) || (U_) == 0)) {                    \
          HS_HAND_P(st_p[i], i, 1 - (U_))                                                      \
          if (!(LAST_)) HS_LOAD_P(i, min(cc + (U_) + 2, n_cc - 1))                             \
        }                                                                                      \
      _Pragma("unroll") for (int g = 0; g < PG; ++g) {                                         \
        if (s * PG + g + BD < SPC * PG) HS_READ_B(U_, s * PG + g + BD)                         \
        acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(                                       \
            __builtin_bit_cast(half8, fa[((U_) * SPC + s) % FR]), bf[(s * PG + g) % (BD + 1)], acc[g], 0, 0, 0); \
        if (PG > 2) __builtin_amdgcn_sched_barrier(0);                                         \
      }                                                                                        \
      if (!(LAST_) || (U_) * SPC + s + FR < 2 * SPC)                                           \
        fa[((U_) * SPC + s) % FR] = load16(w_buf, lane * 16, wf + HS_WOFF((U_) * SPC + s + FR)); \
      __builtin_amdgcn_sched_barrier(0);                                                       \
    }                                                                                          \
  }
  int cc = 0;
  for (; cc + 2 < n_cc; cc += 2) {
    HS_CHUNK(0, false)
    __syncthreads();
    HS_CHUNK(1, false)
    __syncthreads();
    wf += 72 * 1024;
  }
  // residual of the pieces this wavefront finishes (without one: any address, so that the loads are
  // unconditional), fetched behind the last chunks
  u32x4 res_raw[UN];
  {
    const f16* const rsp = p.res ? p.res + n0 + cw * 32 + 4 * QU * h : p.in;
    const int pitch = p.res ? p.res_pitch : 0;
#pragma unroll
    for (int k = 0; k < UN; ++k) {
      const int q = (ks * UN + k) * QU;
      int lds, m;
      pixel(q / 4, lds, m);
      const f16* const at = rsp + (size_t)max(m, 0) * pitch + (p.res ? 8 * (q % 4) : 0);
      if (QU == 2) {
        res_raw[k] = *reinterpret_cast<const u32x4*>(at);
      } else {
        const uint2 v = *reinterpret_cast<const uint2*>(at);
        res_raw[k] = {v.x, v.y, 0u, 0u};
      }
    }
  }
  HS_CHUNK(0, true)
  __syncthreads();
  HS_CHUNK(1, true)
#undef HS_CHUNK
#undef HS_READ_B
#undef HS_WOFF
#undef HS_HAND_P
#undef HS_LOAD_P

  uint32_t touched[kTouched] = {};
  if (p.next_lines) prefetch_next(p, (int)tile, p.tiles_m * p.tiles_n, touched);
  __syncthreads();                   // every wavefront is done with the patches
  float4* const s_red = reinterpret_cast<float4*>(s_raw) + (size_t)(wave / KS) * KS * UNITS * (UB / 16) + lane;
#pragma unroll
  for (int u = 0; u < UNITS; ++u)
    if (u / UN != ks) {
      const int q = u * QU;                                        // first quad of the piece
      const floatx16& a = acc[q / 4];
#pragma unroll
      for (int j = 0; j < QU; ++j) {
        const int o = 4 * (q % 4 + j);
        s_red[(ks * UNITS + u) * (UB / 16) + 64 * j] = make_float4(a[o], a[o + 1], a[o + 2], a[o + 3]);
      }
    }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < UNITS; ++u)
    if (u / UN == ks) {
      const int q = u * QU;
      const floatx16& a = acc[q / 4];
      float4 v[2];
#pragma unroll
      for (int j = 0; j < QU; ++j) {
        const int o = 4 * (q % 4 + j);
        float4 b[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) {
          b[k] = make_float4(a[o], a[o + 1], a[o + 2], a[o + 3]);
          if (k != ks) b[k] = s_red[(k * UNITS + u) * (UB / 16) + 64 * j];
        }
#pragma unroll
        for (int d = KS / 2; d >= 1; d /= 2)                       // in pairs
#pragma unroll
          for (int k = 0; k < d; ++k) {
            b[k].x += b[k + d].x; b[k].y += b[k + d].y; b[k].z += b[k + d].z; b[k].w += b[k + d].w;
          }
        v[j] = b[0];
      }
      const int cbase = n0 + cw * 32 + 8 * (q % 4), m = o_m[q / 4];
      if (p.use_partial) {
        if (m >= 0) {
          float* dst = p.partial + (size_t)m * p.cout_pad + cbase + 4 * h;
#pragma unroll
          for (int j = 0; j < QU; ++j) *reinterpret_cast<float4*>(dst + 8 * j) = v[j];
        }
      } else if (QU == 2) {
        store_half(p.out, p.out_pitch, p.relu != 0, m, cbase, h, v[0], v[1], res_raw[u % UN], p.res != nullptr);
      } else {
        store_quad(p, m, cbase, h, v[0], res_raw[u % UN]);
      }
    }
  asm volatile("" ::"v"(touched[0]), "v"(touched[1]), "v"(touched[2]), "v"(touched[3]));
}
// =============================================================================================
// 3x3 stride-2 pad-1 layers with the block's 1x1 stride-2 projection riding along: k_conv3x3_run's tiles, K splits and
// loads.  What differs:
//   - An output pixel needs four input pixels.  A patch row holds its even pixels first, then the odd ones, so that the
//     lanes of a tap read neighbours; rows are padded so that the next output row (two patch rows further) goes on in the
//     next bank group.
//   - The K loop goes by items of 16 * KS input channels (a chunk, or half of one): every wavefront takes one K-step per
//     tap and item, and one of the projection's, whose pixels are the centre tap's and whose sums are accumulators of
//     their own.  The 64-channel layer's single chunk is one item of four K splits or two of two.
// Per output and K split: item, tap; then the splits in pairs.
// Against the kernels it replaced (4 x 8-pixel tiles with the splits chunk by chunk; 8 x 8 x 128 tiles on large grids), us
// for the layers of 128 / 256 / 512 channels: one 288 x 160 frame 6.0 / 6.7 / 7.8 -> 4.5 / 5.3 / 6.5, one 854 x 480 frame 8.0
// / 8.0 / 8.4 -> 6.9 / 6.6 / 6.9, four 641 x 361 frames 15.9 / 12.3 / 12.9 -> 12.0 / 8.7 / 12.6, sixteen 416 x 240 frames
// 17.7 / 13.9 / 14.0 -> 15.1 / 12.3 / 12.1, twelve 854 x 480 frames 30.9 / 27.6 / 28.8 -> (k_conv3x3s2_dira) / 26.9 / 24.8.
// =============================================================================================
template <int PG, int KS, int CW, int BD, int PL, int LDS, int OCC>
__global__ __launch_bounds__(64 * KS * CW, OCC) void k_conv3x3s2_run(RunParams p) {
  constexpr int NW = KS * CW, C = 32 * CW, VP = 2 * KS, U = VP + 1, PITCH = 8 * U;   // 16-byte vectors, LDS units per pixel
  constexpr int UNITS = 4 * PG;                                    // pieces of 16 channels x 32 pixels, the projection's too
  constexpr int UP = UNITS * NW * 2048 <= 2 * LDS || UNITS * NW * 2048 <= 65536 ? UNITS : UNITS / 2, PASSES = UNITS / UP, UN = UP / KS;
  static_assert(UP % KS == 0, "every K split finishes the same number of pieces");
  constexpr int RED = UP * NW * 2048, SHM = RED > 2 * LDS ? RED : 2 * LDS;
  __shared__ __align__(16) unsigned char s_raw[SHM];
  f16* const s_patch = reinterpret_cast<f16*>(s_raw);

  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave % KS, cw = wave / KS;
  // the parameters of the prologue, all in one round trip
  asm volatile("" ::"s"(p.in), "s"(p.wt_frag), "s"(p.run_in_bytes), "s"(p.run_w_bytes), "s"(p.cin_pitch), "s"(p.chunks_per_tap),
               "s"(p.tiles_per_xcd), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.n_block), "s"(p.run_by_blk), "s"(p.run_nb_shift),
               "s"(p.run.strip_w), "s"(p.run.rows), "s"(p.run.h), "s"(p.run.w), "s"(p.run.by_strip_w), "s"(p.run.by_h),
               "s"(p.run.by_batch), "s"(p.run.by23_row), "s"(p.wt2_frag), "s"(p.run.pitch2), "s"(p.run.by_period), "s"(p.run.hin));
  const uint32_t tile = (blockIdx.x & 7u) * (uint32_t)p.tiles_per_xcd + (blockIdx.x >> 3);
  const RunTile rt = run_tile(tile, p.tiles_m, p.tiles_n, p.n_block, p.run_nb_shift, p.run_by_blk);   // tile order: see above
  const int n0 = (int)rt.channels * C;
  const RunOrigin org = run_origin(p.run, rt.run);
  const int rw = 2 * p.run.strip_w + 1, rp = p.run.pitch2, odd = (p.run.strip_w + 1) * PITCH;   // odd: offset of a row's odd pixels

  const BufferRsrc in_buf = buffer_of(p.in, p.run_in_bytes), w_buf = buffer_of(p.wt_frag, p.run_w_bytes),
                   w2_buf = buffer_of(p.wt2_frag, p.run_w_bytes / 9);
  u32x4 first[PL];
  // ---- patch loader, as in k_conv3x3_run
  int l_poff[PL], l_lds[PL];
  {
    const uint32_t pix = (uint32_t)tid / VP;
    const int v = (tid % VP) * 8;
    uint32_t prow = run_div23(pix, p.run.by23_row), pcol = pix - prow * (uint32_t)rw;
#pragma unroll
    for (int i = 0; i < PL; ++i) {
      int m;
      const bool fits = prow < (uint32_t)p.run.rows, in = run2_patch_pixel(p.run, org, prow, pcol, m) && fits;
      l_poff[i] = in ? (m * p.cin_pitch + v) * 2 : kOutside;
      l_lds[i] = fits ? (int)prow * rp + (int)(pcol >> 1) * PITCH + (pcol & 1u ? odd : 0) + v : LDS / 2 - 64 + v;
      first[i] = load16(in_buf, l_poff[i], 0);
      prow += (uint32_t)p.run.step_q;
      pcol += (uint32_t)p.run.step_r;
      if (pcol >= (uint32_t)rw) { pcol -= (uint32_t)rw; ++prow; }
    }
  }
  u32x4 st_p[PL];
#define HS_LOAD_P(I_, IT_) st_p[I_] = load16(in_buf, l_poff[I_], (IT_) * (VP * 16));
#define HS_HAND_P(V_, I_, B_) *reinterpret_cast<u32x4*>(&s_patch[(B_) * (LDS / 2) + l_lds[I_]]) = (V_);

  // An item is VP * 8 input channels: a chunk, or half of one.  Its K-steps are the KS splits': a wavefront takes one per
  // tap, and one for the projection (on the centre tap's pixels).  n_it items, in pairs; a single one comes second.
  const int n_it = p.chunks_per_tap * (4 / KS), single = n_it & 1;
  constexpr int WI = KS == 4 ? 36 * 1024 : 2 * 1024, WI2 = KS == 4 ? 4 * 1024 : 2 * 1024;   // bytes from item to item of a pair
  constexpr int WP = 36 * 1024 * KS / 2, WP2 = 4 * 1024 * KS / 2;                           // and from pair to pair
  int wf = (n0 / 32 + cw) * p.chunks_per_tap * 36 * 1024 + ks * 1024 - single * WI;
  int wf2 = (n0 / 32 + cw) * p.chunks_per_tap * 4 * 1024 + ks * 1024 - single * WI2;
#pragma unroll
  for (int i = 0; i < PL; ++i) HS_LOAD_P(i, min(1, n_it - 1))
  u32x4 fa[9], fb;
#pragma unroll
  for (int t = 0; t < 9; ++t) fa[t] = load16(w_buf, lane * 16, wf + single * WI + t * 4096);
  fb = load16(w2_buf, lane * 16, wf2 + single * WI2);
  int fpo[PG], o_m[PG];
#pragma unroll
  for (int g = 0; g < PG; ++g) {
    uint32_t row, col;
    run2_pixel(p.run, org, 32 * g + r, row, col, o_m[g]);
    fpo[g] = (int)row * rp + (int)col * PITCH + h * 8 + ks * 16;
  }
  // (Only here: an exit further up would split the loads of the parameters into several round trips.  Beyond the last tile all
  // of the above is the last tile's.)
  if (tile >= (uint32_t)(p.tiles_m * p.tiles_n)) return;
#pragma unroll
  for (int i = 0; i < PL; ++i) HS_HAND_P(first[i], i, single)
  __syncthreads();

  const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  floatx16 acc[2][PG];                                             // the layer's, the projection's
#pragma unroll
  for (int g = 0; g < PG; ++g) acc[0][g] = acc[1][g] = zero16;
  // Pixel fragment F_ = K-step * PG + group of an item; K-step 4 is the centre tap, which the projection shares
  half8 bf[BD + 1];
#define HS_READ_B(U_, F_)                                                                      \
  bf[(F_) % (BD + 1)] = *reinterpret_cast<const half8*>(                                       \
      &s_patch[(U_) * (LDS / 2) + fpo[(F_) % PG] + ((F_) / PG / 3) * rp + (((F_) / PG) % 3 == 1 ? odd : ((F_) / PG) % 3 / 2 * PITCH)]);
#define HS_ITEM(U_, LAST_)                                                                     \
  {                                                                                            \
    _Pragma("unroll") for (int f = 0; f < BD; ++f) HS_READ_B(U_, f)                            \
    _Pragma("unroll") for (int s = 0; s < 9; ++s) {                                            \
      _Pragma("unroll") for (int i = 0; i < PL; ++i)                                           \
        if ((2 * i + 1) * 9 / (2 * PL) == s && (!(LAST_) || (U_) == 0)) {                      \
          HS_HAND_P(st_p[i], i, 1 - (U_))                                                      \
          if (!(LAST_)) HS_LOAD_P(i, min(it + (U_) + 2, n_it - 1))                             \
        }                                                                                      \
      _Pragma("unroll") for (int g = 0; g < PG; ++g) {                                         \
        if (s * PG + g + BD < 9 * PG) HS_READ_B(U_, s * PG + g + BD)                           \
        const half8 b_ = bf[(s * PG + g) % (BD + 1)];                                          \
        acc[0][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, fa[s]), b_, acc[0][g], 0, 0, 0); \
        if (s == 4) acc[1][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, fb), b_, acc[1][g], 0, 0, 0); \
        if (PG > 2) __builtin_amdgcn_sched_barrier(0);                                         \
      }                                                                                        \
      if (!(LAST_) || (U_) == 0) {                                                             \
        fa[s] = load16(w_buf, lane * 16, wf + ((U_) == 0 ? WI : WP) + s * 4096);               \
        if (s == 4) fb = load16(w2_buf, lane * 16, wf2 + ((U_) == 0 ? WI2 : WP2));             \
      }                                                                                        \
      __builtin_amdgcn_sched_barrier(0);                                                       \
    }                                                                                          \
  }
  int it = 0;
  for (; it + 2 < n_it; it += 2) {
    HS_ITEM(0, false)
    __syncthreads();
    HS_ITEM(1, false)
    __syncthreads();
    wf += WP;
    wf2 += WP2;
  }
  if (!single) {
    HS_ITEM(0, true)
    __syncthreads();
  }
  HS_ITEM(1, true)
#undef HS_ITEM
#undef HS_READ_B
#undef HS_HAND_P
#undef HS_LOAD_P

  uint32_t touched[kTouched] = {};
  if (p.next_lines) prefetch_next(p, (int)tile, p.tiles_m * p.tiles_n, touched);
  float4* const s_red = reinterpret_cast<float4*>(s_raw) + wave / KS * KS * UP * 128 + lane;
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    __syncthreads();                 // every wavefront is done with the patches, or with the sums of the pass before
#pragma unroll
    for (int u = 0; u < UP; ++u)
      if (u / UN != ks) {
        const floatx16& a = acc[(ps * UP + u) / (2 * PG)][(ps * UP + u) / 2 % PG];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int o = 8 * (u & 1) + 4 * j;
          s_red[(ks * UP + u) * 128 + 64 * j] = make_float4(a[o], a[o + 1], a[o + 2], a[o + 3]);
        }
      }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < UP; ++u)
      if (u / UN == ks) {
        const int w = (ps * UP + u) / (2 * PG), g = (ps * UP + u) / 2 % PG;
        const floatx16& a = acc[w][g];
        float4 v[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int o = 8 * (u & 1) + 4 * j;
          float4 b[KS];
#pragma unroll
          for (int k = 0; k < KS; ++k) {
            b[k] = make_float4(a[o], a[o + 1], a[o + 2], a[o + 3]);
            if (k != ks) b[k] = s_red[(k * UP + u) * 128 + 64 * j];
          }
#pragma unroll
          for (int d = KS / 2; d >= 1; d /= 2)                     // in pairs
#pragma unroll
            for (int k = 0; k < d; ++k) {
              b[k].x += b[k + d].x; b[k].y += b[k + d].y; b[k].z += b[k + d].z; b[k].w += b[k + d].w;
            }
          v[j] = b[0];
        }
        const int cbase = n0 + cw * 32 + 16 * (u & 1);
        const u32x4 none = {0u, 0u, 0u, 0u};
        if (w == 0) store_half(p.out, p.out_pitch, p.relu != 0, o_m[g], cbase, h, v[0], v[1], none, false);
        else store_half(p.out2, p.out2_pitch, false, o_m[g], cbase, h, v[0], v[1], none, false);   // no ReLU
      }
  }
  asm volatile("" ::"v"(touched[0]), "v"(touched[1]), "v"(touched[2]), "v"(touched[3]));
}
// The instantiations of k_conv3x3s2_run and k_conv3x3_run: the host plans for the tiles, splits and patch buffers of
// kRun2Forms and kRunForms, four wavefronts each; pixel (and weight) fragments in flight and workgroups per CU.
template <int I, int BD, int OCC>
static const void* run2_kernel() {
  constexpr Run2Form f = kRun2Forms[I];
  static_assert(f.step == f.ch && f.units == 2 * f.splits() + 1, "a patch pixel's vectors, and one more unit against bank conflicts");
  return (const void*)k_conv3x3s2_run<f.px / 32, f.splits(), f.ch / 32, BD, f.passes, f.lds, OCC>;
}
static const void* run2_kernel_of(int form) {
  switch (form) {
    case 0: return run2_kernel<0, 5, 2>();
    case 1: return run2_kernel<1, 5, 3>();
    case 2: return run2_kernel<2, 5, 2>();
    case 3: return run2_kernel<3, 5, 2>();
    case 4: return run2_kernel<4, 5, 1>();
    default: return nullptr;
  }
}
template <int I, int FR, int BD, int OCC>
static const void* run_kernel() {
  constexpr RunForm f = kRunForms[I];
  return (const void*)k_conv3x3_run<f.px / 32, f.splits(), f.ch / 32, FR, BD, f.passes, f.lds, OCC>;
}
static const void* run_kernel_of(int form) {
  switch (form) {
    case 0: return run_kernel<0, 9, 8, 3>();
    case 1: return run_kernel<1, 9, 6, 3>();
    case 2: return run_kernel<2, 9, 8, 3>();
    case 3: return run_kernel<3, 9, 4, 3>();
    case 4: return run_kernel<4, 9, 5, 2>();
    case 5: return run_kernel<5, 12, 5, 2>();
    case 6: return run_kernel<6, 9, 8, 1>();
    case 7: return run_kernel<7, 9, 5, 2>();
    default: return nullptr;
  }
}

KernelDesc describe(const ConvParams& p) {
  // 1-D grid, padded to a multiple of 8 so that every XCD owns tiles_per_xcd consecutive tiles
  const dim3 grid(8u * (unsigned)p.tiles_per_xcd);
  switch (p.variant) {
    case CONV_DIRECT: {
      const void* f = p.kc == 16 ? (p.kw_splits == 2 ? (const void*)k_conv_direct<1, 2> : (const void*)k_conv_direct<1, 1>)
                                 : (p.kw_splits == 2 ? (const void*)k_conv_direct<2, 2> : (const void*)k_conv_direct<2, 1>);
      return KernelDesc{f, grid, dim3(256), 0};
    }
    case CONV_TINY_NET:
      return KernelDesc{(const void*)k_tiny_net<false>, dim3((unsigned)(p.wout + 7) / 8, (unsigned)(p.hout + 7) / 8, (unsigned)p.batch),
                        dim3(512), 0};
    case CONV_BLOCK64: return KernelDesc{(const void*)k_block64_fused, grid, dim3(256), 0};
    case CONV_S2_DIRA: return KernelDesc{(const void*)k_conv3x3s2_dira, grid, dim3(256), 0};
    case CONV_KW:
      return KernelDesc{p.stride == 1 ? run_kernel_of(p.run_form) : run2_kernel_of(p.run_form), grid, dim3(256), 0};
    default: return KernelDesc{nullptr, grid, dim3(256), 0};
  }
}

KernelDesc describe(const TinyFrameParams& p) {
  return KernelDesc{(const void*)k_tiny_net<true>, dim3((unsigned)(p.wout + 7) / 8, (unsigned)(p.hout + 7) / 8, (unsigned)p.r.batch), dim3(512), 0};
}

// ---------------------------------------------------------------------------------------------
// ConvLSTM epilogue + 1x1 head: one workgroup per pixel, one thread per hidden channel
// (hid == 256).  Gates and state update in fp32 (c kept in fp32, h stored fp16); the head's
// eight logits of the pixel are the workgroup-wide sums of w[k][j] * h[j] over the stored
// (fp16) h: a wavefront butterfly, then the four wavefront sums in order.
// logits: planar per image, logits[(image*8 + k)*img_m + pixel in image].
// The eight threads that hold a pixel's logits also finish the part of stage 3 that needs no other
// pixel: heat map, mask and the overlay's channel map.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_lstm_epilogue(LstmEpilogueParams p) {
  __shared__ float s_part[4][8];
  const int m = blockIdx.x, j = threadIdx.x, lane = j & 63, wave = j >> 6;
  const size_t t = (size_t)m * p.hid + j;
  const int n4 = 4 * p.hid;
  float g[4] = {0.f, 0.f, 0.f, 0.f};
  const float* row = p.partial + (size_t)m * n4;
#pragma unroll
  for (int k = 0; k < 4; ++k) g[k] += row[k * p.hid + j];
  const float gi = sigmoid_f(g[0]), gf = sigmoid_f(g[1]), gg = tanhf(g[2]), go = sigmoid_f(g[3]);
  const float c_new = gf * p.c[t] + gi * gg;
  p.c[t] = c_new;
  const f16 h16 = (f16)(go * tanhf(c_new));
  p.h_out[(size_t)m * p.h_pitch + j] = h16;

  const float hv = (float)h16;
  float v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = hv * (float)p.w_head[k * p.hid + j];
  // Wavefront sums of the eight products by a halving butterfly: at offset 32 a lane keeps four
  // of the eight (k / 4 == its bit 5) and hands the other four to its partner in the same
  // exchange, at 16 two, at 8 one; offsets 4, 2, 1 finish that one.  Ten exchanges instead of
  // 48, and every sum adds the same pairs level by level as the full butterfly would: lanes
  // 8 * k .. 8 * k + 7 end with the sum of product k.
  float a4[4], a2[2], a1;
  {
    const bool up = (lane & 32) != 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      a4[i] = (up ? v[4 + i] : v[i]) + __shfl_xor(up ? v[i] : v[4 + i], 32, 64);
  }
  {
    const bool up = (lane & 16) != 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      a2[i] = (up ? a4[2 + i] : a4[i]) + __shfl_xor(up ? a4[i] : a4[2 + i], 16, 64);
  }
  {
    const bool up = (lane & 8) != 0;
    a1 = (up ? a2[1] : a2[0]) + __shfl_xor(up ? a2[0] : a2[1], 8, 64);
  }
#pragma unroll
  for (int off = 4; off >= 1; off >>= 1) a1 += __shfl_xor(a1, off, 64);
  if ((lane & 7) == 0) s_part[wave][lane >> 3] = a1;
  __syncthreads();
  if (j < 8) {
    const float sum = ((s_part[0][j] + s_part[1][j]) + s_part[2][j]) + s_part[3][j];
    const int img = m / p.img_m, ml = m - img * p.img_m;
    const size_t at = ((size_t)img * 8 + j) * p.img_m + ml;
    p.logits[at] = sum;
    p.heat[at] = heat_of(sum);
    const bool set = sum > p.theta;
    p.mask[at] = set ? 1 : 0;
    const uint32_t set_channels = (uint32_t)__ballot(set) & 0xffu;
    if (j == 0) {
      p.kmap[m] = set_channels ? (uint8_t)__builtin_ctz(set_channels) : 0xff;
      if (m == p.m - 1) *p.t_end = wall_clock64();
    }
  }
}

KernelDesc describe(const LstmEpilogueParams& p) {
  return KernelDesc{(const void*)k_lstm_epilogue, dim3((unsigned)p.m), dim3(256), 0};
}

// =============================================================================================
// Stem: 7x7 stride-2 convolution (3 -> 64 channels) + ReLU + 3x3 stride-2 max-pool in one
// kernel; the 64-channel convolution output (the largest tensor of the network) never reaches
// memory.
//
// A workgroup produces 8 x 15 pooled pixels, i.e. the 17 x 31 convolution outputs under them
// (one row/column of overlap with the neighbouring tiles), as 17 row fragments of 32 pixels.
// The whole input patch (39 rows x 70 padded 4-channel pixels) sits in LDS; the weight matrix
// (64 x 224 halves, k = (ky*8 + px)*4 + ch) is held as MFMA fragments in registers.  Because the image is stored with 4
// channels per pixel, the 32 K-values of kernel row ky for convolution pixel cx are the 64
// contiguous bytes starting at input pixel 2*cx of row 2*cy + ky: MFMA pixel operands are read
// straight from the patch, no im2col copy.
// Wavefront (wm, wn): convolution rows 8*wm .. 8*wm+8 (row 8 is computed by both halves, it
// feeds pooled rows 3 and 4), channels 32*wn .. +31: nine accumulators.  Pooling: maximum over
// three accumulators (rows), then over lanes r, r+1, r+2 (columns, two DPP wavefront shifts), on
// rounded and clamped values; even lanes store.
// Twelve 854x480 frames against the same pooling in 32-bit floats: 50.8 -> 40.0 us (two boxes, whose
// other kernels differ by 7 %), one frame 8.7 -> 7.4; on one box the whole pass 710 -> 699.
// =============================================================================================
// value of lane + 1 (DPP whole-wavefront shift; lane 63 keeps its own)
__device__ __forceinline__ uint32_t lane_plus_1(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x130, 0xf, 0xf, false);
}
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef f16 half2v __attribute__((ext_vector_type(2)));
// larger of each half of two pairs of non-negative fp16 numbers
__device__ __forceinline__ uint32_t max_pairs(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, a), __builtin_bit_cast(i16x2, b)));
}

__global__ __launch_bounds__(256, 2) void k_stem_pool(StemPoolParams p) {
  constexpr int PROWS = 39, PVEC = 35, PROW_H = PVEC * 8;      // patch rows, vectors, halves per row
  constexpr int NPV = PROWS * PVEC, NPL = (NPV + 255) / 256;   // patch vectors, per thread
  __shared__ __align__(16) f16 s_patch[PROWS * PROW_H];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 31, h = lane >> 5;
  const int tile = (int)(blockIdx.x & 7u) * p.tiles_per_xcd + (int)(blockIdx.x >> 3);
  if (tile >= p.batch * p.tiles_y * p.tiles_x) return;
  const int tx = tile % p.tiles_x, ty = (tile / p.tiles_x) % p.tiles_y;
  const int img = tile / (p.tiles_x * p.tiles_y);
  const int p0 = 8 * ty, q0 = 15 * tx;              // first pooled pixel
  const int cy0 = 2 * p0 - 1, cx0 = 2 * q0 - 1;     // first convolution pixel
  const int iy0 = 2 * cy0, ix0 = 2 * cx0;           // first pixel of the padded image (may be < 0)

  // ---- fill LDS: unconditional loads from clamped addresses, zeros where out of the image
  u32x4 st_p[NPL];
  bool inb[NPL];
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    const int v = min(tid + 256 * i, NPV - 1);
    const int ly = v / PVEC, lv = v - ly * PVEC;
    const int y = iy0 + ly, x = ix0 + 2 * lv;
    inb[i] = y >= 0 && y < p.hin && x >= 0 && x < p.win;
    const f16* src = inb[i] ? p.in + (((size_t)img * p.hin + y) * p.win + x) * 4 : p.in;
    st_p[i] = *reinterpret_cast<const u32x4*>(src);
  }
  // The wavefront's 14 weight fragments come straight from memory (fragment order, one
  // contiguous 1 KB block per wavefront load) and stay in registers.
  const int wm = wave & 1, wn = wave >> 1;
  half8 a[7][2];
  {
    const half8* wfr = reinterpret_cast<const half8*>(p.wt) + (size_t)wn * 14 * 64 + lane;
#pragma unroll
    for (int ky = 0; ky < 7; ++ky)
#pragma unroll
      for (int s = 0; s < 2; ++s) a[ky][s] = wfr[(ky * 2 + s) * 64];
  }
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    const int v = tid + 256 * i;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    if (v < NPV) *reinterpret_cast<u32x4*>(&s_patch[v * 8]) = inb[i] ? st_p[i] : zero;
  }
  __syncthreads();

  // ---- 14 K-steps of 16 (two per kernel row), nine row fragments each
  floatx16 acc[9];
#pragma unroll
  for (int j = 0; j < 9; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0.0f;
  const f16* fp = &s_patch[(16 * wm) * PROW_H + r * 8 + h * 8];   // patch row 2*(8*wm + j) + ky
  // Patch row rho serves every (convolution row j, kernel row ky) with 2*j + ky == rho, so each
  // patch fragment is read once: 46 LDS reads feed the 126 MFMAs.  Per accumulator the K order
  // stays ky = 0..6.
#pragma unroll
  for (int rho = 0; rho < 23; ++rho) {
    if (rho % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // bounds how far reads are hoisted
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const half8 b = *reinterpret_cast<const half8*>(fp + rho * PROW_H + s * 16);
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const int ky = rho - 2 * j;
        if (ky >= 0 && ky <= 6)
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ky < 0 ? 0 : ky > 6 ? 6 : ky][s], b,
                                                         acc[j], 0, 0, 0);
      }
    }
  }

  // ---- ReLU, pool.  Rounding to fp16, ReLU and the maximum commute, so the accumulators are rounded
  // and clamped first, two values per instruction; ReLU also turns a NaN into 0, and what is left
  // is ordered like its bits, so the maxima are 16-bit integer ones (a float maximum costs a second
  // instruction per operand to quieten a NaN that the compiler cannot rule out: of the 850 vector
  // instructions of this part in 32-bit floats 370 are left).  A pooling window always holds its centre row
  // (convolution row 2 * py exists whenever pooled row py does), rows outside the convolution
  // output are skipped (the same for the whole wavefront), columns outside it count as 0, which
  // cannot change the maximum.  Then the lane pair (r, r + 32) exchanges quads and stores 16 bytes
  // per lane (store_quads_to); every lane takes part in the exchange.
  const int cx = cx0 + r;
  const uint32_t col_mask = cx >= 0 && cx < p.wc ? 0xffffffffu : 0u;
  const int q = q0 + (r >> 1);
  const bool writer = (r & 1) == 0 && r <= 28 && q < p.wp;
  i16x2 y[9][8];
#pragma unroll
  for (int j = 0; j < 9; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const half2v t = {(f16)acc[j][2 * i], (f16)acc[j][2 * i + 1]}, zero = {(f16)0.0f, (f16)0.0f};
      y[j][i] = __builtin_bit_cast(i16x2, __builtin_elementwise_max(t, zero));
    }
#pragma unroll
  for (int pl = 0; pl < 4; ++pl) {
    const int py = p0 + 4 * wm + pl;
    const int cy_top = cy0 + 8 * wm + 2 * pl;             // rows cy_top, cy_top + 1 (centre), cy_top + 2
    const bool top_ok = cy_top >= 0, bot_ok = cy_top + 2 < p.hc;
    i16x2 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = y[2 * pl + 1][i];
    if (top_ok) {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = __builtin_elementwise_max(v[i], y[2 * pl][i]);
    }
    if (bot_ok) {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = __builtin_elementwise_max(v[i], y[2 * pl + 2][i]);
    }
    uint32_t o[4][2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t m = __builtin_bit_cast(uint32_t, v[i]) & col_mask;
      const uint32_t m2 = max_pairs(m, lane_plus_1(m));        // columns r, r+1
      o[i >> 1][i & 1] = max_pairs(m2, lane_plus_1(m2));       // columns r .. r+2
    }
    store_quads_to(p.out, 64, writer && py < p.hp, (img * p.hp + py) * p.wp + q, 32 * wn, h, o);
  }
}

KernelDesc describe(const StemPoolParams& p) {
  return KernelDesc{(const void*)k_stem_pool, dim3(8u * (unsigned)p.tiles_per_xcd), dim3(256), 0};
}

// =============================================================================================
// Stage 3's channel maxima: maximum, its lowest index, presence -- one workgroup per tool channel;
// every lane keeps (best value, lowest index), a wavefront butterfly, then one more across the 4
// wavefronts through LDS.  The integer outputs are decided on the logits with exact comparisons.
// Where nothing else waits for the maxima, their workgroups ride along in the overlay's launch
// (k_overlay) instead of a launch of their own.
// =============================================================================================
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
  return v > bv || (v == bv && i < bi);
}

// Maximum of channel k of one image (logits L[0 .. n-1]) into the host-visible record; every thread of
// a 256-thread workgroup.  Thread 0 returns it in bv, bi.
__device__ __forceinline__ void channel_maximum(const float* L, int n, float theta, int k, PostRecord* rec,
                                                float& bv, int& bi) {
  __shared__ float s_v[4];
  __shared__ int s_i[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  bv = -INFINITY;
  bi = 0x7fffffff;
  for (int i = tid; i < n; i += 256) {
    const float x = L[i];
    if (better(x, i, bv, bi)) { bv = x; bi = i; }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const float ov = __shfl_xor(bv, off, 64);
    const int oi = __shfl_xor(bi, off, 64);
    if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
  }
  if (lane == 0) { s_v[wave] = bv; s_i[wave] = bi; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 4; ++w)
      if (better(s_v[w], s_i[w], bv, bi)) { bv = s_v[w]; bi = s_i[w]; }
    rec->argmax_idx[k] = bi;
    rec->peak[k] = heat_of(bv);
    rec->present[k] = bv > theta ? 1 : 0;
  }
}

__global__ __launch_bounds__(256) void k_postprocess(PostParams p) {
  const int k = blockIdx.x, img = blockIdx.y;
  float bv;
  int bi;
  channel_maximum(p.logits + ((size_t)img * 8 + k) * p.n, p.n, p.theta, k, p.rec + img, bv, bi);
  if (threadIdx.x == 0 && p.marks) {
    // anchor of the annotation layer: centre of the argmax cell's footprint in the frame
    int* const mk = p.marks + ((size_t)img * 8 + k) * 2;
    const int ay = bi / p.wm, ax = bi - ay * p.wm;
    mk[0] = bv > p.theta ? ((2 * ax + 1) * p.wf) / (2 * p.wm) : -1;
    mk[1] = bv > p.theta ? ((2 * ay + 1) * p.hf) / (2 * p.hm) : -1;
  }
  if (threadIdx.x == 0 && k == 7 && img == p.batch - 1) *p.t_end = wall_clock64();
}

KernelDesc describe(const PostParams& p) {
  return KernelDesc{(const void*)k_postprocess, dim3(8, p.batch), dim3(256), 0};
}

// =============================================================================================
// Stage 4: pure streaming, one read and one write of the frame, in two forms.
//
// Groups of 16 pixels (FINE == false).  A thread owns 48 bytes, three 16-byte accesses, of one frame
// row; groups are numbered row-major over the frame, 256 per workgroup, so there is no per-row
// prologue and no barrier.  A group sees at most two cells of the channel map (the host takes this
// form only then): both are fetched up front together with the pixels.  A wavefront moves the 192
// vectors of its 64 groups as consecutive 16-byte accesses and regroups them through LDS, instead
// of every lane touching its own 48-byte span.  The last group of a row may hang over the row's
// end: vectors that start beyond the pitch are not fetched, and of a vector that holds the end of
// the pixels only their bytes are stored, so the padding between rows stays what it was.  (Those
// groups used to go pixel by pixel: one such lane held up its wavefront for 45 byte loads, 54 us
// instead of 11 for four 1279 x 719 frames with annotations.)
//
// Quads of 4 pixels (FINE == true).  A thread owns 12 bytes, which a wavefront reads and writes as
// one run of 768, and fetches the channel byte of each pixel: any number of cells.  What bounds a
// small frame is the chain of instructions of one thread, on a chip that it does not fill, so four
// times the threads with a third of the chain each.
//
// Workgroup 0 of an image hands the host the stages' ends, the next n_max find stage 3's channel maxima (see
// channel_maximum).
// =============================================================================================
// 0xffffffff where the condition holds, else 0.
__device__ __forceinline__ uint32_t mask_of(bool c) { return c ? 0xffffffffu : 0u; }
// Bits of a where m is set, else of b.
__device__ __forceinline__ uint32_t pick_bits(uint32_t m, uint32_t a, uint32_t b) { return (a & m) | (b & ~m); }

// Colour of channel k (0..7).  A select chain over the eight scalar palette words: indexing the
// kernel-argument array with a per-lane k would be a vector load from memory, one more full
// memory latency between the channel byte and the blend.
__device__ __forceinline__ uint32_t overlay_colour(const OverlayLayer& L, uint32_t k) {
  uint32_t c = L.pal[0];
#pragma unroll
  for (uint32_t i = 1; i < 8; ++i) c = k == i ? L.pal[i] : c;
  return c;
}

// Where the annotation layer of L may draw on N pixels starting at (X0, Y), held as words w (N = 4 or 16; word j starts with
// channel j mod 3).  A tool's drawing lies in one box; a wavefront visits only the tools whose box some lane meets, tools in
// increasing order (later tools paint over earlier ones).  Lane i of every 16 fetches word i of the eight anchors: one memory
// latency, and the loop reads them as scalars.  What a tool paints is a bit per pixel, spread to the bytes' masks.
template <int N>
__device__ __forceinline__ void overlay_marks(const OverlayLayer& L, uint32_t (&w)[3 * N / 4], int Y, int X0, int by) {
  const int anchors = L.marks[(size_t)by * 16 + (threadIdx.x & 15)];
  const int lab_w = 11 * L.scale, lab_h = 7 * L.scale;
  // the cross-hair's bars are 2 * arm + 1 long and 2 * half + 1 thick; either may be the larger.  The
  // label reaches further to the right than a bar (13 pixels past arm at least, half is at most 8)
  const int ext = max(L.arm, L.half);
#pragma unroll 1
  for (int k = 0; k < 8; ++k) {
    const int cx = __builtin_amdgcn_readlane(anchors, 2 * k), cy = __builtin_amdgcn_readlane(anchors, 2 * k + 1);
    if (cx < 0) continue;
    const int ox = cx + L.arm + 2, oy = cy - lab_h - 2;          // label origin
    const bool met = Y >= min(cy - ext, oy) && Y <= cy + ext && X0 + N - 1 >= cx - ext && X0 < ox + lab_w;
    if (!__any((int)met)) continue;
    // |X - cx| <= reach: the wider of the two bars where the row meets both (-1: it meets neither)
    const int dy = abs(Y - cy), reach = max(dy <= L.half ? L.arm : -1, dy <= L.arm ? L.half : -1);
    uint32_t m[N];
#pragma unroll
    for (int i = 0; i < N; ++i) m[i] = mask_of(abs(X0 + i - cx) <= reach);
    const bool label = Y >= oy && Y < oy + lab_h;
    if (__any((int)label)) {
      // this row's glyph cells as bits, cell 11 empty: what lies outside the label's pixels 0 .. lab_w - 1 takes that one.
      // Pixel to cell: floor(x / scale) = x * ceil(65536 / scale) >> 16 for x <= 88, scale <= 8 (the excess x * scale / 65536
      // stays below 1 / scale)
      const uint32_t inv = (65536u + (uint32_t)L.scale - 1u) / (uint32_t)L.scale;
      const int gy = (int)(mul24((uint32_t)max(0, min(Y - oy, lab_h - 1)), inv) >> 16);
      const uint32_t row = (uint32_t)(L.glyph[0] >> (5 * gy)) & 31u, row_k = (uint32_t)(L.glyph[1 + k] >> (5 * gy)) & 31u;
      const uint32_t cells = label ? row | row_k << 6 : 0u;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const uint32_t lx = min((uint32_t)(X0 + i - ox), (uint32_t)lab_w);
        m[i] |= 0u - (cells >> (mul24(lx, inv) >> 16) & 1u);
      }
    }
    const uint32_t col = L.pal[k], r = col & 0xffu, g = (col >> 8) & 0xffu, b = (col >> 16) & 0xffu;
    const uint32_t c[3] = {r | g << 8 | b << 16 | r << 24, g | b << 8 | r << 16 | g << 24, b | r << 8 | g << 16 | b << 24};
#pragma unroll
    for (int q = 0; q < N / 4; ++q) {                            // four pixels are three words
      w[3 * q] = pick_bits(pick_bits(0x00ffffffu, m[4 * q], m[4 * q + 1]), c[0], w[3 * q]);
      w[3 * q + 1] = pick_bits(pick_bits(0x0000ffffu, m[4 * q + 1], m[4 * q + 2]), c[1], w[3 * q + 1]);
      w[3 * q + 2] = pick_bits(pick_bits(0x000000ffu, m[4 * q + 2], m[4 * q + 3]), c[2], w[3 * q + 2]);
    }
  }
}

// The channel-map cells a group of 16 pixels starting at (X0, Y) sees in layer L: its first
// cell, and the two channel bytes.
struct OverlayCells {
  int mx0;
  uint8_t k0, k1;
};
template <int NL>
__device__ __forceinline__ const uint8_t* overlay_map_row(const OverlayParamsOf<NL>& p, const OverlayLayer& L, int Y, int by) {
  const int my = (int)udiv_est((uint32_t)(Y * L.hm), (uint32_t)p.hf, p.rcp_hf);
  return L.kmap + ((size_t)by * L.hm + my) * L.wm;
}
template <int NL>
__device__ __forceinline__ OverlayCells overlay_cells(const OverlayParamsOf<NL>& p, const OverlayLayer& L,
                                                      int Y, int X0, int by) {
  OverlayCells c;
  const uint8_t* const krow = overlay_map_row(p, L, Y, by);
  c.mx0 = (int)udiv_est((uint32_t)(X0 * L.wm), (uint32_t)p.wf, p.rcp_wf);
  c.k0 = krow[c.mx0];
  c.k1 = krow[min(c.mx0 + 1, L.wm - 1)];
  return c;
}

// One layer of stage 4 applied to a group of 16 pixels held in registers (w[0..11], word j starts
// with channel j mod 3): blend of the layer's channel map, then its annotations.
template <int NL>
__device__ __forceinline__ void overlay_layer_group(const OverlayParamsOf<NL>& p, const OverlayLayer& L,
                                                    const OverlayCells& cells, uint32_t (&w)[12],
                                                    int Y, int X0, int by) {
  const int ia = 256 - L.a;
  const int mx0 = cells.mx0;
  const uint8_t k0 = cells.k0, k1 = cells.k1;
  // Most groups see one channel for all 16 pixels: nothing to draw, or one colour.  Then the
  // blend runs on two bytes per 32-bit operation: even and odd bytes of a word are 16-bit
  // fields, (256 - a) * byte + (a * colour + 128) never exceeds 65408, so no field carries into
  // its neighbour.  The field pair is below 2^24 and the factor at most 256: 24-bit multiplies
  // (full rate; the 32-bit ones run at a quarter of it) are exact.
  const int mx_last = (int)udiv_est((uint32_t)(min(X0 + 15, p.wf - 1) * L.wm), (uint32_t)p.wf, p.rcp_wf);
  if (mx_last == mx0 || k1 == k0) {
    if (k0 != 0xff) {
      const uint32_t col = overlay_colour(L, k0);
      uint32_t t[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) t[c] = mad24((uint32_t)L.a, (col >> (8 * c)) & 0xffu, 128u);
#pragma unroll
      for (int j = 0; j < 12; ++j) {
        const uint32_t ce = t[j % 3] | (t[(j + 2) % 3] << 16);        // bytes 0 and 2
        const uint32_t co = t[(j + 1) % 3] | (t[(j + 3) % 3] << 16);  // bytes 1 and 3
        const uint32_t e = w[j] & 0x00ff00ffu, o = (w[j] >> 8) & 0x00ff00ffu;
        w[j] = ((mad24(e, (uint32_t)ia, ce) >> 8) & 0x00ff00ffu) |
               (mad24(o, (uint32_t)ia, co) & 0xff00ff00u);
      }
    }
  } else {
    // two cells: pixels [0, s) see k0, [s, 16) see k1.  Same packed blend with the colour
    // term chosen per byte (byte index < 3*s), then bytes of an undrawn cell are restored.
    const int rem = X0 * L.wm - mx0 * p.wf;
    const int s3 = 3 * (int)udiv_est((uint32_t)(p.wf - rem + L.wm - 1), (uint32_t)L.wm, L.rcp_wm);
    const uint32_t c0 = k0 != 0xff ? overlay_colour(L, k0) : 0u;
    const uint32_t c1 = k1 != 0xff ? overlay_colour(L, k1) : 0u;
    const uint32_t d0 = k0 != 0xff ? 0xffffffffu : 0u, d1 = k1 != 0xff ? 0xffffffffu : 0u;
    uint32_t t0[3], t1[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      t0[c] = mad24((uint32_t)L.a, (c0 >> (8 * c)) & 0xffu, 128u);
      t1[c] = mad24((uint32_t)L.a, (c1 >> (8 * c)) & 0xffu, 128u);
    }
#pragma unroll
    for (int j = 0; j < 12; ++j) {
      const uint32_t tb0 = 4 * j + 0 < s3 ? t0[j % 3] : t1[j % 3];
      const uint32_t tb1 = 4 * j + 1 < s3 ? t0[(j + 1) % 3] : t1[(j + 1) % 3];
      const uint32_t tb2 = 4 * j + 2 < s3 ? t0[(j + 2) % 3] : t1[(j + 2) % 3];
      const uint32_t tb3 = 4 * j + 3 < s3 ? t0[(j + 3) % 3] : t1[(j + 3) % 3];
      const uint32_t e = w[j] & 0x00ff00ffu, o = (w[j] >> 8) & 0x00ff00ffu;
      const uint32_t blended = ((mad24(e, (uint32_t)ia, tb0 | (tb2 << 16)) >> 8) & 0x00ff00ffu) |
                               (mad24(o, (uint32_t)ia, tb1 | (tb3 << 16)) & 0xff00ff00u);
      const int nb = min(4, max(0, s3 - 4 * j));                    // leading bytes of cell 0
      const uint32_t low = nb == 4 ? 0xffffffffu : ((1u << (8 * nb)) - 1u);
      const uint32_t draw = (low & d0) | (~low & d1);
      w[j] = (blended & draw) | (w[j] & ~draw);
    }
  }
  if (L.marks) overlay_marks<16>(L, w, Y, X0, by);
}

// The channel bytes of a quad of pixels starting at (X0, Y) in layer L, pixel i in byte i (0xff: nothing to draw).
template <int NL>
__device__ __forceinline__ uint32_t overlay_quad_cells(const OverlayParamsOf<NL>& p, const OverlayLayer& L, int Y, int X0, int by) {
  const uint8_t* const krow = overlay_map_row(p, L, Y, by);
  uint32_t k[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) k[i] = krow[udiv_est((uint32_t)(min(X0 + i, p.wf - 1) * L.wm), (uint32_t)p.wf, p.rcp_wf)];
  return k[0] | k[1] << 8 | k[2] << 16 | k[3] << 24;
}
// One layer of stage 4 applied to a quad (three words): the same packed blend, every pixel with its own colour terms
// (a * colour + 128; terms[k] = {red, green in the upper half}, {blue}), then the bytes of undrawn pixels are restored.
__device__ __forceinline__ void overlay_layer_quad(const OverlayLayer& L, const uint2* terms, uint32_t cells, uint32_t (&w)[3],
                                                   int Y, int X0, int by) {
  if (__any((int)(cells != 0xffffffffu))) {
    const uint32_t ia = 256u - (uint32_t)L.a;
    uint2 t[4];
    uint32_t d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t k = (cells >> (8 * i)) & 0xffu;
      d[i] = mask_of(k != 0xffu);
      t[i] = terms[k & 7u];
    }
    // bytes: r0 g0 b0 r1 | g1 b1 r2 g2 | b2 r3 g3 b3; the terms of bytes 0 and 2, of bytes 1 and 3
    const uint32_t te[3] = {(t[0].x & 0xffffu) | t[0].y << 16, t[1].x >> 16 | t[2].x << 16, t[2].y | (t[3].x & 0xffff0000u)};
    const uint32_t to[3] = {t[0].x >> 16 | t[1].x << 16, t[1].y | (t[2].x & 0xffff0000u), (t[3].x & 0xffffu) | t[3].y << 16};
    const uint32_t draw[3] = {pick_bits(0x00ffffffu, d[0], d[1]), pick_bits(0x0000ffffu, d[1], d[2]),
                              pick_bits(0x000000ffu, d[2], d[3])};
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const uint32_t e = w[j] & 0x00ff00ffu, o = (w[j] >> 8) & 0x00ff00ffu;
      const uint32_t blended = ((mad24(e, ia, te[j]) >> 8) & 0x00ff00ffu) | (mad24(o, ia, to[j]) & 0xff00ff00u);
      w[j] = pick_bits(draw[j], blended, w[j]);
    }
  }
  if (L.marks) overlay_marks<4>(L, w, Y, X0, by);
}

// LAYERS == false: exactly one layer (every single-network application).  LAYERS == true: the
// n_layers layers of a multi-network application are applied in order, each on the result of
// the one before, while the pixels sit in registers (one read and one write of the frame).
template <bool LAYERS, bool FINE>
__global__ __launch_bounds__(256) void k_overlay(OverlayParamsOf<LAYERS ? kMaxLayers : 1> p) {
  const int by = (int)blockIdx.y;                                // image of the batch
  const int nl = LAYERS ? p.n_layers : 1;
  const int b = (int)blockIdx.x - 1;
  if (b < 0) {                                                   // (first, so that its stores to the host end beside the drawing)
    const int l = (int)threadIdx.x;
    if (by == 0 && l < nl && p.layer[LAYERS ? l : 0].stamps) {
      const OverlayLayer& L = p.layer[LAYERS ? l : 0];
      L.stamps->pre = L.t_stages[0];
      L.stamps->infer = L.t_stages[1];
      L.stamps->post = L.t_stages[2];
    }
    return;
  }
  if (b < p.n_max) {                                             // eight workgroups per layer
    const OverlayLayer& L = p.layer[LAYERS ? b >> 3 : 0];
    const int k = b & 7, n = L.wm * L.hm;
    if (!L.rec) return;
    const uint64_t t_stage2 = L.t_stages[1];
    float bv;
    int bi;
    channel_maximum(L.logits + ((size_t)by * 8 + k) * n, n, L.theta, k, L.rec + by, bv, bi);
    if (threadIdx.x == 0) L.rec[by].ticks[k] = (int32_t)(wall_clock64() - t_stage2);
    return;
  }
  const uint8_t* const src = p.src[by];
  uint8_t* const dst = p.dst[by];
  // The launch's end as its last workgroup sees it, noted ahead of the pixels' stores, whose way to memory hides the
  // stamp's to the host.  (Behind them it puts 1.8 us on a frame.)
  auto stamp_end = [&] {
    if (p.stamp_end && blockIdx.x == gridDim.x - 1 && by == p.batch - 1 && (int)threadIdx.x < nl) {
      StageStamps* const st = p.layer[LAYERS ? threadIdx.x : 0].stamps;
      if (st) st->drawn = wall_clock64();
    }
  };
  if constexpr (FINE) {
    __shared__ uint2 s_terms[LAYERS ? kMaxLayers : 1][8];
    const int qpr = (p.wf + 3) >> 2, total = qpr * p.hf;         // quads per row, of the frame
    const int q_own = (b - p.n_max) * 256 + (int)threadIdx.x, q = min(q_own, total - 1);
    const int Y = (int)udiv_est((uint32_t)q, (uint32_t)qpr, p.rcp_qpr), X0 = (q - Y * qpr) * 4;
    const size_t at = (size_t)Y * p.pitch + (size_t)X0 * 3;
    const int bytes = min(12, 3 * (p.wf - X0));                  // of the quad that are pixels
    uint32_t cells[LAYERS ? kMaxLayers : 1];
    cells[0] = overlay_quad_cells(p, p.layer[0], Y, X0, by);
    uint32_t w[3];
    if (bytes == 12) {
      const u32x3 v = *reinterpret_cast<const u32x3*>(src + at);
      w[0] = v[0]; w[1] = v[1]; w[2] = v[2];
    } else {                                                     // words that hold pixels lie inside the row's pitch
#pragma unroll
      for (int j = 0; j < 3; ++j) w[j] = 4 * j < bytes ? *reinterpret_cast<const uint32_t*>(src + at + 4 * j) : 0u;
    }
    if constexpr (LAYERS) {
#pragma unroll
      for (int l = 1; l < kMaxLayers; ++l)
        if (l < nl) cells[l] = overlay_quad_cells(p, p.layer[l], Y, X0, by);
    }
    if (threadIdx.x < 8) {
#pragma unroll
      for (int l = 0; l < (LAYERS ? kMaxLayers : 1); ++l) {
        const OverlayLayer& L = p.layer[l];
        const uint32_t col = overlay_colour(L, threadIdx.x), a = (uint32_t)L.a;
        s_terms[l][threadIdx.x] = make_uint2(mad24(a, col & 0xffu, 128u) | mad24(a, (col >> 8) & 0xffu, 128u) << 16,
                                             mad24(a, (col >> 16) & 0xffu, 128u));
      }
    }
    __syncthreads();
    overlay_layer_quad(p.layer[0], s_terms[0], cells[0], w, Y, X0, by);
    if constexpr (LAYERS) {
#pragma unroll
      for (int l = 1; l < kMaxLayers; ++l)
        if (l < nl) overlay_layer_quad(p.layer[l], s_terms[l], cells[l], w, Y, X0, by);
    }
    stamp_end();
    if (q_own < total) {
      if (bytes == 12) {
        *reinterpret_cast<u32x3*>(dst + at) = u32x3{w[0], w[1], w[2]};
      } else {
#pragma unroll
        for (int i = 0; i < 9; ++i)
          if (i < bytes) dst[at + i] = (uint8_t)(w[i >> 2] >> (8 * (i & 3)));
      }
    }
  } else {
    __shared__ u32x4 s_x[4][192];
    const int gpr = (p.wf + 15) >> 4, total = gpr * p.hf;        // groups per row, of the frame
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g_wave = (b - p.n_max) * 256 + wave * 64;          // first group of the wavefront
    if (g_wave >= total) return;
    // rows of whole groups that butt against each other: the frame is one run of vectors
    const bool flat = (p.wf & 15) == 0 && p.pitch == (size_t)48 * gpr;
    // all quotients by float estimate + exact fix-up (operands < 2^31, quotients < 2^22)
    const int g = min(g_wave + lane, total - 1);
    const int Y = (int)udiv_est((uint32_t)g, (uint32_t)gpr, p.rcp_gpr), X0 = (g - Y * gpr) * 16;
    // the first layer's map bytes are requested before the pixels, so the two fetches overlap
    const OverlayCells first = overlay_cells(p, p.layer[0], Y, X0, by);
    // vector 64 * j + lane of the wavefront: byte offset in the frame, and how many of its bytes are pixels
    size_t v_off[3];
    int v_bytes[3];
    u32x4 t[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int v = 64 * j + lane;
      const uint32_t gi = ((uint32_t)v * 171u) >> 9;             // v / 3 for v < 192
      const int gv = g_wave + (int)gi;
      if (flat) {
        const bool in = gv < total;
        v_off[j] = (size_t)(in ? g_wave * 3 + v : g_wave * 3) * 16;
        v_bytes[j] = in ? 16 : 0;
      } else {
        const int yv = (int)udiv_est((uint32_t)min(gv, total - 1), (uint32_t)gpr, p.rcp_gpr);
        const int in_row = (min(gv, total - 1) - yv * gpr) * 48 + (v - 3 * (int)gi) * 16;
        v_bytes[j] = gv < total ? max(0, min(16, 3 * p.wf - in_row)) : 0;
        v_off[j] = (size_t)yv * p.pitch + (v_bytes[j] > 0 ? in_row : 0);
      }
      t[j] = *reinterpret_cast<const u32x4*>(src + v_off[j]);
    }
    s_x[wave][lane] = t[0]; s_x[wave][64 + lane] = t[1]; s_x[wave][128 + lane] = t[2];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    uint32_t w[12];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const u32x4 v = s_x[wave][3 * lane + j];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[4 * j + i] = v[i];
    }
    overlay_layer_group(p, p.layer[0], first, w, Y, X0, by);
    if constexpr (LAYERS) {
#pragma unroll 1
      for (int l = 1; l < nl; ++l)
        overlay_layer_group(p, p.layer[l], overlay_cells(p, p.layer[l], Y, X0, by), w, Y, X0, by);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const u32x4 o = {w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]};
      s_x[wave][3 * lane + j] = o;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    stamp_end();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const u32x4 o = s_x[wave][64 * j + lane];
      if (v_bytes[j] == 16) {
        *reinterpret_cast<u32x4*>(dst + v_off[j]) = o;
      } else if (v_bytes[j] > 0) {                               // the end of a row inside this vector
#pragma unroll
        for (int i = 0; i < 15; ++i)
          if (i < v_bytes[j]) dst[v_off[j] + i] = (uint8_t)(o[i >> 2] >> (8 * (i & 3)));
      }
    }
  }
}

// Quads where a group of 16 pixels may see three cells of some layer's map, and for launches of fewer than 192 workgroups'
// worth of such groups, which leave CUs idle.  Us, groups of 16 / quads (cells of 16 pixels and more): 640 x 360 6.5 / 4.3,
// annotated 8.1 / 5.0; 960 x 540 (32 400 groups) 5.8 / 4.5; 1280 x 720 (57 600) 5.0 / 4.8; 1279 x 719 4.6 / 4.9; 1920 x 1080 6.1 / 5.3,
// annotated 6.3 / 8.1; four 1279 x 719 (230 080) 6.7 / 8.1; twelve 1920 x 1080 24.1 / 30.9.  (One line for all: between it and
// about 130 000 groups a plain frame would be up to 0.8 us faster in quads, an annotated one 1.8 slower.)  Before the quads and the annotations as
// masks (a third cell fetched on demand, labels pixel by pixel): 320 x 240 with cells of 10 pixels 11.0 (4.8 now), annotated
// 322 x 241 21.8 (4.8), four annotated 1279 x 719 15.3 (8.7), twelve annotated 1920 x 1080 37.4 (29.0).
static bool overlay_fine(const OverlayParams& p) {
  for (int l = 0; l < p.n_layers; ++l)
    if (15 * p.layer[l].wm > p.wf) return true;
  return (int64_t)((p.wf + 15) >> 4) * p.hf * p.batch < 192 * 256;
}

KernelDesc describe(const OverlayParams& p) {
  const bool fine = overlay_fine(p);
  const unsigned threads = (unsigned)((fine ? (p.wf + 3) >> 2 : (p.wf + 15) >> 4) * p.hf);
  const void* f = p.n_layers > 1 ? (fine ? (const void*)k_overlay<true, true> : (const void*)k_overlay<true, false>)
                                 : (fine ? (const void*)k_overlay<false, true> : (const void*)k_overlay<false, false>);
  return KernelDesc{f, dim3(1 + (unsigned)p.n_max + (threads + 255) / 256, p.batch), dim3(256), 0};
}

// ---------------------------------------------------------------------------------------------
// Gate scratch for callers that cannot allocate.  In host code the array's name is only a
// handle for hipGetSymbolAddress: every GPU holds its own copy at its own address, looked up
// once per device (with that device current) and used as an ordinary device pointer from then
// on -- the kernels receive it in their parameter blocks like the workspace scratch it replaces.
// ---------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch_address(void** d_ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static void* ptr_of[kMaxDevices] = {nullptr};
  static std::mutex mu;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!ptr_of[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    ptr_of[dev] = ptr;
  }
  *d_ptr = ptr_of[dev];
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_fill_zero(uint4* d, size_t n) {
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride)
    d[i] = make_uint4(0, 0, 0, 0);
}

// Plain streaming copy (16-byte vectors, grid-stride): the known-size kernel that hardware
// byte counters are calibrated against.
__global__ __launch_bounds__(256) void k_copy(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                              size_t n) {
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

void launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 16;
  if (n == 0) return;
  const unsigned blocks = (unsigned)min((size_t)8192, (n + 255) / 256);
  hipLaunchKernelGGL(k_copy, dim3(blocks), dim3(256), 0, s, reinterpret_cast<const uint4*>(src),
                     reinterpret_cast<uint4*>(dst), n);
}

void launch_fill_zero(void* d, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 16;
  if (n == 0) return;
  const unsigned blocks = (unsigned)min((size_t)2048, (n + 255) / 256);
  hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(256), 0, s, reinterpret_cast<uint4*>(d), n);
}

}  // namespace hs
