// Geometry of the tiles of k_conv3x3_run and k_conv3x3s2_run (see there): runs of consecutive pixels of strips of all
// images of a launch, and the patch under a run.  One definition for the kernels and for the host, which plans with it.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

namespace hs {

constexpr int kRunPitch = 64 + 8;        // LDS halves per patch pixel: 64 channels, padded against bank conflicts

// Of a layer: output maps of h x w pixels, input maps of hin x win (stride 1: the same), `batch` images.
struct RunGeometry {
  int px;               // pixels per tile
  int h, w, batch;
  int hin, win;
  int strip_w;          // columns per strip
  int rows;             // patch rows at most, the rows of zeros between images included
  int step_q, step_r;   // quotient and remainder of the patch pixels per loading pass by a patch row's length
  int pitch2;           // stride 2: LDS halves per patch row
  // reciprocals: ceil(2^31 / d) for quotients of scalars, ceil(2^23 / d) for those of lanes
  uint32_t by_strip_w, by_h, by_batch, by_period;   // period: stride 2, patch rows of an image
  uint32_t by23_strip_w, by23_row, by23_h, by23_h1, by23_batch;
};

// LDS halves per patch row.  The pixel behind a row's last one lies in the bank group it would lie in without the two
// border pixels between them (9 x 16 bytes per pixel, 16 bank groups).
constexpr __host__ __device__ __forceinline__ int run_row_pitch(int strip_w) { return kRunPitch * strip_w + 256; }

__host__ __device__ __forceinline__ uint32_t run_mul24(uint32_t a, uint32_t b) {
#ifdef __HIP_DEVICE_COMPILE__
  // written as an instruction because the compiler turns __umul24 back into a 32-bit multiply, at a quarter of the
  // rate, when it knows one factor to be small
  uint32_t r;
  asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
#else
  return (a & 0xffffffu) * (b & 0xffffffu);
#endif
}
__host__ __device__ __forceinline__ uint32_t run_div31(uint32_t n, uint32_t by) {   // n * d below 2^31
#ifdef __HIP_DEVICE_COMPILE__
  return __umulhi(n << 1, by);
#else
  return (uint32_t)(((uint64_t)(n << 1) * by) >> 32);
#endif
}
__host__ __device__ __forceinline__ uint32_t run_div23(uint32_t n, uint32_t by) {   // n * d below 2^23
  return run_mul24(n, by) >> 23;
}

// Workgroup `tile` of a launch of tiles_m runs x tiles_n channel tiles, in blocks of n_block = 1 << nb_shift channel tiles
// (by_blk: reciprocal of tiles_m * n_block): its run, its channel tile.  The surplus workgroups of a grid that is padded to
// whole XCDs get the last tile, so that what they load before they leave lies inside the layer's tensors.
struct RunTile {
  uint32_t run, channels;
};
__host__ __device__ __forceinline__ RunTile run_tile(uint32_t tile, int tiles_m, int tiles_n, int n_block, int nb_shift,
                                                     uint32_t by_blk) {
  const uint32_t nb = (uint32_t)n_block, last = (uint32_t)(tiles_m * tiles_n) - 1;
  tile = tile < last ? tile : last;
  const uint32_t blk = run_div31(tile, by_blk), in_blk = tile - blk * (uint32_t)tiles_m * nb;
  return RunTile{in_blk >> nb_shift, blk * nb + (in_blk & (nb - 1))};
}

// Where tile `tile` starts: row `y` of column `img` (image) of strip `strip`, `rem` pixels into the row.
struct RunOrigin {
  uint32_t rem, y, strip, img;
};
__host__ __device__ __forceinline__ RunOrigin run_origin(const RunGeometry& g, uint32_t tile) {
  const uint32_t q = tile * (uint32_t)g.px, row = run_div31(q, g.by_strip_w), v = run_div31(row, g.by_h);
  RunOrigin o;
  o.rem = q - row * (uint32_t)g.strip_w;
  o.y = row - v * (uint32_t)g.h;
  o.strip = run_div31(v, g.by_batch);
  o.img = v - o.strip * (uint32_t)g.batch;
  return o;
}

// Patch pixel (row, col): true if it is a pixel of the map, at index m of the launch's pixels; else it is a zero (border,
// or the row between two images, or beyond the last strip, which starts at column w or later).
__host__ __device__ __forceinline__ bool run_patch_pixel(const RunGeometry& g, const RunOrigin& o, uint32_t row, uint32_t col,
                                                         int& m) {
  const uint32_t e = o.y + row;          // 0: a row of zeros, then an image's rows, then the next image
  const uint32_t k = run_div23(e, g.by23_h1), f = e - k * (uint32_t)(g.h + 1);
  const uint32_t ds = run_div23(o.img + k, g.by23_batch), img = o.img + k - ds * (uint32_t)g.batch;
  const int x = (int)((o.strip + ds) * (uint32_t)g.strip_w + col) - 1;
  m = ((int)(img * (uint32_t)g.h + f) - 1) * g.w + x;
  return f != 0 && x >= 0 && x < g.w;
}

// Pixel i of the tile: its index m among the launch's pixels, -1 if there is none; (row, col): the patch pixel of its
// first tap.
__host__ __device__ __forceinline__ void run_pixel(const RunGeometry& g, const RunOrigin& o, uint32_t i, uint32_t& row,
                                                   uint32_t& col, int& m) {
  const uint32_t n = o.rem + i, d = run_div23(n, g.by23_strip_w);
  const uint32_t k = run_div23(o.y + d, g.by23_h), y = o.y + d - k * (uint32_t)g.h;
  const uint32_t ds = run_div23(o.img + k, g.by23_batch), img = o.img + k - ds * (uint32_t)g.batch;
  col = n - d * (uint32_t)g.strip_w;
  row = d + k;
  const uint32_t x = (o.strip + ds) * (uint32_t)g.strip_w + col;
  m = x < (uint32_t)g.w ? (int)((img * (uint32_t)g.h + y) * (uint32_t)g.w + x) : -1;
}

// Stride 2 (pad 1).  An output row's taps read input rows 2 y - 1 .. 2 y + 1: an image has 2 h + 1 patch rows, the first
// one zeros, the last one zeros too where hin is odd.  Strips are an even number of columns wide; a patch row holds
// 2 strip_w + 1 pixels, in LDS the even ones first, so that the lanes of a tap read neighbours.
__host__ __device__ __forceinline__ bool run2_patch_pixel(const RunGeometry& g, const RunOrigin& o, uint32_t row, uint32_t col,
                                                          int& m) {
  const uint32_t e = 2 * o.y + row, k = run_div31(e, g.by_period), f = e - k * (uint32_t)(2 * g.h + 1);
  const uint32_t ds = run_div23(o.img + k, g.by23_batch), img = o.img + k - ds * (uint32_t)g.batch;
  const int y = (int)f - 1, x = (int)(2 * (o.strip + ds) * (uint32_t)g.strip_w + col) - 1;
  m = ((int)img * g.hin + y) * g.win + x;
  return y >= 0 && y < g.hin && x >= 0 && x < g.win;
}
// The pixel's first tap: patch row `row`, even pixel `col` of it.
__host__ __device__ __forceinline__ void run2_pixel(const RunGeometry& g, const RunOrigin& o, uint32_t i, uint32_t& row,
                                                    uint32_t& col, int& m) {
  run_pixel(g, o, i, row, col, m);       // row = d + k: d output rows and k images further
  const uint32_t d = run_div23(o.rem + i, g.by23_strip_w);
  row += d;
}
// LDS halves per patch row with u 16-byte units per pixel: two rows further, the next output row's first pixel lies in
// the bank group behind its predecessor's.
constexpr __host__ __device__ __forceinline__ int run2_row_pitch(int strip_w, int u) {
  return 8 * (u * (2 * strip_w + 1) + ((u * strip_w / 2 - u * (2 * strip_w + 1)) % 8 + 8) % 8);
}

inline void run_finish_plan(RunGeometry& g, int px, int h, int w, int hin, int win, int batch, int row, int step) {
  g.px = px; g.h = h; g.w = w; g.hin = hin; g.win = win; g.batch = batch;
  g.step_q = step / row; g.step_r = step % row;
  auto by = [](int bits, int d) { return (uint32_t)((((uint64_t)1 << bits) + (uint64_t)d - 1) / (uint64_t)d); };
  g.by_strip_w = by(31, g.strip_w); g.by_h = by(31, h); g.by_batch = by(31, batch); g.by_period = by(31, 2 * h + 1);
  g.by23_strip_w = by(23, g.strip_w); g.by23_row = by(23, row);
  g.by23_h = by(23, h); g.by23_h1 = by(23, h + 1); g.by23_batch = by(23, batch);
}

// Plans runs of px pixels with patches of at most 32 * passes pixels and lds bytes: the strips as wide as gives the fewest
// tiles and then the smallest patch.  Returns the number of tiles, 0 if no strip width fits.
inline int run_plan(int h, int w, int batch, int px, int passes, int lds, RunGeometry& g) {
  const int64_t rows = (int64_t)batch * h;
  if (h > 2500 || rows * (w + 64) >= (int64_t)1 << 23) return 0;
  int best_tiles = 0, best_px = 0;
  for (int sw = 1; sw <= w && sw <= 64; ++sw) {
    const int64_t strips = (w + sw - 1) / sw, tiles = (rows * strips * sw + px - 1) / px;
    // rows under a run that starts anywhere in its first one, images that begin inside it
    const int d = (px % sw == 0 ? px - 1 : px + sw - 2) / sw, k = (d + h - 1) / h, n_rows = d + k + 3;
    const int n_px = n_rows * (sw + 2);
    if (n_px > 32 * passes || n_rows * run_row_pitch(sw) * 2 + 128 > lds) continue;
    if (tiles * px * sw >= (int64_t)1 << 31 || (rows * strips + px) * h >= (int64_t)1 << 31) continue;
    if (!best_tiles || tiles < best_tiles || (tiles == best_tiles && n_px < best_px)) {
      best_tiles = (int)tiles; best_px = n_px;
      g.strip_w = sw; g.rows = n_rows;
    }
  }
  if (!best_tiles) return 0;
  g.pitch2 = 0;
  run_finish_plan(g, px, h, w, h, w, batch, g.strip_w + 2, 32);
  return best_tiles;
}

// The same at stride 2; a loading pass takes `step` patch pixels of u 16-byte units in LDS.
inline int run2_plan(int hin, int win, int batch, int px, int passes, int lds, int step, int u, RunGeometry& g) {
  const int h = (hin + 1) / 2, w = (win + 1) / 2;
  const int64_t rows = (int64_t)batch * h;
  if (h > 2500 || rows * (w + 64) >= (int64_t)1 << 23) return 0;
  int best_tiles = 0, best_px = 0;
  for (int sw = 2; sw <= w + 1 && sw <= 64; sw += 2) {
    const int64_t strips = (w + sw - 1) / sw, tiles = (rows * strips * sw + px - 1) / px;
    const int d = (px % sw == 0 ? px - 1 : px + sw - 2) / sw, k = (d + h - 1) / h, n_rows = 2 * d + k + 3;
    const int n_px = n_rows * (2 * sw + 1);
    if (n_px > step * passes || n_rows * run2_row_pitch(sw, u) * 2 + 128 > lds) continue;
    if (tiles * px * sw >= (int64_t)1 << 31 || (rows * strips + px) * h >= (int64_t)1 << 31) continue;
    if (!best_tiles || tiles < best_tiles || (tiles == best_tiles && n_px < best_px)) {
      best_tiles = (int)tiles; best_px = n_px;
      g.strip_w = sw; g.rows = n_rows;
    }
  }
  if (!best_tiles) return 0;
  g.pitch2 = run2_row_pitch(g.strip_w, u);
  run_finish_plan(g, px, h, w, hin, win, batch, 2 * g.strip_w + 1, step);
  return best_tiles;
}

}  // namespace hs
