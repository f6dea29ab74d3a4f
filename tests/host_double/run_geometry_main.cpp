// The tiles of k_conv3x3_run against a plain enumeration: every form, maps of one pixel to hundreds, several images.
// Every pixel is in exactly one tile; its nine taps read the patch pixels of its neighbours, or zeros outside the map;
// every patch fits its form's buffer and loading passes.
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "hs_kernels.h"

using namespace hs;

static long checked = 0;

#define CHECK(cond)                                                                                          \
  if (!(cond)) {                                                                                             \
    printf("%dx%d, %d images, form %d, strips of %d, tile %u: %s\n", w, h, batch, form, g.strip_w, t, #cond); \
    exit(1);                                                                                                 \
  }

static void check(int h, int w, int batch, int form) {
  const RunForm& f = kRunForms[form];
  RunGeometry g;
  const int tiles = run_plan(h, w, batch, f.px, f.passes, f.lds, g);
  uint32_t t = 0;
  if (tiles == 0) {
    g.strip_w = 0;
    CHECK(form != kRunFormAnyMap);
    return;
  }
  std::vector<char> seen((size_t)batch * h * w);
  const int rw = g.strip_w + 2;
  for (t = 0; t < (uint32_t)tiles; ++t) {
    const RunOrigin o = run_origin(g, t);
    // the patch, as the loading passes walk it
    std::vector<int> patch((size_t)g.rows * rw, -2);
    for (int thread = 0; thread < 32; ++thread) {
      uint32_t row = run_div23((uint32_t)thread, g.by23_row), col = (uint32_t)thread - row * (uint32_t)rw;
      for (int i = 0; i < f.passes; ++i) {
        CHECK((int)(row * (uint32_t)rw + col) == thread + 32 * i);
        if ((int)row < g.rows) {
          CHECK(((int)row * run_row_pitch(g.strip_w) + (int)col * kRunPitch + 64) * 2 <= f.lds - 128);
          int m;
          patch[row * (uint32_t)rw + col] = run_patch_pixel(g, o, row, col, m) ? m : -1;
        }
        row += (uint32_t)g.step_q;
        col += (uint32_t)g.step_r;
        if (col >= (uint32_t)rw) { col -= (uint32_t)rw; ++row; }
      }
    }
    for (int v : patch) CHECK(v != -2 && v < batch * h * w);
    for (int i = 0; i < f.px; ++i) {
      uint32_t row, col;
      int m;
      run_pixel(g, o, (uint32_t)i, row, col, m);
      CHECK((int)row + 2 < g.rows && (int)col + 2 < rw);
      if (m < 0) continue;
      CHECK(m < batch * h * w && !seen[(size_t)m]);
      seen[(size_t)m] = 1;
      const int img = m / (h * w), y = m / w % h, x = m % w;
      for (int ky = 0; ky < 3; ++ky)
        for (int kx = 0; kx < 3; ++kx) {
          const int iy = y + ky - 1, ix = x + kx - 1;
          const int want = iy >= 0 && iy < h && ix >= 0 && ix < w ? (img * h + iy) * w + ix : -1;
          CHECK(patch[(row + (uint32_t)ky) * (uint32_t)rw + col + (uint32_t)kx] == want);
        }
      ++checked;
    }
  }
  for (char c : seen) CHECK(c);
}

// The same at stride 2, on an input map of hin x win pixels.
static void check2(int hin, int win, int batch, int form) {
  const Run2Form& f = kRun2Forms[form];
  const int h = (hin + 1) / 2, w = (win + 1) / 2;
  RunGeometry g;
  const int tiles = run2_plan(hin, win, batch, f.px, f.passes, f.lds, f.step, f.units, g);
  uint32_t t = 0;
  if (tiles == 0) {
    g.strip_w = 0;
    CHECK(form != kRun2FormAnyMap);
    return;
  }
  std::vector<char> seen((size_t)batch * h * w);
  const int rw = 2 * g.strip_w + 1;
  for (t = 0; t < (uint32_t)tiles; ++t) {
    const RunOrigin o = run_origin(g, t);
    std::vector<int> patch((size_t)g.rows * rw, -2);
    for (int thread = 0; thread < f.step; ++thread) {
      uint32_t row = run_div23((uint32_t)thread, g.by23_row), col = (uint32_t)thread - row * (uint32_t)rw;
      for (int i = 0; i < f.passes; ++i) {
        CHECK((int)(row * (uint32_t)rw + col) == thread + f.step * i);
        if ((int)row < g.rows) {
          const int at = (int)row * g.pitch2 + (int)(col >> 1) * 8 * f.units + (col & 1 ? (g.strip_w + 1) * 8 * f.units : 0);
          CHECK((at + 8 * (f.units - 1)) * 2 <= f.lds - 128 && (int)(row + 1) * g.pitch2 >= at + 8 * f.units);
          int m;
          patch[row * (uint32_t)rw + col] = run2_patch_pixel(g, o, row, col, m) ? m : -1;
        }
        row += (uint32_t)g.step_q;
        col += (uint32_t)g.step_r;
        if (col >= (uint32_t)rw) { col -= (uint32_t)rw; ++row; }
      }
    }
    for (int v : patch) CHECK(v != -2 && v < batch * hin * win);
    for (int i = 0; i < f.px; ++i) {
      uint32_t row, col;
      int m;
      run2_pixel(g, o, (uint32_t)i, row, col, m);
      CHECK((int)row + 2 < g.rows && (int)col < g.strip_w);
      if (m < 0) continue;
      CHECK(m < batch * h * w && !seen[(size_t)m]);
      seen[(size_t)m] = 1;
      const int img = m / (h * w), y = m / w % h, x = m % w;
      for (int ky = 0; ky < 3; ++ky)
        for (int kx = 0; kx < 3; ++kx) {
          const int iy = 2 * y + ky - 1, ix = 2 * x + kx - 1;
          const int want = iy >= 0 && iy < hin && ix >= 0 && ix < win ? (img * hin + iy) * win + ix : -1;
          CHECK(patch[(row + (uint32_t)ky) * (uint32_t)rw + 2 * col + (uint32_t)kx] == want);
        }
      ++checked;
    }
  }
  for (char c : seen) CHECK(c);
}

int main() {
  for (int form = 0; form < kRun2FormCount; ++form) {
    for (int batch : {1, 2, 3, 7, 16})
      for (int h : {1, 2, 3, 4, 5, 7, 8, 15, 16, 29, 30, 60, 61})
        for (int w : {1, 2, 3, 4, 5, 9, 12, 13, 27, 28, 53, 54, 107, 108}) check2(h, w, batch, form);
    for (int h : {271, 1999, 4095, 4096}) check2(h, 32, 2, form);
    check2(32, 4096, 16, form);
    check2(723, 724, 4, form);
  }
  for (int form = 0; form < kRunFormCount; ++form) {
    for (int batch : {1, 2, 3, 7, 16})
      for (int h : {1, 2, 3, 4, 5, 7, 8, 12, 15, 23, 30, 31, 60})
        for (int w : {1, 2, 3, 5, 6, 9, 13, 14, 21, 27, 36, 41, 54, 65, 107}) check(h, w, batch, form);
    for (int h : {135, 999, 2047, 2048}) check(h, 16, 2, form);      // the largest maps the boundary accepts
    check(16, 2048, 16, form);
    check(362, 362, 4, form);
  }
  printf("%ld pixels in their tiles\n", checked);
  return 0;
}
