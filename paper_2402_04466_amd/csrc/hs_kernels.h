// Device-side interface of libhs: parameter blocks and launch functions of the HIP
// kernels behind the four per-frame stages (format conversion, recurrent conv-net
// inference, postprocess, overlay; paper Section III-A).  Host code fills a parameter
// block once per layer at application creation and launches it per frame.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "hs_run.h"

namespace hs {

typedef _Float16 f16;

// How to launch a kernel whose single argument is one of the parameter blocks below:
// hipLaunchKernel(func, grid, block, {&params}, shmem, stream), or the same as a graph node.
struct KernelDesc {
  const void* func;
  dim3 grid, block;
  unsigned shmem;
};

// ---- stage 1: bilinear resize (exact integer) + normalise + interleave ----------------
constexpr int kMaxBatch = 16;   // streams one launch can serve (blockIdx.y = stream)

struct ResizeParams {
  const uint8_t* src[kMaxBatch];   // per stream: frame, RGB bytes, row pitch src_pitch (x16)
  int batch;
  size_t dst_img_stride;           // halves between the streams' padded images
  size_t dst32_img_stride;         // floats between the streams' planar fp32 tensors
  size_t src_pitch;
  int wi, hi, wo, ho;
  f16* dst;             // padded 4-channel fp16 image: pixel (y+pad_t, x+pad_l), pitch dst_w px
  int dst_w, pad_l, pad_t;
  float* dst_f32;       // optional planar fp32 [3][ho][wo]
  const float* lut32;   // 256 entries
  const f16* lut16;     // 256 entries
  float rcp_dx, rcp_dy;         // 1/(2*wo), 1/(2*ho): division estimates
  uint64_t* t_end;      // the launch's end, on the device's constant-rate clock, as its highest-numbered workgroup sees it
  uint32_t d_magic, d_shift;    // floor(n / (4*wo*ho)) = mulhi(n, d_magic) >> d_shift for n < 2^31
};
KernelDesc describe(const ResizeParams& p);

// ---- stage 2: implicit-GEMM convolution on fp16 MFMA ------------------------------------
// Activations are pixel-major ("NHWC"): element (y, x, c) at in[(y*win + x)*cin_pitch + c].
// The K axis is cut into chunks of KC contiguous halves; chunk q belongs to tap
// q / chunks_per_tap = (ky, kx) = (tap / kw, tap % kw) and starts at channel
// (q % chunks_per_tap) * KC of input pixel (stride*oy + ky - pad, stride*ox + kx - pad).
// Out-of-range pixels read as zero.  First layers (3 input channels) use a padded
// 4-channel image and "row taps": kw = 1, a chunk spans several adjacent pixels.
enum ConvVariant {
  CONV_DIRECT,    // <= 32 output channels, one chunk of 16 or 32 halves per tap, <= 9 taps: no LDS tiles,
                  // K splits inside the workgroup (k_conv_direct); wt_frag: [chunk][K-step][lane][8]
  CONV_TINY_NET,  // the whole small network in one launch (k_tiny_net): hin, win the padded image, hout, wout the logits'
                  // map, mid_h, mid_w the first layer's; wt_frag: the four layers' weights as for CONV_DIRECT
  CONV_BLOCK64,   // a whole 64 -> 64 -> 64 channel block (two 3x3/1 convolutions, ReLU between,
                  // shortcut from the input, ReLU) in one launch (k_block64_fused): wt_frag = first,
                  // wt2_frag = second convolution, res = in
  CONV_S2_DIRA,   // 3x3/2 layers (+ fused 1x1/2 projection) of one Cin chunk on large grids: tile 8 x 8 x 128, weights
                  // from wt_frag / wt2_frag, tile walking, no residual (k_conv3x3s2_dira)
  CONV_KW         // 3x3 layers with the K splits inside the workgroup, tiles of consecutive pixels, weights from wt_frag /
                  // wt2_frag.  Stride 1, an even number of Cin chunks: k_conv3x3_run.  Stride 2, always with its fused
                  // projection: k_conv3x3s2_run
};
// The forms of k_conv3x3_run: channels and pixels of a tile, loading passes over a patch (32 pixels each), bytes of a patch
// buffer; cost of a tile in us where its CU works on several, fixed and per Cin chunk (see Builder::choose_form).
struct RunForm {
  int ch, px, passes, lds;
  double cost, chunk_cost;
  constexpr int splits() const { return 128 / ch; }   // K splits: four wavefronts of 32 channels each
};
constexpr RunForm kRunForms[] = {
    {32, 32, 3, 16384, 0.35, 0.47}, {32, 64, 4, 24576, 0.55, 0.57},  {64, 64, 4, 24576, 0.75, 1.03},
    {64, 96, 6, 26624, 1.3, 1.29},  {64, 128, 7, 36864, 1.9, 1.62}, {64, 160, 8, 40960, 2.3, 2.22},
    {32, 32, 7, 44032, 0.35, 0.47},   // patches of maps a few pixels wide or high, which hold mostly border
    {32, 128, 7, 36864, 1.37, 0.745},   // partitions alone
};
constexpr int kRunFormCount = 8, kRunFormAnyMap = 6;
// And of k_conv3x3s2_run: patch pixels per loading pass, 16-byte LDS units per patch pixel besides.
struct Run2Form {
  int ch, px, passes, lds, step, units;
  double cost, chunk_cost;
  constexpr int splits() const { return 128 / ch; }
};
constexpr Run2Form kRun2Forms[] = {
    {32, 32, 6, 28672, 32, 9, 1.2, 0.53}, {64, 32, 3, 16384, 64, 5, 0.4, 1.3}, {64, 64, 5, 28672, 64, 5, 1.4, 1.62},
    {64, 96, 8, 40960, 64, 5, 2.4, 2.0},
    {32, 32, 8, 40960, 32, 9, 1.2, 0.53},   // maps a few pixels wide or high
};
constexpr int kRun2FormCount = 5, kRun2FormAnyMap = 4;
// What k_conv3x3_run and k_conv3x3s2_run read of a layer's parameters, and so all that their launches hand over.
struct RunParams {
  const f16* in;
  const f16* wt_frag;   // weights in MFMA fragment order: [cout_pad / 32][Cin chunk][tap][K-step of 16][lane][8 halves], lane
                        // r + 32 h holding k = 16 * step + 8 * h .. + 7 of channel 32 * group + r
  f16* out;             // out[m*out_pitch + n]
  const f16* res;       // optional residual, res[m*res_pitch + n]
  float* partial;       // [m][cout_pad] fp32
  // CONV_BLOCK64: the second convolution's weights.  Stride 2: fused 1x1 stride-2 projection of the
  // same input (no residual, no ReLU), or NULL: [cout_pad / 32][Cin chunk][K-step of 16][lane][8 halves]
  const f16* wt2_frag;
  f16* out2;
  // CONV_KW: weights of the layer that runs next, to be prefetched, in 128-byte lines (0: none)
  const void* next_wt; int next_lines;
  int cin_pitch, out_pitch, res_pitch, out2_pitch;
  int cout_pad;         // multiple of the block's N tile
  int chunks_per_tap;
  int use_partial;      // 1: store the fp32 sums for the ConvLSTM epilogue, no epilogue here
  int relu;
  int tiles_m, tiles_n; // spatial x channel tiles; the grid is 8 * tiles_per_xcd workgroups
  int tiles_per_xcd;    // ceil(workgroups / 8)
  int n_block;          // channel tiles per block of the tile order (divides tiles_n;
                        // 1: spatial tile fastest, tiles_n: channel tile fastest)
  // bytes of the input (CONV_BLOCK64, too) and of the weights; log2 of n_block, reciprocal of tiles_m * n_block (run_div31); tiles
  uint32_t run_in_bytes, run_w_bytes;
  int run_nb_shift;
  uint32_t run_by_blk;
  RunGeometry run;
};
struct ConvParams : RunParams {
  int hin, win;
  int mid_h, mid_w;     // CONV_TINY_NET
  int hout, wout, m;    // m = batch*hout*wout output pixels (images stacked along m)
  int batch, img_m;     // images per launch, pixels per image (hout*wout)
  int cout;
  int kc;               // 16, 32 or 64
  int variant;          // ConvVariant
  int kw_splits;        // CONV_DIRECT: K splits
  int tiles_x;          // spatial variants: tiles per output row
  uint32_t tiles_img, by_tiles_img, by_tiles_x;   // CONV_BLOCK64: tiles per image; reciprocals (run_div31)
  int ntaps, kw, nchunks, ktot;
  int stride, pad;
  int chunks_per_split; // K split z handles chunks [z*chunks_per_split, ...)
  int tiles_per_wg;     // consecutive spatial tiles one workgroup walks (>= 1);
                        // workgroups = ceil(tiles_m / tiles_per_wg) * tiles_n
  float* out_f32;       // if set: the logits, planar fp32 out_f32[(image*8 + n)*img_m + pixel], instead of
                        // `out`; with them stage 3's per-cell outputs (see PostParams)
  float theta; float* heat; uint8_t* mask; uint8_t* kmap; uint64_t* t_end;
  int run_form;         // CONV_KW: form (kRunForms, kRun2Forms)
};
KernelDesc describe(const ConvParams& p);

// CONV_TINY_NET from the frame on: stage 1 in the same launch (r; its padded image is written, but not read).
struct TinyFrameParams {
  ResizeParams r;
  const f16* wt_frag;
  float* out_f32; float* heat; uint8_t* mask; uint8_t* kmap; uint64_t* t_end;   // as in ConvParams
  float theta;
  int mid_h, mid_w, hout, wout, m, img_m;
};
KernelDesc describe(const TinyFrameParams& p);

// ConvLSTM gate non-linearities and state update from the gate pre-activations, plus the 1x1
// head on the new h.  partial: [m][4*hid], channels ordered i, f, g, o (hid each);
// hid must be 256.  c: fp32 [m][hid] updated in place; h: fp16 written to h_out[m*h_pitch + j];
// logits[(image*8 + k)*img_m + pixel] = sum_j w_head[k][j] * h[pixel][j] (fp16 weights).
struct LstmEpilogueParams {
  const float* partial; int m; int hid;
  float* c; f16* h_out; int h_pitch;
  const f16* w_head; float* logits; int img_m;
  // stage 3's per-cell outputs (see PostParams), from the same logits
  float theta; float* heat; uint8_t* mask; uint8_t* kmap; uint64_t* t_end;
};
KernelDesc describe(const LstmEpilogueParams& p);

// Stem of the ResNet-style backbone: 7x7 stride-2 pad-3 convolution 3 -> 64, ReLU, 3x3 stride-2
// pad-1 max-pool, fused.  in: padded 4-channel fp16 images (pad 3 on the top and left, zeros),
// hin x win pixels each with win even; wt: the [64][224] matrix, k = (ky*8 + px)*4 + ch, zero where
// px == 7 or ch == 3, in MFMA fragment order: [channel half][ky][K-step of 16][lane][8 halves]; out: pooled pixel-major [batch][hp][wp][64].
struct StemPoolParams {
  const f16* in; const f16* wt; f16* out;
  int hin, win;          // padded image
  int hc, wc;            // convolution output
  int hp, wp;            // pooled output
  int batch;
  int tiles_x, tiles_y;  // tiles of 8 x 15 pooled pixels
  int tiles_per_xcd;     // ceil(batch * tiles_y * tiles_x / 8)
};
KernelDesc describe(const StemPoolParams& p);

// ---- stage 3: postprocess -----------------------------------------------------------------
struct PostRecord {           // written by the kernel into pinned host memory
  int32_t argmax_idx[8];
  float peak[8];
  uint8_t present[8];
  // found in the overlay's launch: ticks of the device's constant-rate clock from the end of stage 2
  // (see PostParams) until then
  int32_t ticks[8];
};
// The ends of the stages on the device's constant-rate clock, in pinned host memory, written by the overlay's launch
// (post: where stage 3 has a launch; drawn: where wanted).  drawn is the launch's end as its highest-numbered workgroup
// sees it ahead of its last stores.  (Events attached to the stages' last kernels would say the same, but each of them
// leaves the queue idle for 4.6 us, since such a kernel ends with a release to the host; one for the overlay's begin, for
// its length, leaves it idle for 14.)
struct StageStamps { uint64_t pre, infer, post, drawn; };
// Stage 3.  Per cell (written by the kernel that computes the logits): heat = sigmoid(logit), mask =
// logit > theta, both [batch][8][n], and kmap [batch][n] = the lowest channel whose mask is set, 0xff
// if none (what the overlay draws).  Per channel (here, or in the overlay's launch): PostRecord.
// t_end: that kernel's end, on the device's constant-rate clock (one for all XCDs), as its highest-numbered workgroup sees
// it.
struct PostParams {
  const float* logits; int n;    // [batch][8][n]
  float theta;                   // logit threshold
  PostRecord* rec;               // [batch], host-visible
  int batch;
  // anchors of the annotation layer: marks[(image*8 + k)*2 + {0,1}] = frame position (cx, cy) of
  // the centre of tool k's argmax cell, cx = -1 when the tool is absent; NULL: not wanted
  int* marks;
  int wm, hm, wf, hf;            // map (n == wm*hm) and frame size, for the anchors
  uint64_t* t_end;               // as in ResizeParams
};
KernelDesc describe(const PostParams& p);

// ---- stage 4: overlay ---------------------------------------------------------------------
constexpr int kMaxLayers = 4;   // networks whose results one overlay launch can draw
// What one network contributes to the picture: its channel map, colours and annotations.
struct OverlayLayer {
  const uint8_t* kmap; int wm, hm;   // [batch][hm][wm]: lowest set mask channel or 0xff
  float rcp_wm;                      // 1/wm: division estimate (needs wf*wm and hf*hm below 2^31)
  int a;                             // Q8 alpha, 0..256
  uint32_t pal[8];                   // R | G<<8 | B<<16
  // annotation layer: cross-hair and 'T'<k> label per present tool, opaque, in tool order
  const int* marks;                  // anchors written by the postprocess kernel, NULL: none
  int arm, half, scale;              // marker arm / half thickness, pixels per glyph cell
  // stage 3's channel maxima of this layer's network, found in the overlay's launch: logits
  // [batch][8][hm*wm] and the records [batch] (NULL: a launch of their own has found them)
  const float* logits; PostRecord* rec; float theta;
  // ends of stages 1 to 3 on the device's clock (stage 3's where it has a launch), and where the host wants them (NULL:
  // nowhere)
  const uint64_t* t_stages; StageStamps* stamps;
  uint64_t glyph[9];                 // bit (5*row + col) of glyph g, col 0 = leftmost
};
template <int N>
struct OverlayParamsOf {
  const uint8_t* src[kMaxBatch]; uint8_t* dst[kMaxBatch];   // per stream
  int batch; size_t pitch; int wf, hf;
  float rcp_gpr, rcp_qpr, rcp_hf, rcp_wf;   // 1/ceil(wf/16), 1/ceil(wf/4), 1/hf, 1/wf (ceil(wf/4)*hf below 2^31)
  int n_layers;                      // layers drawn in order, each over the one before
  int n_max;                         // workgroups per image between the first and the drawing ones: 8 * n_layers
                                     // when some layer has a rec, else 0
  int stamp_end;                     // the layers' stamps->drawn is wanted
  OverlayLayer layer[N];
};
typedef OverlayParamsOf<kMaxLayers> OverlayParams;   // begins like OverlayParamsOf<1>, all that a launch of one layer hands over
static_assert(offsetof(OverlayParams, layer) == offsetof(OverlayParamsOf<1>, layer), "the same beginning");
KernelDesc describe(const OverlayParams& p);

// ---- scratch for callers that cannot allocate ---------------------------------------------
// A fixed device array inside the library (one copy per GPU, held until the process ends) that
// can stand in for the gate scratch of an application's workspace.  Returns the array's
// device address ON THE CURRENT DEVICE and its size; the address is looked up once per device.
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
hipError_t static_scratch_address(void** d_ptr, size_t* bytes);

// ---- helpers ------------------------------------------------------------------------------
void launch_fill_zero(void* d, size_t bytes, hipStream_t s);   // bytes multiple of 16
void launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);   // bytes multiple of 16

}  // namespace hs
