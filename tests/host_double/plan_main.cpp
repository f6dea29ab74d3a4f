// The library's own planning code.  Without arguments: plans of layers that no network here has; what the kernels do not do
// is refused.  With arguments, "resnet18_convlstm" or "tiny4" and width, height, batch: prints each layer's kernel and form.
#include "hs_lib.cpp"

#define CHECK(cond)                                   \
  do {                                                \
    if (!(cond)) {                                    \
      printf("line %d: %s\n", __LINE__, #cond);       \
      exit(1);                                        \
    }                                                 \
  } while (0)

static hs_app_desc description() {
  hs_app_desc d;
  memset(&d, 0, sizeof(d));
  d.batch = 2;
  return d;
}

static Tensor tensor(int h, int w, int c, int batch) {
  Tensor t;
  t.h = h; t.w = w; t.c = t.pitch = c;
  t.cap = (size_t)batch * h * w * c;
  return t;
}

// A stride-2 layer of so many Cin chunks, planned with one form.
static bool plans(int chunks, int form) {
  ConvParams c;
  memset(&c, 0, sizeof(c));
  c.batch = 2; c.hin = 24; c.win = 40; c.cin_pitch = 64 * chunks;
  c.hout = 12; c.wout = 20; c.img_m = 240; c.m = 480;
  c.cout = c.cout_pad = 128; c.kc = 64; c.ntaps = 9; c.kw = 3; c.stride = 2; c.pad = 1;
  c.chunks_per_tap = chunks; c.nchunks = 9 * chunks; c.ktot = 64 * c.nchunks;
  return Builder::plan_run2(c, form);
}

static int print_forms(const char* net, int w, int h, int batch) {
  hs_app_desc d = description();
  d.net = strcmp(net, "tiny4") == 0 ? HS_NET_TINY4 : HS_NET_RESNET18_CONVLSTM;
  d.net_w = w; d.net_h = h; d.batch = batch;
  int pw, ph, pad;
  padded_input_geometry(w, h, d.net == HS_NET_TINY4 ? 3 : 7, &pw, &ph, &pad);
  Builder b(d, nullptr, false, false);
  b.walk(ph, pw);
  for (const Op& op : b.ops) {
    if (op.fam != F_CONV && op.fam != F_NET) continue;
    const ConvParams& c = op.conv;
    switch (c.variant) {
      case CONV_DIRECT: printf("direct %d\n", c.kw_splits); break;
      case CONV_TINY_NET: printf("tiny_net 0\n"); break;
      case CONV_BLOCK64: printf("block64 0\n"); break;
      case CONV_S2_DIRA: printf("s2_dira 0\n"); break;
      default: printf("%s %d\n", c.stride == 1 ? "run" : "s2_run", c.run_form);
    }
  }
  return 0;
}

int main(int argc, char** argv) {
  if (argc == 5) return print_forms(argv[1], atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
  for (int form = 0; form < kRun2FormCount; ++form)
    for (int chunks = 1; chunks <= 8; ++chunks)
      // four K splits: whole chunks, in pairs or a single one; two: half chunks, always in pairs
      CHECK(plans(chunks, form) == (kRun2Forms[form].splits() == 2 || chunks == 1 || chunks % 2 == 0));
  // CUs that a mask keeps busy: engines with CUs times the fewest of one
  auto busy = [](int from, int to) {
    uint32_t mask[8] = {0};
    for (int i = from; i < to; ++i) mask[i / 32] |= 1u << (i % 32);
    return effective_cus(mask, 8, 256);
  };
  CHECK(busy(0, 256) == 256 && busy(0, 128) == 128 && busy(0, 80) == 64 && busy(80, 160) == 64 && busy(0, 40) == 32 && busy(0, 16) == 16);
  // a layer planned for fewer CUs: as many K splits; for all of them again: the plan it had
  for (int chunks : {2, 4, 8, 12})
    for (int batch : {1, 2, 3}) {
      ConvParams c;
      memset(&c, 0, sizeof(c));
      c.batch = batch; c.hin = c.hout = 15; c.win = c.wout = 27; c.img_m = 405; c.m = batch * 405; c.cin_pitch = 64 * chunks;
      c.cout = c.cout_pad = 512; c.kc = 64; c.ntaps = 9; c.kw = 3; c.stride = 1; c.pad = 1;
      c.chunks_per_tap = chunks; c.nchunks = 9 * chunks; c.ktot = 64 * c.nchunks;
      Builder::choose_split(c);
      const int form = c.run_form;
      for (int cus : {16, 32, 64, 128, 256}) {
        const ConvParams before = c;
        Builder::choose_split(c, &before, cus);
        CHECK(kRunForms[c.run_form].splits() == kRunForms[form].splits());
      }
      CHECK(c.run_form == form);
    }
  const hs_app_desc d = description();
  for (bool with_projection : {true, false}) {
    Builder b(d, nullptr, false, false);
    Tensor in = tensor(24, 40, 128, d.batch), out = tensor(12, 20, 128, d.batch), proj = out;
    bool refused = false;
    try {
      b.conv_layer(in, 0, 128, 3, 2, 1, true, nullptr, &out, false, false, 0, with_projection ? &proj : nullptr);
    } catch (const std::logic_error&) {
      refused = true;
    }
    CHECK(refused == !with_projection);
  }
  return 0;
}
