// Plans and encodes one dense convolution per input line, or two that read the same tensor, and says what would be launched.  Links the library's planner and
// encoders (net_plan.cpp, launch.cpp) against a kernel table without a device, so that a plan which its own encoder refuses is
// found on the CPU.
// Line: DTYPE(0 fp32, 1 bf16) C_IN H W C_OUT K STRIDE PAD PLAN_CUS, and of the second convolution C_OUT (0: none) K STRIDE PAD.
// Answer, of the first convolution: ENCODED KERNEL_ID PIXELS_PER_WAVE THREADS SPLIT_K SHARES_A_LAUNCH GATHER K_STEPS STEPS_OF_A_WORKGROUP STEPS_OF_A_WAVE WORKGROUPS,
// and what its launch has: KERNEL_ID WORKGROUPS THREADS; or -1 and why not.
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../paper_2504_08795_amd/csrc/aql.h"
#include "../../paper_2504_08795_amd/csrc/kernels.h"
#include "../../paper_2504_08795_amd/csrc/net_plan.h"

using namespace daris;

// Every kernel the table asks for, with the size of its argument block.
const AqlKernel* AqlRuntime::kernel(const std::string& name) const {
  static const struct { const char* base; uint32_t bytes; } sizes[] = {
      {"conv_wave_kernel", sizeof(ConvArgs)}, {"conv_taps_kernel", sizeof(ConvArgs)}, {"conv_taps16_kernel", sizeof(ConvArgs)}, {"conv_image_kernel", sizeof(ImageConvArgs)}, {"conv_wave_pair_kernel", 2 * sizeof(ConvArgs) + 4}, {"conv_wave16_kernel", sizeof(ConvArgs)},
      {"conv_wave16_pair_kernel", 2 * sizeof(ConvArgs) + 4}, {"conv_wave_dw_kernel", sizeof(ConvArgs) + sizeof(DwFusedArgs)},
      {"conv_block_kernel", sizeof(ConvArgs)}, {"conv_large_kernel", sizeof(ConvArgs)}, {"conv_point_kernel", sizeof(ConvArgs)}, {"conv_point_pair_kernel", 2 * sizeof(ConvArgs) + 4}, {"conv_taps_large_kernel", sizeof(ConvArgs)}, {"splitk_reduce_kernel", 48}, {"dwconv_kernel", sizeof(DwArgs)}, {"dwconv_window_kernel", sizeof(DwWindowArgs)},
      {"maxpool_kernel", sizeof(PoolArgs)}, {"maxpool_window_kernel", sizeof(PoolWindowArgs)}, {"gavgpool_kernel", sizeof(PoolArgs)}, {"fc_kernel", sizeof(FcArgs)},
      {"ingest_kernel", 28}, {"egress_kernel", 28}, {"cu_probe_kernel", 12}};
  static AqlKernel known[sizeof(sizes) / sizeof(sizes[0])];
  for (size_t i = 0; i < sizeof(sizes) / sizeof(sizes[0]); ++i) {
    const std::string base = std::string("daris::") + sizes[i].base;
    if (name.compare(0, base.size(), base) == 0 && (name.size() == base.size() || name[base.size()] == '<')) {
      known[i].object = 1;
      known[i].kernarg_size = sizes[i].bytes;
      return &known[i];
    }
  }
  return nullptr;
}

int main() {
  AqlRuntime rt;
  KernelTable kt;
  const std::string missing = kt.resolve(rt);
  if (!missing.empty()) {
    std::fprintf(stderr, "kernel %s\n", missing.c_str());
    return 2;
  }
  int dtype, cin, h, w, cus, cout[2], k[2], s[2], p[2];
  while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d", &dtype, &cin, &h, &w, &cout[0], &k[0], &s[0], &p[0], &cus, &cout[1], &k[1], &s[1], &p[1]) == 13) {
    daris_layer L[2];
    std::memset(L, 0, sizeof L);
    for (int i = 0; i < 2; ++i) {
      L[i].op = DARIS_OP_CONV; L[i].c_in = cin; L[i].c_out = cout[i]; L[i].k = k[i]; L[i].stride = s[i]; L[i].pad = p[i]; L[i].groups = 1;
      L[i].in_from = -1; L[i].res_from = -1;
    }
    daris_dnn d;
    d.n_layers = cout[1] ? 2 : 1; d.in_c = cin; d.in_h = h; d.in_w = w; d.dtype = dtype; d.layers = L;
    NetPlan net;
    const std::string err = build_plan(d, false, true, true, true, true, true, cus, &net);
    if (!err.empty()) {
      std::printf("-1 %s\n", err.c_str());
      continue;
    }
    const TensorInfo& in = net.tensor(0);
    static float ws;
    ConvArgs a[2];
    std::memset(a, 0, sizeof a);
    for (int i = 0; i < d.n_layers; ++i) {
      const LayerPlan& P = net.layers[i];
      ConvArgs& c = a[i];
      c.ws = &ws;
      c.H = in.H; c.W = in.W; c.Cin = in.Cs; c.Ho = P.out.H; c.Wo = P.out.W; c.Cout = P.out.Cs;
      c.kh = c.kw = k[i]; c.stride = s[i]; c.pad = p[i]; c.Kpad = P.Kpad; c.M = P.out.H * P.out.W;
      c.splitk = P.cp.splitk; c.S = P.cp.S; c.sz = P.cp.sz; c.sw = P.cp.sw; c.MT = P.cp.MT; c.NTn = P.cp.NTn; c.G = P.cp.G; c.xmode = P.cp.xmode;
      c.c_real = i == 0 && net.fuse_ingest ? net.in_c : 0;
    }
    std::vector<KernelLaunch> out;
    const LayerPlan &A = net.layers[0], &B = net.layers[d.n_layers - 1];
    const bool pair = A.pair_with >= 0;
    bool ok;
    if (pair) ok = B.macs >= A.macs ? encode_conv_pair(kt, B.cp, a[1], A.cp, a[0], net.bf16, &out) : encode_conv_pair(kt, A.cp, a[0], B.cp, a[1], net.bf16, &out);
    else ok = encode_conv(kt, A.cp, a[0], net.bf16, &out) && (d.n_layers == 1 || encode_conv(kt, B.cp, a[1], net.bf16, &out));
    const KernelLaunch first = out.empty() ? KernelLaunch() : out[0];
    std::printf("%d %d %d %d %d %d %d %d %d %d %u %d %u %u\n", ok ? 1 : 0, A.cp.kernel, A.cp.rows, A.cp.threads, A.cp.splitk, pair ? 1 : 0, A.cp.gather, A.cp.S, A.cp.sz, A.cp.sw, A.cp.grid_x,
                first.kernel_id, first.groups, first.threads);
  }
  return 0;
}
