// Plans and encodes one dense convolution per input line and says what would be launched.  Links the library's planner and
// encoders (net_plan.cpp, launch.cpp) against a kernel table without a device, so that a plan which its own encoder refuses is
// found on the CPU.
// Line: DTYPE(0 fp32, 1 bf16) C_IN H W C_OUT K STRIDE PAD PLAN_CUS.  Answer: ENCODED KERNEL_ID PIXELS_PER_WAVE THREADS SPLIT_K.
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
      {"conv_wave_kernel", sizeof(ConvArgs)}, {"conv_wave_pair_kernel", 2 * sizeof(ConvArgs) + 4}, {"conv_wave16_kernel", sizeof(ConvArgs)},
      {"conv_wave16_pair_kernel", 2 * sizeof(ConvArgs) + 4}, {"conv_wave_dw_kernel", sizeof(ConvArgs) + sizeof(DwFusedArgs)},
      {"conv_block_kernel", sizeof(ConvArgs)}, {"splitk_reduce_kernel", 48}, {"dwconv_kernel", sizeof(DwArgs)}, {"dwconv_window_kernel", sizeof(DwWindowArgs)},
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
  int dtype, cin, h, w, cout, k, s, p, cus;
  while (std::scanf("%d %d %d %d %d %d %d %d %d", &dtype, &cin, &h, &w, &cout, &k, &s, &p, &cus) == 9) {
    daris_layer L;
    std::memset(&L, 0, sizeof L);
    L.op = DARIS_OP_CONV; L.c_in = cin; L.c_out = cout; L.k = k; L.stride = s; L.pad = p; L.groups = 1; L.in_from = -1; L.res_from = -1;
    daris_dnn d;
    d.n_layers = 1; d.in_c = cin; d.in_h = h; d.in_w = w; d.dtype = dtype; d.layers = &L;
    NetPlan net;
    const std::string err = build_plan(d, false, true, true, true, true, true, cus, &net);
    if (!err.empty()) {
      std::printf("-1 %s\n", err.c_str());
      continue;
    }
    const LayerPlan& P = net.layers[0];
    const TensorInfo& in = net.tensor(0);
    static float ws;
    ConvArgs a;
    std::memset(&a, 0, sizeof a);
    a.ws = &ws;
    a.H = in.H; a.W = in.W; a.Cin = in.Cs; a.Ho = P.out.H; a.Wo = P.out.W; a.Cout = P.out.Cs;
    a.kh = a.kw = k; a.stride = s; a.pad = p; a.Kpad = P.Kpad; a.M = P.out.H * P.out.W;
    a.splitk = P.cp.splitk; a.S = P.cp.S; a.sz = P.cp.sz; a.sw = P.cp.sw; a.MT = P.cp.MT; a.NTn = P.cp.NTn; a.G = P.cp.G; a.xmode = P.cp.xmode;
    a.c_real = net.fuse_ingest ? net.in_c : 0;
    std::vector<KernelLaunch> out;
    const bool ok = encode_conv(kt, P.cp, a, net.bf16, &out);
    std::printf("%d %d %d %d %d\n", ok ? 1 : 0, P.cp.kernel, P.cp.rows, P.cp.threads, P.cp.splitk);
  }
  return 0;
}
