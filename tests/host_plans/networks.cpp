// Plans whole networks, cuts them into stages, encodes them as launches and walks the launches: every pointer lies in the buffer of the tensor that the layer
// reads or writes, that buffer holds this tensor when it is read, every tile of every launch is somebody's, and divisions by multiplication are exact as far as
// they are used.  Links the library's planner and encoders (net_plan.cpp, launch.cpp, net_encode.cpp), no GPU needed.
// Lines: DTYPE(0 fp32, 1 bf16) C H W PLAN_CUS STAGES N_LAYERS, then a line for each layer: OP C_IN C_OUT K STRIDE PAD GROUPS ACT IN_FROM RES_FROM.
// Answer: ok LAYER:KERNEL:WORKGROUPS ..., or bad and what.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../../paper_2504_08795_amd/csrc/aql.h"
#include "../../paper_2504_08795_amd/csrc/net_encode.h"

using namespace daris;

static std::map<const AqlKernel*, std::string> g_names;

const AqlKernel* AqlRuntime::kernel(const std::string& name) const {
  static const struct { const char* base; uint32_t bytes; } sizes[] = {
      {"conv_wave_kernel", sizeof(ConvArgs)}, {"conv_taps_kernel", sizeof(ConvArgs)}, {"conv_taps16_kernel", sizeof(ConvArgs)}, {"conv_image_kernel", sizeof(ImageConvArgs)},
      {"conv_wave_pair_kernel", 2 * sizeof(ConvArgs) + 4}, {"conv_wave16_kernel", sizeof(ConvArgs)}, {"conv_wave16_pair_kernel", 2 * sizeof(ConvArgs) + 4},
      {"conv_wave_dw_kernel", sizeof(ConvArgs) + sizeof(DwFusedArgs)}, {"conv_block_kernel", sizeof(ConvArgs)}, {"conv_large_kernel", sizeof(ConvArgs)},
      {"conv_taps_large_kernel", sizeof(ConvArgs)}, {"splitk_reduce_kernel", 48}, {"dwconv_kernel", sizeof(DwArgs)}, {"dwconv_window_kernel", sizeof(DwWindowArgs)},
      {"maxpool_kernel", sizeof(PoolArgs)}, {"maxpool_window_kernel", sizeof(PoolWindowArgs)}, {"gavgpool_kernel", sizeof(PoolArgs)}, {"fc_kernel", sizeof(FcArgs)},
      {"ingest_kernel", 28}, {"egress_kernel", 28}, {"cu_probe_kernel", 12}, {"conv_point_kernel", sizeof(ConvArgs)}, {"conv_point_pair_kernel", 2 * sizeof(ConvArgs) + 4},
      {"conv_image_pool_kernel", sizeof(ImageConvArgs)}, {"conv_expand_dw_kernel", sizeof(ExpandDwArgs)}, {"fc_pooled_kernel", sizeof(FcPooledArgs)},
      {"conv_chain_kernel", sizeof(ConvArgs) + sizeof(ChainArgs)}, {"conv_block_pool_kernel", sizeof(ConvArgs)}, {"conv_taps16_tall_kernel", sizeof(ConvArgs)}};
  static std::map<std::string, AqlKernel> known;
  for (const auto& s : sizes) {
    const std::string base = std::string("daris::") + s.base;
    if (name.compare(0, base.size(), base) == 0 && (name.size() == base.size() || name[base.size()] == '<')) {
      AqlKernel& k = known[name];
      k.object = 1;
      k.kernarg_size = s.bytes;
      g_names[&k] = name.substr(7);
      return &k;
    }
  }
  return nullptr;
}

namespace {

constexpr uint64_t kSlot = 1ull << 40, kWeights = 1ull << 60, kBias = 1ull << 61, kWorkspace = 1ull << 59;

struct Walk {
  const NetPlan& net;
  std::vector<int> holds;  // the tensor in each slot, -1: nothing yet
  std::string bad;
  std::string where;
  std::set<int> read, written;  // slots of the launch

  void fail(const std::string& what) {
    if (bad.empty()) bad = where + ": " + what;
  }
  void check(bool ok, const char* what) {
    if (!ok) fail(what);
  }
  int es() const { return net.bf16 ? 2 : 4; }
  size_t bytes(int tensor) const {
    const TensorInfo& t = net.tensor(tensor);
    return (size_t)t.H * t.W * t.Cs * es();
  }
  int slot_of(const void* p) {
    const uint64_t a = (uint64_t)(uintptr_t)p;
    if (a == 0 || a % kSlot != 0 || a / kSlot > holds.size()) {
      fail("a pointer to no buffer");
      return 0;
    }
    return (int)(a / kSlot) - 1;
  }
  void reads(const void* p, int tensor, size_t n) {
    const int s = slot_of(p);
    check(s == net.tensor(tensor).slot && holds[s] == tensor, ("tensor " + std::to_string(tensor) + " is not there any more").c_str());
    check(n <= net.slot_bytes[s], "reads past its buffer");
    read.insert(s);
  }
  void writes(const void* p, int tensor, size_t n) {
    const int s = slot_of(p);
    check(s == net.tensor(tensor).slot, "another tensor's buffer");
    check(n <= net.slot_bytes[s], "writes past its buffer");
    check(!written.count(s), "two tensors in one buffer");
    written.insert(s);
    holds[s] = tensor;
  }
  void done() {
    for (int s : written) check(!read.count(s), "writes what it reads");
    read.clear();
    written.clear();
  }
  int layer_of_weights(const void* w) { return (int)(((uint64_t)(uintptr_t)w - kWeights) >> 32); }
  int layer_of_bias(const void* b) { return (int)(((uint64_t)(uintptr_t)b - kBias) >> 32); }
  void divides(uint32_t magic, uint64_t d, uint64_t below) {  // fast_div for every n < below, by its edges
    auto one = [&](uint64_t n) { return n >= below || (magic ? (n * magic) >> 32 : n) == n / d; };
    bool ok = true;
    for (uint64_t n = 0; n < 64; ++n) ok = ok && one(n) && (below <= n || one(below - 1 - n));
    const uint64_t last = below ? (below - 1) / d : 0, step = std::max<uint64_t>(last / 500, 1);
    for (uint64_t q = 1; q <= last; q += step) ok = ok && one(q * d - 1) && one(q * d);
    ok = ok && one(last * d) && (last == 0 || one(last * d - 1));
    check(ok, "a division that is not exact");
  }
  // conv_tile_of over a launch's workgroups
  void tiles(const ConvArgs& p, uint32_t groups, int rows) {
    std::vector<char> seen((size_t)p.MT * p.G, 0);
    size_t n = 0;
    for (uint32_t L = 0; L < groups; ++L) {
      const int x = L & 7, q = L >> 3;
      int g, mt;
      if (p.xmode == 2) {
        const int lr = 3 - __builtin_ctz(p.G);
        g = x >> lr;
        mt = (q << lr) + (x & ((1 << lr) - 1));
      } else {
        const int i = p.xmode == 1 ? q : (int)L;
        const int d = p.mg_mt == kNoMagic ? i / p.MT : p.mg_mt ? (int)(((uint64_t)i * p.mg_mt) >> 32) : i;
        g = p.xmode == 1 ? d * 8 + x : d;
        mt = i - d * p.MT;
      }
      if (g >= p.G || mt >= p.MT) continue;
      if (mt < 0 || seen[(size_t)g * p.MT + mt]) return fail("a tile computed twice");
      seen[(size_t)g * p.MT + mt] = 1;
      ++n;
    }
    check(n == seen.size(), "a tile nobody computes");
    check((int64_t)p.MT * rows >= p.M && (int64_t)(p.MT - 1) * rows < p.M, "pixel tiles do not fit the output");
    check(p.G == p.NTn * p.splitk, "weight groups");
    divides(p.mg_wo, (uint64_t)p.Wo, (uint64_t)p.M + 64);
  }
  // rows: pixels of a tile; at: a layer's convolution, whose pixels come from `from`
  void conv(const ConvArgs& p, uint32_t groups, int rows, int from = -1) {
    const int l = layer_of_weights(p.w);
    const LayerPlan& L = net.layers[l];
    tiles(p, groups, rows);
    if (p.c_real == 0) reads(p.x, from >= 0 ? from : L.in_t, bytes(from >= 0 ? from : L.in_t));
    if (p.splitk > 1) {
      check((uint64_t)(uintptr_t)p.ws == kWorkspace && (size_t)p.splitk * p.M * p.Cout * 4 <= net.ws_bytes, "workspace");
      return;
    }
    if (p.res) reads(p.res, L.res_t, bytes(L.res_t));
    check((p.res != nullptr) == (L.res_t >= 0), "residual");
    const size_t sums = (size_t)L.cp.MT * p.Cout * 4;  // (the sums of a tile's pixels in place of its outputs)
    writes(p.y, l + 1, p.act & kActSumPixels ? sums : bytes(l + 1));
  }

  void launch(int l, const KernelLaunch& k) {
    const std::string& name = g_names[k.k];
    const std::string base = name.substr(0, name.find('<'));
    where = "layer " + std::to_string(l) + ", " + name;
    check(k.groups > 0 && k.threads > 0 && k.threads % 64 == 0 && k.threads <= 1024, "geometry");
    ConvArgs p;
    std::memcpy(&p, k.args, sizeof p);
    if (base == "ingest_kernel" || base == "egress_kernel") {
      const void* at[2];
      std::memcpy(at, k.args, sizeof at);
      if (base == "ingest_kernel") writes(at[1], 0, bytes(0));
      else reads(at[0], (int)net.layers.size(), bytes((int)net.layers.size()));
      return done();
    }
    const LayerPlan& L = net.layers[l];
    if (base == "conv_chain_kernel") {
      ChainArgs c;
      std::memcpy(&c, k.args + sizeof p, sizeof c);
      const int wide = L.follows >= 0 ? L.follows : l, first = net.layers[wide].joins;
      check(layer_of_weights(p.w) == first && layer_of_weights(c.w3) == wide, "weights");
      tiles(p, k.groups, 32);
      reads(p.x, net.layers[first].in_t, bytes(net.layers[first].in_t));
      check((c.res3 != nullptr) == (net.layers[wide].res_t >= 0), "residual");
      if (c.res3) reads(c.res3, net.layers[wide].res_t, bytes(net.layers[wide].res_t));
      writes(c.y3, wide + 1, bytes(wide + 1));
      check((c.n1 > 0) == (wide != l) && c.n1 <= 64, "the second 1x1");
      if (c.n1) {
        check(layer_of_weights(c.w1) == l && L.in_t == wide + 1, "the second 1x1");
        writes(c.y1, l + 1, (size_t)p.M * c.n1 * es());
      }
    } else if (base == "conv_expand_dw_kernel") {
      ExpandDwArgs e;
      std::memcpy(&e, k.args, sizeof e);
      check(k.groups == (uint32_t)(e.bands * (e.C / 16)) && e.C % 16 == 0 && e.threads == (int)k.threads && k.threads >= 64 && k.threads <= 512, "workgroups");
      check((int64_t)e.bands * e.band >= e.Ho && (int64_t)(e.bands - 1) * e.band < e.Ho, "bands");
      check((int64_t)((e.band - 1) * e.stride + 3) * e.W <= kExpandPixels, "a band's pixels do not fit LDS");
      divides(e.mg_bands, e.bands, k.groups);
      divides(e.mg_w, e.W, (uint64_t)e.H * e.W + 16);
      divides(e.mg_wo, e.Wo, (uint64_t)e.band * e.Wo);
      reads(e.x, net.layers[L.joins].in_t, bytes(net.layers[L.joins].in_t));
      writes(e.y, l + 1, (size_t)e.Ho * e.Wo * e.C * es());
    } else if (base == "conv_image_pool_kernel" || base == "conv_image_kernel") {
      ImageConvArgs m;
      std::memcpy(&m, k.args, sizeof m);
      const bool pool = base == "conv_image_pool_kernel";
      const int wn = pool || name.find("2>") != std::string::npos ? 2 : 1, nb = (m.Cout + 31) / 32;
      const int high = pool ? kImagePoolRows : 8 / wn, wide = pool ? kImagePoolCols : kImageCols, Ho = pool ? m.pool_h : m.Ho, Wo = pool ? m.pool_w : m.Wo;
      check(nb % wn == 0 && k.groups == (uint32_t)m.tiles * (nb / wn) && m.across == (Wo + wide - 1) / wide && m.tiles == m.across * ((Ho + high - 1) / high), "tiles");
      const int rows = pool ? 2 * kImagePoolRows + 2 : 8 / wn;
      check(m.patch_w == (kImageCols - 1) * m.stride + m.k && m.patch == ((rows - 1) * m.stride + m.k) * m.patch_w && ((rows - 1) * m.stride + m.k) * m.pitch <= (pool ? kImagePoolPatch : kImagePatch), "patch");
      check(k.threads == (pool ? 128u * (kImagePoolRows + 1) : 256u), "threads");
      divides(m.mg_tiles, m.tiles, k.groups);
      divides(m.mg_across, m.across, m.tiles);
      check(m.x == nullptr, "input");
      writes(m.y, l + 1, (size_t)Ho * Wo * m.Cout * es());
    } else if (base == "conv_block_pool_kernel") {
      const LayerPlan& O = net.layers[L.joins];
      check(layer_of_weights(p.w) == L.joins && p.Ho % 2 == 0 && p.Wo % 2 == 0 && p.splitk == 1 && !p.res, "pooled tiles");
      tiles(p, k.groups, 64);
      reads(p.x, O.in_t, bytes(O.in_t));
      writes(p.y, l + 1, (size_t)(p.Ho / 2) * (p.Wo / 2) * p.Cout * es());
    } else if (base == "fc_pooled_kernel") {
      FcPooledArgs f;
      std::memcpy(&f, k.args, sizeof f);
      const LayerPlan& B = net.layers[L.in_t - 1];
      const int from = B.lonely ? L.in_t : B.average_of + 1;
      check(f.tiles >= 1 && f.tiles <= kPooledTiles && f.K <= kPooledInputs && f.pixels == (B.lonely ? 1 : net.tensor(from).H * net.tensor(from).W), "sums");
      check(k.groups * kPooledRows >= (uint32_t)f.Ns && k.threads == 64 * kPooledRows, "rows");
      reads(f.x, from, (size_t)f.tiles * f.K * 4);
      if (f.y) writes(f.y, l + 1, (size_t)f.Ns * es());
      check((f.y == nullptr) == (l + 1 == (int)net.layers.size()), "logits");
    } else if (base == "gavgpool_kernel" && L.lonely) {
      PoolArgs a;
      std::memcpy(&a, k.args, sizeof a);
      reads(a.x, L.in_t, (size_t)a.H * a.C * 4);
      writes(a.y, l + 1, (size_t)a.C * 4);
    } else if (base == "gavgpool_kernel" || base == "maxpool_kernel" || base == "maxpool_window_kernel") {
      PoolArgs a;
      std::memcpy(&a, k.args, sizeof a);
      reads(a.x, L.in_t, bytes(L.in_t));
      writes(a.y, l + 1, bytes(l + 1));
    } else if (base == "dwconv_kernel" || base == "dwconv_window_kernel") {
      DwArgs a;
      std::memcpy(&a, k.args, sizeof a);
      reads(a.x, L.in_t, bytes(L.in_t));
      writes(a.y, l + 1, bytes(l + 1));
    } else if (base == "fc_kernel") {
      FcArgs f;
      std::memcpy(&f, k.args, sizeof f);
      reads(f.x, L.in_t, bytes(L.in_t));
      if (f.y) writes(f.y, l + 1, (size_t)f.Ns * es());
    } else if (base == "splitk_reduce_kernel") {
      struct { const float* ws; const float* bias; const void* res; void* y; int M, N, splitk, act; } r;
      std::memcpy(&r, k.args, sizeof r);
      const int at = layer_of_bias(r.bias);
      if (r.res) reads(r.res, net.layers[at].res_t, bytes(net.layers[at].res_t));
      writes(r.y, at + 1, bytes(at + 1));
    } else if (base == "conv_wave_pair_kernel" || base == "conv_wave16_pair_kernel" || base == "conv_point_pair_kernel") {
      ConvArgs q;
      int n0;
      std::memcpy(&q, k.args + sizeof p, sizeof q);
      std::memcpy(&n0, k.args + 2 * sizeof p, sizeof n0);
      const int rows = base == "conv_wave16_pair_kernel" || name.find(", 16, ") != std::string::npos ? 16 : 32;
      check(n0 % 8 == 0 && n0 < (int)k.groups, "the second problem's workgroups");
      conv(p, (uint32_t)n0, rows);
      conv(q, k.groups - (uint32_t)n0, rows);
    } else if (base == "conv_wave_dw_kernel") {
      conv(p, k.groups, 32, net.layers[L.pair_with].in_t);
    } else {
      const int rows = base == "conv_block_kernel" ? 64 : base == "conv_taps16_tall_kernel" ? 32 : base == "conv_wave16_kernel" || base == "conv_taps16_kernel" || (base == "conv_point_kernel" && name.find(", 16, ") != std::string::npos) ? 16 : 32;
      conv(p, k.groups, rows);
    }
    done();
  }
};

}  // namespace

int main() {
  AqlRuntime rt;
  KernelTable kt;
  JoinedTable joined;
  std::string missing = kt.resolve(rt);
  if (missing.empty()) missing = joined.resolve(rt);
  if (!missing.empty()) {
    std::fprintf(stderr, "kernel %s\n", missing.c_str());
    return 2;
  }
  daris_dnn d;
  int cus, stages, n, dtype;
  while (std::scanf("%d %d %d %d %d %d %d", &dtype, &d.in_c, &d.in_h, &d.in_w, &cus, &stages, &n) == 7) {
    std::vector<daris_layer> layers(n);
    for (daris_layer& L : layers) {
      std::memset(&L, 0, sizeof L);
      if (std::scanf("%d %d %d %d %d %d %d %d %d %d", &L.op, &L.c_in, &L.c_out, &L.k, &L.stride, &L.pad, &L.groups, &L.act, &L.in_from, &L.res_from) != 10) return 3;
    }
    d.n_layers = n;
    d.dtype = dtype;
    d.layers = layers.data();
    NetPlan net;
    std::string err = build_plan(d, false, true, true, true, true, true, cus, &net);
    if (err.empty() && !split_stages(&net, std::min(stages, 1 + (int)net.legal_cuts.size()))) err = "stages";
    if (!err.empty()) {
      std::printf("bad %s\n", err.c_str());
      continue;
    }
    join_layers(&net);
    std::vector<void*> slots;
    for (size_t s = 0; s < net.slot_bytes.size(); ++s) slots.push_back((void*)(uintptr_t)((s + 1) * kSlot));
    for (int l = 0; l < n; ++l) {
      net.layers[l].w_dev = (void*)(uintptr_t)(kWeights + ((uint64_t)l << 32));
      net.layers[l].b_dev = (float*)(uintptr_t)(kBias + ((uint64_t)l << 32));
    }
    LaunchSeq seq;
    err = encode_network(net, false, kt, joined, slots, (float*)(uintptr_t)kWorkspace, &seq);
    Walk walk{net, std::vector<int>(slots.size(), -1), "", "", {}, {}};
    std::string out;
    if (err.empty()) {
      if (!net.fuse_ingest) walk.launch(0, seq.launches[0].kl);
      for (int l = 0; l < n && walk.bad.empty(); ++l)
        for (int i = seq.layer_lo[l]; i < seq.layer_lo[l + 1]; ++i) {
          const KernelLaunch& k = seq.launches[i].kl;
          out += " " + std::to_string(l) + ":" + g_names[k.k].substr(0, g_names[k.k].find('<')) + ":" + std::to_string(k.groups);
          walk.launch(l, k);
        }
      if (!net.final_direct && walk.bad.empty()) walk.launch(n, seq.launches.back().kl);
      for (size_t s = 0; s < net.stage_first.size(); ++s)
        if (seq.layer_lo[s + 1 < net.stage_first.size() ? net.stage_first[s + 1] : n] <= seq.layer_lo[net.stage_first[s]]) walk.fail("a stage without launches");
      err = walk.bad;
    }
    if (err.empty()) std::printf("ok%s\n", out.c_str());
    else std::printf("bad %s\n", err.c_str());
  }
  return 0;
}
