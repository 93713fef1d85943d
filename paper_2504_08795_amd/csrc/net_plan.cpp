#include "net_plan.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <limits>

namespace daris {

static inline int round_up(int a, int b) { return (a + b - 1) / b * b; }

uint16_t host_f32_to_bf16(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN
  u += 0x7fffu + ((u >> 16) & 1u);                                           // nearest, ties to even
  return (uint16_t)(u >> 16);
}

// f as the sum of three bf16 numbers, exact for every finite f of 2^-110 and more (and 0); below that up to 2^-134 is lost.
static void split_bf16(float f, uint16_t out[3]) {
  for (int p = 0; p < 3; ++p) {
    uint16_t h = host_f32_to_bf16(f);
    if ((h & 0x7fffu) == 0x7f80u && std::isfinite(f)) h -= 1;  // rounding up would overflow: the largest finite number
    const uint32_t u = (uint32_t)h << 16;
    float v;
    std::memcpy(&v, &u, 4);
    out[p] = h;
    f = std::isfinite(v) ? f - v : 0.f;
  }
}

std::string build_plan(const daris_dnn& dnn, bool keep_activations, bool pair_launches, bool fuse_ingest, bool staged_rows, bool small_tiles, bool fuse_dw,
                       int plan_cus, NetPlan* out, bool tall_tiles, bool join) {
  NetPlan& net = *out;
  net = NetPlan();
  if (dnn.n_layers < 1 || !dnn.layers) return "DNN has no layers";
  if (dnn.in_c < 1 || dnn.in_h < 1 || dnn.in_w < 1) return "bad input shape";
  if (dnn.dtype != DARIS_FP32 && dnn.dtype != DARIS_BF16) return "bad dtype";
  net.bf16 = dnn.dtype == DARIS_BF16;
  net.plan_cus = plan_cus;
  const int vec = net.bf16 ? 8 : 4, es = net.bf16 ? 2 : 4;
  net.in_c = dnn.in_c;
  net.in_h = dnn.in_h;
  net.in_w = dnn.in_w;
  net.ingest.C = dnn.in_c;
  net.ingest.Cs = round_up(dnn.in_c, vec);
  net.ingest.H = dnn.in_h;
  net.ingest.W = dnn.in_w;
  net.ingest.bytes = (size_t)net.ingest.H * net.ingest.W * net.ingest.Cs * es;
  const int n = dnn.n_layers;
  net.layers.resize(n);
  auto rows_taken = [&](const LayerPlan& L) {
    const TensorInfo& in = net.tensor(L.in_t);
    return conv_rows_take(in.H, in.W, in.Cs, (uint64_t)L.out.H * (uint64_t)L.out.W, L.out.Cs, L.Kpad, net.bf16);
  };
  auto rows_taken_large = [&](const LayerPlan& L) {
    const TensorInfo& in = net.tensor(L.in_t);
    return conv_rows_take_large(in.H, in.W, in.Cs, L.out.W, L.out.Cs, L.d.k, L.d.stride, L.Kpad, net.bf16);
  };
  // the channel stride that lets plan_conv choose 16-pixel tiles, which only whole 64-byte rows feed; 0: it may not
  auto small_tile_stride = [&](const LayerPlan& L) { return small_tiles && rows_taken(L) ? net.tensor(L.in_t).Cs : 0; };

  for (int l = 0; l < n; ++l) {
    LayerPlan& L = net.layers[l];
    L.d = dnn.layers[l];
    L.d.w = nullptr;
    L.d.b = nullptr;
    const daris_layer& d = L.d;
    if (d.in_from < -1 || d.in_from >= l) return "layer " + std::to_string(l) + ": in_from must name an earlier layer or -1";
    if (d.res_from < -1 || d.res_from >= l) return "layer " + std::to_string(l) + ": res_from must name an earlier layer or -1";
    L.in_t = d.in_from + 1;
    L.res_t = d.res_from < 0 ? -1 : d.res_from + 1;
    const TensorInfo& in = net.tensor(L.in_t);
    TensorInfo& o = L.out;
    switch (d.op) {
      case DARIS_OP_CONV: {
        if (d.c_in != in.C) return "layer " + std::to_string(l) + ": c_in does not match its input";
        if (d.k < 1 || d.stride < 1 || d.pad < 0 || d.c_out < 1) return "layer " + std::to_string(l) + ": bad conv geometry";
        L.depthwise = d.groups != 1;
        if (L.depthwise && !(d.groups == d.c_in && d.c_in == d.c_out))
          return "layer " + std::to_string(l) + ": only dense (groups=1) and depthwise (groups=c_in=c_out) convolutions";
        o.C = d.c_out;
        o.Cs = round_up(d.c_out, vec);
        o.H = (in.H + 2 * d.pad - d.k) / d.stride + 1;
        o.W = (in.W + 2 * d.pad - d.k) / d.stride + 1;
        if (o.H < 1 || o.W < 1) return "layer " + std::to_string(l) + ": empty output";
        L.macs = (int64_t)o.H * o.W * d.c_out * (d.c_in / d.groups) * d.k * d.k;
        if (!L.depthwise) {
          L.K = d.k * d.k * in.Cs;
          L.Kpad = round_up(L.K, 16);  // what one matrix instruction takes: one K step (bf16), two (fp32)
          // the kernels divide pixel and k indices by Wo, Cin and kw with 32-bit multipliers: operands must stay small
          if ((uint64_t)(o.H * (uint64_t)o.W + 64) * (uint64_t)o.W >= (1ull << 32) || (uint64_t)(L.Kpad + 64) * (uint64_t)in.Cs >= (1ull << 32))
            return "layer " + std::to_string(l) + ": tensor too large for the kernels' index arithmetic";
          L.cp = plan_conv(o.H * o.W, o.Cs, L.Kpad, net.bf16, staged_rows && conv_rows_staged(in.Cs, net.bf16) ? 2 : 1, small_tile_stride(L), plan_cus,
                           conv_block_takes(in.H, in.W, in.Cs, d.k, d.pad, L.Kpad),
                           !staged_rows || !conv_three_taps(d.k, d.stride, d.pad) ? kNoTaps : rows_taken(L) ? kTaps : rows_taken_large(L) ? kTapsLarge : kNoTaps);
          net.ws_bytes = std::max(net.ws_bytes, L.cp.ws_bytes);
        } else {
          L.kernel_id = K_DWCONV;
        }
        break;
      }
      case DARIS_OP_MAXPOOL:
        if (d.k < 1 || d.stride < 1 || d.pad < 0 || 2 * d.pad > d.k) return "layer " + std::to_string(l) + ": bad pool geometry";
        o.C = in.C;
        o.Cs = in.Cs;
        o.H = (in.H + 2 * d.pad - d.k) / d.stride + 1;
        o.W = (in.W + 2 * d.pad - d.k) / d.stride + 1;
        if (o.H < 1 || o.W < 1) return "layer " + std::to_string(l) + ": empty output";
        L.kernel_id = K_MAXPOOL;
        break;
      case DARIS_OP_GAVGPOOL:
        o.C = in.C;
        o.Cs = in.Cs;
        o.H = o.W = 1;
        L.kernel_id = K_GAVGPOOL;
        break;
      case DARIS_OP_FC:
        if (d.c_in != in.C * in.H * in.W) return "layer " + std::to_string(l) + ": FC c_in must equal C*H*W of its input";
        if (d.c_out < 1) return "layer " + std::to_string(l) + ": bad FC size";
        o.C = d.c_out;
        o.Cs = round_up(d.c_out, vec);
        o.H = o.W = 1;
        L.macs = (int64_t)d.c_in * d.c_out;
        L.K = in.H * in.W * in.Cs;
        L.Kpad = L.K;
        L.kernel_id = K_FC;
        break;
      default:
        return "layer " + std::to_string(l) + ": unknown op";
    }
    if (d.act < DARIS_ACT_NONE || d.act > DARIS_ACT_RELU6) return "layer " + std::to_string(l) + ": unknown activation";
    if (L.res_t >= 0) {
      const TensorInfo& r = net.tensor(L.res_t);
      if (d.op != DARIS_OP_CONV || L.depthwise) return "layer " + std::to_string(l) + ": residual only on dense convolutions";
      if (r.C != o.C || r.H != o.H || r.W != o.W) return "layer " + std::to_string(l) + ": residual shape mismatch";
    }
    o.bytes = (size_t)o.H * o.W * o.Cs * es;
  }
  // Launch pairs (a residual block's first convolution and its shortcut convolution).  A pair saves one launch and its gap; the
  // kernel for pairs has no 64 x 64 tiles, so a heavy member that has them gives them up.  All kernels of a network with
  // pairs and without, on 128 CUs: ResNet-18 fp32 109.0 us / 115.5, bf16 (192 CUs) 62.9 / 68.4; ResNet-50 bf16 161.8 / 169.3, fp32 270.9 /
  // 275.8, and on 64 CUs, where a heavy member gives its 64 x 64 tiles up, 427.0 / 433.9.
  for (int l = 0; l + 1 < n && pair_launches; ++l) {
    LayerPlan& A = net.layers[l];
    LayerPlan& B = net.layers[l + 1];
    if (A.d.op != DARIS_OP_CONV || B.d.op != DARIS_OP_CONV || A.depthwise || B.depthwise) continue;
    if (A.in_t != B.in_t || B.res_t == l + 1) continue;
    if (conv_rows_staged(net.tensor(A.in_t).Cs, net.bf16) && (!rows_taken(A) || !rows_taken(B))) continue;  // large tensors: a launch matters little, fetching them in rows does
    LayerPlan& heavy = A.macs > B.macs ? A : B;
    LayerPlan& light = A.macs > B.macs ? B : A;
    const ConvPlan own = heavy.cp;
    const int sa = staged_rows && conv_rows_staged(net.tensor(heavy.in_t).Cs, net.bf16) ? 2 : 1;
    if (heavy.cp.rows == 64 || heavy.cp.gather == kGatherTaps)  // (kernels that have no form for two problems)
      heavy.cp = plan_conv(heavy.out.H * heavy.out.W, heavy.out.Cs, heavy.Kpad, net.bf16, sa, small_tile_stride(heavy), plan_cus, false);
    const int sb = staged_rows && conv_rows_staged(net.tensor(light.in_t).Cs, net.bf16) ? 2 : 1;
    ConvPlan like = plan_conv_like(heavy.cp, light.out.H * light.out.W, light.out.Cs, light.Kpad, net.bf16, sb, plan_cus);
    heavy.cp = plan_conv_beside(heavy.cp, like, heavy.out.H * heavy.out.W, heavy.out.Cs, heavy.Kpad, net.bf16, sa, plan_cus);
    like = plan_conv_like(heavy.cp, light.out.H * light.out.W, light.out.Cs, light.Kpad, net.bf16, sb, plan_cus);
    if (like.kernel == K_NONE || (like.rows == 16 && small_tile_stride(light) == 0)) {
      heavy.cp = own;
      continue;
    }
    net.ws_bytes = std::max(net.ws_bytes, heavy.cp.ws_bytes);
    light.cp = like;
    A.pair_with = l + 1;
    B.pair_with = l;
    B.pair_lead = true;
    ++l;
  }
  // depthwise 3x3 + the 1x1 convolution that alone reads it: one launch, the depthwise output is never stored
  for (int l = 0; l + 1 < n && fuse_dw && staged_rows && !keep_activations; ++l) {
    LayerPlan& A = net.layers[l];
    LayerPlan& B = net.layers[l + 1];
    if (A.d.op != DARIS_OP_CONV || !A.depthwise || A.d.k != 3 || A.d.pad != 1 || (A.d.stride != 1 && A.d.stride != 2)) continue;
    if (B.d.op != DARIS_OP_CONV || B.depthwise || B.d.k != 1 || B.d.stride != 1 || B.d.pad != 0 || B.in_t != l + 1 || B.pair_with >= 0) continue;
    bool only_reader = true;
    for (int q = l + 2; q < n; ++q)
      if (net.layers[q].in_t == l + 1 || net.layers[q].res_t == l + 1) only_reader = false;
    if (!only_reader || !conv_rows_staged(A.out.Cs, net.bf16)) continue;
    ConvPlan cp = B.cp;
    if (cp.rows != 32)  // the fused producer exists for 32-pixel tiles
      cp = plan_conv(B.out.H * B.out.W, B.out.Cs, B.Kpad, net.bf16, 2, 0, plan_cus, false);
    if (!conv_dw_fusable(cp, net.bf16)) continue;  // the separate launch is faster (or no such kernel variant)
    B.cp = cp;
    net.ws_bytes = std::max(net.ws_bytes, cp.ws_bytes);
    A.pair_with = l + 1;
    B.pair_with = l;
    B.pair_lead = true;
    A.fused_dw = B.fused_dw = true;
    A.fusable_dw = B.fusable_dw = true;
    ++l;
  }
  // Layer 0 can gather straight from the caller's input when that is its only reader and one filter tap is exactly
  // one 16-byte vector of the padded layout (1..4 real channels).
  {
    const LayerPlan& L0 = net.layers[0];
    bool only_reader = true;
    for (int l = 1; l < n; ++l)
      if (net.layers[l].in_t == 0 || net.layers[l].res_t == 0) only_reader = false;
    net.fuse_ingest = !keep_activations && fuse_ingest && (uint64_t)dnn.in_c * dnn.in_h * dnn.in_w * 4 < (1ull << 31) && L0.d.op == DARIS_OP_CONV && !L0.depthwise &&
                      L0.in_t == 0 && L0.res_t < 0 && L0.pair_with < 0 && only_reader && net.ingest.Cs == vec && dnn.in_c <= 4;
  }
  // how each dense convolution comes by its pixels, which the layers' links decide too
  for (int l = 0; l < n; ++l) {
    LayerPlan& L = net.layers[l];
    if (L.d.op != DARIS_OP_CONV || L.depthwise) continue;
    const bool joint = L.pair_with >= 0 && !net.layers[L.pair_with].depthwise;
    if (l == 0 && net.fuse_ingest) plan_input(&L.cp, L.out.H, L.out.W, L.out.Cs, L.d.k, L.d.stride, plan_cus, net.bf16);
    else if (joint) plan_gather(&L.cp, net.tensor(L.in_t).Cs, rows_taken(L) && rows_taken(net.layers[L.pair_with]) && net.layers[L.pair_with].cp.staged, net.bf16);
    else plan_gather(&L.cp, net.tensor(L.in_t).Cs, rows_taken(L) || (L.cp.rows == 32 && L.cp.nw == 2 && rows_taken_large(L)), net.bf16);
    L.kernel_id = L.cp.kernel;
    L.tall = tall_tiles && tall_takes(L.cp, L.out.H * L.out.W, plan_cus) && rows_taken(L);
  }
  // layers that join the one in front, which nobody else reads
  for (int l = 0; l + 1 < n && !keep_activations && join; ++l) {
    LayerPlan& A = net.layers[l];
    LayerPlan& B = net.layers[l + 1];
    if (A.d.op != DARIS_OP_CONV || A.depthwise || A.pair_with >= 0 || B.in_t != l + 1 || B.pair_with >= 0) continue;
    bool only_reader = true;
    for (int q = l + 2; q < n; ++q)
      if (net.layers[q].in_t == l + 1 || net.layers[q].res_t == l + 1) only_reader = false;
    if (!only_reader) continue;
    if (B.d.op == DARIS_OP_MAXPOOL) {
      if (B.d.k == 3 && B.d.stride == 2 && B.d.pad == 1 && image_pool_takes(A.cp, A.out.H, A.out.W, A.out.Cs, A.d.k, A.d.stride, plan_cus, net.bf16)) B.can_join = l;
      if (B.d.k == 2 && B.d.stride == 2 && B.d.pad == 0 && A.res_t < 0 && block_pool_takes(A.cp, A.out.H, A.out.W)) B.can_join = l;
    } else if (B.d.op == DARIS_OP_CONV && B.depthwise && staged_rows && small_tiles) {
      if (B.d.k == 3 && B.d.pad == 1 && (B.d.stride == 1 || B.d.stride == 2) && A.d.k == 1 && A.d.stride == 1 && A.d.pad == 0 && A.res_t < 0 && rows_taken(A) && !(l == 0 && net.fuse_ingest) &&
          plan_expand_dw(&A.cp, A.out.H, A.out.W, net.tensor(A.in_t).Cs, A.out.Cs, A.Kpad, B.d.stride, plan_cus, net.bf16)) {
        if (fuse_dw) B.can_join = l;
        // (Launches of their own have this plan too and give the same sums.  Parted, the convolution takes, against the plan that it would have alone, -0.6 to 0.5 us in fp32,
        // faster in 80 of 82 random layers whose plans differ, and -0.5 to 0.5 in bf16, slower by more than 0.1 in 12 of 159.)
        A.kernel_id = A.cp.kernel;
      }
    }
  }
  // convolution, global average pooling and FC layer, which nobody else reads
  for (int l = 0; l + 2 < n && !keep_activations && join; ++l) {
    LayerPlan& A = net.layers[l];
    LayerPlan& B = net.layers[l + 1];
    LayerPlan& C = net.layers[l + 2];
    if (A.d.op != DARIS_OP_CONV || A.depthwise || A.pair_with >= 0 || B.d.op != DARIS_OP_GAVGPOOL || B.in_t != l + 1 || C.d.op != DARIS_OP_FC || C.in_t != l + 2) continue;
    bool only_reader = true;
    for (int q = l + 2; q < n; ++q)
      if (net.layers[q].in_t == l + 1 || net.layers[q].res_t == l + 1 || (q > l + 2 && net.layers[q].in_t == l + 2) || net.layers[q].res_t == l + 2) only_reader = false;
    if (!only_reader || !rows_taken(A) || !sums_pixels(A.cp, A.out.Cs)) continue;
    A.sums_pixels = true;
    A.pair_with = l + 2;
    A.out.bytes = std::max(A.out.bytes, (size_t)A.cp.MT * A.out.Cs * 4);
    B.out.bytes = std::max(B.out.bytes, (size_t)B.out.Cs * 4);
    B.average_of = l;
    B.kernel_id = A.kernel_id;
  }
  // a 3x3 convolution, the 1x1 that alone reads it, and the 1x1 behind that
  for (int l = 0; l + 1 < n && !keep_activations && staged_rows && join; ++l) {
    LayerPlan& A = net.layers[l];
    LayerPlan& B = net.layers[l + 1];
    auto plain = [&](const LayerPlan& L) { return L.d.op == DARIS_OP_CONV && !L.depthwise && L.pair_with < 0 && L.can_join < 0 && !L.sums_pixels && rows_taken(L); };
    auto point = [&](const LayerPlan& L) { return plain(L) && L.d.k == 1 && L.d.stride == 1 && L.d.pad == 0; };
    if (!plain(A) || A.res_t >= 0 || (l == 0 && net.fuse_ingest) || !point(B) || B.in_t != l + 1 || B.res_t == l + 1 || !chain_takes(A.cp, A.out.Cs, B.cp, B.out.Cs, nullptr, net.bf16)) continue;
    bool only_reader = true;
    for (int q = l + 2; q < n; ++q)
      if (net.layers[q].in_t == l + 1 || net.layers[q].res_t == l + 1) only_reader = false;
    if (!only_reader) continue;
    B.can_join = l;
    if (l + 2 >= n) break;
    LayerPlan& C = net.layers[l + 2];
    if (point(C) && C.in_t == l + 2 && C.res_t < 0 && C.out.Cs <= 64 && chain_takes(A.cp, A.out.Cs, B.cp, B.out.Cs, &C.cp, net.bf16)) C.can_follow = l + 1;
  }
  const TensorInfo& fin = net.layers[n - 1].out;
  net.n_out = fin.C * fin.H * fin.W;
  net.final_direct = net.layers[n - 1].d.op == DARIS_OP_FC;

  // legal cuts: after layer l, when every later layer reads only tensors produced at or after l
  for (int l = 0; l + 1 < n; ++l) {
    bool ok = true;
    for (int q = l + 1; q < n && ok; ++q) {
      const daris_layer& d = net.layers[q].d;
      if (d.in_from < l) ok = false;
      if (d.res_from >= 0 && d.res_from < l) ok = false;
    }
    if (ok) net.legal_cuts.push_back(l);
  }
  net.stage_first.assign(1, 0);
  join_layers(&net);

  // activation slots: a tensor's slot is free again once its last reader has been issued (same stream, in order)
  // The earlier member of a launch pair is issued with the later one (and its split-K reduction after that launch):
  // what it reads must stay in place until then, so its reads count as reads of the later layer; and what it writes, read or not,
  // must not be given to the later member.
  std::vector<int> last_use(n + 1, -1);
  for (int l = 0; l < n; ++l) {
    const LayerPlan& L = net.layers[l];
    int at = net.joined_away(l) ? l + 1 : std::max(l, L.pair_with);
    if (net.followed(at)) ++at;
    last_use[l + 1] = std::max(last_use[l + 1], at);
    last_use[L.in_t] = std::max(last_use[L.in_t], at);
    if (L.res_t >= 0) last_use[L.res_t] = std::max(last_use[L.res_t], at);
  }
  std::vector<int> slot_owner;  // tensor currently held by each slot, -1 = free
  auto take_slot = [&](int tensor, size_t bytes) {
    int s = -1;
    if (!keep_activations)
      for (size_t i = 0; i < slot_owner.size(); ++i)
        if (slot_owner[i] < 0) { s = (int)i; break; }
    if (s < 0) {
      slot_owner.push_back(-1);
      net.slot_bytes.push_back(0);
      s = (int)slot_owner.size() - 1;
    }
    slot_owner[s] = tensor;
    net.slot_bytes[s] = std::max(net.slot_bytes[s], bytes);
    return s;
  };
  net.ingest.slot = take_slot(0, net.ingest.bytes);
  for (int l = 0; l < n; ++l) {
    for (size_t i = 0; i < slot_owner.size(); ++i)
      if (slot_owner[i] >= 0 && last_use[slot_owner[i]] < l) slot_owner[i] = -1;
    if (l == n - 1 && net.final_direct) break;  // logits go straight to the caller's buffer
    net.layers[l].out.slot = take_slot(l + 1, net.layers[l].out.bytes);
  }
  return "";
}

bool join_layers(NetPlan* net) {
  bool changed = false;
  for (int l = 0; l + 1 < (int)net->layers.size(); ++l) {
    LayerPlan& A = net->layers[l];
    LayerPlan& B = net->layers[l + 1];
    const bool cut = std::find(net->stage_first.begin(), net->stage_first.end(), l + 1) != net->stage_first.end();
    // A depthwise layer is computed inside the next layer's launch only while both lie in one stage: a cut between them makes
    // the depthwise layer's output the tensor that crosses the boundary (and a stage of that layer alone would have no launch).
    if (A.fusable_dw && A.depthwise && A.fused_dw == cut) {
      A.fused_dw = B.fused_dw = !cut;
      A.pair_with = cut ? -1 : l + 1;
      B.pair_with = cut ? -1 : l;
      B.pair_lead = !cut;
      changed = true;
    }
    // ... and so with the layers that are computed in the next one's launch.
    if (B.can_join == l && (B.joins == l) == cut) {
      const bool pool = B.d.op == DARIS_OP_MAXPOOL;
      B.joins = cut ? -1 : l;
      if (pool && A.cp.rows != 64) A.pair_with = cut ? -1 : l + 1;  // (64-pixel tiles: what a plan says is the same with the cut and without)
      if (pool && A.cp.rows != 64) B.kernel_id = cut ? (int32_t)K_MAXPOOL : K_IMAGE_POOL_F32 + net->bf16;
      if (B.depthwise) B.kernel_id = cut ? (int32_t)K_DWCONV : K_EXPAND_DW_F32 + net->bf16;  // (a dense convolution keeps the name of the plan whose sums it has)
      changed = true;
    }
    const bool follows = B.can_follow == l && A.joins >= 0 && !cut;
    if (follows != (B.follows >= 0)) {
      B.follows = follows ? l : -1;
      changed = true;
    }
  }
  for (int l = 0; l + 1 < (int)net->layers.size(); ++l) {
    LayerPlan& B = net->layers[l];
    if (B.average_of < 0) continue;
    auto starts = [&](int q) { return std::find(net->stage_first.begin(), net->stage_first.end(), q) != net->stage_first.end(); };
    const bool lonely = starts(l) && starts(l + 1);
    if (B.lonely != lonely) changed = true;
    B.lonely = lonely;
    B.kernel_id = lonely ? (int32_t)K_GAVGPOOL : net->layers[B.average_of].kernel_id;
  }
  return changed;
}

bool split_stages(NetPlan* net, int k) {
  const int n = (int)net->layers.size();
  if (k < 1 || k - 1 > (int)net->legal_cuts.size()) return false;
  std::vector<int64_t> pre(n + 1, 0);
  for (int l = 0; l < n; ++l) pre[l + 1] = pre[l] + net->layers[l].macs;
  auto sum = [&](int a, int b) { return pre[b + 1] - pre[a]; };  // layers a..b inclusive
  const int64_t INF = std::numeric_limits<int64_t>::max();
  std::vector<char> legal(n, 0);
  for (int c : net->legal_cuts) legal[c] = 1;
  // f[r][s]: least possible largest-stage MACs when layers s..n-1 form r stages
  std::vector<std::vector<int64_t>> f(k + 1, std::vector<int64_t>(n + 1, INF));
  for (int s = 0; s < n; ++s) f[1][s] = sum(s, n - 1);
  for (int r = 2; r <= k; ++r)
    for (int s = 0; s < n; ++s)
      for (int c = s; c + 1 < n; ++c) {
        if (!legal[c] || f[r - 1][c + 1] == INF) continue;
        f[r][s] = std::min(f[r][s], std::max(sum(s, c), f[r - 1][c + 1]));
      }
  const int64_t best = f[k][0];
  if (best == INF) return false;
  std::vector<int> first(1, 0);
  int pos = 0;
  for (int r = k; r >= 2; --r) {
    int chosen = -1;
    for (int c = pos; c + 1 < n; ++c) {
      if (!legal[c] || f[r - 1][c + 1] == INF) continue;
      if (std::max(sum(pos, c), f[r - 1][c + 1]) <= best) { chosen = c; break; }
    }
    if (chosen < 0) return false;
    pos = chosen + 1;
    first.push_back(pos);
  }
  net->stage_first = first;
  return true;
}

template <typename T>
static void put(std::vector<unsigned char>* buf, size_t idx, float v, bool bf16) {
  if (bf16) reinterpret_cast<uint16_t*>(buf->data())[idx] = host_f32_to_bf16(v);
  else reinterpret_cast<float*>(buf->data())[idx] = v;
}

void pack_conv(const NetPlan& net, const LayerPlan& L, const float* w, const float* b, std::vector<unsigned char>* wp,
               std::vector<float>* bp) {
  const daris_layer& d = L.d;
  const TensorInfo& in = net.tensor(L.in_t);
  const bool bf = net.bf16;
  const size_t es = bf ? 2 : 4;
  const int kk = d.k * d.k;
  bp->assign(L.out.Cs, 0.f);
  if (b)
    for (int o = 0; o < d.c_out; ++o) (*bp)[o] = b[o];
  if (L.depthwise) {
    // [tap][C]
    wp->assign((size_t)kk * in.Cs * es, 0);
    for (int c = 0; c < d.c_out; ++c)
      for (int t = 0; t < kk; ++t) put<float>(wp, (size_t)t * in.Cs + c, w[(size_t)c * kk + t], bf);
    return;
  }
  // Where weight (tap t, channel ci) lies along K: tap by tap, or, where a fetch of rows serves three taps, chunk by chunk in the order
  // (ky, channels of a chunk, kx)
  const int per_chunk = (L.cp.rows == 16 ? 128 : 64) / (int)es;
  auto k_of = [&](int t, int ci) { return L.cp.gather == kGatherTaps ? ((t / 3 * (in.Cs / per_chunk) + ci / per_chunk) * 3 + t % 3) * per_chunk + ci % per_chunk : t * in.Cs + ci; };
  if (!bf) {
    // fp32: three bf16 parts per weight (see split8 in device_common.h), [channel block of R][chunk][part][lane = i + R q][8],
    // element e of lane (i, q) in chunk s is W[n = R nb + i][k = s * CK + 8 q + e]; a chunk is what one matrix instruction
    // takes, CK = 16 (R = 32) or 32 (R = 16)
    const int R = L.cp.rows == 16 ? 16 : 32, ck = R == 16 ? 32 : 16, nch = L.Kpad / ck;
    const int nblocks = (L.out.Cs + R - 1) / R;
    const int nb_alloc = (nblocks + L.cp.tn - 1) / L.cp.tn * L.cp.tn;
    wp->assign((size_t)nb_alloc * nch * 3 * 1024 + 12 * 1024, 0);  // + slack for refills past the last chunk (32- and 64-pixel tiles)
    uint16_t* out = reinterpret_cast<uint16_t*>(wp->data());
    for (int o = 0; o < d.c_out; ++o)
      for (int ci = 0; ci < d.c_in; ++ci)
        for (int t = 0; t < kk; ++t) {
          const int k = k_of(t, ci);
          const int s = k / ck, q = (k % ck) / 8, e = k % 8;
          const size_t at = ((size_t)(o / R) * nch + s) * 3 * 512 + (size_t)(o % R + R * q) * 8 + e;
          uint16_t part[3];
          split_bf16(w[((size_t)o * d.c_in + ci) * kk + t], part);
          for (int p = 0; p < 3; ++p) out[at + (size_t)p * 512] = part[p];
        }
    return;
  }
  if (L.cp.rows == 16) {
    // 16-row kernel: [channel block of 16][step][lane = j + 16 q][VEC], element e of lane (j, q) at step s is
    // W[n = 16 nb + j][k = s * 4 VEC + q * VEC + e], k = tap * Cs_in + ci; blocks padded to a multiple of TN
    const int vec = bf ? 8 : 4, ks = 4 * vec, S = L.cp.S;
    const int nblocks = (L.out.Cs + 15) / 16;
    const int nb_alloc = (nblocks + L.cp.tn - 1) / L.cp.tn * L.cp.tn;
    wp->assign((size_t)nb_alloc * S * 64 * 16, 0);  // (nothing is requested past the last step)
    for (int o = 0; o < d.c_out; ++o)
      for (int ci = 0; ci < d.c_in; ++ci)
        for (int t = 0; t < kk; ++t) {
          const int k = k_of(t, ci);
          const int st = k / ks, q = (k % ks) / vec, e = k % vec;
          const size_t lane = (size_t)(o % 16) + 16 * q;
          put<float>(wp, (((size_t)(o / 16) * S + st) * 64 + lane) * vec + e, w[((size_t)o * d.c_in + ci) * kk + t], bf);
        }
    return;
  }
  // [channel block of 32][step][lane = i + 32 h][VEC], element e of lane (i, h) at step s is
  // W[n = 32 nb + i][k = s*KS + h*VEC + e], k = tap * Cs_in + ci; blocks padded to a multiple of TN, zeros elsewhere
  const int vec = bf ? 8 : 4, ks = 2 * vec, S = L.cp.S;
  const int nblocks = (L.out.Cs + 31) / 32;
  const int nb_alloc = (nblocks + L.cp.tn - 1) / L.cp.tn * L.cp.tn;
  wp->assign((size_t)nb_alloc * S * 64 * 16 + 8 * 1024, 0);  // + slack for the kernel's pipeline refills past the last step
  for (int o = 0; o < d.c_out; ++o)
    for (int ci = 0; ci < d.c_in; ++ci)
      for (int t = 0; t < kk; ++t) {
        const int k = k_of(t, ci);
        const int st = k / ks, h = (k % ks) / vec, e = k % vec;
        const size_t lane = (size_t)(o % 32) + 32 * h;
        put<float>(wp, (((size_t)(o / 32) * S + st) * 64 + lane) * vec + e, w[((size_t)o * d.c_in + ci) * kk + t], bf);
      }
}

void pack_fc(const NetPlan& net, const LayerPlan& L, const float* w, const float* b, std::vector<unsigned char>* wp,
             std::vector<float>* bp) {
  const daris_layer& d = L.d;
  const TensorInfo& in = net.tensor(L.in_t);
  const bool bf = net.bf16;
  const size_t es = bf ? 2 : 4;
  const int hw = in.H * in.W;
  bp->assign(d.c_out, 0.f);
  if (b)
    for (int o = 0; o < d.c_out; ++o) (*bp)[o] = b[o];
  // [N][H*W*Cs]: caller order is (c, y, x); device tensors are (y, x, c) with channel stride Cs
  wp->assign((size_t)d.c_out * L.K * es, 0);
  for (int o = 0; o < d.c_out; ++o)
    for (int c = 0; c < in.C; ++c)
      for (int px = 0; px < hw; ++px)
        put<float>(wp, (size_t)o * L.K + (size_t)px * in.Cs + c, w[(size_t)o * d.c_in + (size_t)c * hw + px], bf);
}

}  // namespace daris
