// A network's plan as launches: which kernel each layer runs and with which arguments (host logic, no GPU needed).
#include "net_encode.h"

namespace daris {

static ConvArgs conv_args(const NetPlan& net, int l, bool wave_prio, void* y, const std::vector<void*>& slots, float* ws) {
  const LayerPlan& L = net.layers[l];
  const TensorInfo& in = net.tensor(L.in_t);
  ConvArgs a;
  a.x = slots[in.slot]; a.w = L.w_dev; a.bias = L.b_dev; a.y = y; a.ws = ws; a.wave_prio = wave_prio ? 1 : 0;
  a.res = L.res_t >= 0 ? slots[net.tensor(L.res_t).slot] : nullptr;
  a.H = in.H; a.W = in.W; a.Cin = in.Cs; a.Ho = L.out.H; a.Wo = L.out.W; a.Cout = L.out.Cs;
  a.kh = a.kw = L.d.k; a.stride = L.d.stride; a.pad = L.d.pad;
  a.Kpad = L.Kpad; a.M = L.out.H * L.out.W; a.act = L.d.act | (L.sums_pixels ? kActSumPixels : 0);
  a.splitk = L.cp.splitk; a.S = L.cp.S; a.sz = L.cp.sz; a.sw = L.cp.sw;
  a.MT = L.cp.MT; a.NTn = L.cp.NTn; a.G = L.cp.G; a.xmode = L.cp.xmode;
  a.mg_wo = div_magic((uint32_t)a.Wo); a.mg_cin = div_magic((uint32_t)a.Cin); a.mg_kw = div_magic((uint32_t)a.kw); a.mg_mt = tile_magic(L.cp.grid_x, a.MT);
  a.c_real = 0;
  if (l == 0 && net.fuse_ingest) {  // layer 0 gathers from the job's fp32 [C][H][W] input: the pointer is filled in per job
    a.x = nullptr;
    a.c_real = net.in_c;
  }
  return a;
}

std::string encode_network(const NetPlan& net, bool wave_prio, const KernelTable& kt, const JoinedTable& joined, const std::vector<void*>& slots, float* ws, LaunchSeq* seq) {
  const int n = (int)net.layers.size();
  const int bf16 = net.bf16;
  std::vector<KernelLaunch> ks;
  *seq = LaunchSeq();
  seq->layer_lo.assign(n + 1, 0);
  auto take = [&](double flops) {
    for (size_t i = 0; i < ks.size(); ++i) {
      LaunchRt r;
      r.kl = ks[i];
      r.flops = i == 0 ? flops : 0;
      seq->launches.push_back(r);
    }
    ks.clear();
  };
  if (!net.fuse_ingest) {
    if (!encode_ingest(kt, nullptr, slots[net.ingest.slot], net.ingest.C, net.ingest.Cs, net.ingest.H, net.ingest.W, bf16, &ks))
      return "input conversion launch";
    seq->in_launch = 0;
    seq->in_off = kIngestInputOffset;
    take(0);
  }
  for (int l = 0; l < n; ++l) {
    seq->layer_lo[l] = (int)seq->launches.size();
    const LayerPlan& L = net.layers[l];
    const TensorInfo& in = net.tensor(L.in_t);
    const void* x = slots[in.slot];
    const bool direct = l == n - 1 && net.final_direct;  // writes the job's logits
    void* y = direct ? nullptr : slots[L.out.slot];
    bool ok = false;
    double flops = 0;
    switch (L.d.op) {
      case DARIS_OP_CONV:
        if ((L.depthwise && L.fused_dw) || net.joined_away(l) || net.followed(l)) {
          ok = true;  // computed inside the next layer's launch
        } else if (!L.depthwise && (L.joins >= 0 || L.follows >= 0)) {
          const int wide = L.follows >= 0 ? L.follows : l, first = net.layers[wide].joins;
          const LayerPlan& W = net.layers[wide];
          const ConvArgs a = conv_args(net, first, wave_prio, nullptr, slots, ws), b = conv_args(net, wide, wave_prio, slots[W.out.slot], slots, ws), c = conv_args(net, l, wave_prio, y, slots, ws);
          flops = 2.0 * (double)(net.layers[first].macs + W.macs + (wide == l ? 0 : L.macs));
          ok = encode_chain(joined, net.layers[first].cp, a, W.cp, b, wide == l ? nullptr : &L.cp, wide == l ? nullptr : &c, bf16, &ks);
        } else if (L.depthwise) {
          DwArgs a = DwArgs();
          a.x = x; a.w = L.w_dev; a.bias = L.b_dev; a.y = y;
          a.H = in.H; a.W = in.W; a.C = in.Cs; a.Ho = L.out.H; a.Wo = L.out.W;
          a.k = L.d.k; a.stride = L.d.stride; a.pad = L.d.pad; a.act = L.d.act;
          if (L.joins >= 0) {
            flops = 2.0 * (double)(L.macs + net.layers[L.joins].macs);
            ok = encode_expand_dw(joined, net.layers[L.joins].cp, conv_args(net, L.joins, wave_prio, nullptr, slots, ws), a, net.plan_cus, bf16, &ks);
          } else {
            ok = encode_dwconv(kt, a, bf16, &ks);
          }
        } else if (L.pair_with >= 0 && !L.pair_lead && !L.sums_pixels) {
          ok = true;  // issued together with the next layer
        } else {
          const ConvArgs a = conv_args(net, l, wave_prio, y, slots, ws);
          flops = 2.0 * (double)L.macs;
          if (L.fused_dw) {
            const LayerPlan& O = net.layers[L.pair_with];  // the depthwise layer: this launch reads ITS input
            const TensorInfo& din = net.tensor(O.in_t);
            ConvArgs b = a;
            b.x = slots[din.slot];
            DwFusedArgs d;
            d.w = O.w_dev; d.bias = O.b_dev; d.H = din.H; d.W = din.W; d.stride = O.d.stride; d.act = O.d.act;
            flops += 2.0 * (double)O.macs;
            ok = encode_conv_dw(kt, L.cp, b, d, bf16, &ks);
          } else if (L.pair_with >= 0 && !L.sums_pixels) {
            const LayerPlan& O = net.layers[L.pair_with];
            const ConvArgs b = conv_args(net, L.pair_with, wave_prio, slots[O.out.slot], slots, ws);
            flops += 2.0 * (double)O.macs;
            // the heavier convolution is the first problem (its plan was kept)
            ok = L.macs >= O.macs ? encode_conv_pair(kt, L.cp, a, O.cp, b, bf16, &ks) : encode_conv_pair(kt, O.cp, b, L.cp, a, bf16, &ks);
          } else {
            if (l == 0 && net.fuse_ingest) {
              seq->in_launch = (int)seq->launches.size();
              seq->in_off = kConvInputOffset;
            }
            ok = L.tall ? encode_conv_tall(joined, L.cp, a, bf16, &ks) : encode_conv(kt, L.cp, a, bf16, &ks);
          }
        }
        break;
      case DARIS_OP_MAXPOOL:
      case DARIS_OP_GAVGPOOL: {
        if (L.average_of >= 0) {
          const LayerPlan& O = net.layers[L.average_of];
          ok = !L.lonely || encode_pooled_sums(kt, (const float*)x, (float*)y, in.Cs, O.cp.MT, in.H * in.W, &ks);
          break;
        }
        PoolArgs a = PoolArgs();
        a.x = x; a.y = y; a.H = in.H; a.W = in.W; a.C = in.Cs; a.Ho = L.out.H; a.Wo = L.out.W;
        a.k = L.d.k; a.stride = L.d.stride; a.pad = L.d.pad;
        if (L.joins >= 0) {  // the convolution in front, which pools its outputs
          const LayerPlan& O = net.layers[L.joins];
          flops = 2.0 * (double)O.macs;
          if (L.joins == 0 && net.fuse_ingest) {
            seq->in_launch = (int)seq->launches.size();
            seq->in_off = kConvInputOffset;
          }
          const ConvArgs conv = conv_args(net, L.joins, wave_prio, nullptr, slots, ws);
          ok = O.cp.rows == 64 ? encode_block_pool(joined, O.cp, conv, a, &ks) : encode_image_pool(joined, O.cp, conv, a, bf16, &ks);
          break;
        }
        ok = L.d.op == DARIS_OP_MAXPOOL ? encode_maxpool(kt, a, bf16, &ks) : encode_gavgpool(kt, a, bf16, &ks);
        break;
      }
      case DARIS_OP_FC: {
        FcArgs a = FcArgs();
        a.x = x; a.w = L.w_dev; a.bias = L.b_dev; a.y = y;
        a.K = L.K; a.N = L.d.c_out; a.Ns = direct ? L.d.c_out : L.out.Cs;
        a.act = L.d.act; a.out_f32 = direct ? 1 : 0;
        if (direct) {
          seq->out_launch = (int)seq->launches.size();
          seq->out_off = kFcOutputOffset;
        }
        if (L.in_t > 0 && net.layers[L.in_t - 1].average_of >= 0) {
          const LayerPlan& B = net.layers[L.in_t - 1];
          const LayerPlan& O = net.layers[B.average_of];
          a.x = B.lonely ? x : slots[O.out.slot];
          ok = encode_fc_pooled(joined, a, B.lonely ? 1 : O.cp.MT, B.lonely ? 1 : O.out.H * O.out.W, bf16, &ks);
          break;
        }
        ok = encode_fc(kt, a, bf16, &ks);
        break;
      }
    }
    if (!ok) return "launch of layer " + std::to_string(l) + " (" + kernel_name(L.kernel_id) + ")";
    take(flops);
  }
  seq->layer_lo[n] = (int)seq->launches.size();
  if (!net.final_direct) {
    const TensorInfo& o = net.layers[n - 1].out;
    if (!encode_egress(kt, slots[o.slot], nullptr, o.C, o.Cs, o.H, o.W, bf16, &ks)) return "output conversion launch";
    seq->out_launch = (int)seq->launches.size();
    seq->out_off = kEgressOutputOffset;
    take(0);
  }
  return "";
}

}  // namespace daris
