// Host-side plan of one task's DNN: tensor shapes, buffer slots, legal stage cuts, the MAC-balanced stage split
// (Sec. III-B1), weight packing for the HIP kernels, and the per-stage launch sequence.
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/daris.h"
#include "kernels.h"

namespace daris {

struct TensorInfo {
  int C = 0, Cs = 0, H = 0, W = 0;  // logical channels, channel stride (padded), spatial size
  int slot = -1;                    // activation buffer slot, -1 = none (written straight to the caller's logits)
  size_t bytes = 0;
};

struct LayerPlan {
  daris_layer d;  // descriptor with the host pointers cleared
  TensorInfo out;
  int in_t = 0, res_t = -1;  // tensor indices: 0 = ingested network input, l + 1 = output of layer l
  int64_t macs = 0;
  bool depthwise = false;
  int K = 0, Kpad = 0;       // GEMM K (conv: kh*kw*Cs_in, fc: H*W*Cs_in) and its zero-padded length
  ConvPlan cp;
  bool tall = false;         // cp runs in tiles of two blocks of pixels (tall_takes)
  // Two dense convolutions that read the same tensor and do not depend on each other share one launch: it is issued
  // at the later layer (pair_lead), the earlier one issues nothing; the lighter of the two is planned like the heavier.
  int pair_with = -1;
  bool pair_lead = false;
  // A 3x3 depthwise convolution whose only reader is the 1x1 convolution right after it is computed inside that
  // convolution's launch and never stored: the two layers are linked like a launch pair (the depthwise layer issues
  // nothing, the 1x1 convolution leads) and both carry this mark.
  bool fused_dw = false;
  bool fusable_dw = false;  // the plan allows it; fused_dw is switched off while a stage cut separates the two layers
  // Two layers in a row whose first is read by the second alone and never stored: the first is computed in the second one's launch and issues nothing.
  // joins = the first layer, at the second, and how; can_join: the plan allows it; switched off while a stage cut separates the two.  (A
  // convolution that a pooling layer joins has that layer as pair_with, like the earlier member of a launch pair.)
  int joins = -1, can_join = -1;
  // The 1x1 convolution behind such a pair (a 3x3 convolution that joins a 1x1), which nobody else needs to wait for: follows = that pair's second layer,
  // whose launch is then issued here and stores both outputs.  can_follow as can_join.
  int follows = -1, can_follow = -1;
  // A global average pooling that issues nothing: average_of = the convolution in front, which leaves sums over the pixels of its tiles in place of its
  // output (sums_pixels; pair_with = the FC layer behind, which takes the sums).  lonely: alone in its stage, where it makes the averages from the sums.
  int average_of = -1;
  bool sums_pixels = false, lonely = false;
  int32_t kernel_id = K_NONE;
  void* w_dev = nullptr;
  float* b_dev = nullptr;
};

struct NetPlan {
  int bf16 = 0;
  int plan_cus = 128;             // the partition size that the plans are made for
  int in_c = 0, in_h = 0, in_w = 0;
  TensorInfo ingest;              // tensor 0
  std::vector<LayerPlan> layers;
  std::vector<size_t> slot_bytes; // activation slots after liveness-based reuse
  size_t ws_bytes = 0;            // split-K workspace
  std::vector<int> legal_cuts;    // l such that a cut after layer l is legal
  std::vector<int> stage_first;   // first layer of each stage (size = number of stages)
  int n_out = 0;                  // elements of the final output (C*H*W)
  bool final_direct = false;      // last layer is an FC writing fp32 logits itself
  bool fuse_ingest = false;       // layer 0 reads the caller's fp32 [C][H][W] input itself: no layout conversion launch

  const TensorInfo& tensor(int t) const { return t == 0 ? ingest : layers[t - 1].out; }
  // Whether layer l is computed in the launch of the next one, and its output never stored.
  bool joined_away(int l) const { return l + 1 < (int)layers.size() && layers[l + 1].joins == l; }
  // Whether a plan's reader is told that layer l is never stored: not of a convolution in 64-pixel tiles that a pooling layer joins.
  bool hidden(int l) const { return joined_away(l) && layers[l].cp.rows != 64; }
  // Whether layer l's launch is the next one's.
  bool followed(int l) const { return l + 1 < (int)layers.size() && layers[l + 1].follows == l; }
};

// Builds shapes, MACs, legal cuts, buffer slots and kernel plans.  pair_launches: two independent convolutions on one
// tensor share a launch; fuse_ingest: the first convolution may read the caller's input layout itself; staged_rows:
// convolutions whose pixels are whole 64-byte rows fetch them coalesced through LDS; small_tiles: deep, skinny layers
// get 16-pixel tiles instead of a K split across workgroups; fuse_dw: a depthwise convolution is computed inside the 1x1
// convolution that alone reads it, or the 1x1 in front in its; tall_tiles: LayerPlan::tall; join: LayerPlan::joins,
// follows and average_of.  Returns "" or an error text.
// plan_cus: the partition size the convolution grids are balanced for.
std::string build_plan(const daris_dnn& dnn, bool keep_activations, bool pair_launches, bool fuse_ingest, bool staged_rows, bool small_tiles, bool fuse_dw,
                       int plan_cus, NetPlan* out, bool tall_tiles = true, bool join = true);
// Joins what can share a launch across layers (LayerPlan::joins, fused depthwise layers) wherever no stage cut separates the layers, and
// parts the others.  Returns whether anything changed.
bool join_layers(NetPlan* net);
// Chooses k - 1 cuts minimising the largest per-stage MAC count, ties to the lexicographically smallest cut
// list.  Returns false when k exceeds the number of legal cuts + 1.
bool split_stages(NetPlan* net, int k);

// Weight packing (host): results are byte buffers in the device layouts of kernels.h.
void pack_conv(const NetPlan& net, const LayerPlan& L, const float* w, const float* b, std::vector<unsigned char>* wp,
               std::vector<float>* bp);
void pack_fc(const NetPlan& net, const LayerPlan& L, const float* w, const float* b, std::vector<unsigned char>* wp,
             std::vector<float>* bp);
uint16_t host_f32_to_bf16(float f);

}  // namespace daris
