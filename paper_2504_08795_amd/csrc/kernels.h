// Interface between the host runtime and the HIP kernels (gfx950 only): argument structures shared by both sides,
// the host-side launch plans, and the encoders that turn a layer into ready-to-dispatch AQL launches.
//
// Device tensor format: NHWC, element type float (fp32 tasks) or bfloat16 stored as uint16 (bf16 tasks),
// channel stride Cs = channel count rounded up to one 16-byte vector (4 floats / 8 bf16); pad channels hold 0.
#pragma once
#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

namespace daris {

enum KernelId : int32_t {
  K_NONE = 0,
  // wave-tile implicit GEMM: TN 32-channel blocks per wave, NW waves splitting K inside the workgroup
  K_CONVW_F32_T1W2, K_CONVW_F32_T1W4, K_CONVW_F32_T1W8, K_CONVW_F32_T2W2, K_CONVW_F32_T2W4, K_CONVW_F32_T2W8,
  K_CONVW_BF16_T1W2, K_CONVW_BF16_T1W4, K_CONVW_BF16_T1W8, K_CONVW_BF16_T2W2, K_CONVW_BF16_T2W4, K_CONVW_BF16_T2W8,
  // the same with 16-pixel tiles of TN 16-channel blocks (deep, skinny layers)
  K_CONV16_F32_T1W2, K_CONV16_F32_T1W4, K_CONV16_F32_T1W8, K_CONV16_F32_T2W2, K_CONV16_F32_T2W4, K_CONV16_F32_T2W8,
  K_CONV16_BF16_T1W2, K_CONV16_BF16_T1W4, K_CONV16_BF16_T1W8, K_CONV16_BF16_T2W2, K_CONV16_BF16_T2W4, K_CONV16_BF16_T2W8,
  // the same with 64 pixels x 64 channels per wave (fp32 layers of many tiles)
  K_CONV64_F32_T2W2, K_CONV64_F32_T2W4, K_CONV64_F32_T2W8,
  K_SPLITK_REDUCE, K_DWCONV, K_MAXPOOL, K_GAVGPOOL, K_FC, K_INGEST, K_EGRESS,
  // one fetch of rows for the three taps of a window's row: the tiles that plan_conv chooses it for, 32-, 16- and 64-pixel ones
  K_TAPS_F32_T1W2, K_TAPS_F32_T1W4, K_TAPS_F32_T1W8, K_TAPS_F32_T2W2, K_TAPS_F32_T2W8,
  K_TAPS_BF16_T1W2, K_TAPS_BF16_T1W4, K_TAPS_BF16_T2W2, K_TAPS_BF16_T2W4,
  K_TAPS16_F32_T1W8, K_TAPS16_F32_T2W8, K_TAPS16_BF16_T1W4, K_TAPS16_BF16_T1W8, K_TAPS16_BF16_T2W4, K_TAPS16_BF16_T2W8,
  K_TAPS64_F32_T2W2, K_TAPS64_F32_T2W4, K_TAPS64_F32_T2W8,
  // the network input in patches: workgroups of one channel block, or of two
  K_IMAGE_F32_N1, K_IMAGE_F32_N2, K_IMAGE_BF16_N1, K_IMAGE_BF16_N2,
  K_IMAGE_POOL_F32, K_IMAGE_POOL_BF16,  // ... with the 3 x 3 max pooling behind it
  K_EXPAND_DW_F32, K_EXPAND_DW_BF16,    // a 1 x 1 convolution and the depthwise one behind it
  K_CHAIN_F32, K_CHAIN_BF16,            // a 3 x 3 convolution and the one or two 1 x 1 behind it
  K_BLOCK_POOL_F32,                     // 64-pixel tiles with three taps per fetch and the 2 x 2 max pooling behind them
  K_COUNT  // at most 64: what a caller of daris_kernel_timing_read has to provide
};
static_assert(K_COUNT <= 64, "see daris_kernel_timing_read");
const char* kernel_name(int32_t id);

// How a convolution's waves come by their pixels.
enum ConvGather : int {
  kGatherAligned = 0,    // straight into registers, no K step straddles a filter tap (bf16)
  kGatherGeneral = 1,    // straight into registers, any channel count
  kGatherInput = 2,      // layer 0: the caller's fp32 [C][H][W] input, straight into registers
  kGatherRows = 3,       // whole 64-byte rows, through LDS
  kGatherDepthwise = 4,  // computed from the input of the depthwise layer in front
  kGatherTaps = 5,       // whole 64-byte rows, each fetch for the three taps of a 3 x 3 window's row; K in the order (ky, channels of a chunk, kx)
  kGatherImage = 6,      // layer 0: the caller's input, a patch per workgroup through LDS
};

constexpr uint32_t kNoMagic = 0xffffffffu;

// ConvArgs::act: the activation, and whether the launch stores its outputs' sums over the pixels of each tile (float [MT][Cout]) in place of the outputs.
constexpr int kActMask = 3, kActSumPixels = 4;
struct ConvArgs {
  const void* x;      // [H][W][Cin]; with c_real > 0: the network input as the caller gives it, float [c_real][H][W]
  const void* w;      // packed weights in MFMA fragment order (see pack_conv)
  const float* bias;  // [Cout]
  const void* res;    // [Ho*Wo][Cout] or nullptr
  void* y;            // [Ho*Wo][Cout]
  float* ws;          // split-K partial sums (splitk > 1)
  int H, W, Cin, Ho, Wo, Cout;
  int kh, kw, stride, pad;
  uint32_t mg_mt;  // multiplier for division by MT, or kNoMagic
  int Kpad, M;
  int act;
  int splitk;  // grid.z
  int S, sz, sw;  // K steps in total, per K slice of a workgroup, per wave
  uint32_t mg_wo, mg_cin, mg_kw;  // multipliers for division by Wo, Cin, kw (see div_magic)
  int MT, NTn, G, xmode;  // pixel tiles, channel tiles, weight groups (= NTn * splitk), XCD mapping mode
  int c_real;             // > 0: layer 0 reads the fp32 [C][H][W] network input directly (Cin == one 16-byte vector, c_real <= 4)
  int wave_prio;          // 1: the waves raise their issue priority (stages of high-priority tasks on shared CUs)
};

// The first convolution of a network for conv_image_body: x is the network input as the caller gives it, float [c_real][H][W].
struct ImageConvArgs {
  const void* x;
  const void* w;  // as ConvArgs::w
  const float* bias;
  void* y;
  int H, W, Ho, Wo, Cout, k, stride, pad;
  int act, S, M, c_real, wave_prio;
  int tiles, across;   // pixel tiles in all, from left to right
  int patch_w, patch;  // input pixels of a tile: a row of them, all
  int phase, pitch;    // places between columns of a row that differ by one (mod stride), between rows
  uint32_t mg_tiles, mg_across, mg_patch_w, mg_stride, mg_wo, mg_k;  // multipliers for division
  int pool_h, pool_w;  // size of the pooled output (conv_image_kernel with POOL, where y is that output)
  int unused[5];  // to one of the sizes that grab() reads
};
constexpr int kImageCols = 16;     // output pixels of a tile's row
constexpr int kImagePatch = 864;   // places for the input pixels of a tile
constexpr int kImageTaps = 512;    // and for its taps: of whole chunks and two more
constexpr int kImagePoolRows = 4, kImagePoolCols = 7;  // conv_image_pool_kernel: a workgroup's pooled pixels, from 9 x 15 convolution outputs
constexpr int kImagePoolPatch = 1024;  // and the places for their input pixels

// The 3x3 depthwise convolution (pad 1) that conv_wave_dw_kernel computes on the fly in front of a 1x1 convolution; the
// ConvArgs beside it describe that 1x1 convolution, except that ConvArgs::x is the DEPTHWISE layer's input tensor
// [H][W][Cin] (ConvArgs::H, W stay the 1x1 convolution's own input size = the depthwise layer's output size).
struct DwFusedArgs {
  const void* w = nullptr;      // [9][C]
  const float* bias = nullptr;  // [C]
  int H = 0, W = 0;             // the depthwise layer's input size
  int stride = 1, act = 0;
};

// A 1x1 convolution and the 3x3 depthwise convolution (pad 1) behind it for conv_expand_dw_kernel.
struct ExpandDwArgs {
  const void* x;         // [H][W][Cin]
  const void* w;         // the 1x1 convolution's weights, packed for 16-pixel tiles
  const float* bias;     // [C]
  const void* dw_w;      // [9][C]
  const float* dw_bias;  // [C]
  void* y;               // [Ho][Wo][C]
  int H, W, Cin, Ho, Wo, C;
  int stride, act, dw_act;  // the depthwise layer's stride, both activations
  int band, bands;          // output rows of a workgroup, workgroups of a channel block
  int S;                    // K steps, as ConvArgs::S
  int threads, wave_prio;
  uint32_t mg_bands, mg_w, mg_wo;  // multipliers for division
  int unused[11];  // to one of the sizes that grab() reads
};
constexpr int kExpandPixels = 320;  // most input pixels of a workgroup
constexpr int kExpandRow = 20;      // floats of a pixel's 16 channels in LDS, spread over the banks
constexpr int kExpandChunks = 5;    // most chunks of 32 k

// The 1x1 convolutions behind the 3x3 one, whose ConvArgs these follow in the arguments of conv_chain_kernel.
struct ChainArgs {
  const void* w3;      // the first: [kChainWide][64], packed for 32-pixel tiles
  const float* bias3;  // [kChainWide]
  const void* res3;    // [M][kChainWide] or nullptr
  void* y3;            // [M][kChainWide]
  const void* w1;      // the second, which reads y3: [n1][kChainWide], as packed
  const float* bias1;  // [n1]
  void* y1;            // [M][n1]
  int act3;
  int n1, act1;        // n1 = 0: there is no second
  int unused[5];       // to one of the sizes that grab() reads
};
constexpr int kChainWide = 256;  // channels of the first

struct DwArgs {
  const void* x;      // [H][W][C]
  const void* w;      // [k*k][C]
  const float* bias;  // [C]
  void* y;            // [Ho][Wo][C]
  int H, W, C, Ho, Wo, k, stride, pad, act;
};

struct PoolArgs {
  const void* x;
  void* y;
  int H, W, C, Ho, Wo, k, stride, pad;
};

// The kernels for windows of a size known at compile time (dwconv_window_kernel, maxpool_window_kernel) find a thread's place
// by multiplications.
struct PointPlace {
  uint32_t mg_cv, mg_wo;  // multipliers for division by the channel vectors of a pixel and by Wo, or kNoMagic
  uint32_t per_xcd;       // workgroups of one XCD
};
struct DwWindowArgs {
  DwArgs a;
  PointPlace at;
};
struct PoolWindowArgs {
  PoolArgs a;
  PointPlace at;
};

struct FcArgs {
  const void* x;      // [K]
  const void* w;      // [N][K]
  const float* bias;  // [N]
  void* y;            // [Ns], element type of the task, or float when out_f32; outputs N..Ns-1 are written as 0
  int K, N, Ns, act, out_f32;
  int stream;    // 1: the matrix is read past the last cache (set by encode_fc)
};

// An FC layer behind a global average pooling whose convolution has added its outputs up over the pixels of its tiles.
struct FcPooledArgs {
  const float* x;  // [tiles][K]
  const void* w;
  const float* bias;
  void* y;         // as FcArgs::y
  int K, N, Ns, act, out_f32;
  int tiles, pixels;  // sums of a channel, pixels they are the sums of
  int unused;
};
constexpr int kPooledTiles = 8;       // most sums of a channel
constexpr int kPooledRows = 8;        // rows of the FC layer's matrix, and waves, in a workgroup
constexpr int kPooledInputs = 4096;   // most channels: they lie in LDS

// Kernel and tile configuration chosen on the host for one dense convolution.
struct ConvPlan {
  int32_t kernel;  // KernelId
  int splitk;      // K slices across workgroups (1 = none); > 1 needs the workspace and the reduction launch
  int rows;                        // pixels per wave tile: 32 (conv_wave_*), 64 (conv_block_*), both with channel blocks of 32, or 16 (conv_wave16_*: blocks of 16)
  int tn, nw, S, sz, sw, MT, NTn, G, xmode;
  int step_align;                  // K slices are multiples of this many steps
  int staged;                      // the pixel operand may be fetched in whole 64-byte rows through LDS
  int gather;                      // ConvGather (kGatherDepthwise never: that is a matter of the launch, LayerPlan::fused_dw)
  int tiles;                       // output tiles per grid.z slice
  size_t ws_bytes;                 // split-K workspace this launch needs
  uint32_t grid_x;                 // workgroups of the launch
  int threads;
};
// True when every pixel's channel vector is a whole number of 64-byte rows, the shape for which the convolution kernel
// fetches the pixel operand in coalesced rows through LDS (chunks of two K steps).
inline bool conv_rows_staged(int cin_stride, int bf16) { return cin_stride > 0 && (cin_stride * (bf16 ? 2 : 4)) % 64 == 0; }
// Whether the kernels that fetch such rows (conv_rows_body) can run a convolution: their byte offsets into the input, the output
// (for the residual operand) and a wave's slice of the weights are 31-bit numbers.
inline bool conv_rows_take(int H, int W, int cin_stride, uint64_t M, int cout_stride, int Kpad, int bf16) {
  const uint64_t es = bf16 ? 2 : 4, limit = 1ull << 31;
  return conv_rows_staged(cin_stride, bf16) && (uint64_t)H * (uint64_t)W * (uint64_t)cin_stride * es < limit && M * (uint64_t)cout_stride * es < limit && (uint64_t)Kpad * 192 < limit;
}
// The same for larger tensors, of plans of two waves and 32 pixels (conv_large_kernel, conv_taps_large_kernel): the offsets of a tile
// count from what it touches of the input and of the output.
inline bool conv_rows_take_large(int H, int W, int cin_stride, int Wo, int cout_stride, int k, int stride, int Kpad, int bf16) {
  const uint64_t es = bf16 ? 2 : 4, limit = 1ull << 31, tile_rows = (uint64_t)(31 / Wo + 1) * (uint64_t)stride + (uint64_t)k, rows = tile_rows < (uint64_t)H ? tile_rows : (uint64_t)H;
  return conv_rows_staged(cin_stride, bf16) && rows * (uint64_t)W * (uint64_t)cin_stride * es < limit && 32 * (uint64_t)cout_stride * es < limit && (uint64_t)Kpad * 192 < limit;
}
// Whether the kernel of 64 x 64 tiles can run an fp32 convolution of this geometry: it keeps one bit per filter tap in a word
// and walks the rows of taps inside the image as a rectangle of them, and its byte offsets into the input and into the weights
// of two channel blocks are signed 32-bit numbers.
inline bool conv_block_takes(int H, int W, int cin_stride, int k, int pad, int Kpad) {
  return k * k <= 31 && pad < k && conv_rows_staged(cin_stride, 0) && (uint64_t)(H + pad) * (uint64_t)W * (uint64_t)cin_stride * 4 < (1ull << 31) &&
         (uint64_t)(Kpad / 8) * 3072 + 12288 < (1ull << 31);
}
// Whether one fetch of rows can serve the three taps of a window's row (conv_taps_body, conv_block_kernel): the pixels of a tile and
// their neighbours are then consecutive in the input.
inline bool conv_three_taps(int k, int stride, int pad) { return k == 3 && stride == 1 && pad == 1; }
// bf16 = 0/1.  Chooses tile shape, waves per workgroup and split-K from (M, N, Kpad), allow_block and the nominal partition
// size (nominal_cus: how many CUs the grid is balanced for) only, so results do not depend on the partition a stage runs in.  step_align = 2 cuts K in whole chunks of two steps (for conv_rows_staged shapes), else 1.
// cin_stride = the input tensor's channel stride: when it is a whole number of the 16-row kernel's K steps and the 32-row
// plan would split K across workgroups or leave half of the CUs idle, a 16-row plan is chosen instead (cin_stride 0: never).
// allow_block = false: no 64-pixel tiles (a convolution that conv_block_takes refuses, shares its launch or computes its input on the fly);
// three_taps: kTaps where conv_three_taps and conv_rows_take hold, kTapsLarge where conv_rows_take_large does in the latter's place.  The
// plan's gather is kGatherTaps or kGatherRows; plan_gather settles the rest.
enum ThreeTaps : int { kNoTaps = 0, kTaps = 1, kTapsLarge = 2 };
ConvPlan plan_conv(int M, int N, int Kpad, int bf16, int step_align, int cin_stride, int nominal_cus, bool allow_block, ThreeTaps three_taps = kNoTaps);
// Plan for a second convolution that is to share a launch with `first`: the same wave-tile kernel variant, K not split
// across workgroups.  Returns a plan with kernel == K_NONE when that is not possible.
ConvPlan plan_conv_like(const ConvPlan& first, int M, int N, int Kpad, int bf16, int step_align, int nominal_cus = 128);
// The plan `own` of the heavier convolution once `light` shares its launch: with the waves a workgroup that so many tiles want (those of the lighter one
// count by their share of K).  us on 128 CUs, fp32: 3136 x 128 x 256 beside 784 x 512 x 256 13.6 -> 8.6, 784 x 256 x 512 beside 196 x 1024 x 512 9.9 -> 7.5, 196 x 512 x
// 1024 beside 49 x 2048 x 1024 9.0 -> 8.6; bf16 the first of them 4.9 -> 4.2.
ConvPlan plan_conv_beside(const ConvPlan& own, const ConvPlan& light, int M, int N, int Kpad, int bf16, int step_align, int nominal_cus);
// Settles the gather of a plan without kGatherTaps; rows = conv_rows_take holds (for both members of a launch pair), or conv_rows_take_large.
void plan_gather(ConvPlan* pl, int cin_stride, bool rows, int bf16);
// The first convolution of a network, whose plan reads the caller's input: turns it into one for conv_image_body, or leaves it
// (kGatherInput) where that cannot run or is the slower one.
void plan_input(ConvPlan* pl, int Ho, int Wo, int cout_stride, int k, int stride, int nominal_cus, int bf16);
// Multiplier for fast_div: floor(2^32 / d) + 1, or 0 for d == 1.  Exact for every n >= 0 with n * d < 2^32.
inline uint32_t div_magic(uint32_t d) { return d <= 1 ? 0u : (uint32_t)((1ull << 32) / d) + 1u; }
// ... for the tile order of a convolution: the multiplier for division of a workgroup number by MT.
inline uint32_t tile_magic(uint64_t groups, int MT) { return groups * (uint64_t)MT < (1ull << 32) ? div_magic((uint32_t)MT) : kNoMagic; }

// ---- launches ------------------------------------------------------------------------------------------------------------
//
// The kernels are dispatched by AQL packets written by the library itself (aql.h).  An encoder turns the arguments of
// a layer into one or two Launch records: kernel, geometry and the exact argument bytes the kernel expects.

struct AqlKernel;
class AqlRuntime;

struct KernelLaunch {
  const AqlKernel* k = nullptr;
  uint32_t groups = 0, threads = 0;  // workgroups, threads per workgroup
  uint32_t nbytes = 0;               // bytes of args in use
  int32_t kernel_id = K_NONE;
  alignas(8) unsigned char args[336];
};

// Every kernel of the code object, looked up once.
struct KernelTable {
  const AqlKernel* conv[2][6][4] = {};  // [bf16][(tn - 1) * 3 + log2(nw) - 1][gather 0..3] (fp32: no kGatherAligned)
  const AqlKernel* taps[2][6] = {};     // the same with kGatherTaps, where there is a kernel id
  const AqlKernel* large[2][2][2] = {}; // conv_rows_take_large: [bf16][kGatherTaps][tn - 1]
  const AqlKernel* image[2][2] = {};    // kGatherImage: [bf16][128 pixels x 32 channels, 64 x 64]
  const AqlKernel* pair[2][6][3] = {};  // kGatherAligned, kGatherGeneral, kGatherRows
  const AqlKernel* conv16[2][2][6] = {};  // 16-row tiles: [bf16][kGatherTaps][(tn - 1) * 3 + log2(nw) - 1]
  const AqlKernel* pair16[2][6] = {};
  const AqlKernel* block[2][3] = {};    // 64-pixel tiles: [kGatherTaps][log2(nw) - 1]
  const AqlKernel* convdw[2][6] = {};   // 1x1 convolution with a fused depthwise producer (fp32: tn = 1 only)
  const AqlKernel *reduce[2] = {}, *dwconv[2] = {}, *maxpool[2] = {}, *gavgpool[2] = {}, *fc[2] = {}, *ingest[2] = {}, *egress[2] = {};
  const AqlKernel *dwconv3[2] = {}, *maxpool_k[2][2] = {};  // 3x3 windows; 2x2 and 3x3 windows
  const AqlKernel *point[2][2][6] = {}, *point_pair[2][2][6] = {};  // 1x1 windows without padding over whole rows: [bf16][16-row tiles][(tn - 1) * 3 + log2(nw) - 1] (bf16 32-row tiles: no eight waves)
  const AqlKernel* cu_probe = nullptr;
  // "" or the name of the first kernel that is missing or whose argument size is not what this header declares
  std::string resolve(const AqlRuntime& rt);
};

// The kernels that compute several layers in a row, and those that run a plan of KernelTable's in tiles of another shape.
struct JoinedTable {
  const AqlKernel* image_pool[2] = {};  // kGatherImage and the 3 x 3 max pooling behind it
  const AqlKernel* expand_dw[2][kExpandChunks] = {};
  const AqlKernel* fc_pooled[2] = {};
  const AqlKernel* chain[2] = {};
  const AqlKernel* block_pool[3] = {};  // [log2(nw) - 1]
  const AqlKernel* tall[2] = {};
  std::string resolve(const AqlRuntime& rt);  // as KernelTable::resolve
};

// Dense convolution: the main kernel, then the split-K reduction if the plan has one.  False on an inconsistent plan.
bool encode_conv(const KernelTable& kt, const ConvPlan& pl, const ConvArgs& a, int bf16, std::vector<KernelLaunch>* out);
// A plan of 16-pixel tiles with three taps per fetch and two blocks of channels to a wave, run with two blocks of pixels in place of them (conv_taps_body,
// TM = 2): the same K slices, hence the same sums.  Whether it should be, and the launch.  Not where it would take more rounds of the CUs, nor with four waves (bf16 with
// K below 2048) or less than twelve groups of taps for eight, whose loops are short: us with blocks of channels / of pixels, 450 x 256 x 1152 on 256 CUs 2.83 / 2.97, 252 x 128 x 1728 on 64 2.95 / 3.23, 210 x 512 x 1728 on
// 256 3.13 / 3.34; with eight, 374 x 64 x 2304 on 64 3.43 / 3.35, 84 x 512 x 4608 on 128 4.62 / 4.36;
// fp32 375 x 128 x 864 on 128 4.10 / 4.42, 304 x 256 x 864 on 160 4.41 / 4.50, 377 x 64 x 1152 on 64 4.61 / 4.30.
bool tall_takes(const ConvPlan& pl, int M, int nominal_cus);
bool encode_conv_tall(const JoinedTable& kt, const ConvPlan& pl, const ConvArgs& a, int bf16, std::vector<KernelLaunch>* out);
// Two independent convolutions in one launch: pl0/a0 as planned by plan_conv, pl1/a1 by plan_conv_like(pl0, ...).
bool encode_conv_pair(const KernelTable& kt, const ConvPlan& pl0, const ConvArgs& a0, const ConvPlan& pl1, const ConvArgs& a1, int bf16,
                      std::vector<KernelLaunch>* out);
// A depthwise 3x3 convolution (pad 1, stride d.stride) followed by the 1x1 convolution pl/a in one launch.  a.x must be the
// depthwise layer's input; the plan must be a staged 32-row one (conv_rows_staged shape, step_align 2).
bool encode_conv_dw(const KernelTable& kt, const ConvPlan& pl, const ConvArgs& a, const DwFusedArgs& d, int bf16, std::vector<KernelLaunch>* out);
// Whether a depthwise 3x3 layer in front of the 1x1 convolution planned as pl should be computed inside that convolution's
// launch.  Measured on MobileNetV2's blocks: the producer re-reads the depthwise input up to nine times through one CU's
// vector cache and pays a memory latency per chunk of 64 bytes of channels, so it can only win where the convolution has enough
// workgroups to fill a partition and a single channel block (no repetition per block, few chunks per wave); elsewhere the
// separate, fully parallel depthwise launch is faster (by 1.3 to 5 us per block).  There it saves a launch: MobileNetV2's kernels fused / with
// the three blocks' layers in launches of their own, fp32 128 CUs 134.5 / 135.5 us, 64 CUs 163.5 / 165.1 (the frame on 128 169.7 / 172.4); bf16 on 128 CUs 109.6 /
// 108.7 (two blocks).
bool conv_dw_fusable(const ConvPlan& pl, int bf16);
// The first convolution and the 3 x 3 max pooling with stride 2 and padding 1 that alone reads it, in one launch: whether the convolution planned
// as pl should be computed so, and the launch itself (pool: the pooling layer).  us of the two launches / of one, 12544 x 64 x 7 x 7 with stride 2: fp32 on
// 128 CUs 8.2 / 7.2, bf16 on 192 CUs 6.3 / 4.9; in the chain of a frame the pooling launch takes 1.3 more than alone, and ResNet-18's frame goes from 133.9 to
// 132.1 us in fp32 and from 81.8 to 79.0 in bf16.  It computes 1.4 outputs for one that counts, and fp32 is bound by the matrix pipe, so that it gains while a CU has one
// workgroup at most: up to one, and where the CUs of an XCD do not come out even over its four shader engines (multiples of 32 in all) up to eight ninths, above which some CU gets
// two while others idle.  Frames of the ResNets of 40 random sizes on such partitions, apart / joined in the geometric mean: 0.84 to 0.885 workgroups a CU 1.008, 0.89 to 1 0.993 (ResNet-18 planned
// for 96 with 112 workgroups 193.3 us / 194.8); bf16, 40 sizes with 1.8 to 6.2 workgroups a CU, 1.003, with no trend.
bool image_pool_takes(const ConvPlan& pl, int Ho, int Wo, int cout_stride, int k, int stride, int nominal_cus, int bf16);
bool encode_image_pool(const JoinedTable& kt, const ConvPlan& pl, const ConvArgs& a, const PoolArgs& pool, int bf16, std::vector<KernelLaunch>* out);
// An fp32 convolution in 64-pixel tiles with three taps per fetch and the 2 x 2 max pooling with stride 2 that alone reads it, in one launch: whether the plan
// (of an output of Ho x Wo) is one, and the launch.
bool block_pool_takes(const ConvPlan& pl, int Ho, int Wo);
bool encode_block_pool(const JoinedTable& kt, const ConvPlan& pl, const ConvArgs& a, const PoolArgs& pool, std::vector<KernelLaunch>* out);
// A 1x1 convolution and the 3x3 depthwise convolution with padding 1 that alone reads it, in one launch.  Turns pl into the plan of the convolution by
// itself whose sums have the same order, and returns whether the two should be joined.
bool plan_expand_dw(ConvPlan* pl, int H, int W, int cin_stride, int c_stride, int Kpad, int dw_stride, int nominal_cus, int bf16);
bool encode_expand_dw(const JoinedTable& kt, const ConvPlan& pl, const ConvArgs& a, const DwArgs& d, int nominal_cus, int bf16, std::vector<KernelLaunch>* out);
// A 3x3 convolution planned as `conv`, the 1x1 convolution that alone reads it (`wide`) and, unless null, the 1x1 convolution that reads that one
// (`narrow`), all with the same pixels, in one launch: whether the kernel has the plans' tiles and K slices, and the launch.
bool chain_takes(const ConvPlan& conv, int channels, const ConvPlan& wide, int wide_channels, const ConvPlan* narrow, int bf16);
bool encode_chain(const JoinedTable& kt, const ConvPlan& conv, const ConvArgs& a, const ConvPlan& wide, const ConvArgs& b, const ConvPlan* narrow, const ConvArgs* c, int bf16,
                  std::vector<KernelLaunch>* out);
bool encode_dwconv(const KernelTable& kt, const DwArgs& a, int bf16, std::vector<KernelLaunch>* out);
bool encode_maxpool(const KernelTable& kt, const PoolArgs& a, int bf16, std::vector<KernelLaunch>* out);
bool encode_gavgpool(const KernelTable& kt, const PoolArgs& a, int bf16, std::vector<KernelLaunch>* out);
// Global average pooling without a launch: the convolution in front adds its outputs up over the pixels of each tile (kActSumPixels), the FC layer behind adds
// those sums, divides by the number of pixels and rounds.  Whether a convolution planned as pl can; the average alone from its sums (where stage cuts
// leave the pooling layer by itself; y: float [C], which the FC layer then takes as the sums of one tile of one pixel); the FC layer.
bool sums_pixels(const ConvPlan& pl, int channels);
bool encode_pooled_sums(const KernelTable& kt, const float* x, float* y, int C, int tiles, int pixels, std::vector<KernelLaunch>* out);
bool encode_fc_pooled(const JoinedTable& kt, const FcArgs& a, int tiles, int pixels, int bf16, std::vector<KernelLaunch>* out);
bool encode_fc(const KernelTable& kt, const FcArgs& a, int bf16, std::vector<KernelLaunch>* out);
// x: float [C][H][W] -> y: [H][W][Cs]
bool encode_ingest(const KernelTable& kt, const float* x, void* y, int C, int Cs, int H, int W, int bf16, std::vector<KernelLaunch>* out);
// x: [H][W][Cs] -> y: float [C][H][W]
bool encode_egress(const KernelTable& kt, const void* x, float* y, int C, int Cs, int H, int W, int bf16, std::vector<KernelLaunch>* out);
// Records, per workgroup, the XCC id and the hardware id register of the CU it ran on (mask probing).
bool encode_cu_probe(const KernelTable& kt, uint32_t* out_dev, int n_groups, int spin, std::vector<KernelLaunch>* out);

// Byte offsets inside a launch's argument block of the pointers that change from job to job.
constexpr uint32_t kConvInputOffset = 0;     // ConvArgs::x (layer 0 gathering from the job's input)
constexpr uint32_t kIngestInputOffset = 0;   // ingest: x
constexpr uint32_t kFcOutputOffset = 24;     // FcArgs::y
constexpr uint32_t kEgressOutputOffset = 8;  // egress: y

}  // namespace daris
