// Body of the implicit-GEMM convolution of large fp32 layers on gfx950: 64 pixels x 64 channels per wave.
#pragma once
#include <hip/hip_runtime.h>

#include "layer_bodies.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

// A layer of many tiles is bound by what the waves load, not by its launch.  Per 16 k a 32 x 64 wave tile reads 2 KB of
// pixels and 6 KB of weights (three bf16 parts each) for 384 cycles of matrix work; the four SIMDs of a CU together ask for
// 32 KB in that time and the vector cache delivers 24.  A 64 x 64 tile reads 10 KB for 768 cycles, so the matrix pipe is
// the narrower one again.  128 CUs, against the 32 x 64 tiles: 784 x 512 x 4608 59.5 -> 40 us, 3136 x 256 x 2304 62.5 -> 42,
// 50176 x 64 x 576 57.3 -> 50 (fp32 matrix instructions: 69.7, 76.8, 76.5).  With rows and weights from fixed addresses and
// no exchange through LDS the first takes 32 us: that much is the matrix pipe.  Rows fetched 128 bytes at a time: 42 us.
// (bf16 layers gain nothing from it: 239.7 us for VGG-16's kernels either way.)
//
// The NW waves of a workgroup own the same tile and split K, as in conv_wave_body: no barrier in the K loop, the pixel
// rows pass through a corner of LDS of the wave's own (coalesced 64-byte rows in, matrix order out), two chunks of rows and
// weights are in flight (TAPS: the weights of three chunks, and one fetch of rows for them).  The four 32 x 32 blocks of the partial
// tiles are then summed in wave order, NT / 256 blocks at a time, and finished by the same epilogue.  LDS for 2, 4 and 8 waves: 8, 16 and
// 64 KB (TAPS: 10, 20 and 64, the corners being larger).
//
// TAPS: 3 x 3 windows with stride 1 and padding 1, where a tile's 64 pixels and their left and right neighbours are 66 consecutive
// pixels of the input, whatever row of the image they lie in.  K is walked as (ky, 16 channels, kx): one fetch of the 66 rows
// serves the three taps of a window's row, 23 load instructions for three chunks instead of 30, and these bind the walk together
// with the matrix pipe (a CU's vector memory unit takes about twenty cycles for each: with ten loads a chunk 1600 cycles for eight waves' chunks,
// which need 1536 on its four matrix pipes).  A neighbour on the other side of the image's edge is read from a row of zeros; above and below
// the image the rows are offsets outside the tensor.  us on 128 CUs without and with: 50176 x 64 x
// 576 48.0, 38.9; 12544 x 128 x 1152 41.7, 33.9; 3136 x 256 x 2304 41.3, 33.8; 784 x 512 x 4608 39.4, 31.8.
//
// POOL (with TAPS): the 2 x 2 max pooling with stride 2 behind the convolution, whose output is never stored (p.y: the pooled one).  A tile's two blocks of
// pixels are then 32 places of two rows of the image one above the other, counted row pair by row pair, so that the four outputs under a pooled pixel lie in
// both blocks at places s and s + 1; a fetch is 34 rows for each.  The sums are the same, bit for bit.  It costs nothing that can be measured, and saves the
// pooling launch (us on 128 CUs of the two / of one: 50176 x 64 x 576 42.0, 39.1; 12544 x 128 x 1152 36.3, 33.7; 3136 x 256 x 2304 35.8, 32.6; 784 x 512 x 4608
// 33.3, 31.7) and its gap: VGG-16's frame 433.0 -> 423.4.
template <int NW, bool TAPS>
constexpr int conv_block_lds() {  // floats of LDS
  constexpr int stage = NW * (TAPS ? 5 : 4) * 16 * 4 * 4, sums = NW * (NW * 64 >= 256 ? NW * 64 / 256 : 1) * 1024;
  return stage > sums ? stage : sums;
}
template <int NW, bool TAPS, bool POOL>
__device__ __forceinline__ void conv_block_body(const ConvArgs& p, float* const red) {
  static_assert(TAPS || !POOL, "pooling is for three taps per fetch");
  constexpr int ES = 4;
  constexpr int KS = 8;                      // k per step of the plan; a chunk is two steps
  constexpr int NT = NW * 64;
  constexpr int NP = 3;                      // parts of a weight
  constexpr int NROWS = TAPS ? 5 : 4;        // load instructions for the rows of a fetch
  constexpr int STAGE_V = NROWS * 16 * 4;    // one wave's staging buffer: 64 or 80 pixels x 4 pieces of 16 bytes
  constexpr int NSLOT = TAPS ? 3 : 2;        // chunks of weights in flight
  constexpr int BPP = NT >= 256 ? NT / 256 : 1;  // 32 x 32 blocks summed per pass: a channel quad per thread (NW = 2: two)
  static_assert(NW == 2 || NW == 4 || NW == 8, "one or two blocks per pass");

  if (p.wave_prio) __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, lh = lane >> 5;
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  const int zi = p.splitk == 1 ? 0 : g / p.NTn;
  const int m0 = mt * 64, s0 = mt * 32, nb0 = (g - zi * p.NTn) * 2;
  const int s_wg0 = zi * p.sz;
  const int s_wg1 = min(s_wg0 + p.sz, p.S);
  int sbeg = min(s_wg0 + wave * p.sw, s_wg1), nsteps = min(sbeg + p.sw, s_wg1) - sbeg;
  if constexpr (TAPS) tap_slice<false, NW>(s_wg0, s_wg1, p.sw, wave, &sbeg, &nsteps);
  const int nchunks = nsteps >> 1;  // TAPS: in threes

  const auto xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)((uint32_t)(p.H * p.W) * (uint32_t)p.Cin * ES), 0x00027000);
  const int piece = lane & 3, prow = lane >> 2;
  const int wstride = (p.S >> 1) * NP * 1024;  // bytes of one channel block
  const auto wrsrc = __builtin_amdgcn_make_buffer_rsrc((unsigned char*)const_cast<void*>(p.w) + (size_t)nb0 * wstride, 0, 2 * wstride + 12 * 1024, 0x00027000);
  int woff = (sbeg >> 1) * NP * 1024;
  uint4 bw[NSLOT][2][NP];
  auto load_w = [&](int s) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < NP; ++q)
        bw[s][j][q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, lane * 16, woff + j * wstride + q * 1024, 0));
    woff += NP * 1024;
  };

  f32x16 acc[4];  // block (i, j) of 32 pixels x 32 channels at 2 i + j
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;

  uint4* const st = reinterpret_cast<uint4*>(red) + wave * STAGE_V;
  // A wave issues in order and the matrix pipe takes 32 cycles per instruction, so everything else a chunk needs is laid
  // between the matrix instructions, and the scheduler is told to leave it there: the rows of the next chunk go to LDS
  // and come back in matrix order, those of the chunk after the next are requested, and the operand just fetched is split.
  Split8 cur[2], nxt[2];
  uint4 a4[2][2];
  // lanes exchange data through the wave's buffer: order the accesses of the whole wave, not only of each lane
  auto wave_order = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto put_rows = [&](const uint4 (&rows)[NROWS]) {
    wave_order();
#pragma unroll
    for (int r = 0; r < NROWS; ++r) st[(16 * r + prow) * 4 + (piece ^ ((prow >> 1) & 3))] = rows[r];
    wave_order();
  };
  auto row_at = [&](int row) { return row * 4 + ((2 * lh) ^ ((row >> 1) & 3)); };  // (spread over the banks) the lane's first piece of a row; the second: ^ 1
  float r0, r1;
  uint32_t mid;
  auto split_piece = [&](int u) {  // piece u of 16: half of the work on two of the lane's sixteen values (see split8)
    const int i = u >> 3, e = (u >> 1) & 3;
    const uint4& v = a4[i][e >> 1];
    const uint32_t u0 = (e & 1) ? v.z : v.x, u1 = (e & 1) ? v.w : v.y;
    uint4* to = nxt[i].p;
    auto set = [&](uint4& d, uint32_t w) { (e == 0 ? d.x : e == 1 ? d.y : e == 2 ? d.z : d.w) = w; };
    if ((u & 1) == 0) {
      set(to[0], __builtin_amdgcn_perm(u1, u0, 0x07060302u));
      r0 = __uint_as_float(u0) - __uint_as_float(u0 & 0xffff0000u);
      r1 = __uint_as_float(u1) - __uint_as_float(u1 & 0xffff0000u);
      mid = pack_bf16_rne(r0, r1);
      set(to[1], mid);
    } else {
      set(to[2], pack_bf16_rne(r0 - __uint_as_float(mid << 16), r1 - __uint_as_float(mid & 0xffff0000u)));
    }
  };
  auto take_next = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i) cur[i] = nxt[i];
  };
  constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};  // from the smallest terms to the largest
  if constexpr (TAPS) {
    const int groups = nchunks / 3;  // of three taps
    const int gk = (sbeg >> 1) / 3 * 16;
    int ky = fast_div(gk, p.mg_cin), ci = gk - ky * p.Cin;
    const int row_bytes = p.Cin * ES;
    const uint32_t first = (uint32_t)(m0 - 1 + prow - p.W) * (uint32_t)row_bytes + (uint32_t)(piece * 16);  // of the row of pixel m0 - 1 + prow above, at channel 0
    uint32_t pair_first[POOL ? 5 : 1];  // POOL: the same of the pixel that lands in place 16 r + prow, by r
    bool pair_used[POOL ? 5 : 1];
    if constexpr (POOL) {
#pragma unroll
      for (int r = 0; r < 5; ++r) {  // places 0 to 33: the upper rows, 40 to 73: the lower ones, the others zeros
        const int place = 16 * r + prow, below = place >= 40 ? 1 : 0, s = s0 - 1 + place - 40 * below, y = fast_div(max(s, 0), p.mg_wo);
        pair_used[r] = place - 40 * below < 34 && s >= 0 && 2 * s < p.M;
        pair_first[r] = (uint32_t)(s + (y + below - 1) * p.W) * (uint32_t)row_bytes + (uint32_t)(piece * 16);
      }
    }
    uint4 rows[5];
    auto load_row = [&](int r) {  // r < 4: sixteen rows; 4: the last two, and zeros into rows 66 to 79
      const uint32_t at = POOL ? pair_first[POOL ? r : 0] + (uint32_t)(ky * p.W) * (uint32_t)row_bytes : first + (uint32_t)(16 * r + ky * p.W) * (uint32_t)row_bytes;
      const bool used = POOL ? pair_used[POOL ? r : 0] : r < 4 || prow < 2;
      rows[r] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, used ? (int)(at + (uint32_t)(ci * ES)) : (int)0x80000000, 0, 0));
    };
    auto advance = [&]() {
      ci += 2 * KS;
      const bool next = ci >= p.Cin;
      ci = next ? 0 : ci;
      ky += next ? 1 : 0;
    };
    constexpr int BLOCK = POOL ? 40 : 32, ZEROS = POOL ? 34 : 66;  // places between the blocks' pixels, a place of zeros
    int left_at[2], right_at[2];
    const int mid_at = row_at(li + 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = POOL ? s0 + li : m0 + 32 * i + li, y = fast_div(m, p.mg_wo), x = m - y * p.Wo;
      left_at[i] = x == 0 ? row_at(ZEROS) : row_at(BLOCK * i + li);
      right_at[i] = x == p.Wo - 1 ? row_at(ZEROS) : row_at(BLOCK * i + li + 2);
    }
    auto get_rows = [&](auto kx) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) a4[i][h] = st[(kx == 0 ? left_at[i] : kx == 1 ? mid_at + 4 * BLOCK * i : right_at[i]) ^ h];
    };
    auto chunk = [&](auto kx, auto more) {  // tap kx of a group; more: another group follows
      constexpr bool next = kx < 2 || more;
      if constexpr (kx == 2 && more) put_rows(rows);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < 24; ++n) {
        const int t = n >> 2, i = (n >> 1) & 1, j = n & 1;
        acc[2 * i + j] = mfma_bf16(cur[i].p[PA[t]], bw[kx][j][PB[t]], acc[2 * i + j]);
        if constexpr (next) {
          if (n == 0) get_rows(std::integral_constant<int, (kx + 1) % 3>());
          if (n >= 6 && n < 22) split_piece(n - 6);
        }
        if constexpr (kx == 0 && more) {  // the rows of the next group
          if (n >= 1 && n < 6) load_row(n - 1);
          if (n == 6) advance();
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (more) load_w(kx);
      if constexpr (next) take_next();
      __builtin_amdgcn_sched_barrier(0);
    };
    if (groups > 0) {
#pragma unroll
      for (int r = 0; r < 5; ++r) load_row(r);
      advance();
      static_for<0, 3>(load_w);
      put_rows(rows);
      get_rows(std::integral_constant<int, 0>());
#pragma unroll
      for (int u = 0; u < 16; ++u) split_piece(u);
      take_next();
      for (int g = groups; g > 1; --g) static_for<0, 3>([&](auto kx) { chunk(kx, std::true_type()); });
      static_for<0, 3>([&](auto kx) { chunk(kx, std::false_type()); });
    }
  } else {
    // Walk over k = (tap, ci): a chunk never straddles a tap, so the walk is wave-uniform and lives in scalars.  A lane keeps
    // the byte offset of its piece of each row at tap (0, 0) and one bit per tap that says whether that pixel lies inside the
    // image; the loads go through a buffer descriptor, which returns 0 for an offset past the tensor's end, so padding and
    // the pixels past M need no blanking and the loop body no branch.
    const int kbeg = sbeg * KS;
    const int tap0 = fast_div(kbeg, p.mg_cin);
    int ci = kbeg - tap0 * p.Cin;
    int ky = fast_div(tap0, p.mg_kw), kx = tap0 - ky * p.kw;
    int tap = tap0;
    int rbase[4];
    uint32_t taps[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 16 * r + prow;
      const int y = fast_div(m, p.mg_wo), x = m - y * p.Wo;
      const int iy0 = y * p.stride - p.pad, ix0 = x * p.stride - p.pad;
      rbase[r] = (iy0 * p.W + ix0) * p.Cin * ES + piece * 16;
      // the taps inside the image form a rectangle: rows [ya, yb), columns [xa, xb)
      const int ya = max(0, -iy0), yb = min(p.kh, p.H - iy0), xa = max(0, -ix0), xb = min(p.kw, p.W - ix0);
      const uint32_t cols = m < p.M && xb > xa ? ((xb - xa >= 32 ? 0u : (1u << (xb - xa))) - 1u) << xa : 0u;
      taps[r] = 0u;
      for (int t = ya; t < yb; ++t) taps[r] |= cols << (t * p.kw);
    }
    uint4 rows[2][4];
    auto load_row = [&](int s, int r) {
      const int off = ((ky * p.W + kx) * p.Cin + ci) * ES;
      const uint32_t bit = tap < 32 ? 1u << tap : 0u;  // past the last tap: nothing is inside
      const int o = (taps[r] & bit) ? rbase[r] + off : -16;
      rows[s][r] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, o, 0, 0));
    };
    auto advance = [&]() {  // to the next chunk
      ci += 2 * KS;
      const bool next = ci >= p.Cin;
      ci = next ? ci - p.Cin : ci;
      tap += next ? 1 : 0;
      kx += next ? 1 : 0;
      const bool wrap = kx == p.kw;
      kx = wrap ? 0 : kx;
      ky += wrap ? 1 : 0;
    };
    auto get_rows = [&]() {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) a4[i][h] = st[row_at(32 * i + li) ^ h];
    };
    auto chunk = [&](int s) {  // slot s of the weights holds this chunk's, slot s ^ 1 of the rows the next chunk's
      put_rows(rows[s ^ 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < 24; ++n) {
        const int t = n >> 2, i = (n >> 1) & 1, j = n & 1;
        acc[2 * i + j] = mfma_bf16(cur[i].p[PA[t]], bw[s][j][PB[t]], acc[2 * i + j]);
        if (n == 0) get_rows();
        if (n < 4) load_row(s ^ 1, n);  // two chunks ahead (past the end of the slice: nothing is read, or never used)
        if (n == 3) advance();
        if (n >= 6 && n < 22) split_piece(n - 6);
        __builtin_amdgcn_sched_barrier(0);
      }
      load_w(s);  // (spread over the chunk instead, each part as it falls free: 7 % slower)
      take_next();
      __builtin_amdgcn_sched_barrier(0);
    };
    auto load_rows = [&](int s) {
#pragma unroll
      for (int r = 0; r < 4; ++r) load_row(s, r);
      advance();
    };
    load_rows(0);
    load_w(0);
    load_rows(1);
    load_w(1);
    put_rows(rows[0]);
    load_rows(0);
    get_rows();
#pragma unroll
    for (int u = 0; u < 16; ++u) split_piece(u);
    take_next();
    int c = 0;
    for (; c + 2 <= nchunks; c += 2) {
      chunk(0);
      chunk(1);
    }
    if (c < nchunks) chunk(0);
  }

  // --- sum the NW partial tiles in wave order, BPP blocks (i, j) per pass; epilogue per quad of consecutive channels:
  // quad q of a block = elements 4q..4q+3 of [v][lane], i.e. pixel 8*(v/4) + 4*(lane/32) + v%4, channels lane%32 .. +3.
  // Loads and stores are counted together, so a load that is waited for behind a store waits for the store's way to memory as
  // well: the bias is fetched once ahead of all passes and the residual ahead of the stores of the pass before (a load of both per
  // quad made eight such waits of a workgroup of two waves: 50176 x 64 x 576 53.4 us, 48.0 without;
  // 12544 x 128 x 576 26.1, 23.6).
  constexpr int RQ = 256 * BPP / NT;  // quads of a thread per pass
  const bool own_epilogue = p.splitk == 1;
  const int b = BPP == 1 ? 0 : tid >> 8;  // the thread's block of a pass
  // the block of a pass, or the first of two: POOL takes the two that meet under the pooled pixels one after the other
  auto block_of = [](int pass) { return POOL && BPP == 1 ? 2 * (pass & 1) + (pass >> 1) : pass * BPP; };
  auto park = [&](int pass) {
    __syncthreads();  // the partial tiles reuse the staging buffers, then the pass before
#pragma unroll
    for (int k = 0; k < BPP; ++k) {
#pragma unroll
      for (int w = 0; w < 16; ++w) red[(wave * BPP + k) * 1024 + w * 64 + lane] = acc[block_of(pass) + k][w];
    }
  };
  auto place = [&](int pass, int r, int* mm, int* n) {  // pixel and first channel of the thread's quad r
    const int blk = block_of(pass) + b, e = 4 * ((tid & 255) + r * NT), v = e >> 6, l = e & 63;
    *mm = (POOL ? s0 : m0 + 32 * (blk >> 1)) + (v >> 2) * 8 + (l >> 5) * 4 + (v & 3);
    *n = (nb0 + (blk & 1)) * 32 + (l & 31);
  };
  float4 bias[BPP == 1 ? 2 : 1];  // of both blocks of channels; two blocks a pass: of the thread's own
#pragma unroll
  for (int k = 0; k < (BPP == 1 ? 2 : 1); ++k) {
    int mm, n;
    place(POOL ? 2 * k : k, 0, &mm, &n);
    bias[k] = *(const float4*)(p.bias + (n < p.Cout ? n : 0));
  }
  float4 res[RQ];
  const bool use_res = !POOL && own_epilogue && p.res != nullptr;
  auto fetch_res = [&](int pass) {
    if (!use_res) return;
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      int mm, n;
      place(pass, r, &mm, &n);
      res[r] = *(const float4*)((const float*)p.res + (mm < p.M && n < p.Cout ? (size_t)mm * p.Cout + n : 0));
    }
  };
  fetch_res(0);
  park(0);
  if (TAPS && __builtin_expect(m0 + 64 > p.M, 0)) {
#pragma unroll
    for (int k = 0; k < 4; ++k) drop_pixels(acc[k], POOL ? p.M / 2 - s0 : p.M - m0 - 32 * (k >> 1));
  }
  spoil_unless_in_range(acc, red + wave * BPP * 1024, BPP * 16);
  __syncthreads();
  if (__builtin_expect(spoiled(red[lane % NW * BPP * 1024 + lane]), 0)) {  // every thread of the workgroup or none
    const bool small = all_small(acc);
    const f32x16 had[4] = {acc[0], acc[1], acc[2], acc[3]};
    plain_products<POOL ? 7 : TAPS ? 5 : 3, 32, 2, 2>(p, DwFusedArgs(), POOL ? s0 : m0, nb0, sbeg, 2 * nchunks, acc);
#pragma unroll
    for (int k = 0; k < 4; ++k) take_second(small, had[k], acc[k]);
    park(0);
    __syncthreads();
  }
  float best[POOL ? 4 * RQ : 1];
#pragma unroll
  for (int pass = 0; pass < 4 / BPP; ++pass) {
    if (pass > 0) {
      park(pass);
      __syncthreads();
    }
    float val[4 * RQ];
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      float* const v = val + 4 * r;
      const int e = 4 * ((tid & 255) + r * NT);
      v[0] = v[1] = v[2] = v[3] = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float4 t = *(const float4*)&red[(w * BPP + b) * 1024 + e];
        v[0] += t.x; v[1] += t.y; v[2] += t.z; v[3] += t.w;
      }
    }
    if (POOL || own_epilogue) {
      const float4 bi = bias[BPP != 1 ? 0 : POOL ? pass >> 1 : pass & 1];
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        float* const v = val + 4 * r;
        v[0] += bi.x; v[1] += bi.y; v[2] += bi.z; v[3] += bi.w;
        if (use_res) {
          v[0] += res[r].x; v[1] += res[r].y; v[2] += res[r].z; v[3] += res[r].w;
        }
      }
      apply_act(val, p.act);
    }
    if constexpr (POOL) {
#pragma unroll
      for (int i = 0; i < 4 * RQ; ++i) best[i] = fmaxf((pass & 1) == 0 ? -INFINITY : best[i], val[i]);
      if ((pass & 1) == 0) continue;
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        int s, n;
        place(pass, r, &s, &n);
        float4 v;  // (the neighbour's quad: sixteen lanes further on)
        v.x = fmaxf(best[4 * r], __shfl_xor(best[4 * r], 16, 64)); v.y = fmaxf(best[4 * r + 1], __shfl_xor(best[4 * r + 1], 16, 64));
        v.z = fmaxf(best[4 * r + 2], __shfl_xor(best[4 * r + 2], 16, 64)); v.w = fmaxf(best[4 * r + 3], __shfl_xor(best[4 * r + 3], 16, 64));
        if ((s & 1) == 0 && 2 * s < p.M && n < p.Cout) put((float*)p.y + (size_t)(s >> 1) * p.Cout + n, v);
      }
      continue;
    }
    if (pass + 1 < 4 / BPP) fetch_res(pass + 1);
    float* const to = own_epilogue ? (float*)p.y : p.ws + (size_t)zi * p.M * p.Cout;  // (partial sums of this K slice: splitk_reduce_kernel finishes the layer)
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      int mm, n;
      place(pass, r, &mm, &n);
      if (mm < p.M && n < p.Cout) put(to + (size_t)mm * p.Cout + n, make_float4(val[4 * r], val[4 * r + 1], val[4 * r + 2], val[4 * r + 3]));
    }
  }
}

}  // namespace daris
