// Spatial SwiGLU for gfx950 (MI355X): paper Sec. 3.1, "Spatial SwiGLU",
//   Y = [SiLU(X W_g) * DWConv3x3(X W_v)] W_o,
// X the patch tokens of one image in row-major grid order, the value branch
// convolved depthwise over the H x W grid (zero padding), the gate tokenwise.
//
// Two launches (three when the output product splits K):
//   1. gated_conv_kernel: H = SiLU(X W_g^T) * (DWConv3x3(X W_v^T) + bias) per
//      tile of tokens, both products on MFMA with the input dtype's operands
//      (fp16 or bf16) and float32 accumulation, rounded to fp16 on chip, the
//      convolution's halo recomputed per tile; H is stored in fp16, the
//      operand type of the next product;
//   2. gemm_ring_kernel or gemm_staged_kernel: Y = H W_o^T (fp16 operands; bf16 weights are widened),
//      float32 partial products per K slice summed by ksplit_reduce_kernel.
// Weights use the layout of a linear layer (output features first), so both
// operands of every product are read along K in 16-byte pieces.
#include <hip/hip_runtime.h>

#include "gemm.h"
#include "gtr.h"
#include "gtr_device.h"
#include "gtr_internal.h"

namespace gtr {

constexpr int KB = 4;     // minimum 64-wide K-steps per slice when splitting K
// C = sum over the ksplit float32 partial products, converted to C's dtype;
// 4 elements per thread.
__global__ void __launch_bounds__(256) ksplit_reduce_kernel(const float* part, void* C, int64_t n4, int ksplit,
                                                            int cdt, const void* res) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n4) return;
  f4 s = reinterpret_cast<const f4*>(part)[i];
  for (int z = 1; z < ksplit; ++z) s += reinterpret_cast<const f4*>(part)[(int64_t)z * n4 + i];
  if (res) {  // a residual in C's dtype
    float r[4];
    load4(res, cdt, 4 * i, r);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] += r[e];
  }
  if (cdt == GTR_F32) {
    reinterpret_cast<f4*>(C)[i] = s;
  } else {
    float x[4] = {s[0], s[1], s[2], s[3]};
    store_n<4>(C, cdt, 4 * i, x);
  }
}

// H[b][t][c] = SiLU(G[b][t][c]) * (sum_{u,v} V[b][t + (u-1, v-1)][c] * cw[c][u][v] + cb[c]),
// G = X W_g^T and V = X W_v^T, in one launch. A work-group owns a tile of
// kFH x kFW tokens of one image and kFN channels. Its K loop multiplies the
// tile's (kFH + 2) x (kFW + 2)-token halo of X by the kFN rows of W_v, and the
// tile's own tokens (each tile row is a run of 16 consecutive halo rows) by the
// kFN rows of W_g, with the transfers to LDS, the swizzle and the C^T
// accumulator layout of gemm_ring_kernel (two stages of 64-deep K steps, 80 KB:
// two work-groups per CU). Halo rows outside the image read some row of it and
// their V is zeroed. The epilogue rounds both products to fp16 into the LDS the
// K loop used and forms the gated convolution there: G and V never leave the
// chip, and the halo's extra V rows are the price (180 V rows per 128 tokens).
// One-dimensional grid of tiles * (hidden / kFN) work-groups; as in
// gemm_ring_kernel each XCD takes a contiguous range of the order (tile, channel
// block), channel blocks fastest, so the work-groups that read the same X halo
// share one XCD's L2. (Measured at 40x40 tokens, one image, us per SwiGLU call
// with an earlier K loop: GTR-L 34.4, GTR-X 45.9 with this order; 35.1 / 46.9
// with channel blocks slowest; 34.2 / 46.6 with the plain two-dimensional grid.)
constexpr int kFH = 8, kFW = 16;         // tile: 8 rows of 16 tokens
constexpr int kFHW = kFW + 2;            // halo row length
constexpr int kFV = (kFH + 2) * kFHW;    // halo tokens (180)
constexpr int kFVT = (kFV + 15) / 16;    // MFMA row blocks of V (12; rows 180..191 are padding)
constexpr int kFN = 64;                  // channels per work-group
constexpr int kFWaves = 8;               // 4 row groups x 2 halves of the channels
constexpr int kFA = kFVT * 16 / 8 / kFWaves;  // transfers of the halo per wave per K step (3)
constexpr int kFB = 2 * kFN / 8 / kFWaves;    // of W_g and W_v (2)
constexpr int kFP = kFN / 8;             // 16-byte pieces (8 channels) of one token's kFN channels
static_assert(kFN == 64 && kFWaves == 8 && kFH == 8 && kFW == 16, "wave and thread split");
static_assert(kFVT * 2 % kFWaves == 0, "transfers split evenly over the waves");
// A launch takes less than 2^32 threads: more work-groups go in several launches.
constexpr int64_t kLaunchWgs = 0xffffffffu / (64 * kFWaves);

struct GatedConvArgs {
  const void* X;
  const void* Wg;
  const void* Wv;
  const float* cw;  // [hidden][9]
  const float* cb;  // [hidden] or null
  _Float16* H;      // [B * Hh * W][hidden]
  int Hh, W, d, hidden;
  int B;            // images
  int first, count;  // positions of the (tile, channel block) order this launch takes
};

template <int DT>
__global__ void __launch_bounds__(64 * kFWaves) __attribute__((amdgpu_waves_per_eu(4)))
gated_conv_kernel(GatedConvArgs f) {
  typedef Operand<DT, DT> OP;
  constexpr int NT = 64 * kFWaves;
  constexpr int SA = kFVT * 16 * kPitch64, SB = kFN * kPitch64;  // 16-bit elements per stage: halo, each weight tile
  constexpr int ST = SA + 2 * SB;
  constexpr int VT = kFVT / 4, GT = kFH / 4;                     // row blocks of V and G per wave
  constexpr int NJ = kFN / 32;                                   // column blocks per wave
  constexpr int kTiles = (kFVT * 16 + kFH * kFW) * kFN;          // 16-bit elements of the epilogue's V and G
  static_assert(2 * ST * 2 >= kTiles * 2 + (9 * kFN + kFN) * 4, "epilogue tiles and conv weights fit the stages");
  __shared__ __attribute__((aligned(1024))) unsigned short ring[2 * ST];

  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wr = w >> 1, wc = w & 1;  // row group, channel half
  const int r16 = lane & 15, kq = lane >> 4;
  const int tiles_x = (f.W + kFW - 1) / kFW, tiles_y = (f.Hh + kFH - 1) / kFH;
  const int T = f.count, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int ncb = f.hidden / kFN;
  const int j = f.first + xcd * (T >> 3) + min(xcd, T & 7) + slot;  // position in the (tile, channel block) order
  const int tile = j / ncb;
  const int tx = tile % tiles_x;
  const int ty = (tile / tiles_x) % tiles_y;
  const int64_t b = tile / (tiles_x * tiles_y);
  const int y0 = ty * kFH, x0 = tx * kFW;
  const int c0 = (j % ncb) * kFN;
  const int64_t L = (int64_t)f.Hh * f.W, K = f.d;

  // this lane's global pieces: transfer q of the wave fills halo rows 8 (w + 8 q) ..,
  // then rows 8 w .. of W_g and of W_v
  const char* ga[kFA];
  const char* gb[kFB];
  const int lr = lane >> 3;
#pragma unroll
  for (int q = 0; q < kFA; ++q) {
    const int row = 8 * (w + kFWaves * q) + lr, col = (lane & 7) ^ kSwz64(row);
    const int hy = row / kFHW, hx = row - hy * kFHW;
    const int y = min(max(y0 - 1 + hy, 0), f.Hh - 1), x = min(max(x0 - 1 + hx, 0), f.W - 1);
    ga[q] = static_cast<const char*>(f.X) + ((b * L + (int64_t)y * f.W + x) * K + 8 * col) * 2;
  }
#pragma unroll
  for (int q = 0; q < kFB; ++q) {
    const int row = 8 * w + lr, col = (lane & 7) ^ kSwz64(row);
    gb[q] = static_cast<const char*>(q ? f.Wv : f.Wg) + ((int64_t)(c0 + row) * K + 8 * col) * 2;
  }
  const unsigned lbase = lds_addr(ring) + w * 1024;
  auto issue = [&](int buf) {
    const unsigned l = lbase + buf * ST * 2;
#pragma unroll
    for (int q = 0; q < kFA; ++q) {
      dma16(ga[q], l + kFWaves * 1024 * q);
      ga[q] += 128;
    }
#pragma unroll
    for (int q = 0; q < kFB; ++q) {
      dma16(gb[q], l + (SA + q * SB) * 2);
      gb[q] += 128;
    }
  };
  issue(0);

  // conv weights and bias of the work-group's channels, for the epilogue
  f4 cwv = {0.f, 0.f, 0.f, 0.f};
  if (tid < kFN * 9 / 4)
    cwv = reinterpret_cast<const f4*>(f.cw + (int64_t)c0 * 9)[tid];
  else if (tid < kFN * 10 / 4 && f.cb)
    cwv = reinterpret_cast<const f4*>(f.cb + c0)[tid - kFN * 9 / 4];

  f4 av[VT][NJ], ag[GT][NJ];
#pragma unroll
  for (int t = 0; t < VT; ++t)
#pragma unroll
    for (int j = 0; j < NJ; ++j) av[t][j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < GT; ++t)
#pragma unroll
    for (int j = 0; j < NJ; ++j) ag[t][j] = f4{0.f, 0.f, 0.f, 0.f};

  const int steps = f.d / 64;
  for (int s = 0; s < steps; ++s) {
    ring_wait<0>();  // this step's stage has landed, every wave is done with the other one
    if (s + 1 < steps) issue((s & 1) ^ 1);
    const unsigned short* S = ring + (s & 1) * ST;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      auto frag = [&](const unsigned short* base, int row) {
        return OP::get(*reinterpret_cast<const w4*>(&base[row * kPitch64 + 8 * ((4 * h + kq) ^ kSwz64(row))]));
      };
      typename OP::T fg[NJ], fv[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        fv[j] = frag(S + SA + SB, 32 * wc + 16 * j + r16);
        fg[j] = frag(S + SA, 32 * wc + 16 * j + r16);
      }
#pragma unroll
      for (int t = 0; t < VT; ++t) {
        const typename OP::T fa = frag(S, 16 * (VT * wr + t) + r16);
#pragma unroll
        for (int j = 0; j < NJ; ++j) av[t][j] = mfma(fv[j], fa, av[t][j]);  // V^T tiles
      }
#pragma unroll
      for (int t = 0; t < GT; ++t) {
        const int ci = GT * wr + t;  // tile row: halo rows (ci + 1) * kFHW + 1 .. + 16
        const typename OP::T fa = frag(S, (ci + 1) * kFHW + 1 + r16);
#pragma unroll
        for (int j = 0; j < NJ; ++j) ag[t][j] = mfma(fg[j], fa, ag[t][j]);  // G^T tiles
      }
    }
  }

  // epilogue: V [192 halo rows][kFN] and G [128 tile tokens][kFN] in fp16, in
  // the stages. The 16-byte piece p of row r sits at piece p ^ eswz(r): the C^T
  // writes (16 rows x 2 half-pieces per 32 lanes) and the convolution's reads (4
  // consecutive rows x 8 pieces per 32 lanes) then both spread over all banks;
  // unswizzled, the writes of rows r, r + 2, r + 4, ... hit the same banks.
  ring_sync();  // every wave is past the K loop's last LDS read
  _Float16* Vt = reinterpret_cast<_Float16*>(ring);
  _Float16* Gt = Vt + kFVT * 16 * kFN;
  float* wsm = reinterpret_cast<float*>(ring + kTiles);  // [9 taps][kFN], then the bias [kFN]
  auto eswz = [](int row) { return (row >> 1) & (kFP - 1); };
  if (tid < kFN * 9 / 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 4 * tid + e, ch = i / 9;
      wsm[(i - 9 * ch) * kFN + ch] = cwv[e];
    }
  } else if (tid < kFN * 10 / 4) {
    reinterpret_cast<f4*>(wsm)[tid] = cwv;
  }
#pragma unroll
  for (int t = 0; t < VT; ++t) {
    const int row = 16 * (VT * wr + t) + r16;
    const int hy = row / kFHW, hx = row - hy * kFHW;
    const bool in = (unsigned)(y0 - 1 + hy) < (unsigned)f.Hh && (unsigned)(x0 - 1 + hx) < (unsigned)f.W;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      h4 hv = {(_Float16)av[t][j][0], (_Float16)av[t][j][1], (_Float16)av[t][j][2], (_Float16)av[t][j][3]};
      if (!in) hv = h4{0, 0, 0, 0};
      *reinterpret_cast<h4*>(&Vt[row * kFN + 8 * ((4 * wc + 2 * j + (kq >> 1)) ^ eswz(row)) + 4 * (kq & 1)]) = hv;
    }
  }
#pragma unroll
  for (int t = 0; t < GT; ++t)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int row = 16 * (GT * wr + t) + r16;
      const h4 hg = {(_Float16)ag[t][j][0], (_Float16)ag[t][j][1], (_Float16)ag[t][j][2], (_Float16)ag[t][j][3]};
      *reinterpret_cast<h4*>(&Gt[row * kFN + 8 * ((4 * wc + 2 * j + (kq >> 1)) ^ eswz(row)) + 4 * (kq & 1)]) = hg;
    }
  __syncthreads();

  // gated convolution: 8 channels (piece pc) of NR tokens one below the other
  // per thread, which share the halo rows between them
  constexpr int NR = kFH * kFW * kFP / NT;  // 2
  const int pc = tid & (kFP - 1), tg = tid / kFP, cj = tg % kFW, ci = tg / kFW * NR;
  h8 out[NR];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {  // 4 of the 8 channels at a time: the 9 taps of all 8 take 72 registers
    float acc[NR][4];
    const f4 bias = *reinterpret_cast<const f4*>(&wsm[9 * kFN + 8 * pc + 4 * hf]);
#pragma unroll
    for (int m = 0; m < NR; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[m][e] = bias[e];
    f4 wt[3][3];  // wt[u][v][e]: tap (u, v) of channel 8 pc + 4 hf + e
#pragma unroll
    for (int hr = 0; hr < NR + 2; ++hr) {
      if (hr < 3)
#pragma unroll
        for (int v = 0; v < 3; ++v) wt[hr][v] = *reinterpret_cast<const f4*>(&wsm[(3 * hr + v) * kFN + 8 * pc + 4 * hf]);
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        const int row = (ci + hr) * kFHW + cj + v;
        const h4 x = *reinterpret_cast<const h4*>(&Vt[row * kFN + 8 * (pc ^ eswz(row)) + 4 * hf]);
#pragma unroll
        for (int m = 0; m < NR; ++m) {
          const int u = hr - m;  // the tap row of token ci + m that this halo row is under
          if (u < 0 || u > 2) continue;
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[m][e] = fmaf((float)x[e], wt[u][v][e], acc[m][e]);
        }
      }
    }
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int ct = (ci + m) * kFW + cj;
      const h4 g4 = *reinterpret_cast<const h4*>(&Gt[ct * kFN + 8 * (pc ^ eswz(ct)) + 4 * hf]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float z = (float)g4[e];
        acc[m][e] *= z * __builtin_amdgcn_rcpf(1.f + __expf(-z));
        // computed here: sunk into the guarded store, the products hold every operand in registers till then
        asm volatile("" : "+v"(acc[m][e])::"memory");
        out[m][4 * hf + e] = (_Float16)acc[m][e];
      }
    }
  }
#pragma unroll
  for (int m = 0; m < NR; ++m) {
    const int y = y0 + ci + m, x = x0 + cj;
    if (y < f.Hh && x < f.W) *reinterpret_cast<h8*>(f.H + (b * L + (int64_t)y * f.W + x) * f.hidden + c0 + 8 * pc) = out[m];
  }
}

// ---------------------------------------------------------------------------
// Tile of a product. The CUs run in lockstep through ceil(tiles / CUs) tiles
// each, so the time goes with that count times the tile's area; per area a larger
// tile is faster, as it reads fewer operand bytes per product: at 12800 x 384 x
// 2304 64 x 192, 64 x 128 and 64 x 64 take 1.08, 1.08 and 1.25 times as long as 128 x
// 192 (36 us), at 12800 x 1920 x 384 1.19, 1.19 and 1.28 times (36 us). The weights
// below lie between. Where the larger tile leaves CUs idle the
// smaller one wins, as the rule says: 8300 x 384 x 1536 20.1 in 64 x 128 (390
// tiles) against 25.3 in 128 x 192 (130); 1600 x 384 x 1536 9.7 in 64 x 64 (150)
// against 14.2 in 64 x 128 (75); with LN 1600 x 1920 x 384 10.6 in 64 x 192 (250)
// against 11.4 in 64 x 64 (750), 1600 x 960 x 192 6.9 in 64 x 64 (375) against 8.0 in
// 64 x 192 (125). All widths that no wider tile divides run in 64 x 64. Known
// misses: 3200 to 5000 x 384 x 1536 and 2304 with inputs from cache, 64 x 64 up to 14 %
// faster than the 64 x 128 taken (from HBM 8 % slower); from 20000 rows on, 128 x 192
// up to 12 % faster than 64 x 192; 10000 x 1920 x 384 with LN 42.5 against 38.4.
// ---------------------------------------------------------------------------
constexpr int kCUs = 256;
constexpr int kGemmBM = 64, kGemmBN = 64;  // the smallest tile
struct GemmTile {
  int bm, bn;
  float weight;
};
constexpr GemmTile kGemmTiles[] = {{128, 192, 1.f}, {64, 192, 1.05f}, {64, 128, 1.15f}, {64, 64, 1.25f}};

static int pick_tile(int64_t M, int N, bool ln) {
  int best = 3;
  float cost = 0.f;
  for (int i = 3; i >= 0; --i) {
    const GemmTile& t = kGemmTiles[i];
    if (N % t.bn || (ln && i == 2)) continue;
    const int64_t tiles = (M + t.bm - 1) / t.bm * (N / t.bn);
    const float c = (float)((tiles + kCUs - 1) / kCUs) * t.bm * t.bn * t.weight;
    if (i == 3 || c < cost) best = i, cost = c;
  }
  return best;
}

template <int ADT, int BDT, int MT, int BM, int BN, int WM, int WN, int S, int LN, int KH = 1>
static void launch_tile(const GemmArgs& g, hipStream_t stream) {
  const int64_t wgs = (int64_t)((g.M + BM - 1) / BM) * ((g.N / BN + g.cols - 1) / g.cols) * g.ksplit;
  hipLaunchKernelGGL((gemm_ring_kernel<ADT, BDT, MT, BM, BN, WM, WN, S, LN, KH>), dim3((unsigned)wgs), dim3(64 * WM * WN), 0,
                     stream, g);
}

// Column tiles per work-group of the row-normalised product in wide tiles: the
// statistics of a row block cost about half a tile, once per work-group, and
// two work-groups share a CU, so the time goes with max(1, work-groups / (2
// CUs)) (cols + 1/2). Measured (us with one, two and three column tiles): 12800 x
// 1920 x 384 44.0, 40.4 (500 work-groups), 52.5; 8300 x 1920 x 384 31.7, 36.3, 48.0;
// 30500 x 1920 x 384 113, 104, 115; 15300 x 960 x 384 24.8, 25.4, 24.6 (takes three).
static int pick_cols(int64_t M, int N, const GemmTile& t) {
  const int64_t rows = (M + t.bm - 1) / t.bm, ntile = N / t.bn;
  int best = 1;
  float cost = 0.f;
  for (int c = 1; c <= 4 && c <= ntile; ++c) {
    const float rounds = (float)(rows * ((ntile + c - 1) / c)) / (2 * kCUs);
    const float x = (rounds > 1.f ? rounds : 1.f) * (c + 0.5f);
    if (c == 1 || x < cost) best = c, cost = x;
  }
  return best;
}

// Grids of fewer than kCUs 64 x 64 tiles leave one work-group on a CU, and its K
// loop is a chain of dependent steps: there the two 32-deep halves of a step are
// summed apart (KH = 2, or on separate waves in gemm_staged_kernel, which round
// alike), which cuts the chain of dependent MFMAs and of float32 additions in
// half. The registers are free at that size; larger grids gain nothing from it.
// gemm_staged_kernel takes the row-normalised products of that size and the long
// chains (K of kStagedK and more); the measurements are beside it.
constexpr int kStagedK = 2048;
template <int ADT, int BDT, int MT, bool LN>
static void launch_gemm(GemmArgs g, hipStream_t stream) {
  const int t = g.ksplit > 1 ? 3 : pick_tile(g.M, g.N, LN);
  const int64_t tiles = ((int64_t)g.M + 63) / 64 * (g.N / 64) * g.ksplit;  // of 64 x 64
  g.cols = LN && t < 2 ? pick_cols(g.M, g.N, kGemmTiles[t]) : 1;
  if (t == 0)
    launch_tile<ADT, BDT, MT, 128, 192, 2, 4, 2, LN ? 2 : 0>(g, stream);
  else if (t == 1)
    launch_tile<ADT, BDT, MT, 64, 192, 2, 4, 2, LN ? 2 : 0>(g, stream);
  else if (!LN && t == 2 && tiles <= 2 * kCUs)  // one work-group per CU: a third stage covers the wait
    launch_tile<ADT, BDT, MT, 64, 128, 2, 2, 3, 0>(g, stream);
  else if (!LN && t == 2)
    launch_tile<ADT, BDT, MT, 64, 128, 2, 2, 2, 0>(g, stream);
  else if (tiles < kCUs && (LN || g.K >= kStagedK))
    hipLaunchKernelGGL((gemm_staged_kernel<ADT, BDT, MT, LN ? 1 : 0>), dim3((unsigned)tiles), dim3(512), 0, stream, g);
  else if (!LN && tiles < kCUs)
    launch_tile<ADT, BDT, MT, 64, 64, 2, 2, 3, 0, 2>(g, stream);
  else
    launch_tile<ADT, BDT, MT, 64, 64, 2, 2, LN ? 2 : 3, LN ? 1 : 0>(g, stream);
}

// K is split into the fewest slices that give 64 work-groups when M x d alone
// does not (small grids only): every slice costs a float32 partial product and
// its share of the reduction.
static int out_ksplit(int64_t M, int d, int hidden) {
  const int64_t wgs = ((M + kGemmBM - 1) / kGemmBM) * (d / kGemmBN);
  int s = 1;
  while (wgs * s < 64 && s < 8 && hidden / 64 >= 2 * s * KB) s *= 2;
  return s;
}

struct SwigluLayout {
  size_t h_off, part_off, total;
};

static SwigluLayout swiglu_layout(int64_t M, int d, int64_t hidden) {
  auto a256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
  SwigluLayout l;
  l.h_off = 0;
  l.part_off = a256((size_t)M * hidden * 2);
  const int ks = out_ksplit(M, d, (int)hidden);
  l.total = a256(l.part_off + (ks > 1 ? (size_t)ks * M * d * 4 : 0));
  return l;
}

// All checks but the workspace size and the pointers when !check_pointers.
static gtr_status swiglu_check(const gtr_swiglu_args* a, int64_t* M_out, bool check_pointers) {
  if (a->B <= 0 || a->H <= 0 || a->W <= 0 || a->d <= 0 || a->hidden <= 0) return GTR_ERR_SHAPE;
  if (a->d % 64 || a->hidden % 64) return GTR_ERR_UNSUPPORTED;
  if (a->dtype != GTR_F16 && a->dtype != GTR_BF16) return GTR_ERR_UNSUPPORTED;
  if (a->y_dtype != a->dtype && a->y_dtype != GTR_F32) return GTR_ERR_UNSUPPORTED;
  int64_t L, M, n;
  if (__builtin_mul_overflow((int64_t)a->H, (int64_t)a->W, &L) || __builtin_mul_overflow(L, (int64_t)a->B, &M))
    return GTR_ERR_SHAPE;
  if (M > 0x7fffffff - 128 || __builtin_mul_overflow(M, (int64_t)a->hidden, &n) || n > ((int64_t)1 << 40))
    return GTR_ERR_SHAPE;
  // both launches number their work-groups with 32-bit ints
  const int64_t tiles = (int64_t)a->B * ((a->H + kFH - 1) / kFH) * ((a->W + kFW - 1) / kFW);
  if (tiles * (a->hidden / kFN) > 0x7fffffff || ((M + kGemmBM - 1) / kGemmBM) * (a->d / kGemmBN) * 8 > 0x7fffffff)
    return GTR_ERR_SHAPE;
  *M_out = M;
  if (!check_pointers) return GTR_OK;
  if (!a->x || !a->w_gate || !a->w_value || !a->w_out || !a->conv_w || !a->y) return GTR_ERR_NULL;
  const uintptr_t mis = reinterpret_cast<uintptr_t>(a->x) | reinterpret_cast<uintptr_t>(a->w_gate) |
                        reinterpret_cast<uintptr_t>(a->w_value) | reinterpret_cast<uintptr_t>(a->w_out) |
                        reinterpret_cast<uintptr_t>(a->conv_w) | reinterpret_cast<uintptr_t>(a->conv_b) |
                        reinterpret_cast<uintptr_t>(a->y);
  if (mis & 15u) return GTR_ERR_UNSUPPORTED;
  const SwigluLayout lay = swiglu_layout(M, a->d, a->hidden);
  if (!a->workspace || (reinterpret_cast<uintptr_t>(a->workspace) & 255u)) return GTR_ERR_WORKSPACE;
  if (a->workspace_bytes < lay.total) return GTR_ERR_WORKSPACE;
  const size_t es = dtype_size(a->dtype);
  struct R {
    uintptr_t lo, hi;
  };
  auto rng = [](const void* p, size_t bytes) {
    const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
    return R{lo, lo + bytes};
  };
  auto ovl = [](R x, R y) { return x.lo < y.hi && y.lo < x.hi; };
  const R ry = rng(a->y, (size_t)M * a->d * dtype_size(a->y_dtype));
  const R rw = rng(a->workspace, lay.total);
  const R ins[] = {rng(a->x, (size_t)M * a->d * es), rng(a->w_gate, (size_t)a->hidden * a->d * es),
                   rng(a->w_value, (size_t)a->hidden * a->d * es), rng(a->w_out, (size_t)a->d * a->hidden * es),
                   rng(a->conv_w, (size_t)a->hidden * 9 * 4),
                   a->conv_b ? rng(a->conv_b, (size_t)a->hidden * 4) : R{0, 0}};
  for (const R& r : ins)
    if (ovl(ry, r) || ovl(rw, r)) return GTR_ERR_ALIAS;
  if (ovl(ry, rw)) return GTR_ERR_ALIAS;
  if (a->residual) {  // read-only like the inputs, or y itself (each element read, then written, by one thread)
    if (reinterpret_cast<uintptr_t>(a->residual) & 15u) return GTR_ERR_UNSUPPORTED;
    const R rr = rng(a->residual, (size_t)M * a->d * dtype_size(a->y_dtype));
    if ((a->residual != a->y && ovl(rr, ry)) || ovl(rr, rw)) return GTR_ERR_ALIAS;
  }
  return GTR_OK;
}

}  // namespace gtr

using namespace gtr;

extern "C" size_t gtr_spatial_swiglu_workspace_size(const gtr_swiglu_args* a) {
  int64_t M;
  if (!a || swiglu_check(a, &M, false) != GTR_OK) return 0;
  return swiglu_layout(M, a->d, a->hidden).total;
}

extern "C" gtr_status gtr_spatial_swiglu(const gtr_swiglu_args* a, hipStream_t stream) {
  if (!a) return GTR_ERR_NULL;
  int64_t M;
  gtr_status st = swiglu_check(a, &M, true);
  if (st != GTR_OK) return st;
  const SwigluLayout lay = swiglu_layout(M, a->d, a->hidden);
  char* ws = static_cast<char*>(a->workspace);
  _Float16* Hb = reinterpret_cast<_Float16*>(ws + lay.h_off);
  const bool bf = a->dtype == GTR_BF16;

  GatedConvArgs gc{a->x, a->w_gate, a->w_value, a->conv_w, a->conv_b, Hb, a->H, a->W, a->d, a->hidden, a->B, 0, 0};
  const int64_t tiles = (int64_t)a->B * ((a->H + kFH - 1) / kFH) * ((a->W + kFW - 1) / kFW);
  const int64_t wgs = tiles * (a->hidden / kFN);
  for (int64_t first = 0; first < wgs; first += kLaunchWgs) {
    gc.first = (int)first;
    gc.count = (int)(wgs - first < kLaunchWgs ? wgs - first : kLaunchWgs);
    if (bf)
      hipLaunchKernelGGL(gated_conv_kernel<GTR_BF16>, dim3((unsigned)gc.count), dim3(64 * kFWaves), 0, stream, gc);
    else
      hipLaunchKernelGGL(gated_conv_kernel<GTR_F16>, dim3((unsigned)gc.count), dim3(64 * kFWaves), 0, stream, gc);
    if (hipGetLastError() != hipSuccess) return GTR_ERR_HIP;
  }

  const int ks = out_ksplit(M, a->d, a->hidden);
  float* part = reinterpret_cast<float*>(ws + lay.part_off);
  GemmArgs g3{Hb, a->w_out, a->y, part, (int)M, a->d, a->hidden, a->y_dtype, ks, nullptr, ks == 1 ? a->residual : nullptr};
  if (bf)
    launch_gemm<GTR_F16, GTR_BF16, GTR_F16, false>(g3, stream);
  else
    launch_gemm<GTR_F16, GTR_F16, GTR_F16, false>(g3, stream);
  if (hipGetLastError() != hipSuccess) return GTR_ERR_HIP;
  if (ks > 1) {
    const int64_t n4 = M * a->d / 4;
    hipLaunchKernelGGL(ksplit_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, stream, part, a->y,
                       n4, ks, (int)a->y_dtype, a->residual);
  }
  return hipGetLastError() == hipSuccess ? GTR_OK : GTR_ERR_HIP;
}

// ---------------------------------------------------------------------------
// gtr_gemm: C = A B^T (+ bias) (+ res) through launch_gemm, K in one slice.
// ---------------------------------------------------------------------------
static gtr_status gemm_check(const gtr_gemm_args* a) {
  if (a->M <= 0 || a->N <= 0 || a->K <= 0 || a->a_tokens < 0 || a->c_tokens < 0) return GTR_ERR_SHAPE;
  if (a->N % 64 || a->K % 64) return GTR_ERR_UNSUPPORTED;
  if (a->a_tokens && a->M % a->a_tokens) return GTR_ERR_SHAPE;
  if (a->c_tokens) {
    if (a->c_heads <= 0 || a->c_head_dim <= 0 || a->M % a->c_tokens) return GTR_ERR_SHAPE;
    if (a->c_head_dim % 4 || a->N % ((int64_t)a->c_heads * a->c_head_dim) || a->res) return GTR_ERR_UNSUPPORTED;
  }
  if ((a->a_dtype != GTR_F16 && a->a_dtype != GTR_BF16) || a->b_dtype != a->a_dtype) return GTR_ERR_UNSUPPORTED;
  if (a->c_dtype != GTR_F16 && a->c_dtype != GTR_BF16 && a->c_dtype != GTR_F32) return GTR_ERR_UNSUPPORTED;
  if (a->row_norm && (a->row_norm != 1 || a->a_tokens || !(a->row_norm_eps >= 0.f && a->row_norm_eps < 1e30f)))
    return GTR_ERR_UNSUPPORTED;
  if (a->M > 0x7fffffff - 128 || ((a->M + kGemmBM - 1) / kGemmBM) * (a->N / kGemmBN) > 0x7fffffff)
    return GTR_ERR_SHAPE;
  if (!a->a || !a->b || !a->c) return GTR_ERR_NULL;
  const uintptr_t mis = reinterpret_cast<uintptr_t>(a->a) | reinterpret_cast<uintptr_t>(a->b) |
                        reinterpret_cast<uintptr_t>(a->c) | reinterpret_cast<uintptr_t>(a->bias) |
                        reinterpret_cast<uintptr_t>(a->res);
  if (mis & 15u) return GTR_ERR_UNSUPPORTED;
  const size_t es = dtype_size(a->a_dtype);
  auto ovl = [](const void* p, size_t pb, const void* q, size_t qb) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(p), y = reinterpret_cast<uintptr_t>(q);
    return q && x < y + qb && y < x + pb;
  };
  const size_t cb = (size_t)a->M * a->N * dtype_size(a->c_dtype);
  // C may be res itself (an in-place residual: each element is read, then
  // written, by one thread), not any other input
  if (ovl(a->c, cb, a->a, (size_t)a->M * a->K * es) || ovl(a->c, cb, a->b, (size_t)a->N * a->K * es) ||
      ovl(a->c, cb, a->bias, (size_t)a->N * 4) || (a->res != a->c && ovl(a->c, cb, a->res, cb)))
    return GTR_ERR_ALIAS;
  return GTR_OK;
}

extern "C" gtr_status gtr_gemm(const gtr_gemm_args* a, hipStream_t stream) {
  if (!a) return GTR_ERR_NULL;
  const gtr_status st = gemm_check(a);
  if (st != GTR_OK) return st;
  GemmArgs g{a->a, a->b, a->c, nullptr, (int)a->M, a->N, a->K, (int)a->c_dtype, 1, a->bias, a->res,
             a->a_tokens, a->c_tokens, a->c_tokens ? a->c_heads : 0, a->c_tokens ? a->c_head_dim : 0,
             a->row_norm ? a->row_norm_eps : 0.f, 1};
  if (a->a_dtype == GTR_BF16) {
    if (a->row_norm)
      launch_gemm<GTR_BF16, GTR_BF16, GTR_BF16, true>(g, stream);
    else
      launch_gemm<GTR_BF16, GTR_BF16, GTR_BF16, false>(g, stream);
  } else {
    if (a->row_norm)
      launch_gemm<GTR_F16, GTR_F16, GTR_F16, true>(g, stream);
    else
      launch_gemm<GTR_F16, GTR_F16, GTR_F16, false>(g, stream);
  }
  return hipGetLastError() == hipSuccess ? GTR_OK : GTR_ERR_HIP;
}
