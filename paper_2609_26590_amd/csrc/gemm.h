// The matrix products of the block on gfx950: C = A B^T in work-group tiles
// whose operands go from memory straight to LDS (global_load_lds_dwordx4), a
// ring of S stages of 64-deep K steps.
#pragma once

#include <hip/hip_runtime.h>

#include "gtr.h"
#include "gtr_device.h"

namespace gtr {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned int w4 __attribute__((ext_vector_type(4)));

// 8 consecutive K elements of one row as an MFMA operand. DT is the dtype of
// the matrix in memory, MT the operand type (GTR_F16 or GTR_BF16).
template <int DT, int MT>
struct Operand;
template <>
struct Operand<GTR_F16, GTR_F16> {
  typedef h8 T;
  static __device__ __forceinline__ T get(w4 raw) { return __builtin_bit_cast(T, raw); }
};
template <>
struct Operand<GTR_BF16, GTR_BF16> {
  typedef bf8 T;
  static __device__ __forceinline__ T get(w4 raw) { return __builtin_bit_cast(T, raw); }
};
template <>
struct Operand<GTR_BF16, GTR_F16> {  // bf16 weights against fp16 activations
  typedef h8 T;
  static __device__ __forceinline__ T get(w4 raw) {
    T r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned int u = raw[e];
      r[2 * e] = (_Float16)__builtin_bit_cast(float, u << 16);
      r[2 * e + 1] = (_Float16)__builtin_bit_cast(float, u & 0xffff0000u);
    }
    return r;
  }
};

__device__ __forceinline__ f4 mfma(const h8& a, const h8& b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma(const bf8& a, const bf8& b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 4 consecutive elements of dtype dt at element offset off, as floats.
__device__ __forceinline__ void load4(const void* base, int dt, int64_t off, float (&x)[4]) {
  if (dt == GTR_F32) {
    const f4 v = *reinterpret_cast<const f4*>(static_cast<const float*>(base) + off);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = v[e];
  } else if (dt == GTR_F16) {
    const h4 v = *reinterpret_cast<const h4*>(static_cast<const _Float16*>(base) + off);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = (float)v[e];
  } else {
    typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
    const u16x4 v = *reinterpret_cast<const u16x4*>(static_cast<const unsigned short*>(base) + off);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = bf16_bits_to_f32(v[e]);
  }
}

// ---------------------------------------------------------------------------
// Memory straight to LDS: lane l's 16 bytes at g go to LDS byte lds + 16 l (lds
// wave-uniform). The instruction writes no register, so nothing the compiler
// tracks is in flight; it does not know of the transfer either, and every use
// of the data is behind ring_wait. M0, which holds the LDS address, is reserved:
// the compiler allocates nothing to it and warns when it is named as clobbered, so
// a kernel with these transfers must hold no other instruction that reads M0 (the
// tests check the listing for one).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void dma16(const void* g, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(g) : "memory");
}
// Waits until at most N of this wave's transfers are in flight and its LDS
// reads are done, then for the work-group: behind it every wave sees the stages
// all but the last N transfers filled, and a stage that was read before it may
// be overwritten. (Loads and stores the compiler issues besides only make the
// wait longer: vmcnt counts them too, in order.)
template <int N>
__device__ __forceinline__ void ring_wait() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
// The barrier alone, LDS accesses done.
__device__ __forceinline__ void ring_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// LDS rows of 64 K elements (128 bytes, 8 pieces of 16): piece c of row r sits
// at c ^ kSwz64(r). ds_read_b128 serves 32 lanes at a time from 32 distinct
// 16-byte slots (address / 16 mod 32); the operand reads (16 rows x 2 pieces
// per 32 lanes) then hit 32 of them: rows r, r + 4, r + 8, r + 12 share a slot
// up to the piece, and the swizzle gives them 4 disjoint piece pairs. A transfer
// to LDS fills 8 whole rows in order, whatever the swizzle (its lanes fetch the
// pieces of a row in swizzled order).
constexpr int kPitch64 = 64;
__device__ __forceinline__ int kSwz64(int r) { return ((r >> 2) & 3) << 1; }

struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  float* part;
  int M, N, K;
  int cdt;     // dtype of C (GTR_F32 / GTR_F16 / GTR_BF16)
  int ksplit;  // number of K slices (1: none)
  const float* bias;  // [N] float32 added to every row, or null (ksplit = 1 only)
  const void* res;    // [M][N] in C's dtype added elementwise (a residual), or null (ksplit = 1 only)
  // head-major operands (ksplit = 1 only; 0: row-major):
  int64_t a_tokens;   // A is [M / a_tokens][K / 64][a_tokens][64]: row m = (image m / a_tokens, token
                      // m % a_tokens), K step s = head s (a head concat read in place)
  int64_t c_tokens;   // C is written [N / (c_heads c_dim)][M / c_tokens][c_heads][c_tokens][c_dim]
  int c_heads, c_dim;
  float ln_eps;       // the row normalisation's epsilon (kernels with LN != 0)
  int cols;           // column tiles a work-group takes one after the other
};

// Adds the sum and the sum of squares of a piece's 8 elements about the shift.
// `one` is 1 and not known to the compiler, which then converts an fp16 element
// and subtracts in one instruction (v_fma_mix_f32).
template <int ADT>
__device__ __forceinline__ void piece_stats(const w4& v, float one, float shift, float& s, float& q) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const unsigned u = v[e];
    float d0, d1;
    if constexpr (ADT == GTR_F16) {
      const unsigned short lo = (unsigned short)(u & 0xffffu), hi = (unsigned short)(u >> 16);
      d0 = fmaf((float)__builtin_bit_cast(_Float16, lo), one, -shift);
      d1 = fmaf((float)__builtin_bit_cast(_Float16, hi), one, -shift);
    } else {
      d0 = __builtin_bit_cast(float, u << 16) - shift;
      d1 = __builtin_bit_cast(float, u & 0xffff0000u) - shift;
    }
    s += d0;
    q = fmaf(d0, d0, q);
    s += d1;
    q = fmaf(d1, d1, q);
  }
}
// Adds a piece's 8 elements, in their order.
template <int BDT>
__device__ __forceinline__ void piece_sum(const w4& v, float one, float& s) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const unsigned u = v[e];
    if constexpr (BDT == GTR_F16) {
      const unsigned short lo = (unsigned short)(u & 0xffffu), hi = (unsigned short)(u >> 16);
      s = fmaf((float)__builtin_bit_cast(_Float16, lo), one, s);
      s = fmaf((float)__builtin_bit_cast(_Float16, hi), one, s);
    } else {
      s += __builtin_bit_cast(float, u << 16);
      s += __builtin_bit_cast(float, u & 0xffff0000u);
    }
  }
}
template <int ADT>
__device__ __forceinline__ float first_elem(unsigned u) {
  const unsigned short lo = (unsigned short)(u & 0xffffu);
  return ADT == GTR_F16 ? (float)__builtin_bit_cast(_Float16, lo) : __builtin_bit_cast(float, u << 16);
}

// Mean and 1 / sqrt(var + eps) of the BM rows of A from row mb on, over K
// columns, into st: 8 lanes per row (lane l takes pieces l, l + 8, .., the order of
// LN = 1's sums), BM / NW rows per wave, from memory (the rows the ring reads
// next). Squares are taken about the row's first element, so that a mean large
// next to the spread costs no precision.
template <int ADT, int BM, int NW>
__device__ __forceinline__ void row_stats(const GemmArgs& g, int mb, int wave, int lane, f2* st) {
  constexpr int RW = BM / NW, G = RW % 16 == 0 ? 2 : 1, U = 6;  // rows per wave; groups of 8 rows, pieces in flight
  static_assert(RW % (8 * G) == 0, "rows split evenly over the waves");
  const int l = lane & 7, np = g.K / 8;
  const float inv = 1.f / (float)g.K;
  float one = 1.f;
  asm volatile("" : "+v"(one));
#pragma unroll 1
  for (int r0 = wave * RW; r0 < (wave + 1) * RW; r0 += 8 * G) {
    const w4* p[G];
    float sh[G], s[G], q[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      p[u] = reinterpret_cast<const w4*>(static_cast<const unsigned short*>(g.A) +
                                         (int64_t)min(mb + r0 + 8 * u + (lane >> 3), g.M - 1) * g.K);
      sh[u] = s[u] = q[u] = 0.f;
    }
#pragma unroll 1
    for (int c = 0; c < np; c += 8 * U) {
      w4 v[G][U];
#pragma unroll
      for (int u = 0; u < G; ++u)
#pragma unroll
        for (int x = 0; x < U; ++x) v[u][x] = p[u][c + 8 * x + l < np ? c + 8 * x + l : l];
      if (c == 0)
#pragma unroll
        for (int u = 0; u < G; ++u) sh[u] = __shfl(first_elem<ADT>(v[u][0][0]), lane & ~7, kWave);
#pragma unroll
      for (int x = 0; x < U; ++x)
        if (c + 8 * x < np)  // K is a multiple of 64: all lanes or none
#pragma unroll
          for (int u = 0; u < G; ++u) piece_stats<ADT>(v[u][x], one, sh[u], s[u], q[u]);
    }
#pragma unroll
    for (int u = 0; u < G; ++u) {
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) {
        s[u] += __shfl_xor(s[u], o, kWave);
        q[u] += __shfl_xor(q[u], o, kWave);
      }
      const float m1 = s[u] * inv;
      if (l == 0) st[r0 + 8 * u + (lane >> 3)] = f2{sh[u] + m1, rsqrtf(fmaxf(q[u] * inv - m1 * m1, 0.f) + g.ln_eps)};
    }
  }
}

// C[M][N] = A[M][K] * B[N][K]^T (+ bias) (+ res), row-major or head-major, K a
// multiple of 64, N a multiple of BN. WM x WN waves; each holds a (BM / WM) x
// (BN / WN) block of 16 x 16 MFMA tiles. Rows past M are read from row M - 1 and
// not stored. With ksplit > 1, K is cut into ksplit slices whose partial
// products go to part + slice * M * N (float32) for ksplit_reduce_kernel.
//
// What bounds it: with the operands staged through registers (four K steps in
// flight, 64 x 64 tiles) a 64-deep step took about 1,000 cycles against 256 of
// MFMA work, most of it the chain load -> register -> LDS -> register. The
// transfers straight to LDS take the registers and the LDS writes out of that
// chain, and free the registers that larger tiles need: 128 x 192 tiles move
// 2.4 times fewer operand bytes per product than 64 x 64. Stages: two for the
// large tiles, where the second work-group of a CU covers the wait (12800 x 1920
// x 384 in 128 x 128 tiles 68 us with three, which leave room for one work-group,
// 39 with two); three for 64 x 64, whose grids are small and whose operands come
// from beyond the L2 (1600 x 384 x 1536 over rotating weights 13.8 us with two,
// 10.4 with three, 10.6 with four); three for 64 x 128 where each CU has one
// work-group (two against three, operands from HBM: 4150 x 384 x 1536 21.7 against
// 15.1, 1600 x 768 x 3072 39 against 25; from cache 13.2 against 13.7, 27.8 against
// 23.2). Measured (us, operands staged through registers -> straight to LDS, operands
// from HBM): 12800 x 1920 x 384 with LN 62.7 -> 39.9, 8300 x 1920 x 384 with LN
// 43.4 -> 33.9, 12800 x 384 x 1536 37.2 -> 31.4, 12800 x 384 x 384 16.8 -> 13.3,
// 1600 x 1920 x 384 with LN 12.3 -> 10.6, 1600 x 384 x 384 5.6 -> 5.0; 1600 x 384 x
// 1536 10.3 -> 10.4.
//
// A work-group takes `cols` column tiles of its row block one after the other
// (one transfer chain across them), so that the row statistics of LN = 2 are
// paid once per `cols` tiles.
//
// LN: every row of A is normalised over its K columns (A' = (A - mu) / sqrt(var
// + eps), a layer normalisation without affine weights, which the caller folds
// into B and the bias) inside the product: the MFMAs multiply the raw A, the
// row sums of B are taken from the operands as they are read, and the
// epilogue forms rs_m (C_mn - mu_m rowsum_n), which is A' B^T in real arithmetic.
// The row sums and the statistics are taken in one fixed order for every tile (8
// lanes per row, pieces l, l + 8, ..), so that a product rounds alike in all of
// them; an MFMA against ones for the sums would take 0.5 us less at 1600 x 1920 x
// 384 and round another way.
// The statistics come from the operands as they are read (LN = 1: no extra
// load, for small tiles and short chains) or from a pass over the rows before
// the loop (LN = 2: no extra registers in the loop, for the larger tiles).
// Both need K in one slice and a row-major A, LN = 1 also cols = 1. (In 128 x 192
// tiles LN = 2 spills two registers, stored once before the products and loaded
// once in the epilogue of a tile.)
//
// KH = 2 sums the two 32-deep halves of every step apart (grids of fewer 64 x 64
// tiles than CUs).
//
// The grid is one-dimensional. Work-group b runs on XCD b % 8 (round-robin
// dispatch), and each XCD takes a contiguous range of the order (slice, row
// block, column group), column groups fastest: the work-groups that read the
// same rows of A share one XCD's L2.
template <int ADT, int BDT, int MT, int BM, int BN, int WM, int WN, int S, int LN, int KH>
__global__ void __launch_bounds__(64 * WM * WN)
__attribute__((amdgpu_waves_per_eu(WM * WN == 8 ? 4 : 2))) gemm_ring_kernel(GemmArgs g) {
  typedef Operand<ADT, MT> OA;
  typedef Operand<BDT, MT> OB;
  constexpr int NW = WM * WN;                            // waves
  constexpr int TI = BM / (16 * WM), TJ = BN / (16 * WN);  // MFMA tiles per wave
  constexpr int PA = BM / 8 / NW, PB = BN / 8 / NW;      // transfers per wave per step
  constexpr int PL = PA + PB;
  constexpr int SA = BM * kPitch64, SB = BN * kPitch64;  // elements per stage
  static_assert(S == 2 || S == 3, "stages");
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tiles split evenly over the waves");
  __shared__ __attribute__((aligned(1024))) unsigned short ring[S * (SA + SB)];
  __shared__ f2 lnp[LN == 1 ? WN : 1][LN == 1 ? BM : 1];  // LN = 1: per tile row, the waves' sums and squares

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wmi = wave / WN, wni = wave % WN;
  const int r16 = lane & 15, kq = lane >> 4;
  const int gx = (g.M + BM - 1) / BM, ntile = g.N / BN, gy = (ntile + g.cols - 1) / g.cols;
  const int T = gx * gy * g.ksplit, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int jt = xcd * (T >> 3) + min(xcd, T & 7) + slot;
  const int by = jt % gy, bxz = jt / gy, bx = bxz % gx, bz = bxz / gx;
  const int mb = bx * BM;
  int nb = by * g.cols * BN;
  const int tiles = min(g.cols, ntile - by * g.cols);
  const int wm = wmi * (BM / WM), wn = wni * (BN / WN);
  const int64_t K = g.K;
  const int allsteps = g.K / 64;
  const int s_per = (allsteps + g.ksplit - 1) / g.ksplit;
  const int s0 = g.ksplit > 1 ? bz * s_per : 0;
  const int steps = max(0, min(s0 + s_per, allsteps) - s0);
  const int total = steps * tiles;

  // this lane's global pieces; transfer q of the wave fills rows 8 (wave + NW q) ..
  const char* ga[PA];
  const char* gb[PB];
  const int64_t ast = (g.a_tokens ? 64 * g.a_tokens : 64) * 2;  // bytes from one K step of A to the next
  const int lr = lane >> 3;
#pragma unroll
  for (int q = 0; q < PA; ++q) {
    const int row = 8 * (wave + NW * q) + lr, col = (lane & 7) ^ kSwz64(row);
    const unsigned m = (unsigned)min(mb + row, g.M - 1), at = g.a_tokens ? (unsigned)g.a_tokens : 1u;
    ga[q] = static_cast<const char*>(g.A) +
            ((g.a_tokens ? ((int64_t)(m / at) * (K / 64) * at + m % at) * 64 : (int64_t)m * K) + 8 * col) * 2 + s0 * ast;
  }
#pragma unroll
  for (int q = 0; q < PB; ++q) {
    const int row = 8 * (wave + NW * q) + lr, col = (lane & 7) ^ kSwz64(row);
    gb[q] = static_cast<const char*>(g.B) + ((int64_t)(nb + row) * K + 8 * col) * 2 + (int64_t)s0 * 128;
  }
  const unsigned lbase = lds_addr(ring) + wave * 1024;
  const int64_t arew = -(int64_t)steps * ast, brew = (BN * K - (int64_t)steps * 64) * 2;
  int ik = 0, ibuf = 0;  // K step within its tile and ring buffer of the next transfer
  auto issue = [&]() {
    const unsigned l = lbase + ibuf * (SA + SB) * 2;
#pragma unroll
    for (int q = 0; q < PA; ++q) {
      dma16(ga[q], l + NW * 1024 * q);
      ga[q] += ast;
    }
#pragma unroll
    for (int q = 0; q < PB; ++q) {
      dma16(gb[q], l + SA * 2 + NW * 1024 * q);
      gb[q] += 128;
    }
    ibuf = ibuf + 1 == S ? 0 : ibuf + 1;
    if (++ik == steps) {  // the same rows of A again, the next BN rows of B
      ik = 0;
#pragma unroll
      for (int q = 0; q < PA; ++q) ga[q] += arew;
#pragma unroll
      for (int q = 0; q < PB; ++q) gb[q] += brew;
    }
  };

  f4 acc[KH][TI][TJ];  // KH = 2: one set for each 32-deep half of a step
  float bs[TJ][2];     // LN: sums of B's row r16 of tile j over this lane's pieces kq and 4 + kq

  float sh[TI], sa[TI], sq[TI];  // LN = 1: row statistics from the operands as they are read
  float one = 1.f;
  asm volatile("" : "+v"(one));
#pragma unroll
  for (int i = 0; i < TI; ++i) sh[i] = sa[i] = sq[i] = 0.f;
  auto mma = [&](int buf) {
    const unsigned short* As = ring + buf * (SA + SB);
    const unsigned short* Bs = As + SA;
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // the 32-deep halves of the step
      const int pc = (4 * h + kq) ^ kSwz64(r16);
      w4 ra[TI], rb[TJ];
#pragma unroll
      for (int j = 0; j < TJ; ++j) rb[j] = *reinterpret_cast<const w4*>(&Bs[(wn + 16 * j + r16) * kPitch64 + 8 * pc]);
#pragma unroll
      for (int i = 0; i < TI; ++i) ra[i] = *reinterpret_cast<const w4*>(&As[(wm + 16 * i + r16) * kPitch64 + 8 * pc]);
      typename OB::T fb[TJ];
#pragma unroll
      for (int j = 0; j < TJ; ++j) fb[j] = OB::get(rb[j]);
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const typename OA::T fa = OA::get(ra[i]);
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[h % KH][i][j] = mfma(fb[j], fa, acc[h % KH][i][j]);  // C^T tiles
      }
      if constexpr (LN != 0) {
#pragma unroll
        for (int j = 0; j < TJ; ++j) piece_sum<BDT>(rb[j], one, bs[j][h]);
      }
      if constexpr (LN == 1) {  // every (row block, half) of A is read by WN waves: wave wni takes its share
#pragma unroll
        for (int i = 0; i < TI; ++i)
          if ((2 * i + h) % WN == wni) piece_stats<ADT>(ra[i], one, sh[i], sa[i], sq[i]);
      }
    }
  };

#pragma unroll
  for (int q = 0; q < S - 1; ++q)
    if (q < total) issue();
  static_assert(TI <= 4, "lane kq keeps the statistics of row block kq");
  f2 lst = {0.f, 1.f};  // LN: mean and 1 / sqrt(var + eps) of row 16 kq + r16 of this wave's block
  if constexpr (LN == 2) {  // through the last stage, which no transfer has been issued to
    f2* st = reinterpret_cast<f2*>(ring + (S - 1) * (SA + SB));
    row_stats<ADT, BM, NW>(g, mb, wave, lane, st);
    ring_sync();
    lst = st[wm + 16 * min(kq, TI - 1) + r16];
    ring_sync();
  }
  int f = 0, buf = 0;  // step of the whole run, its ring buffer
  for (int t = 0; t < tiles; ++t) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      bs[j][0] = bs[j][1] = 0.f;
#pragma unroll
      for (int q = 0; q < KH * TI; ++q) acc[q / TI][q % TI][j] = f4{0.f, 0.f, 0.f, 0.f};
    }
    for (int k = 0; k < steps; ++k, ++f) {
      // this step's stage has landed (the stages after it may be in flight), and
      // every wave is done with the one before it, which the next transfer fills
      const int rem = total - 1 - f;  // steps after this one
      if (S == 3 && rem >= 1)
        ring_wait<PL>();
      else
        ring_wait<0>();
      if (rem >= S - 1) issue();
      if constexpr (LN == 1) {
        if (f == 0) {  // the shift of each row: its first element
#pragma unroll
          for (int i = 0; i < TI; ++i) {
            const int row = wm + 16 * i + r16;
            sh[i] = first_elem<ADT>(ring[row * kPitch64 + 8 * kSwz64(row)]);
          }
        }
      }
      mma(buf);
      buf = buf + 1 == S ? 0 : buf + 1;
    }

    if constexpr (LN == 1) {  // (one column tile)
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        sa[i] += __shfl_xor(sa[i], 16, kWave);
        sq[i] += __shfl_xor(sq[i], 16, kWave);
        sa[i] += __shfl_xor(sa[i], 32, kWave);
        sq[i] += __shfl_xor(sq[i], 32, kWave);
        if (kq == 0) lnp[wni][wm + 16 * i + r16] = f2{sa[i], sq[i]};
      }
      ring_sync();
      const float inv = 1.f / (float)g.K;
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        float a = 0.f, q = 0.f;
#pragma unroll
        for (int p = 0; p < WN; ++p) {
          const f2 v = lnp[p][wm + 16 * i + r16];
          a += v[0];
          q += v[1];
        }
        const float m1 = a * inv;
        if (kq == i) lst = f2{sh[i] + m1, rsqrtf(fmaxf(q * inv - m1 * m1, 0.f) + g.ln_eps)};
      }
    }

    // lane holds C[row 16i + r16][columns 16j + 4kq .. 16j + 4kq + 3] of this
    // wave's block (the products above are C^T tiles): one 4-element store each
    void* C = g.ksplit > 1 ? static_cast<void*>(g.part + (int64_t)bz * g.M * g.N) : g.C;
    const int cdt = g.ksplit > 1 ? (int)GTR_F32 : g.cdt;
    const bool hmc = g.ksplit == 1 && g.c_tokens != 0;
    const unsigned tokens = hmc ? (unsigned)g.c_tokens : 1u, cdim = hmc ? (unsigned)g.c_dim : 1u;
    const unsigned hd = hmc ? (unsigned)(g.c_heads * g.c_dim) : 1u, img = (unsigned)g.M / tokens;
    int64_t coloff[TJ];
    f4 cs[TJ];  // LN: row sums of B for the lane's four columns
    if constexpr (LN != 0) {
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        float s2[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          s2[h] = bs[j][h] + __shfl_xor(bs[j][h], 16, kWave);
          s2[h] += __shfl_xor(s2[h], 32, kWave);
        }
        const float sum = s2[0] + s2[1];
#pragma unroll
        for (int e = 0; e < 4; ++e) cs[j][e] = __shfl(sum, 4 * kq + e, kWave);
      }
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const unsigned n0 = (unsigned)(nb + wn + 16 * j + 4 * kq);
      const unsigned p = n0 / hd, r = n0 - p * hd, h = r / cdim;
      coloff[j] = hmc ? ((int64_t)p * img * g.c_heads * tokens + (int64_t)h * tokens) * cdim + (r - h * cdim) : n0;
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      const unsigned m = (unsigned)(mb + wm + 16 * i + r16);
      f2 st = {0.f, 1.f};
      if (LN != 0) st = f2{__shfl(lst[0], 16 * i + r16, kWave), __shfl(lst[1], 16 * i + r16, kWave)};
      if (m >= (unsigned)g.M) continue;
      const int64_t rowoff = hmc ? ((int64_t)(m / tokens) * g.c_heads * tokens + m % tokens) * cdim : (int64_t)m * g.N;
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const int n0 = nb + wn + 16 * j + 4 * kq;
        const int64_t off = rowoff + coloff[j];
        f4 sum = acc[0][i][j];
        if constexpr (KH == 2) sum += acc[1][i][j];
        float x[4] = {sum[0], sum[1], sum[2], sum[3]};
        if constexpr (LN != 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = st[1] * (x[e] - st[0] * cs[j][e]);
        }
        if (g.ksplit == 1 && g.bias) {
          const f4 bv = *reinterpret_cast<const f4*>(g.bias + n0);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] += bv[e];
        }
        if (g.ksplit == 1 && g.res) {  // (row-major C)
          float rv[4];
          load4(g.res, cdt, off, rv);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] += rv[e];
        }
        store_n<4>(C, cdt, off, x);
      }
    }
    nb += BN;
  }
}

// The same product in 64 x 64 tiles with the operands staged through registers
// (16-byte loads, four K steps in flight, written to two LDS stages a step before
// they are multiplied), 8 waves: the waves kh = 0 and kh = 1 take the first and
// the second 32-deep half of every step, and their sums meet through LDS at the
// end. LN = 1 as above, the statistics taken from the pieces as they pass through
// registers: per thread and step one piece of A and one of B, a step before the
// MFMAs that need them, so that they run beside the waits.
//
// For grids of fewer tiles than CUs (see launch_gemm), where one work-group's
// chain of K steps is the whole time and a second work-group covers no wait.
// Measured there against the transfers straight to LDS (us, f16 / bf16): 400 x 960 x
// 192 with LN 5.2 / 5.5 against 5.6 / 6.0, 1600 x 384 x 384 with LN 6.4 / 6.6
// against 7.0 / 7.6, 1600 x 192 x 768 with LN 8.4 / 8.5 against 9.6 / 10.5; 1600 x 384
// x 2304 12.5 against 13.0, operands from HBM 14.0 against 15.6; but 1600 x 384 x 384
// 5.3 against 5.0 and 1600 x 384 x 1536 9.8 against 9.7.
template <int ADT, int BDT, int MT, int LN>
__global__ void __launch_bounds__(512) gemm_staged_kernel(GemmArgs g) {
  typedef Operand<ADT, MT> OA;
  typedef Operand<BDT, MT> OB;
  constexpr int BM = 64, BN = 64, TI = 2, TJ = 2;  // tile; MFMA tiles per wave
  constexpr int D = 4;                             // K steps of loads in flight
  static_assert(BM * BN * 4 <= 2 * BM * kPitch64 * 2, "the second halves' sums fit in As");
  __shared__ __attribute__((aligned(16))) unsigned short As[2][BM * kPitch64];
  __shared__ __attribute__((aligned(16))) unsigned short Bs[2][BN * kPitch64];
  __shared__ f2 lnst[LN ? BM : 1];     // per tile row: mean, 1 / sqrt(var + eps)
  __shared__ float lncs[LN ? BN : 1];  // per tile column: the row sum of B

  const int w = (threadIdx.x >> 6) & 3, kh = threadIdx.x >> 8, lane = threadIdx.x & 63;
  const int r16 = lane & 15, kq = lane >> 4;
  const int gx = (g.M + BM - 1) / BM, gy = g.N / BN;
  const int T = gx * gy * g.ksplit, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int jt = xcd * (T >> 3) + min(xcd, T & 7) + slot;
  const int by = jt % gy, bxz = jt / gy, bx = bxz % gx, bz = bxz / gx;
  const int mb = bx * BM, nb = by * BN;
  const int wm = (w >> 1) * (BM / 2), wn = (w & 1) * (BN / 2);
  const int64_t K = g.K;
  const int allsteps = g.K / 64;
  const int s_per = (allsteps + g.ksplit - 1) / g.ksplit;
  const int s0 = g.ksplit > 1 ? bz * s_per : 0;
  const int s1 = min(s0 + s_per, allsteps);

  // this thread's piece of each operand: row prow of the tile, 16-byte column threadIdx % 8
  const int prow = threadIdx.x >> 3, pcol = threadIdx.x & 7;
  const unsigned m = (unsigned)min(mb + prow, g.M - 1), at = g.a_tokens ? (unsigned)g.a_tokens : 1u;
  const w4* ga = reinterpret_cast<const w4*>(
      static_cast<const unsigned short*>(g.A) +
      (g.a_tokens ? ((int64_t)(m / at) * (K / 64) * at + m % at) * 64 : (int64_t)m * K) + 8 * pcol);
  const w4* gb = reinterpret_cast<const w4*>(static_cast<const unsigned short*>(g.B) + (int64_t)(nb + prow) * K + 8 * pcol);
  const int64_t ast = g.a_tokens ? 8 * g.a_tokens : 8;  // 16-byte pieces from one K step of A to the next
  const int at_lds = prow * kPitch64 + 8 * (pcol ^ kSwz64(prow));

  f4 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  w4 ra[D], rb[D];
  float sh = 0.f, sa = 0.f, sq = 0.f, sb = 0.f;  // LN: of the pieces staged so far
  auto fetch = [&](int st, int q) {
    ra[q] = ga[ast * st];
    rb[q] = gb[8 * st];
  };
  auto stage = [&](int buf, int q) {
    *reinterpret_cast<w4*>(&As[buf][at_lds]) = ra[q];
    *reinterpret_cast<w4*>(&Bs[buf][at_lds]) = rb[q];
  };
  float one = 1.f;
  asm volatile("" : "+v"(one));
  auto stats = [&](int q) {
    if constexpr (LN != 0) {
      piece_stats<ADT>(ra[q], one, sh, sa, sq);
      piece_sum<BDT>(rb[q], one, sb);
    }
  };
  auto mma = [&](int buf) {
    const int pc = (4 * kh + kq) ^ kSwz64(r16);
    typename OA::T fa[TI];
    typename OB::T fb[TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
      fa[i] = OA::get(*reinterpret_cast<const w4*>(&As[buf][(wm + 16 * i + r16) * kPitch64 + 8 * pc]));
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      fb[j] = OB::get(*reinterpret_cast<const w4*>(&Bs[buf][(wn + 16 * j + r16) * kPitch64 + 8 * pc]));
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) acc[i][j] = mfma(fb[j], fa[i], acc[i][j]);  // C^T tiles
  };
  // The loop runs whole groups of D steps in which every step issues the same
  // loads (past the slice's last step they re-read that step, never used): with
  // no load under a branch the compiler's waits count exactly, so a step waits
  // for the loads of the step it stages, not for the newer ones. The last (steps
  // mod D) steps follow with their loads already in flight.
  if (s1 > s0) {
#pragma unroll
    for (int q = 0; q < D; ++q) fetch(min(s0 + q, s1 - 1), q);
    if constexpr (LN != 0) sh = __shfl(first_elem<ADT>(ra[0][0]), lane & ~7, kWave);  // the row's first element
    stage(0, 0);
    stats(0);
    __syncthreads();
    int sb0 = s0;
    for (; sb0 + D <= s1; sb0 += D) {
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const int st = sb0 + q, buf = (st - s0) & 1;
        fetch(min(st + D, s1 - 1), q);  // slot q was staged before this step
        mma(buf);
        stage(buf ^ 1, (q + 1) % D);  // nobody reads buf ^ 1 now
        if (st + 1 < s1) stats((q + 1) % D);  // past the last step: a re-read
        __syncthreads();
      }
    }
#pragma unroll
    for (int q = 0; q < D - 1; ++q) {
      const int st = sb0 + q, buf = (st - s0) & 1;
      if (st < s1) {
        mma(buf);
        if (st + 1 < s1) {
          stage(buf ^ 1, (q + 1) % D);
          stats((q + 1) % D);
        }
        __syncthreads();
      }
    }
  }

  if constexpr (LN != 0) {  // the 8 threads of a row combine; the first of each stores
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      sa += __shfl_xor(sa, o, kWave);
      sq += __shfl_xor(sq, o, kWave);
      sb += __shfl_xor(sb, o, kWave);
    }
    if (pcol == 0) {
      const float inv = 1.f / (float)g.K, m1 = sa * inv;
      lnst[prow] = f2{sh + m1, rsqrtf(fmaxf(sq * inv - m1 * m1, 0.f) + g.ln_eps)};
      lncs[prow] = sb;
    }
  }
  f4* red = reinterpret_cast<f4*>(&As[0][0]) + w * TI * TJ * 64 + lane;
  __syncthreads();  // every wave is past the K loop's last LDS read
  if (kh == 1) {
#pragma unroll
    for (int q = 0; q < TI * TJ; ++q) red[64 * q] = acc[q / TJ][q % TJ];
  }
  __syncthreads();
  if (kh == 1) return;
#pragma unroll
  for (int q = 0; q < TI * TJ; ++q) acc[q / TJ][q % TJ] += red[64 * q];

  // the stores of gemm_ring_kernel
  void* C = g.ksplit > 1 ? static_cast<void*>(g.part + (int64_t)bz * g.M * g.N) : g.C;
  const int cdt = g.ksplit > 1 ? (int)GTR_F32 : g.cdt;
  const bool hmc = g.ksplit == 1 && g.c_tokens != 0;
  const unsigned tokens = hmc ? (unsigned)g.c_tokens : 1u, cdim = hmc ? (unsigned)g.c_dim : 1u;
  const unsigned hd = hmc ? (unsigned)(g.c_heads * g.c_dim) : 1u, img = (unsigned)g.M / tokens;
  int64_t coloff[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const unsigned n0 = (unsigned)(nb + wn + 16 * j + 4 * kq);
    const unsigned p = n0 / hd, r = n0 - p * hd, h = r / cdim;
    coloff[j] = hmc ? ((int64_t)p * img * g.c_heads * tokens + (int64_t)h * tokens) * cdim + (r - h * cdim) : n0;
  }
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    const int lr = wm + 16 * i + r16;
    const unsigned row = (unsigned)(mb + lr);
    if (row >= (unsigned)g.M) continue;
    const int64_t rowoff = hmc ? ((int64_t)(row / tokens) * g.c_heads * tokens + row % tokens) * cdim : (int64_t)row * g.N;
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int lc = wn + 16 * j + 4 * kq;
      const int64_t off = rowoff + coloff[j];
      float x[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
      if constexpr (LN != 0) {
        const f2 st = lnst[lr];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = st[1] * (x[e] - st[0] * lncs[lc + e]);
      }
      if (g.ksplit == 1 && g.bias) {
        const f4 bv = *reinterpret_cast<const f4*>(g.bias + nb + lc);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] += bv[e];
      }
      if (g.ksplit == 1 && g.res) {  // (row-major C)
        float rv[4];
        load4(g.res, cdt, off, rv);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] += rv[e];
      }
      store_n<4>(C, cdt, off, x);
    }
  }
}

}  // namespace gtr
