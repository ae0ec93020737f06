// The cloud's token-wise connector on the transmitted rows (arXiv
// 2607.27952: Sec. 3.4 applies phi_c to the rows of Eq. 12, H_S = phi_c(X_S);
// Sec. 3.2 defines phi_c as a token-wise connector) for gfx950, bf16:
//
//   xhat = LayerNorm(x) = (x - mean) / sqrt(var + eps) * gamma + beta
//   h    = GELU(W1 xhat + b1)        (GELU with erf)
//   y    = W2 h + b2
//
// for every kept row x. The paper gives no formula for phi_c; this is the
// token-wise connector structure of the model family it uses.
//
//   k_layernorm   one wave per row, fp32 statistics in a fixed order; xhat
//                 rounded to bf16 (the matrix cores' input type).
//   k_gemm_nt     C[m][n] = sum_k A[n][k] B[m][k] (both operands row-major
//                 with k contiguous: weights one output feature per row,
//                 tokens one row each) plus bias, optionally GELU, rounded to
//                 bf16. Block tiles from 32 features x 32 tokens (few rows:
//                 enough blocks to pull the weights through every compute
//                 unit) to 256 x 256 (four waves of 4 x 4
//                 v_mfma_f32_32x32x16_bf16 tiles; many rows); the weights are
//                 the MFMA's A operand. Operands stream through an LDS ring
//                 by LDS DMA, one barrier per stage; the output tile leaves
//                 through the same LDS, so that its stores cover whole rows.
#include <algorithm>
#include <cmath>

#include "last_internal.h"

using namespace last_dev;

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const f32x2_t x = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
}

// ---------------------------------------------------------------- LayerNorm
// One wave per row, 16-byte pieces (8 values): lane l takes pieces l, l + 64,
// ... Rows of up to 64 NP pieces are loaded once into registers (all loads
// in flight together); longer rows stream, reading the row again from cache
// for the deviations and the output. Sums are fp32, each lane's in piece
// order, then across the wave in a fixed order.
constexpr int kLnWaves = 4;

__device__ __forceinline__ void unpack8(const uint4 &w, float *v) {
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = bf16_lo(u[i]);
    v[2 * i + 1] = bf16_hi(u[i]);
  }
}

__device__ __forceinline__ uint4 norm8(const uint4 &w, float mean, float rstd, const float *__restrict__ gamma,
                                       const float *__restrict__ beta, int p) {
  float v[8];
  unpack8(w, v);
  const float4 *g4 = reinterpret_cast<const float4 *>(gamma);
  const float4 *b4 = reinterpret_cast<const float4 *>(beta);
  const float4 ga = g4[2 * p], gb = g4[2 * p + 1], ba = b4[2 * p], bb = b4[2 * p + 1];
  const float g[8] = {ga.x, ga.y, ga.z, ga.w, gb.x, gb.y, gb.z, gb.w};
  const float b[8] = {ba.x, ba.y, ba.z, ba.w, bb.x, bb.y, bb.z, bb.w};
  float y[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) y[i] = (v[i] - mean) * rstd * g[i] + b[i];
  return make_uint4(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]), pack_bf16(y[4], y[5]), pack_bf16(y[6], y[7]));
}

// NP > 0: at most NP pieces per lane, held in registers; NP == 0: streaming.
template <int NP>
__global__ __launch_bounds__(64 * kLnWaves) void k_layernorm(const uint16_t *__restrict__ x,
                                                             const float *__restrict__ gamma,
                                                             const float *__restrict__ beta, int64_t K,
                                                             int Dv, float eps, uint16_t *__restrict__ xn) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * kLnWaves + (threadIdx.x >> 6);
  if (t >= K) return;
  const uint4 *row = reinterpret_cast<const uint4 *>(x + t * Dv);
  uint4 *out = reinterpret_cast<uint4 *>(xn + t * Dv);
  const int np = Dv / 8;
  float v[8];
  if constexpr (NP > 0) {
    uint4 w[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) w[i] = lane + 64 * i < np ? row[lane + 64 * i] : make_uint4(0, 0, 0, 0);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      unpack8(w[i], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) s += v[j];
    }
    const float mean = wave_sum(s) / (float)Dv;
    float c2 = 0.f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      if (lane + 64 * i >= np) break;
      unpack8(w[i], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) c2 = fmaf(v[j] - mean, v[j] - mean, c2);
    }
    const float rstd = 1.0f / sqrtf(wave_sum(c2) / (float)Dv + eps);
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (lane + 64 * i < np) out[lane + 64 * i] = norm8(w[i], mean, rstd, gamma, beta, lane + 64 * i);
  } else {
    float s = 0.f;
    for (int p = lane; p < np; p += 64) {
      unpack8(row[p], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) s += v[j];
    }
    const float mean = wave_sum(s) / (float)Dv;
    float c2 = 0.f;
    for (int p = lane; p < np; p += 64) {
      unpack8(row[p], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) c2 = fmaf(v[j] - mean, v[j] - mean, c2);
    }
    const float rstd = 1.0f / sqrtf(wave_sum(c2) / (float)Dv + eps);
    for (int p = lane; p < np; p += 64) out[p] = norm8(row[p], mean, rstd, gamma, beta, p);
  }
}

// ---------------------------------------------------------------- GEMM
// Block tile TN features x TM tokens on WN x WM computing waves of FN x FM
// v_mfma_f32_32x32x16_bf16 tiles each; all four waves copy. A stage holds KC
// columns of both operands; RING stages live in LDS, filled by LDS DMA
// RING - 1 stages ahead of use. A group of SG 16-column steps' fragments is
// read from LDS while the previous group's products run, and the stage's last
// group is multiplied after the barrier that publishes the next stage, so the
// matrix cores keep busy across it.
//
// Every output element is one chain of the same instruction over ascending
// 16-column steps, whatever the tile: all tiles give the same bits, and a
// row's result does not depend on the batch it came in.
template <int TN_, int TM_, int WN_, int WM_, int KC_, int RING_, int SG_>
struct Tile {
  static constexpr int TN = TN_, TM = TM_, WN = WN_, WM = WM_, KC = KC_, RING = RING_, SG = SG_;
  static constexpr int FN = TN / (32 * WN), FM = TM / (32 * WM);   // 32 x 32 tiles a wave
  static constexpr int RP = KC * 2 / 16;                           // 16-byte pieces of one row of a stage
  static constexpr int APieces = TN * RP, BPieces = TM * RP;       // weights, tokens
  static constexpr int StagePieces = APieces + BPieces;
  static constexpr int Waves = 4;
  static constexpr int PerWave = StagePieces / 64 / Waves;         // DMA instructions a wave and stage
  static constexpr int PerWaveA = APieces / 64 / Waves;
  static constexpr int Groups = KC / 16 / SG;
  static constexpr int OP = TN / 8;                                // 16-byte pieces of one output row
  static_assert(WN * WM <= Waves && FN * 32 * WN == TN && FM * 32 * WM == TM, "wave split");
  static_assert(APieces % (64 * Waves) == 0 && BPieces % (64 * Waves) == 0, "even DMA split");
  static_assert((KC / 16) % SG == 0 && PerWave % Groups == 0, "DMA chunks per step group");
  static_assert(RP == 8 || RP == 16 || RP == 32, "swizzle assumes 8, 16 or 32 pieces a row");
  static_assert(TM * OP <= RING * StagePieces, "the output tile is staged in the ring");
  static_assert(RING * StagePieces * 16 <= 160 * 1024, "LDS");
};
constexpr int kGWaves = 4, kGThreads = 64 * kGWaves;
constexpr int kGK = 64;                      // every reduction length is a multiple of this

// A row's pieces are permuted so that 16 consecutive rows read at one piece
// index hit 16 distinct 16-byte bank groups.
template <int RP>
__device__ __forceinline__ int gperm(int row) {
  return RP == 8 ? (row >> 1) & 7 : row & (RP - 1);
}

// GELU(u) = u (1 + erf(u / sqrt 2)) / 2 with erf from Abramowitz and Stegun,
// Handbook of Mathematical Functions, formula 7.1.26: for x >= 0,
// erfc(x) = (a1 t + ... + a5 t^5) e^(-x^2), t = 1 / (1 + p x), within
// 1.5e-7. With q = erfc(|u| / sqrt 2), GELU is u (1 - q / 2) for u >= 0 and
// u q / 2 below; in fp32 the result stays within 1e-6 (1 + |u|), far under
// the bf16 rounding that follows. One reciprocal and one exponential, where
// a full-precision erf costs several times more in this one-wave-per-SIMD
// epilogue.
__device__ __forceinline__ float gelu(float u) {
  const float x = fabsf(u) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
  float poly = fmaf(1.061405429f, t, -1.453152027f);
  poly = fmaf(poly, t, 1.421413741f);
  poly = fmaf(poly, t, -0.284496736f);
  poly = fmaf(poly, t, 0.254829592f);
  poly *= t;
  const float q = poly * __builtin_amdgcn_exp2f(-(x * x) * 1.4426950408889634f);
  return u >= 0.0f ? u * fmaf(-0.5f, q, 1.0f) : 0.5f * u * q;
}

template <class T>
struct Frags {
  bf16x8_t a[T::SG][T::FN], b[T::SG][T::FM];
};

template <class T, bool GELU>
__global__ __launch_bounds__(kGThreads, 1) void k_gemm_nt(const uint16_t *__restrict__ A,   // [N][Kd]
                                                          const uint16_t *__restrict__ B,   // [M][Kd]
                                                          const float *__restrict__ bias,   // [N]
                                                          int64_t M, int N, int Kd, int n_tiles,
                                                          int blocks_xcd,
                                                          uint16_t *__restrict__ C) {       // [M][N]
  constexpr int FN = T::FN, FM = T::FM, RP = T::RP, SG = T::SG, RING = T::RING;
  __shared__ uint4 ring[RING][T::StagePieces];
  // Blocks are dealt to the 8 XCDs in turn; renumber them so that each XCD
  // runs a contiguous range of tiles, taken 8 token tiles at a time across
  // the feature tiles, which keeps the operands it shares in its own L2.
  const int64_t b = blockIdx.x;
  const int64_t l = b < (int64_t)blocks_xcd * 8 ? (b % 8) * blocks_xcd + b / 8 : b;
  const int64_t band = l / (8 * (int64_t)n_tiles), in_band = l % (8 * (int64_t)n_tiles);
  const int64_t m_tiles = (M + T::TM - 1) / T::TM;
  const int64_t band_rows = std::min<int64_t>(8, m_tiles - band * 8);
  const int64_t mt = band * 8 + in_band % band_rows;
  const int nt = (int)(in_band / band_rows);
  const int n0 = nt * T::TN;
  const int64_t m0 = mt * T::TM;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const bool computes = wave < T::WN * T::WM;
  const int wn = wave / T::WM, wm = wave % T::WM;

  // This wave's DMA instructions q = wave + 4 x: the first APieces / 64 fill
  // the weight rows of a stage, the rest the token rows. The base is the
  // block's first row of the operand (64-bit, wave-uniform), a lane's byte
  // offset from it (under 256 rows) is fixed for the block, and each stage
  // moves the base by KC columns. Rows past the end repeat the last row.
  const char *baseA = (const char *)uniform_ptr((const char *)A + (int64_t)n0 * Kd * 2);
  const char *baseB = (const char *)uniform_ptr((const char *)B + m0 * Kd * 2);
  uint32_t voff[T::PerWave], dst[T::PerWave];
#pragma unroll
  for (int x = 0; x < T::PerWave; ++x) {
    const int q = wave + kGWaves * x;
    const bool isA = x < T::PerWaveA;   // q < APieces / 64
    const int sl = (isA ? q : q - T::APieces / 64) * 64 + lane;
    const int row = sl / RP, slot = sl % RP;
    const int p = slot ^ gperm<RP>(row);
    const int64_t first = isA ? n0 : m0, last_row = (isA ? (int64_t)N : M) - 1;
    const int64_t grow = std::min<int64_t>(first + row, last_row);
    voff[x] = (uint32_t)((grow - first) * Kd * 2 + p * 16);
    dst[x] = __builtin_amdgcn_readfirstlane(lds_u32(&ring[0][(isA ? 0 : T::APieces) + (sl - lane)]));
  }
  constexpr uint32_t kStageBytes = T::StagePieces * 16;
  // Instructions x in [x0, x1) of stage st's DMA.
  auto issue = [&](int st, int x0, int x1) {
    const int64_t col = (int64_t)st * T::KC * 2;
    const uint32_t so = (uint32_t)(st % RING) * kStageBytes;
#pragma unroll
    for (int x = 0; x < T::PerWave; ++x)
      if (x >= x0 && x < x1) dma16(dst[x] + so, (x < T::PerWaveA ? baseA : baseB) + col, voff[x]);
  };

  // Fragment addresses: lane row lane % 32 of every 32-row tile; the piece
  // for k-step ks is 2 ks + lane / 32.
  const int r32 = lane & 31, half = lane >> 5;
  auto load = [&](Frags<T> &f, int st, int grp) {
    const uint4 *sa = ring[st % RING];
    const uint4 *sb = sa + T::APieces;
#pragma unroll
    for (int s = 0; s < SG; ++s) {
      const int piece = 2 * (grp * SG + s) + half;
#pragma unroll
      for (int i = 0; i < FN; ++i) {
        const int row = 32 * FN * wn + 32 * i + r32;
        f.a[s][i] = __builtin_bit_cast(bf16x8_t, sa[row * RP + (piece ^ gperm<RP>(row))]);
      }
#pragma unroll
      for (int j = 0; j < FM; ++j) {
        const int row = 32 * FM * wm + 32 * j + r32;
        f.b[s][j] = __builtin_bit_cast(bf16x8_t, sb[row * RP + (piece ^ gperm<RP>(row))]);
      }
    }
  };

  f32x16_t acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = f32x16_t{};
  auto mma = [&](const Frags<T> &f) {
#pragma unroll
    for (int s = 0; s < SG; ++s)
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[s][i], f.b[s][j], acc[i][j], 0, 0, 0);
  };

  // The look-ahead stage's DMA goes out a step group at a time, kChunk
  // instructions after each group's fragment reads: one burst at the top of
  // the stage backs up the memory queue and stalls the products (measured on
  // the 256 x 256 tile: a 4096-cube product takes 141 us with one burst, 130
  // us over two steps, 125 us over four).
  constexpr int kChunk = T::PerWave / T::Groups;
  const int nst = Kd / T::KC;
#pragma unroll
  for (int st = 0; st < RING - 1; ++st)
    if (st < nst) issue(st, 0, T::PerWave);
  Frags<T> cur, nxt;
  for (int st = 0; st < nst; ++st) {
    // stage st has landed for this wave once at most the later stages' loads
    // are outstanding; the barrier publishes it and retires every read of
    // the slot the look-ahead DMA overwrites
    if (st + RING - 2 < nst && RING > 2) vm_wait<(RING - 2) * T::PerWave>();
    else vm_wait<0>();
    __syncthreads();
    const bool ahead = st + RING - 1 < nst;
    if (computes) {
      load(nxt, st, 0);
      if (ahead) issue(st + RING - 1, 0, kChunk);
      if (st > 0) mma(cur);
#pragma unroll
      for (int g = 1; g < T::Groups; ++g) {
        cur = nxt;
        load(nxt, st, g);
        if (ahead) issue(st + RING - 1, g * kChunk, (g + 1) * kChunk);
        mma(cur);
      }
      cur = nxt;
    } else if (ahead) {
      issue(st + RING - 1, 0, T::PerWave);
    }
  }
  if (computes) mma(cur);

  // Epilogue, in two passes through the ring (free once every wave is past
  // its last fragment read). A lane's accumulators hold one token and
  // scattered groups of four features (token 32 FM wm + 32 j + lane % 32,
  // features 32 FN wn + 32 i + 8 g + 4 (lane / 32) + 0..3 at elements
  // 4 g .. 4 g + 3); stored as they are, every 8-byte piece would land in a
  // different cache line. So the block's tile goes to LDS as bf16 (rows of
  // OP 16-byte pieces, piece index XOR token % OP so that the 32 tokens of a
  // write spread over the banks), then leaves row by row.
  __syncthreads();
  if (computes) {
    uint2 *ot2 = reinterpret_cast<uint2 *>(&ring[0][0]);
#pragma unroll
    for (int j = 0; j < FM; ++j) {
      const int t = 32 * FM * wm + 32 * j + r32;
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int nl = 32 * FN * wn + 32 * i + 8 * g;
          const int n = n0 + nl + 4 * half;
          const float4 bb = n < N ? *reinterpret_cast<const float4 *>(bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
          float y0 = acc[i][j][4 * g + 0] + bb.x, y1 = acc[i][j][4 * g + 1] + bb.y;
          float y2 = acc[i][j][4 * g + 2] + bb.z, y3 = acc[i][j][4 * g + 3] + bb.w;
          if (GELU) {
            y0 = gelu(y0);
            y1 = gelu(y1);
            y2 = gelu(y2);
            y3 = gelu(y3);
          }
          ot2[(t * T::OP + ((nl >> 3) ^ (t & (T::OP - 1)))) * 2 + half] =
              make_uint2(pack_bf16(y0, y1), pack_bf16(y2, y3));
        }
    }
  }
  __syncthreads();
  const uint4 *ot = &ring[0][0];
  const int piece = threadIdx.x % T::OP;
  const int n = n0 + 8 * piece;
  // N is a multiple of 4: a piece is whole, half (8-byte aligned rows when
  // N % 8 == 4) or past the end.
  const bool whole = N % 8 == 0;
  constexpr int kRows = kGThreads / T::OP;   // rows a pass of the block
#pragma unroll 4
  for (int k = 0; k < (T::TM + kRows - 1) / kRows; ++k) {
    const int t = k * kRows + (int)threadIdx.x / T::OP;
    const int64_t m = m0 + t;
    if (t >= T::TM || m >= M || n >= N) continue;
    const uint4 v = ot[t * T::OP + (piece ^ (t & (T::OP - 1)))];
    uint16_t *dst = C + m * N + n;
    if (whole) {
      *reinterpret_cast<uint4 *>(dst) = v;
    } else {
      *reinterpret_cast<uint2 *>(dst) = make_uint2(v.x, v.y);
      if (n + 4 < N) *reinterpret_cast<uint2 *>(dst + 4) = make_uint2(v.z, v.w);
    }
  }
}

// The tiles, smallest first. The small ones stream: their time is the operand
// rows a compute unit pulls through its L1, so they keep deep rings (three
// stages in flight) and long stages (few barriers); a reduction that is no
// multiple of the long stage takes 64-column stages.
template <int KC>
using T32 = Tile<32, 32, 1, 1, KC, 4, KC == 64 ? 4 : 8>;
template <int KC>
using T64x32 = Tile<64, 32, 2, 1, KC, 4, 4>;
template <int KC>
using T64 = Tile<64, 64, 2, 2, KC, 4, 4>;
using T128 = Tile<128, 128, 2, 2, 64, 4, 1>;
using T256x128 = Tile<256, 128, 2, 2, 64, 3, 1>;
using T256 = Tile<256, 256, 2, 2, 64, 2, 1>;

template <class T, bool GELU>
hipError_t launch_tile(const void *A, const void *B, const float *bias, int64_t M, int N, int Kd, void *C,
                       hipStream_t s) {
  const int n_tiles = (N + T::TN - 1) / T::TN;
  const int64_t blocks = (int64_t)n_tiles * ((M + T::TM - 1) / T::TM);
  last::launch_begin(GELU ? "connector_gemm1" : "connector_gemm2", s);
  hipLaunchKernelGGL((k_gemm_nt<T, GELU>), dim3((unsigned)blocks), dim3(kGThreads), 0, s, (const uint16_t *)A,
                     (const uint16_t *)B, bias, M, N, Kd, n_tiles, (int)(blocks / 8), (uint16_t *)C);
  return last::launch_end(s);
}

// The tile of a product. A block holds its compute unit alone (its ring), so
// a product takes ceil(blocks / CUs) rounds of the time one block takes, and
// few rows want small tiles: with 256 x 256 alone, 64 rows of a 4096 x 4096
// product are 16 blocks on 256 units. The weights are the measured times of a
// full round (us for both 4096-wide products of last_connector); a round that
// leaves units idle costs less, down to 0.8 of it. All are proportional to
// the reduction length. Whole call, 4096 -> 4096 -> 4096, before (256 x 256
// only) and with the tile chosen: 64 rows 186 -> 26.7 us (32 x 32; 209 -> 56 on
// operands that no cache holds yet), 96 rows
// 184 -> 33 (64 x 32), 256 rows 198 -> 43 (64 x 64), 1024 rows 200 -> 86 (128
// x 128), 2048 rows 205 -> 145 (256 x 128), 4096 rows 250 (256 x 256 either
// way; 308 with 128 x 128); 1536 wide, 1024 rows 101 -> 40.
enum TileId { kT32, kT64x32, kT64, kT128, kT256x128, kT256, kTiles };
constexpr int kTileN[kTiles] = {T32<64>::TN, T64x32<64>::TN, T64<64>::TN, T128::TN, T256x128::TN, T256::TN};
constexpr int kTileM[kTiles] = {T32<64>::TM, T64x32<64>::TM, T64<64>::TM, T128::TM, T256x128::TM, T256::TM};
constexpr float kTileTime[kTiles] = {22.f, 26.f, 37.f, 80.f, 139.f, 245.f};

TileId pick_tile(int64_t M, int N) {
  const int cus = last::device_cus();
  TileId best = kT256;
  float best_time = INFINITY;
  for (int t = kTiles - 1; t >= 0; --t) {
    const int64_t blocks = (M + kTileM[t] - 1) / kTileM[t] * ((N + kTileN[t] - 1) / kTileN[t]);
    if (blocks > INT32_MAX) break;   // 256 x 256 always fits (connector_shape_ok)
    const float fill = (float)(blocks % cus) / cus;
    const float time = kTileTime[t] * ((float)(blocks / cus) + (fill > 0.f ? 0.8f + 0.2f * fill * fill : 0.f));
    if (time < best_time) {
      best_time = time;
      best = (TileId)t;
    }
  }
  return best;
}

template <bool GELU>
hipError_t launch_gemm(const void *A, const void *B, const float *bias, int64_t M, int N, int Kd, void *C,
                       hipStream_t s) {
  switch (pick_tile(M, N)) {
    case kT32:
      return Kd % 256 == 0 ? launch_tile<T32<256>, GELU>(A, B, bias, M, N, Kd, C, s)
                           : launch_tile<T32<64>, GELU>(A, B, bias, M, N, Kd, C, s);
    case kT64x32:
      return Kd % 128 == 0 ? launch_tile<T64x32<128>, GELU>(A, B, bias, M, N, Kd, C, s)
                           : launch_tile<T64x32<64>, GELU>(A, B, bias, M, N, Kd, C, s);
    case kT64:
      return Kd % 128 == 0 ? launch_tile<T64<128>, GELU>(A, B, bias, M, N, Kd, C, s)
                           : launch_tile<T64<64>, GELU>(A, B, bias, M, N, Kd, C, s);
    case kT128: return launch_tile<T128, GELU>(A, B, bias, M, N, Kd, C, s);
    case kT256x128: return launch_tile<T256x128, GELU>(A, B, bias, M, N, Kd, C, s);
    default: return launch_tile<T256, GELU>(A, B, bias, M, N, Kd, C, s);
  }
}

}  // namespace

namespace last {

bool connector_shape_ok(int64_t K, int32_t Dv, int32_t Dh, int32_t Do) {
  const int64_t blocks = (K + T256::TM - 1) / T256::TM * ((std::max(Dh, Do) + T256::TN - 1) / T256::TN);
  return Dv % kGK == 0 && Dh % kGK == 0 && Do % 4 == 0 && blocks <= INT32_MAX;
}

hipError_t launch_connector(int64_t K, int32_t Dv, int32_t Dh, int32_t Do, float eps, const void *x,
                            const float *gamma, const float *beta, const void *w1, const float *b1,
                            const void *w2, const float *b2, void *out, void *xn, void *hid,
                            hipStream_t s) {
  if (K == 0) return hipSuccess;
  launch_begin("connector_layernorm", s);
  const dim3 grid((unsigned)((K + kLnWaves - 1) / kLnWaves)), block(64 * kLnWaves);
  const int per_lane = (Dv / 8 + 63) / 64;
  if (per_lane <= 4)
    hipLaunchKernelGGL(k_layernorm<4>, grid, block, 0, s, (const uint16_t *)x, gamma, beta, K, Dv, eps,
                       (uint16_t *)xn);
  else if (per_lane <= 8)
    hipLaunchKernelGGL(k_layernorm<8>, grid, block, 0, s, (const uint16_t *)x, gamma, beta, K, Dv, eps,
                       (uint16_t *)xn);
  else
    hipLaunchKernelGGL(k_layernorm<0>, grid, block, 0, s, (const uint16_t *)x, gamma, beta, K, Dv, eps,
                       (uint16_t *)xn);
  hipError_t e = launch_end(s);
  if (e != hipSuccess) return e;
  e = launch_gemm<true>(w1, xn, b1, K, Dh, Dv, hid, s);
  if (e != hipSuccess) return e;
  return launch_gemm<false>(w2, hid, b2, K, Do, Dh, out, s);
}

}  // namespace last
