// Causal prefill attention of the guidance model with the LAST statistics
// of each request's last row as a by-product (arXiv 2607.27952, Sec. 3.3:
// the relevance is read from the attention of the same prefill pass), for
// gfx950, bf16 inputs:
//
//   out_p = sum_{j <= p} softmax_j(sigma q_p . k_j) v_j      for every position p
//
// and, for the last position p* = P_r - 1, the scaled logits of the visual
// keys and the row's (max, sum exp, visual sum exp), in the layout the
// last-token score pass uses, so that its merge and finalize kernels turn
// them into w~ (Eq. 7-8) without another pass over the keys.
//
// One block per (layer, request, query head, 128 query positions); each of
// its four waves owns 32 positions. Keys and values go through LDS 64 at a
// time, both row-major with XOR-swizzled 16-byte pieces, copied straight from
// memory by LDS DMA (global_load_lds_dwordx4: no registers, no transposing
// stores) one stage ahead of their use. The value fragments are read with the
// LDS transpose load (ds_read_b64_tr_b16): in each group of 16 lanes, lane i's
// element j comes from element i % 4 of the 8 bytes lane 4 j + i / 4 points
// at, so lanes pointing at 4 keys x 4 four-dimension chunks receive 4 keys of
// one dimension each.
//
// The product runs transposed so that every lane owns one query:
//   S^T = K Q^T   (v_mfma_f32_32x32x16_bf16, A = 32 keys, B = the wave's 32
//                  queries, kept in registers): lane l holds query l % 32 and
//                  16 of the 32 keys of a tile, the other 16 being in lane
//                  l ^ 32. The tile's keys are loaded into the MFMA rows in a
//                  permuted order, so that lane half h holds keys
//                  8h .. 8h + 7 and 16 + 8h .. 16 + 8h + 7 of the tile.
//   O^T = V^T P^T (A = 32 value dimensions x 16 keys from the transposed
//                  LDS stage, B = 8 probabilities of the lane, packed to bf16):
//                  the permutation above makes each lane's probabilities
//                  exactly the keys its half of the B operand needs.
// The softmax runs online per lane in base-2 units (the scale times log2 e
// folded into the exponent's fma): a stage of 64 keys at a time, its maximum
// first, so that every probability is at most 1, a row's largest exactly 1,
// and the sums stay as finite as the values; what was summed is rescaled only
// when some lane's maximum has moved.
//
// What bounds it: long sequences, the matrix and vector units sharing the
// issue (matrix cores busy 53% of the cycles, at 1.93 GHz of 2.4 nominal, on 8 x
// 16512 tokens); short ones, latency (busy 26% on 64 x 640). The
// loop is pipelined by stages: the matrix cores form the next stage's logits
// and then this stage's products with the values while the vector ALU forms
// this stage's probabilities, and the next stage's maximum is taken under the
// last products. 8 x 16512 tokens, 28/4 heads, one layer: 23.1 ms with the
// same arithmetic one phase after the other, 15.3 now (1.02 PFLOP/s, where
// torch's 8192^3 product reaches 1.22). 64 x 640 tokens, 32 heads, 2 layers:
// 1.27 -> 0.88 ms. A reference that moves only past 2^16 instead of the
// maximum took 2% less, but rounds a row's largest probability and lets
// values past 2^90 overflow. With the products one stage behind, the
// registers spill (20.3 and 1.45 ms).
#include <algorithm>
#include <math.h>
#include <type_traits>

#include "last_internal.h"

using namespace last_dev;

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kKS = 64;                       // keys per LDS stage: two units of 32
constexpr float kLog2e = 1.4426950408889634f;

constexpr int kNW = 4;                        // waves a block, of 32 query positions each
constexpr int kThreads = 64 * kNW, kQB = 32 * kNW;
constexpr int kRing = 2;                      // stages of keys, and of values, in LDS

template <int DH>
struct Shape {
  static constexpr int kPieces = DH * 2 / 16;            // 16-byte pieces per key row
  static constexpr int kSteps = kPieces / 2;             // S^T MFMA steps per key tile
  static constexpr int kDT = DH / 32;                    // value-dimension tiles of O^T
  static constexpr int kDma = kKS * kPieces / 64 / kNW;  // DMA instructions per operand stage and wave
  static_assert(kKS * kPieces % (64 * kNW) == 0, "stage split");
  static_assert(kSteps == 2 * kDT, "chunk split");
};

// Physical 16-byte piece of logical piece p in row j of a stage (keys and
// values alike): an XOR that gives the 16 rows a key fragment reads at one
// piece 16 different bank groups, and the 4 rows a transpose read takes 64
// bytes of four different quarters of the banks. (The plain p ^ (j % 16) put
// those four rows' 64 bytes on the same banks: a third of the time of the
// long prefill went into the conflicts.)
template <int NP>
__device__ __forceinline__ int pswz(int j, int p) {
  return p ^ (NP >= 16 ? ((j & 3) << 2) | ((j >> 2) & 3) : ((j & 2) << 1) | ((j >> 2) & 3));
}

typedef short s16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ s16x4_t read_tr(const uint16_t *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)p);
}

// Key of a 32-key tile that MFMA row i carries: lane half h, element v of the
// accumulator (row 4h + v % 4 + 8 (v / 4)) then holds key 8h + v (v < 8) or
// 16 + 8h + v - 8 (v >= 8).
__device__ __forceinline__ int perm_key(int i) {
  const int h = (i >> 2) & 1, v = (i & 3) + 4 * (i >> 3);
  return 8 * h + v + (v >= 8 ? 8 : 0);
}
__device__ __forceinline__ int acc_key(int half, int v) { return 8 * half + v + (v >= 8 ? 8 : 0); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
// two floats to bf16, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const f32x2_t x = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
}

// max over the two halves of the wave (lanes l and l ^ 32), in both
__device__ __forceinline__ float half_max(float v) {
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float v) {
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The request's last row against its visual keys (the first of them at kp):
// its logits again (the same products, bit for bit, with that row in every
// column and the keys straight from memory, mostly from L2), written in the
// score pass's base-2 units, and the sum of their terms against the row's
// maximum mr, of this wave's share. One tile's keys are in flight; with four, the
// attention loop above it lost its registers to them (64 x 640 tokens: 1003
// -> 1114 us, and 1070 as a call of its own); inside the loop, beside the row's
// own stages, it costs every wave registers too (893 -> 1009 us).
template <int DH>
__device__ __forceinline__ float last_row(const uint16_t *qrow, const uint16_t *kp, int64_t kvstride, int nvis,
                                          float s2, float mr, float *vl, int Hq) {
  constexpr int kSteps = Shape<DH>::kSteps;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int tiles = (nvis + 31) / 32;
  bf16x8_t bq[kSteps], kf[kSteps];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) bq[s] = *reinterpret_cast<const bf16x8_t *>(qrow + (2 * s + half) * 8);
  auto load_k = [&](int tile) {
    const uint16_t *row = kp + min(32 * tile + perm_key(col), nvis - 1) * kvstride;
#pragma unroll
    for (int s = 0; s < kSteps; ++s) kf[s] = *reinterpret_cast<const bf16x8_t *>(row + (2 * s + half) * 8);
  };
  float vsum = 0.f;
  if (wave < tiles) load_k(wave);
  for (int tile = wave; tile < tiles; tile += kNW) {
    f32x16_t sc = f32x16_t{};
#pragma unroll
    for (int s = 0; s < kSteps; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], bq[s], sc, 0, 0, 0);
    if (tile + kNW < tiles) load_k(tile + kNW);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int i = 32 * tile + acc_key(half, e);
      const float x2 = sc[e] * s2;
      if (i < nvis) {
        vsum += __builtin_amdgcn_exp2f(x2 - mr);
        if (col == e) vl[(int64_t)i * Hq] = x2;   // every column holds the row: one of them writes
      }
    }
  }
  return half_sum(vsum);
}

// One (layer, request, head, block of query positions) per block.
template <int DH>
__global__ __launch_bounds__(kThreads, 2) void k_prefill(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
    const int32_t *__restrict__ cu_seqlens, const int32_t *__restrict__ vis_start,
    const int32_t *__restrict__ cu_vis, const int32_t *__restrict__ qb_off,
    const int32_t *__restrict__ qb_req, int R, int Hq, int Hkv, int64_t QB_total,
    int64_t T_total, int64_t N_total, float scale, uint16_t *__restrict__ out,
    float *__restrict__ vlog, float4 *__restrict__ stats) {
  using SH = Shape<DH>;
  constexpr int NP = SH::kPieces;
  __shared__ uint4 s_kv[2][kRing][kKS * NP];
  static_assert(kNW * 32 <= 2 * kRing * kKS, "the output rows are staged in the ring");
  auto &s_k = s_kv[0], &s_v = s_kv[1];

  // Order: layer, request, head, query block (the longest, last, block of a
  // request first). XCD-contiguous numbering runs neighbours together on one
  // XCD: the query blocks of one head re-read its keys and values from that
  // L2, and the heads running beside each other cover whole token rows (Hq Dh
  // elements apart). With every request's blocks of one head before the next
  // head, all running blocks read the same few 256-byte slots of the rows,
  // and so the same memory channels: 64 x 640 tokens, 32 heads 1137 us.
  const int64_t bid = xcd_contiguous(blockIdx.x, gridDim.x), per_layer = (int64_t)Hq * QB_total;
  const int l = (int)(bid / per_layer);
  const int64_t in_layer = bid % per_layer;
  const int r = qb_req[in_layer / Hq];
  const int in_req = (int)(in_layer - (int64_t)Hq * qb_off[r]), nqb = qb_off[r + 1] - qb_off[r];
  const int h = in_req / nqb, qb = nqb - 1 - in_req % nqb;
  const int g = Hq / Hkv, kv = h / g;
  const int64_t tok0 = cu_seqlens[r];
  const int P = cu_seqlens[r + 1] - (int)tok0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int q0 = qb * kQB + wave * 32;       // the wave's first query position
  const int qpos = q0 + col;                     // this lane's query
  const int kend = min(P, qb * kQB + kQB);   // keys the block needs: 0 .. kend - 1
  const int nst = (kend + kKS - 1) / kKS;            // stages of the block, and of the wave
  const int wst = q0 < P ? (min(P, q0 + 32) - 1) / kKS + 1 : 0;
  const float s2 = scale * kLog2e;

  // B operand of S^T: the lane's query row, pieces 2 st + half
  bf16x8_t bq[SH::kSteps];
  auto load_q = [&](int pos) {
    const char *qp = reinterpret_cast<const char *>(q + (((int64_t)l * T_total + tok0 + pos) * Hq + h) * DH);
#pragma unroll
    for (int st = 0; st < SH::kSteps; ++st)
      bq[st] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(qp + (2 * st + half) * 16));
  };
  load_q(min(qpos, P - 1));

  const int64_t kvstride = (int64_t)Hkv * DH;    // elements between consecutive tokens
  const uint16_t *kbase = k + ((int64_t)l * T_total + tok0) * kvstride + (int64_t)kv * DH;
  const uint16_t *vbase = v + ((int64_t)l * T_total + tok0) * kvstride + (int64_t)kv * DH;

  // One operand stage: rows 64 st .. 64 st + 63 (clamped to the block's last
  // needed key). DMA instruction x of this wave covers 16-byte slots 64 i +
  // lane, i = wave + kNW x, of the stage: row (slot / NP), physical piece
  // (slot % NP), which holds logical piece pswz(row, physical) (an XOR, its
  // own inverse). The rows of x are 64 kNW / NP x below those of x = 0 and the
  // piece is the same, so a lane's offset is one register and only the base
  // moves, but in a last stage that reaches past the keys.
  constexpr int kRows = 64 * kNW / NP;
  static_assert(kRows % 16 == 0, "the swizzle repeats every 16 rows");
  const int drow = (wave * 64 + lane) / NP, dpiece = pswz<NP>(drow, lane % NP) * 16;
  const uint32_t rowb = (uint32_t)(kvstride * 2), voff0 = drow * rowb + dpiece;
  auto issue = [&](const uint16_t *base, uint4 *to, int st) {
    const char *from = reinterpret_cast<const char *>(base) + (int64_t)st * kKS * rowb;
    if ((st + 1) * kKS <= kend) {
#pragma unroll
      for (int x = 0; x < SH::kDma; ++x)
        dma16(__builtin_amdgcn_readfirstlane(lds_u32(to + (wave + kNW * x) * 64)),
              uniform_ptr(from + (int64_t)(kRows * x) * rowb), voff0);
    } else {
#pragma unroll
      for (int x = 0; x < SH::kDma; ++x)
        dma16(__builtin_amdgcn_readfirstlane(lds_u32(to + (wave + kNW * x) * 64)), uniform_ptr(from),
              (uint32_t)min(kRows * x + drow, kend - 1 - st * kKS) * rowb + dpiece);
    }
  };
  // group g: the keys and values that stage g of the loop below reads
  auto issue_group = [&](int g) {
    if (g + 1 < nst) issue(kbase, s_k[(g + 1) % kRing], g + 1);
    if (g < nst) issue(vbase, s_v[g % kRing], g);
  };

  // Fragment offsets in an operand stage (elements). Keys: row 32 t +
  // perm_key(col), piece 2 s + half; the swizzle does not depend on t.
  // Values (A = V^T): lane l needs dimension 32 dt + l % 32 of keys 16 s + 8
  // half .. + 7, as two transpose reads of 4 keys; lane i of its 16-lane group
  // points at key i / 4 of the four and dimensions 4 (i % 4) .. + 3 of the
  // group's 16; the swizzle does not depend on s.
  int koff[SH::kSteps], voffs[SH::kDT][2];
  {
    const int krow = perm_key(col);
#pragma unroll
    for (int s = 0; s < SH::kSteps; ++s) koff[s] = (krow * NP + pswz<NP>(krow, 2 * s + half)) * 8;
    const int gr = lane >> 4, pl = lane & 15;
#pragma unroll
    for (int dt = 0; dt < SH::kDT; ++dt)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int key = 8 * (gr >> 1) + 4 * c + (pl >> 2), d = dt * 32 + 16 * (gr & 1) + 4 * (pl & 3);
        voffs[dt][c] = key * DH + pswz<NP>(key, d >> 3) * 8 + (d & 7);
      }
  }
  auto kfrag = [&](const uint16_t *ks, int t, int s) {   // key tile t of the stage, step s
    return *reinterpret_cast<const bf16x8_t *>(ks + koff[s] + t * 32 * DH);
  };
  auto vfrag = [&](const uint16_t *vs, int s, int dt) {  // 16-key step s of the stage
    typedef short s16x8_t __attribute__((ext_vector_type(8)));
    const s16x4_t a0 = read_tr(vs + voffs[dt][0] + s * 16 * DH), a1 = read_tr(vs + voffs[dt][1] + s * 16 * DH);
    const s16x8_t av = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
    return __builtin_bit_cast(bf16x8_t, av);
  };

  // Per lane (= per query), in both halves alike: the running maximum m of the
  // stages so far (base-2 units) and the sum of the terms against it.
  float m = -INFINITY, lsum = 0.f;
  f32x16_t o[SH::kDT];
#pragma unroll
  for (int dt = 0; dt < SH::kDT; ++dt) o[dt] = f32x16_t{};

  // The maximum with stage j (logits in x, whose keys a query does not see
  // become -inf), what its exponents subtract, the factor of the sums so far,
  // and whether any query's maximum moved. (s2 > 0, so the largest dot gives
  // the largest logit. A query with no key seen yet keeps -inf; its terms and
  // sums are 0.)
  float mref = 0.f, alpha = 1.f;
  bool moved = false;
  auto maximum = [&](f32x16_t (&x)[2], int j) {
    if (kKS * j + kKS - 1 > q0) {   // causal mask, and past the block's end
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = kKS * j + 32 * t + acc_key(half, e);
          x[t][e] = (key <= qpos && key < kend) ? x[t][e] : -INFINITY;
        }
    }
    float mx = x[0][0];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, x[t][e]);
    const float mnew = fmaxf(m, half_max(mx) * s2);
    mref = mnew == -INFINITY ? 0.f : mnew;
    alpha = __builtin_amdgcn_exp2f(m - mref);
    moved = __any(mnew != m);
    m = mnew;
  };

  issue(kbase, s_k[0], 0);
  issue_group(0);
  if (nst > 1)
    vm_wait<2 * SH::kDma>();
  else
    vm_wait<0>();
  __syncthreads();
  f32x16_t sc[2][2];   // logits of a stage's two 32-key tiles, by stage parity
  if (wst > 0) {
    const uint16_t *ks = reinterpret_cast<const uint16_t *>(s_k[0]);
    sc[0][0] = sc[0][1] = f32x16_t{};
#pragma unroll
    for (int s = 0; s < SH::kSteps; ++s)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        sc[0][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag(ks, t, s), bq[s], sc[0][t], 0, 0, 0);
    maximum(sc[0], 0);
  }
  // Stage j (slot S = j % 2) in chunks of one MFMA: the logits of stage j + 1
  // (if LOGITS), then the stage's probabilities times the values, 16 keys at a
  // time; the probabilities are formed beside both, a pair every 1.6 chunks at
  // DH = 128, so that each group of 16 keys is there before its products. A
  // chunk's fragment is read from LDS two chunks ahead.
  auto body = [&](auto logits, auto parity, int j, int vslot) {
    constexpr bool LOGITS = decltype(logits)::value;
    constexpr int S = decltype(parity)::value, kHalf = 2 * SH::kSteps, kChunks = 2 * kHalf;
    constexpr int kDone = 15 * kChunks / 20;   // the chunk with the last probabilities
    const uint16_t *ks = reinterpret_cast<const uint16_t *>(s_kv[0][1 - S]);
    const uint16_t *vs = reinterpret_cast<const uint16_t *>(s_kv[1][vslot]);
    f32x16_t(&cur)[2] = sc[S], (&next)[2] = sc[1 - S];
    uint32_t pb[16];
    bf16x8_t fr[3];
    auto read = [&](int c) {
      if (c < kHalf) {
        if (LOGITS) fr[c % 3] = kfrag(ks, c / SH::kSteps, c % SH::kSteps);
      } else {
        fr[c % 3] = vfrag(vs, (c - kHalf) / SH::kDT, (c - kHalf) % SH::kDT);
      }
    };
    float ps = 0.f;
    read(0);
    read(1);
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      if (c + 2 < kChunks) read(c + 2);
      // the maximum moves rarely after the first stages: rescale only then
      if (c == kHalf && moved) {
#pragma unroll
        for (int dt = 0; dt < SH::kDT; ++dt) o[dt] *= alpha;
      }
      if (c >= kHalf) {
        const int s = (c - kHalf) / SH::kDT;
        f32x16_t &od = o[(c - kHalf) % SH::kDT];
        od = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            fr[c % 3],
            __builtin_bit_cast(bf16x8_t, make_uint4(pb[4 * s], pb[4 * s + 1], pb[4 * s + 2], pb[4 * s + 3])), od, 0, 0, 0);
      } else if (LOGITS) {
        f32x16_t &n = next[c / SH::kSteps];
        n = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[c % 3], bq[c % SH::kSteps],
                                                    c % SH::kSteps == 0 ? f32x16_t{} : n, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i * kChunks / 20 != c) continue;
        const f32x16_t &x = cur[i / 8];
        const int e = 2 * (i % 8);
        // the raw dots stay in place and the scale goes into the exponent
        const float p0 = __builtin_amdgcn_exp2f(fmaf(x[e], s2, -mref));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(x[e + 1], s2, -mref));
        ps += p0 + p1;
        pb[i] = pack_bf16(p0, p1);
      }
      // (after that chunk the maximum's steps go among the remaining products)
      if (c == kDone) {
        lsum = fmaf(lsum, alpha, half_sum(ps));
        if (LOGITS) maximum(next, j + 1);
      }
      if (c < kDone) __builtin_amdgcn_sched_barrier(0);
    }
    static_assert(kDone < kHalf + 3 * SH::kDT && 11 * kChunks / 20 < kHalf + 2 * SH::kDT &&
                      7 * kChunks / 20 < kHalf + SH::kDT && 3 * kChunks / 20 < kHalf,
                  "probabilities before their products");
  };
  // Every wave of the block passes turn(0) .. turn(nst - 1). At turn(j) the
  // keys of stage j + 1 and the values of stage j have landed for this wave;
  // the barrier publishes them and retires every read of the slots that the
  // next group overwrites.
  auto turn = [&](int j) {
    vm_wait<0>();
    __syncthreads();
    issue_group(j + 1);
  };
  // Stages in pairs, so that the ring slots, and with them every fragment's
  // address but the lane's part, are constants.
  static_assert(kRing == 2, "slot parity");
  constexpr std::true_type more{};
  constexpr std::false_type final{};
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  int j = 0;
  if (wst > 0) {
    for (; j + 2 < wst; j += 2) {
      turn(j);
      body(more, even, j, 0);
      turn(j + 1);
      body(more, odd, j + 1, 1);
    }
    if (j + 1 < wst) {
      turn(j);
      body(more, even, j++, 0);
      sc[0][0] = sc[1][0];
      sc[0][1] = sc[1][1];
    }
    turn(j);
    body(final, even, j, j % kRing);   // the logits are in sc[0] either way
    ++j;
  }
  for (; j < nst; ++j) turn(j);

  // out_p = O^T column / sum; lane half h holds dimensions 4 h + e % 4 + 8 (e /
  // 4) of its query. The wave's 32 rows go through LDS (free once every wave
  // is past its last read; rows of NP 16-byte pieces, swizzled like a stage)
  // and leave as whole rows.
  __syncthreads();
  if (wst > 0) {
    uint4 *rows = &s_kv[0][0][0] + wave * 32 * NP;
    const float inv = 1.0f / lsum;
#pragma unroll
    for (int dt = 0; dt < SH::kDT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; e += 4) {
        const int d = dt * 32 + 4 * half + 8 * (e / 4);
        uint2 w;
        w.x = pack_bf16(o[dt][e] * inv, o[dt][e + 1] * inv);
        w.y = pack_bf16(o[dt][e + 2] * inv, o[dt][e + 3] * inv);
        reinterpret_cast<uint2 *>(rows + col * NP + pswz<NP>(col, d >> 3))[half] = w;
      }
    // (the wave's own rows: its LDS operations complete in order; the fence
    // keeps the compiler from moving the loads, of other lanes' pieces, above
    // the stores)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint16_t *ob = out + (((int64_t)l * T_total + tok0 + q0) * Hq + h) * DH;
#pragma unroll 4
    for (int x = 0; x < NP / 2; ++x) {
      const int slot = x * 64 + lane, row = slot / NP, pp = slot % NP;
      const uint4 w = rows[row * NP + pswz<NP>(row, pp)];
      if (q0 + row < P) *reinterpret_cast<uint4 *>(ob + (int64_t)row * Hq * DH + pp * 8) = w;
    }
  }

  // The LAST extraction, by the block that holds the request's last row.
  if (kend != P) return;
  __shared__ float s_last[2], s_vsum[kNW];
  if (q0 <= P - 1 && P - 1 < q0 + 32 && qpos == P - 1 && half == 0) {
    s_last[0] = m;
    s_last[1] = lsum;
  }
  __syncthreads();
  const float mlast = s_last[0];
  const float vsum =
      last_row<DH>(q + (((int64_t)l * T_total + tok0 + P - 1) * Hq + h) * DH, kbase + vis_start[r] * kvstride, kvstride,
                   cu_vis[r + 1] - cu_vis[r], s2, mlast == -INFINITY ? 0.f : mlast,
                   vlog + ((int64_t)l * N_total + cu_vis[r]) * Hq + h, Hq);
  if (lane == 0) s_vsum[wave] = vsum;
  __syncthreads();
  if (threadIdx.x == 0) {
    float vs = 0.f;
#pragma unroll
    for (int w = 0; w < kNW; ++w) vs += s_vsum[w];
    stats[((int64_t)l * Hq + h) * R + r] = make_float4(mlast, s_last[1], vs, 0.f);
  }
}

// Per request: the number of 128-position query blocks, their prefix and the
// block -> request map.
__global__ __launch_bounds__(256) void k_prefill_plan(const int32_t *__restrict__ cu_seqlens, int R,
                                                      int64_t cap, int32_t *__restrict__ qb_off,
                                                      int32_t *__restrict__ qb_req) {
  __shared__ int sh[4];
  int carry = 0;
  for (int base = 0; base < R; base += 256) {
    const int r = base + (int)threadIdx.x;
    int n = 0;
    if (r < R) n = (cu_seqlens[r + 1] - cu_seqlens[r] + kQB - 1) / kQB;
    int tot;
    const int pre = block_exclusive_scan(n, sh, &tot) + carry;
    if (r < R) {
      qb_off[r] = pre;
      for (int i = 0; i < n; ++i)
        if (pre + i < cap) qb_req[pre + i] = r;
    }
    carry += tot;
  }
  if (threadIdx.x == 0) qb_off[R] = carry;
}

template <int DH>
hipError_t launch_dh(const last_batch *b, int64_t QB_total, const int32_t *qb_off, const int32_t *qb_req,
                        const void *q, const void *k, const void *v, void *out, float *vlog, float4 *stats,
                        float scale, hipStream_t s) {
  const int64_t blocks = (int64_t)b->G * b->Hq * QB_total;
  const int64_t T_total = b->cu_seqlens_h[b->R], N_total = b->cu_vis_h[b->R];
  last::launch_begin("prefill", s);
  hipLaunchKernelGGL(k_prefill<DH>, dim3((unsigned)blocks), dim3(kThreads), 0, s, (const uint16_t *)q,
                     (const uint16_t *)k, (const uint16_t *)v, b->cu_seqlens, b->vis_start, b->cu_vis, qb_off,
                     qb_req, b->R, b->Hq, b->Hkv, QB_total, T_total, N_total, scale, (uint16_t *)out, vlog, stats);
  return last::launch_end(s);
}

}  // namespace

namespace last {

int64_t prefill_query_blocks(const last_batch *b) {
  int64_t n = 0;
  for (int r = 0; r < b->R; ++r) n += (b->cu_seqlens_h[r + 1] - b->cu_seqlens_h[r] + kQB - 1) / kQB;
  return n;
}

hipError_t launch_prefill(const last_batch *b, int64_t QB_total, int32_t *qb_off, int32_t *qb_req,
                          const void *q, const void *k, const void *v, void *out, float *vlog,
                          float4 *stats, float scale, hipStream_t s) {
  launch_begin("prefill_plan", s);
  hipLaunchKernelGGL(k_prefill_plan, dim3(1), dim3(256), 0, s, b->cu_seqlens, b->R, QB_total, qb_off, qb_req);
  hipError_t e = launch_end(s);
  if (e != hipSuccess) return e;
  return b->Dh == 64 ? launch_dh<64>(b, QB_total, qb_off, qb_req, q, k, v, out, vlog, stats, scale, s)
                     : launch_dh<128>(b, QB_total, qb_off, qb_req, q, k, v, out, vlog, stats, scale, s);
}

}  // namespace last
