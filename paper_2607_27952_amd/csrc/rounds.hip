// The exact greedy k-center of LAST (arXiv 2607.27952, Sec. 3.4, Eq. 9-11)
// without the N x N coverage matrix, for gfx950.
//
// Step t of the greedy needs the coverage distance of every token to the
// newest pick (Eq. 10). gram.hip forms all N_r^2 distances up front; this file
// forms, as the paper's own incremental form does, only the distances to the
// tokens actually picked (about K_r N_r of them), yet keeps the matrix cores
// busy by taking the picks in rounds:
//
//   - at the start of a round every token's running minimum distance
//     delta_i is exact (every pick so far folded in), hence so is every
//     objective o_i = w_i delta_i and its key (o_i bits, lowest index first);
//   - the round's candidates are the kRB tokens with the largest keys, and T
//     is the largest key left outside them. delta only decreases, so every
//     outside key stays <= T for the rest of the round;
//   - the greedy then runs on the candidates alone, with their mutual
//     distances (a kRB x kRB Gram on the matrix cores): while its best key is
//     above T, that token is the best of the whole request, i.e. exactly the
//     pick the full greedy makes; the round ends at the first key that is
//     not, or after kRP picks;
//   - the round's picks are folded into every token's delta in one pass over
//     the request's features: a kRP-column product on the matrix cores.
// Each round makes at least one pick (the request's best key is a candidate).
// A round whose best objective is 0 (or not a number for every token) ends
// the greedy the way Eq. 9-11 with lowest-index ties do: the rest of the
// budget goes to the lowest-index tokens not yet picked.
//
// Every distance is the number gram.hip stores for the same ordered pair:
// dot products on v_mfma_f32_32x32x16_bf16 in 128-column chunks of fp32
// partial sums, folded into fp64 in column order; the squared norms from
// the same arithmetic; and 1 - dot / (|x_a| |x_b|) multiplied in the order
// gram.hip uses for that pair (its row block's token first). So this form and
// the matrix form pick the same tokens, bit for bit.
//
// Kernels:
//   k_rnorm    |x_i|^2 and 1 / |x_i| of every token (one pass over X).
//   k_reven    (where the form is chosen on the device) whether a request's
//              relevance is too even for the rounds.
//   k_rprep    fold-tile prefixes, the per-request state and that choice.
//   k_rounds   the rounds, as a queue of tasks on a persistent grid; per
//              request and round: S (select the candidates), G (the
//              candidates' distances and the greedy on them), F (fold the
//              picks into 256 tokens each), listed round by round and, within
//              a round, phase by phase. A block takes the next task index from
//              a global counter and waits until the tasks it depends on (all
//              with smaller indices, so already taken by running blocks) have
//              completed: no block ever waits for a block that has not started,
//              so the grid needs no co-residency. Every wait is bounded by a
//              wall-clock limit.
//   k_rfail    after a timeout, marks the unfinished requests invalid.
//
// What bounds it: the folds, which read X once a round, and the chain of one
// request's rounds, on relevance with peaks. Video batch, 8 x 16384 tokens of
// 3584: 10.6 rounds of up to 128 picks, each a chain of S 23 us, G 89 and F 89;
// its 5440 folds on 256 units are 1.9 of the 2.5 ms; 10.1 GB fetched (4.0 TB/s
// over the kernel), matrix cores busy 20%. 128 ragged requests of 256 to 16384
// tokens of 1536: 15.3 GB in 4.7 ms, some 19400 folds of 42 us (3.2 ms over the
// units), the longest request's chain about 2.9 ms, busy 15%. 32 x 2880 tokens
// of 4096: 3.6 GB in 1.05 ms, busy 13%. Rounds of 64 picks took 3.53, 10.9 and
// 1.52 ms.
#include <algorithm>
#include <cstdlib>
#include <math.h>

#include "last_internal.h"

using namespace last_dev;

namespace last {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kRThreads = 512;
constexpr int kRWaves = kRThreads / 64;
constexpr int kRB = kRoundCands;              // candidates a round at most
constexpr int kRSub = kRB / 32;               // 32-slot blocks of the candidate list
constexpr int kRP = kRoundPicks;              // picks a round at most
constexpr int kFRows = kRoundFoldRows;        // tokens a fold task
constexpr int kFRing = 3;                     // fold ring stages (two in flight)
constexpr int kFCols = 64;                    // columns a ring stage
constexpr int kFTokPieces = kFRows * kFCols * 2 / 16;   // 16-byte pieces of tokens a stage
constexpr int kFPickPieces = kRP * kFCols * 2 / 16;     // ... of picks
constexpr int kFStagePieces = kFTokPieces + kFPickPieces;
constexpr int kFTokInstr = kFTokPieces / 64 / kRWaves;  // LDS-DMA instructions a wave, tokens
constexpr int kFTiles = kRP / 32;                       // 32-pick tiles of a fold task
constexpr int kFPickInstr = kFPickPieces / 64 / kRWaves;   // ... picks, of a fold with every tile
static_assert(kFTiles % 2 == 0 && kFPickInstr == kFTiles / 2, "a pick DMA instruction a wave per two tiles");
constexpr int kGRing = 6;                      // candidate-Gram ring stages (five in flight)
constexpr int kGStagePieces = kRB * kFCols * 2 / 16;    // 16-byte pieces of candidates a stage
constexpr int kGPerWave = kGStagePieces / 64 / kRWaves;  // LDS-DMA instructions a wave
static_assert(kGPerWave * 64 * kRWaves == kGStagePieces, "even DMA split");
constexpr int kGStride = kRB + 1;              // floats of a row of the candidate matrix (odd: its mirror
                                               // writes, one column a lane group, spread over the banks)
constexpr int kSelLds = kRoundMaxN;           // keys of a request held in LDS by the select
constexpr int kFtLds = 2048;                  // fold-tile prefixes held in LDS (batches of fewer requests)
static_assert(kRB % 64 == 0 && kRB <= 256, "candidate slots: whole waves");
static_assert(kFRows == 32 * kRWaves, "a fold task: 32 tokens a wave");

// Every word one task hands to a task of another block (delta, candidates,
// their distances, picks, state) is written with a device-scope (agent)
// atomic store and read with a device-scope atomic load (the sc1 forms),
// which go to the device's coherence point past the XCDs' separate L2
// caches: a device-scope store is acknowledged there, so once every wave has
// waited for its stores (s_waitcnt) and the block has met at its barrier,
// raising the completion count cannot overtake them. No task writes such a
// word with a plain store, which would need the L2 written back (a release
// fence) before the count; that fence on every task costs 10% of a video
// batch's selection.
__device__ __forceinline__ int ld_i32(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_i32(int32_t *p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_u32(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_u32(uint32_t *p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_u64(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_u64(unsigned long long *p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_f32(const float *p) {
  return __uint_as_float(ld_u32(reinterpret_cast<const uint32_t *>(p)));
}
__device__ __forceinline__ void st_f32(float *p, float v) {
  st_u32(reinterpret_cast<uint32_t *>(p), __float_as_uint(v));
}

__device__ __forceinline__ float clean_score(float w) { return w > 0.f ? w : 0.f; }   // NaN -> 0

// Values that steer branches or loops around barriers are made wave-uniform
// as the compiler sees them (read from the first active lane): a branch on a
// value it takes as per-lane is lowered with exec masks, and around a loop
// with barriers the compiler may then give lanes loop nests of their own,
// in which a block repeats barriers without the lane that fetches its next
// task ever running. All lanes hold the same value wherever these are used.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uniu(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ unsigned long long uni64(unsigned long long v) {
  return ((unsigned long long)uniu((uint32_t)(v >> 32)) << 32) | uniu((uint32_t)v);
}
__device__ __forceinline__ int64_t uni_i64(int64_t v) { return (int64_t)uni64((unsigned long long)v); }

// Eq. 10 term for the ordered pair (row token, column token) as gram.hip
// stores it: 1 - cos clamped at 0, zero-norm rows at distance 1, bitwise
// duplicates at 0; dot * inv_a * inv_b multiplied with a = the token of the
// lower 32-row block (the row token within one block), which is the order in
// which the Gram tile that owns the pair evaluates it. The pick's own entry is
// -inf (its selection mark).
__device__ __forceinline__ float coverage_ab(double dot, double nna, double nnb, double inva, double invb) {
  const double t = 1.0 - dot * inva * invb;
  float c = t > 0.0 ? (float)t : 0.0f;
  c = (dot == nna && nna == nnb) ? 0.0f : c;
  c = (nna <= 0.0 || nnb <= 0.0) ? 1.0f : c;
  return c;
}
__device__ __forceinline__ float coverage_dir(int x, int y, double dot, double nnx, double nny, double invx,
                                              double invy) {
  // selects only: a branch per distance costs more than the distance
  const bool fwd = (x >> 5) <= (y >> 5);
  const float c = coverage_ab(dot, nnx, nny, fwd ? invx : invy, fwd ? invy : invx);
  return x == y ? -INFINITY : c;
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

struct RArgs {
  const float *scores;
  const uint16_t *X;
  const double *nn, *inv;
  const int32_t *cu_vis, *cu_keep;
  int32_t *kept, *order;
  float *gains;
  float *dl;                       // [N_total] running minimum distance (+inf before the first pick, -inf once picked)
  int32_t *cand;                   // [R][kRB] this round's candidates (request-local token indices)
  int32_t *picks;                  // [R][kRP] this round's picks
  int32_t *st;                     // [R][4] picks so far, picks this round, candidates, finished
  unsigned long long *st_T;        // [R] the bound key T
  uint32_t *dcnt;                  // [R] completed tasks
  const int64_t *ftoff;            // [R + 1] fold-tile prefixes
  const unsigned long long *ctl;   // live (low word) and abort (high word), read together
  const uint32_t *form;            // null, or the form chosen on the device
  unsigned long long *head;        // next task index
  uint32_t *live;                  // unfinished requests
  uint32_t *abort_word;            // set on a timeout or an impossible state
  int R, Dv;
  int64_t Q;                       // tasks a round
  int64_t limit;                   // wall-clock ticks a wait may take
};
enum { kStT = 0, kStNp = 1, kStNb = 2, kStFin = 3 };

// ------------------------------------------------------------- LDS layouts
struct SmFold {
  uint4 ring[kFRing][kFStagePieces];
  int pick[kRP];
  double pnn[kRP], pinv[kRP];
};
struct SmGreedy {
  union {
    uint4 ring[kGRing][kGStagePieces];
    float mat[kRB * kGStride];
  };
  double nn[kRB], inv[kRB];
  int tok[kRB];
};
struct SmSelect {
  uint32_t v[kSelLds];            // key of each token: objective bits + 1, or 0
  uint32_t hist[kRWaves][257];    // per-wave digit counts (padded: waves on different banks)
  uint32_t tot[256];
};
union SmAll {
  SmFold f;
  SmGreedy g;
  SmSelect s;
};

// ----------------------------------------------------------- block helpers
__device__ unsigned long long block_max_u64(unsigned long long k, unsigned long long *sh) {
  k = wave_max_key((uint32_t)(k >> 32), (uint32_t)k);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = k;
  __syncthreads();
  unsigned long long m = sh[0];
#pragma unroll
  for (int w = 1; w < kRWaves; ++w) m = sh[w] > m ? sh[w] : m;
  __syncthreads();
  return uni64(m);
}
__device__ uint32_t block_max_u32(uint32_t v, unsigned long long *sh) {
  return (uint32_t)(block_max_u64((unsigned long long)v << 32, sh) >> 32);
}
__device__ uint32_t block_sum_u32(uint32_t v, unsigned long long *sh) {
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t s = 0;
#pragma unroll
  for (int w = 0; w < kRWaves; ++w) s += (uint32_t)sh[w];
  __syncthreads();
  return uniu(s);
}

// Tokens 0..N-1 in index order: thread t owns the contiguous run of E =
// ceil(N / kRThreads) <= 64 tokens from t E, tests them (loads issued eight at
// a time) into a bit mask, and one block-wide scan of the counts orders the
// runs. emit(rank, i) for the first `limit` tokens with test(load(i), i), on
// the thread that owns i. Returns how many were emitted.
template <typename Load, typename Test, typename Emit>
__device__ int ordered_scan(int N, int limit, Load load, Test test, Emit emit, int *sh) {
  const int E = (N + kRThreads - 1) / kRThreads;
  const int i0 = (int)threadIdx.x * E;
  // each thread starts its run at a different offset, so that the lanes of a
  // wave read different LDS banks
  const int rot = E > 1 ? (int)threadIdx.x % E : 0;
  unsigned long long flags = 0ull;
  for (int k0 = 0; k0 < E; k0 += 8) {
    uint32_t v[8];
    int e[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      e[u] = k0 + u + rot;
      e[u] -= e[u] >= E ? E : 0;
      const int i = i0 + e[u];
      v[u] = (k0 + u < E && i < N) ? load(i) : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + e[u];
      if (k0 + u < E && i < N && test(v[u], i)) flags |= 1ull << e[u];
    }
  }
  int total = 0;
  int rank = block_exclusive_scan(__popcll(flags), sh, &total);
  while (flags) {
    const int e = __ffsll((long long)flags) - 1;
    flags &= flags - 1ull;
    if (rank < limit) emit(rank, i0 + e);
    ++rank;
  }
  return min(uni(total), limit);
}
static_assert(kRoundMaxN <= 64 * kRThreads, "ordered_scan: one 64-bit mask a thread");

// ------------------------------------------------------------------- norms
// |x_i|^2 as the diagonal of a 32 x 32 MFMA Gram of 32 consecutive rows with
// themselves, in the Gram's 128-column chunks; 1 / |x_i| in fp64 (0 for a
// zero row). One wave per 32 rows; two chunks of loads in flight.
__global__ __launch_bounds__(256) void k_rnorm(const uint16_t *__restrict__ X, int64_t N_total, int Dv,
                                               const uint32_t *__restrict__ form, double *__restrict__ nn,
                                               double *__restrict__ inv) {
  if (form && *form != 0u) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * 32;
  if (row0 >= N_total) return;
  const int64_t row = min<int64_t>(row0 + (lane & 31), N_total - 1);
  const uint16_t *p = X + row * (int64_t)Dv + 8 * (lane >> 5);
  const int nc = Dv / 128;   // even
  // this lane's diagonal element, if any: column c = lane % 32 sits in half
  // (c % 8) / 4 at accumulator element 4 (c / 8) + c % 4
  const int c = lane & 31;
  const bool has = ((c & 7) >> 2) == (lane >> 5);
  const int vsel = 4 * (c >> 3) + (c & 3);
  double d = 0.0;
  uint4 f0[8], f1[8];
  auto load = [&](uint4 (&f)[8], int ch) {
#pragma unroll
    for (int s = 0; s < 8; ++s) f[s] = *reinterpret_cast<const uint4 *>(p + ch * 128 + 16 * s);
  };
  auto chunk = [&](const uint4 (&f)[8]) {
    f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f[0]), as_bf16x8(f[0]), f32x16{}, 0, 0, 0);
#pragma unroll
    for (int s = 1; s < 8; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f[s]), as_bf16x8(f[s]), acc, 0, 0, 0);
    float x = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) x = v == vsel ? acc[v] : x;
    d += (double)x;
  };
  load(f0, 0);
  for (int ch = 0; ch < nc; ch += 2) {
    load(f1, ch + 1);
    chunk(f0);
    if (ch + 2 < nc) load(f0, ch + 2);
    chunk(f1);
  }
  if (has && row0 + c < N_total) {
    nn[row0 + c] = d;
    inv[row0 + c] = d > 0.0 ? 1.0 / sqrt(d) : 0.0;
  }
}

// ------------------------------------------------------------------- prep
// even[r kEvenStride] = whether request r's relevance is too even for the rounds: its
// N/16-th largest value within kEvenBins bins of its median, a bin being 1/32
// of an octave (2 to 3%). The objectives of even relevance fall below the
// bound after few picks of a round, whatever the features. (A request of at
// most kRB tokens is its own candidates: no bound, so never too even.) Values
// are binned by their float bits relative to the mean's. One block a request,
// bound by the latency of its two passes over the relevance. Measured with
// log-normal relevance of spread s (gap in bins; select call, matrix / rounds
// in us), 32 x 2880 tokens 4096 wide, 1/9 kept: s 0.001 (0) 2027 / 2155, 0.1
// (5) 1938 / 1266, 0.3 (14) 1960 / 1177; 64 x 1024 tokens, 1/16 kept: 0.03 (2)
// 585 / 662, 0.1 (5) 569 / 573, 0.2 (10) 556 / 416.
constexpr int kEvenThreads = 1024, kEvenBins = 8;
__global__ __launch_bounds__(kEvenThreads) void k_reven(const float *__restrict__ scores,
                                                        const int32_t *__restrict__ cu_vis,
                                                        uint32_t *__restrict__ even) {
  constexpr int kWaves = kEvenThreads / 64;
  __shared__ uint32_t hist[kWaves][257];   // per-wave counts (padded: waves on different banks)
  __shared__ uint32_t tot[256];
  __shared__ float sh[kWaves];
  const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t n0 = cu_vis[r];
  const int N = cu_vis[r + 1] - (int)n0;
  if (N <= kRB) {
    if (tid == 0) even[r * SelectWs::kEvenStride] = 0u;
    return;
  }
  float sum = 0.f;
  for (int i = tid; i < N; i += kEvenThreads) sum += clean_score(scores[n0 + i]);
  for (int x = tid; x < kWaves * 257; x += kEvenThreads) (&hist[0][0])[x] = 0u;
  sum = wave_sum(sum);
  if (lane == 0) sh[wave] = sum;
  __syncthreads();
  float mean = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) mean += sh[w];
  const int mid = (int)__float_as_uint(mean / (float)N);
  for (int i = tid; i < N; i += kEvenThreads) {
    const int b = ((int)__float_as_uint(clean_score(scores[n0 + i])) - mid) >> 18;
    atomicAdd(&hist[wave][min(max(b, -128), 127) + 128], 1u);
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c += hist[w][tid];
    tot[tid] = c;
  }
  __syncthreads();
  if (tid >= 64) return;
  // lane l holds bins 4 l .. 4 l + 3: the highest bin with at least `want`
  // values in it and above
  uint32_t above = 0;   // values in the bins of later lanes
  for (int x = 0; x < 4; ++x) above += tot[4 * lane + x];
  const uint32_t mine = above;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_down(above, o);
    if (lane + o < 64) above += y;
  }
  above -= mine;
  auto quantile = [&](uint32_t want) {
    int b = -1;
    uint32_t acc = above;
    for (int x = 3; x >= 0; --x) {
      acc += tot[4 * lane + x];
      if (b < 0 && acc >= want) b = 4 * lane + x;
    }
    const unsigned long long m = __ballot(b >= 0);   // lane 0 counts all N values, so never empty
    return __shfl(b, 63 - __clzll((long long)m));
  };
  const int hi = quantile((uint32_t)N / 16), med = quantile((uint32_t)N / 2);
  if (lane == 0) even[r * SelectWs::kEvenStride] = hi - med < kEvenBins ? 1u : 0u;
}

// Fold-tile prefixes (one F task per kFRows tokens of a request), the state,
// the counters; the form, where the device chooses it: the matrix (1) if any
// request's relevance is too even. One block.
__global__ __launch_bounds__(1024) void k_rprep(const int32_t *__restrict__ cu_vis, int R, int64_t *__restrict__ ftoff,
                                                int32_t *__restrict__ st, uint32_t *__restrict__ dcnt,
                                                unsigned long long *__restrict__ head, uint32_t *__restrict__ live,
                                                uint32_t *__restrict__ abort_word, const uint32_t *__restrict__ even,
                                                uint32_t *__restrict__ form) {
  __shared__ int64_t sh[16];
  __shared__ int64_t s_run;
  __shared__ uint32_t s_form;
  if (threadIdx.x == 0) {
    s_run = 0;
    s_form = 0u;
    *head = 0ull;
    *live = (uint32_t)R;
    *abort_word = 0u;
  }
  __syncthreads();
  if (form) {
    for (int r = threadIdx.x; r < R; r += blockDim.x)
      if (even[r * SelectWs::kEvenStride] != 0u) s_form = 1u;
    __syncthreads();
    if (threadIdx.x == 0) *form = s_form;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int base = 0; base < R; base += blockDim.x) {
    const int r = base + (int)threadIdx.x;
    int64_t c = 0;
    if (r < R) {
      const int N = cu_vis[r + 1] - cu_vis[r];
      c = (N + kFRows - 1) / kFRows;
      st[4 * r + kStT] = 0;
      st[4 * r + kStNp] = 0;
      st[4 * r + kStNb] = 0;
      st[4 * r + kStFin] = 0;
      dcnt[r] = 0u;
    }
    int64_t x = c;
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) sh[wave] = x;
    __syncthreads();
    int64_t before = 0, tot = 0;
    for (int w = 0; w < nw; ++w) {
      if (w < wave) before += sh[w];
      tot += sh[w];
    }
    if (r < R) ftoff[r] = s_run + before + x - c;
    __syncthreads();
    if (threadIdx.x == 0) s_run += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) ftoff[R] = s_run;
}

// ------------------------------------------------------------------ tasks
struct Req {
  int r;
  int64_t n0, k0;
  int N, K;
};

__device__ void finish_request(const RArgs &a, const Req &q, int *shi) {
  // kept = the tokens marked -inf, ascending (Eq. 12)
  const uint32_t *dl = reinterpret_cast<const uint32_t *>(a.dl + q.n0);
  ordered_scan(
      q.N, q.K, [&](int i) { return ld_u32(dl + i); },
      [&](uint32_t v, int) { return v == __float_as_uint(-INFINITY); },
      [&](int rank, int i) { a.kept[q.k0 + rank] = i; }, shi);
  if (threadIdx.x == 0) {
    st_i32(a.st + 4 * q.r + kStFin, 1);
    __hip_atomic_fetch_add(a.live, 0xFFFFFFFFu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// S: the round's candidates, or the first pick, the degenerate end, the end.
__device__ void task_select(const RArgs &a, SmAll &sm, const Req &q, unsigned long long *shk, int *shi) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int t = uni(ld_i32(a.st + 4 * q.r + kStT));
  if (t == 0) {
    // delta starts at +inf; the first pick is the most relevant token (Eq. 9)
    unsigned long long best = 0ull;
    for (int i = tid; i < q.N; i += kRThreads) {
      st_f32(a.dl + q.n0 + i, INFINITY);
      const float w = clean_score(a.scores[q.n0 + i]);
      const unsigned long long k = ((unsigned long long)__float_as_uint(w) << 32) | (0xFFFFFFFFu - (unsigned)i);
      best = k > best ? k : best;
    }
    best = block_max_u64(best, shk);
    const int j = (int)(0xFFFFFFFFu - (uint32_t)best);
    vm_wait<0>();   // the +inf stores are complete before the pick's mark
    __syncthreads();
    if (tid == 0) {
      a.order[q.k0] = j;
      a.gains[q.k0] = __uint_as_float((uint32_t)(best >> 32));
      st_f32(a.dl + q.n0 + j, -INFINITY);
      st_i32(a.picks + (int64_t)q.r * kRP, j);
      st_i32(a.st + 4 * q.r + kStNp, 1);
      st_i32(a.st + 4 * q.r + kStNb, 0);
      st_i32(a.st + 4 * q.r + kStT, 1);
    }
    if (q.K == 1) {
      vm_wait<0>();
      __syncthreads();
      finish_request(a, q, shi);
    }
    return;
  }
  if (t >= q.K) {
    finish_request(a, q, shi);
    return;
  }

  // keys: v_i = objective bits + 1, or 0 when w_i delta_i is not a number
  // >= 0 (picked tokens: -inf or NaN)
  SmSelect &s = sm.s;
  uint32_t vmax = 0u, vmin = 0xFFFFFFFFu, nvalid = 0u;
  for (int base = 0; base < q.N; base += 8 * kRThreads) {
    float d[8], w[8];   // eight loads in flight a thread
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = base + u * kRThreads + tid;
      d[u] = i < q.N ? ld_f32(a.dl + q.n0 + i) : 0.f;
      w[u] = i < q.N ? a.scores[q.n0 + i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = base + u * kRThreads + tid;
      if (i >= q.N) continue;
      const float o = clean_score(w[u]) * d[u];
      const uint32_t v = o >= 0.f ? __float_as_uint(o) + 1u : 0u;
      s.v[i] = v;
      vmax = max(vmax, v);
      if (v != 0u) {
        vmin = min(vmin, v);
        ++nvalid;
      }
    }
  }
  vmax = block_max_u32(vmax, shk);
  vmin = ~block_max_u32(~vmin, shk);
  nvalid = block_sum_u32(nvalid, shk);

  if (vmax <= 1u) {
    // the best objective is 0 (or none is a number): from here on every step
    // takes the lowest-index token not yet picked
    const int t0 = t, need = q.K - t;
    const uint32_t *dl = reinterpret_cast<const uint32_t *>(a.dl + q.n0);
    ordered_scan(
        q.N, need, [&](int i) { return ld_u32(dl + i); },
        [&](uint32_t v, int) { return v != __float_as_uint(-INFINITY); },
        [&](int rank, int i) {
          a.order[q.k0 + t0 + rank] = i;
          a.gains[q.k0 + t0 + rank] = 0.f;
          st_f32(a.dl + q.n0 + i, -INFINITY);
        },
        shi);
    vm_wait<0>();
    __syncthreads();
    if (tid == 0) st_i32(a.st + 4 * q.r + kStT, q.K);
    finish_request(a, q, shi);
    return;
  }

  // Candidates: the tokens whose v exceeds a cut, at most kRB of them. The
  // cut is a boundary of 256 bins of width 2^shift over [lo, hi], refined
  // inside the bin that overflows kRB until at least kRB / 2 tokens lie above
  // it; if that bin has shrunk to a single value, its lowest-index tokens
  // fill the candidates up to kRB (at most four passes). T, the largest key
  // not taken, bounds every other token for the rest of the round.
  __shared__ uint32_t s_bin, s_acc;
  __shared__ int s_tie;
  uint32_t cut = 0u;   // candidates: v > cut, and (tie mode) v == cut at indices below tie
  int tie = 0;
  unsigned long long T = 0ull;
  if (nvalid > (uint32_t)kRB) {
    uint32_t lo = vmin, hi = vmax, above = 0u;   // `above`: valid tokens with v > hi
    bool tied = false;
    for (;;) {
      const uint32_t d = hi - lo;
      const int shift = d < 256u ? 0 : 24 - __clz(d);   // (hi - lo) >> shift < 256
      for (int x = tid; x < kRWaves * 257; x += kRThreads) (&s.hist[0][0])[x] = 0u;
      __syncthreads();
      const int wave = tid >> 6;
      for (int i = tid; i < q.N; i += kRThreads) {
        const uint32_t v = s.v[i];
        if (v >= lo && v <= hi && v != 0u) atomicAdd(&s.hist[wave][(v - lo) >> shift], 1u);
      }
      __syncthreads();
      if (tid < 256) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kRWaves; ++w) c += s.hist[w][tid];
        s.tot[tid] = c;
      }
      __syncthreads();
      if (tid < 64) {
        // bins 4 lane .. 4 lane + 3; the one bin whose tokens push the count
        // (from the top) past kRB, and the count above it
        const uint32_t c0 = s.tot[4 * lane], c1 = s.tot[4 * lane + 1], c2 = s.tot[4 * lane + 2],
                       c3 = s.tot[4 * lane + 3];
        const uint32_t mine = c0 + c1 + c2 + c3;
        uint32_t incl = mine;   // suffix sum over lanes >= lane
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t y = __shfl_down(incl, o);
          if (lane + o < 64) incl += y;
        }
        const uint32_t after = above + incl - mine;
        if (after <= (uint32_t)kRB && after + mine > (uint32_t)kRB) {
          uint32_t acc = after, b;
          if (acc + c3 > (uint32_t)kRB) {
            b = 4 * lane + 3;
          } else if ((acc += c3) + c2 > (uint32_t)kRB) {
            b = 4 * lane + 2;
          } else if ((acc += c2) + c1 > (uint32_t)kRB) {
            b = 4 * lane + 1;
          } else {
            acc += c1;
            b = 4 * lane;
          }
          s_bin = b;
          s_acc = acc;
        }
      }
      __syncthreads();
      const uint32_t b = uniu(s_bin), acc = uniu(s_acc);
      __syncthreads();
      const uint32_t blo = lo + (b << shift);
      const uint32_t bhi = (uint32_t)min<uint64_t>((uint64_t)hi, (uint64_t)blo + ((1ull << shift) - 1ull));
      if (acc >= (uint32_t)kRB / 2) {
        cut = bhi;
        break;
      }
      if (shift == 0) {   // one value: its lowest-index tokens fill the rest
        cut = blo;
        tied = true;
        above = acc;
        break;
      }
      lo = blo;
      hi = bhi;
      above = acc;
    }
    if (tied) {
      // the (kRB - above + 1)-th token (in index order) with v == cut bounds the rest
      const int want = kRB - (int)above + 1;
      if (tid == 0) s_tie = q.N;
      __syncthreads();
      const uint32_t c = cut;
      ordered_scan(
          q.N, want, [&](int i) { return s.v[i]; }, [&](uint32_t v, int) { return v == c; },
          [&](int rank, int i) {
            if (rank == want - 1) s_tie = i;
          },
          shi);
      tie = uni(s_tie);
      T = ((unsigned long long)(cut - 1u) << 32) | (0xFFFFFFFFu - (unsigned)tie);
    } else {
      // T: the largest key among the valid tokens at or below the cut
      unsigned long long best = 0ull;
      for (int i = tid; i < q.N; i += kRThreads) {
        const uint32_t v = s.v[i];
        const unsigned long long k =
            (v != 0u && v <= cut) ? ((unsigned long long)(v - 1u) << 32) | (0xFFFFFFFFu - (unsigned)i) : 0ull;
        best = k > best ? k : best;
      }
      T = block_max_u64(best, shk);
    }
  }
  const uint32_t vs = cut;
  const int ti = tie;
  const int nb = ordered_scan(
      q.N, kRB, [&](int i) { return s.v[i]; },
      [&](uint32_t v, int i) { return v > vs || (v == vs && v != 0u && i < ti); },
      [&](int rank, int i) { st_i32(a.cand + (int64_t)q.r * kRB + rank, i); }, shi);
  if (tid == 0) {
    st_i32(a.st + 4 * q.r + kStNb, nb);
    st_i32(a.st + 4 * q.r + kStNp, 0);
    st_u64(a.st_T + q.r, T);
  }
}

// G: the candidates' mutual distances, then the greedy of Eq. 9-11 on them
// while each pick is certified (its key above T), at most kRP picks.
//
// The distances: the upper triangle of the kRB x kRB Gram in 32 x 32 blocks
// on the matrix cores, both directions of every pair, into LDS. The
// candidates' rows stream through an LDS ring (LDS DMA, 64 columns a stage);
// wave w owns up to three blocks of one block row or column, in the Gram's
// 128-column chunks folded into fp64. One block forms the whole matrix, so
// it never leaves LDS: as 21 tasks of one block each, the pairs cost a
// dequeue and a wait apiece and the matrix a round trip through memory
// (ragged batch of 128 requests: 16400 such tasks, 27 us each with the waits,
// 1.7 of 7.5 ms).
__device__ void task_greedy(const RArgs &a, SmAll &sm, const Req &q) {
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int nb = uni(ld_i32(a.st + 4 * q.r + kStNb));
  if (nb == 0) return;
  SmGreedy &g = sm.g;
  if (tid < kRB) {
    // slots past nb repeat the last candidate; their distances are not used
    const int p = ld_i32(a.cand + (int64_t)q.r * kRB + min(tid, nb - 1));
    g.tok[tid] = p;
    g.nn[tid] = a.nn[q.n0 + p];
    g.inv[tid] = a.inv[q.n0 + p];
  }
  __syncthreads();
  {
    const int Dv = a.Dv, nst = Dv / kFCols;   // even
    uint32_t dst[kGPerWave], voff[kGPerWave];
#pragma unroll
    for (int x = 0; x < kGPerWave; ++x) {
      const int slot = (wave + kRWaves * x) * 64 + lane, row = slot >> 3, piece = (slot & 7) ^ ((row >> 1) & 7);
      dst[x] = __builtin_amdgcn_readfirstlane(lds_u32(&g.ring[0][(wave + kRWaves * x) * 64]));
      voff[x] = (uint32_t)(((int64_t)g.tok[row] * Dv + piece * 8) * 2);
    }
    const char *base = (const char *)uniform_ptr(a.X + q.n0 * (int64_t)Dv);
    auto issue = [&](int st) {
      const uint32_t add = (uint32_t)(st % kGRing) * (kGStagePieces * 16);
#pragma unroll
      for (int x = 0; x < kGPerWave; ++x) dma16(dst[x] + add, base + (int64_t)st * kFCols * 2, voff[x]);
    };
    // Blocks (sa, sb), sa <= sb < 6, three a wave (the last wave none of its
    // third), as one A block row against three B block rows: wave 0 (0; 0 1 2),
    // 1 (0; 3 4 5), 2 (1; 1 2 3), 3 (2; 2 3 4), 4 (3; 3 4 5), 5 (5; 1 2 5),
    // 6 (4; 1 4 5), 7: none. Wave 5's first two and wave 6's first are the
    // mirrors of (1, 5), (2, 5) and (1, 4): the product of a pair of rows is
    // the same number either way round.
    static_assert(kRSub == 6 && kRWaves == 8, "the blocks of a wave");
    const int ra = wave < 2 ? 0 : wave < 5 ? wave - 1 : wave == 5 ? 5 : 4;
    const int rb[3] = {wave == 0 ? 0 : wave == 1 || wave == 4 ? 3 : wave == 3 ? 2 : 1,
                       wave == 0 ? 1 : wave == 1 || wave == 4 || wave == 6 ? 4 : wave == 3 ? 3 : 2,
                       wave == 0 ? 2 : wave == 2 ? 3 : wave == 3 ? 4 : 5};
    const bool works = wave < 7;
    int aslot[4], bslot[4];   // of block row 0; block row x is 256 x pieces on
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int c = lane & 31, sl = c * 8 + ((2 * s + (lane >> 5)) ^ ((c >> 1) & 7));
      aslot[s] = 256 * ra + sl;
      bslot[s] = sl;
    }
    double acc64[3][16];
    f32x16 acc[3];
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc64[x][v] = 0.0;
#pragma unroll
    for (int st = 0; st < kGRing - 1; ++st)
      if (st < nst) issue(st);
    for (int st = 0; st < nst; st += 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // stage st + h has landed; the barrier publishes it and retires every
        // read of the slot that is filled next
        if (st + h + kGRing - 2 < nst)
          vm_wait<(kGRing - 2) * kGPerWave>();
        else
          vm_wait<0>();
        __syncthreads();
        if (st + h + kGRing - 1 < nst) issue(st + h + kGRing - 1);
        const uint4 *ring = g.ring[(st + h) % kGRing];
        if (works) {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const bf16x8 fa = as_bf16x8(ring[aslot[s]]);
#pragma unroll
            for (int x = 0; x < 3; ++x)
              acc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, as_bf16x8(ring[bslot[s] + 256 * rb[x]]),
                                                               (h == 0 && s == 0) ? f32x16{} : acc[x], 0, 0, 0);
          }
        }
      }
      if (works) {
#pragma unroll
        for (int x = 0; x < 3; ++x)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc64[x][v] += (double)acc[x][v];
      }
    }
    __syncthreads();   // the ring is free: the matrix takes its place
    if (works) {
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        const int sj = 32 * rb[x] + (lane & 31), tj = g.tok[sj];
        const double nnj = g.nn[sj], invj = g.inv[sj];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int si = 32 * ra + (lane >> 5) * 4 + (v & 3) + 8 * (v >> 2), ti = g.tok[si];
          const double nni = g.nn[si], invi = g.inv[si];
          const float c = coverage_dir(ti, tj, acc64[x][v], nni, nnj, invi, invj);
          g.mat[si * kGStride + sj] = c;
          if (ra != rb[x]) {
            // the two directions differ only inside one 32-row block of X
            float m = c;
            if (__any((ti >> 5) == (tj >> 5))) m = coverage_dir(tj, ti, acc64[x][v], nnj, nni, invj, invi);
            g.mat[sj * kGStride + si] = m;
          }
        }
      }
    }
  }
  __syncthreads();
  if (wave != 0) return;
  constexpr int E = kRB / 64;
  const unsigned long long T = uni64(ld_u64(a.st_T + q.r));
  const int t = uni(ld_i32(a.st + 4 * q.r + kStT));
  int np = 0;
  float w[E], d[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int c = lane + 64 * e;
    const bool in = c < nb;
    const int tok = g.tok[c];
    w[e] = in ? clean_score(a.scores[q.n0 + tok]) : 0.f;
    d[e] = in ? ld_f32(a.dl + q.n0 + tok) : -INFINITY;
  }
  // One wave, one dependent step a pick, so the chain is kept short.
  // Objectives are compared as floats (a picked token's -inf or NaN counts
  // as 0). Candidates are listed by ascending index, so the lowest index
  // among equal objectives is the lowest slot, and the token itself is
  // needed only when a best objective equals the bound's. Pick p of the round
  // is kept by lane p % 64 (of two) as a slot; all are stored at the end.
  static_assert(kRP <= 128 && E == 3, "two picks and three slots a lane");
  const uint32_t Thi = (uint32_t)(T >> 32);
  int ps[2] = {0, 0};
  float pg[2] = {0.f, 0.f};
  for (;;) {
    float o[E];
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = w[e] * d[e];   // Eq. 11
    const float best = fmaxf(fmaxf(o[0], o[1]), fmaxf(o[2], 0.f));
    const float mb = wave_max(best);
    const uint32_t mbits = __float_as_uint(mb);
    if (mbits == 0u || mbits < Thi) break;   // the degenerate end, or not certified
    const unsigned long long m0 = __ballot(o[0] == mb), m1 = __ballot(o[1] == mb), m2 = __ballot(o[2] == mb);
    const unsigned long long ms = m0 ? m0 : m1 ? m1 : m2;
    const int slot = (int)__ffsll((long long)ms) - 1 + (m0 ? 0 : m1 ? 64 : 128);
    if (mbits == Thi && (0xFFFFFFFFu - (unsigned)uni(g.tok[slot])) <= (uint32_t)T) break;   // not certified
    const bool mine = lane == (np & 63), low = np < 64;
    ps[0] = mine && low ? slot : ps[0];
    pg[0] = mine && low ? mb : pg[0];
    ps[1] = mine && !low ? slot : ps[1];
    pg[1] = mine && !low ? mb : pg[1];
    ++np;
    if (t + np >= q.K || np >= kRP) break;
    const float *row = g.mat + slot * kGStride + lane;
#pragma unroll
    for (int e = 0; e < E; ++e) d[e] = fminf(d[e], row[64 * e]);   // Eq. 10 (slots past nb keep -inf)
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int x = lane + 64 * h;
    if (x < np) {
      const int j = g.tok[ps[h]];
      a.order[q.k0 + t + x] = j;
      a.gains[q.k0 + t + x] = pg[h];
      st_f32(a.dl + q.n0 + j, -INFINITY);
      st_i32(a.picks + (int64_t)q.r * kRP + x, j);
    }
  }
  if (lane == 0) {
    st_i32(a.st + 4 * q.r + kStT, t + np);
    st_i32(a.st + 4 * q.r + kStNp, np);
  }
}

// F: fold the round's picks into delta of tokens [kFRows f, kFRows f + kFRows):
// a kFRows x (32 NT) product (tokens x picks) on the matrix cores, both
// operands streamed through an LDS ring by LDS DMA, 64 columns a stage; each
// wave owns 32 tokens against the NT 32-pick tiles. Bound by the token rows,
// which every round reads again: so a round takes as many picks as the
// accumulators hold (fp32 and fp64 of 32 x 128 a wave).
template <int NT>
__device__ __forceinline__ void fold_tiles(const RArgs &a, SmFold &F, const Req &q, int f) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kPick = NT / 2;                  // pick DMA instructions a wave and stage
  constexpr int kPerWave = kFTokInstr + kPick;
  const int i0 = f * kFRows;
  const int nrows = min(kFRows, q.N - i0);
  const int Dv = a.Dv;

  // DMA: token instructions x < kFTokInstr cover slots (wave + 8 x) * 64 + lane
  // (rows 0..255); pick instruction y covers slots (wave + 8 y) * 64 + lane of
  // the pick part. Slot = row * 8 + (piece ^ ((row >> 1) & 7)).
  constexpr uint32_t kStageBytes = kFStagePieces * 16;
  uint32_t dst[kPerWave], voff[kPerWave];
#pragma unroll
  for (int x = 0; x < kFTokInstr; ++x) {
    const int slot = (wave + kRWaves * x) * 64 + lane, row = slot >> 3, piece = (slot & 7) ^ ((row >> 1) & 7);
    dst[x] = __builtin_amdgcn_readfirstlane(lds_u32(&F.ring[0][(wave + kRWaves * x) * 64]));
    voff[x] = (uint32_t)(((int64_t)min(row, nrows - 1) * Dv + piece * 8) * 2);
  }
#pragma unroll
  for (int y = 0; y < kPick; ++y) {
    const int slot = (wave + kRWaves * y) * 64 + lane, row = slot >> 3, piece = (slot & 7) ^ ((row >> 1) & 7);
    dst[kFTokInstr + y] =
        __builtin_amdgcn_readfirstlane(lds_u32(&F.ring[0][kFTokPieces + (wave + kRWaves * y) * 64]));
    voff[kFTokInstr + y] = (uint32_t)(((int64_t)F.pick[row] * Dv + piece * 8) * 2);
  }
  const char *tokbase = (const char *)uniform_ptr(a.X + (q.n0 + i0) * (int64_t)Dv);
  const char *pickbase = (const char *)uniform_ptr(a.X + q.n0 * (int64_t)Dv);
  const int nst = Dv / kFCols;   // even
  auto issue = [&](int st) {
    const uint32_t add = (uint32_t)(st % kFRing) * kStageBytes;
#pragma unroll
    for (int x = 0; x < kFTokInstr; ++x) dma16_nt(dst[x] + add, tokbase + (int64_t)st * kFCols * 2, voff[x]);
#pragma unroll
    for (int y = kFTokInstr; y < kPerWave; ++y) dma16(dst[y] + add, pickbase + (int64_t)st * kFCols * 2, voff[y]);
  };

  // Fragment slots: a row's piece is 2 s + lane / 32, XOR (row / 2) % 8; the
  // rows of a tile are 32 apart, so every tile's slot is the first one's plus
  // 256 (the XOR does not change).
  int aslot[4], bslot[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int piece = 2 * s + (lane >> 5), c = lane & 31;
    const int sl = c * 8 + (piece ^ ((c >> 1) & 7));
    aslot[s] = 32 * wave * 8 + sl;
    bslot[s] = kFTokPieces + sl;
  }

  double acc64[NT][16];
#pragma unroll
  for (int tn = 0; tn < NT; ++tn)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc64[tn][v] = 0.0;
  f32x16 acc[NT];

  issue(0);
  if (nst > 1) issue(1);
  for (int st = 0; st < nst; st += 2) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (st + h + 1 < nst)
        vm_wait<kPerWave>();
      else
        vm_wait<0>();
      __syncthreads();
      if (st + h + 2 < nst) issue(st + h + 2);
      const uint4 *ring = F.ring[(st + h) % kFRing];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bf16x8 fa = as_bf16x8(ring[aslot[s]]);
#pragma unroll
        for (int tn = 0; tn < NT; ++tn)
          acc[tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, as_bf16x8(ring[bslot[s] + 256 * tn]),
                                                            (h == 0 && s == 0) ? f32x16{} : acc[tn], 0, 0, 0);
      }
    }
#pragma unroll
    for (int tn = 0; tn < NT; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc64[tn][v] += (double)acc[tn][v];
  }

  // distances, their minimum over the picks (lanes of a half hold one pick
  // column each), and the fold into delta (Eq. 10). Rows past the end repeat
  // the last one (not stored), and pick slots past np the last pick (folding
  // it twice changes nothing).
  int pk[NT];
  double pnn[NT], pinv[NT];
#pragma unroll
  for (int tn = 0; tn < NT; ++tn) {
    const int k = 32 * tn + (lane & 31);
    pk[tn] = F.pick[k];
    pnn[tn] = F.pnn[k];
    pinv[tn] = F.pinv[k];
  }
  const int il0 = 32 * wave + (lane >> 5) * 4;
  float m[16];
  // Where no token's norm equals a pick's (no duplicate of a pick, no pick
  // itself) and all are finite, a distance is max(0, 1 - dot inv inv) alone
  // (a zero row has inv 0, so 1), and its minimum over the picks that of the
  // largest product: 4 operations a pair instead of 15.
  bool special = false;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const double nni = a.nn[q.n0 + i0 + min(il0 + (v & 3) + 8 * (v >> 2), nrows - 1)];
    special |= !(nni < (double)INFINITY);
#pragma unroll
    for (int tn = 0; tn < NT; ++tn) special |= nni == pnn[tn];
  }
#pragma unroll
  for (int tn = 0; tn < NT; ++tn) special |= !(pnn[tn] < (double)INFINITY);
  if (!__any(special)) {
    bool fwd[NT];   // the pick's 32-row block of X is not above the wave's tokens'
#pragma unroll
    for (int tn = 0; tn < NT; ++tn) fwd[tn] = (pk[tn] >> 5) <= (i0 >> 5) + wave;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const double invi = a.inv[q.n0 + i0 + min(il0 + (v & 3) + 8 * (v >> 2), nrows - 1)];
      double u = 0.0;
#pragma unroll
      for (int tn = 0; tn < NT; ++tn) {
        const double t = acc64[tn][v] * (fwd[tn] ? pinv[tn] : invi) * (fwd[tn] ? invi : pinv[tn]);
        u = tn == 0 ? t : fmax(u, t);
      }
      const double c = 1.0 - u;
      m[v] = c > 0.0 ? (float)c : 0.0f;
    }
  } else {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = i0 + min(il0 + (v & 3) + 8 * (v >> 2), nrows - 1);
      const double nni = a.nn[q.n0 + i], invi = a.inv[q.n0 + i];
      float mv = INFINITY;
#pragma unroll
      for (int tn = 0; tn < NT; ++tn)
        mv = fminf(mv, coverage_dir(pk[tn], i, acc64[tn][v], pnn[tn], nni, pinv[tn], invi));
      m[v] = mv;
    }
  }
  // the minimum over the 32 lanes, each step halving the values a lane keeps
  // (bit 4 of the lane chooses rows 8.., bit 3 rows 4.. of those, and so on)
#pragma unroll
  for (int w = 8, o = 16; w >= 1; w >>= 1, o >>= 1) {
    const bool up = (lane & o) != 0;
#pragma unroll
    for (int v = 0; v < w; ++v) {
      const float keep = up ? m[v + w] : m[v], give = up ? m[v] : m[v + w];
      m[v] = fminf(keep, __shfl_xor(give, o));
    }
  }
  const float mv = fminf(m[0], __shfl_xor(m[0], 1));
  if ((lane & 1) == 0) {
    const int vs = (lane >> 1) & 15;   // bits 4..1 of the lane, as the steps above chose them
    const int il = il0 + (vs & 3) + 8 * (vs >> 2);
    if (il < nrows) {
      float *p = a.dl + q.n0 + i0 + il;
      st_f32(p, fminf(ld_f32(p), mv));
    }
  }
}

__device__ void task_fold(const RArgs &a, SmAll &sm, const Req &q, int f) {
  const int tid = threadIdx.x;
  const int t = uni(ld_i32(a.st + 4 * q.r + kStT));
  if (t >= q.K) return;   // the last round's picks need no fold (they are marked)
  const int np = uni(ld_i32(a.st + 4 * q.r + kStNp));
  if (np <= 0) return;
  SmFold &F = sm.f;
  if (tid < kRP) {
    const int p = ld_i32(a.picks + (int64_t)q.r * kRP + min(tid, np - 1));
    F.pick[tid] = p;
    F.pnn[tid] = a.nn[q.n0 + p];
    F.pinv[tid] = a.inv[q.n0 + p];
  }
  __syncthreads();
  if (np > 64)
    fold_tiles<kFTiles>(a, F, q, f);
  else
    fold_tiles<2>(a, F, q, f);
}

// ------------------------------------------------------------- the rounds
// The task at position u of a macro-round. The requests form two halves,
// A = [0, RA) and B = [RA, R), half a round apart, so that one half's serial
// chain (select, candidate Gram, greedy) runs while the other half folds.
// Macro-round m lists, in this order:
//   S of A's round m; the first half of B's folds of round m - 1; G of A's
//   round m; the rest of B's folds; S of B's round m; the first half of A's
//   folds of round m; G of B's round m; the rest of A's folds.
// The folds listed between a select and its greedy keep the blocks busy while
// the select runs. Each task depends only on tasks listed before it. Sets kind
// (0 S, 1 G, 2 F), the request and the sub-index (F: the fold tile within the
// request); returns -1 for B's folds (they belong to round m - 1), else 0.
// `ft(i)` is the first fold tile of request i (ft(R) the total). Every value
// is wave-uniform.
template <typename Ft>
__device__ __forceinline__ int64_t decode_task(int64_t u, int64_t R, Ft ft, int &kind, int &r, int &sub) {
  const int64_t RA = (R + 1) / 2, RB = R - RA;
  const int64_t FA = ft(RA), FB = ft(R) - FA, hA = FA / 2, hB = FB / 2;
  // fold tile g of the requests [r0, r0 + nr) (g counts from the first of them)
  auto fold = [&](int64_t r0, int64_t nr, int64_t g) {
    const int64_t f = ft(r0) + g;
    int64_t lo = r0, hi = r0 + nr - 1;   // the last request whose first tile is <= f
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) >> 1;
      if (ft(mid) <= f)
        lo = mid;
      else
        hi = mid - 1;
    }
    kind = 2;
    r = (int)lo;
    sub = (int)(f - ft(lo));
  };
  int64_t x = u;
  if (x < RA) {
    kind = 0;
    r = (int)x;
    return 0;
  }
  x -= RA;
  if (x < hB) {
    fold(RA, RB, x);
    return -1;
  }
  x -= hB;
  if (x < RA) {
    kind = 1;
    r = (int)x;
    return 0;
  }
  x -= RA;
  if (x < FB - hB) {
    fold(RA, RB, hB + x);
    return -1;
  }
  x -= FB - hB;
  if (x < RB) {
    kind = 0;
    r = (int)(RA + x);
    return 0;
  }
  x -= RB;
  if (x < hA) {
    fold(0, RA, x);
    return 0;
  }
  x -= hA;
  if (x < RB) {
    kind = 1;
    r = (int)(RA + x);
    return 0;
  }
  x -= RB;
  fold(0, RA, hA + x);
  return 0;
}

// Tasks of a request of `tiles` fold tiles a round, and how many of its tasks are
// complete before one of this kind may start in round n: every task of earlier
// rounds and, in its own, S before G, and both before F.
__device__ __forceinline__ int64_t tasks_a_round(int64_t tiles) { return 2 + tiles; }
__device__ __forceinline__ int64_t tasks_before(int64_t n, int kind, int64_t tiles) { return n * tasks_a_round(tiles) + kind; }

// Whether a task of round n whose dependencies are complete shows a fault: the
// first round makes one pick and every later one at least one, so the select of
// round K finds K picks and ends the request, and no task of a later round ever
// has its dependencies. (How far the queue's head has run says nothing: blocks
// pass over the tasks of finished requests without waiting, so beside one
// unfinished request of c tasks a round the head runs up to grid / c rounds
// ahead of it.)
__device__ __forceinline__ bool past_last_round(int64_t n, int64_t K) { return n > K; }

__global__ __launch_bounds__(kRThreads) void k_rounds(RArgs a) {
  __shared__ SmAll sm;
  __shared__ unsigned long long shk[kRWaves];
  __shared__ int shi[kRWaves];
  __shared__ int s_task[5];   // status (0 run, 2 exit), request, kind, sub-index, round
  __shared__ int s_ft[kFtLds];   // fold-tile prefixes of batches of fewer than kFtLds requests
  if (a.form && *a.form != 0u) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uni(tid >> 6);
  if (a.R < kFtLds)
    for (int x = tid; x <= a.R; x += kRThreads) s_ft[x] = (int)a.ftoff[x];
  __syncthreads();
  auto ft_at = [&](int64_t i) -> int64_t { return uni_i64(a.R < kFtLds ? (int64_t)s_ft[i] : a.ftoff[i]); };
  int prev = -1;   // the request of the task this block has just completed
  for (;;) {
    // Wave 0 publishes the completed task (every wave waited for its stores
    // before the last barrier) and takes the next one, passing over those of
    // finished requests; all its lanes poll the same words, so its branches
    // stay uniform. The words of one step are loaded together: each load goes
    // to the device's coherence point, about a microsecond away.
    if (wave == 0) {
      if (lane == 0 && prev >= 0)
        __hip_atomic_fetch_add(a.dcnt + prev, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int status = 0, r = 0, kind = 0, sub = 0;
      int64_t n = 0;
      do {
        unsigned long long qi = 0ull;
        if (lane == 0) qi = __hip_atomic_fetch_add(a.head, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned long long ctl = ld_u64(a.ctl);   // live requests | abort word << 32
        qi = uni64(qi);
        ctl = uni64(ctl);
        status = 0;
        if ((ctl >> 32) != 0ull || (uint32_t)ctl == 0u) {
          status = 2;
          break;
        }
        const int64_t m = (int64_t)(qi / (unsigned long long)a.Q);   // macro-round
        const int64_t u = (int64_t)qi - m * a.Q;
        const int64_t tq = decode_task(u, a.R, ft_at, kind, r, sub);
        n = m + tq;   // tq = -1: B's folds of the previous round
        if (n < 0) {
          status = 1;   // B's folds before its first round: no task
          continue;
        }
        const int64_t need = tasks_before(n, kind, ft_at(r + 1) - ft_at(r));
        const uint64_t t0 = wall_clock64();
        for (;;) {
          uint32_t done = ld_u32(a.dcnt + r);
          int fin = ld_i32(a.st + 4 * r + kStFin);
          uint32_t ab = ld_u32(a.abort_word);
          done = uniu(done);
          fin = uni(fin);
          ab = uniu(ab);
          if (fin != 0) {
            status = 1;   // finished: nothing waits for its counts any more
            break;
          }
          if ((int64_t)done >= need) {
            // The loads above may be served out of order: read the end mark
            // again now that the counts are there. A fold needs no second
            // look (it returns when the picks are complete).
            if (kind != 2 && uni(ld_i32(a.st + 4 * r + kStFin)) != 0) status = 1;
            break;
          }
          if (ab != 0u) {
            status = 2;
            break;
          }
          if ((int64_t)(wall_clock64() - t0) > a.limit) {
            if (lane == 0) st_u32(a.abort_word, 1u);
            status = 2;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
      } while (status == 1);
      if (lane == 0) {
        s_task[0] = status;
        s_task[1] = r;
        s_task[2] = kind;
        s_task[3] = sub;
        s_task[4] = (int)n;   // below 2^31: the counts reached it
      }
    }
    __syncthreads();
    const int status = uni(s_task[0]);
    if (status == 2) break;
    const int r = uni(s_task[1]), kind = uni(s_task[2]), sub = uni(s_task[3]), n = uni(s_task[4]);
    __syncthreads();
    Req q;
    q.r = r;
    q.n0 = uni(a.cu_vis[r]);
    q.N = uni(a.cu_vis[r + 1]) - (int)q.n0;
    q.k0 = uni(a.cu_keep[r]);
    q.K = uni(a.cu_keep[r + 1]) - (int)q.k0;
    if (past_last_round(n, q.K)) {
      if (tid == 0) st_u32(a.abort_word, 1u);
      break;
    }
    if (kind == 0)
      task_select(a, sm, q, shk, shi);
    else if (kind == 1)
      task_greedy(a, sm, q);
    else
      task_fold(a, sm, q, sub);
    // this task's stores are complete before wave 0 publishes it
    vm_wait<0>();
    __syncthreads();
    prev = r;
  }
}

// After a timeout: every request not finished gets kept = order = -1 and
// gains = NaN.
__global__ __launch_bounds__(256) void k_rfail(const uint32_t *__restrict__ abort_word, const int32_t *__restrict__ st,
                                               const int32_t *__restrict__ cu_keep, int R, int32_t *__restrict__ kept,
                                               int32_t *__restrict__ order, float *__restrict__ gains) {
  if (*abort_word == 0u) return;
  for (int r = blockIdx.x; r < R; r += gridDim.x) {
    if (st[4 * r + kStFin] != 0) continue;
    for (int k = cu_keep[r] + (int)threadIdx.x; k < cu_keep[r + 1]; k += blockDim.x) {
      kept[k] = -1;
      order[k] = -1;
      gains[k] = __builtin_nanf("");
    }
  }
}

}  // namespace

// ------------------------------------------------------------------- host
bool rounds_supported(int32_t N_max, int32_t Dv, last_dtype fdtype) {
  return fdtype == LAST_BF16 && Dv % 256 == 0 && Dv <= kRoundMaxDv && N_max <= kRoundMaxN &&
         (int64_t)N_max * Dv * 2 < ((int64_t)1 << 32);
}

hipError_t launch_round_prep(int32_t R, const SelectWs &w, const float *scores, const int32_t *cu_vis, hipStream_t s) {
  launch_begin("rounds_prep", s);
  if (w.form) hipLaunchKernelGGL(k_reven, dim3((unsigned)R), dim3(kEvenThreads), 0, s, scores, cu_vis, w.even);
  uint32_t *live = reinterpret_cast<uint32_t *>(w.r_ctl + 1);
  hipLaunchKernelGGL(k_rprep, dim3(1), dim3(1024), 0, s, cu_vis, R, w.r_qoff, w.r_st, w.r_dcnt, w.r_ctl, live, live + 1,
                     w.even, w.form);
  return launch_end(s);
}

hipError_t launch_round_norms(int32_t Dv, const SelectPlan &p, const SelectWs &w, const void *feats,
                              hipStream_t s) {
  if (p.N_total == 0) return hipSuccess;
  launch_begin("norms", s);
  hipLaunchKernelGGL(k_rnorm, dim3((unsigned)((p.N_total + 127) / 128)), dim3(256), 0, s,
                     static_cast<const uint16_t *>(feats), p.N_total, Dv, w.form, w.nn, w.inv);
  return launch_end(s);
}

hipError_t launch_round_pick(int32_t R, int32_t Dv, const SelectPlan &p, const SelectWs &w, const float *scores,
                             const void *feats, const int32_t *cu_vis, const int32_t *cu_keep, int32_t *kept,
                             int32_t *order, float *gains, hipStream_t s) {
  const int64_t Q = p.round_Q;
  int64_t wait_us = 10000000;
  if (const char *env = getenv("LAST_MC_WAIT_US")) wait_us = std::max<int64_t>(0, atoll(env));
  RArgs a{};
  a.scores = scores;
  a.X = static_cast<const uint16_t *>(feats);
  a.nn = w.nn;
  a.inv = w.inv;
  a.cu_vis = cu_vis;
  a.cu_keep = cu_keep;
  a.kept = kept;
  a.order = order;
  a.gains = gains;
  a.dl = w.r_dl;
  a.cand = w.r_cand;
  a.picks = w.r_picks;
  a.st = w.r_st;
  a.st_T = w.r_T;
  a.dcnt = w.r_dcnt;
  a.ftoff = w.r_qoff;
  a.form = w.form;
  a.head = w.r_ctl;
  a.live = reinterpret_cast<uint32_t *>(w.r_ctl + 1);
  a.abort_word = reinterpret_cast<uint32_t *>(w.r_ctl + 1) + 1;
  a.ctl = w.r_ctl + 1;
  a.R = R;
  a.Dv = Dv;
  const int grid = std::max(1, device_cus());
  a.Q = Q;
  a.limit = device_wall_khz() * wait_us / 1000;
  launch_begin("rounds", s);
  hipLaunchKernelGGL(k_rounds, dim3((unsigned)grid), dim3(kRThreads), 0, s, a);
  hipLaunchKernelGGL(k_rfail, dim3((unsigned)std::min(R, 1024)), dim3(256), 0, s, a.abort_word, w.r_st, cu_keep, R,
                     kept, order, gains);
  return launch_end(s);
}

}  // namespace last
