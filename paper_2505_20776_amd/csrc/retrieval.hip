// Cross-model Retrieval kernels (SpecExtend Sec. 3.2.1 and Alg. 1):
//   chunk_scores_kernel  - normalise the per-chunk exponential sums left by
//                          the prefix pass, average over chunk tokens and heads
//   select_*_kernel      - SelectChunks: top-k by ranking (short inputs) or radix select, ascending output
//   gather_*_kernel      - UpdateDraftCache: copy the chosen chunks verbatim
#include "common.h"
#include "score_row.h"

namespace specext {
namespace {

// --------------------------------------------------------------------------
// chunk scores
// --------------------------------------------------------------------------

// scores[r][c] = (1/Hq) * sum_h  sum_blocks  blocksum(h, t) * exp2(ref - lse2(h, t)) / |c|
// The prefix pass leaves one (sum, ref) pair per score block (score_gran keys;
// a chunk is a whole number of blocks).  The heads of a chunk are dealt to the four lanes of a
// quad (head h to lane h mod 4: with four heads per group a quad's load is 32 consecutive bytes);
// each adds its heads in ascending order, and the four sums are combined in a fixed order: a
// deterministic fp32 sum.  The blocks of a longer chunk are dealt to 4, 16 or 64 quads, whose sums
// are combined in a fixed order too.
//
// What bounds it: every pair group is a 32-byte piece of a line of its own (the pairs of a block are
// [rows], as the prefix kernels write them), fetched from behind another XCD's L2, so the kernel is one
// trip to memory if all of a thread's loads are in flight together and enough compute units ask.  Hence
// one wavefront and 16 chunks per workgroup; 64 chunks per workgroup with a head's loads one after the
// other took 5.5 us for 512 chunks of one block and 7.9 us for 512 of two (32 heads in 8 groups), so
// 2.9 and 3.65 us; with the inputs among the first arguments and no divisions by the group size 2.7 and 3.2.
constexpr int kHeadsAtOnce = 8;                // heads of one thread whose loads are in flight together

// NSUB score blocks per lane and step, QUADS quads per chunk: the smallest pair whose product covers a chunk's blocks
// (chunks beyond 256 blocks take several steps).
template <int NSUB, int QUADS>
struct ScoreShape {
  static constexpr int kBlocks = NSUB;
  static constexpr int kQuads = QUADS;
  static constexpr int kLanes = 4 * QUADS;                         // per chunk
  static constexpr int kThreads = kLanes > 64 ? kLanes : 64;       // of a workgroup of chunk_scores_kernel
  static constexpr int kChunks = kThreads / kLanes;
};
// Measured, us for the scores of one row over 8K fp32 keys (32 heads in 8 groups) in chunks of 16, 64 and 512 blocks: 17, 66
// and 490 with one quad per chunk, whose blocks beyond the first four come one after the other; 4.1, 4.0 and 5.7 so.
template <class F>
__host__ void with_score_shape(int blocks, F&& f) {
  if (blocks <= 1) f(ScoreShape<1, 1>{});
  else if (blocks <= 2) f(ScoreShape<2, 1>{});
  else if (blocks <= 4) f(ScoreShape<4, 1>{});
  else if (blocks <= 8) f(ScoreShape<2, 4>{});
  else if (blocks <= 16) f(ScoreShape<4, 4>{});
  else if (blocks <= 32) f(ScoreShape<2, 16>{});
  else if (blocks <= 64) f(ScoreShape<4, 16>{});
  else if (blocks <= 128) f(ScoreShape<2, 64>{});
  else f(ScoreShape<4, 64>{});
}

// The scores' inputs, the first arguments of both kernels (in registers at their start: common.h).
#define SPECEXT_SCORE_PARAMS uint64_t path_at, uint64_t count_at, uint64_t part_at, uint64_t lse2_at, int T, int M, int G, int Hq, int n_sub, int per_chunk
#define SPECEXT_SCORE_ARGS(p) address_of(row_path), address_of(row_count), address_of((p).chunk_part), address_of((p).lse2), (p).T, (p).M, (p).G, (p).Hq, (p).n_sub, (p).B / (p).score_gran
struct ScoreInputs {
  const float *part, *lse2;      // AttnParams::chunk_part, lse2
  int M, G, Hq, n_sub, per_chunk;      // per_chunk: score blocks of a chunk
};

// value of quad lane I in every lane of the quad
template <int I>
__device__ __forceinline__ float quad_lane(float v) {
  return SPECEXT_DPP(v, I * 0x55);
}

// The four partial sums of chunk c that chunk_score adds, by the chunk's lanes; `lane` = number among them.  QUADS = 1: lane
// p returns the p-th.  4 or 16: every lane returns the first, the others are zero.  64: the lanes of wave p return the p-th.
template <class Shape>
__device__ __forceinline__ float chunk_partial(const ScoreInputs& p, int t, int c, int lane) {
  constexpr int kBlocks = Shape::kBlocks;
  const int part = lane & 3;
  const int sub_lo = min(c * p.per_chunk, (p.n_sub - 1) / p.per_chunk * p.per_chunk);      // chunks past the end re-read the last one, unused
  const int sub_hi = min(sub_lo + p.per_chunk, p.n_sub);
  const float inv_g = 1.0f / static_cast<float>(p.G);
  float acc = 0.f;
  for (int sb0 = sub_lo + (lane >> 2); sb0 < sub_hi; sb0 += kBlocks * Shape::kQuads) {
    for (int hb = part; hb < p.Hq; hb += 4 * kHeadsAtOnce) {
      float l2[kHeadsAtOnce];
      float2 pair[kHeadsAtOnce][kBlocks];
#pragma unroll
      for (int u = 0; u < kHeadsAtOnce; ++u) {
        const int h = min(hb + 4 * u, p.Hq - 1);                 // heads past the end re-read the last one, unused
        const int g = static_cast<int>((static_cast<float>(h) + 0.5f) * inv_g);      // h / G, exact for h < 2^20
        const int m = t * p.G + (h - g * p.G);
        l2[u] = p.lse2[g * p.M + m];
        const float* src = p.part + (static_cast<int64_t>(g) * p.n_sub * p.M + m) * 2;
#pragma unroll
        for (int b = 0; b < kBlocks; ++b)                         // blocks past the chunk's end re-read its last one, unused
          pair[u][b] = *reinterpret_cast<const float2*>(src + static_cast<int64_t>(min(sb0 + b * Shape::kQuads, sub_hi - 1)) * p.M * 2);
      }
#pragma unroll
      for (int u = 0; u < kHeadsAtOnce; ++u) {
        if (hb + 4 * u < p.Hq) {
#pragma unroll
          for (int b = 0; b < kBlocks; ++b)
            if (sb0 + b * Shape::kQuads < sub_hi) acc += pair[u][b].x * exp2f(pair[u][b].y - l2[u]);
        }
      }
    }
  }
  return Shape::kQuads == 1 ? acc : Shape::kQuads == 4 ? row16_sum(acc) : wave_sum(acc);
}

// of chunk c of B keys of L
__device__ __forceinline__ float chunk_score(int c, int B, int L, int Hq, float p0, float p1, float p2, float p3) {
  const int size = min(B, L - c * B);
  return (((p0 + p1) + p2) + p3) / (static_cast<float>(size) * static_cast<float>(Hq));
}

template <class Shape>
__global__ __launch_bounds__(Shape::kThreads) void chunk_scores_kernel(SPECEXT_SCORE_PARAMS, int C, int B, int L, int first_row,
                                                                       float* scores) {
  const ScoreInputs in = {in_global<const float>(part_at), in_global<const float>(lse2_at), M, G, Hq, n_sub, per_chunk};
  const int t = scored_row(in_global<const int>(path_at), in_global<const int>(count_at), T, first_row + blockIdx.y);
  const int c = blockIdx.x * Shape::kChunks + threadIdx.x / Shape::kLanes;
  const int lane = threadIdx.x % Shape::kLanes;
  const float acc = chunk_partial<Shape>(in, t, c, lane);
  float parts[4] = {acc, 0.f, 0.f, 0.f};
  if constexpr (Shape::kQuads == 1) {
    parts[0] = quad_lane<0>(acc), parts[1] = quad_lane<1>(acc), parts[2] = quad_lane<2>(acc), parts[3] = quad_lane<3>(acc);
  } else if constexpr (Shape::kQuads == 64) {
    __shared__ float of_wave[4];
    if ((lane & 63) == 0) of_wave[lane >> 6] = acc;
    __syncthreads();
    for (int w = 0; w < 4; ++w) parts[w] = of_wave[w];
  }
  if (lane == 0 && c < C)
    scores[static_cast<int64_t>(blockIdx.y) * C + c] = chunk_score(c, B, L, Hq, parts[0], parts[1], parts[2], parts[3]);
}

// --------------------------------------------------------------------------
// top-k selection
// --------------------------------------------------------------------------

constexpr int kSelThreads = 1024;

// Map a finite float to a uint32 whose unsigned order is the float order.
__device__ __forceinline__ uint32_t orderable(float f) {
  f += 0.0f;                                   // -0 -> +0 so they compare equal
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inclusive prefix sum over the wave, in registers (six data-parallel-primitive steps, no LDS round trips).
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8 within rows of 16 lanes
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);      // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);      // row_bcast:31 into rows 2 and 3
  return v;
}

// Exclusive block prefix sum of one int per thread; returns the block total in `total`.
__device__ __forceinline__ int block_exclusive_scan(int v, int* wave_sums, int& total) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int incl = wave_inclusive_scan(v);
  __syncthreads();                              // wave_sums may still be read from the previous call
  if (lane == 63) wave_sums[wave] = incl;
  __syncthreads();
  int base = 0;
  total = 0;
  const int n_waves = blockDim.x >> 6;
  for (int w = 0; w < n_waves; ++w) {
    const int s = wave_sums[w];
    if (w < wave) base += s;
    total += s;
  }
  return base + incl - v;
}

// Block-wide count of a predicate (up to 32 flags per thread, bit u of
// `flags` = flag u); every thread gets the total.  Wave counts come from ballots;
// `slots` must hold blockDim.x / 64 ints and alternate between two buffers from
// call to call so that one barrier per call is enough.
__device__ __forceinline__ int block_count(unsigned flags, int n_flags, int* slots) {
  int c = 0;
  for (int u = 0; u < n_flags; ++u) c += __popcll(__ballot((flags >> u) & 1u));
  if ((threadIdx.x & 63) == 0) slots[threadIdx.x >> 6] = c;
  __syncthreads();
  // all sixteen slots are read at once (slots of absent waves hold zero), one LDS round trip
  const int4 a = *reinterpret_cast<const int4*>(slots), b = *reinterpret_cast<const int4*>(slots + 4),
             cc = *reinterpret_cast<const int4*>(slots + 8), d = *reinterpret_cast<const int4*>(slots + 12);
  return ((a.x + a.y) + (a.z + a.w)) + ((b.x + b.y) + (b.z + b.w)) + ((cc.x + cc.y) + (cc.z + cc.w)) +
         ((d.x + d.y) + (d.z + d.w));
}

// One workgroup.  The key value V of the k-th largest score is built bit by bit from
// the top: a bit stays set if at least k keys are >= the candidate.  Scores above V
// are all taken; of the scores equal to V the lowest-indexed ones fill what is left.
// A last pass in index order (block scans over the keep flags) writes the output
// ascending.  For inputs that the byte-wise selection does not take; the keys are re-read from memory.

__global__ __launch_bounds__(kSelThreads) void select_kernel(const float* __restrict__ scores, int n, int k,
                                                            int* __restrict__ idx_out, int* __restrict__ n_out) {
  __shared__ __attribute__((aligned(16))) int slots[2][kSelThreads / 64];
  __shared__ int wave_sums[kSelThreads / 64];

  const int k_eff = min(k, n);
  if (threadIdx.x == 0) *n_out = k_eff;
  for (int i = k_eff + threadIdx.x; i < k; i += blockDim.x) idx_out[i] = -1;
  if (k_eff == 0) return;
  if (threadIdx.x < 2 * (kSelThreads / 64)) slots[0][threadIdx.x] = 0;      // slots of absent waves stay zero
  __syncthreads();

  // how many keys are >= cand (block-wide), 32 keys per thread per round of ballots
  auto count_ge = [&](uint32_t cand, int* slot) {
    int total = 0;
    for (int base = 0; base < n; base += blockDim.x * 32) {
      unsigned flags = 0;
      for (int u = 0; u < 32; ++u) {
        const int i = base + u * blockDim.x + threadIdx.x;
        flags |= ((i < n && orderable(scores[i]) >= cand) ? 1u : 0u) << u;
      }
      // (an extra barrier keeps the slot buffer of the previous call intact)
      __syncthreads();
      total += block_count(flags, 32, slot);
    }
    return total;
  };
  uint32_t v = 0;
  int round = 0;
  for (int bit = 31; bit >= 0; --bit, ++round) {
    const uint32_t cand = v | (1u << bit);
    if (count_ge(cand, slots[round & 1]) >= k_eff) v = cand;
  }
  // v is the k-th largest key.  Keys above it: n_gt < k_eff; ties needed: k_eff - n_gt >= 1
  const int n_gt = v == 0xffffffffu ? 0 : count_ge(v + 1u, slots[round & 1]);
  const int need = k_eff - n_gt;
  int out_base = 0, tie_base = 0;
  for (int start = 0; start < n; start += blockDim.x) {
    const int i = start + threadIdx.x;
    uint32_t key = 0;
    if (i < n) key = orderable(scores[i]);
    const int is_tie = (i < n && key == v) ? 1 : 0;
    const int is_gt = (i < n && key > v) ? 1 : 0;
    int tie_total;
    const int tie_rank = tie_base + block_exclusive_scan(is_tie, wave_sums, tie_total);
    const int take = is_gt | (is_tie & (tie_rank < need ? 1 : 0));
    int take_total;
    const int pos = out_base + block_exclusive_scan(take, wave_sums, take_total);
    if (take) idx_out[pos] = i;
    out_base += take_total;
    tie_base += tie_total;
  }
}

// Inputs of at most kRankMax scores take the byte-wise selection below with one key per thread, those of at most
// kRadixMax with four (4096 scores of a 128K prefix: 25 us bit by bit as below, 8.2 us so).
constexpr int kRankMax = 1024;
constexpr int kRadixMax = 4 * kSelThreads;
constexpr int kScoreGroupsOneLaunch = 1600;
constexpr int kScoreChunksOneLaunch = 128;

// One workgroup (blockDim.x a multiple of 64), thread i holding the scores of chunks i, i + blockDim.x, ... (KPT of
// them).  The key of the k-th largest score is found a byte at a time from the top:
// a 256-bin histogram (LDS atomics) of the keys that match the bytes fixed so far, a
// suffix scan over the bins, and the bin that holds the k-th key fixes the next byte - four
// rounds instead of one compare of every key with every other.  Scores of one row share
// their leading bits, so the lanes of a wave that hold its first key's bin add as one.  Every wave does the scan
// for itself (four bins per lane), so a round costs one barrier.  Keys above the threshold
// are all taken; of the keys equal to it the lowest-indexed ones fill what is left; ballots
// and one exchange of per-wave counts give the ascending output.
template <int KPT>
struct RadixLds {
  __attribute__((aligned(16))) int hist[4][256];     // one histogram per round, all cleared up front
  int2 wave_counts[KPT * (kSelThreads / 64)];        // per key of a thread and wave: keys above the threshold, equal to it
};

template <int KPT>
__device__ __forceinline__ void radix_select_and_write(const float (&score)[KPT], int n, int k, int* __restrict__ idx_out,
                                                       int* __restrict__ n_out, RadixLds<KPT>& sh) {
  const int i = threadIdx.x;
  const int lane = i & 63;
  const int wave = __builtin_amdgcn_readfirstlane(i >> 6);
  const int n_waves = blockDim.x >> 6;
  static_assert(KPT * (kSelThreads / 64) <= 64, "the waves' counts fit one wave");
  const int k_eff = min(k, n);
  if (i == 0) *n_out = k_eff;
  for (int u = k_eff + i; u < k; u += blockDim.x) idx_out[u] = -1;
  if (k_eff == 0) return;
  uint32_t key[KPT];
  bool live[KPT];
#pragma unroll
  for (int v = 0; v < KPT; ++v) {
    live[v] = i + v * static_cast<int>(blockDim.x) < n;
    key[v] = live[v] ? orderable(score[v]) : 0u;
  }
  // Up to a wave of scores: every lane counts the keys above its own, no barrier and no LDS.  Scores and selection of one row
  // in one launch, 16 chunks 4.3 us with the rounds below, 2.9 so; 64 chunks 4.4 and 3.4.
  if (KPT == 1 && n <= 64) {
    if (wave > 0) return;
    int above = 0;                       // keys larger than this lane's
#pragma unroll
    for (int q = 0; q < 64; q += 16)
      if (q < n) {                       // lanes behind the last score hold zero, which is above nothing
#pragma unroll
        for (int j = q; j < q + 16; ++j) above += static_cast<uint32_t>(__builtin_amdgcn_readlane(key[0], j)) > key[0] ? 1 : 0;
      }
    bool take = live[0] && above < k_eff;
    const uint64_t most = __ballot(take);
    if (__popcll(most) > k_eff) {
      // the smallest keys of these are equal, and not all of them fit: the lowest-indexed ones do
      // (theirs is the largest count, found a bit at a time from the top: lane by lane, half of 64 equal scores took 4.1 us, so 2.4)
      uint64_t ties = most;
#pragma unroll
      for (int bit = 5; bit >= 0; --bit) {
        const uint64_t with = __ballot((above >> bit) & 1) & ties;
        if (with) ties = with;
      }
      const int last = __builtin_amdgcn_readlane(above, __builtin_ctzll(ties));
      if ((ties >> lane) & 1) take = __popcll(ties & ((uint64_t{1} << lane) - 1)) < k_eff - last;
    }
    const uint64_t taken = __ballot(take);
    if (take) idx_out[__popcll(taken & ((uint64_t{1} << lane) - 1))] = lane;
    return;
  }
  for (int u = i; u < 4 * 256; u += blockDim.x) (&sh.hist[0][0])[u] = 0;
  __syncthreads();
  uint32_t prefix = 0;           // the bytes of the threshold fixed so far (higher bytes first)
  int need = k_eff;              // keys still to take among those that match `prefix` in the fixed bytes
#pragma unroll
  for (int round = 0; round < 4; ++round) {
    const int shift = 24 - 8 * round;
#pragma unroll
    for (int v = 0; v < KPT; ++v) {
      const bool match = live[v] && (round == 0 || (key[v] >> (shift + 8)) == (prefix >> (shift + 8)));
      const uint64_t matching = __ballot(match);
      if (matching) {
        const int first = __ffsll(static_cast<long long>(matching)) - 1;
        const uint32_t bin = (key[v] >> shift) & 255u;
        const uint32_t first_bin = __builtin_amdgcn_readlane(bin, first);
        const uint64_t same = __ballot(match && bin == first_bin);
        if (lane == first) atomicAdd(&sh.hist[round][first_bin], __popcll(same));
        if (match && bin != first_bin) atomicAdd(&sh.hist[round][bin], 1);
      }
    }
    __syncthreads();
    // lane l looks at bins 255 - 4l (first) down to 252 - 4l; `above` = keys in higher bins
    const int4 h = *reinterpret_cast<const int4*>(&sh.hist[round][252 - 4 * lane]);
    const int bins[4] = {h.w, h.z, h.y, h.x};
    const int mine = (h.x + h.y) + (h.z + h.w);
    int above = wave_inclusive_scan(mine) - mine;
    int bin = -1, left = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (above < need && need <= above + bins[j]) {
        bin = 255 - 4 * lane - j;
        left = need - above;
      }
      above += bins[j];
    }
    // exactly one lane found the bin (1 <= need <= number of matching keys)
    const int src = __ffsll(static_cast<long long>(__ballot(bin >= 0))) - 1;
    prefix |= static_cast<uint32_t>(__builtin_amdgcn_readlane(bin, src)) << shift;
    need = __builtin_amdgcn_readlane(left, src);
  }
  // prefix is the k-th largest key; `need` of the keys equal to it are taken, lowest index first
#pragma unroll
  for (int v = 0; v < KPT; ++v) {
    const uint64_t bal_greater = __ballot(live[v] && key[v] > prefix), bal_tie = __ballot(live[v] && key[v] == prefix);
    if (lane == 0) sh.wave_counts[v * n_waves + wave] = make_int2(__popcll(bal_greater), __popcll(bal_tie));
  }
  __syncthreads();
  // lane e of every wave takes the e-th count in index order: ties before it, then outputs before it
  const int2 count = lane < KPT * n_waves ? sh.wave_counts[lane] : make_int2(0, 0);
  const int ties_before = wave_inclusive_scan(count.y) - count.y;
  const int taken = count.x + min(max(need - ties_before, 0), count.y);
  const int pos_before = wave_inclusive_scan(taken) - taken;
  const uint64_t lower = (uint64_t{1} << lane) - 1;
#pragma unroll
  for (int v = 0; v < KPT; ++v) {
    const bool is_tie = live[v] && key[v] == prefix;
    const int tie_rank = __builtin_amdgcn_readlane(ties_before, v * n_waves + wave) + __popcll(__ballot(is_tie) & lower);
    const bool take = (live[v] && key[v] > prefix) || (is_tie && tie_rank < need);
    const int pos = __builtin_amdgcn_readlane(pos_before, v * n_waves + wave) + __popcll(__ballot(take) & lower);
    if (take) idx_out[pos] = i + v * static_cast<int>(blockDim.x);
  }
}

template <int KPT>
__global__ __launch_bounds__(kSelThreads) void select_radix_kernel(const float* __restrict__ scores, int n, int k,
                                                                 int* __restrict__ idx_out, int* __restrict__ n_out) {
  __shared__ RadixLds<KPT> radix;
  float mine[KPT];
#pragma unroll
  for (int v = 0; v < KPT; ++v) {
    const int i = threadIdx.x + v * blockDim.x;
    mine[v] = i < n ? scores[i] : 0.f;
  }
  radix_select_and_write<KPT>(mine, n, k, idx_out, n_out, radix);
}

// Chunk scores of one tree row and the top-k over them in one launch (at most kRankMax
// chunks, up to 1024 threads), for problems whose pairs one compute unit takes in faster than a second launch
// costs.  Scores with the arithmetic of chunk_scores_kernel: the same bits.  scores may be null.
template <class Shape>
__global__ __launch_bounds__(kRankMax) void score_select_kernel(SPECEXT_SCORE_PARAMS, int C, int B, int L, int score_row, int k,
                                                               float* scores, int* __restrict__ idx_out, int* __restrict__ n_out) {
  __shared__ RadixLds<1> radix;
  __shared__ float partial[kRankMax][4];
  const ScoreInputs in = {in_global<const float>(part_at), in_global<const float>(lse2_at), M, G, Hq, n_sub, per_chunk};
  const int t = scored_row(in_global<const int>(path_at), in_global<const int>(count_at), T, score_row);
  const int lane = threadIdx.x % Shape::kLanes;
  for (int c = threadIdx.x / Shape::kLanes; c < C; c += blockDim.x / Shape::kLanes) {
    const float acc = chunk_partial<Shape>(in, t, c, lane);
    if constexpr (Shape::kQuads == 1) partial[c][lane] = acc;
    else if constexpr (Shape::kQuads == 64) partial[c][lane >> 6] = acc;
    else if (lane < 4) partial[c][lane] = lane == 0 ? acc : 0.f;
  }
  __syncthreads();
  const int c = threadIdx.x;
  float score[1] = {0.f};
  if (c < C) {
    score[0] = chunk_score(c, B, L, Hq, partial[c][0], partial[c][1], partial[c][2], partial[c][3]);
    if (scores) scores[c] = score[0];
  }
  radix_select_and_write<1>(score, C, k, idx_out, n_out, radix);
}

// --------------------------------------------------------------------------
// draft-KV gather
// --------------------------------------------------------------------------

__device__ __forceinline__ int chunk_tokens(int c, int n_chunks, int src_len, int chunk_size) {
  if (c < 0 || c >= n_chunks) return 0;
  return min(chunk_size, src_len - c * chunk_size);
}

// grid (max_idx, n_layers * n_heads, 2): one workgroup copies one chunk of one
// (layer, head) of K (z = 0) or V (z = 1), 16 bytes per thread, kGatherAtOnce of them in flight.  The workgroups
// of (layer, head) 0 of K also do the bookkeeping: each writes the original positions of
// its chunk's tokens, and the one of list entry 0 the total and the -1 behind it.
//
// What bounds it: the launch and two trips to memory, the list and then the rows.  So the list's length, the workgroup's
// entry and the first 64 entries are requested together, and every wave adds up the tokens ahead for itself; with the three
// behind one another and a workgroup-wide sum, 32 chunks of 32 tokens of 8 heads (4 MB of cold bf16 rows) took 4.7 us, this 4.2;
// of 32 heads 7.2 and 6.6; four chunks of one fp32 head 2.8 and 2.5.  Behind more than kGatherAlone entries the waves share
// the sum: each for itself, 256 chunks took 9.85 us as shared, but 1024 chunks of 16 tokens of 8 heads 39 instead of 32 us, 4096 of
// 4 tokens of 2 heads 53 instead of 27.
constexpr int kGatherAtOnce = 4;
constexpr int kGatherThreads = 256;
constexpr int kGatherAlone = 256;
__global__ __launch_bounds__(kGatherThreads) void gather_copy_kernel(const int* __restrict__ idx, const int* __restrict__ n_idx, int max_idx,
                                                         int src_len, int chunk_size, int row_vecs, int src_cap, int dst_cap,
                                                         const uint4* __restrict__ k_src, const uint4* __restrict__ v_src,
                                                         uint4* __restrict__ k_dst, uint4* __restrict__ v_dst,
                                                         int* __restrict__ pos_out, int* __restrict__ len_out) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x;
  int c = idx[r], first = idx[min(lane, max_idx - 1)];
  int n_used = n_idx ? *n_idx : max_idx;
  asm volatile("" : "+s"(c), "+v"(first), "+s"(n_used));        // all three requested before the first is waited for
  n_used = min(max(n_used, 0), max_idx);
  const int n_chunks = (src_len + chunk_size - 1) / chunk_size;
  // tokens of the first `end` list entries (the same `end` in the whole workgroup)
  __shared__ int wave_tokens[kGatherThreads / 64];
  auto tokens_of = [&](int end) {
    if (__builtin_expect(end > kGatherAlone, 0)) {
      int part = 0;
      for (int i = threadIdx.x; i < end; i += kGatherThreads) part += chunk_tokens(idx[i], n_chunks, src_len, chunk_size);
      part = __builtin_amdgcn_readlane(wave_inclusive_scan(part), 63);
      __syncthreads();                 // the sum before has been read
      if (lane == 0) wave_tokens[threadIdx.x >> 6] = part;
      __syncthreads();
      int total = 0;
      for (int w = 0; w < kGatherThreads / 64; ++w) total += wave_tokens[w];
      return total;
    }
    int part = lane < end ? chunk_tokens(first, n_chunks, src_len, chunk_size) : 0;
    for (int i = 64 + lane; i < end; i += 64) part += chunk_tokens(idx[i], n_chunks, src_len, chunk_size);
    return __builtin_amdgcn_readlane(wave_inclusive_scan(part), 63);
  };
  const bool book = blockIdx.y == 0 && blockIdx.z == 0 && (pos_out || len_out);
  if (book && r == 0) {
    const int total = tokens_of(n_used);
    if (pos_out)
      for (int i = total + threadIdx.x; i < dst_cap; i += kGatherThreads) pos_out[i] = -1;
    if (len_out && threadIdx.x == 0) *len_out = total;
  }
  if (r >= n_used) return;
  const int tokens = chunk_tokens(c, n_chunks, src_len, chunk_size);
  if (tokens == 0) return;
  const int dst_tok = tokens_of(r);              // tokens of all earlier list entries

  const int64_t lh = blockIdx.y;
  const uint4* src = (blockIdx.z == 0 ? k_src : v_src) + (lh * src_cap + static_cast<int64_t>(c) * chunk_size) * row_vecs;
  uint4* dst = (blockIdx.z == 0 ? k_dst : v_dst) + (lh * dst_cap + dst_tok) * row_vecs;
  const int n_vecs = tokens * row_vecs;
  for (int i0 = threadIdx.x; i0 < n_vecs; i0 += kGatherAtOnce * kGatherThreads) {
    uint4 v[kGatherAtOnce];
#pragma unroll
    for (int u = 0; u < kGatherAtOnce; ++u) v[u] = src[min(i0 + u * kGatherThreads, n_vecs - 1)];      // past the end: the last one again, unused
#pragma unroll
    for (int u = 0; u < kGatherAtOnce; ++u)
      if (i0 + u * kGatherThreads < n_vecs) dst[i0 + u * kGatherThreads] = v[u];
  }
  if (book && pos_out)
    for (int tk = threadIdx.x; tk < tokens; tk += kGatherThreads) pos_out[dst_tok + tk] = c * chunk_size + tk;
}

// The bookkeeping alone (an empty list or no (layer, head) to copy): original positions of
// the kept tokens, -1 behind them, and the total.  One workgroup; entry r of the list is
// handled by thread r (lists longer than the block go round by round, carrying the
// running offset), offsets come from a block scan.
__global__ __launch_bounds__(256) void gather_meta_kernel(const int* __restrict__ idx, const int* __restrict__ n_idx,
                                                         int max_idx, int src_len, int dst_cap, int chunk_size,
                                                         int* __restrict__ pos_out, int* __restrict__ len_out) {
  __shared__ int wave_sums[4];
  const int n_used = n_idx ? min(max(*n_idx, 0), max_idx) : max_idx;
  const int n_chunks = (src_len + chunk_size - 1) / chunk_size;
  int base = 0;
  for (int r0 = 0; r0 < n_used; r0 += blockDim.x) {
    const int r = r0 + threadIdx.x;
    int c = -1, tokens = 0;
    if (r < n_used) {
      c = idx[r];
      tokens = chunk_tokens(c, n_chunks, src_len, chunk_size);
    }
    int total;
    const int off = base + block_exclusive_scan(tokens, wave_sums, total);
    if (pos_out)
      for (int tk = 0; tk < tokens; ++tk) pos_out[off + tk] = c * chunk_size + tk;
    base += total;
  }
  if (pos_out)
    for (int i = base + threadIdx.x; i < dst_cap; i += blockDim.x) pos_out[i] = -1;
  if (len_out && threadIdx.x == 0) *len_out = base;
}

}  // namespace

// (The launchers stand in this order so that the compiler places the code of the kernels that follow one another in a step
// - scores, selection, gather - side by side: with the score kernels of long chunks between them the selection took 0.3 us more.)
hipError_t launch_select_chunks(const float* scores, int32_t n_chunks, int32_t k, int32_t* idx_out,
                                int32_t* n_out, hipStream_t stream) {
  // a small input needs only as many waves as it has scores (fewer waves, cheaper barriers)
  const int threads = n_chunks >= kSelThreads ? kSelThreads : ((n_chunks + 63) / 64) * 64;
  const auto kernel = n_chunks <= kRankMax ? select_radix_kernel<1> : n_chunks <= kRadixMax ? select_radix_kernel<4> : select_kernel;
  return launch_kernel(kernel, dim3(1), dim3(threads), 0, stream, scores, n_chunks, k, idx_out, n_out);
}

hipError_t launch_chunk_scores(const AttnParams& p, int32_t score_row, const int32_t* row_path,
                               const int32_t* row_count, float* scores, hipStream_t stream) {
  const int rows = (score_row < 0 && !row_path) ? p.T : 1;
  const int first = score_row < 0 ? 0 : score_row;
  hipError_t e = hipErrorInvalidValue;
  with_score_shape(p.B / p.score_gran, [&](auto shape) {
    using Shape = decltype(shape);
    const dim3 grid((p.C + Shape::kChunks - 1) / Shape::kChunks, rows), block(Shape::kThreads);
    e = launch_kernel(chunk_scores_kernel<Shape>, grid, block, 0, stream, SPECEXT_SCORE_ARGS(p), p.C, p.B, p.L, first, scores);
  });
  return e;
}

hipError_t launch_score_select(const AttnParams& p, int32_t score_row, const int32_t* row_path,
                               const int32_t* row_count, int32_t k, float* scores, int32_t* idx_out, int32_t* n_out,
                               hipStream_t stream) {
  if (p.C > kRankMax) return hipErrorInvalidValue;
  // One compute unit takes in the pair groups (KV heads x score blocks) at some 600 per us; from 1600 on, and from 128 chunks
  // on, where the selection takes sixteen waves, a launch of its own for the scores, which every compute unit shares, is the
  // shorter way.  Measured with the pairs as the attention left them, us in one launch / in two; whole iterations of one
  // layer, then of two, launched from Python (the two in turn in one process):
  //   8 heads, 32-key chunks   100 chunks 28.3 / 29.0, 41.7 / 42.4;  128 28.8 / 29.6, 43.2 / 43.7;  160 31.5 / 31.1, 47.3 / 46.8
  //   8 heads, 64-key chunks   80 (1280 groups) 32.1 / 32.2, 47.5 / 48.3;  100 (1600) 33.1 / 33.3, 50.3 / 50.3;  113 (1800) 34.9 / 34.6
  //   32 heads, 32-key chunks  41 (1312) 28.9 / 29.4, 42.1 / 42.8;  50 (1600) 30.3 / 30.5, 44.1 / 44.3;  64 (2048) 31.2 / 30.8, 45.6 / 45.1
  // and the selection alone in a captured graph: 8 heads 1280 groups 5.8 / 6.2, 1600 6.1 / 6.4, 2048 6.4 / 6.2, 2944 6.2 / 5.1; 2 heads
  // 129 chunks 5.6 / 5.2, 256 6.5 / 5.5 (with one or two heads and 129 to 192 chunks the iteration is bounded by the host and
  // equal to 0.3 us either way, with a slow host up to 1 - 2 us longer in two).
  if (scores && (p.C > kScoreChunksOneLaunch || static_cast<int64_t>(p.Hkv) * p.n_sub > kScoreGroupsOneLaunch)) {
    const hipError_t e = launch_chunk_scores(p, score_row, row_path, row_count, scores, stream);
    return e != hipSuccess ? e : launch_select_chunks(scores, p.C, k, idx_out, n_out, stream);
  }
  // at least one thread per chunk (selection), four or more for the scores as far as 1024 go
  hipError_t e = hipErrorInvalidValue;
  with_score_shape(p.B / p.score_gran, [&](auto shape) {
    using Shape = decltype(shape);
    const int threads = Shape::kQuads > 1 ? 1024 : p.C <= 64 ? 256 : p.C <= 128 ? 512 : 1024;
    e = launch_kernel(score_select_kernel<Shape>, dim3(1), dim3(threads), 0, stream, SPECEXT_SCORE_ARGS(p), p.C, p.B, p.L, score_row, k,
                      scores, idx_out, n_out);
  });
  return e;
}

hipError_t launch_gather(const void* k_src, const void* v_src, void* k_dst, void* v_dst,
                         const int32_t* idx, const int32_t* n_idx, int32_t max_idx, int32_t n_lh,
                         int32_t src_len, int32_t src_cap, int32_t dst_cap, int32_t row_bytes,
                         int32_t chunk_size, int32_t* pos_out, int32_t* len_out, hipStream_t stream) {
  if (max_idx > 0 && n_lh > 0) {
    dim3 grid(max_idx, n_lh, 2);
    return launch_kernel(gather_copy_kernel, grid, dim3(kGatherThreads), 0, stream, idx, n_idx, max_idx, src_len, chunk_size, row_bytes / 16,
                         src_cap, dst_cap, static_cast<const uint4*>(k_src), static_cast<const uint4*>(v_src),
                         static_cast<uint4*>(k_dst), static_cast<uint4*>(v_dst), pos_out, len_out);
  }
  if (pos_out || len_out) {
    return launch_kernel(gather_meta_kernel, dim3(1), dim3(256), 0, stream, idx, n_idx, max_idx, src_len, dst_cap, chunk_size, pos_out,
                         len_out);
  }
  return hipSuccess;
}

}  // namespace specext
