// Prefix pass of Hybrid Tree Attention (SpecExtend Sec. 3.1) on the gfx950 matrix cores with
// fp32 probabilities: fp32 inputs, and the bf16 problems that the two bf16 kernels do not take
// (chunk sizes that are no multiple of 32, prefixes shorter than their key tile, head_dim 64
// with strided keys), which keep the fp32 arithmetic they always had.
//
// What bounds it.  With fp32 inputs both products run on v_mfma_f32_16x16x4_f32, 256 flop per
// clock and compute unit (157 TFLOP/s, 1/16 of the bf16 rate): a tree of 60 nodes with four
// heads per group is matrix-bound (0.12 us of K/V traffic per us of matrix work), everything
// else - softmax, LDS reads, loads - fits beside it.  One thread per query row on the vector
// ALUs, which this replaces, left three of a compute unit's four SIMDs idle and read every K/V
// element from LDS once per row: 3370 us at fp32, 2K tokens, 32/8 heads, 60 nodes; here 24.5 us
// (13.6 us of matrix instructions at 2.4 GHz; the rest is the way to the first tile, 2 us, the
// workgroup's own merge and stores, 3 us, and the loop's other instructions: products of fp32 run on
// the vector multipliers, so while one wave of a SIMD issues them the other's vector instructions
// wait).
// With bf16 inputs Q K^T is exact in bf16 products, and the probabilities go into P V as three
// bf16 terms whose sum is the fp32 value (8 + 8 + 8 mantissa bits), so that nothing is rounded
// and the product runs at a third of the bf16 rate instead of the fp32 one's sixteenth (4109
// keys, 60 nodes: 6250 us before, 16.0 us here).
// The range is that of plain fp32 attention but for |V| near its end (the lagging reference lets
// P reach 2^10: an exact running maximum takes 25.4 instead of 24.4 us at 2K and 77.3 instead of
// 73.0 at 8K): infinite V, logits of minus infinity, of any finite size and scales of any size
// are answered, for which the queries are scaled in the prologue.
//
// Shape.  A workgroup owns 16 * NSUB * RB query rows of one KV head and one split of the keys.
// Its waves form RB row groups x KG key groups: the key groups take the split's tiles in turns
// and are merged through LDS at the end, so that few rows (a draft level, a toy) still keep four
// SIMDs busy and the split count - the partial outputs that cross memory - stays low.
//   tile    one key group's step: 16 keys (fp32) or 32 keys (bf16), the same bytes
//   stage   KG tiles, one workgroup barrier; the ring in LDS holds 128 KB of stages (two of
//           64 KB, four for head_dim 64), requested ahead by direct global->LDS loads.  A compute
//           unit takes in 64 bytes per clock: issuing a stage keeps its waves for 1000 cycles
//           when all do it at once, so the upper half of a workgroup of eight waves begins a
//           stage with the products that it still has to do (bf16 8K 22.6 -> 21.1 us per launch).
// Workgroups of 128 rows with two key groups (half as many reads of every key, twice the partial
// outputs) measured slower in an earlier form of this kernel, under the profiler: 32 against 29 us
// (fp32, 2K), 20.0 against 18.7 us (bf16, 4109).
// Matrix-core mapping, transposed so that a lane owns one query row (l & 15) in both products:
//   S^T[key][row]   = K Q^T     A = K rows from LDS, B = Q in registers.  The contraction index
//                               is permuted alike on both sides: a lane quarter (l >> 4) takes
//                               the 16-byte pieces 4 j + quarter of a row.
//   O^T[dcol][row] += V^T P^T   B = P^T straight from the S^T accumulators (lane quarter q holds
//                               keys 4 q .. 4 q + 3), A = V.  fp32: one 16-byte read per key gives
//                               four consecutive columns, each the operand of its own product.
//                               bf16: ds_read_b64_tr_b16 as in the other kernels.
#include "mfma_util.h"

namespace specext {
namespace {

constexpr int KG = 4;                             // key groups of a workgroup
constexpr int kRingBytes = 128 * 1024;

template <int D, bool BF16>
struct Tile {
  static constexpr int kElem = BF16 ? 2 : 4;
  static constexpr int kKeys = BF16 ? 32 : 16;
  static constexpr int kRowBytes = D * kElem;              // 128, 256 or 512
  static constexpr int kPieces = kRowBytes / 16;           // 16-byte pieces of a row
  static constexpr int kBytes = kKeys * kRowBytes;         // 8 KB (D = 128) or 4 KB
  static constexpr int kLoads = kBytes / 1024;             // direct loads of one wave per K or V tile
  static constexpr int kRowsPerLoad = 1024 / kRowBytes;
  // 16-byte piece `c` of row `r` sits at piece c ^ k_swz(r) (K) or c ^ v_swz(r) (V) of its LDS row, so that the
  // operand reads spread over the banks: 16 rows x one piece for K; for a bf16 V 8 rows x 32 bytes (an fp32 V row is
  // read 256 consecutive bytes at a time and needs none)
  // (k_swz repeats after 16 rows, v_swz after eight, which is so many loads)
  static constexpr int kKPeriod = 16 / kRowsPerLoad;
  static constexpr int kVPeriod = BF16 ? 8 / kRowsPerLoad : 1;
  static __device__ __forceinline__ int k_swz(int r) { return kRowBytes == 128 ? (r >> 1) & 7 : r & 15; }
  static __device__ __forceinline__ int v_swz(int r) {
    return !BF16 ? 0 : kRowBytes == 128 ? ((r >> 1) & 3) << 1 : (r & 7) << 1;
  }
};

// The exponent is one fused multiply-add, logit * c - reference, with the reference the rounded product for the row's largest
// logit: the rounding is left in every exponent alike, up to 2^-24 of the reference, and cancels in the row's sum.  From
// references of 2^24 on it could no longer be left in; there the product is rounded before the subtraction, as it was for the
// reference, and the largest logit's exponent is zero again.
constexpr float kFarLog2 = 16777216.f;

constexpr int stages_of(int stage_bytes) { return kRingBytes / stage_bytes < 4 ? kRingBytes / stage_bytes : 4; }

// value + the value of the lane 16 away (within a pair of 16-lane rows)
__device__ __forceinline__ float rows16_sum(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float rows16_max(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int D, bool BF16, int NSUB, int RB, int SCORES>
__global__ __launch_bounds__(RB * KG * 64) void prefix_f32_kernel(uint64_t k_at, uint64_t v_at, uint64_t q_at, int64_t kp_sh, int L, int keys_per_split, int M, int G,
                                                            int kp_sl, int head_fastest, AttnParams p) {
  p.kp = in_global<const void>(k_at);
  p.vp = in_global<const void>(v_at);
  p.q = in_global<const void>(q_at);
  p.kp_sh = kp_sh, p.L = L, p.keys_per_split = keys_per_split, p.M = M, p.G = G, p.kp_sl = kp_sl, p.head_fastest = head_fastest;
  using T = Tile<D, BF16>;
  constexpr int kStageBytes = KG * 2 * T::kBytes;
  constexpr int kStages = stages_of(kStageBytes);
  constexpr int kSlotBytes = 2 * T::kBytes;                // one key group's place for a stage: K tile, V tile
  constexpr int kGroupBytes = kStages * kSlotBytes;        // its ring; the key groups' rings stand side by side
  constexpr int kTileLoads = T::kLoads / RB;               // direct loads of one wave per K or V tile
  constexpr int kLoadsPerStage = 2 * kTileLoads;
  // The first stage's V tiles, requested behind its K tiles, are waited for behind the first products only.  fp32 with 512-byte
  // rows, whose products take long enough: 8 nodes of 4 heads, 1000 keys 6.26 -> 5.8 us, 80 rows at 2K 11.15 -> 10.3; the
  // others are 0.1 - 0.3 us faster without the second barrier.
  constexpr bool kSplitV = !BF16 && D == 128;
  constexpr int kSubTiles = T::kKeys / 16;                 // S^T blocks of 16 keys per tile
  constexpr int kQRegs = BF16 ? D / 32 : D / 16;           // 16-byte pieces of a query row per lane
  constexpr int kOBlocks = D / 16;                         // 16 x 16 output blocks per 16 rows
  constexpr int kRows = 16 * NSUB;                         // query rows of a wave
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb = wave % RB;                                // row group
  const int kg = wave / RB;                                // key group
  const int li = lane & 15;
  const int qt = lane >> 4;                                // lane quarter

  const int split = p.head_fastest ? blockIdx.y : blockIdx.x;
  const int g = p.head_fastest ? blockIdx.x : blockIdx.y;
  const int row0 = (blockIdx.z * RB + rb) * kRows;
  const int key_lo = split * p.keys_per_split;
  const int key_hi = min(p.L, key_lo + p.keys_per_split);
  const int n_tiles = (key_hi - key_lo + T::kKeys - 1) / T::kKeys;
  const int n_stages = (n_tiles + KG - 1) / KG;
  const int my_tiles = (n_tiles - kg + KG - 1) / KG;       // tiles of this key group: one in each of the first stages

  const int64_t key_bytes = p.kp_sl * T::kElem;
  const unsigned char* kbase = static_cast<const unsigned char*>(p.kp) + static_cast<int64_t>(g) * p.kp_sh * T::kElem;
  const unsigned char* vbase = static_cast<const unsigned char*>(p.vp) + static_cast<int64_t>(g) * p.kp_sh * T::kElem;
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((lds_void*)lds));
  const int ld_row = lane / T::kPieces;                    // row within one load
  const int ld_piece = lane % T::kPieces;

  // The loads of a stage, which is requested in order.  A whole tile's take a lane's offset within the tile, which stays the same,
  // and a uniform base that moves on: no vector instructions, which would stand still while the other wave of the SIMD issues
  // fp32 products (those run on the vector multipliers).  Keys past the split's end repeat its last one (masked below).
  constexpr int kKOffs = T::kKPeriod > RB ? (kTileLoads < T::kKPeriod / RB ? kTileLoads : T::kKPeriod / RB) : 1;
  constexpr int kVOffs = T::kVPeriod > RB ? T::kVPeriod / RB : 1;
  const unsigned row_off = static_cast<unsigned>(ld_row) * static_cast<unsigned>(key_bytes);
  unsigned k_off[kKOffs], v_off[kVOffs];
#pragma unroll
  for (int i = 0; i < kKOffs; ++i) k_off[i] = row_off + ((ld_piece ^ T::k_swz((rb + i * RB) * T::kRowsPerLoad + ld_row)) << 4);
#pragma unroll
  for (int i = 0; i < kVOffs; ++i) v_off[i] = row_off + ((ld_piece ^ T::v_swz((rb + i * RB) * T::kRowsPerLoad + ld_row)) << 4);
  const int64_t first_off = (static_cast<int64_t>(key_lo) + kg * T::kKeys + rb * T::kRowsPerLoad) * key_bytes;
  const unsigned char *k_next = kbase + first_off, *v_next = vbase + first_off;
  const int64_t load_step = RB * T::kRowsPerLoad * key_bytes, stage_step = KG * T::kKeys * key_bytes;
  const int whole_tiles = ((key_hi - key_lo) / T::kKeys - kg + KG - 1) / KG;       // of this key group
  const unsigned group_lds = lds0 + kg * kGroupBytes;
  auto issue_stage = [&](auto slot_c, int st) __attribute__((always_inline)) {
    if (st >= my_tiles) return;
    const unsigned dst = group_lds + decltype(slot_c)::value * kSlotBytes + rb * 1024;
    if (__builtin_expect(st < whole_tiles, 1)) {
      const unsigned char *ksrc = k_next, *vsrc = v_next;
#pragma unroll
      for (int i = 0; i < kTileLoads; ++i) {
        load_to_lds_16(dst + i * RB * 1024, k_off[i % kKOffs], ksrc);
        ksrc += load_step;
      }
#pragma unroll
      for (int i = 0; i < kTileLoads; ++i) {
        load_to_lds_16(dst + T::kBytes + i * RB * 1024, v_off[i % kVOffs], vsrc);
        vsrc += load_step;
      }
      k_next += stage_step;
      v_next += stage_step;
    } else {
      const int key0 = key_lo + (st * KG + kg) * T::kKeys;
      const int last = key_hi - 1 - key0;
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const unsigned char* src = (v ? vbase : kbase) + key0 * key_bytes;
#pragma unroll
        for (int i = 0; i < kTileLoads; ++i) {
          const int r = (rb + i * RB) * T::kRowsPerLoad + ld_row;
          const unsigned off = static_cast<unsigned>(min(r, last)) * static_cast<unsigned>(key_bytes);
          load_to_lds_16(dst + v * T::kBytes + i * RB * 1024, off + ((ld_piece ^ (v ? T::v_swz(r) : T::k_swz(r))) << 4), src);
        }
      }
    }
  };

  // Queries (B operand of S^T) go through LDS, too, each row group's rows loaded once for all key groups, into the place of the
  // last stage of the ring, which is requested when they have left it.  (Loaded into registers by every wave for itself they
  // were four times the bytes, and the compiler, which counts only such loads, waited for the first stage behind them before
  // their scaling.)  Rows past the last one repeat it and are never stored.
  constexpr int kQLoads = kRows * T::kRowBytes / 1024;     // of a row group
  static_assert(kRows * T::kRowBytes <= kSlotBytes && RB <= KG, "a row group's queries fit one key group's slot");
  constexpr int kQSlot = kStages - 1;
  const unsigned q_lds = lds0 + rb * kGroupBytes + kQSlot * kSlotBytes;
#pragma unroll
  for (int i = 0; i < (kQLoads + KG - 1) / KG; ++i) {
    const int u = kg + i * KG;
    if (u < kQLoads) {
      const int r = u * T::kRowsPerLoad + ld_row;
      const int m = min(row0 + r, p.M - 1);
      const int t = static_cast<int>((static_cast<float>(m) + 0.5f) * (1.0f / static_cast<float>(p.G)));      // m / G, exact for m < 2^20
      const int h = g * p.G + (m - t * p.G);
      load_to_lds_16_at(q_lds + u * 1024, static_cast<const unsigned char*>(p.q) + (t * p.q_st + h * p.q_sh) * T::kElem + ((ld_piece ^ T::k_swz(r)) << 4));
    }
  }
  static_for<0, kStages - 1>([&](auto st_c) { issue_stage(st_c, decltype(st_c)::value); });
  const int ahead = min(my_tiles, kStages - 1);            // stages requested so far

  // Operand reads take these as LDS addresses plus immediates (again no vector instructions in a stage), pinned in registers so
  // that the compiler does not rebuild them.  K (and query) piece 4 j + quarter of row 16 u + li: from j = 4 on 256 bytes further.
  constexpr int kKAddrs = kQRegs < 4 ? kQRegs : 4;
  unsigned kq_off[kKAddrs], k_addr[kKAddrs];
#pragma unroll
  for (int j = 0; j < kKAddrs; ++j) {
    kq_off[j] = li * T::kRowBytes + (((4 * j + qt) ^ T::k_swz(li)) << 4);
    k_addr[j] = group_lds + kq_off[j];
    asm volatile("" : "+v"(k_addr[j]));
  }
  // V: fp32 key 4 quarter + i, 16 bytes of a 64-column block; bf16 transposing reads of keys 16 u + 4 quarter ..
  constexpr int kVAddrs = BF16 ? kOBlocks : 1;
  unsigned v_addr[kVAddrs];
#pragma unroll
  for (int b = 0; b < kVAddrs; ++b) {
    if constexpr (BF16) {
      const int r = 4 * qt + (li >> 2);
      v_addr[b] = group_lds + T::kBytes + r * T::kRowBytes + (((2 * b + ((li & 3) >> 1)) ^ T::v_swz(r)) << 4) + ((li & 1) << 3);
    } else {
      v_addr[b] = group_lds + T::kBytes + 4 * qt * T::kRowBytes + (li << 4);
    }
    asm volatile("" : "+v"(v_addr[b]));
  }
  auto lds_read = [&](unsigned addr) { return *reinterpret_cast<const lds_uintx4*>(static_cast<uintptr_t>(addr)); };

  // The scale's power of two goes into the queries (exact), so that a logit that is finite scaled is finite as the product
  // leaves it: 1 / sqrt(d) and the factor of base 2 make it a sixth to an eighth.
  const int scale_exp = max(-16, min(0, static_cast<int>(__float_as_uint(p.scale_log2) >> 23) - 127));
  const float q_scale = __uint_as_float(static_cast<uint32_t>(127 + scale_exp) << 23);
  uintx4 qf[NSUB][kQRegs];
  wait_vmcnt_even(kLoadsPerStage * ahead);                 // this wave's query rows have landed
  lds_barrier();
#pragma unroll
  for (int s = 0; s < NSUB; ++s)
#pragma unroll
    for (int j = 0; j < kQRegs; ++j) qf[s][j] = lds_read(q_lds + kq_off[j % kKAddrs] + 16 * s * T::kRowBytes + 256 * (j / kKAddrs));
#pragma unroll
  for (int s = 0; s < NSUB; ++s)
#pragma unroll
    for (int j = 0; j < kQRegs; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t w = qf[s][j][e];
        if constexpr (BF16)
          qf[s][j][e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{__uint_as_float(w << 16) * q_scale,
                                                                                     __uint_as_float(w & 0xffff0000u) * q_scale}, bf16x2));
        else
          qf[s][j][e] = __float_as_uint(__uint_as_float(w) * q_scale);
      }

  floatx4 acc[NSUB][kOBlocks];
#pragma unroll
  for (int s = 0; s < NSUB; ++s)
#pragma unroll
    for (int b = 0; b < kOBlocks; ++b) acc[s][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  float ref[NSUB], run_sum[NSUB];      // reference (scaled logit, base 2) the exponentials are taken against; lane-partial sum
#pragma unroll
  for (int s = 0; s < NSUB; ++s) {
    ref[s] = -INFINITY;
    run_sum[s] = 0.f;
  }
  const float c = p.scale_log2 * __uint_as_float(static_cast<uint32_t>(127 - scale_exp) << 23);      // what is left of the scale
  const int gran_log2 = __builtin_ctz(p.score_gran);
  // of block 0 and this lane's first row
  float* score_row = SCORES == 2 ? p.chunk_part + (static_cast<int64_t>(g) * p.n_sub * p.M + row0 + li) * 2 : nullptr;
  bool far = false;                    // some reference of this wave is beyond kFarLog2

  // A tile in three parts: the logits (and the V fragments: all that reads the ring), the softmax, the second product (from
  // registers).  With every wave in the same order both waves of a SIMD would be in their softmax at the same time and the
  // matrix pipe idle; so the upper half of a workgroup of eight waves (wave w + 4 shares wave w's SIMD) starts a stage with
  // the second product of the tile before (bf16 inputs, 4109 keys: 16.1 instead of 17.1 us, 8K 23.3 instead of 25.2; fp32 inputs, 2K:
  // 24.4 instead of 24.8).
  floatx4 s_acc[NSUB][kSubTiles];      // the tile's logits, then its probabilities
  float score_part[NSUB][kSubTiles];   // a lane's sums of them
  uintx4 pf[NSUB][3];                  // bf16 inputs: the probabilities as three terms
  uintx4 vf[kOBlocks];                 // fp32: [key i of the quarter][64-column block]; bf16: [16-column block]
  auto tile_logits = [&](auto slot_c, int st) __attribute__((always_inline)) {
    constexpr unsigned slot = decltype(slot_c)::value * kSlotBytes;
    // all K fragments of the tile are requested before the first product (one at a time, every product would wait for
    // its own LDS read)
    uintx4 kf[kSubTiles][kQRegs];
#pragma unroll
    for (int u = 0; u < kSubTiles; ++u)
#pragma unroll
      for (int j = 0; j < kQRegs; ++j) kf[u][j] = lds_read(k_addr[j % kKAddrs] + (slot + 16 * u * T::kRowBytes + 256 * (j / kKAddrs)));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kSubTiles; ++u) {
#pragma unroll
      for (int s = 0; s < NSUB; ++s) s_acc[s][u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < kQRegs; ++j) {
        if constexpr (BF16) {
#pragma unroll
          for (int s = 0; s < NSUB; ++s)
            s_acc[s][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[u][j]),
                                                                  __builtin_bit_cast(bf16x8, qf[s][j]), s_acc[s][u], 0, 0, 0);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int s = 0; s < NSUB; ++s) {
              const uint32_t kb = kf[u][j][e], qb = qf[s][j][e];
              s_acc[s][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(kb), __uint_as_float(qb), s_acc[s][u], 0, 0, 0);
            }
        }
      }
    }
    if (kSplitV && st == 0) {
      __builtin_amdgcn_sched_barrier(0);
      wait_vmcnt_even(kLoadsPerStage * max(0, min(my_tiles, kStages) - 1));
      lds_barrier();
    }
    // and the V fragments before the softmax, which hides their reads
#pragma unroll
    for (int b = 0; b < kOBlocks; ++b) {
      if constexpr (BF16) {
        shortx4 half[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
          half[u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)static_cast<uintptr_t>(v_addr[b] + (slot + 16 * u * T::kRowBytes)));
        vf[b] = __builtin_bit_cast(uintx4, __builtin_shufflevector(half[0], half[1], 0, 1, 2, 3, 4, 5, 6, 7));
      } else {
        vf[b] = lds_read(v_addr[0] + (slot + b / (D / 64) * T::kRowBytes + 256 * (b % (D / 64))));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // A product's result may be read ten wait states after its issue at the earliest.  The compiler counts them, but where
    // the branch below follows the last product directly it counts along the branch's long side only and reads too early
    // on the short one (seen in its output: two states, and the register's previous content in the row maximum), so the
    // states are spelled out here.
#pragma unroll
    for (int s = 0; s < NSUB; ++s)
#pragma unroll
      for (int u = 0; u < kSubTiles; ++u) asm volatile("" : "+v"(s_acc[s][u]));
    asm volatile("s_nop 9");
  };
  auto tile_softmax = [&](int st) __attribute__((always_inline)) {
    // online softmax; lane quarter qt holds keys 16 u + 4 qt + i of the tile
    const int key0 = key_lo + (st * KG + kg) * T::kKeys;
    const int left = key_hi - key0;
    if (__builtin_expect(left < T::kKeys, 0)) {
#pragma unroll
      for (int u = 0; u < kSubTiles; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (16 * u + 4 * qt + i >= left) {
#pragma unroll
            for (int s = 0; s < NSUB; ++s) s_acc[s][u][i] = -INFINITY;
          }
    }
    float mx[NSUB];
    bool grow = false;
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      mx[s] = -INFINITY;
#pragma unroll
      for (int u = 0; u < kSubTiles; ++u)
        mx[s] = fmaxf(mx[s], fmaxf(fmaxf(s_acc[s][u][0], s_acc[s][u][1]), fmaxf(s_acc[s][u][2], s_acc[s][u][3])));
      mx[s] *= c;
      grow |= mx[s] > ref[s] + kLazyLog2;
    }
    if (__builtin_expect(__any(grow), 0)) {                 // some row of this wave outgrew its reference: move every reference up
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        const float new_ref = fmaxf(ref[s], halves_max(rows16_max(mx[s])));
        // 0 on the first tile; a row may have seen nothing but logits of minus infinity yet
        const float alpha = new_ref > -INFINITY ? fast_exp2(ref[s] - new_ref) : 1.f;
        ref[s] = new_ref;
        run_sum[s] *= alpha;
#pragma unroll
        for (int b = 0; b < kOBlocks; ++b) acc[s][b] *= alpha;
        far |= __any(new_ref > kFarLog2 || (new_ref < -kFarLog2 && new_ref > -INFINITY));
      }
    }
    float base[NSUB];
#pragma unroll
    for (int s = 0; s < NSUB; ++s) base[s] = ref[s] > -INFINITY ? ref[s] : 0.f;
    if (__builtin_expect(far, 0)) {
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int u = 0; u < kSubTiles; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float scaled = s_acc[s][u][i] * c;
            asm volatile("" : "+v"(scaled));               // rounded before the subtraction
            s_acc[s][u][i] = scaled - base[s];
          }
    } else {
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int u = 0; u < kSubTiles; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) s_acc[s][u][i] = fmaf(s_acc[s][u][i], c, -base[s]);
    }
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
#pragma unroll
      for (int u = 0; u < kSubTiles; ++u) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s_acc[s][u][i] = fast_exp2(s_acc[s][u][i]);
        const float part = (s_acc[s][u][0] + s_acc[s][u][1]) + (s_acc[s][u][2] + s_acc[s][u][3]);
        run_sum[s] += part;
        if (SCORES) score_part[s][u] = part;
      }
    }
    if constexpr (BF16) {
      // P as three bf16 terms, each the leading eight bits of what is just below the rest: their sum is P exactly and none is
      // zero or negative while P is not zero, so an infinite V gives that infinity as in one product.
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          float x0 = s_acc[s][e >> 2][e & 3], x1 = s_acc[s][e >> 2][(e & 3) + 1];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const uint32_t b0 = k < 2 ? __builtin_elementwise_sub_sat(__float_as_uint(x0), 1u) : __float_as_uint(x0);
            const uint32_t b1 = k < 2 ? __builtin_elementwise_sub_sat(__float_as_uint(x1), 1u) : __float_as_uint(x1);
            pf[s][k][e / 2] = __builtin_amdgcn_perm(b1, b0, 0x07060302);          // the upper halves
            x0 -= __uint_as_float(b0 & 0xffff0000u);
            x1 -= __uint_as_float(b1 & 0xffff0000u);
          }
        }
    }
  };
  // The (sum, reference) pairs of the score blocks of the tile that the softmax was last done for, in stage st.  The upper waves
  // end a stage with their softmax, which nothing overlaps, so they store behind the second product that follows (fp32 4K 41.3
  // -> 40.5 us, bf16 4109 keys 16.3 -> 16.0; the lower ones doing so as well: 24.5 -> 24.7 us at fp32 2K, 16.0 -> 16.1).
  auto store_scores = [&](int st) __attribute__((always_inline)) {
    const int key0 = key_lo + (st * KG + kg) * T::kKeys;
    const int left = key_hi - key0;
#pragma unroll
    for (int s = 0; s < NSUB; ++s)
#pragma unroll
      for (int u = 0; u < kSubTiles; ++u) {
        float part = score_part[s][u];
        if constexpr (SCORES == 2) {
          // blocks of 16 keys, the usual case: no choices
          part = halves_sum(rows16_sum(part));
          if (16 * u < left && qt == 0 && row0 + 16 * s + li < p.M)
            *reinterpret_cast<floatx2*>(score_row + (static_cast<int64_t>(key0 / 16 + u) * p.M + 16 * s) * 2) = floatx2{part, ref[s]};
        } else if constexpr (SCORES == 1) {
          // one (sum, reference) pair per score_gran keys: 4 (a lane quarter), 8 or 16
          if (p.score_gran >= 8) part = rows16_sum(part);
          if (p.score_gran >= 16) part = halves_sum(part);
          const int key = key0 + 16 * u + 4 * qt;
          const int m = row0 + 16 * s + li;
          if (((4 * qt) & (p.score_gran - 1)) == 0 && key < key_hi && m < p.M)
            *reinterpret_cast<floatx2*>(p.chunk_part + ((static_cast<int64_t>(g) * p.n_sub + (key >> gran_log2)) * p.M + m) * 2) =
                floatx2{part, ref[s]};
        }
      }
  };
  auto second_product = [&]() __attribute__((always_inline)) {
    if constexpr (BF16) {
#pragma unroll
      for (int b = 0; b < kOBlocks; ++b)
#pragma unroll
        for (int k = 2; k >= 0; --k)                        // smallest terms first
#pragma unroll
          for (int s = 0; s < NSUB; ++s)
            acc[s][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[b]), __builtin_bit_cast(bf16x8, pf[s][k]), acc[s][b], 0, 0, 0);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int db = 0; db < D / 64; ++db)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t vb = vf[i * (D / 64) + db][e];
#pragma unroll
            for (int s = 0; s < NSUB; ++s)
              acc[s][4 * db + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(vb), s_acc[s][0][i], acc[s][4 * db + e], 0, 0, 0);
          }
    }
  };
  auto key_loop = [&](auto rotated_c) __attribute__((always_inline)) {
    constexpr bool kRotated = decltype(rotated_c)::value;
    for (int s0 = 0; s0 < n_stages; s0 += kStages) {
      static_for<0, kStages>([&](auto slot_c) {
        constexpr int slot = decltype(slot_c)::value;
        const int st = s0 + slot;
        if (__builtin_expect(st < n_stages, 1)) {
          // this wave's loads of stage st (in the first perhaps of its K tile alone) have landed when no more than those requested behind
          // them are pending (score stores in between only make the wait longer); its reads of the stage before, whose place is
          // filled next, are done
          if (__builtin_expect(st == 0, 0)) wait_vmcnt_even(my_tiles > 0 ? kLoadsPerStage * (ahead - 1) + (kSplitV ? kTileLoads : 0) : 0);
          else if (kStages == 2) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          else wait_vmcnt_even(kLoadsPerStage * max(0, min(my_tiles - 1 - st, kStages - 2)));
          if (kRotated || slot == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          lds_barrier();
          if (kRotated) {
            if (st > 0 && st <= my_tiles) {
              second_product();
              store_scores(st - 1);
            }
            issue_stage(ic<(slot + kStages - 1) % kStages>{}, st + kStages - 1);
            if (st < my_tiles) {
              tile_logits(slot_c, st);
              tile_softmax(st);
            } else if (kSplitV && st == 0) lds_barrier();
          } else {
            issue_stage(ic<(slot + kStages - 1) % kStages>{}, st + kStages - 1);
            if (st < my_tiles) {
              tile_logits(slot_c, st);
              tile_softmax(st);
              store_scores(st);
              second_product();
            } else if (kSplitV && st == 0) lds_barrier();
          }
        }
      });
    }
    if (kRotated && my_tiles == n_stages) {
      second_product();
      store_scores(n_stages - 1);
    }
  };
  if (RB * KG == 8 && wave >= 4) key_loop(std::integral_constant<bool, true>{});
  else key_loop(std::integral_constant<bool, false>{});

  // ---- the key groups' partials meet in LDS; key group w finishes the w-th share of the columns and leaves the others ----
  lds_barrier();                                     // every wave has left the ring
  constexpr int kShare = kOBlocks / KG;
  constexpr int kDumpBytes = NSUB * kOBlocks * 1024;       // a wave's O^T, one floatx4 per lane and block
  float* ml = reinterpret_cast<float*>(lds + RB * KG * kDumpBytes);      // [wave][2][kRows]
  unsigned char* dump = lds + wave * kDumpBytes + lane * 16;
  auto columns = [&](int s, int b) {
    if constexpr (BF16) return acc[s][b];
    // accumulator 4 db + e holds columns 64 db + 16 qt + 4 i + e: regrouped so that a lane stores consecutive columns
    return floatx4{acc[s][b & ~3][b & 3], acc[s][(b & ~3) + 1][b & 3], acc[s][(b & ~3) + 2][b & 3], acc[s][(b & ~3) + 3][b & 3]};
  };
#pragma unroll
  for (int s = 0; s < NSUB; ++s) {
    const float sum = halves_sum(rows16_sum(run_sum[s]));
#pragma unroll
    for (int b = 0; b < kOBlocks; ++b)
      if (b / kShare != kg) *reinterpret_cast<floatx4*>(dump + (s * kOBlocks + b) * 1024) = columns(s, b);
    if (qt == 0) {
      ml[(wave * 2 + 0) * kRows + 16 * s + li] = ref[s];
      ml[(wave * 2 + 1) * kRows + 16 * s + li] = sum;
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  lds_barrier();
#pragma unroll
  for (int s = 0; s < NSUB; ++s) {
    const int m = row0 + 16 * s + li;
    float mw[KG], lw[KG];
    float top = -INFINITY;
#pragma unroll
    for (int w = 0; w < KG; ++w) {
      mw[w] = ml[((w * RB + rb) * 2 + 0) * kRows + 16 * s + li];
      lw[w] = ml[((w * RB + rb) * 2 + 1) * kRows + 16 * s + li];
      top = fmaxf(top, mw[w]);
    }
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < KG; ++w) {
      mw[w] = lw[w] > 0.f ? fast_exp2(mw[w] - top) : 0.f;      // a key group without tiles contributes nothing
      total = fmaf(lw[w], mw[w], total);
    }
    const int64_t slot = static_cast<int64_t>(split) * p.Hq * p.T + g * p.M + m;
#pragma unroll
    for (int b = 0; b < kOBlocks; ++b) {
      if (b / kShare != kg) continue;
      floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < KG; ++w)                             // in key-group order
        o += (w == b / kShare ? columns(s, b)
                              : *reinterpret_cast<const floatx4*>(lds + (w * RB + rb) * kDumpBytes + (s * kOBlocks + b) * 1024 + lane * 16)) *
             mw[w];
      const int col = BF16 ? 16 * b + 4 * qt : 64 * (b >> 2) + 16 * qt + 4 * (b & 3);
      if (m < p.M) *reinterpret_cast<floatx4*>(p.part_o + slot * D + col) = o;
    }
    if (kg == 0 && qt == 0 && m < p.M)
      *reinterpret_cast<floatx2*>(p.part_ml + slot * 2) = floatx2{top, total};
  }
}

template <int D, bool BF16, int NSUB, int RB, int SCORES>
hipError_t launch_one(const AttnParams& p, hipStream_t stream) {
  // a split begins with a score block: the kernel stores a block's pair from one tile of one split
  if (SCORES && p.keys_per_split % p.score_gran != 0) return hipErrorInvalidValue;
  using T = Tile<D, BF16>;
  constexpr int kWaves = RB * KG;
  constexpr int kStageBytes = KG * 2 * T::kBytes;
  constexpr int kRing = stages_of(kStageBytes) * kStageBytes;
  constexpr int kMergeBytes = kWaves * (NSUB * (D / 16) * 1024 + 2 * 16 * NSUB * 4);
  constexpr int kLdsBytes = kMergeBytes > kRing ? kMergeBytes : kRing;
  static_assert(kLdsBytes <= 160 * 1024, "ring and merge area must fit the 160 KB of LDS");
  auto kernel = prefix_f32_kernel<D, BF16, NSUB, RB, SCORES>;
  if (kLdsBytes > 64 * 1024) {
    // more than the default 64 KB of dynamic LDS: raise the cap once per device
    static std::atomic<bool> attr_set[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!attr_set[dev].load(std::memory_order_acquire)) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
      if (e != hipSuccess) return e;
      attr_set[dev].store(true, std::memory_order_release);
    }
  }
  const int rows_per_wg = 16 * NSUB * RB;
  dim3 grid(p.head_fastest ? p.Hkv : p.S, p.head_fastest ? p.S : p.Hkv, (p.M + rows_per_wg - 1) / rows_per_wg);
  return launch_kernel(kernel, grid, dim3(kWaves * 64), kLdsBytes, stream, address_of(p.kp), address_of(p.vp), address_of(p.q), p.kp_sh, p.L,
                       p.keys_per_split, p.M, p.G, static_cast<int>(p.kp_sl), p.head_fastest, p);
}

template <int D, bool BF16, int NSUB, int RB>
hipError_t launch_shape(const AttnParams& p, hipStream_t stream) {
  if (!p.want_scores) return launch_one<D, BF16, NSUB, RB, 0>(p, stream);
  // 64-row workgroups have a form for 16-key score blocks (chunks that are a multiple of 16 keys) without the run-time choices
  // and the 64-bit address of every pair: bf16 8K in 32 rows x 2, chunks of 16, 28.4 -> 27.6 us, fp32 8K 80.4 -> 79.7; with
  // fewer rows there are too few tiles to pay for its prologue (toy 5.5 -> 5.6).
  if constexpr (RB == 2)
    if (p.score_gran == 16) return launch_one<D, BF16, NSUB, RB, 2>(p, stream);
  return launch_one<D, BF16, NSUB, RB, 1>(p, stream);
}

template <int D, bool BF16>
hipError_t launch_rows(const AttnParams& p, hipStream_t stream) {
  switch (p.rows_per_group) {
    case 16: return launch_shape<D, BF16, 1, 1>(p, stream);
    case 32: return launch_shape<D, BF16, 2, 1>(p, stream);
    default: return launch_shape<D, BF16, 2, 2>(p, stream);
  }
}

}  // namespace

hipError_t launch_prefix_f32(const AttnParams& p, hipStream_t stream) {
  if (p.S <= 0) return hipSuccess;
  const bool bf16 = p.in_dtype == SPECEXT_BF16;
  if (p.d == 128) return bf16 ? launch_rows<128, true>(p, stream) : launch_rows<128, false>(p, stream);
  return bf16 ? launch_rows<64, true>(p, stream) : launch_rows<64, false>(p, stream);
}

}  // namespace specext
