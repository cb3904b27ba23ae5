// Prefill attention (SpecExtend Sec. 3.1: FlashAttention for the prefill stage of the
// target and the draft model): exact causal self-attention with an online softmax, no
// score matrix in memory, on the gfx950 matrix cores.  bf16 Q/K/V, head_dim 128, fp32
// accumulation.
//
// Shape.  The query rows of a KV head (row m = token * G + head-in-group, as in the
// verification kernels) are cut into groups of 256 / KG rows; a workgroup of 8 wavefronts
// owns one group and walks the keys 0 .. position of the group's last token in tiles of 32.
// The waves form 8 / KG row groups (32 rows each, queries and running output in registers) x
// KG key groups, which take the tiles in turns and are merged through LDS at the end.  KG = 1
// where the rows fill the chip; a piece of a prompt or a short prompt takes 2 or 4, so that
// four times as many workgroups share its work (each K/V byte then enters four times as many
// compute units, which the L2 delivers; the rule and its figures are at the launcher).
// K and V tiles arrive by direct global->LDS loads into a ring of stages (KG tiles each), one
// workgroup barrier per stage.  Only the tiles on the diagonal are masked (a key is hidden from
// a row whose token comes before it), and a wave leaves out the tiles that all of its rows
// come before.  At the end every row is normalised and written.
//
//   grid = (KV heads, row groups); row groups are taken from the last (longest key range)
//   to the first so that the long workgroups start first, and neighbouring workgroups in
//   dispatch order are the KV heads of one row group, which land on different XCDs: the
//   workgroups that share a head's K/V share an L2.
//
// Matrix-core mapping as in the verification prefix kernel: S^T = K Q^T (A = K tile from
// LDS, B = Q registers), O^T += V^T P^T (A = V^T by LDS transpose reads, B = P^T straight
// from the S^T accumulators), so that a lane owns one query row in both products.  As there,
// the two waves of a SIMD take the steps of a tile in different orders behind a barrier, so
// that one is in its softmax while the other issues matrix products.
#include "mfma_util.h"

namespace specext {
namespace {

constexpr int kTile = 32;
constexpr int kD = 128;
constexpr int kRowBytes = kD * 2;
constexpr int kTileBytes = kTile * kRowBytes;     // 8 KB
constexpr int kWaves = 8;
// Stages of the ring: 16 KB, 32 KB or 64 KB of K and V each.
constexpr int stages(int kg) { return kg == 4 ? 2 : 4; }
constexpr int ring_bytes(int kg) { return 2 * kg * stages(kg) * kTileBytes; }      // 64 KB, then 128 KB
// Behind the ring: the staging of the 256 / KG query rows (256 B each), later the row statistics
// that the key groups exchange (KG > 1) or, per wave, the staging of its 32 output rows, 256 bytes
// at a time (KG = 1; rows padded to 264 B so that the 8-byte column writes fall into distinct banks).
constexpr int kPatchStride = kRowBytes + 8;
constexpr int kPrivBytes = 32 * kPatchStride;
constexpr int lds_bytes(int kg) { return ring_bytes(kg) + (kg == 1 ? kWaves * kPrivBytes : kWaves / kg * 32 * kRowBytes); }
static_assert(lds_bytes(1) <= 160 * 1024 && lds_bytes(2) <= 160 * 1024 && lds_bytes(4) <= 160 * 1024, "must fit the 160 KB of LDS");

template <int KG>
__global__ __launch_bounds__(kWaves * 64) void prefill_rows_kernel(PrefillParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int kRowWaves = kWaves / KG;
  constexpr int kRows = kRowWaves * 32;                           // query rows of a workgroup
  constexpr int kStages = stages(KG);
  constexpr int kLoads = 8 / kRowWaves;                           // 1 KB blocks of a K (or V) tile that one wave fills
  constexpr int kLoadsPerStage = 2 * kLoads;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rw = wave % kRowWaves;
  const int kg = wave / kRowWaves;
  const int c32 = lane & 31;
  const int hf = lane >> 5;

  const int g = blockIdx.x;
  const int grp = gridDim.y - 1 - blockIdx.y;
  const int row0 = grp * kRows + rw * 32;
  const int m = row0 + c32;                                       // this lane's query row of the KV head
  const int m_last = min(p.M, (grp + 1) * kRows) - 1;              // last real row of the group
  const int key_hi = p.q_off + m_last / p.G + 1;                  // keys that row sees (<= N)
  const int load_hi = max(key_hi, kTile);                         // whole tiles are loaded; N >= 32
  const int n_tiles = (load_hi + kTile - 1) / kTile;              // tiles of this workgroup
  const int n_stages = (n_tiles + KG - 1) / KG;
  const int my_tiles = (n_tiles - kg + KG - 1) / KG;              // tiles of this key group: kg, kg + KG, ...
  const int my_pos = p.q_off + min(m, p.M - 1) / p.G;             // newest key this lane's row sees
  const int wave_first_pos = p.q_off + min(row0, p.M - 1) / p.G;  // ... the wave's first row sees
  const int wave_last_pos = p.q_off + min(row0 + 31, p.M - 1) / p.G;
  // tiles of this key group that some row of the wave sees
  const int live_tiles = min(my_tiles, (wave_last_pos / kTile - kg + KG) / KG);

  const int64_t row_bytes = p.k_sl * 2;
  const unsigned char* kbase = static_cast<const unsigned char*>(p.k) + static_cast<int64_t>(g) * p.k_sh * 2;
  const unsigned char* vbase = static_cast<const unsigned char*>(p.v) + static_cast<int64_t>(g) * p.k_sh * 2;

  // LDS ring: a tile is 32 rows x 256 B; one direct load writes 1 KB = 4 consecutive rows,
  // lane i landing at byte 16*i.  The 16-byte chunks of a row are XOR-swizzled (K: chunk ^
  // (row & 15), V: chunk ^ ((row & 3) << 2)) so that the operand reads are free of bank
  // conflicts; the LDS side of a direct load being fixed, the swizzle is applied to the
  // global address.  All K tiles come first, then all V tiles.
  const unsigned kring_lds = static_cast<unsigned>(reinterpret_cast<uintptr_t>((lds_void*)lds));
  const unsigned my_lds = kring_lds + kg * kTileBytes;
  constexpr int kVOff = kStages * KG * kTileBytes;
  const int ld_row = lane >> 4;
  const int ld_slot = lane & 15;
  unsigned k_voff[kLoads];
#pragma unroll
  for (int u = 0; u < kLoads; ++u)
    k_voff[u] = static_cast<unsigned>(ld_row * row_bytes) + ((ld_slot ^ ((4 * (kLoads * rw + u) + ld_row) & 15)) << 4);
  const unsigned v_voff = static_cast<unsigned>(ld_row * row_bytes) + ((ld_slot ^ (ld_row << 2)) << 4);

  // Tile t covers keys [32t, 32t+32); the last tile is shifted back so that it ends exactly
  // at load_hi (no load leaves the cache); its rows below 32t belong to the tile before
  // and are masked.
  auto tile_first_row = [&](int t) { return min(t * kTile, load_hi - kTile); };
  // this wave's share of its key group's tile of stage st, into ring stage SLOT: block u of kLoads (K and V)
  auto issue_block = [&](auto slot_c, int st, int u) __attribute__((always_inline)) {
    constexpr unsigned slot = decltype(slot_c)::value * (KG * kTileBytes);
    const int64_t off = (static_cast<int64_t>(tile_first_row(st * KG + kg)) + 4 * (kLoads * rw + u)) * row_bytes;
    load_to_lds_16(my_lds + slot + (kLoads * rw + u) * 1024, k_voff[u], kbase + off);
    load_to_lds_16(my_lds + kVOff + slot + (kLoads * rw + u) * 1024, v_voff, vbase + off);
  };
  auto issue_stage = [&](auto slot_c, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kLoads; ++u) issue_block(slot_c, st, u);
  };

  // prologue: stage 0, then the queries, then stages 1 .. kStages-2
  if (0 < my_tiles) issue_stage(ic<0>{}, 0);
  const unsigned q_lds = kring_lds + ring_bytes(KG) + rw * (KG == 1 ? kPrivBytes : 32 * kRowBytes);
  {
    // load u brings rows 4u..4u+3 of the 32 rows (1 KB); the lane that fills LDS chunk slot
    // `ld_slot` of row r fetches chunk ld_slot ^ (r & 15) of that query row (the K swizzle,
    // so that the fragment reads below use the K read offsets).  The key groups share the loads.
    const int t0 = min(row0, p.M - 1) / p.G;
    const unsigned char* qbase = static_cast<const unsigned char*>(p.q) + static_cast<int64_t>(t0) * p.q_st * 2;
#pragma unroll
    for (int i = 0; i < 8 / KG; ++i) {
      const int u = i * KG + kg;
      const int r = 4 * u + ld_row;
      const int mq = min(row0 + r, p.M - 1);               // padding rows repeat the last real row (never stored)
      const int tq = mq / p.G;
      const int hq = g * p.G + (mq - tq * p.G);
      const unsigned voff = static_cast<unsigned>(((tq - t0) * p.q_st + hq * p.q_sh) * 2) + ((ld_slot ^ (r & 15)) << 4);
      load_to_lds_16(q_lds + u * 1024, voff, qbase);
    }
  }
  static_for<1, kStages - 1>([&](auto u_c) {
    constexpr int u = decltype(u_c)::value;
    if (u < my_tiles) issue_stage(ic<u>{}, u);
  });

  // K operand read: row c32, chunk (2*ks + hf) ^ (c32 & 15)
  unsigned k_rd[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) k_rd[ks] = c32 * kRowBytes + ((((2 * ks) ^ (c32 & 14)) | (hf ^ (c32 & 1))) << 4);
  // V transpose read: a group of 16 lanes reads 4 keys x 16 dcols
  const int li = lane & 15;
  const int grp_col = (lane >> 4) & 1;
  const int v_key_in = 4 * hf + (li >> 2);
  const int v_q4 = li >> 2;
  // the operand reads of the loop: LDS addresses, pinned in registers, plus the ring stage's immediate
  unsigned k_addr[8], v_addr[4];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    k_addr[ks] = my_lds + k_rd[ks];
    asm volatile("" : "+v"(k_addr[ks]));
  }
#pragma unroll
  for (int db = 0; db < 4; ++db) {
    v_addr[db] = my_lds + kVOff + v_key_in * kRowBytes + ((db ^ v_q4) << 6) + ((2 * grp_col + ((li & 3) >> 1)) << 4) +
                 ((li & 1) << 3);
    asm volatile("" : "+v"(v_addr[db]));
  }

  bf16x8 qf[8];
  floatx16 acc_o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_o[db][r] = 0.f;
  float ref = -INFINITY;       // reference logit (raw units) the exponentials are taken against
  float run_sum = 0.f;         // lane-partial row sum
  const float c = p.scale_log2;
  const float lazy_raw = kLazyLog2 / c;
  const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // One tile in three steps: logits and V^T fragments (all that reads the ring), mask and online softmax (one query
  // row per lane pair, the reference moves lazily), O^T += V^T P^T.
  floatx16 s;
  bf16x8 vf[4][2];
  bf16x8 pf[2];
  auto tile_front = [&](auto slot_c) __attribute__((always_inline)) {
    constexpr int slot = decltype(slot_c)::value * (KG * kTileBytes);
    s = zero16;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uintx4 kw = *reinterpret_cast<const lds_uintx4*>(static_cast<uintptr_t>(k_addr[ks] + slot));
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kw), qf[ks], s, 0, 0, 0);
    }
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      const unsigned col = v_addr[db] + slot;
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)static_cast<uintptr_t>(col + (16 * jj) * kRowBytes));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)static_cast<uintptr_t>(col + (16 * jj + 8) * kRowBytes));
        const shortx8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        vf[db][jj] = __builtin_bit_cast(bf16x8, both);
      }
    }
  };
  auto tile_softmax = [&](int st) __attribute__((always_inline)) {
    const int key0 = (st * KG + kg) * kTile;
    const int first_row = tile_first_row(st * KG + kg);
    if (first_row < key0 || first_row + kTile - 1 > wave_first_pos) {
      // register r holds key first_row + 4*hf + 8*(r/4) + r%4: hidden when it belongs to the
      // tile before (shifted last tile) or comes after this row's token
      const int lo_thr = key0 - first_row - 4 * hf;
      const int hi_thr = my_pos - first_row - 4 * hf;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int idx = 8 * (r >> 2) + (r & 3);
        if (idx < lo_thr || idx > hi_thr) s[r] = -INFINITY;
      }
    }
    float mx = fmaxf(s[0], s[1]);
#pragma unroll
    for (int r = 2; r < 16; r += 2) mx = fmaxf(mx, fmaxf(s[r], s[r + 1]));
    if (__builtin_expect(__any(mx > ref + lazy_raw), 0)) {     // some row of this wave outgrew its reference: move every reference up
      mx = halves_max(mx);
      const float new_ref = fmaxf(ref, mx);
      // 0 on the first tile; with several key groups a row may not have seen any key yet
      const float alpha = KG == 1 || new_ref > -INFINITY ? fast_exp2((ref - new_ref) * c) : 1.f;
      ref = new_ref;
      run_sum *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[db][r] *= alpha;
    }
    const float mc = KG == 1 || ref > -INFINITY ? ref * c : 0.f;
    float part = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = fast_exp2(fmaf(s[r], c, -mc));
      part += s[r];
    }
    run_sum += part;
    pf[0] = pack8(s, 0);
    pf[1] = pack8(s, 8);
  };
  auto second_product = [&](auto between) __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][0], pf[0], acc_o[db], 0, 0, 0);
      acc_o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][1], pf[1], acc_o[db], 0, 0, 0);
      between(db);
    }
  };

  // Before stage st is read every wave waits for its own share of it and meets the others at a
  // barrier; behind that barrier every wave has also left stage st-1, whose ring stage takes
  // stage st + kStages - 1.  The loop exists once per order of the steps, so that each order gets its
  // own register allocation: the upper four waves (wave w + 4 shares wave w's SIMD) do the softmax and
  // second product of the tile before, then this tile's logits; the lower four the second product of
  // the tile before, this tile's logits, its softmax.
  auto key_loop = [&](auto upper_c) __attribute__((always_inline)) {
    constexpr bool kUpper = decltype(upper_c)::value;
    for (int s0 = 0; s0 < n_stages; s0 += kStages) {
      static_for<0, kStages>([&](auto u_c) {
        constexpr int u = decltype(u_c)::value;
        const int st = s0 + u;
        if (__builtin_expect(st < n_stages, 1)) {
          if (__builtin_expect(st > 0 && st + kStages - 2 < my_tiles, 1)) {
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kLoadsPerStage * (kStages - 2)) : "memory");
          } else {
            wait_vmcnt_even(kLoadsPerStage * max(0, min(my_tiles - 1 - st, kStages - 2)));   // also covers the queries
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // this wave's reads of stage st-1 are done
          lds_barrier();
          // With several key groups the loads of stage st + kStages - 1 go out one block at a time between the second
          // product's instructions: a load takes the address unit 16 cycles, and behind the barrier all waves would queue
          // for it before their first matrix instruction (0.82 instead of 0.99 us per stage with two key groups, 0.99
          // instead of 1.23 us with four; a single group's two loads per wave cost less than the interruption, 2 %).
          const bool more = st + kStages - 1 < my_tiles;
          auto next = [&](int b) __attribute__((always_inline)) {
            if (KG > 1 && b < kLoads && more) {
              __builtin_amdgcn_sched_barrier(0);
              issue_block(ic<(u + kStages - 1) % kStages>{}, st + kStages - 1, b);
              __builtin_amdgcn_sched_barrier(0);
            }
          };
          if ((KG == 1 || st == 0 || st > live_tiles) && more) issue_stage(ic<(u + kStages - 1) % kStages>{}, st + kStages - 1);
          if (__builtin_expect(st == 0, 0)) {
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
              qf[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const lds_uintx4*>(static_cast<uintptr_t>(q_lds + k_rd[ks])));
          }
          if constexpr (kUpper) {
            if (__builtin_expect(st > 0 && st <= live_tiles, 1)) {
              tile_softmax(st - 1);
              second_product(next);
            }
            if (__builtin_expect(st < live_tiles, 1)) tile_front(ic<u>{});
          } else {
            if (__builtin_expect(st > 0 && st <= live_tiles, 1)) second_product(next);
            if (__builtin_expect(st < live_tiles, 1)) {
              tile_front(ic<u>{});
              tile_softmax(st);
            }
          }
        }
      });
    }
    if (live_tiles == n_stages) {
      if (kUpper) tile_softmax(live_tiles - 1);
      second_product([](int) {});
    }
  };
  if (wave & 4) key_loop(ic<1>{});
  else key_loop(ic<0>{});

  if constexpr (KG > 1) {
    // ---- the key groups' partials meet in LDS; key group w finishes and writes the w-th share of the columns ----
    constexpr int kShare = 4 / KG;                                  // 32-column blocks
    lds_barrier();                                                  // every wave has left the ring and the queries
    float* ml = reinterpret_cast<float*>(lds + ring_bytes(KG));      // [wave][2][32]
    unsigned char* dump = lds + wave * (16 * 1024) + lane * 16;
    const float sum = halves_sum(run_sum);
#pragma unroll
    for (int db = 0; db < 4; ++db)
      if (db / kShare != kg) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *reinterpret_cast<floatx4*>(dump + (4 * db + r4) * 1024) =
              floatx4{acc_o[db][4 * r4], acc_o[db][4 * r4 + 1], acc_o[db][4 * r4 + 2], acc_o[db][4 * r4 + 3]};
      }
    if (hf == 0) {
      ml[wave * 64 + c32] = ref * c;
      ml[wave * 64 + 32 + c32] = sum;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    lds_barrier();
    float wgt[KG];
    float top = -INFINITY, total = 0.f;
#pragma unroll
    for (int w = 0; w < KG; ++w) top = fmaxf(top, ml[(w * kRowWaves + rw) * 64 + c32]);
#pragma unroll
    for (int w = 0; w < KG; ++w) {
      const float mw = ml[(w * kRowWaves + rw) * 64 + c32], lw = ml[(w * kRowWaves + rw) * 64 + 32 + c32];
      wgt[w] = lw > 0.f ? fast_exp2(mw - top) : 0.f;                // a key group that this row does not see contributes nothing
      total = fmaf(lw, wgt[w], total);
    }
    const float inv = 1.0f / total;
    const int tr = m / p.G;
    const int hr = g * p.G + (m - tr * p.G);
    const int64_t o = static_cast<int64_t>(tr) * p.o_st + static_cast<int64_t>(hr) * p.o_sh + 4 * hf;
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      if (db / kShare != kg) continue;
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < KG; ++w) {                              // in key-group order
          if (w == db / kShare) v += floatx4{acc_o[db][4 * r4], acc_o[db][4 * r4 + 1], acc_o[db][4 * r4 + 2], acc_o[db][4 * r4 + 3]} * wgt[w];
          else v += *reinterpret_cast<const floatx4*>(lds + (w * kRowWaves + rw) * (16 * 1024) + (4 * db + r4) * 1024 + lane * 16) * wgt[w];
        }
        v *= inv;
        if (m < p.M) {
          if (p.out_dtype == SPECEXT_BF16) {
            uintx2 w;
            w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{v[0], v[1]}, bf16x2));
            w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{v[2], v[3]}, bf16x2));
            *reinterpret_cast<uintx2*>(static_cast<uint16_t*>(p.out) + o + 32 * db + 8 * r4) = w;
          } else {
            *reinterpret_cast<floatx4*>(static_cast<float*>(p.out) + o + 32 * db + 8 * r4) = v;
          }
        }
      }
    }
    if (p.lse && kg == 0 && hf == 0 && m < p.M)
      p.lse[static_cast<int64_t>(hr) * p.Tq + tr] = (top + __builtin_amdgcn_logf(total)) * kLn2;
    return;
  }

  // ---- normalise and write.  O^T sits in registers with a lane owning one row; it goes
  // through the wave's private LDS area, 256 bytes per row at a time (all 128 columns as
  // bf16, or 64 columns as fp32), so that the global stores are whole 256-byte pieces.
  unsigned char* priv = lds + ring_bytes(1) + wave * kPrivBytes;
  const float l_tot = halves_sum(run_sum);
  const float inv = 1.0f / l_tot;
  const int rows_here = min(32, p.M - row0);       // <= 0 for a wave of padding rows only
  const int passes = p.out_dtype == SPECEXT_BF16 ? 1 : 2;
  for (int pass = 0; pass < passes; ++pass) {
    if (pass == 1) __builtin_amdgcn_wave_barrier();
    if (p.out_dtype == SPECEXT_BF16) {
#pragma unroll
      for (int db = 0; db < 4; ++db) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          uintx2 w;
          const floatx2 f0 = {acc_o[db][4 * r4] * inv, acc_o[db][4 * r4 + 1] * inv};
          const floatx2 f1 = {acc_o[db][4 * r4 + 2] * inv, acc_o[db][4 * r4 + 3] * inv};
          w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f0, bf16x2));
          w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f1, bf16x2));
          *reinterpret_cast<uintx2*>(priv + c32 * kPatchStride + (32 * db + 8 * r4 + 4 * hf) * 2) = w;
        }
      }
    } else {
#pragma unroll
      for (int d2 = 0; d2 < 2; ++d2) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          floatx4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = (pass == 0 ? acc_o[d2][4 * r4 + e] : acc_o[2 + d2][4 * r4 + e]) * inv;
          // 16 bytes at column 32*d2 + 8*r4 + 4*hf of the 64-column half; rows padded by 8 B
          // are only 8-byte aligned, so two 8-byte writes
          unsigned char* dst = priv + c32 * kPatchStride + (32 * d2 + 8 * r4 + 4 * hf) * 4;
          *reinterpret_cast<floatx2*>(dst) = floatx2{w[0], w[1]};
          *reinterpret_cast<floatx2*>(dst + 8) = floatx2{w[2], w[3]};
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int row = 4 * it + (lane >> 4);
      const uintx2* src = reinterpret_cast<const uintx2*>(priv + row * kPatchStride + 16 * (lane & 15));
      const uintx2 a = src[0], b = src[1];
      if (row < rows_here) {
        const int mr = row0 + row;
        const int tr = mr / p.G;
        const int hr = g * p.G + (mr - tr * p.G);
        const int64_t o = static_cast<int64_t>(tr) * p.o_st + static_cast<int64_t>(hr) * p.o_sh;
        unsigned char* dst = p.out_dtype == SPECEXT_BF16
                                 ? static_cast<unsigned char*>(p.out) + o * 2 + 16 * (lane & 15)
                                 : static_cast<unsigned char*>(p.out) + o * 4 + 256 * pass + 16 * (lane & 15);
        *reinterpret_cast<uintx4*>(dst) = uintx4{a[0], a[1], b[0], b[1]};
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
  if (p.lse && hf == 0 && m < p.M) {
    const int tr = m / p.G;
    const int hr = g * p.G + (m - tr * p.G);
    p.lse[static_cast<int64_t>(hr) * p.Tq + tr] = (ref * c + __builtin_amdgcn_logf(l_tot)) * kLn2;
  }
}

template <int KG>
hipError_t launch_key_groups(const PrefillParams& p, hipStream_t stream) {
  auto kernel = prefill_rows_kernel<KG>;
  static std::atomic<bool> attr_set[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!attr_set[dev].load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(KG));
    if (e != hipSuccess) return e;
    attr_set[dev].store(true, std::memory_order_release);
  }
  const int rows_per_wg = kWaves / KG * 32;
  dim3 grid(p.Hkv, (p.M + rows_per_wg - 1) / rows_per_wg);
  return launch_kernel(kernel, grid, dim3(kWaves * 64), lds_bytes(KG), stream, p);
}

}  // namespace

// Key groups per workgroup.  In units of a tile's period the launch takes as long as the longer of its longest
// workgroup and its total work over the compute units; more key groups shorten the first and leave the second, but a
// period costs more (every K/V byte enters more compute units): at a full chip 0.95 us with one group, 1.00 with two, 1.21
// with four (and 0.75, 0.82, 0.99 us where most of the chip idles).  Measured, us for 1 / 2 / 4 groups at 32 query and 8
// KV heads: 512 new tokens behind 15851 374 / 206 / 156; 1024 behind 7168 191 / 129 / 146; 2048 behind 6144 225 / 229 /
// 272; whole prompts of 512 18.3 / 13.4 / 9.8, of 1024 30.5 / 21.2 / 20.2, of 2048 56 / 45 / 54, of 4096 133 / 147 / 174.
hipError_t launch_prefill_rows(const PrefillParams& p, hipStream_t stream) {
  const int rows = kWaves * 32;
  const int groups = (p.M + rows - 1) / rows;
  const float longest = static_cast<float>((p.N + kTile - 1) / kTile);
  const float shortest = static_cast<float>((p.q_off + (rows + p.G - 1) / p.G + kTile - 1) / kTile);
  const float share = static_cast<float>(p.Hkv) * groups * 0.5f * (longest + (shortest < longest ? shortest : longest)) / p.n_cus;
  auto periods = [&](int kg) { return longest / kg > share ? longest / kg : share; };
  if (1.15f * periods(2) >= periods(1)) return launch_key_groups<1>(p, stream);
  return 1.2f * periods(4) >= periods(2) ? launch_key_groups<2>(p, stream) : launch_key_groups<4>(p, stream);
}

}  // namespace specext
