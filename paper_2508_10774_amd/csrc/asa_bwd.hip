// Block-sparse attention backward for gfx950, mask held constant (the paper restricts attention
// with the block mask "during both training and inference", Sec. 3.3 Step 2.1).
//
//   Delta = rowsum(dO * O), LSE in log2 units     delta_kernel (both padded to whole blocks)
//   dQ    = scale * dS K     per query block      dq_kernel   (walks the row list, CSR)
//   dK    = scale * dS^T Q,  dV = P^T dO  per key block   dkv_kernel  (walks the column list, CSC)
// with P = exp(scale*S - LSE), dS = P * (dO V^T - Delta) recomputed per tile in both kernels,
// so no atomics are needed and the result does not depend on scheduling.
//
// Operand orientation (32x32x16 bf16 MFMA, see asa_fwd.hip for kappa / rho):
//   dq_kernel : keys on the M axis, queries on lanes: S^T = K Q^T and dP^T = V dO^T share the
//               accumulator layout, LSE and Delta are per-lane scalars, and bf16(dS^T) is directly
//               the B operand of dQ^T = K^T dS^T (K^T operand by transposing LDS reads of the K rows).
//   dkv_kernel: queries on the M axis, keys on lanes: S = Q K^T, dP = dO V^T with K, V of the
//               wave's 32 keys resident in registers; bf16(P) and bf16(dS) are the B operands of
//               dV^T = dO^T P and dK^T = Q^T dS (dO^T, Q^T operands by transposing LDS reads of
//               the row tiles).
#include <stdlib.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "asa_common.hpp"
#include "asa_tiles.hpp"

namespace asa {

constexpr float kLog2e = 1.44269504088896340736f;

// ---------------------------------------------------------------------------------------
// Row statistics of the backward, three rows of Lpad values per slab, padded to whole blocks so that the
// kernels can fetch 64 of them without a bounds test:
//   ndelta[slab][row] = - sum_x dO[row][x] * (O[row][x] + O_lo[row][x])  (fp32), 0 past L
//   lse2[slab][row]  = LSE[row] * log2(e), +inf past L (every probability of such a row is 0)
//   lse2g            = lse2 - bias (for keys whose scores carry an additive bias), if asked for
// D / 8 lanes per row, 16 bytes each (bound: HBM; with 16 lanes per row at d = 64, half of them idle,
// 81 us for 48 heads of 17 776 rows, 59 us now).
// ---------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void delta_kernel(const void *o, const void *o_lo,
                                                    const void *d_o, TensorView to, int H, int L,
                                                    int Lpad, const float *lse, float bias_log2,
                                                    float *ndelta, float *lse2, float *lse2g) {
  constexpr int kLanes = D / 8;
  const int slab = blockIdx.y;
  const int row = blockIdx.x * (256 / kLanes) + threadIdx.x / kLanes;
  const int sub = threadIdx.x % kLanes;
  float acc = 0.f;
  if (row < L) {
    const int64_t at = (int64_t)row * to.sL + 8 * sub;
    const bf16x8 a = *reinterpret_cast<const bf16x8 *>(slab_ptr(o, to, slab, H) + at);
    const bf16x8 b = *reinterpret_cast<const bf16x8 *>(slab_ptr(d_o, to, slab, H) + at);
    const bf16x8 lo = *reinterpret_cast<const bf16x8 *>(slab_ptr(o_lo, to, slab, H) + at);
#pragma unroll
    for (int x = 0; x < 8; ++x) acc += ((float)a[x] + (float)lo[x]) * (float)b[x];
  }
#pragma unroll
  for (int off = kLanes / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (row < Lpad && sub == 0) {
    const int64_t at = 3 * (int64_t)slab * Lpad + row;
    const float l2 = row < L ? lse[(int64_t)slab * L + row] * kLog2e : INFINITY;
    ndelta[at] = -acc;
    lse2[at] = l2;
    if (lse2g) lse2g[at] = l2 - bias_log2;
  }
}

// The same without Delta, one thread per row: where Delta is formed from the tiles (DELTA_ONLY below), O and
// dO need not be read for it (block 64, d 128, 40 slabs of 5 000 rows, four blocks per row, whole
// backward: 274 us with the two reads, 254 us without).
__global__ __launch_bounds__(256) void lse2_kernel(int L, int Lpad, const float *lse, float bias_log2,
                                                   float *lse2, float *lse2g) {
  const int slab = blockIdx.y, row = blockIdx.x * 256 + threadIdx.x;
  if (row >= Lpad) return;
  const int64_t at = 3 * (int64_t)slab * Lpad + row;
  const float l2 = row < L ? lse[(int64_t)slab * L + row] * kLog2e : INFINITY;
  lse2[at] = l2;
  if (lse2g) lse2g[at] = l2 - bias_log2;
}

struct BwdArgs {
  const void *q, *k, *v, *d_o;
  const float *lse2, *ndelta; // [slab][Lpad], slabs 3 Lpad apart: LSE * log2(e) (minus this launch's key bias), -Delta; padded with +inf, 0
  float *ndelta_out;          // where the Delta-only walk of dq_kernel writes (the same array as ndelta)
  const int32_t *row_ptr, *col_idx, *col_ptr, *row_idx;
  void *dq, *dk, *dv;
  TensorView tq, tk, tv, to;
  int H, L, Lpad, Nb, n_slabs;
  float scale, scale_log2e;
  const int32_t *order;   // dK/dV: work item of each workgroup slot, longest column first inside an XCD's share (null: natural order)
  const int32_t *order_q; // dQ: the same by rows
  int lead;               // one launch for both: items of an XCD's share of dQ that come before the rest of dK / dV
  // ---- global tokens of ASA_G (all zero / null when they are not used)
  // dK/dV kernels: the key side of a launch may be the pooled tokens instead of K, V
  int Lk, Nbk;            // valid key rows and key blocks of this launch (= L, Nb normally)
  float *gk32, *gv32;     // non-null: write fp32 gradients [chunk][slab][Nbk * block][d] here instead of dk / dv
  int q_chunks;           // with gk32 / gv32: the query blocks are split into this many ranges, one workgroup each
  const float *pool_gk, *pool_gv;   // non-null: add pool_g*[slab][row / pool_n] / count(window) to row's gradient
  int pool_n, pool_rows;  // pooling window; rows per slab of pool_gk / pool_gv
  // dQ kernel: pooled tiles appended to every query block's list
  const void *kg, *vg;    // [slab][Nbg * block][d] bf16
  int Lg, Nbg;
  float pooled_bias_log2;
};

template <int BLK, int D>
struct BwdCfg {
  static constexpr int kWaves = BLK / 32;
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kST = 32;                       // rows (keys or queries) per tile
  static constexpr int kSub = BLK / kST;               // tiles per block
  static constexpr int kStages = 4;                    // LDS stages
  static constexpr int kTile = kST * D * 2;            // bytes of one row tile
  static constexpr int kDqStage = 2 * kTile;                   // K rows, V rows
  static constexpr int kDkvStage = 2 * kTile + 2 * kST * 4;    // Q rows, dO rows, LSE, -Delta
  static constexpr int kDqLds = kStages * kDqStage;
  static constexpr int kDkvLds = kStages * kDkvStage;
  static constexpr int kWavesPerSimd = D == 128 ? 1 : 2;              // dK / dV
  // dQ at block 128 / d 128 just fits 256 registers: two workgroups per compute unit hide each other's
  // starts and barriers (2.12 -> 2.00 ms at 12 heads of 32 760 tokens).  At block 64 / d 128 the copy
  // offsets of two wavefronts do not fit (spills: 98 -> 130 us at 12 slabs of 4 332).
  static constexpr int kDqWavesPerSimd = D == 128 && BLK == 64 ? 1 : 2;
};

// ---------------------------------------------------------------------------------------
// The tile loop of dq_kernel and dkv_kernel: a software pipeline inside ONE wavefront.
//
// Two wavefronts of a SIMD that each run "matrix products, then vector work, then products" hardly
// overlap on this chip: the cycles of a step were the SUM of its matrix, vector and copy cycles
// (dQ at block 128 / d 128: 2640 of them for 1536 matrix cycles).  But one wavefront hides two
// exponentials and three multiply-adds under every 32-cycle MFMA it issues itself (33..38 cycles
// measured).  So a tile is 32 rows, and an iteration has two phases:
//   A: the S and dP products of tile t + 1; between them, two instructions here and there, the
//      exponentials, products and packs that turn S and dP of tile t into P and dS;
//   B: the products that add tile t to the gradients; between them the copies of tile t + 3.
// Everything is pinned slot by slot (one MFMA, its share of the other work, a scheduling barrier),
// LDS operands are read 5..6 products ahead through a ring that runs on across iterations, and
// there is one workgroup barrier per tile.  A wavefront issues one instruction every ~5 cycles, so
// the number of instructions matters as much as the MFMAs: four LDS stages with the loop unrolled
// by four make every LDS address a register plus an immediate; -Delta is the initial value of the
// dP accumulator; at d = 128 the copies take their addresses from RunningTileCopy, all but those of dQ at block 128 or with pooled
// tokens (dK / dV at block 128 / d 128 231 -> 210 instructions per tile; whole backward at block 64 / d 128, 8 heads of
// 17 776 tokens, 990 -> 970 us; block 128 / d 128, 12 heads of 32 760, no change beyond the noise of 0.5 %).  Operands two at a time,
// with one wait for both, change nothing.
// Registers: dK / dV at d = 128 (and dQ at block 64 / d 128) run one wavefront per SIMD with the
// gradients in accumulation registers (the instruction is written out for that: the compiler would
// move S and P there as well, at a vector instruction per register and tile), the others two.
// Bound: the matrix cores at the power limit (Wan2.1 shape: dK / dV 1.18 PFLOP/s executed, matrix pipe
// busy 73 % of the cycles at 1.53 GHz, dQ 1.23 PFLOP/s, 86 % at 1.37 GHz; with neither copies nor
// vector work the same loop runs at 1.4).  Against two unpipelined wavefronts per SIMD, 25 % density, MI355X:
//   block 128 / d 128, 12 heads of 32 760:  dK+dV 3.19 -> 2.75 ms, dQ 2.40 -> 2.00 ms
//   block 64 / d 64, 48 heads of 17 776:    dK+dV 1.93 -> 1.67 ms, dQ 1.52 -> 1.33 ms
//   block 64 / d 128, 12 slabs of 4 332:    dK+dV 235 -> 118 us, dQ 177 -> 98 us, Delta 144 -> 75 us
// Eight stages instead of four are 1.5 % slower (longer start of a workgroup), 4 or 7 operands ahead
// instead of 6 change nothing.
// ---------------------------------------------------------------------------------------

// ---------------------------------------------------------------------------------------
// dQ: one workgroup per query block, one wavefront per 32 query rows (its Q and dO rows stay
// in registers as B operands).  The "channels x keys" operand of dQ^T = K^T dS^T is gathered from
// the K row tile by the transposing LDS read.
// ---------------------------------------------------------------------------------------
// GT: with the pooled (global) tokens of ASA_G appended to every query block's list
// DELTA_ONLY: no gradient; the same walk forms Delta_q = sum_c P_qc dP_qc (= rowsum(dO * O) with
// the exact O, since the P of a row sum to 1) from the unrounded fp32 P and dP and writes -Delta to
// a.ndelta_out.  Used when the caller has not kept the low half of O: Delta from the bf16 O alone
// is off by up to 0.05 in rows whose soft-max is spread over keys with similar values, and that
// error goes into dQ and dK times the size of the keys / queries.
template <int BLK, int D, bool GT, bool DELTA_ONLY>
__device__ __forceinline__ void dq_walk(const BwdArgs &a, int workgroup, uint32_t smem_addr, int *cols) {
  using C = BwdCfg<BLK, D>;
  constexpr int kVOff = C::kTile, kStage = C::kDqStage;
  constexpr int kPooled = 1 << 30;             // flag of an entry of cols[]: a block of pooled tokens

  const int slot = xcd_contiguous_work(workgroup, a.n_slabs * a.Nb);
  if (slot < 0) return;
  const int work = a.order_q ? a.order_q[slot] : slot;
  const int slab = work / a.Nb;
  const int qb = work - slab * a.Nb;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, hl = lane >> 5, n = lane & 31;

  const bf16 *qs = slab_ptr(a.q, a.tq, slab, a.H);
  const bf16 *ks = slab_ptr(a.k, a.tk, slab, a.H);
  const bf16 *vs = slab_ptr(a.v, a.tv, slab, a.H);
  const bf16 *gs = slab_ptr(a.d_o, a.to, slab, a.H);
  const bool dense = a.row_ptr == nullptr;   // no index lists: every key block
  const int t_begin = dense ? 0 : a.row_ptr[slab * (a.Nb + 1) + qb];
  const int n_own_blocks = dense ? a.Nb : a.row_ptr[slab * (a.Nb + 1) + qb + 1] - t_begin;
  const int n_blocks = n_own_blocks + (GT ? a.Nbg : 0);   // pooled blocks come after the row's own list
  {
    const int32_t *g = a.col_idx + (int64_t)slab * a.Nb * a.Nb + t_begin;
    for (int t = tid; t < n_blocks; t += C::kThreads)
      cols[t] = t >= n_own_blocks ? (t - n_own_blocks) | kPooled : (dense ? t : g[t]);
  }
  // pooled keys / values of this slab: rows of D elements, padded to whole blocks
  const bf16 *kgs = reinterpret_cast<const bf16 *>(a.kg) + (int64_t)slab * a.Nbg * BLK * D;
  const bf16 *vgs = reinterpret_cast<const bf16 *>(a.vg) + (int64_t)slab * a.Nbg * BLK * D;

  const int qrow = qb * BLK + wave * 32 + n;
  const bool qvalid = qrow < a.L;
  const int qrow_c = qvalid ? qrow : a.L - 1;
  bf16x8 qreg[D / 16], greg[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    qreg[s] = *reinterpret_cast<const bf16x8 *>(qs + (int64_t)qrow_c * a.tq.sL + 16 * s + 8 * hl);
    greg[s] = *reinterpret_cast<const bf16x8 *>(gs + (int64_t)qrow_c * a.to.sL + 16 * s + 8 * hl);
  }
  // rows past L have LSE = +inf there, so that every probability is exactly zero
  const float lse2 = a.lse2[3 * (int64_t)slab * a.Lpad + qrow];
  // dP starts from -Delta instead of zero (the subtraction then costs nothing) where 16 registers for
  // it do not cost a wavefront
  const float ndelta = DELTA_ONLY ? 0.f : a.ndelta[3 * (int64_t)slab * a.Lpad + qrow];
  constexpr bool kInitDelta = !(BLK == 128 && D == 128) || DELTA_ONLY;
  f32x16 nd16;
#pragma unroll
  for (int i = 0; i < 16; ++i) nd16[i] = kInitDelta ? ndelta : 0.f;
  float dsum = 0.f;   // DELTA_ONLY: sum of P * dP over my keys

  f32x16 acc[D / 32];
#pragma unroll
  for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[dm][i] = 0.f;

  using Copy = TrTileCopy<C::kST, D, C::kWaves>;
  // (at block 128 / d 128 the 256 registers of dQ are full without the running copies' offsets: the walk for Delta 2065
  // -> 2156 us at 4 heads of 32 760 tokens; d 64, small calls: 0.98x)
  constexpr bool kRun = !GT && BLK == 64 && D == 128;
  using RunCopy = RunningTileCopy<C::kST, D, C::kWaves>;
  Copy copy_k, copy_v;
  RunCopy run_k, run_v;
  LastTileWatch watch;
  if constexpr (!kRun) {
    copy_k.init(wave, lane, a.tk.sL, a.L);
    copy_v.init(wave, lane, a.tv.sL, a.L);
  } else {
    run_k.init(wave, lane, ks, a.tk.sL, a.L);
    run_v.init(wave, lane, vs, a.tv.sL, a.L);
    watch.init(RunCopy::last_row0(a.L));
  }
  constexpr int kI = Copy::kInstr;
  constexpr int kBatch = 2 * kI;                // copy instructions per tile and wavefront
  const int last_row0 = Copy::last_row0(a.L);
  Copy copy_p;                                  // pooled rows: D elements apart, never ragged
  if (GT) copy_p.init(wave, lane, D, C::kST);

  // (stages are absolute LDS addresses, multiples of 256: the XORs below touch lower bits only)
  // row-wise A fragments (S^T = K Q^T, dP^T = V dO^T): row kappa(n) of the 32 keys
  const int kr = kappa(n);
  uint32_t row_at[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    row_at[s] = (smem_addr + (uint32_t)(kr * D * 2 + (hl ^ t_swz<D>(kr)) * 16)) ^ (uint32_t)(32 * s);
  // transposed A fragments "32 channels x 16 keys" of dQ^T += K^T dS^T (see dkv_kernel)
  const int tr_i = lane & 15, tr_w = tr_i & 3, tr_j = tr_i >> 2, tr_b = (lane >> 4) & 1;
  const uint32_t tr_lane = smem_addr + tr_piece<D>(8 * hl + tr_j, 16 * (tr_w & 1) + 8 * tr_b + 4 * (tr_w >> 1));
  uint32_t tr_at[2 * (D / 32)];
#pragma unroll
  for (int dm = 0; dm < D / 32; ++dm) {
    tr_at[2 * dm] = tr_lane ^ (uint32_t)(((4 * dm) ^ t_swz<D>(0)) * 16);
    tr_at[2 * dm + 1] = tr_lane ^ (uint32_t)(((4 * dm) ^ t_swz<D>(4)) * 16);
  }
  const float c = a.scale_log2e;
  const int n_it = n_blocks * C::kSub;

  // The tile whose copies come next (see dkv_kernel)
  int entry_v = 0, entry_at = 0, key_c = 0;
  bool last_tile = false, pooled_c = false;
  const char *base_k = nullptr, *base_v = nullptr;
  auto fetch_entry = [&]() __attribute__((always_inline)) {
    entry_v = cols[entry_at < n_blocks ? entry_at : n_blocks - 1];
    ++entry_at;
  };
  auto next_tile = [&](auto part_tag, auto new_block_tag) __attribute__((always_inline)) {
    constexpr int part = decltype(part_tag)::value;
    constexpr bool new_block = decltype(new_block_tag)::value;
    if constexpr (part == 0) {
      if constexpr (new_block) {
        const int e = __builtin_amdgcn_readfirstlane(entry_v);
        if (GT) pooled_c = (e & kPooled) != 0;
        key_c = (GT ? e & (kPooled - 1) : e) * BLK;
      } else {
        key_c += C::kST;
      }
    } else if constexpr (part == 1 && kRun) {
      if constexpr (new_block) run_k.block(key_c);
      else run_k.step();
    } else if constexpr (kRun) {
      if constexpr (new_block) run_v.block(key_c);
      else run_v.step();
      watch.tile(key_c, a.L, run_k, run_v);
    } else if constexpr (part == 1) {
      base_k = reinterpret_cast<const char *>(ks) + (int64_t)min(key_c, last_row0) * (a.tk.sL * 2);
      last_tile = key_c >= last_row0;
      if (GT) base_k = pooled_c ? reinterpret_cast<const char *>(kgs) + (int64_t)key_c * (D * 2) : base_k;
    } else {
      base_v = reinterpret_cast<const char *>(vs) + (int64_t)min(key_c, last_row0) * (a.tv.sL * 2);
      if (GT) base_v = pooled_c ? reinterpret_cast<const char *>(vgs) + (int64_t)key_c * (D * 2) : base_v;
    }
  };
  uint64_t started = 0;
  auto copy_one = [&](auto i_tag, uint32_t st) __attribute__((always_inline)) {
    constexpr int i = decltype(i_tag)::value, x = i < kI ? i : i - kI;
    if constexpr (!kRun) {
      const Copy &own = i < kI ? copy_k : copy_v;
      const uint32_t off = GT && pooled_c ? copy_p.off[x] : (last_tile ? own.off_last[x] : own.off[x]);
      lds_dma16_sv(i < kI ? base_k : base_v, off, st + (i < kI ? 0 : kVOff) + own.lds0 + x * 1024);
    } else if constexpr (i < kI) {
      if constexpr (x == 0) started = run_k.start(st);
      run_k.template load<x>(started);
    } else {
      if constexpr (x == 0) started = run_v.start(st + kVOff);
      run_v.template load<x>(started);
    }
  };
  auto copy_some = [&](auto from_tag, auto n_tag, uint32_t st) __attribute__((always_inline)) {
    constexpr int from = decltype(from_tag)::value;
    [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
      (copy_one(std::integral_constant<int, from + I>{}, st), ...);
    }(std::make_integer_sequence<int, decltype(n_tag)::value>{});
  };
  auto wait_copies = [&](auto n_tag) __attribute__((always_inline)) {
    constexpr int N = decltype(n_tag)::value;    // at most N instructions still in flight
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  };
  // The block of the tile in work, for the masks of the last block and the bias of pooled keys
  int cur_v = 0, cur_at = 0, key_t = 0, key_end = 0;
  float lse_t = lse2;
  auto fetch_current = [&]() __attribute__((always_inline)) {
    cur_v = cols[cur_at < n_blocks ? cur_at : n_blocks - 1];
    ++cur_at;
  };
  auto next_current = [&](auto new_block_tag) __attribute__((always_inline)) {
    if constexpr (decltype(new_block_tag)::value) {
      const int e = __builtin_amdgcn_readfirstlane(cur_v);
      key_t = (GT ? e & (kPooled - 1) : e) * BLK;
      const bool pooled = GT && (e & kPooled) != 0;
      key_end = pooled ? a.Lg : a.L;             // keys at or past it do not exist
      if (GT) lse_t = pooled ? lse2 - a.pooled_bias_log2 : lse2;
    } else {
      key_t += C::kST;
    }
  };

  // One iteration handles tile t of 32 keys: phase A computes S^T and dP^T of tile t + 1 while the
  // vector ALU turns those of tile t into dS^T, phase B adds tile t's product to dQ^T (see
  // dkv_kernel for the ring of operands, the stages and the unrolling by four tiles).
  constexpr int kNA = 2 * (D / 16), kNB = DELTA_ONLY ? 0 : 2 * (D / 32), kN = kNA + kNB;
  constexpr int kRing = kN % 8 == 0 && (kInitDelta || kN % 6) ? 8 : 6, kDepth = kRing == 8 ? 6 : 5;
  static_assert(kN % kRing == 0, "the ring continues across iterations");
  constexpr int kBar = kNA < kN - kDepth ? kNA : kN - kDepth;   // the barrier comes before this product
  bf16x8 ring[kRing];
  auto read_row = [&](auto e_tag, auto stage_tag) __attribute__((always_inline)) {   // operand e of phase A
    constexpr int e = decltype(e_tag)::value, st = decltype(stage_tag)::value * kStage;
    ring[e % kRing] = lds_read<bf16x8>(row_at[e / 2] + (uint32_t)(st + (e & 1) * kVOff));
  };
  auto read_tr = [&](auto f_tag, auto stage_tag) __attribute__((always_inline)) {    // operand f of phase B
    constexpr int f = decltype(f_tag)::value, dm = f % (D / 32), tt = f / (D / 32);
    constexpr int at = decltype(stage_tag)::value * kStage + 16 * tt * D * 2;
    const bf16x4 lo = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm] + (uint32_t)at));
    const bf16x4 hi = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm + 1] + (uint32_t)(at + 4 * D * 2)));
    ring[(kNA + f) % kRing] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr bool kWrittenOut = C::kDqWavesPerSimd == 1 && !DELTA_ONLY;
  auto accumulate = [](f32x16 &d, bf16x8 x, bf16x8 y) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (C::kDqWavesPerSimd == 1)
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(x), "v"(y));
    else
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, d, 0, 0, 0);
#endif
  };

  f32x16 s0, p0, s1, p1;
  auto body = [&](auto u_tag, f32x16 &sc, f32x16 &pc, f32x16 &sn, f32x16 &pn) __attribute__((always_inline)) {
    constexpr int U = decltype(u_tag)::value;        // tile index mod 4
    using St = std::integral_constant<int, U>;
    using St1 = std::integral_constant<int, (U + 1) & 3>;
    using St2 = std::integral_constant<int, (U + 2) & 3>;
    constexpr bool kNewBlock = (U + C::kStages - 1) % C::kSub == 0;   // of the tile copied here
    constexpr bool kNextNewBlock = (U + C::kStages) % C::kSub == 0;
    if (key_t + C::kST > key_end) {                  // (uniform, rare) keys past the end
      const int left = key_end - key_t - 8 * hl;     // (compared with constants: nothing to keep in registers)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (16 * (i >> 3) + (i & 7) >= left) sc[i] = -INFINITY;
    }
    uint32_t db[8];
    // (accumulator register i of lane half hl is key 16 (i / 8) + 8 hl + i % 8)
    auto finish = [&](int i) __attribute__((always_inline)) {
      if (DELTA_ONLY) {
        dsum = fmaf(sc[i], pc[i], dsum);
      } else {
        pc[i] = kInitDelta ? pc[i] * sc[i] : (pc[i] + ndelta) * sc[i];
        if (i & 1) db[i >> 1] = pack_bf16x2(pc[i - 1], pc[i]);
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    [&]<int... X>(std::integer_sequence<int, X...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int x = X;
        if constexpr (x == kBar) {
          // tile t + 2 has landed (everyone's copies) and nobody reads tile t - 1 any more
          wait_copies(std::integral_constant<int, (C::kStages - 4) * kBatch>{});
          asm volatile("s_barrier" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (x + kDepth < kNA) read_row(std::integral_constant<int, x + kDepth>{}, St1{});
        else if constexpr (x + kDepth < kN) read_tr(std::integral_constant<int, x + kDepth - kNA>{}, St{});
        else read_row(std::integral_constant<int, x + kDepth - kN>{}, St2{});
        if constexpr (x < kNA) {
          constexpr int s = x / 2;
          if constexpr ((x & 1) == 0)
            sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[x % kRing], qreg[s], s == 0 ? zero16 : sn, 0, 0, 0);
          else
            pn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[x % kRing], greg[s], s == 0 ? nd16 : pn, 0, 0, 0);
          constexpr int per = 16 / kNA;                // elements of tile t that belong to this slot
#pragma unroll
          for (int u = 0; u < per; ++u) {
            const int i = x * per + u;
            sc[i] = fast_exp2(fmaf(sc[i], c, -lse_t));
          }
          if constexpr (x > 0) {
#pragma unroll
            for (int u = 0; u < per; ++u) finish((x - 1) * per + u);
          }
          if constexpr (x == kNA - 1) {
#pragma unroll
            for (int u = 0; u < per; ++u) finish(x * per + u);
          }
        } else {
          constexpr int f = x - kNA, dm = f % (D / 32), tt = f / (D / 32);
          const u32x4 raw = {db[4 * tt], db[4 * tt + 1], db[4 * tt + 2], db[4 * tt + 3]};
          accumulate(acc[dm], ring[x % kRing], __builtin_bit_cast(bf16x8, raw));
        }
        if constexpr (x == 1) next_tile(std::integral_constant<int, 0>{}, std::bool_constant<kNewBlock>{});
        if constexpr (x == 3) next_tile(std::integral_constant<int, 1>{}, std::bool_constant<kNewBlock>{});
        if constexpr (x == 5) next_tile(std::integral_constant<int, 2>{}, std::bool_constant<kNewBlock>{});
        if constexpr (x == 2 && (U + 1) % C::kSub == 0) fetch_current();
        if constexpr (x == kN - 2 && kNextNewBlock) fetch_entry();
        // copies of tile t + kStages - 1, spread over the slots behind the barrier
        if constexpr (x >= kBar) {
          constexpr int i0 = (x - kBar) * kBatch / (kN - kBar), i1 = (x - kBar + 1) * kBatch / (kN - kBar);
          copy_some(std::integral_constant<int, i0>{}, std::integral_constant<int, i1 - i0>{}, smem_addr + ((U + 3) & 3) * kStage);
        }
        if constexpr (x == kN - 1) next_current(std::bool_constant<(U + 1) % C::kSub == 0>{});
        __builtin_amdgcn_sched_barrier(0);
      }(), ...);
    }(std::make_integer_sequence<int, kN>{});
  };

  __syncthreads();   // cols[] is written
  if (n_it > 0) {
    // The loop takes four tiles at a time, one per stage.  Blocks of 64 rows are two tiles: with an
    // odd number of them tile 0 goes to stage 2 and the first two tiles come before the loop.
    const bool odd = C::kSub == 2 && (n_blocks & 1);
    const uint32_t first_stage = odd ? 2u : 0u, first_off = first_stage * kStage;
    // tiles 0 .. kStages - 2
    for (int t = 0; t < C::kStages - 1; ++t) {
      auto all_parts = [&](auto new_block_tag) __attribute__((always_inline)) {
        next_tile(std::integral_constant<int, 0>{}, new_block_tag);
        next_tile(std::integral_constant<int, 1>{}, new_block_tag);
        next_tile(std::integral_constant<int, 2>{}, new_block_tag);
      };
      if (t % C::kSub == 0) {
        fetch_entry();
        all_parts(std::true_type{});
      } else {
        all_parts(std::false_type{});
      }
      copy_some(std::integral_constant<int, 0>{}, std::integral_constant<int, kBatch>{}, smem_addr + ((t + first_stage) & 3u) * kStage);
    }
    if ((C::kStages - 1) % C::kSub == 0) fetch_entry();
    fetch_current();
    next_current(std::true_type{});
    wait_copies(std::integral_constant<int, (C::kStages - 3) * kBatch>{});   // tiles 0 and 1
    __syncthreads();
    // S^T and dP^T of tile 0, first operands of tile 1
#pragma unroll
    for (int s = 0; s < D / 16; ++s) row_at[s] += first_off;
    s0 = zero16;
    p0 = nd16;
    [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int e = E;
        read_row(std::integral_constant<int, e>{}, std::integral_constant<int, 0>{});
        if constexpr ((e & 1) == 0) s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[e % kRing], qreg[e / 2], s0, 0, 0, 0);
        else p0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[e % kRing], greg[e / 2], p0, 0, 0, 0);
      }(), ...);
    }(std::make_integer_sequence<int, kNA>{});
    [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
      (read_row(std::integral_constant<int, E>{}, std::integral_constant<int, 1>{}), ...);
    }(std::make_integer_sequence<int, kDepth>{});
#pragma unroll
    for (int s = 0; s < D / 16; ++s) row_at[s] -= first_off;
    if constexpr (kWrittenOut) settle_acc(acc);
    if (odd) {
      body(std::integral_constant<int, 2>{}, s0, p0, s1, p1);
      body(std::integral_constant<int, 3>{}, s1, p1, s0, p0);
    }
    for (int t = odd ? 2 : 0; t < n_it; t += 4) {
      body(std::integral_constant<int, 0>{}, s0, p0, s1, p1);
      body(std::integral_constant<int, 1>{}, s1, p1, s0, p0);
      body(std::integral_constant<int, 2>{}, s0, p0, s1, p1);
      body(std::integral_constant<int, 3>{}, s1, p1, s0, p0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);          // stray copies must land before the LDS is given up
    if constexpr (kWrittenOut) settle_acc(acc);
  }

  if (DELTA_ONLY) {
    // the two lane halves hold different keys of the same query; rows past L get 0 (their P is 0)
    const float total = dsum + swap_halves(dsum);
    if (hl == 0) a.ndelta_out[3 * (int64_t)slab * a.Lpad + qrow] = -total;
    return;
  }
  if (qvalid) {
    bf16 *dst_row = slab_ptr(a.dq, a.tq, slab, a.H) + (int64_t)qrow * a.tq.sL;
#pragma unroll
    for (int dm = 0; dm < D / 32; ++dm) {
      uint32_t w[8];
#pragma unroll
      for (int i = 0; i < 16; i += 2)
        w[i >> 1] = pack_bf16x2(acc[dm][i] * a.scale, acc[dm][i + 1] * a.scale);
      uint4 *dst = reinterpret_cast<uint4 *>(dst_row + dm * 32 + 16 * hl);
      dst[0] = make_uint4(w[0], w[1], w[2], w[3]);
      dst[1] = make_uint4(w[4], w[5], w[6], w[7]);
    }
  }
}

// ---------------------------------------------------------------------------------------
// dK, dV: one workgroup per key block, one wavefront per 32 keys; its K and V rows stay in
// registers as B operands and both 32 x d fp32 accumulators live in registers, so S and P are
// computed once per tile for both gradients.  A tile is the Q rows and dO rows of 32 queries and
// their LSE and -Delta values.  The products with P^T and dS^T need "channels x queries" operands:
// they are gathered from the same row tiles by the transposing LDS read, so no transposed copy of
// Q or dO exists, in LDS or in memory.
// ---------------------------------------------------------------------------------------
template <int BLK, int D>
__device__ __forceinline__ void dkv_walk(const BwdArgs &a, int workgroup, uint32_t smem_addr, int *rows) {
  using C = BwdCfg<BLK, D>;
  constexpr int kGOff = C::kTile, kStatOff = 2 * C::kTile, kStage = C::kDkvStage;

  const int work_c = xcd_contiguous_work(workgroup, a.n_slabs * a.Nbk * a.q_chunks);
  if (work_c < 0) return;
  const int chunk = work_c % a.q_chunks;      // range of query blocks (1 range unless pooled keys)
  const int work = a.order ? a.order[work_c] : work_c / a.q_chunks;
  const int slab = work / a.Nbk;
  const int kb = work - slab * a.Nbk;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, hl = lane >> 5, n = lane & 31;

  const bf16 *qs = slab_ptr(a.q, a.tq, slab, a.H);
  const bf16 *ks = slab_ptr(a.k, a.tk, slab, a.H);
  const bf16 *vs = slab_ptr(a.v, a.tv, slab, a.H);
  const bf16 *gs = slab_ptr(a.d_o, a.to, slab, a.H);
  // lanes 0..31 fetch the 32 LSE values of a tile, lanes 32..63 its 32 negated Deltas (both arrays
  // are padded to whole blocks: no bounds test; the LSE values of a slab stand one or two rows of Lpad
  // values behind its Deltas, so the distance fits 32 bits)
  const float *stat_s = a.ndelta + 3 * (int64_t)slab * a.Lpad;
  const uint32_t stat_off = (uint32_t)(n * 4) + (hl ? 0u : (uint32_t)((a.lse2 - a.ndelta) * 4));
  const bool dense = a.col_ptr == nullptr;   // no index lists: every query block
  const int t_begin = dense ? 0 : a.col_ptr[slab * (a.Nb + 1) + kb];
  const int per_chunk = (a.Nb + a.q_chunks - 1) / a.q_chunks;
  const int first = chunk * per_chunk;          // dense: my range of query blocks
  const int n_blocks = dense ? max(0, min(per_chunk, a.Nb - first))
                             : a.col_ptr[slab * (a.Nb + 1) + kb + 1] - t_begin;
  {
    const int32_t *g = a.row_idx + (int64_t)slab * a.Nb * a.Nb + t_begin;
    for (int t = tid; t < n_blocks; t += C::kThreads) rows[t] = dense ? first + t : g[t];
  }
  const int krow = kb * BLK + wave * 32 + n;
  const bool kvalid = krow < a.Lk;
  const int krow_c = kvalid ? krow : a.Lk - 1;
  bf16x8 kreg[D / 16], vreg[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    kreg[s] = *reinterpret_cast<const bf16x8 *>(ks + (int64_t)krow_c * a.tk.sL + 16 * s + 8 * hl);
    vreg[s] = *reinterpret_cast<const bf16x8 *>(vs + (int64_t)krow_c * a.tv.sL + 16 * s + 8 * hl);
  }
  f32x16 kacc[D / 32], vacc[D / 32];   // dK^T and dV^T of my 32 keys
#pragma unroll
  for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
    for (int i = 0; i < 16; ++i) kacc[dm][i] = vacc[dm][i] = 0.f;

  using Copy = TrTileCopy<C::kST, D, C::kWaves>;
  using RunCopy = RunningTileCopy<C::kST, D, C::kWaves>;
  constexpr bool kRun = D == 128;               // (d 64, small calls: 0.98x)
  Copy copy_q, copy_g;
  RunCopy run_q, run_g;
  LastTileWatch watch;
  if constexpr (kRun) {
    run_q.init(wave, lane, qs, a.tq.sL, a.L);
    run_g.init(wave, lane, gs, a.to.sL, a.L);
    watch.init(RunCopy::last_row0(a.L));
  } else {
    copy_q.init(wave, lane, a.tq.sL, a.L);
    copy_g.init(wave, lane, a.to.sL, a.L);
  }
  constexpr int kI = Copy::kInstr;
  constexpr int kBatch = 2 * kI + 1;            // copy instructions per tile and wavefront
  const int last_row0 = Copy::last_row0(a.L);

  // (stages are absolute LDS addresses, multiples of 256: the XORs below touch lower bits only)
  // row-wise A fragments (S = Q K^T, dP = dO V^T): row kappa(n) of the 32 queries, 16-byte chunk
  // (2 s + hl) ^ t_swz(row)
  const int kr = kappa(n);
  uint32_t row_at[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    row_at[s] = (smem_addr + (uint32_t)(kr * D * 2 + (hl ^ t_swz<D>(kr)) * 16)) ^ (uint32_t)(32 * s);
  // transposed A fragments "32 channels x 16 queries" (dV^T += dO^T P, dK^T += Q^T dS): lane i of
  // a 16-lane group addresses query i / 4 of 4 consecutive ones and 4 of the channels that
  // the MFMA rows of its group stand for (row order rho); two reads make the 8 queries of a lane
  const int tr_i = lane & 15, tr_w = tr_i & 3, tr_j = tr_i >> 2, tr_b = (lane >> 4) & 1;
  const uint32_t tr_lane = smem_addr + tr_piece<D>(8 * hl + tr_j, 16 * (tr_w & 1) + 8 * tr_b + 4 * (tr_w >> 1));
  uint32_t tr_at[2 * (D / 32)];
#pragma unroll
  for (int dm = 0; dm < D / 32; ++dm) {
    tr_at[2 * dm] = tr_lane ^ (uint32_t)(((4 * dm) ^ t_swz<D>(0)) * 16);
    tr_at[2 * dm + 1] = tr_lane ^ (uint32_t)(((4 * dm) ^ t_swz<D>(4)) * 16);
  }
  const float c = a.scale_log2e;
  const int n_it = n_blocks * C::kSub;

  // The tile whose copies come next: query block `cb` (entry of the list) and its first row, base
  // addresses.  Tiles past the end repeat the last block: the number of copies in flight stays the
  // same and their data is not used.
  int entry_v = 0, entry_at = 0, q0 = 0;
  bool last_tile = false;
  const char *base_q = nullptr, *base_g = nullptr, *base_st = nullptr;
  auto fetch_entry = [&]() __attribute__((always_inline)) {      // (read well before it is used)
    entry_v = rows[entry_at < n_blocks ? entry_at : n_blocks - 1];
    ++entry_at;
  };
  // three parts, so that a kernel slot holds a few scalar instructions only
  auto next_tile = [&](auto part_tag, auto new_block_tag) __attribute__((always_inline)) {
    constexpr int part = decltype(part_tag)::value;
    constexpr bool new_block = decltype(new_block_tag)::value;
    if constexpr (part == 0) {
      q0 = new_block ? __builtin_amdgcn_readfirstlane(entry_v) * BLK : q0 + C::kST;
      if constexpr (!kRun || new_block) base_st = reinterpret_cast<const char *>(stat_s) + (int64_t)q0 * 4;
      else base_st += C::kST * 4;
    } else if constexpr (part == 1 && kRun) {
      if constexpr (new_block) run_q.block(q0);
      else run_q.step();
    } else if constexpr (kRun) {
      if constexpr (new_block) run_g.block(q0);
      else run_g.step();
      watch.tile(q0, a.L, run_q, run_g);
    } else if constexpr (part == 1) {
      base_q = reinterpret_cast<const char *>(qs) + (int64_t)min(q0, last_row0) * (a.tq.sL * 2);
      last_tile = q0 >= last_row0;
    } else {
      base_g = reinterpret_cast<const char *>(gs) + (int64_t)min(q0, last_row0) * (a.to.sL * 2);
    }
  };
  uint64_t started = 0;
  auto copy_one = [&](auto i_tag, uint32_t st) __attribute__((always_inline)) {
    constexpr int i = decltype(i_tag)::value;
    if constexpr (i < kI && kRun) {
      if constexpr (i == 0) started = run_q.start(st);
      run_q.template load<i>(started);
    } else if constexpr (i < 2 * kI && kRun) {
      if constexpr (i == kI) started = run_g.start(st + kGOff);
      run_g.template load<i - kI>(started);
    } else if constexpr (i < kI) {
      copy_q.issue_one(i, st, base_q, last_tile);
    } else if constexpr (i < 2 * kI) {
      copy_g.issue_one(i - kI, st + kGOff, base_g, last_tile);
    } else {
      lds_dma4_sv(base_st, stat_off, st + kStatOff);
    }
  };
  auto copy_some = [&](auto from_tag, auto n_tag, uint32_t st) __attribute__((always_inline)) {
    constexpr int from = decltype(from_tag)::value;
    [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
      (copy_one(std::integral_constant<int, from + I>{}, st), ...);
    }(std::make_integer_sequence<int, decltype(n_tag)::value>{});
  };
  auto wait_copies = [&](auto n_tag) __attribute__((always_inline)) {
    constexpr int N = decltype(n_tag)::value;    // at most N instructions still in flight
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  };

  // One iteration handles tile t: phase A computes S and dP of tile t + 1 (matrix pipe) while the
  // vector ALU turns S and dP of tile t into P and dS; phase B adds tile t's products to dV and dK.
  // The A operands are read kDepth products ahead through a ring that runs on from iteration to
  // iteration.  The loop is unrolled by four tiles, one per stage: every LDS address is a
  // register plus an immediate.
  constexpr int kNA = 2 * (D / 16), kNB = 4 * (D / 32), kN = kNA + kNB;
  constexpr int kRing = 8, kDepth = 6;
  static_assert(kN % kRing == 0, "the ring continues across iterations");
  bf16x8 ring[kRing];
  auto read_row = [&](auto e_tag, auto stage_tag) __attribute__((always_inline)) {   // operand e of phase A
    constexpr int e = decltype(e_tag)::value, st = decltype(stage_tag)::value * kStage;
    ring[e % kRing] = lds_read<bf16x8>(row_at[e / 2] + (uint32_t)(st + (e & 1) * kGOff));
  };
  auto read_tr = [&](auto f_tag, auto stage_tag) __attribute__((always_inline)) {    // operand f of phase B
    constexpr int f = decltype(f_tag)::value, st = decltype(stage_tag)::value * kStage;
    constexpr int dm = (f / 2) % (D / 32), tt = f / (2 * (D / 32));
    constexpr int at = st + ((f & 1) == 0 ? kGOff : 0) + 16 * tt * D * 2;
    const bf16x4 lo = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm] + (uint32_t)at));
    const bf16x4 hi = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm + 1] + (uint32_t)(at + 4 * D * 2)));
    ring[(kNA + f) % kRing] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // LSE and -Delta of the 8 + 8 queries of my lane half, from stage `st`
  f32x4 lse_v[4];
  uint32_t stat_at = smem_addr + kStatOff + 32 * hl;
  auto read_lse = [&](int q, int st) __attribute__((always_inline)) {
    lse_v[q] = lds_read<f32x4>(stat_at + (uint32_t)(st * kStage + ((q >> 1) * 16 + (q & 1) * 4) * 4));
  };
  auto read_ndelta = [&](int q, int st, f32x16 &p) __attribute__((always_inline)) {
    const f32x4 v = lds_read<f32x4>(stat_at + (uint32_t)(st * kStage + C::kST * 4 + ((q >> 1) * 16 + (q & 1) * 4) * 4));
#pragma unroll
    for (int x = 0; x < 4; ++x) p[4 * q + x] = v[x];
  };
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto accumulate = [](f32x16 &acc, bf16x8 x, bf16x8 y) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (C::kWavesPerSimd == 1)
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(x), "v"(y));
    else
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, acc, 0, 0, 0);
#endif
  };

  f32x16 s0, p0, s1, p1;
  auto body = [&](auto u_tag, f32x16 &sc, f32x16 &pc, f32x16 &sn, f32x16 &pn) __attribute__((always_inline)) {
    constexpr int U = decltype(u_tag)::value;        // tile index mod 4
    using St = std::integral_constant<int, U>;
    using St1 = std::integral_constant<int, (U + 1) & 3>;
    using St2 = std::integral_constant<int, (U + 2) & 3>;
    // the tile copied in this iteration, t + kStages - 1, starts a new query block?
    constexpr bool kNewBlock = (U + C::kStages - 1) % C::kSub == 0;
    constexpr bool kNextNewBlock = (U + C::kStages) % C::kSub == 0;
    uint32_t pb[8], db[8];
    auto pack = [&](int i) __attribute__((always_inline)) {
      pc[i] *= sc[i];
      if (i & 1) {
        pb[i >> 1] = pack_bf16x2(sc[i - 1], sc[i]);
        db[i >> 1] = pack_bf16x2(pc[i - 1], pc[i]);
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int e = E;
        if constexpr (e + kDepth < kNA) read_row(std::integral_constant<int, e + kDepth>{}, St1{});
        else read_tr(std::integral_constant<int, e + kDepth - kNA>{}, St{});
        constexpr int s = e / 2;
        if constexpr ((e & 1) == 0)
          sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[e % kRing], kreg[s], s == 0 ? zero16 : sn, 0, 0, 0);
        else
          pn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[e % kRing], vreg[s], pn, 0, 0, 0);
        constexpr int per = 16 / kNA;                // elements of tile t that belong to this slot
#pragma unroll
        for (int u = 0; u < per; ++u) {
          const int i = e * per + u;
          sc[i] = fast_exp2(fmaf(sc[i], c, -lse_v[i >> 2][i & 3]));
        }
        if constexpr (e > 0) {
#pragma unroll
          for (int u = 0; u < per; ++u) pack((e - 1) * per + u);
        }
        if constexpr (e == kNA - 1) {
#pragma unroll
          for (int u = 0; u < per; ++u) pack(e * per + u);
        }
        if constexpr (e == 1) next_tile(std::integral_constant<int, 0>{}, std::bool_constant<kNewBlock>{});
        if constexpr (e == 3) next_tile(std::integral_constant<int, 1>{}, std::bool_constant<kNewBlock>{});
        if constexpr (e == 5) next_tile(std::integral_constant<int, 2>{}, std::bool_constant<kNewBlock>{});
        __builtin_amdgcn_sched_barrier(0);
      }(), ...);
    }(std::make_integer_sequence<int, kNA>{});

    // tile t + 2 has landed (everyone's copies) and nobody reads tile t - 1 any more
    wait_copies(std::integral_constant<int, (C::kStages - 4) * kBatch>{});
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    [&]<int... F>(std::integer_sequence<int, F...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int f = F, e = kNA + f;
        if constexpr (f + kDepth < kNB) read_tr(std::integral_constant<int, f + kDepth>{}, St{});
        else read_row(std::integral_constant<int, f + kDepth - kNB>{}, St2{});
        constexpr int dm = (f / 2) % (D / 32), tt = f / (2 * (D / 32));
        if constexpr ((f & 1) == 0) {
          const u32x4 raw = {pb[4 * tt], pb[4 * tt + 1], pb[4 * tt + 2], pb[4 * tt + 3]};
          accumulate(vacc[dm], ring[e % kRing], __builtin_bit_cast(bf16x8, raw));
        } else {
          const u32x4 raw = {db[4 * tt], db[4 * tt + 1], db[4 * tt + 2], db[4 * tt + 3]};
          accumulate(kacc[dm], ring[e % kRing], __builtin_bit_cast(bf16x8, raw));
        }
        if constexpr (f < 4) read_lse(f, (U + 1) & 3);
        else if constexpr (f < 8) read_ndelta(f - 4, (U + 2) & 3, pc);
        if constexpr (f == 0 && kNextNewBlock) fetch_entry();
        // copies of tile t + kStages - 1, spread over the slots
        constexpr int i0 = f * kBatch / kNB, i1 = (f + 1) * kBatch / kNB;
        copy_some(std::integral_constant<int, i0>{}, std::integral_constant<int, i1 - i0>{}, smem_addr + ((U + 3) & 3) * kStage);
        __builtin_amdgcn_sched_barrier(0);
      }(), ...);
    }(std::make_integer_sequence<int, kNB>{});
  };

  __syncthreads();   // rows[] is written
  if (n_it > 0) {
    // The loop takes four tiles at a time, one per stage.  Blocks of 64 rows are two tiles: with an
    // odd number of them tile 0 goes to stage 2 and the first two tiles come before the loop.
    const bool odd = C::kSub == 2 && (n_blocks & 1);
    const uint32_t first_stage = odd ? 2u : 0u, first_off = first_stage * kStage;
    // tiles 0 .. kStages - 2
    for (int t = 0; t < C::kStages - 1; ++t) {
      auto all_parts = [&](auto new_block_tag) __attribute__((always_inline)) {
        next_tile(std::integral_constant<int, 0>{}, new_block_tag);
        next_tile(std::integral_constant<int, 1>{}, new_block_tag);
        next_tile(std::integral_constant<int, 2>{}, new_block_tag);
      };
      if (t % C::kSub == 0) {
        fetch_entry();
        all_parts(std::true_type{});
      } else {
        all_parts(std::false_type{});
      }
      copy_some(std::integral_constant<int, 0>{}, std::integral_constant<int, kBatch>{}, smem_addr + ((t + first_stage) & 3u) * kStage);
    }
    if ((C::kStages - 1) % C::kSub == 0) fetch_entry();
    wait_copies(std::integral_constant<int, (C::kStages - 3) * kBatch>{});   // tiles 0 and 1
    __syncthreads();
    // S and dP of tile 0, first operands of tile 1
#pragma unroll
    for (int s = 0; s < D / 16; ++s) row_at[s] += first_off;
    stat_at += first_off;
    s0 = zero16;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      read_lse(q, 0);
      read_ndelta(q, 0, p0);
      read_ndelta(q, 1, p1);
    }
    [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int e = E;
        read_row(std::integral_constant<int, e>{}, std::integral_constant<int, 0>{});
        if constexpr ((e & 1) == 0) s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[e % kRing], kreg[e / 2], s0, 0, 0, 0);
        else p0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[e % kRing], vreg[e / 2], p0, 0, 0, 0);
      }(), ...);
    }(std::make_integer_sequence<int, kNA>{});
    [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
      (read_row(std::integral_constant<int, E>{}, std::integral_constant<int, 1>{}), ...);
    }(std::make_integer_sequence<int, kDepth>{});
#pragma unroll
    for (int s = 0; s < D / 16; ++s) row_at[s] -= first_off;
    stat_at -= first_off;
    if constexpr (C::kWavesPerSimd == 1) {
      settle_acc(kacc);
      settle_acc(vacc);
    }
    if (odd) {
      body(std::integral_constant<int, 2>{}, s0, p0, s1, p1);
      body(std::integral_constant<int, 3>{}, s1, p1, s0, p0);
    }
    for (int t = odd ? 2 : 0; t < n_it; t += 4) {
      body(std::integral_constant<int, 0>{}, s0, p0, s1, p1);
      body(std::integral_constant<int, 1>{}, s1, p1, s0, p0);
      body(std::integral_constant<int, 2>{}, s0, p0, s1, p1);
      body(std::integral_constant<int, 3>{}, s1, p1, s0, p0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);          // stray copies must land before the LDS is given up
    if constexpr (C::kWavesPerSimd == 1) {
      settle_acc(kacc);
      settle_acc(vacc);
    }
  }

  // epilogue of one gradient: acc holds its transpose for my 32 keys
  auto emit = [&](f32x16 *acc, const bool is_dv) {
    const float mul = is_dv ? 1.f : a.scale;
    float *out32 = is_dv ? a.gv32 : a.gk32;
    if (out32) {
      // gradients of pooled tokens: kept in fp32 for the launch that spreads them over the windows
      if (kvalid) {
        float *row = out32 + (((int64_t)chunk * a.n_slabs + slab) * a.Nbk * BLK + krow) * D;
#pragma unroll
        for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            f32x4 v = {acc[dm][4 * q4] * mul, acc[dm][4 * q4 + 1] * mul, acc[dm][4 * q4 + 2] * mul,
                       acc[dm][4 * q4 + 3] * mul};
            *reinterpret_cast<f32x4 *>(row + dm * 32 + 16 * hl + 4 * q4) = v;
          }
      }
      return;
    }
    if (!kvalid) return;
    bf16 *out_row = is_dv ? slab_ptr(a.dv, a.tv, slab, a.H) + (int64_t)krow * a.tv.sL
                          : slab_ptr(a.dk, a.tk, slab, a.H) + (int64_t)krow * a.tk.sL;
    const float *pool = is_dv ? a.pool_gv : a.pool_gk;
#pragma unroll
    for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[dm][i] *= mul;
    if (pool) {
      // the mean over a window passes 1 / count of the pooled token's gradient to each token
      const int w = krow / a.pool_n;
      const int cnt = min(a.pool_n, a.Lk - w * a.pool_n);
      const float inv = 1.f / (float)cnt;
      const float *prow = pool + ((int64_t)slab * a.pool_rows + w) * D;
#pragma unroll
      for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const f32x4 v = *reinterpret_cast<const f32x4 *>(prow + dm * 32 + 16 * hl + 4 * q4);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[dm][4 * q4 + e] += v[e] * inv;
        }
    }
#pragma unroll
    for (int dm = 0; dm < D / 32; ++dm) {
      uint32_t w[8];
#pragma unroll
      for (int i = 0; i < 16; i += 2)
        w[i >> 1] = pack_bf16x2(acc[dm][i], acc[dm][i + 1]);
      uint4 *po = reinterpret_cast<uint4 *>(out_row + dm * 32 + 16 * hl);
      po[0] = make_uint4(w[0], w[1], w[2], w[3]);
      po[1] = make_uint4(w[4], w[5], w[6], w[7]);
    }
  };
  emit(kacc, false);
  emit(vacc, true);
}

static size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }
template <int BLK, int D, bool GT, bool DELTA_ONLY = false>
__global__ __launch_bounds__(BLK * 2, (BwdCfg<BLK, D>::kDqWavesPerSimd)) void dq_kernel(BwdArgs a) {
  extern __shared__ __align__(1024) unsigned char smem[];
  __shared__ int cols[kMaxNb];
  dq_walk<BLK, D, GT, DELTA_ONLY>(a, blockIdx.x, ASA_LDS_ADDR_OF(smem), cols);
}

template <int BLK, int D>
__global__ __launch_bounds__(BLK * 2, (BwdCfg<BLK, D>::kWavesPerSimd)) void dkv_kernel(BwdArgs a) {
  extern __shared__ __align__(1024) unsigned char smem[];
  __shared__ int rows[kMaxNb];
  dkv_walk<BLK, D>(a, blockIdx.x, ASA_LDS_ADDR_OF(smem), rows);
}

// dK / dV and dQ in one launch: neither needs the other's results, so the dQ workgroups fill the compute
// units that the last round of dK / dV leaves idle, and a small call is one chain of workgroups instead of two.
// Bound of such calls: the longest workgroup and the start of a launch.  Backward of two launches -> one, same
// bits (d 64 / block 64 unless stated): 34 workgroups per gradient 20.7 -> 15.3 us, 378 67 -> 51, 1016 180 -> 148,
// 3048 380 -> 377; block 64 / d 128: 378 83 -> 69, 1016 267 -> 256, 3048 737 -> 732; block 128 / d 64: 192
// 60 -> 44, 512 166 -> 137, 1536 362 -> 357; block 128 / d 128: 18 33 -> 22, 192 83 -> 75, 320 129 -> 115.
// Many rounds hide the last one, and two kinds of lists at a time share less of the L2: 6144 workgroups of block 64
// 1192 -> 1206 us at d 64, 2331 -> 2372 at d 128; block 128 / d 128, where dQ here has one wavefront per SIMD instead
// of two, 768 equal, 1024 319 -> 324, 1280 581 -> 602.
// The rows and columns of always-kept prefix blocks are as long as the sequence, and a workgroup takes one alone: those of dQ
// start right behind those of dK / dV (`lead` of each XCD's share) and not behind all of dK / dV.  Same bits; us: block 64, 17 776 tokens of
// which 226 are text, d 64: 1 head 313 -> 244, 3 heads 330 -> 309, d 128: 3 heads 495 -> 442; 4 heads of 4 276 85 -> 68; block 128 /
// d 128, 3 heads of 12 780, 300 text, 346 -> 295.  (prefix_rows_last: where. Also where
// all workgroups start at once: without it there, 1 head 311 us.) (All of dQ between dK / dV, one by
// one: 0.96-0.98x where there is no prefix.)
template <int BLK, int D, bool GT>
__global__ __launch_bounds__(BLK * 2, (BwdCfg<BLK, D>::kWavesPerSimd)) void dkv_dq_kernel(BwdArgs a) {
  extern __shared__ __align__(1024) unsigned char smem[];
  __shared__ int list[kMaxNb];
  const int first_dq = gridDim.x / 2;          // (a multiple of the number of XCDs)
  bool dkv = (int)blockIdx.x < first_dq;
  int workgroup = dkv ? (int)blockIdx.x : (int)blockIdx.x - first_dq;
  if (a.lead > 0) {
    // in an XCD's share: the first `lead` of dK / dV, the first `lead` of dQ, the rest of dK / dV, the rest of dQ
    const int share = first_dq / kNumXcd, turn = blockIdx.x / kNumXcd;
    dkv = turn < a.lead || (turn >= 2 * a.lead && turn < share + a.lead);
    const int at = turn < a.lead ? turn : (turn < 2 * a.lead || turn < share + a.lead ? turn - a.lead : turn - share);
    workgroup = at * kNumXcd + blockIdx.x % kNumXcd;
  }
  if (dkv) dkv_walk<BLK, D>(a, workgroup, ASA_LDS_ADDR_OF(smem), list);
  else dq_walk<BLK, D, GT, false>(a, workgroup, ASA_LDS_ADDR_OF(smem), list);
}

static size_t order_bytes(const Problem &pb) {
  return round256((size_t)pb.n_slabs * pb.Nb * sizeof(int32_t));
}
static size_t rowstat_bytes(const Problem &pb) {
  return round256((size_t)pb.n_slabs * pb.Lpad * sizeof(float));
}
size_t bwd_workspace_bytes(const Problem &pb) {
  // [slab][3][Lpad] fp32 (-Delta, LSE in log2 units, the same minus the pooled keys'
  // bias), then the orders of the dK / dV and of the dQ workgroups
  return 3 * rowstat_bytes(pb) + 2 * order_bytes(pb);
}
// sum of the per-range partial gradients of the pooled tokens into range 0's buffer
__global__ void pooled_reduce_kernel(float *buf, int chunks, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  f32x4 acc = reinterpret_cast<const f32x4 *>(buf)[i];
  for (int c = 1; c < chunks; ++c) {
    const f32x4 v = reinterpret_cast<const f32x4 *>(buf + c * n * 4)[i];
    acc += v;
  }
  reinterpret_cast<f32x4 *>(buf)[i] = acc;
}
static int pooled_chunks(const Problem &pb, int Nbg) {
  // enough workgroups to fill the chip, at most 16 ranges (each costs a partial buffer)
  int c = (1024 + pb.n_slabs * Nbg - 1) / (pb.n_slabs * Nbg);
  c = c > 16 ? 16 : c;
  return c > pb.Nb ? pb.Nb : (c < 1 ? 1 : c);
}
static size_t pooled_rows_bytes(const Problem &pb, int Nbg, size_t elem) {
  return round256((size_t)pb.n_slabs * Nbg * pb.block * pb.d * elem);
}
size_t bwd_g_workspace_bytes(const Problem &pb, int Nbg) {
  // ... then the pooled tokens' dK, dV (fp32, one buffer per range of query blocks)
  return bwd_workspace_bytes(pb) + 2 * pooled_chunks(pb, Nbg) * pooled_rows_bytes(pb, Nbg, 4);
}

// Do two [B, H, L, d] bf16 tensors share memory, or stand in one another's gaps?
static bool overlap(const Problem &pb, const void *x, const TensorView &tx, const void *y, const TensorView &ty) {
  auto last = [&](const void *t, const TensorView &v) {
    return reinterpret_cast<const bf16 *>(t) + (pb.B - 1) * v.sB + (pb.H - 1) * v.sH + (pb.L - 1) * v.sL + pb.d - 1;
  };
  return x <= static_cast<const void *>(last(y, ty)) && y <= static_cast<const void *>(last(x, tx));
}

// workgroups of dK / dV on the chip
static int bwd_resident(int block, int d) { return block == 64 && d == 64 ? 1024 : (block == 128 && d == 128 ? 256 : 512); }
// Would a prefix row end the launch late?  From 1.2 times what each resident workgroup has to do on average, where such rows are a
// fifth of all at most.  (373 calls with text: early rows 0.98-1.28x in the 248 that this takes, 1.05x on average, 1.00x in the
// others; with more of them, long rows of both kinds share compute units, down to 0.93x.)
static bool prefix_rows_last(const Problem &pb) {
  if (pb.n_prefix_blocks == 0 || 5 * pb.n_prefix_blocks > pb.Nb) return false;
  return 5 * (int64_t)pb.Nb * bwd_resident(pb.block, pb.d) > 6 * pb.n_slabs * listed_blocks(pb);
}

// dq_over_inputs: dQ is written into memory that dK / dV reads (asa.h allows it): dK / dV must have ended before
template <int BLK, int D>
static hipError_t launch_bwd_t(const BwdArgs &a, const BwdArgs *pooled_launch, bool dq_over_inputs, hipStream_t st) {
  using C = BwdCfg<BLK, D>;
  {
    const void *dq_fns[4] = {reinterpret_cast<const void *>(&dq_kernel<BLK, D, false>),
                             reinterpret_cast<const void *>(&dq_kernel<BLK, D, true>),
                             reinterpret_cast<const void *>(&dq_kernel<BLK, D, false, true>),
                             reinterpret_cast<const void *>(&dq_kernel<BLK, D, true, true>)};
    for (const void *fn : dq_fns) {
      hipError_t e0 = set_dynamic_lds_once(fn, C::kDqLds);
      if (e0 != hipSuccess) return e0;
    }
    hipError_t e0 = set_dynamic_lds_once(reinterpret_cast<const void *>(&dkv_kernel<BLK, D>), C::kDkvLds);
    if (e0 != hipSuccess) return e0;
    const void *both_fns[2] = {reinterpret_cast<const void *>(&dkv_dq_kernel<BLK, D, false>),
                               reinterpret_cast<const void *>(&dkv_dq_kernel<BLK, D, true>)};
    for (const void *fn : both_fns) {
      e0 = set_dynamic_lds_once(fn, C::kDkvLds);
      if (e0 != hipSuccess) return e0;
    }
  }
  const int grid = xcd_grid(a.n_slabs * a.Nb);
  // One launch or two (see dkv_dq_kernel): the line is where the gain of filling the last round has gone.
  const int resident = bwd_resident(BLK, D);
  const bool together = !dq_over_inputs && a.n_slabs * a.Nb <= (BLK == D ? 3 : 6) * resident;
  hipError_t e = hipSuccess;
  if (a.ndelta_out) {
    // no low half of O from the caller: Delta from the tiles themselves, before anything uses it
    if (pooled_launch)
      hipLaunchKernelGGL((dq_kernel<BLK, D, true, true>), dim3(grid), dim3(C::kThreads), C::kDqLds, st, a);
    else
      hipLaunchKernelGGL((dq_kernel<BLK, D, false, true>), dim3(grid), dim3(C::kThreads), C::kDqLds, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  timing_begin(st);
  if (pooled_launch) {
    // gradients of the pooled tokens first (fp32, every query block attends them) ...
    const BwdArgs &g = *pooled_launch;
    const int ggrid = xcd_grid(g.n_slabs * g.Nbk * g.q_chunks);
    hipLaunchKernelGGL((dkv_kernel<BLK, D>), dim3(ggrid), dim3(C::kThreads), C::kDkvLds, st, g);
    e = hipGetLastError();
    if (e == hipSuccess && g.q_chunks > 1) {
      const int64_t n4 = (int64_t)g.n_slabs * g.Nbk * BLK * D / 4;
      const int rgrid = (int)((n4 + 255) / 256);
      hipLaunchKernelGGL(pooled_reduce_kernel, dim3(rgrid), dim3(256), 0, st, g.gv32, g.q_chunks, n4);
      hipLaunchKernelGGL(pooled_reduce_kernel, dim3(rgrid), dim3(256), 0, st, g.gk32, g.q_chunks, n4);
      e = hipGetLastError();
    }
  }
  // ... then the tokens' own gradients, which add their share of the pooled ones
  if (e == hipSuccess && together) {
    if (pooled_launch)
      hipLaunchKernelGGL((dkv_dq_kernel<BLK, D, true>), dim3(2 * grid), dim3(C::kThreads), C::kDkvLds, st, a);
    else
      hipLaunchKernelGGL((dkv_dq_kernel<BLK, D, false>), dim3(2 * grid), dim3(C::kThreads), C::kDkvLds, st, a);
    e = hipGetLastError();
    timing_end(st);
    return e;
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL((dkv_kernel<BLK, D>), dim3(grid), dim3(C::kThreads), C::kDkvLds, st, a);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    if (pooled_launch)
      hipLaunchKernelGGL((dq_kernel<BLK, D, true>), dim3(grid), dim3(C::kThreads), C::kDqLds, st, a);
    else
      hipLaunchKernelGGL((dq_kernel<BLK, D, false>), dim3(grid), dim3(C::kThreads), C::kDqLds, st, a);
    e = hipGetLastError();
  }
  timing_end(st);
  return e;
}

hipError_t launch_bwd(const Problem &pb, const void *q, const void *k, const void *v,
                      const void *o, const void *o_lo, const void *d_o, const float *lse,
                      const int32_t *row_ptr, const int32_t *col_idx, const int32_t *col_ptr,
                      const int32_t *row_idx, void *dq, void *dk, void *dv, void *workspace,
                      hipStream_t st, const GlobalTokens *gt) {
  unsigned char *ws = reinterpret_cast<unsigned char *>(workspace);
  const size_t rb = rowstat_bytes(pb);
  float *ndelta = reinterpret_cast<float *>(ws);
  float *lse2 = ndelta + pb.Lpad;
  float *lse2g = ndelta + 2 * pb.Lpad;
  int32_t *order = reinterpret_cast<int32_t *>(ws + 3 * rb);

  hipError_t e = hipSuccess;
  const float pooled_bias = gt ? log2f((float)gt->n) : 0.f;
  const int rows = 2048 / pb.d;      // rows per workgroup of delta_kernel
  dim3 dgrid((pb.Lpad + rows - 1) / rows, pb.n_slabs);
  if (!o_lo)
    hipLaunchKernelGGL(lse2_kernel, dim3((pb.Lpad + 255) / 256, pb.n_slabs), dim3(256), 0, st, pb.L, pb.Lpad,
                       lse, pooled_bias, lse2, gt ? lse2g : nullptr);
  else if (pb.d == 128)
    hipLaunchKernelGGL(delta_kernel<128>, dgrid, dim3(256), 0, st, o, o_lo, d_o, pb.o, pb.H, pb.L,
                       pb.Lpad, lse, pooled_bias, ndelta, lse2, gt ? lse2g : nullptr);
  else
    hipLaunchKernelGGL(delta_kernel<64>, dgrid, dim3(256), 0, st, o, o_lo, d_o, pb.o, pb.H, pb.L,
                       pb.Lpad, lse, pooled_bias, ndelta, lse2, gt ? lse2g : nullptr);
  e = hipGetLastError();
  if (e != hipSuccess) return e;

  BwdArgs a;
  a.q = q; a.k = k; a.v = v; a.d_o = d_o;
  a.lse2 = lse2; a.ndelta = ndelta;
  a.ndelta_out = o_lo ? nullptr : ndelta;
  a.row_ptr = row_ptr; a.col_idx = col_idx; a.col_ptr = col_ptr; a.row_idx = row_idx;
  a.dq = dq; a.dk = dk; a.dv = dv;
  a.tq = pb.q; a.tk = pb.k; a.tv = pb.v; a.to = pb.o;
  a.H = pb.H; a.L = pb.L; a.Lpad = pb.Lpad; a.Nb = pb.Nb; a.n_slabs = pb.n_slabs;
  a.scale = pb.scale;
  a.scale_log2e = pb.scale * kLog2e;
  a.order = nullptr;
  a.order_q = nullptr;
  a.lead = 0;
  {
    const int total = pb.n_slabs * pb.Nb;
    if (col_ptr && length_order_wanted(total)) {
      int32_t *order_q = reinterpret_cast<int32_t *>(ws + 3 * rb + order_bytes(pb));
      e = launch_length_order(col_ptr, pb.Nb, total, order, st, row_ptr, order_q);
      if (e != hipSuccess) return e;
      a.order = order;
      a.order_q = order_q;
      if (prefix_rows_last(pb))
        a.lead = std::min((pb.n_slabs + kNumXcd - 1) / kNumXcd * pb.n_prefix_blocks, (total + kNumXcd - 1) / kNumXcd);
    }
  }
  a.Lk = pb.L; a.Nbk = pb.Nb;
  a.gk32 = a.gv32 = nullptr; a.q_chunks = 1; a.pool_gk = a.pool_gv = nullptr; a.pool_n = 1; a.pool_rows = 0;
  a.kg = a.vg = nullptr; a.Lg = a.Nbg = 0; a.pooled_bias_log2 = 0.f;
  BwdArgs g;                       // the launch whose key side is the pooled tokens
  const BwdArgs *pooled = nullptr;
  if (gt) {
    unsigned char *wg = ws + bwd_workspace_bytes(pb);
    float *gk32 = reinterpret_cast<float *>(wg);
    const int chunks = pooled_chunks(pb, gt->Nbg);
    float *gv32 = reinterpret_cast<float *>(wg + chunks * pooled_rows_bytes(pb, gt->Nbg, 4));
    TensorView tvg;                // the pooled tensors: [slab][Nbg * block][d], rows of d elements
    tvg.sL = pb.d; tvg.sH = (int64_t)gt->Nbg * pb.block * pb.d; tvg.sB = tvg.sH * pb.H;
    const float bias = pooled_bias;
    g = a;
    g.order = nullptr;
    g.order_q = nullptr;
    g.k = gt->kg; g.v = gt->vg; g.tk = tvg; g.tv = tvg;
    g.col_ptr = nullptr; g.row_idx = nullptr;          // every query block attends the pooled tokens
    g.Lk = gt->Lg; g.Nbk = gt->Nbg; g.lse2 = lse2g;
    g.gk32 = gk32; g.gv32 = gv32; g.q_chunks = chunks;
    pooled = &g;
    a.pool_gk = gk32; a.pool_gv = gv32; a.pool_n = gt->n; a.pool_rows = gt->Nbg * pb.block;
    a.kg = gt->kg; a.vg = gt->vg; a.Lg = gt->Lg; a.Nbg = gt->Nbg;
    a.pooled_bias_log2 = bias;
  }
  const bool over = overlap(pb, dq, pb.q, q, pb.q) || overlap(pb, dq, pb.q, d_o, pb.o);
  if (pb.block == 128 && pb.d == 128) return launch_bwd_t<128, 128>(a, pooled, over, st);
  if (pb.block == 128 && pb.d == 64) return launch_bwd_t<128, 64>(a, pooled, over, st);
  if (pb.block == 64 && pb.d == 128) return launch_bwd_t<64, 128>(a, pooled, over, st);
  if (pb.block == 64 && pb.d == 64) return launch_bwd_t<64, 64>(a, pooled, over, st);
  return hipErrorInvalidValue;
}

}  // namespace asa
