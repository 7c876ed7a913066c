// Block-sparse flash-attention forward for gfx950 (Sec. 3.3 Step 2.2 of the paper: the
// binary block mask "directly integrated with a block-sparse attention kernel").
//
// One workgroup owns one query block of one slab and walks that row's list of kept key
// blocks.  A wavefront owns 32 query rows.  Per key tile:
//   S^T = K Q^T      MFMA 32x32x16 bf16, keys on the M axis, queries on the N axis, so a
//                    lane holds 16 keys of ONE query and the row maximum / row sum of the
//                    online soft-max need a single cross-lane exchange;
//   O^T += V^T P^T   the accumulator of S^T, rounded to bf16, already IS the B operand of
//                    this product, provided the rows of K are read in the permuted order
//                    kappa; the V^T operand comes from a per-block transposed copy of V (both
//                    LDS operand reads are then 16-byte loads) or, where making the copy costs
//                    more than it gains, from V's rows by the transposing LDS read.
// Four kernels (launch_fwd_t says which runs where): lock-step, ping-pong, pipelined, wide.  A key block is
// walked in steps of 64 (pipelined, wide: 32) keys.  The K rows and the V^T slice (or V rows) of a step are copied
// straight from global memory into LDS (no register staging) with an XOR swizzle of 16-byte
// chunks instead of row padding, which keeps the 16-byte fragment reads conflict-free.
#include <stdlib.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "asa_common.hpp"
#include "asa_tiles.hpp"

namespace asa {

// ---------------------------------------------------------------------------------------
// [slab][L][d] -> [slab][Nb][d][block] bf16: every block of `block` positions becomes one
// contiguous transposed tile (channels major), zero-filled for positions >= L.  A tile is then
// a single contiguous run in memory for the attention kernels, instead of d rows that are
// Lpad * 2 bytes apart (a power-of-two pitch that lands every row on the same memory channel).
// ---------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void transpose_kernel(const void *src, TensorView tv, int H,
                                                        int L, int Lpad, int block, bf16 *dst,
                                                        const int32_t *row_ptr, int Nb, int min_tiles) {
  constexpr int TL = 64;  // positions per workgroup
  __shared__ uint16_t tile[TL][D + 2];
  const int slab = blockIdx.y;
  // (with lists: slabs of fewer tiles go to a kernel that reads the rows of V themselves)
  if (row_ptr && row_ptr[slab * (Nb + 1) + Nb] < min_tiles) return;
  const int l0 = blockIdx.x * TL;
  const uint16_t *s = reinterpret_cast<const uint16_t *>(slab_ptr(src, tv, slab, H));
  const int tid = threadIdx.x;
  constexpr int CH = D / 8;  // 16-byte chunks per row
  for (int c = tid; c < TL * CH; c += 256) {
    int r = c / CH, cc = c % CH;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (l0 + r < L) val = *reinterpret_cast<const uint4 *>(s + (int64_t)(l0 + r) * tv.sL + cc * 8);
    const uint16_t *e = reinterpret_cast<const uint16_t *>(&val);
#pragma unroll
    for (int x = 0; x < 8; ++x) tile[r][cc * 8 + x] = e[x];
  }
  __syncthreads();
  // the 64 positions of this workgroup lie inside one block (block is a multiple of 64)
  uint16_t *out = reinterpret_cast<uint16_t *>(dst) + (int64_t)slab * D * Lpad +
                  (int64_t)(l0 / block) * D * block + (l0 % block);
  for (int c = tid; c < D * (TL / 8); c += 256) {
    int dd = c / (TL / 8), lc = c % (TL / 8);
    uint4 val;
    uint16_t *e = reinterpret_cast<uint16_t *>(&val);
#pragma unroll
    for (int x = 0; x < 8; ++x) e[x] = tile[lc * 8 + x][dd];
    *reinterpret_cast<uint4 *>(out + (int64_t)dd * block + lc * 8) = val;
  }
}

static hipError_t launch_transpose(const void *src, const TensorView &tv, int H, int L, int Lpad, int block,
                                   int d, int n_slabs, const bf16 *dst, hipStream_t st,
                                   const int32_t *row_ptr = nullptr, int Nb = 0, int min_tiles = 0) {
  dim3 grid(Lpad / 64, n_slabs);
  if (d == 128)
    hipLaunchKernelGGL(transpose_kernel<128>, grid, dim3(256), 0, st, src, tv, H, L, Lpad, block,
                       const_cast<bf16 *>(dst), row_ptr, Nb, min_tiles);
  else
    hipLaunchKernelGGL(transpose_kernel<64>, grid, dim3(256), 0, st, src, tv, H, L, Lpad, block,
                       const_cast<bf16 *>(dst), row_ptr, Nb, min_tiles);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Global tokens of ASA_G (Sec. 3.3): MeanPool_n over the token axis, K and V in one launch.  The mean
// of a window's valid tokens is formed in fp32 and rounded to bf16 (the tensor type of K_aug /
// V_aug); rows past Lg are zero.
//
// Bound: HBM (every token is read once).  D / 8 lanes read one token row as 16-byte pieces; the
// 2048 / D rows that a workgroup of 256 threads has in hand at a time are split over `parts`
// (a power of two, at most the window) interleaved shares of each window, whose sums meet in LDS.
// Small windows share a workgroup, a large one gets all of its threads.  At 12 heads of 32 760
// tokens, d = 128, window 128: 0.035 ms for K and V (5.8 TB/s), 0.115 ms with one thread per
// channel walking the window two bytes at a time, one launch per tensor.
// ---------------------------------------------------------------------------------------
struct PoolArgs {
  const void *src[2];
  bf16 *dst[2];
  TensorView tv[2];
  int H, L, n, Lg, Lg_pad, log2_parts;
};

template <int D>
__global__ __launch_bounds__(256) void pool_kernel(PoolArgs a) {
  constexpr int kLanes = D / 8, kRows = 256 / kLanes;   // lanes per row; rows per workgroup
  __shared__ float part_sum[kRows][D + 4];
  const int which = blockIdx.z, slab = blockIdx.y;
  const int c = threadIdx.x % kLanes, g = threadIdx.x / kLanes;
  const int parts = 1 << a.log2_parts;
  const int windows = kRows >> a.log2_parts;            // windows of this workgroup
  const int w0 = blockIdx.x * windows;
  const int w = w0 + (g >> a.log2_parts), part = g & (parts - 1);
  float acc[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) acc[x] = 0.f;
  if (w < a.Lg) {
    const bf16 *x0 = slab_ptr(a.src[which], a.tv[which], slab, a.H) + 8 * c;
    const int64_t pitch = a.tv[which].sL;
    const int64_t first = (int64_t)w * a.n;             // (the last window may be short)
    const int64_t last = min((int64_t)a.L, first + a.n);
#pragma unroll 8
    for (int64_t r = first + part; r < last; r += parts) {
      const bf16x8 v = *reinterpret_cast<const bf16x8 *>(x0 + r * pitch);
#pragma unroll
      for (int x = 0; x < 8; ++x) acc[x] += (float)v[x];
    }
  }
#pragma unroll
  for (int x = 0; x < 8; ++x) part_sum[g][8 * c + x] = acc[x];
  __syncthreads();
  if (part != 0 || w >= a.Lg_pad) return;
#pragma unroll
  for (int x = 0; x < 8; ++x) acc[x] = 0.f;
  for (int p = 0; p < parts; ++p)
#pragma unroll
    for (int x = 0; x < 8; ++x) acc[x] += part_sum[g + p][8 * c + x];
  const int count = max(1, min(a.L - w * a.n, a.n));
  uint32_t out[4];
#pragma unroll
  for (int x = 0; x < 8; x += 2)
    out[x >> 1] = w < a.Lg ? pack_bf16x2(acc[x] / (float)count, acc[x + 1] / (float)count) : 0u;
  *reinterpret_cast<uint4 *>(a.dst[which] + ((int64_t)slab * a.Lg_pad + w) * D + 8 * c) =
      make_uint4(out[0], out[1], out[2], out[3]);
}

hipError_t launch_pool(const Problem &pb, int n, const void *k, const void *v, void *kg, void *vg,
                       hipStream_t st) {
  PoolArgs a;
  a.src[0] = k; a.src[1] = v;
  a.dst[0] = reinterpret_cast<bf16 *>(kg); a.dst[1] = reinterpret_cast<bf16 *>(vg);
  a.tv[0] = pb.k; a.tv[1] = pb.v;
  a.H = pb.H; a.L = pb.L; a.n = n;
  a.Lg = (pb.L + n - 1) / n;
  a.Lg_pad = ((a.Lg + pb.block - 1) / pb.block) * pb.block;
  const int rows = 2048 / pb.d;
  a.log2_parts = 0;
  while ((2 << a.log2_parts) <= rows && (2 << a.log2_parts) <= n) ++a.log2_parts;
  const int windows = rows >> a.log2_parts;
  const dim3 grid((a.Lg_pad + windows - 1) / windows, pb.n_slabs, 2);
  if (pb.d == 128) hipLaunchKernelGGL(pool_kernel<128>, grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL(pool_kernel<64>, grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// forward kernel
// ---------------------------------------------------------------------------------------
struct FwdArgs {
  const void *q, *k, *v;
  const bf16 *vt;  // [slab][Nb][d][block]: V, one transposed tile per key block
  const int32_t *row_ptr, *col_idx;
  void *o, *o_lo;
  float *lse;
  TensorView tq, tk, tv, to;
  int H, L, Lpad, Nb, n_slabs;
  float scale_log2e;  // scale * log2(e)
  // global tokens (ASA_G); Nbg = 0 switches them off
  const void *kg;     // [slab][Nbg * block][d] bf16 pooled keys, zero rows past Lg
  const bf16 *vgt;    // [slab][Nbg][d][block]: pooled values, transposed tiles
  const void *vg;     // [slab][Nbg * block][d] bf16 pooled values
  int Lg, Nbg;        // pooled tokens per slab, key blocks they fill
  float bias_log2;    // log2(n): the additive ln(n) of the pooled scores, in the exp2 domain
  // Choice between two kernels (lock-step and another) per (batch, head) slab, made on the device from the
  // slab's tile count: 0 = this launch takes every slab; +1 = only slabs whose rows hold at least
  // `select_min_tiles` tiles on average; -1 = only the others.
  int select, select_min_tiles;
  const int32_t *order;   // work item of each workgroup slot (longest row first inside an XCD's share), or null
};

// does this launch leave the slab to the other kernel?  (wave-uniform; before any barrier)
__device__ __forceinline__ bool slab_not_mine(const FwdArgs &a, int slab) {
  if (a.select == 0) return false;
  const int tiles = a.row_ptr[slab * (a.Nb + 1) + a.Nb];
  const bool long_rows = tiles >= a.select_min_tiles * a.Nb;
  return (a.select > 0) != long_rows;
}

template <int BLK, int D>
struct FwdCfg {
  static constexpr int kWaves = BLK / 32;
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kKT = 64;                   // keys per pipeline step
  static constexpr int kSub = BLK / kKT;           // steps per key block
  static constexpr int kKElems = kKT * D;          // one K stage:   [64 keys][D]  (unpadded)
  static constexpr int kVElems = D * kKT;          // one V^T stage: [D][64 keys]  (unpadded)
  // LDS stages of the lock-step kernel: two where the second does not cost a resident workgroup
  // (block 128: registers allow 2-3 workgroups per CU anyway), one at block 64 (measured at
  // block 64 / d 64: two stages 1.43 ms, one 1.29 ms; at block 128 / d 128: 1.695 vs 1.73 ms)
  static constexpr int kStages = BLK == 128 ? 2 : 1;
};

// The running maximum (and with it O and the row sum) is rescaled only on steps where some row
// of the wavefront actually found a larger logit; on all other steps the factor would be 1.
// The maximum is never allowed to lag behind: a row dominated by one key then has that key's
// probability equal to exactly 1, free of bf16 rounding, which the backward's Delta relies on.
//
// Lock-step kernel: one workgroup per query block, all wavefronts in lock step.  With two LDS
// stages (2 x 32 KB at d = 128) the copies of step s + 1 are requested right after the barrier
// that opens step s; with one, the copies of a step are waited for right away and the other
// workgroups on the CU compute meanwhile.  It serves large block 64 / d 64 calls, large dense calls at the
// mixed shapes and, at block 128 / d 128, short rows (launch_fwd_t draws the line) and tensors that the ping-pong
// kernel below does not take (slabs of 4 GiB and more).
// VT: the operand of the second product comes from the transposed copy of V (one 16-byte read)
// instead of the rows of V (two transposing reads).
template <int BLK, int D, bool VT>
// (block 64 / d 64 fits 128 registers: four wavefronts per SIMD, 2 % faster than three)
__global__ __launch_bounds__(BLK * 2, (BLK == 64 && D == 64) ? 4 : 2) void fwd_kernel(FwdArgs a) {
  using C = FwdCfg<BLK, D>;
  extern __shared__ __align__(1024) unsigned char smem[];
  bf16 *lds = reinterpret_cast<bf16 *>(smem);
  __shared__ int cols[kMaxNb];

  const int slot = xcd_contiguous_work(blockIdx.x, a.n_slabs * a.Nb);
  if (slot < 0) return;
  const int work = a.order ? a.order[slot] : slot;
  const int slab = work / a.Nb;
  if (slab_not_mine(a, slab)) return;
  const int qb = work - slab * a.Nb;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, hl = lane >> 5, n = lane & 31;

  const bf16 *qs = slab_ptr(a.q, a.tq, slab, a.H);
  const bf16 *ks = slab_ptr(a.k, a.tk, slab, a.H);
  const bf16 *vs = slab_ptr(a.v, a.tv, slab, a.H);
  const bf16 *vts = a.vt + (int64_t)slab * D * a.Lpad;
  // no index lists: dense attention, every key block in order
  const bool dense = a.row_ptr == nullptr;
  const int t_begin = dense ? 0 : a.row_ptr[slab * (a.Nb + 1) + qb];
  const int n_tiles = dense ? a.Nb : a.row_ptr[slab * (a.Nb + 1) + qb + 1] - t_begin;
  {
    const int32_t *g = a.col_idx + (int64_t)slab * a.Nb * a.Nb + t_begin;
    for (int t = tid; t < n_tiles; t += C::kThreads) cols[t] = dense ? t : g[t];
  }
  const int qrow = qb * BLK + wave * 32 + n;
  const bool qvalid = qrow < a.L;
  const int qrow_c = qvalid ? qrow : a.L - 1;
  bf16x8 qreg[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    qreg[s] = *reinterpret_cast<const bf16x8 *>(qs + (int64_t)qrow_c * a.tq.sL + 16 * s + 8 * hl);
  f32x16 oacc[D / 32];
#pragma unroll
  for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dm][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c = a.scale_log2e;

  RowTileCopy<C::kKT, D, C::kWaves> copy_k;
  TrTileCopy<C::kKT, D, C::kWaves> copy_v;
  ColTileCopy<BLK, D, C::kWaves> copy_vt;
  copy_k.init(wave, lane, a.tk.sL);
  if (VT) copy_vt.init(wave, lane);
  else copy_v.init(wave, lane, a.tv.sL, a.L);
  const int last_row0 = copy_v.last_row0(a.L);
  const int kr = kappa(n), cr = rho(n);
  const int kx = (hl ^ k_swz<D>(kr)) * 8, cx = (hl ^ v_swz(cr)) * 8;
  // transposed A fragments "32 channels x 16 keys" of O^T += V^T P^T, gathered from the rows of V by
  // the transposing LDS read (see asa_bwd.hip)
  const int tr_i = lane & 15, tr_w = tr_i & 3, tr_j = tr_i >> 2, tr_b = (lane >> 4) & 1;
  const uint32_t tr_lane = tr_piece<D>(8 * hl + tr_j, 16 * (tr_w & 1) + 8 * tr_b + 4 * (tr_w >> 1));
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  const int n_steps = n_tiles * C::kSub;
  constexpr int kStageElems = C::kKElems + C::kVElems;
  const uint32_t lds_addr = ASA_LDS_ADDR_OF(smem);
  // copies of one step into one of the two stages, issued in the form the compiler does not
  // track (it would otherwise wait for them before the next LDS read of the other stage)
  // (M0 and base in common for a wavefront's loads of a tile where their distances fit the instruction: lds_dma16_next adds 1024 i
  // to both addresses, the offsets are less by that; a load's rows are at least 1024 bytes from the next one's)
  constexpr bool kShared = VT && copy_k.kInstr <= 4 && copy_vt.kInstr <= 4;
  if constexpr (kShared) {
#pragma unroll
    for (int i = 0; i < copy_k.kInstr; ++i) copy_k.off[i] -= 1024u * i;
#pragma unroll
    for (int i = 0; i < copy_vt.kInstr; ++i) copy_vt.off[i] -= 1024u * i;
  }
  auto fetch = [&](int j, int sub, int stage) __attribute__((always_inline)) {
    const int row0 = j * BLK + sub * C::kKT;
    const uint32_t st = lds_addr + stage * kStageElems * 2;
    const char *kbase = reinterpret_cast<const char *>(ks) + (uint64_t)(uint32_t)row0 * (uint32_t)(a.tk.sL * 2);
    const int lim = a.L - 1 - row0;
    if constexpr (kShared) {
      const char *vtbase = reinterpret_cast<const char *>(vts) + (uint64_t)(uint32_t)j * (D * BLK * 2) + sub * (C::kKT * 2);
      if (lim >= C::kKT - 1) {
        const uint64_t k0 = lds_dma_begin(kbase, st + copy_k.lds_chunk(0));
        [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
          (lds_dma16_next<I * 1024>(k0, copy_k.off[I]), ...);
        }(std::make_integer_sequence<int, copy_k.kInstr>{});
      } else {                              // (rare) rows past the last one re-read it; the whole tile may lie past it
        const char *base = lim < 0 ? kbase + (int64_t)lim * (a.tk.sL * 2) : kbase;
#pragma unroll
        for (int i = 0; i < copy_k.kInstr; ++i) {
          const int past = max(0, copy_k.row_of(i) - max(lim, 0));
          lds_dma16_sv(base, copy_k.off[i] + 1024u * i - (uint32_t)past * (uint32_t)(a.tk.sL * 2), st + copy_k.lds_chunk(i));
        }
      }
      const uint64_t v0 = lds_dma_begin(vtbase, st + C::kKElems * 2 + copy_vt.wave * copy_vt.kInstr * 1024);
      [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
        (lds_dma16_next<I * 1024>(v0, copy_vt.off[I]), ...);
      }(std::make_integer_sequence<int, copy_vt.kInstr>{});
      return;
    }
    if (lim >= C::kKT - 1) copy_k.issue_at(st, kbase);
    else copy_k.issue_at_ragged(st, kbase, lim);
    if (VT) {
      copy_vt.issue_at(st + C::kKElems * 2, reinterpret_cast<const char *>(vts + (int64_t)j * D * BLK + sub * C::kKT));
      return;
    }
    const char *vbase = reinterpret_cast<const char *>(vs) + (int64_t)min(row0, last_row0) * a.tv.sL * 2;
#pragma unroll
    for (int i = 0; i < copy_v.kInstr; ++i) copy_v.issue_one(i, st + C::kKElems * 2, vbase, row0 >= last_row0);
  };
  if (C::kStages == 2) {
    __syncthreads();                      // cols[] is complete
    if (n_steps > 0) fetch(cols[0], 0, 0);
  }
  // With one stage the next step's entry of the list is read during this one: the copies are requested right behind the barrier.
  int j_now = 0, j_next = 0;
  if (C::kStages == 1) {
    __syncthreads();                      // cols[] is complete
    j_now = __builtin_amdgcn_readfirstlane(n_steps > 0 ? cols[0] : 0);
  }
  for (int step = 0; step < n_steps; ++step) {
    if (C::kStages == 1) {
      if (step > 0) __syncthreads();      // the stage is free again
      fetch(j_now, step % C::kSub, 0);
      j_next = cols[min(step + 1, n_steps - 1) / C::kSub];
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // my copies of this step have landed
    __syncthreads();                      // everyone's have; everyone is done with the other stage
    if (C::kStages == 2 && step + 1 < n_steps) fetch(cols[(step + 1) / C::kSub], (step + 1) % C::kSub, (step + 1) & 1);
    const bf16 *Ks = lds + (C::kStages == 2 ? (step & 1) : 0) * kStageElems;
    const uint32_t v_at = lds_addr + ((C::kStages == 2 ? (step & 1) : 0) * kStageElems + C::kKElems) * 2;
    const int key0 = (C::kStages == 1 ? j_now : cols[step / C::kSub]) * BLK + (step % C::kSub) * C::kKT;
    if (!VT && key0 + C::kKT > a.L) {
      // (uniform, once at most) keys past the end have P = 0: their V rows must be finite
      const int first = max(0, a.L - key0);
      for (int x = first * (D / 8) + tid; x < C::kKT * (D / 8); x += C::kThreads)
        reinterpret_cast<u32x4 *>(const_cast<bf16 *>(Ks) + C::kKElems)[x] = u32x4{0, 0, 0, 0};
      __syncthreads();
    }
    f32x16 sacc[C::kKT / 32];
#pragma unroll
    for (int mt = 0; mt < C::kKT / 32; ++mt) {
      const bf16 *krow = Ks + (mt * 32 + kr) * D;
      sacc[mt] = zero16;
#pragma unroll
      for (int s = 0; s < D / 16; ++s) {
        bf16x8 ka = *reinterpret_cast<const bf16x8 *>(krow + ((16 * s) ^ kx));
        sacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qreg[s], sacc[mt], 0, 0, 0);
      }
    }
    if (key0 + C::kKT > a.L) {
#pragma unroll
      for (int mt = 0; mt < C::kKT / 32; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          int key = key0 + mt * 32 + 16 * (i >> 3) + 8 * hl + (i & 7);
          if (key >= a.L) sacc[mt][i] = -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < C::kKT / 32; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[mt][i]);
    mx = max_of_halves(mx) * c;
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = fast_exp2(m_run - ((m_new == -INFINITY) ? 0.f : m_new));
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[dm][i] *= alpha;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    float lsum = 0.f;
#pragma unroll
    for (int mt = 0; mt < C::kKT / 32; ++mt) {
      uint32_t pb[8];
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float p0 = fast_exp2(fmaf(sacc[mt][i], c, -m_use));
        const float p1 = fast_exp2(fmaf(sacc[mt][i + 1], c, -m_use));
        lsum += p0 + p1;
        pb[i >> 1] = pack_bf16x2(p0, p1);
      }
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        uint4 praw = make_uint4(pb[4 * tt], pb[4 * tt + 1], pb[4 * tt + 2], pb[4 * tt + 3]);
        bf16x8 pf = *reinterpret_cast<bf16x8 *>(&praw);
#pragma unroll
        for (int dm = 0; dm < D / 32; ++dm) {
          const uint32_t x0 = (uint32_t)(((4 * dm) ^ t_swz<D>(0)) * 16), x1 = (uint32_t)(((4 * dm) ^ t_swz<D>(4)) * 16);
          const uint32_t at = v_at + (uint32_t)((32 * mt + 16 * tt) * D * 2);
          bf16x8 va;
          if (VT) {
            va = *reinterpret_cast<const bf16x8 *>(Ks + C::kKElems + (dm * 32 + cr) * C::kKT + ((16 * (2 * mt + tt)) ^ cx));
          } else {
            const bf16x4 lo = lds_read_tr16((const lds_char *)(uintptr_t)((tr_lane ^ x0) + at));
            const bf16x4 hi = lds_read_tr16((const lds_char *)(uintptr_t)((tr_lane ^ x1) + at + 4 * D * 2));
            va = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          }
          oacc[dm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pf, oacc[dm], 0, 0, 0);
        }
      }
    }
    l_run += lsum;
    if (C::kStages == 1) j_now = __builtin_amdgcn_readfirstlane(j_next);
  }

  const float l_tot = l_run + swap_halves(l_run);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  if (qvalid) {
    bf16 *os = slab_ptr(a.o, a.to, slab, a.H) + (int64_t)qrow * a.to.sL;
    bf16 *ls = a.o_lo ? slab_ptr(a.o_lo, a.to, slab, a.H) + (int64_t)qrow * a.to.sL : nullptr;
#pragma unroll
    for (int dm = 0; dm < D / 32; ++dm) {
      uint32_t w[8], r[8];
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float v0 = oacc[dm][i] * inv, v1 = oacc[dm][i + 1] * inv;
        const uint32_t pk = pack_bf16x2(v0, v1);
        w[i >> 1] = pk;
        r[i >> 1] = pack_bf16x2(v0 - bf16_bits_to_float(pk & 0xffffu),
                                v1 - bf16_bits_to_float(pk >> 16));
      }
      uint4 *dst = reinterpret_cast<uint4 *>(os + dm * 32 + 16 * hl);
      dst[0] = make_uint4(w[0], w[1], w[2], w[3]);
      dst[1] = make_uint4(w[4], w[5], w[6], w[7]);
      if (ls) {
        uint4 *dl = reinterpret_cast<uint4 *>(ls + dm * 32 + 16 * hl);
        dl[0] = make_uint4(r[0], r[1], r[2], r[3]);
        dl[1] = make_uint4(r[4], r[5], r[6], r[7]);
      }
    }
    if (hl == 0)
      a.lse[(int64_t)slab * a.L + qrow] =
          l_tot > 0.f ? m_run * 0.69314718055994530942f + __logf(l_tot) : -INFINITY;
  }
}

// ---------------------------------------------------------------------------------------
// Ping-pong forward.  The workgroup has two groups of BLK/32 wavefronts that own the SAME
// query rows; group g processes the 64-key steps s with s mod 2 = g and keeps its own
// (maximum, row sum, O) partial, merged once at the end.  Time is cut into phases separated by
// workgroup barriers.  In phase p group (p mod 2) is in its MATRIX phase -- P V of step p-2, then
// S^T of step p -- while the other group is in its VECTOR phase -- soft-max of step p-1.  The
// two groups share every SIMD pairwise (wavefronts w and w + BLK/32), so at any time one
// wavefront per SIMD feeds the matrix pipe and the other the vector ALU.
//
// What was measured on MI355X and shaped this kernel:
//  * A wavefront whose next instruction is an MFMA that waits for the matrix pipe keeps the
//    SIMD's issue slot: with equal priorities the older wavefront starves the other one's vector
//    instructions completely.  With the VECTOR wavefront at the higher priority both run: the
//    MFMA stream loses nothing and the vector stream runs at ~80 % of its stand-alone rate.
//  * One 64 x 16 B direct-to-LDS load occupies the issuing wavefront for 65..90 cycles (much
//    more on a low-priority wavefront that competes with a busy one).  The copies of a phase
//    are requested by its vector group (it has the priority and no MFMA stream to hold up), one
//    at a time between blocks of soft-max arithmetic.  Never as a burst behind the barrier.
//  * Scalar bookkeeping shows up directly as idle matrix time (the scalar unit is shared):
//    the phase loop is unrolled so that p mod 4 is a compile-time constant, every LDS address
//    is an immediate, and the column list is turned once into byte offsets of the K and V^T
//    tiles (LDS tables padded by repeats of the last entry, so copies past the last step need
//    no clamping).
// Tiles: four LDS buffers each for K and V^T steps, buffer = step mod 4.  Phase p requests K
// of step p+3 and V of step p+1; both buffers were last read in phase p-1.
// ---------------------------------------------------------------------------------------
template <int BLK, int D>
struct PpCfg {
  static constexpr int kGroupWaves = BLK / 32;
  static constexpr int kWaves = 2 * kGroupWaves;
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kKT = 64;
  static constexpr int kSub = BLK / kKT;
  static constexpr int kKElems = kKT * D;
  static constexpr int kVElems = D * kKT;
  static constexpr int kStages = 4;
  static constexpr int kTabPad = 8;
  static constexpr int kLdsBytes = kStages * (kKElems + kVElems) * 2;
};

template <int N>
using Int = std::integral_constant<int, N>;

// GT: with the pooled (global) tokens of ASA_G appended to every query block's list
template <int BLK, int D, bool GT>
__global__ __launch_bounds__(BLK * 4, (BLK == 64 && D == 64) ? 2 : 1) void fwd_pp_kernel(FwdArgs a) {   // (2: its LDS allows it)
  using C = PpCfg<BLK, D>;
  extern __shared__ __align__(1024) unsigned char smem[];
  bf16 *ldsK = reinterpret_cast<bf16 *>(smem);
  bf16 *ldsV = ldsK + C::kStages * C::kKElems;
  const uint32_t ldsK_addr = ASA_LDS_ADDR_OF(smem);                       // for the copies
  const uint32_t ldsV_addr = ldsK_addr + C::kStages * C::kKElems * 2;
  __shared__ uint32_t tabK[kMaxNb + C::kTabPad], tabV[kMaxNb + C::kTabPad];

  const int slot = xcd_contiguous_work(blockIdx.x, a.n_slabs * a.Nb);
  if (slot < 0) return;
  const int work = a.order ? a.order[slot] : slot;
  const int slab = work / a.Nb;
  if (slab_not_mine(a, slab)) return;
  const int qb = work - slab * a.Nb;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / C::kGroupWaves;       // 0 or 1
  const int wq = wave % C::kGroupWaves;        // which 32 query rows
  const int lane = tid & 63, hl = lane >> 5, n = lane & 31;

  const bf16 *qs = slab_ptr(a.q, a.tq, slab, a.H);
  const bf16 *ks = slab_ptr(a.k, a.tk, slab, a.H);
  const bf16 *vts = a.vt + (int64_t)slab * D * a.Lpad;
  // no index lists: dense attention, every key block in order
  const bool dense = a.row_ptr == nullptr;
  const int t_begin = dense ? 0 : a.row_ptr[slab * (a.Nb + 1) + qb];
  const int n_own_tiles = dense ? a.Nb : a.row_ptr[slab * (a.Nb + 1) + qb + 1] - t_begin;
  // global tokens: Nbg more key blocks that every query block visits, after its own list
  const int n_tiles = n_own_tiles + (GT ? a.Nbg : 0);
  const int n_steps = n_tiles * C::kSub;
  const int n_own_steps = n_own_tiles * C::kSub;
  const uint32_t pitch_bytes = (uint32_t)a.tk.sL * 2u;
  const uint32_t k_tile_bytes = BLK * pitch_bytes;     // host checked: Nb * this < 2^32
  constexpr uint32_t v_tile_bytes = D * BLK * 2;
  {
    const int32_t *g = a.col_idx + (int64_t)slab * a.Nb * a.Nb + t_begin;
    for (int t = tid; t < n_tiles + C::kTabPad; t += C::kThreads) {
      const int tc = t < n_tiles ? t : n_tiles - 1;      // (-1 where the list is empty: no entry to read)
      if (tc >= 0 && tc < n_own_tiles) {
        const uint32_t j = dense ? (uint32_t)tc : (uint32_t)g[tc];
        tabK[t] = j * k_tile_bytes;
        tabV[t] = j * v_tile_bytes;
      } else if (n_tiles > 0) {   // pooled tile tc - n_own_tiles, rows of D elements
        tabK[t] = (uint32_t)(tc - n_own_tiles) * (BLK * D * 2);
        tabV[t] = (uint32_t)(tc - n_own_tiles) * v_tile_bytes;
      } else {
        tabK[t] = 0;
        tabV[t] = 0;
      }
    }
  }
  const int qrow = qb * BLK + wq * 32 + n;
  const bool qvalid = qrow < a.L;
  const int qrow_c = qvalid ? qrow : a.L - 1;
  bf16x8 qreg[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    qreg[s] = *reinterpret_cast<const bf16x8 *>(qs + (int64_t)qrow_c * a.tq.sL + 16 * s + 8 * hl);
  f32x16 oacc[D / 32];
#pragma unroll
  for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dm][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c = a.scale_log2e;

  // Copies: wavefront wq of the requesting group copies a quarter (BLK = 64: half) of a tile.
  RowTileCopy<C::kKT, D, C::kGroupWaves> copy_k;
  ColTileCopy<BLK, D, C::kGroupWaves> copy_v;
  copy_k.init(wq, lane, a.tk.sL);
  copy_v.init(wq, lane);
  // The first kMatrixCopies of a phase's copy requests are made by its matrix group behind its
  // last MFMA (it finishes before the vector group and would wait at the barrier), the rest by
  // the vector group between blocks of its arithmetic.
#ifndef ASA_FWD_MATRIX_COPIES
#define ASA_FWD_MATRIX_COPIES 4   // the K rows (measured 0..4: within 3 % of each other, 4 ahead by 1 %)
#endif
  constexpr int kInstrK = RowTileCopy<C::kKT, D, C::kGroupWaves>::kInstr;
  constexpr int kBatchInstr = kInstrK + ColTileCopy<BLK, D, C::kGroupWaves>::kInstr;
  constexpr int kMatrixCopies = (BLK == 128 && D == 128) ? ASA_FWD_MATRIX_COPIES : 0;
  static_assert(kBatchInstr == 4 || kBatchInstr == 8 || kBatchInstr == 16, "unexpected copy size");
  const int kr = kappa(n), cr = rho(n);
  const int kx = (hl ^ k_swz<D>(kr)) * 8, cx = (hl ^ v_swz(cr)) * 8;
  const int k_frag0 = kr * D + kx;          // element offset of my K fragment 0 in a 32-key group
  const int v_frag0 = cr * C::kKT + cx;     // of my V^T fragment 0 in a 32-channel group
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // Only the last key block can be ragged.  Per 64-key half of a block: the table entry that
  // means "this step reaches past L" (or an impossible value if that half of the last block is
  // complete).
  const int last_row0 = (a.Nb - 1) * BLK;
  uint32_t k_tail[C::kSub], v_tail[C::kSub];
  const char *k_base[C::kSub], *v_base[C::kSub];
#pragma unroll
  for (int sb = 0; sb < C::kSub; ++sb) {
    const bool ragged = last_row0 + sb * C::kKT + C::kKT > a.L;
    k_tail[sb] = ragged ? (uint32_t)(a.Nb - 1) * k_tile_bytes : 0xFFFFFFFFu;
    v_tail[sb] = ragged ? (uint32_t)(a.Nb - 1) * v_tile_bytes : 0xFFFFFFFFu;
    k_base[sb] = reinterpret_cast<const char *>(ks) + (int64_t)sb * C::kKT * pitch_bytes;
    v_base[sb] = reinterpret_cast<const char *>(vts) + sb * C::kKT * 2;
  }
  // pooled keys / values of this slab (rows of D elements; tiles like V's)
  const char *kg_slab = reinterpret_cast<const char *>(a.kg) + (int64_t)slab * a.Nbg * BLK * D * 2;
  const char *vg_slab = reinterpret_cast<const char *>(a.vgt) + (int64_t)slab * a.Nbg * D * BLK * 2;
  // is step s one over pooled tokens?  (steps past the end repeat the last step)
  auto pooled_step = [&](int step) __attribute__((always_inline)) {
    return GT && (step < n_steps ? step : n_steps - 1) >= n_own_steps;
  };

  __syncthreads();   // tables complete
  // Before phase 0: K of steps 0, 1, 2 and V of step 0 (group 0: K(0), K(2); group 1: K(1),
  // V(0)).  Any of the K tiles may be the ragged one.
  {
    const char *kb = reinterpret_cast<const char *>(ks);
    auto k_step = [&](int step) __attribute__((always_inline)) {
      const int j = (int)(__builtin_amdgcn_readfirstlane(tabV[step / C::kSub]) / v_tile_bytes);
      const int r = j * BLK + (step % C::kSub) * C::kKT;
      if (pooled_step(step)) {
#pragma unroll
        for (int i = 0; i < kInstrK; ++i)   // (with pooled tokens the rows of K are D elements apart, like theirs)
          lds_dma16_sv(kg_slab + (int64_t)r * (D * 2), copy_k.off[i],
                       ldsK_addr + step * C::kKElems * 2 + copy_k.lds_chunk(i));
      } else {
        copy_k.issue_at_ragged(ldsK_addr + step * C::kKElems * 2, kb + (int64_t)r * pitch_bytes, a.L - 1 - r);
      }
    };
    if (grp == 0) {
      k_step(0);
      k_step(2);
    } else {
      k_step(1);
      copy_v.issue_at(ldsV_addr, (pooled_step(0) ? vg_slab : v_base[0]) + __builtin_amdgcn_readfirstlane(tabV[0]));
    }
  }
  // Table entries of the copies of phase 0 (K of step 3, V of step 1) and the V entries of the
  // three phases before, which tell the soft-max whether its step is the ragged one.
  uint32_t ek_next = tabK[3 / C::kSub], ev_next = tabV[1 / C::kSub];
  uint32_t ek_cur = 0, ev_cur = tabV[0], ev_last = 0xFFFFFFFFu, ev_older = 0xFFFFFFFFu;
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)

  f32x16 sacc[C::kKT / 32];
  uint32_t pb[(C::kKT / 32) * 8];
#pragma unroll
  for (int mt = 0; mt < C::kKT / 32; ++mt) sacc[mt] = zero16;
#pragma unroll
  for (int e = 0; e < (C::kKT / 32) * 8; ++e) pb[e] = 0;

  // Start of phase p (R = p mod 4).  During phase p, K of step p+3 and V of step p+1 are
  // requested (their buffers were last read in phase p-1); every wavefront requests the same
  // number of loads per two phases.  Data needed in phase p -- K(p), V(p-2) -- was requested
  // during phase p-3: "all of my copies but the newest kBatchInstr have landed" on every
  // wavefront, followed by the barrier, makes it visible to all.
  int phase_now = 0;   // the phase in progress, set by phase_sync
  auto phase_sync = [&](int p) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    if (kBatchInstr == 4) __builtin_amdgcn_s_waitcnt(0x0F74);
    else if (kBatchInstr == 8) __builtin_amdgcn_s_waitcnt(0x0F78);
    else __builtin_amdgcn_s_waitcnt(0x4F70);   // vmcnt(16): low bits 0, high bits (15:14) 1
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    phase_now = p;
    ek_cur = __builtin_amdgcn_readfirstlane(ek_next);
    ev_older = ev_last;
    ev_last = ev_cur;
    ev_cur = __builtin_amdgcn_readfirstlane(ev_next);
    ek_next = tabK[(p + 4) / C::kSub];
    ev_next = tabV[(p + 2) / C::kSub];
    __builtin_amdgcn_sched_barrier(0);
  };

  // The K copy of this phase: wave-uniform base and per-lane offsets.  Normally the offsets are
  // the tile's own; for the one ragged step they are bent back to the last row (rare branch).
  const char *kdma_base = nullptr, *vdma_base = nullptr;
  uint32_t kdma_off[kInstrK];
  auto dma_prepare = [&](auto r_tag) __attribute__((always_inline)) {
    constexpr int sb = (decltype(r_tag)::value + 1) % C::kSub;
    kdma_base = k_base[sb] + ek_cur;
    vdma_base = v_base[sb] + ev_cur;
#pragma unroll
    for (int i = 0; i < kInstrK; ++i) kdma_off[i] = copy_k.off[i];
    if (GT) {   // K of step p+3, V of step p+1 may be pooled tiles (rows of D elements)
      if (pooled_step(phase_now + 1)) vdma_base = vg_slab + sb * C::kKT * 2 + ev_cur;
      if (pooled_step(phase_now + 3)) {
        // the host admits pooled tokens only where K's rows are D elements apart, like theirs:
        // the per-lane offsets are the same
        kdma_base = kg_slab + sb * C::kKT * (D * 2) + ek_cur;
        return;   // pooled rows are padded to whole blocks: never ragged
      }
    }
    if (ek_cur == k_tail[sb]) {
      int lim = a.L - 1 - (last_row0 + sb * C::kKT);
      if (lim < 0) {
        kdma_base += (int64_t)lim * pitch_bytes;
        lim = 0;
      }
#pragma unroll
      for (int i = 0; i < kInstrK; ++i) {
        const int row = copy_k.row_of(i);
        if (row > lim) kdma_off[i] -= (uint32_t)(row - lim) * pitch_bytes;
      }
    }
  };
  // i-th load of this wavefront's share of the batch of phase R: K of step R+3, V of step R+1
  auto dma_one = [&](auto r_tag, int i) __attribute__((always_inline)) {
    constexpr int R = decltype(r_tag)::value;
    if (i < kInstrK)
      lds_dma16_sv<GT>(kdma_base, kdma_off[i], ldsK_addr + ((R + 3) & 3) * C::kKElems * 2 + copy_k.lds_chunk(i));
    else
      copy_v.template issue_one_at<GT>(i - kInstrK, ldsV_addr + ((R + 1) & 3) * C::kVElems * 2, vdma_base);
  };
  // (idle phases) matrix_slot: this group is the phase's matrix group
  auto dma_idle = [&](auto r_tag, bool matrix_slot) __attribute__((always_inline)) {
    const int first = matrix_slot ? 0 : kMatrixCopies, last = matrix_slot ? kMatrixCopies : kBatchInstr;
    if (first < last) {
      dma_prepare(r_tag);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kBatchInstr; ++i)
        if (i >= first && i < last) dma_one(r_tag, i);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // MATRIX phase p (R = p mod 4): P V of step p-2 followed by S^T of step p.  One wavefront
  // per SIMD runs it at a time, so the LDS fragment reads are software-pipelined kDepth tile
  // products ahead of the MFMA that consumes them.  Runs at the low priority.
  constexpr int kNPv = (C::kKT / 16) * (D / 32);
  constexpr int kNS = (D / 16) * (C::kKT / 32);
  constexpr int kDepth = 6, kRing = kDepth + 1;
  auto do_matrix = [&](auto r_tag, auto with_pv, auto with_s) __attribute__((always_inline)) {
    constexpr int R = decltype(r_tag)::value;
    constexpr bool kPv = decltype(with_pv)::value, kS = decltype(with_s)::value;
    constexpr int n0 = kPv ? 0 : kNPv, n1 = kS ? kNPv + kNS : kNPv;
    const bf16 *Vs = ldsV + ((R + 2) & 3) * C::kVElems;
    const bf16 *Ks = ldsK + R * C::kKElems;
    bf16x8 ring[kRing];
    int zero = 0;
    if (GT) asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int i = n0; i < n1 + kDepth; ++i) {
      if (i < n1) {
        // fragment addresses are formed here from two per-lane bases (the swizzle is an XOR of
        // the low address bits, so (base + x) ^ (16 s) = base + (x ^ 16 s)); `zero` keeps the
        // compiler from hoisting twelve loop-invariant address registers out of the loop
        // (only the pooled-token variant, which is short of registers; the other one keeps the
        // twelve addresses in registers and saves the XORs)
        if (i < kNPv) {
          const int t = i / (D / 32), dm = i % (D / 32);
          if (GT)
            ring[i % kRing] = *reinterpret_cast<const bf16x8 *>(Vs + dm * 32 * C::kKT + ((v_frag0 ^ (16 * t)) ^ zero));
          else
            ring[i % kRing] = *reinterpret_cast<const bf16x8 *>(Vs + (dm * 32 + cr) * C::kKT + ((16 * t) ^ cx));
        } else {
          const int e = i - kNPv, sk = e / (C::kKT / 32), mt = e % (C::kKT / 32);
          if (GT)
            ring[i % kRing] = *reinterpret_cast<const bf16x8 *>(Ks + mt * 32 * D + ((k_frag0 ^ (16 * sk)) ^ zero));
          else
            ring[i % kRing] = *reinterpret_cast<const bf16x8 *>(Ks + (mt * 32 + kr) * D + ((16 * sk) ^ kx));
        }
      }
      const int c_i = i - kDepth;
      if (c_i >= n0) {
        if (c_i < kNPv) {
          const int t = c_i / (D / 32), dm = c_i % (D / 32);
          const u32x4 praw = {pb[4 * t], pb[4 * t + 1], pb[4 * t + 2], pb[4 * t + 3]};
          oacc[dm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[c_i % kRing], __builtin_bit_cast(bf16x8, praw),
                                                            oacc[dm], 0, 0, 0);
        } else {
          const int e = c_i - kNPv, sk = e / (C::kKT / 32), mt = e % (C::kKT / 32);
          sacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[c_i % kRing], qreg[sk],
                                                            sk == 0 ? zero16 : sacc[mt], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(3);
    if (kMatrixCopies > 0) {
      // all MFMAs of the phase are issued: this wavefront's share of the copy requests
      dma_prepare(r_tag);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kMatrixCopies; ++i) dma_one(r_tag, i);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // VECTOR phase p: online soft-max of step p-1 (RX = that step mod 4), whose S^T is in sacc;
  // leaves bf16 P in pb.  Runs at the high priority and requests the phase's copies, an eighth
  // of them at a time between blocks of arithmetic.
  auto do_x = [&](auto rx_tag) __attribute__((always_inline)) {
    constexpr int sb = decltype(rx_tag)::value % C::kSub;
    const Int<(decltype(rx_tag)::value + 1) & 3> r_tag{};   // the phase this runs in
    constexpr int kPortion = kBatchInstr / 8 > 0 ? kBatchInstr / 8 : 1;
    int next_copy = kMatrixCopies;
    auto request = [&](int n_instr) __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < n_instr; ++e)
        if (next_copy < kBatchInstr) dma_one(r_tag, next_copy++);
      __builtin_amdgcn_sched_barrier(0);
    };
    __builtin_amdgcn_s_setprio(3);
    if (kMatrixCopies < kBatchInstr) dma_prepare(r_tag);
    float bias = 0.f;   // added to the scaled scores of pooled keys (log2 domain)
    if (GT && pooled_step(phase_now - 1)) {
      bias = a.bias_log2;
      const int key0 = (int)(ev_older / v_tile_bytes) * BLK + sb * C::kKT;
      if (key0 + C::kKT > a.Lg) {
#pragma unroll
        for (int mt = 0; mt < C::kKT / 32; ++mt)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            int key = key0 + mt * 32 + 16 * (i >> 3) + 8 * hl + (i & 7);
            if (key >= a.Lg) sacc[mt][i] = -INFINITY;
          }
      }
    } else if (ev_older == v_tail[sb]) {
      const int key0 = last_row0 + sb * C::kKT;
#pragma unroll
      for (int mt = 0; mt < C::kKT / 32; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          int key = key0 + mt * 32 + 16 * (i >> 3) + 8 * hl + (i & 7);
          if (key >= a.L) sacc[mt][i] = -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < C::kKT / 32; ++mt)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[mt][i]);
    request(kPortion);
    mx = max_of_halves(mx) * c + bias;
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = fast_exp2(m_run - ((m_new == -INFINITY) ? 0.f : m_new));
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[dm][i] *= alpha;
    }
    request(kPortion);
    const float m_use = ((m_run == -INFINITY) ? 0.f : m_run) - bias;
    float lsum = 0.f;
#pragma unroll
    for (int mt = 0; mt < C::kKT / 32; ++mt) {
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        if (i == 4 || i == 8 || i == 12) request(kPortion);
        const float p0 = fast_exp2(fmaf(sacc[mt][i], c, -m_use));
        const float p1 = fast_exp2(fmaf(sacc[mt][i + 1], c, -m_use));
        lsum += p0 + p1;
        pb[mt * 8 + (i >> 1)] = pack_bf16x2(p0, p1);
      }
    }
    l_run += lsum;
    request(kBatchInstr);   // whatever is left
  };

  const std::true_type yes{};
  const std::false_type no{};
  // Group g owns steps g, g+2, ...; its k-th own step is step (= phase) 2k + g.
  auto run_group = [&](auto g_tag) __attribute__((always_inline)) {
    constexpr int G = decltype(g_tag)::value;
    using R0 = Int<G>;
    using R2 = Int<(G + 2) & 3>;
    int p = 0;
    if (G == 1) { phase_sync(p); dma_idle(Int<0>{}, false); ++p; }   // group 0's matrix slot
    const int n_own = n_steps > G ? (n_steps - G + 1) / 2 : 0;
    if (n_own > 0) {
      phase_sync(p); do_matrix(R0{}, no, yes); ++p;
      phase_sync(p); do_x(R0{}); ++p;
      int k = 1;
      for (; k + 1 < n_own; k += 2) {
        phase_sync(p); do_matrix(R2{}, yes, yes); ++p;
        phase_sync(p); do_x(R2{}); ++p;
        phase_sync(p); do_matrix(R0{}, yes, yes); ++p;
        phase_sync(p); do_x(R0{}); ++p;
      }
      if (k < n_own) {
        phase_sync(p); do_matrix(R2{}, yes, yes); ++p;
        phase_sync(p); do_x(R2{}); ++p;
        phase_sync(p); do_matrix(R0{}, yes, no); ++p;
      } else {
        phase_sync(p); do_matrix(R2{}, yes, no); ++p;
      }
    }
    // the other group may still have phases to run: keep the barriers and copies in step
    for (; p < n_steps + 2; ++p) {
      switch (p & 3) {
        case 0: phase_sync(p); dma_idle(Int<0>{}, G == 0); break;
        case 1: phase_sync(p); dma_idle(Int<1>{}, G == 1); break;
        case 2: phase_sync(p); dma_idle(Int<2>{}, G == 0); break;
        default: phase_sync(p); dma_idle(Int<3>{}, G == 1); break;
      }
    }
  };
  if (grp == 0) run_group(Int<0>{});
  else run_group(Int<1>{});

  // ---- merge the two groups' partials (group 1 -> LDS -> group 0), then write out
  __builtin_amdgcn_s_waitcnt(0x0F70);   // stray copies must land before the buffers are reused
  __syncthreads();
  f32x4 *xbuf = reinterpret_cast<f32x4 *>(smem);          // [4 * D/32][BLK * 2] f32x4
  float *xm = reinterpret_cast<float *>(xbuf + 4 * (D / 32) * (BLK * 2));
  float *xl = xm + BLK * 2;
  const int xslot = wq * 64 + lane;
  float l_half = l_run + swap_halves(l_run);
  if (grp == 1) {
#pragma unroll
    for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 v = {oacc[dm][4 * q4], oacc[dm][4 * q4 + 1], oacc[dm][4 * q4 + 2], oacc[dm][4 * q4 + 3]};
        xbuf[(dm * 4 + q4) * (BLK * 2) + xslot] = v;
      }
    xm[xslot] = m_run;
    xl[xslot] = l_half;
  }
  __syncthreads();
  if (grp == 1) return;
  {
    const float m_o = xm[xslot], l_o = xl[xslot];
    const float m_all = fmaxf(m_run, m_o);
    const float ms = (m_all == -INFINITY) ? 0.f : m_all;
    const float fa = fast_exp2(m_run - ms), fb = fast_exp2(m_o - ms);
    l_half = l_half * fa + l_o * fb;
#pragma unroll
    for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4 v = xbuf[(dm * 4 + q4) * (BLK * 2) + xslot];
#pragma unroll
        for (int e = 0; e < 4; ++e) oacc[dm][4 * q4 + e] = oacc[dm][4 * q4 + e] * fa + v[e] * fb;
      }
    m_run = m_all;
  }
  const float l_tot = l_half;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  if (qvalid) {
    bf16 *os = slab_ptr(a.o, a.to, slab, a.H) + (int64_t)qrow * a.to.sL;
    bf16 *ls = a.o_lo ? slab_ptr(a.o_lo, a.to, slab, a.H) + (int64_t)qrow * a.to.sL : nullptr;
#pragma unroll
    for (int dm = 0; dm < D / 32; ++dm) {
      uint32_t w[8], r[8];
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float v0 = oacc[dm][i] * inv, v1 = oacc[dm][i + 1] * inv;
        const uint32_t pk = pack_bf16x2(v0, v1);
        w[i >> 1] = pk;
        r[i >> 1] = pack_bf16x2(v0 - bf16_bits_to_float(pk & 0xffffu),
                                v1 - bf16_bits_to_float(pk >> 16));
      }
      uint4 *dst = reinterpret_cast<uint4 *>(os + dm * 32 + 16 * hl);
      dst[0] = make_uint4(w[0], w[1], w[2], w[3]);
      dst[1] = make_uint4(w[4], w[5], w[6], w[7]);
      if (ls) {
        uint4 *dl = reinterpret_cast<uint4 *>(ls + dm * 32 + 16 * hl);
        dl[0] = make_uint4(r[0], r[1], r[2], r[3]);
        dl[1] = make_uint4(r[4], r[5], r[6], r[7]);
      }
    }
    if (hl == 0)
      a.lse[(int64_t)slab * a.L + qrow] =
          l_tot > 0.f ? m_run * 0.69314718055994530942f + __logf(l_tot) : -INFINITY;
  }
}

// ---------------------------------------------------------------------------------------
// Pipelined forward: the software pipeline of the backward kernels (see asa_bwd.hip).  One workgroup per
// query block, one wavefront per 32 query rows, tiles of 32 keys.  In iteration t a wavefront
// computes S^T of tile t + 1 and adds P V of tile t - 1, and between those MFMAs turns S^T of tile t
// into P; O is rescaled at the end of an iteration whose rows found a larger logit (the maximum is
// never allowed to lag behind, as in the other kernels).  The V operand is gathered from V's rows by the
// transposing LDS read: no transposed copy of V.  K and V have four LDS stages each.
//
// Bound: at large sizes the direct-to-LDS copies (every wavefront of a workgroup requests its share
// at the same point, ~75 cycles each, twice as many per product as in the backward: without them
// the block 128 / d 128 loop runs 24 % faster) and, at d = 64, vector issue.  Its place is where a
// wavefront's own speed counts: few workgroups, or shapes whose lock-step workgroup leaves the SIMDs
// idle (launch_fwd_t has the figures).
// ---------------------------------------------------------------------------------------
template <int BLK, int D, int KS>
struct PipeCfg {
  static constexpr int kWaves = BLK / 32;              // of a group
  static constexpr int kThreads = kWaves * 64;         // of a group
  static constexpr int kST = 32;                       // keys per tile
  static constexpr int kSub = BLK / kST / KS;          // tiles of a block that a group takes
  static constexpr int kStages = 4;
  static constexpr int kTile = kST * D * 2;            // bytes of one row tile
  static constexpr int kLds = 2 * kStages * kTile;     // K stages, then V stages
  static constexpr int kWavesPerSimd = (BLK == 64 && D == 128) ? 1 : 2;
};

// GT: with the pooled (global) tokens of ASA_G appended to every query block's list
// KS: groups of wavefronts that share a row.  Two groups walk the same list, each with tiles in LDS of its own and half
// of every block's keys (so both have as many tiles, and one list of any length is two of half the length); their O,
// maxima and sums are put together at the end.  A row takes half as long, and a compute unit holds half as many rows: pipe_in_two says
// where that pays.  (Two rows to such a workgroup where rows are short, so that only the long ones are split: the groups
// wait for one another at every barrier, 10-18 % slower than two workgroups.)
template <int BLK, int D, bool GT, int KS>
__global__ __launch_bounds__(BLK * 2 * KS, (PipeCfg<BLK, D, KS>::kWavesPerSimd)) void fwd_pipe_kernel(FwdArgs a) {
  using C = PipeCfg<BLK, D, KS>;
  extern __shared__ __align__(1024) unsigned char smem[];
  __shared__ int cols[kMaxNb];
  constexpr int kStage = C::kTile, kVBase = C::kStages * C::kTile;
  constexpr int kPooled = 1 << 30;             // flag of an entry of cols[]: a block of pooled tokens

  const int slot = xcd_contiguous_work(blockIdx.x, a.n_slabs * a.Nb);
  if (slot < 0) return;
  const int work = a.order ? a.order[slot] : slot;
  const int slab = work / a.Nb;
  if (slab_not_mine(a, slab)) return;
  const int qb = work - slab * a.Nb;
  const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / C::kThreads);
  const int tid = KS == 1 ? threadIdx.x : threadIdx.x % C::kThreads;      // in the group
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, hl = lane >> 5, n = lane & 31;

  const bf16 *qs = slab_ptr(a.q, a.tq, slab, a.H);
  const bf16 *ks = slab_ptr(a.k, a.tk, slab, a.H);
  const bf16 *vs = slab_ptr(a.v, a.tv, slab, a.H);
  const bool dense = a.row_ptr == nullptr;   // no index lists: dense attention, every key block in order
  const int t_begin = dense ? 0 : a.row_ptr[slab * (a.Nb + 1) + qb];
  const int n_own_blocks = dense ? a.Nb : a.row_ptr[slab * (a.Nb + 1) + qb + 1] - t_begin;
  const int n_blocks = n_own_blocks + (GT ? a.Nbg : 0);   // pooled blocks come after the row's own list
  {
    const int32_t *g = a.col_idx + (int64_t)slab * a.Nb * a.Nb + t_begin;
    for (int t = threadIdx.x; t < n_blocks; t += C::kThreads * KS)
      cols[t] = t >= n_own_blocks ? (t - n_own_blocks) | kPooled : (dense ? t : g[t]);
  }
  const bf16 *kgs = reinterpret_cast<const bf16 *>(a.kg) + (int64_t)slab * a.Nbg * BLK * D;
  const bf16 *vgs = reinterpret_cast<const bf16 *>(a.vg) + (int64_t)slab * a.Nbg * BLK * D;

  const int qrow = qb * BLK + wave * 32 + n;
  const bool qvalid = qrow < a.L;
  const int qrow_c = qvalid ? qrow : a.L - 1;
  bf16x8 qreg[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    qreg[s] = *reinterpret_cast<const bf16x8 *>(qs + (int64_t)qrow_c * a.tq.sL + 16 * s + 8 * hl);
  f32x16 oacc[D / 32];
#pragma unroll
  for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dm][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c = a.scale_log2e;

  using Copy = TrTileCopy<C::kST, D, C::kWaves>;
  Copy copy_k, copy_v, copy_p;
  // Running copies where one wavefront per SIMD issues everything (block 64 / d 128: 1.05x); with two of them the branches
  // they bring cost more (d 64 0.88-1.0x, block 128 / d 128 0.97-1.01x).
  constexpr bool kRun = !GT && C::kWavesPerSimd == 1;
  using RunCopy = RunningTileCopy<C::kST, D, C::kWaves>;
  RunCopy run_k, run_v;
  LastTileWatch watch_k, watch_v;
  if constexpr (!kRun) {
    copy_k.init(wave, lane, a.tk.sL, a.L);
    copy_v.init(wave, lane, a.tv.sL, a.L);
  } else {
    run_k.init(wave, lane, ks, a.tk.sL, a.L);
    run_v.init(wave, lane, vs, a.tv.sL, a.L);
    watch_k.init(RunCopy::last_row0(a.L));
    watch_v.init(RunCopy::last_row0(a.L));
  }
  constexpr int kI = Copy::kInstr;
  const int last_row0 = Copy::last_row0(a.L);
  if (GT) copy_p.init(wave, lane, D, C::kST);   // pooled rows: D elements apart, never ragged

  unsigned char *group_smem = smem + group * C::kLds;
  const uint32_t smem_addr = ASA_LDS_ADDR_OF(smem) + (uint32_t)(group * C::kLds);
  const int group_key = group * (BLK / KS);    // my part of a block
  // A fragments of S^T = K Q^T: row kappa(n) of the 32 keys (see asa_bwd.hip)
  const int kr = kappa(n);
  uint32_t row_at[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    row_at[s] = (smem_addr + (uint32_t)(kr * D * 2 + (hl ^ t_swz<D>(kr)) * 16)) ^ (uint32_t)(32 * s);
  // transposed A fragments "32 channels x 16 keys" of O^T += V^T P^T
  const int tr_i = lane & 15, tr_w = tr_i & 3, tr_j = tr_i >> 2, tr_b = (lane >> 4) & 1;
  const uint32_t tr_lane = smem_addr + kVBase + tr_piece<D>(8 * hl + tr_j, 16 * (tr_w & 1) + 8 * tr_b + 4 * (tr_w >> 1));
  uint32_t tr_at[2 * (D / 32)];
#pragma unroll
  for (int dm = 0; dm < D / 32; ++dm) {
    tr_at[2 * dm] = tr_lane ^ (uint32_t)(((4 * dm) ^ t_swz<D>(0)) * 16);
    tr_at[2 * dm + 1] = tr_lane ^ (uint32_t)(((4 * dm) ^ t_swz<D>(4)) * 16);
  }
  const int n_it = n_blocks * C::kSub;

  // The tile whose K rows are copied next, and the tile before it, whose V rows are
  int entry_v = 0, entry_at = 0, key_c = 0, key_v = 0;
  bool last_k = false, last_v = false, pooled_k = false, pooled_v = false;
  const char *base_k = nullptr, *base_v = nullptr, *base_v_next = nullptr;
  auto fetch_entry = [&]() __attribute__((always_inline)) {
    entry_v = cols[entry_at < n_blocks ? entry_at : n_blocks - 1];
    ++entry_at;
  };
  // (new_block_v: of the tile whose V rows are copied)
  auto next_tile = [&](auto part_tag, auto new_block_tag, auto new_block_v_tag) __attribute__((always_inline)) {
    constexpr int part = decltype(part_tag)::value;
    constexpr bool new_block = decltype(new_block_tag)::value, new_block_v = decltype(new_block_v_tag)::value;
    if constexpr (part == 0) {
      last_v = last_k;
      pooled_v = pooled_k;
      base_v = base_v_next;
      key_v = key_c;
      if constexpr (new_block) {
        const int e = __builtin_amdgcn_readfirstlane(entry_v);
        if (GT) pooled_k = (e & kPooled) != 0;
        key_c = (GT ? e & (kPooled - 1) : e) * BLK + group_key;
      } else {
        key_c += C::kST;
      }
      last_k = key_c >= last_row0;
    } else if constexpr (kRun) {
      if constexpr (part == 1) {
        if constexpr (new_block) run_k.block(key_c);
        else run_k.step();
        watch_k.tile(key_c, a.L, run_k);
      } else {
        if constexpr (new_block_v) run_v.block(key_v);
        else run_v.step();
        watch_v.tile(key_v, a.L, run_v);
      }
    } else if constexpr (part == 1) {
      base_k = reinterpret_cast<const char *>(ks) + (int64_t)min(key_c, last_row0) * (a.tk.sL * 2);
      if (GT) base_k = pooled_k ? reinterpret_cast<const char *>(kgs) + (int64_t)key_c * (D * 2) : base_k;
    } else {
      base_v_next = reinterpret_cast<const char *>(vs) + (int64_t)min(key_c, last_row0) * (a.tv.sL * 2);
      if (GT) base_v_next = pooled_k ? reinterpret_cast<const char *>(vgs) + (int64_t)key_c * (D * 2) : base_v_next;
    }
  };
  uint64_t started = 0;
  auto copy_k_one = [&](auto i_tag, uint32_t st) __attribute__((always_inline)) {
    constexpr int i = decltype(i_tag)::value;
    if constexpr (GT) {
      lds_dma16_sv(base_k, pooled_k ? copy_p.off[i] : (last_k ? copy_k.off_last[i] : copy_k.off[i]), st + copy_k.lds0 + i * 1024);
    } else if constexpr (!kRun) {
      copy_k.issue_one(i, st, base_k, last_k);
    } else {
      if constexpr (i == 0) started = run_k.start(st);
      run_k.template load<i>(started);
    }
  };
  auto copy_v_one = [&](auto i_tag, uint32_t st) __attribute__((always_inline)) {
    constexpr int i = decltype(i_tag)::value;
    if constexpr (GT) {
      lds_dma16_sv(base_v, pooled_v ? copy_p.off[i] : (last_v ? copy_v.off_last[i] : copy_v.off[i]), st + kVBase + copy_v.lds0 + i * 1024);
    } else if constexpr (!kRun) {
      copy_v.issue_one(i, st + kVBase, base_v, last_v);
    } else {
      if constexpr (i == 0) started = run_v.start(st + kVBase);
      run_v.template load<i>(started);
    }
  };
  // copies from .. from + n - 1 of a turn's: K's to stage `to_k`, then V's to stage `to_v`
  auto copy_some = [&](auto from_tag, auto n_tag, uint32_t to_k, uint32_t to_v) __attribute__((always_inline)) {
    constexpr int from = decltype(from_tag)::value;
    [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int i = from + I;
        if constexpr (i < kI) copy_k_one(std::integral_constant<int, i>{}, to_k);
        else copy_v_one(std::integral_constant<int, i - kI>{}, to_v);
      }(), ...);
    }(std::make_integer_sequence<int, decltype(n_tag)::value>{});
  };
  // The block of the tile in work, for the masks of the last block and the bias of pooled keys
  int cur_v = 0, cur_at = 0, key_t = 0, key_end = 0;
  float bias = 0.f;
  auto fetch_current = [&]() __attribute__((always_inline)) {
    cur_v = cols[cur_at < n_blocks ? cur_at : n_blocks - 1];
    ++cur_at;
  };
  auto next_current = [&](auto new_block_tag) __attribute__((always_inline)) {
    if constexpr (decltype(new_block_tag)::value) {
      const int e = __builtin_amdgcn_readfirstlane(cur_v);
      key_t = (GT ? e & (kPooled - 1) : e) * BLK + group_key;
      const bool pooled = GT && (e & kPooled) != 0;
      key_end = pooled ? a.Lg : a.L;             // keys at or past it do not exist
      if (GT) bias = pooled ? a.bias_log2 : 0.f;
    } else {
      key_t += C::kST;
    }
  };

  constexpr int kNS = D / 16, kNV = 2 * (D / 32), kN = kNS + kNV;
  constexpr int kRing = 8, kDepth = 6;
  static_assert(kN % kRing == 0, "the ring continues across iterations");
  constexpr int kBar = kNS < kN - kDepth ? kNS : kN - kDepth;   // the barrier comes before this product
  bf16x8 ring[kRing];
  auto read_row = [&](auto e_tag, auto stage_tag) __attribute__((always_inline)) {
    constexpr int e = decltype(e_tag)::value;
    ring[e % kRing] = lds_read<bf16x8>(row_at[e] + (uint32_t)(decltype(stage_tag)::value * kStage));
  };
  auto read_tr = [&](auto f_tag, auto stage_tag) __attribute__((always_inline)) {
    constexpr int f = decltype(f_tag)::value, dm = f % (D / 32), tt = f / (D / 32);
    constexpr int at = decltype(stage_tag)::value * kStage + 16 * tt * D * 2;
    const bf16x4 lo = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm] + (uint32_t)at));
    const bf16x4 hi = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm + 1] + (uint32_t)(at + 4 * D * 2)));
    ring[(kNS + f) % kRing] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 s0, s1;
  uint32_t pb[8];                        // bf16 P of the tile before the one in work
#pragma unroll
  for (int i = 0; i < 8; ++i) pb[i] = 0;
  auto pv = [&](auto f_tag) __attribute__((always_inline)) {
    constexpr int f = decltype(f_tag)::value, dm = f % (D / 32), tt = f / (D / 32);
    const u32x4 raw = {pb[4 * tt], pb[4 * tt + 1], pb[4 * tt + 2], pb[4 * tt + 3]};
    oacc[dm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[(kNS + f) % kRing], __builtin_bit_cast(bf16x8, raw), oacc[dm], 0, 0, 0);
  };

  auto body = [&](auto u_tag, f32x16 &sc, f32x16 &sn) __attribute__((always_inline)) {
    constexpr int U = decltype(u_tag)::value;        // tile index mod 4
    using StK1 = std::integral_constant<int, (U + 1) & 3>;
    using StK2 = std::integral_constant<int, (U + 2) & 3>;
    using StVp = std::integral_constant<int, (U + 3) & 3>;   // V rows of tile t - 1
    constexpr bool kNewBlock = (U + C::kStages - 1) % C::kSub == 0;   // of the K tile copied here
    constexpr bool kNextNewBlock = (U + C::kStages) % C::kSub == 0;
    constexpr bool kNewBlockV = (U + C::kStages - 2) % C::kSub == 0;  // of the V tile copied here
    if (key_t + C::kST > key_end) {                  // (uniform, rare) keys past the end
      const int left = key_end - key_t - 8 * hl;     // (compared with constants: nothing to keep in registers)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (16 * (i >> 3) + (i & 7) >= left) sc[i] = -INFINITY;
      // their V rows (in LDS since the last barrier, read after the next one) must be finite
      u32x4 *z = reinterpret_cast<u32x4 *>(group_smem + kVBase + U * kStage);
      for (int x = max(0, key_end - key_t) * (D / 8) + tid; x < kStage / 16; x += C::kThreads) z[x] = u32x4{0, 0, 0, 0};
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    }
    uint32_t pn[8];
    float mx = -INFINITY, m_use = 0.f, alpha = 1.f, sum0 = 0.f, sum1 = 0.f;
    bool grew = false;
    constexpr int kFirst = kN == 16 ? 5 : 2;         // slot of the first exponentials
    __builtin_amdgcn_sched_barrier(0);
    [&]<int... X>(std::integer_sequence<int, X...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int x = X;
        if constexpr (x == kBar) {
          // K of tile t + 2 and V of tile t + 1 have landed (everyone's copies).  V of tile t landed one
          // barrier earlier: the zeros that a ragged tile writes into it above rely on that.
          __builtin_amdgcn_s_waitcnt(0x0F70);
          asm volatile("s_barrier" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (x + kDepth < kNS) read_row(std::integral_constant<int, x + kDepth>{}, StK1{});
        else if constexpr (x + kDepth < kN) read_tr(std::integral_constant<int, x + kDepth - kNS>{}, StVp{});
        else if constexpr (x + kDepth - kN < kNS) read_row(std::integral_constant<int, x + kDepth - kN>{}, StK2{});
        else read_tr(std::integral_constant<int, x + kDepth - kN - kNS>{}, std::integral_constant<int, U>{});
        if constexpr (x < kNS)
          sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[x % kRing], qreg[x], x == 0 ? zero16 : sn, 0, 0, 0);
        else
          pv(std::integral_constant<int, x - kNS>{});
        // row maximum of tile t
        if constexpr (x < kFirst - 1) {
          constexpr int nm = kFirst >= 5 ? kFirst - 2 : 1;     // slots that take part
          constexpr int i0 = x < nm ? x * 16 / nm : 16, i1 = x < nm ? (x + 1) * 16 / nm : 16;
#pragma unroll
          for (int i = i0; i < i1; ++i) mx = fmaxf(mx, sc[i]);
        }
        if constexpr (x == (kFirst >= 5 ? kFirst - 2 : 1)) mx = max_of_halves(mx) * c + bias;
        if constexpr (x == kFirst - 1) {
          grew = mx > m_run;
          const float m_new = fmaxf(m_run, mx);
          const float m_fin = (m_new == -INFINITY) ? 0.f : m_new;
          alpha = fast_exp2(m_run - m_fin);
          m_use = m_fin - bias;
          m_run = m_new;
        }
        if constexpr (x >= kFirst) {
          constexpr int i0 = (x - kFirst) * 16 / (kN - kFirst), i1 = (x - kFirst + 1) * 16 / (kN - kFirst);
#pragma unroll
          for (int i = i0; i < i1; ++i) {
            sc[i] = fast_exp2(fmaf(sc[i], c, -m_use));
            if (i & 1) {
              sum1 += sc[i];
              pn[i >> 1] = pack_bf16x2(sc[i - 1], sc[i]);
            } else {
              sum0 += sc[i];
            }
          }
        }
        if constexpr (x == 1) next_tile(std::integral_constant<int, 0>{}, std::bool_constant<kNewBlock>{}, std::bool_constant<kNewBlockV>{});
        if constexpr (x == 2) next_tile(std::integral_constant<int, 1>{}, std::bool_constant<kNewBlock>{}, std::bool_constant<kNewBlockV>{});
        if constexpr (x == 3) next_tile(std::integral_constant<int, 2>{}, std::bool_constant<kNewBlock>{}, std::bool_constant<kNewBlockV>{});
        if constexpr (x == 2 && (U + 1) % C::kSub == 0) fetch_current();
        if constexpr (x == kN - 2 && kNextNewBlock) fetch_entry();
        // copies of K of tile t + 3 and V of tile t + 2, spread over the slots behind the barrier
        // (their stages were last read in iteration t - 1)
        if constexpr (x >= kBar) {
          constexpr int i0 = (x - kBar) * 2 * kI / (kN - kBar), i1 = (x - kBar + 1) * 2 * kI / (kN - kBar);
          copy_some(std::integral_constant<int, i0>{}, std::integral_constant<int, i1 - i0>{}, smem_addr + ((U + 3) & 3) * kStage,
                    smem_addr + ((U + 2) & 3) * kStage);
        }
        if constexpr (x == kN - 1) next_current(std::bool_constant<(U + 1) % C::kSub == 0>{});
        __builtin_amdgcn_sched_barrier(0);
      }(), ...);
    }(std::make_integer_sequence<int, kN>{});
    l_run = fmaf(l_run, alpha, sum0 + sum1);
#pragma unroll
    for (int i = 0; i < 8; ++i) pb[i] = pn[i];
    if (__any(grew)) {
#pragma unroll
      for (int dm = 0; dm < D / 32; ++dm)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[dm][i] *= alpha;
    }
  };

  if (n_it > 0) {
    // The loop takes four tiles at a time, one per stage: what is left over comes first.
    const int first = C::kSub == 4 ? 0 : -n_it & 3;
    const uint32_t first_stage = (uint32_t)first;
    {
      // the products of tile -1 have P = 0: their V operand only has to be finite
      u32x4 *z = reinterpret_cast<u32x4 *>(group_smem + kVBase + ((first_stage + 3) & 3) * kStage);
      for (int x = tid; x < kStage / 16; x += C::kThreads) z[x] = u32x4{0, 0, 0, 0};
    }
    __syncthreads();   // cols[] is written
    // K of tiles 0, 1, 2 and V of tiles 0, 1
    [&]<int... T>(std::integer_sequence<int, T...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int t = T;
        constexpr bool new_block = t % C::kSub == 0, new_block_v = t > 0 && (t - 1) % C::kSub == 0;
        if constexpr (new_block) fetch_entry();
        next_tile(std::integral_constant<int, 0>{}, std::bool_constant<new_block>{}, std::bool_constant<new_block_v>{});
        next_tile(std::integral_constant<int, 1>{}, std::bool_constant<new_block>{}, std::bool_constant<new_block_v>{});
        if constexpr (t > 0 || !kRun) next_tile(std::integral_constant<int, 2>{}, std::bool_constant<new_block>{}, std::bool_constant<new_block_v>{});
        copy_some(std::integral_constant<int, 0>{}, std::integral_constant<int, t == 0 ? kI : 2 * kI>{},
                  smem_addr + ((t + first_stage) & 3u) * kStage, smem_addr + ((t + 3 + first_stage) & 3u) * kStage);
      }(), ...);
    }(std::make_integer_sequence<int, 3>{});
    if (3 % C::kSub == 0) fetch_entry();
    fetch_current();
    next_current(std::true_type{});
    __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * kI));   // K of tiles 0 and 1
    __syncthreads();
    auto move_rows = [&](uint32_t by) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < D / 16; ++s) row_at[s] += by;
    };
    const uint32_t stage0 = first_stage * kStage, stage1 = ((first_stage + 1) & 3u) * kStage;
    move_rows(stage0);
    s0 = zero16;
    [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        read_row(std::integral_constant<int, E>{}, std::integral_constant<int, 0>{});
        s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[E % kRing], qreg[E], s0, 0, 0, 0);
      }(), ...);
    }(std::make_integer_sequence<int, kNS>{});
    // first operands of iteration 0 (all of them where it has fewer rows than the ring is deep)
    move_rows(stage1 - stage0);
    [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
      (read_row(std::integral_constant<int, E>{}, std::integral_constant<int, 0>{}), ...);
    }(std::make_integer_sequence<int, (kNS < kDepth ? kNS : kDepth)>{});
    move_rows(0u - stage1);
    if constexpr (kNS < kDepth) {
      const uint32_t stage3 = ((first_stage + 3) & 3u) * kStage;         // (of tile -1)
#pragma unroll
      for (int x = 0; x < 2 * (D / 32); ++x) tr_at[x] += stage3;
      [&]<int... F>(std::integer_sequence<int, F...>) __attribute__((always_inline)) {
        (read_tr(std::integral_constant<int, F>{}, std::integral_constant<int, 0>{}), ...);
      }(std::make_integer_sequence<int, kDepth - kNS>{});
#pragma unroll
      for (int x = 0; x < 2 * (D / 32); ++x) tr_at[x] -= stage3;
    }
    if constexpr (BLK == 128 && D == 128) {
      // What is left over is part of a first pass through the loop: with tiles of its own in front of it the kernel spilled 42 of its
      // 256 registers, and reloads in the loop waited for copies in flight (so and, behind it, this way, us: 9 heads of 8 blocks, 4 tiles
      // a row, 16.7 and 14.8; 11 heads of 17, 2 tiles, 14.9 and 13.1; 1 head of 143, prefix rows, 251 and 232).  Elsewhere
      // registers suffice, and the branches cost 1-2 % at block 64.
      static_assert(C::kSub == 2, "no or two tiles are left over");
      bool half = first != 0;
      for (int left = (n_it + 3) & ~3; left > 0; left -= 4) {
        if (!half) {
          body(std::integral_constant<int, 0>{}, s0, s1);
          body(std::integral_constant<int, 1>{}, s1, s0);
        }
        half = false;
        body(std::integral_constant<int, 2>{}, s0, s1);
        body(std::integral_constant<int, 3>{}, s1, s0);
      }
    } else {
      if constexpr (C::kSub == 1) {
        if (first & 1) s1 = s0;
        if (first == 1) body(std::integral_constant<int, 1>{}, s1, s0);
      }
      if constexpr (C::kSub <= 2) {
        if (first == 2 || (C::kSub == 1 && first == 1)) body(std::integral_constant<int, 2>{}, s0, s1);
        if (first != 0) body(std::integral_constant<int, 3>{}, s1, s0);
      }
      for (int t = -first & 3; t < n_it; t += 4) {
        body(std::integral_constant<int, 0>{}, s0, s1);
        body(std::integral_constant<int, 1>{}, s1, s0);
        body(std::integral_constant<int, 2>{}, s0, s1);
        body(std::integral_constant<int, 3>{}, s1, s0);
      }
    }
    // the last tile's P V (stage 3: the loop ends on a multiple of four)
    __builtin_amdgcn_s_waitcnt(0x0F70);          // stray copies must land before the LDS is given up
    [&]<int... F>(std::integer_sequence<int, F...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        read_tr(std::integral_constant<int, F>{}, std::integral_constant<int, 3>{});
        pv(std::integral_constant<int, F>{});
      }(), ...);
    }(std::make_integer_sequence<int, kNV>{});
  }

  float l_tot = l_run + swap_halves(l_run);
  if constexpr (KS > 1) {
    // the groups' parts of the row meet in the LDS that the tiles have left
    constexpr int kPart = (D / 8 + 1) * 64 * 16;   // bytes per wavefront: O, then maximum and sum
    static_assert(KS == 2 && C::kWaves * kPart <= KS * C::kLds, "the second group's part");
    __syncthreads();                               // (nobody reads a tile any more, no copy is in flight)
    f32x4 *part = reinterpret_cast<f32x4 *>(smem + wave * kPart) + lane;
    if (group > 0) {
#pragma unroll
      for (int x = 0; x < D / 8; ++x)
        part[64 * x] = f32x4{oacc[x / 4][4 * (x % 4)], oacc[x / 4][4 * (x % 4) + 1], oacc[x / 4][4 * (x % 4) + 2], oacc[x / 4][4 * (x % 4) + 3]};
      part[64 * (D / 8)] = f32x4{m_run, l_tot, 0.f, 0.f};
    }
    __syncthreads();
    if (group > 0) return;
    const f32x4 ml = part[64 * (D / 8)];
    const float m_new = fmaxf(m_run, ml[0]), m_fin = (m_new == -INFINITY) ? 0.f : m_new;
    const float mine = fast_exp2(m_run - m_fin), other = fast_exp2(ml[0] - m_fin);
    m_run = m_new;
    l_tot = fmaf(l_tot, mine, ml[1] * other);
#pragma unroll
    for (int x = 0; x < D / 8; ++x) {
      const f32x4 v = part[64 * x];
#pragma unroll
      for (int e = 0; e < 4; ++e) oacc[x / 4][4 * (x % 4) + e] = fmaf(oacc[x / 4][4 * (x % 4) + e], mine, v[e] * other);
    }
  }
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  if (qvalid) {
    bf16 *os = slab_ptr(a.o, a.to, slab, a.H) + (int64_t)qrow * a.to.sL;
    bf16 *ls = a.o_lo ? slab_ptr(a.o_lo, a.to, slab, a.H) + (int64_t)qrow * a.to.sL : nullptr;
#pragma unroll
    for (int dm = 0; dm < D / 32; ++dm) {
      uint32_t w[8], r[8];
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float v0 = oacc[dm][i] * inv, v1 = oacc[dm][i + 1] * inv;
        const uint32_t pk = pack_bf16x2(v0, v1);
        w[i >> 1] = pk;
        r[i >> 1] = pack_bf16x2(v0 - bf16_bits_to_float(pk & 0xffffu),
                                v1 - bf16_bits_to_float(pk >> 16));
      }
      uint4 *dst = reinterpret_cast<uint4 *>(os + dm * 32 + 16 * hl);
      dst[0] = make_uint4(w[0], w[1], w[2], w[3]);
      dst[1] = make_uint4(w[4], w[5], w[6], w[7]);
      if (ls) {
        uint4 *dl = reinterpret_cast<uint4 *>(ls + dm * 32 + 16 * hl);
        dl[0] = make_uint4(r[0], r[1], r[2], r[3]);
        dl[1] = make_uint4(r[4], r[5], r[6], r[7]);
      }
    }
    if (hl == 0)
      a.lse[(int64_t)slab * a.L + qrow] =
          l_tot > 0.f ? m_run * 0.69314718055994530942f + __logf(l_tot) : -INFINITY;
  }
}

// ---------------------------------------------------------------------------------------
// Wide forward: 64 query rows per wavefront, one wavefront per SIMD, with the software pipeline of the backward kernels
// (see asa_bwd.hip) inside it.  QW wavefronts share the tiles of 32 keys: two (one query block of 128) with index lists,
// four (256 rows of a dense call, whatever its block size).  In iteration t a wavefront computes S^T of tile t + 1 for
// its two halves of 32 rows, adds P V of tile t - 1, and between those MFMAs turns S^T of tile t into P.  Every operand
// read from LDS feeds two MFMAs.  V comes from its rows by the transposing LDS read: no transposed copy.  O lives in
// accumulation registers.
//
// Bound: power and issue.  At one wavefront per SIMD every instruction, scalar ones too, takes an issue slot of 4-5
// cycles; 200 of them per iteration stand beside 1024 matrix cycles.  12 heads of 32 760 tokens, a quarter of the tiles:
// matrix duty 0.65 at 1.53-1.59 GHz (ping-pong 0.62 at 1.58), dense 0.68 at 1.70; a build without the copies in the loop has 8
// and 4 % fewer cycles.  What follows from that:
//  * No row maximum per tile.  The exponentials are relative to a reference per row: the largest logit of the first tile
//    and, where the list holds the query block itself, among the 32 keys of the row's own group (one extra product in the
//    prologue).  As long as no row sum of a tile passes 2^30 the reference stays; then the tile is redone and O scaled.
//  * The rounding of P to bf16 shows where few keys carry a row (a key at the reference has P = 1 exactly, one above it
//    has not; with the running maximum every key that was ever the largest is exact).  Where the square of a tile's row
//    sum is large against those before it, what the rounding left out is added as a second product.  The own block comes
//    first in a row's order so that this and new references are rare.
//    Error of O + o_lo against 64 bits, relative, 1e-4, in brackets ping-pong with its running maximum, 13 x 30 x 45
//    tokens, a quarter of the tiles: keys and queries with a smooth field of twice the noise 1.0 (3.7), as strong as the
//    noise 1.8 (5.9), half as strong 5.6 (8.6); noise alone 14.8 (15.3), 1.5 times that 10.7 (12.3), twice 5.6 (8.8),
//    three times 2.3 (5.3).  With a quarter to all of the tiles, 1 014 to 32 760 tokens, it is nowhere larger than with
//    the running maximum.  (A row sum of more than half of everything before as the condition: 1.4, 3.1, 9.0; 16.4,
//    15.6, 12.5, 5.9.  That saves 1 % with the strong field and most of the second products with noise, which is where
//    they cost: 12 heads of 32 760 tokens, noise alone 1.56 ms, 1.5 times that 1.83, twice 2.05, half a field 1.69,
//    ping-pong 1.58 .. 1.60.)
//  * The loop has no ragged or pooled tiles: those are in a second copy of it behind the first.
//  * A wavefront sets M0 and the base of its copies once per tile; addresses advance by scalar additions.
//  * What a rare branch redefines the compiler would compute behind that branch, away from the MFMAs: pinned.
// Times (with the transposition where there was one): a quarter of the tiles 1.58 -> 1.49 ms, dense 5.9 -> 5.4 ms, pooled
// tokens 1.85 -> 1.57 ms against the ping-pong kernel.  (Row sums of the rounded P by v_dot2, as a normaliser, cost 14
// cycles each beside MFMAs, by small MFMAs 64 cycles per tile; the second product serves better.)
// ---------------------------------------------------------------------------------------
template <int BLK, int D, int QW>
struct WideCfg {
  static constexpr int kWaves = QW;                    // QW x 64 query rows per workgroup
  static constexpr int kThreads = QW * 64;
  static constexpr int kRows = QW * 64;
  static constexpr int kST = 32;                       // keys per tile
  static constexpr int kSub = BLK / kST;
  static constexpr int kStages = 4;
  static constexpr int kTile = kST * D * 2;            // bytes of one row tile
  static constexpr int kLds = 2 * kStages * kTile;     // K stages, then V stages
  static_assert(BLK == 128, "the plain loop ends in front of the last block: four tiles in it");
};

template <int BLK, int D, int QW, bool GT>
__global__ __launch_bounds__(QW * 64, 1) void fwd_wide_kernel(FwdArgs a) {
  using C = WideCfg<BLK, D, QW>;
  extern __shared__ __align__(1024) unsigned char smem[];
  __shared__ int cols[kMaxNb];
  __shared__ int again;
  constexpr int kStage = C::kTile, kVBase = C::kStages * C::kTile;
  constexpr int kPooled = 1 << 30;             // flag of an entry of cols[]: a block of pooled tokens
  constexpr int kDm = D / 32;
  // For the row sum of a tile (16 keys of a lane): passes kRedo: new reference; its square passes kLeast + the sum of all
  // squares before, times kEarly (those of the first fifth of the row) or kLate over the number of tiles: second product
  constexpr float kRedo = 1073741824.f, kEarly = 25.f, kLate = 60.f, kLeast = 2.25f;

  const int n_q = C::kRows == BLK ? a.Nb : (a.L + C::kRows - 1) / C::kRows;   // query blocks of a slab
  const int slot = xcd_contiguous_work(blockIdx.x, a.n_slabs * n_q);
  if (slot < 0) return;
  const int work = a.order ? a.order[slot] : slot;
  const int slab = work / n_q;
  if (slab_not_mine(a, slab)) return;
  const int qb = work - slab * n_q;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, hl = lane >> 5, n = lane & 31;

  const bf16 *qs = slab_ptr(a.q, a.tq, slab, a.H);
  const bf16 *ks = slab_ptr(a.k, a.tk, slab, a.H);
  const bf16 *vs = slab_ptr(a.v, a.tv, slab, a.H);
  const bool dense = a.row_ptr == nullptr;   // no index lists: dense attention, every key block in order
  const int t_begin = dense ? 0 : a.row_ptr[slab * (a.Nb + 1) + qb];
  const int n_own_blocks = dense ? a.Nb : a.row_ptr[slab * (a.Nb + 1) + qb + 1] - t_begin;
  const int n_blocks = n_own_blocks + (GT ? a.Nbg : 0);   // pooled blocks come after the row's own list
  // Order of a row's own blocks: the query block's own tokens first where they are in the list (attention is strongest
  // there as a rule), the block with the last row last (the loop below relies on it; a list that does not ascend may have
  // it elsewhere).  Every wavefront looks through the list itself.
  bool own_listed = dense;
  {
    constexpr int kOwn = C::kRows / BLK;       // key blocks of the workgroup's own tokens
    const int32_t *g = a.col_idx + (int64_t)slab * a.Nb * a.Nb + t_begin;
    const bool own_first = (qb + 1) * kOwn < a.Nb;
    int own_at = qb * kOwn, last_at = n_own_blocks - 1;
    if (!dense) {
      own_at = 0;
      for (int t0 = 0; t0 < n_own_blocks; t0 += 64) {
        const int e = t0 + lane < n_own_blocks ? g[t0 + lane] : -1;
        const uint64_t own = __ballot(e == qb), last = __ballot(e == a.Nb - 1);
        if (own) {
          own_listed = true;
          own_at = t0 + (int)__builtin_ctzll(own);
        }
        if (last) last_at = t0 + (int)__builtin_ctzll(last);
      }
      if (own_at == n_own_blocks - 1) own_at = last_at;      // (where the exchange below puts it)
    }
    for (int t = tid; t < n_blocks; t += C::kThreads) {
      int from = t;
      if (t >= n_own_blocks) {
        cols[t] = (t - n_own_blocks) | kPooled;
        continue;
      }
      if (own_first) from = t < kOwn ? own_at + t : (t >= own_at && t < own_at + kOwn ? t - own_at : t);
      from = from == last_at ? n_own_blocks - 1 : (from == n_own_blocks - 1 ? last_at : from);
      cols[t] = dense ? from : g[from];
    }
  }
  const bf16 *kgs = reinterpret_cast<const bf16 *>(a.kg) + (int64_t)slab * a.Nbg * BLK * D;
  const bf16 *vgs = reinterpret_cast<const bf16 *>(a.vg) + (int64_t)slab * a.Nbg * BLK * D;

  const int qrow0 = qb * C::kRows + wave * 64 + n;       // rows of my halves: qrow0, qrow0 + 32
  bf16x8 qa[D / 16], qc[D / 16];
  {
    const bf16 *ra = qs + (int64_t)min(qrow0, a.L - 1) * a.tq.sL, *rc = qs + (int64_t)min(qrow0 + 32, a.L - 1) * a.tq.sL;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
      qa[s] = *reinterpret_cast<const bf16x8 *>(ra + 16 * s + 8 * hl);
      qc[s] = *reinterpret_cast<const bf16x8 *>(rc + 16 * s + 8 * hl);
    }
  }
  // Largest logit of each row among the 32 rows of its own group, where their keys are in the list
  float own_a = -INFINITY, own_c = -INFINITY;
  if (own_listed) {
    const bf16 *ra = ks + (int64_t)min(qrow0, a.L - 1) * a.tk.sL + 8 * hl, *rc = ks + (int64_t)min(qrow0 + 32, a.L - 1) * a.tk.sL + 8 * hl;
    f32x16 sa, sc;
#pragma unroll
    for (int i = 0; i < 16; ++i) sa[i] = sc[i] = 0.f;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
      sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(ra + 16 * s), qa[s], sa, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(rc + 16 * s), qc[s], sc, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      own_a = fmaxf(own_a, sa[i]);
      own_c = fmaxf(own_c, sc[i]);
    }
    own_a = max_of_halves(own_a) * a.scale_log2e;
    own_c = max_of_halves(own_c) * a.scale_log2e;
  }
  f32x16 oa[kDm], oc[kDm];                               // O^T of the two halves
  // per row: reference of the exponentials (log2 units), sum of P over my lane half's keys
  float ma = 0.f, mc = 0.f, la = 0.f, lc = 0.f;
  const float c = a.scale_log2e;
  float wa = 0.f, wc = 0.f;                              // what the square of a tile's row sum must pass for a second product
  // limits of this walk over the list (see the end): for the row sums of a tile that move the references, and for a second product
  float redo_at = kRedo, least = kLeast;

  using Copy = TrTileCopy<C::kST, D, C::kWaves>;
  Copy copy_k, copy_v, copy_p;
  copy_k.init(wave, lane, a.tk.sL, a.L);
  copy_v.init(wave, lane, a.tv.sL, a.L);
  constexpr int kI = Copy::kInstr;
  const int last_row0 = Copy::last_row0(a.L);
  if (GT) copy_p.init(wave, lane, D, C::kST);   // pooled rows: D elements apart, never ragged

  const uint32_t smem_addr = ASA_LDS_ADDR_OF(smem);
  // A fragments of S^T = K Q^T: row kappa(n) of the 32 keys (see asa_bwd.hip)
  const int kr = kappa(n);
  uint32_t row_at[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    row_at[s] = (smem_addr + (uint32_t)(kr * D * 2 + (hl ^ t_swz<D>(kr)) * 16)) ^ (uint32_t)(32 * s);
  // transposed A fragments "32 channels x 16 keys" of O^T += V^T P^T
  const int tr_i = lane & 15, tr_w = tr_i & 3, tr_j = tr_i >> 2, tr_b = (lane >> 4) & 1;
  const uint32_t tr_lane = smem_addr + kVBase + tr_piece<D>(8 * hl + tr_j, 16 * (tr_w & 1) + 8 * tr_b + 4 * (tr_w >> 1));
  uint32_t tr_at[2 * kDm];
#pragma unroll
  for (int dm = 0; dm < kDm; ++dm) {
    tr_at[2 * dm] = tr_lane ^ (uint32_t)(((4 * dm) ^ t_swz<D>(0)) * 16);
    tr_at[2 * dm + 1] = tr_lane ^ (uint32_t)(((4 * dm) ^ t_swz<D>(4)) * 16);
  }
  const int n_it = n_blocks * C::kSub;
  const int t_late = n_it / 5;
  const float early = kEarly / (float)n_it, late = kLate / (float)n_it;
  float share = early;
  if (tid == 0) again = 0;

  // Copies.  The kI loads of a wavefront's share of a tile have M0 and a scalar base in common (lds_dma_begin) and
  // differ by the offset inside the instruction, which moves the LDS and the global address alike: the offsets per
  // lane are lowered by as much (and raised by kBack, which the bases lack, to stay positive).
  constexpr int kBack = (kI - 1) * 1024;
  // offsets of the K and V loads of this iteration; others only where a tile with the last row, or a pooled one, is near
  uint32_t off_k[kI], off_v[kI];
  auto lane_offset = [&](const Copy &own, int i, bool last, bool pooled) __attribute__((always_inline)) {
    return (GT && pooled ? copy_p.off[i] : (last ? own.off_last[i] : own.off[i])) + (uint32_t)(kBack - i * 1024);
  };
  // The tile whose K rows are copied next, and the tile before it, whose V rows are
  int entry_v = 0, entry_at = 0, key_c = 0, block_c = 0;
  bool last_k = false, last_v = false, pooled_k = false, pooled_v = false;
  const char *base_k = nullptr, *base_v = nullptr, *base_v_next = nullptr;
  // > 0: one of the tiles that the coming iteration copies, works on or has just worked on holds the last row, lies past
  // it or is pooled (its K rows were copied at most five iterations ago)
  int special = 0;
  auto fetch_entry = [&]() __attribute__((always_inline)) {
    entry_v = cols[entry_at < n_blocks ? entry_at : n_blocks - 1];
    ++entry_at;
  };
  const char *const ks_b = reinterpret_cast<const char *>(ks) - kBack, *const vs_b = reinterpret_cast<const char *>(vs) - kBack;
  const char *const kgs_b = reinterpret_cast<const char *>(kgs) - kBack, *const vgs_b = reinterpret_cast<const char *>(vgs) - kBack;
  const int64_t tile_k = C::kST * a.tk.sL * 2, tile_v = C::kST * a.tv.sL * 2;   // bytes from tile to tile
  // TAIL: the tile may hold the last row, lie past it or be pooled
  auto next_tile = [&](auto part_tag, auto new_block_tag, auto tail_tag) __attribute__((always_inline)) {
    constexpr int part = decltype(part_tag)::value;
    constexpr bool new_block = decltype(new_block_tag)::value;
    if constexpr (!decltype(tail_tag)::value) {
      if constexpr (part == 0) {
        base_v = base_v_next;
        if constexpr (new_block) block_c = __builtin_amdgcn_readfirstlane(entry_v);
        key_c = new_block ? block_c * BLK : key_c + C::kST;
      } else if constexpr (part == 1) {
        base_k = new_block ? ks_b + block_c * (C::kSub * tile_k) : base_k + tile_k;
      } else {
        base_v_next = new_block ? vs_b + block_c * (C::kSub * tile_v) : base_v_next + tile_v;
      }
    } else if constexpr (part == 0) {
      last_v = last_k;
      pooled_v = pooled_k;
      base_v = base_v_next;
      if constexpr (new_block) {
        const int e = __builtin_amdgcn_readfirstlane(entry_v);
        if (GT) pooled_k = (e & kPooled) != 0;
        block_c = GT ? e & (kPooled - 1) : e;
        key_c = block_c * BLK;
      } else {
        key_c += C::kST;
      }
      last_k = key_c >= last_row0;
      special = (last_k || (GT && pooled_k)) ? 5 : max(special - 1, 0);
    } else if constexpr (part == 1) {
      if constexpr (new_block) {
        base_k = ks_b + block_c * (C::kSub * tile_k);
        if (GT) base_k = pooled_k ? kgs_b + (int64_t)key_c * (D * 2) : base_k;
      } else {
        // (a tile wholly past the last row is replaced by the one that holds it; pooled rows fill whole blocks)
        if (GT) base_k += pooled_k ? C::kTile : (key_c <= last_row0 ? tile_k : 0);
        else base_k += key_c <= last_row0 ? tile_k : 0;
      }
    } else {
      if constexpr (new_block) {
        base_v_next = vs_b + block_c * (C::kSub * tile_v);
        if (GT) base_v_next = pooled_k ? vgs_b + (int64_t)key_c * (D * 2) : base_v_next;
      } else {
        if (GT) base_v_next += pooled_k ? C::kTile : (key_c <= last_row0 ? tile_v : 0);
        else base_v_next += key_c <= last_row0 ? tile_v : 0;
      }
    }
  };
  auto set_offsets = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kI; ++i) {
      off_k[i] = lane_offset(copy_k, i, last_k, pooled_k);
      off_v[i] = lane_offset(copy_v, i, last_v, pooled_v);
    }
  };
  auto copy_one = [&](auto i_tag, uint64_t base, const uint32_t *off) __attribute__((always_inline)) {
    constexpr int i = decltype(i_tag)::value;
    lds_dma16_next<i * 1024>(base, off[i]);
  };
  auto wait_copies = [&](auto n_tag) __attribute__((always_inline)) {
    constexpr int N = decltype(n_tag)::value;    // at most N instructions still in flight
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  };
  // The block of the tile in work, for the masks of the last block and the bias of pooled keys
  int cur_v = 0, cur_at = 0, key_t = 0, key_end = 0;
  int left = C::kST;                             // keys that the tile before it had (32 and more: all)
  float bias = 0.f;
  auto fetch_current = [&]() __attribute__((always_inline)) {
    cur_v = cols[cur_at < n_blocks ? cur_at : n_blocks - 1];
    ++cur_at;
  };
  auto next_current = [&](auto new_block_tag) __attribute__((always_inline)) {
    left = key_end - key_t;
    if constexpr (decltype(new_block_tag)::value) {
      const int e = __builtin_amdgcn_readfirstlane(cur_v);
      key_t = (GT ? e & (kPooled - 1) : e) * BLK;
      const bool pooled = GT && (e & kPooled) != 0;
      key_end = pooled ? a.Lg : a.L;             // keys at or past it do not exist
      if (GT) bias = pooled ? a.bias_log2 : 0.f;
    } else {
      key_t += C::kST;
    }
  };

  // An iteration is kN slots, one MFMA each.  Fragment f of the kF operands of an iteration (K rows of tile
  // t + 1, then V of tile t - 1) feeds the slots 2 f and 2 f + 1 and is read kDepth fragments ahead, through a
  // ring that runs on from iteration to iteration.
  constexpr int kNS = D / 16, kNV = 2 * kDm, kF = kNS + kNV, kN = 2 * kF;
  constexpr int kRing = 8, kDepth = 4;
  static_assert(kF % kRing == 0 && kDepth <= kNS, "the ring continues across iterations");
  constexpr int kHalf = 17;                         // exponentials in front of it
  constexpr int kBar = 2 * kNS;                     // the barrier comes before this slot
  bf16x8 row_ring[kRing];
  bf16x4 lo_ring[kRing], hi_ring[kRing];
  auto read_row = [&](auto f_tag, auto stage_tag) __attribute__((always_inline)) {
    constexpr int f = decltype(f_tag)::value;
    row_ring[f % kRing] = lds_read<bf16x8>(row_at[f] + (uint32_t)(decltype(stage_tag)::value * kStage));
  };
  auto read_tr = [&](auto f_tag, auto stage_tag, auto half_tag) __attribute__((always_inline)) {
    constexpr int f = decltype(f_tag)::value, dm = f % kDm, tt = f / kDm, half = decltype(half_tag)::value;
    constexpr int at = decltype(stage_tag)::value * kStage + 16 * tt * D * 2;
    if constexpr (half == 0)
      lo_ring[(kNS + f) % kRing] = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm] + (uint32_t)at));
    else
      hi_ring[(kNS + f) % kRing] = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm + 1] + (uint32_t)(at + 4 * D * 2)));
  };
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // LDS reads issued behind the last one of fragment f0 up to slot x of the iteration: a row fragment is one read, in its
  // even slot, a transposed one two
  constexpr auto reads_behind = [](int f0, int x) constexpr {
    int n = 0;
    for (int y = 2 * (f0 - kDepth) + 2; y <= x; ++y) {
      const int f = ((y >> 1) + kDepth + kF) % kF;      // fragment read in slot y (of the iteration before if y < 0)
      n += f < kNS ? ((y & 1) == 0) : 1;
    }
    return n;
  };
  auto wait_lds = [&](auto n_tag) __attribute__((always_inline)) {
    constexpr int N = decltype(n_tag)::value;
    __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
  };
  f32x16 s0a, s0c, s1a, s1c;
  uint32_t p0[16], p1[16];               // bf16 P of two tiles, both halves
  auto accumulate = [](f32x16 &acc, bf16x8 x, bf16x8 y) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(x), "v"(y));
#endif
  };
  auto pv = [&](auto f_tag, auto half_tag, const uint32_t *p) __attribute__((always_inline)) {
    constexpr int f = decltype(f_tag)::value, dm = f % kDm, tt = f / kDm, half = decltype(half_tag)::value;
    const u32x4 raw = {p[8 * half + 4 * tt], p[8 * half + 4 * tt + 1], p[8 * half + 4 * tt + 2], p[8 * half + 4 * tt + 3]};
    const bf16x8 x = __builtin_shufflevector(lo_ring[(kNS + f) % kRing], hi_ring[(kNS + f) % kRing], 0, 1, 2, 3, 4, 5, 6, 7);
    accumulate(half == 0 ? oa[dm] : oc[dm], x, __builtin_bit_cast(bf16x8, raw));
  };
  // (what the rare branch of an iteration overwrites would be computed behind it, without MFMAs to hide under)
  auto pin = [](auto &x) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x));
#endif
  };
  auto pin_s = [](auto &x) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(x));
#endif
  };
  auto mask_tile = [&](f32x16 &sa, f32x16 &sc) __attribute__((always_inline)) {
    const int mine = key_end - key_t - 8 * hl;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (16 * (i >> 3) + (i & 7) >= mine) sa[i] = sc[i] = -INFINITY;
  };
  // keys past the end have P = 0: their V rows (in `stage`, read after this by my own wavefront) must be finite.
  // Every wavefront writes all of the zeros itself.
  auto zero_rows = [&](int stage, int left) __attribute__((always_inline)) {
    u32x4 *z = reinterpret_cast<u32x4 *>(smem + kVBase + stage * kStage);
    for (int r = max(0, left) * (D / 8) + lane; r < kStage / 16; r += 64) z[r] = u32x4{0, 0, 0, 0};
  };
  auto row_max = [&](const f32x16 &s, float bias_t) __attribute__((always_inline)) {
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
    return max_of_halves(mx) * c + bias_t;
  };
  auto settle = [&]() __attribute__((always_inline)) {
    settle_acc(oa);
    settle_acc(oc);
  };

  float sq_a = 0.f, sq_c = 0.f;                      // squares of the row sums of the tile before, not yet in wa, wc
  float ta_last = 0.f, tc_last = 0.f;                // row sums of the tile before, not yet in la, lc
  auto body = [&](auto u_tag, auto tail_tag, f32x16 &sa, f32x16 &sc, f32x16 &na, f32x16 &nc, uint32_t *pn, const uint32_t *po) __attribute__((always_inline)) {
    constexpr int U = decltype(u_tag)::value;        // tile index mod 4
    constexpr bool kTail = decltype(tail_tag)::value;
    using StK1 = std::integral_constant<int, (U + 1) & 3>;
    using StK2 = std::integral_constant<int, (U + 2) & 3>;
    using StVp = std::integral_constant<int, (U + 3) & 3>;   // V rows of tile t - 1
    constexpr bool kNextNewBlock = (U + C::kStages) % C::kSub == 0;   // of the K tile that the next iteration copies
    if constexpr (kTail) {
      if (special > 0) {
        set_offsets();
        if (key_t + C::kST > key_end) mask_tile(sa, sc);
        if (left < C::kST) zero_rows((U + 3) & 3, left);
      }
    }
    const float bias_t = GT && kTail ? bias : 0.f;
    const int left_now = kTail ? key_end - key_t : C::kST;
    const float nma = GT && kTail ? bias_t - ma : -ma, nmc = GT && kTail ? bias_t - mc : -mc;
    uint64_t from_k = 0, from_v = 0;
    float ta = 0.f, tc = 0.f;                        // sums of this tile
    float w[32];                                     // argument, then value of each exponential
    constexpr int kES = kN - 2;                      // slots with exponentials
    // first element of slot g
    auto first = [](int g) constexpr { return g <= kBar ? g * kHalf / kBar : kHalf + (g - kBar) * (32 - kHalf) / (kES - kBar); };
    auto arg = [&](auto g_tag) __attribute__((always_inline)) {
      constexpr int g = decltype(g_tag)::value;
#pragma unroll
      for (int e = first(g); e < first(g + 1); ++e)
        w[e] = e < 16 ? fmaf(sa[e & 15], c, nma) : fmaf(sc[e & 15], c, nmc);
    };
    auto finish = [&](auto g_tag) __attribute__((always_inline)) {
      constexpr int g = decltype(g_tag)::value;
#pragma unroll
      for (int e = first(g); e < first(g + 1); ++e) {
        if (e == 0) ta = w[e];
        else if (e < 16) ta += w[e];
        else if (e == 16) tc = w[e];
        else tc += w[e];
        if (e & 1) {
          pn[e >> 1] = pack_bf16x2(w[e - 1], w[e]);
          pin(pn[e >> 1]);
        }
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    [&]<int... X>(std::integer_sequence<int, X...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int x = X, f = x / 2;
        if constexpr (x == kBar) {
          // K of tile t + 2 and V of tile t have landed (everyone's copies)
          wait_copies(std::integral_constant<int, 2 * kI>{});
          asm volatile("s_barrier" ::: "memory");
          from_v = lds_dma_begin(base_v, smem_addr + kVBase + ((U + 2) & 3) * kStage + copy_v.lds0);
          __builtin_amdgcn_sched_barrier(0);
        }
        // operand reads
        constexpr int r = f + kDepth;
        using Half = std::integral_constant<int, x & 1>;
        if constexpr (r < kNS) { if constexpr ((x & 1) == 0) read_row(std::integral_constant<int, r>{}, StK1{}); }
        else if constexpr (r < kF) read_tr(std::integral_constant<int, r - kNS>{}, StVp{}, Half{});
        else { if constexpr ((x & 1) == 0) read_row(std::integral_constant<int, r - kF>{}, StK2{}); }
        // (one wait for two fragments)
        if constexpr (x % 4 == 0) wait_lds(std::integral_constant<int, reads_behind(f + 1, x)>{});
        // the MFMA of this slot
        if constexpr (f < kNS) {
          if constexpr ((x & 1) == 0) na = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_ring[f % kRing], qa[f], f == 0 ? zero16 : na, 0, 0, 0);
          else nc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_ring[f % kRing], qc[f], f == 0 ? zero16 : nc, 0, 0, 0);
        } else {
          pv(std::integral_constant<int, f - kNS>{}, Half{}, po);
        }
        // soft-max of tile t
        if constexpr (x == 0) arg(std::integral_constant<int, 0>{});
        if constexpr (x < kES) {
#pragma unroll
          for (int e = first(x); e < first(x + 1); ++e) w[e] = fast_exp2(w[e]);
        }
        if constexpr (x + 1 < kES) arg(std::integral_constant<int, x + 1>{});
        if constexpr (x >= 1 && x <= kES) finish(std::integral_constant<int, x - 1>{});
        if constexpr (x == 3) {
          la += ta_last;
          lc += tc_last;
          wa = fmaf(share, sq_a, wa);
          wc = fmaf(share, sq_c, wc);
        }
        // K of tile t + 3 in front of the barrier, V of tile t + 2 behind it (their stages were last read in
        // iterations t - 2 and t - 1)
        if constexpr (x == 0) from_k = lds_dma_begin(base_k, smem_addr + ((U + 3) & 3) * kStage + copy_k.lds0);
        if constexpr (x >= 1 && x < kBar) {
          constexpr int i0 = (x - 1) * kI / (kBar - 1), i1 = x * kI / (kBar - 1);
          if constexpr (i1 > i0) copy_one(std::integral_constant<int, i0>{}, from_k, off_k);
          static_assert(i1 - i0 <= 1, "a load per slot");
        }
        if constexpr (x >= kBar) {
          constexpr int i0 = (x - kBar) * kI / (kN - kBar), i1 = (x - kBar + 1) * kI / (kN - kBar);
          if constexpr (i1 > i0) copy_one(std::integral_constant<int, i0>{}, from_v, off_v);
        }
        // the tiles of the next iteration
        if constexpr (x == kN - 8 && kNextNewBlock) fetch_entry();
        if constexpr (kTail && x == kN - 8 && (U + 1) % C::kSub == 0) fetch_current();
        if constexpr (x >= kN - 4 && x <= kN - 2) {
          next_tile(std::integral_constant<int, x - (kN - 4)>{}, std::bool_constant<kNextNewBlock>{}, tail_tag);
          if constexpr (x == kN - 3) pin_s(base_k);
          if constexpr (x == kN - 2) pin_s(base_v_next);
        }
        if constexpr (kTail && x == kN - 1) next_current(std::bool_constant<(U + 1) % C::kSub == 0>{});
        __builtin_amdgcn_sched_barrier(0);
      }(), ...);
    }(std::make_integer_sequence<int, kN>{});
    if (__builtin_expect(__any(fmaxf(ta, tc) > redo_at), 0)) {
      // some row grew far beyond its reference.  New references, this tile's P again, O and the sums scaled.
      const float xa = fmaxf(ma, row_max(sa, bias_t)), xc = fmaxf(mc, row_max(sc, bias_t));
      const float fa = fast_exp2(ma - xa), fc = fast_exp2(mc - xc);
      ma = xa;
      mc = xc;
      ta = tc = 0.f;
#pragma unroll
      for (int e = 0; e < 32; e += 2) {
        const float u = e < 16 ? fast_exp2(fmaf(sa[e & 15], c, bias_t - xa)) : fast_exp2(fmaf(sc[e & 15], c, bias_t - xc));
        const float v = e < 16 ? fast_exp2(fmaf(sa[(e & 15) + 1], c, bias_t - xa)) : fast_exp2(fmaf(sc[(e & 15) + 1], c, bias_t - xc));
        pn[e >> 1] = pack_bf16x2(u, v);
        if (e < 16) ta += u + v;
        else tc += u + v;
      }
      la *= fa;
      lc *= fc;
      wa = fmaf(wa - least, fa * fa, least);
      wc = fmaf(wc - least, fc * fc, least);
      settle();
#pragma unroll
      for (int dm = 0; dm < kDm; ++dm)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          oa[dm][i] *= fa;
          oc[dm][i] *= fc;
        }
      settle();
    }
    sq_a = ta * ta;
    sq_c = tc * tc;
    if (__builtin_expect(__any(sq_a > wa || sq_c > wc), 0)) {
      // what the rounding of P left out, as a second product
      if constexpr (kTail) {
        if (left_now < C::kST) zero_rows(U, left_now);
      }
      uint32_t rest[16];
#pragma unroll
      for (int e = 0; e < 32; e += 2) {
        const float u = e < 16 ? fast_exp2(fmaf(sa[e & 15], c, bias_t - ma)) : fast_exp2(fmaf(sc[e & 15], c, bias_t - mc));
        const float v = e < 16 ? fast_exp2(fmaf(sa[(e & 15) + 1], c, bias_t - ma)) : fast_exp2(fmaf(sc[(e & 15) + 1], c, bias_t - mc));
        rest[e >> 1] = pack_bf16x2(u - bf16_bits_to_float(pn[e >> 1] & 0xffffu), v - bf16_bits_to_float(pn[e >> 1] >> 16));
      }
#if defined(__HIP_DEVICE_COMPILE__)
      asm volatile("s_nop 1");                       // (vector results and the first MFMA that reads them)
#endif
      [&]<int... F>(std::integer_sequence<int, F...>) __attribute__((always_inline)) {
        ([&]() __attribute__((always_inline)) {
          constexpr int dm = F % kDm, tt = F / kDm, at = U * kStage + 16 * tt * D * 2;
          const bf16x4 lo = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm] + (uint32_t)at));
          const bf16x4 hi = lds_read_tr16((const lds_char *)(uintptr_t)(tr_at[2 * dm + 1] + (uint32_t)(at + 4 * D * 2)));
          const bf16x8 x = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          const u32x4 ra4 = {rest[4 * tt], rest[4 * tt + 1], rest[4 * tt + 2], rest[4 * tt + 3]};
          const u32x4 rc4 = {rest[8 + 4 * tt], rest[8 + 4 * tt + 1], rest[8 + 4 * tt + 2], rest[8 + 4 * tt + 3]};
          accumulate(oa[dm], x, __builtin_bit_cast(bf16x8, ra4));
          accumulate(oc[dm], x, __builtin_bit_cast(bf16x8, rc4));
        }(), ...);
      }(std::make_integer_sequence<int, kNV>{});
    }
    ta_last = ta;
    tc_last = tc;
  };

  // true if some value of the row is not finite
  auto emit = [&](f32x16 (&acc)[kDm], int qrow, float m, float l_half) __attribute__((always_inline)) {
    const float l_tot = l_half + swap_halves(l_half);
    if (qrow >= a.L) return false;
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    bf16 *os = slab_ptr(a.o, a.to, slab, a.H) + (int64_t)qrow * a.to.sL;
    bf16 *ls = a.o_lo ? slab_ptr(a.o_lo, a.to, slab, a.H) + (int64_t)qrow * a.to.sL : nullptr;
    float top = 0.f;
#pragma unroll
    for (int dm = 0; dm < kDm; ++dm) {
      uint32_t w[8], r[8];
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float v0 = acc[dm][i] * inv, v1 = acc[dm][i + 1] * inv;
        top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(top, fabsf(v0)), fabsf(v1));   // (keeps a NaN)
        const uint32_t pk = pack_bf16x2(v0, v1);
        w[i >> 1] = pk;
        r[i >> 1] = pack_bf16x2(v0 - bf16_bits_to_float(pk & 0xffffu),
                                v1 - bf16_bits_to_float(pk >> 16));
      }
      uint4 *dst = reinterpret_cast<uint4 *>(os + dm * 32 + 16 * hl);
      dst[0] = make_uint4(w[0], w[1], w[2], w[3]);
      dst[1] = make_uint4(w[4], w[5], w[6], w[7]);
      if (ls) {
        uint4 *dl = reinterpret_cast<uint4 *>(ls + dm * 32 + 16 * hl);
        dl[0] = make_uint4(r[0], r[1], r[2], r[3]);
        dl[1] = make_uint4(r[4], r[5], r[6], r[7]);
      }
    }
    if (hl == 0) {
#pragma clang fp contract(off)
      a.lse[(int64_t)slab * a.L + qrow] =
          l_tot > 0.f ? m * 0.69314718055994530942f + __logf(l_tot) : -INFINITY;
    }
    return !(top < INFINITY);
  };
  // One walk over the list, as a rule.  But P above 1 can overflow with a large V where P <= 1 would not, and the second
  // product makes NaN of an infinite one (what the rounding left out is of either sign, and 0 where P was exact).  So a
  // workgroup with a result that is not finite walks once more: the running maximum as the reference, P <= 1, no second
  // product.  (The look at the results and the loop around the walk: 0.3 % of 12 heads of 32 760 tokens, a quarter of the tiles.)
  for (int walk = 0;; ++walk) {
#pragma unroll
    for (int dm = 0; dm < kDm; ++dm)
#pragma unroll
      for (int i = 0; i < 16; ++i) oa[dm][i] = oc[dm][i] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) p0[i] = p1[i] = 0;
    la = lc = ta_last = tc_last = sq_a = sq_c = 0.f;
    wa = wc = least;
    entry_at = cur_at = special = 0;
    last_k = last_v = pooled_k = pooled_v = false;
    if (n_it > 0) {
      {
        // the products of tile -1 have P = 0: their V operand only has to be finite
        u32x4 *z = reinterpret_cast<u32x4 *>(smem + kVBase + 3 * kStage);
        for (int x = tid; x < kStage / 16; x += C::kThreads) z[x] = u32x4{0, 0, 0, 0};
      }
      __syncthreads();   // cols[] is written
      // K of tiles 0, 1, 2 and V of tiles 0, 1
      for (int t = 0; t < 3; ++t) {
        auto advance = [&](auto new_block) __attribute__((always_inline)) {
          next_tile(std::integral_constant<int, 0>{}, new_block, std::true_type{});
          next_tile(std::integral_constant<int, 1>{}, new_block, std::true_type{});
          next_tile(std::integral_constant<int, 2>{}, new_block, std::true_type{});
        };
        if (t % C::kSub == 0) {
          fetch_entry();
          advance(std::true_type{});
        } else {
          advance(std::false_type{});
        }
        set_offsets();
        auto issue = [&]<int... I>(std::integer_sequence<int, I...>, uint64_t base, const uint32_t *off) __attribute__((always_inline)) {
          (copy_one(std::integral_constant<int, I>{}, base, off), ...);
        };
        issue(std::make_integer_sequence<int, kI>{}, lds_dma_begin(base_k, smem_addr + t * kStage + copy_k.lds0), off_k);
        if (t > 0)
          issue(std::make_integer_sequence<int, kI>{}, lds_dma_begin(base_v, smem_addr + kVBase + (t - 1) * kStage + copy_v.lds0), off_v);
      }
      {
        // the tiles of iteration 0
        next_tile(std::integral_constant<int, 0>{}, std::false_type{}, std::true_type{});
        next_tile(std::integral_constant<int, 1>{}, std::false_type{}, std::true_type{});
        next_tile(std::integral_constant<int, 2>{}, std::false_type{}, std::true_type{});
        set_offsets();
      }
      fetch_current();
      next_current(std::true_type{});
      left = C::kST;
      wait_copies(std::integral_constant<int, 3 * kI>{});   // K of tiles 0 and 1
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      s0a = s0c = zero16;
      [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
        ([&]() __attribute__((always_inline)) {
          read_row(std::integral_constant<int, E>{}, std::integral_constant<int, 0>{});
          s0a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_ring[E % kRing], qa[E], s0a, 0, 0, 0);
          s0c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_ring[E % kRing], qc[E], s0c, 0, 0, 0);
        }(), ...);
      }(std::make_integer_sequence<int, kNS>{});
      // first operands of iteration 0
      [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
        (read_row(std::integral_constant<int, E>{}, std::integral_constant<int, 1>{}), ...);
      }(std::make_integer_sequence<int, kDepth>{});
      // the first references: the row maxima of tile 0, which always has a key
      if (key_t + C::kST > key_end) mask_tile(s0a, s0c);
      ma = fmaxf(own_a, row_max(s0a, bias));
      mc = fmaxf(own_c, row_max(s0c, bias));
      // (no finite logit yet: the lowest reference there is, which the first tile with one moves)
      ma = fmaxf(ma, -3.402823466e38f);
      mc = fmaxf(mc, -3.402823466e38f);
      own_a = own_c = -INFINITY;                 // (not kept in registers for another walk)
#pragma unroll
      for (int i = 0; i < 16; ++i) pin(p1[i]);     // (zeros in registers here, not right in front of an MFMA)
      settle();
      const std::true_type tail{};
      const std::false_type plain{};
      const std::integral_constant<int, 0> u0{};
      const std::integral_constant<int, 1> u1{};
      const std::integral_constant<int, 2> u2{};
      const std::integral_constant<int, 3> u3{};
      int t = 0;
      share = early;
      // As long as the copies (three tiles ahead) stay inside the blocks in front of the last one of the row's own
      // list nothing is ragged or pooled.
      const int n_plain = (n_own_blocks - 1) * C::kSub - 6;
      if (n_plain >= 0) {
        for (; t <= n_plain; t += 4) {
          body(u0, plain, s0a, s0c, s1a, s1c, p0, p1);
          body(u1, plain, s1a, s1c, s0a, s0c, p1, p0);
          body(u2, plain, s0a, s0c, s1a, s1c, p0, p1);
          body(u3, plain, s1a, s1c, s0a, s0c, p1, p0);
          if (t >= t_late) share = late;
        }
        cur_at = t / C::kSub;
        fetch_current();
        next_current(tail);
        left = C::kST;
      }
      for (; t < n_it; t += 4) {
        body(u0, tail, s0a, s0c, s1a, s1c, p0, p1);
        body(u1, tail, s1a, s1c, s0a, s0c, p1, p0);
        body(u2, tail, s0a, s0c, s1a, s1c, p0, p1);
        body(u3, tail, s1a, s1c, s0a, s0c, p1, p0);
        if (t >= t_late) share = late;
      }
      // the last tile's P V (stage 3: the loop ends on a multiple of four)
      __builtin_amdgcn_s_waitcnt(0x0F70);          // stray copies must land before the LDS is given up
      if (left < C::kST) zero_rows(3, left);
      la += ta_last;
      lc += tc_last;
      [&]<int... F>(std::integer_sequence<int, F...>) __attribute__((always_inline)) {
        ([&]() __attribute__((always_inline)) {
          read_tr(std::integral_constant<int, F>{}, std::integral_constant<int, 3>{}, std::integral_constant<int, 0>{});
          read_tr(std::integral_constant<int, F>{}, std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{});
          pv(std::integral_constant<int, F>{}, std::integral_constant<int, 0>{}, p1);
          pv(std::integral_constant<int, F>{}, std::integral_constant<int, 1>{}, p1);
        }(), ...);
      }(std::make_integer_sequence<int, kNV>{});
      settle();
    }

    const bool bad_a = emit(oa, qrow0, ma, la), bad_c = emit(oc, qrow0 + 32, mc, lc);
    if (walk > 0) return;
    if (__any(bad_a || bad_c)) again = 1;
    __syncthreads();                               // (everyone has also read its last V rows)
    if (!__builtin_amdgcn_readfirstlane(again)) return;
    redo_at = 1.f;
    least = INFINITY;
  }
}

template <int BLK, int D, bool VT>
static hipError_t launch_lock_step(const FwdArgs &a, int grid, hipStream_t st) {
  using C = FwdCfg<BLK, D>;
  constexpr int lds = C::kStages * (C::kKElems + C::kVElems) * 2;
  const hipError_t e = set_dynamic_lds_once(reinterpret_cast<const void *>(&fwd_kernel<BLK, D, VT>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((fwd_kernel<BLK, D, VT>), dim3(grid), dim3(C::kThreads), lds, st, a);
  return hipGetLastError();
}

template <int BLK, int D, bool GT, int KS>
static hipError_t launch_pipe(const FwdArgs &a, int grid, hipStream_t st) {
  using X = PipeCfg<BLK, D, KS>;
  const hipError_t e = set_dynamic_lds_once(reinterpret_cast<const void *>(&fwd_pipe_kernel<BLK, D, GT, KS>), KS * X::kLds);
  if (e != hipSuccess) return e;
  if (a.select >= 0) timing_begin(st);       // (else the first kernel of the pair has)
  hipLaunchKernelGGL((fwd_pipe_kernel<BLK, D, GT, KS>), dim3(grid), dim3(X::kThreads * KS), KS * X::kLds, st, a);
  return hipGetLastError();
}

template <int BLK, int D, int QW, bool GT>
static hipError_t launch_wide(const FwdArgs &a, hipStream_t st) {
  using X = WideCfg<BLK, D, QW>;
  const int n_q = X::kRows == BLK ? a.Nb : (a.L + X::kRows - 1) / X::kRows;
  const hipError_t e = set_dynamic_lds_once(reinterpret_cast<const void *>(&fwd_wide_kernel<BLK, D, QW, GT>), X::kLds);
  if (e != hipSuccess) return e;
  timing_begin(st);
  hipLaunchKernelGGL((fwd_wide_kernel<BLK, D, QW, GT>), dim3(xcd_grid(a.n_slabs * n_q)), dim3(X::kThreads), X::kLds, st, a);
  return hipGetLastError();
}

// with a.select: the slabs of fewer than select_min_tiles tiles per row are left out
template <int BLK, int D, bool GT>
static hipError_t launch_ping_pong(const FwdArgs &a, int grid, hipStream_t st) {
  using P = PpCfg<BLK, D>;
  hipError_t e = launch_transpose(a.v, a.tv, a.H, a.L, a.Lpad, BLK, D, a.n_slabs, a.vt, st,
                                  a.select ? a.row_ptr : nullptr, a.Nb, a.select_min_tiles * a.Nb);
  if (e == hipSuccess && GT) {
    // the pooled values: contiguous [slab][Nbg * block][d]
    TensorView tvg;
    tvg.sL = D; tvg.sH = (int64_t)a.Nbg * BLK * D; tvg.sB = tvg.sH * a.H;
    e = launch_transpose(a.vg, tvg, a.H, a.Lg, a.Nbg * BLK, BLK, D, a.n_slabs, a.vgt, st);
  }
  if (e == hipSuccess) e = set_dynamic_lds_once(reinterpret_cast<const void *>(&fwd_pp_kernel<BLK, D, GT>), P::kLdsBytes);
  if (e != hipSuccess) return e;
  timing_begin(st);
  hipLaunchKernelGGL((fwd_pp_kernel<BLK, D, GT>), dim3(grid), dim3(P::kThreads), P::kLdsBytes, st, a);
  return hipGetLastError();
}

// The rules of the shapes other than block 128 / d 128 (see launch_fwd_t for what they rest on).  Without lists the size of
// a block means nothing: 256 rows share the tiles of the wide kernel.
static bool small_shape_wide(const Problem &pb, bool dense, bool pooled) {
  if (!dense || pooled) return false;
  if (forced_fwd_kernel() != 0) return forced_fwd_kernel() == 4;
  const int wide = pb.n_slabs * ((pb.L + 255) / 256), rounds = (wide + 255) / 256;
  const bool filled = pb.d == 128 ? 4 * wide >= 3 * 256 * rounds : 16 * wide >= 15 * 256 * rounds;
  return filled && pb.L >= (pb.d == 128 ? 4000 : 8000);
}
// (with pooled tokens, d 64)
static bool small_shape_ping_pong(const Problem &pb, bool dense) {
  const int total = pb.n_slabs * pb.Nb, tiles = dense ? pb.Nb : pb.Nb / 8, forced = forced_fwd_kernel();
  const bool few_and_long = total <= (pb.block == 128 ? 256 : 512) && tiles >= (pb.block == 128 ? 16 : 24);
  return forced == 2 || ((forced == 0 || forced == 4) && few_and_long);
}
// (of what the wide kernel has left, without pooled tokens)
static bool small_shape_pipe(const Problem &pb, bool dense) {
  const bool small_tile = pb.block == 64 && pb.d == 64;
  const int resident = small_tile ? 1024 : 512, total = pb.n_slabs * pb.Nb;      // pipelined workgroups on the chip
  bool fits = total <= resident || (!small_tile && !dense);
  if (pb.block == 64 && pb.d == 128)
    fits |= (total + resident - 1) / resident * resident - total <= total / 20 || (total > 2 * resident && total <= 3 * resident);
  return fits && forced_fwd_kernel() != 1;
}
// Do two groups of wavefronts share a row (fwd_pipe_kernel)?  Where both halves of every row start at once, and where prefix rows,
// as long as the sequence, end the launch late: from 2.4 times what each resident group has to do on average, a row's start
// and end counted as a block.  A full chip holds half as many rows then and is 0.71-0.9x as fast: of 377 calls with text
// beyond the first line 160 lie above the second, 1.01-1.77x with two groups; of the others 146 lose by them and 59 gain.  (From 1.6
// times on with the prefix columns counted half, and for uneven rows without a prefix, whose lengths the host cannot know: down to
// 0.71x, the latter 0.95x on average of 274 calls.)  Forward alone, one group and two, us: d 64: 1 head of 2 266 tokens, block
// 64, a quarter of the tiles, 12.1 and 8.8; 3 heads of 17 776, text, block 64, 245 and 143; 24 heads of 4 332, text, block 128, 81 and 89;
// d 128: 12 slabs of 4 332, text, block 64, 87 and 80, below the line.
static bool pipe_in_two(const Problem &pb, bool dense, int pooled_blocks) {
  const int resident = pb.block == 64 && pb.d == 64 ? 1024 : 512;      // groups on the chip
  if (2 * (int64_t)pb.n_slabs * pb.Nb <= resident) return true;
  if (dense || pb.n_prefix_blocks == 0) return false;
  const int64_t rows = pb.Nb * (int64_t)(pooled_blocks + 1);           // what a slab's rows have besides the blocks of their lists
  return 5 * (int64_t)(pb.Nb + pooled_blocks + 1) * resident > 12 * pb.n_slabs * (listed_blocks(pb) + rows);
}

template <int BLK, int D>
static hipError_t launch_fwd_t(const FwdArgs &a, const Problem &pb, hipStream_t st) {
  const int total = a.n_slabs * a.Nb, grid = xcd_grid(total);
  // Which kernel.  Measured on MI355X, the transposition of V included where a kernel needs it:
  //   block 128 / d 128: lock-step (V's rows) for short rows; ping-pong, the fastest on a single row, where few rows run at a
  //     time; wide, two of whose workgroups share a compute unit, for long rows where its rounds of 512 query blocks are
  //     filled.  The two long-row kernels meet lock-step at 16-20 tiles.  Time of the others relative to the wide
  //     kernel (taken when that was 1 % faster), keys and queries with a smooth field of twice the noise, 1 014 to
  //     32 760 tokens:
  //       up to 256 query blocks: lock-step 0.55-0.83, ping-pong 0.45-0.70 (4 .. 16 tiles).
  //       lists of one length (a fixed budget), ping-pong at 20, 28 and 60 tiles:
  //            512 query blocks   0.97-1.0   0.98-1.01  1.03         1100 .. 1280  0.91-0.95  0.92-0.97  0.93-0.97
  //            600 .. 700         0.81-0.84  0.81-0.85  0.84-0.87    1500          0.98-1.02  1.0-1.06   1.05
  //            800 .. 1024        0.96-1.03  1.0-1.04   1.04         1600          0.96-0.98  0.96-0.97  0.97
  //                                                                  2000 .. 3072  1.0-1.04   1.02-1.04  1.05
  //         lock-step at 12, 16, 20, 28 tiles: 1024 blocks 0.86-0.91, 0.93-0.96, 0.98-1.0, 1.03-1.06; 2000 .. 3072
  //         0.88-0.92, 0.94-0.97, 0.99-1.01, 1.05.
  //       uneven lists (the threshold alone, 15 .. 85 tiles on average, the longest 2-6 times that), where one long
  //         row holds a wide workgroup for twice as long, ping-pong: 320 .. 768 blocks 0.57-0.93, 1024 0.66-1.0,
  //         1280 0.68-1.02, 1500 .. 1800 0.76-1.07, 2048 0.90-1.08.
  //       always-kept prefix blocks, whose rows are as long as the sequence, 20 tiles on average, ping-pong: 0.52-0.99
  //         up to 1100 blocks; beyond, 0.55-0.87 where such a row is longer than one and a half times what half a
  //         compute unit has to do in all, else 0.91-1.05.
  //       no lists: lock-step (from 18 tiles on ping-pong) at 8 .. 22 tiles 1.0-1.09 where the wide kernel needs at most
  //         half of the ping-pong kernel's rounds, at 27 .. 46 tiles 0.94-0.99 in one round and 0.96-1.07 in more, at 56
  //         and more 1.02-1.10, and 1.0-1.04 from 2048 blocks on with half-filled rounds too; elsewhere 0.53-0.98.
  //     Without lists the choice is made here.  With them the host has only the parameters of the rule to go by, which say how
  //     even the rows are, and both kernels of a pair are launched: each workgroup leaves at once if its (batch, head) slab's
  //     tile count belongs to the other (an empty launch costs 3-10 us).
  //   block 64 / d 64: 48 heads of 17 776 tokens, 13 344 workgroups: lock-step 1.24 ms, pipelined 1.31 ms
  //     (four wavefronts per SIMD against two: vector throughput decides); 2 heads of 1 024 tokens,
  //     32 workgroups: pipelined 12 us, lock-step 17 us (one wavefront's own speed decides).  The
  //     line is drawn where the pipelined kernel's workgroups (four per compute unit) stop being all
  //     resident at once.
  //   block 128 / d 64 and block 64 / d 128: the pipelined kernel has two workgroups per compute unit and
  //     is the faster one as long as they all start at once (512; block 64 / d 128, 16 .. 512 workgroups:
  //     1.25-1.5x) and where a few long rows decide (lists with always-kept prefix blocks or uneven rows:
  //     up to 1.5x).  With more workgroups and rows of one length the lock-step kernel shares a compute
  //     unit between more of them.  Without lists, 632 workgroups of 79 tiles: 303 us against 325 at
  //     block 128 / d 64, 166 us against 197 at block 64 / d 128.  There full rounds of 512 are an
  //     exception (three of 128 tiles: 565 against 500) and so are 1025 .. 1536 workgroups, three rounds
  //     that the lock-step kernel's 1024 at a time do not fill either (1264: 302 and 292).  Lists hide their
  //     lengths from the host and stay pipelined: rows of one length are then 2-6 % slower than
  //     lock-step beyond 1000 workgroups (11 % at 1600 of 10 tiles, block 64 / d 128), uneven ones up to
  //     1.5x faster.
  //   block 64 without lists: the wide kernel, whose workgroups of 256 rows move a quarter of the bytes per product, where
  //     rows are long and its rounds of 256 workgroups are filled.  d 128, workgroups x tokens: 192 x 4 030 146 -> 131 us,
  //     256 x 8 100 332 -> 256, 384 x 8 100 492 -> 432, 768 x 8 100 982 -> 741, 3072 x 32 760 15.8 -> 10.8 ms; 384 x 4 030
  //     equal, 128 x 8 100 169 and 208.  d 64: 256 x 8 100 193 -> 180, 768 x 8 100 555 -> 507, 3072 x 32 760 8.06 -> 6.97
  //     ms; 384 x 8 100 307 and 326, 448 x 8 100 316 and 335, 256 x 4 030 98 and 103.  (Block 128 / d 64: 1.03-1.05x at 32 760 tokens, 0.8-1.0
  //     below: not taken.  With lists at d 64 a wavefront's own copies bound it: 1461 us and 1526 at block 64, 48 heads
  //     of 17 776 tokens.)
  //   pooled tokens, block 128 / d 128, ping-pong relative to wide, the same inputs: 896 .. 1600 query blocks 1.02-1.20 (12 heads of
  //     32 760 tokens 1.85 -> 1.57 ms); 512 of one length 1.03-1.3, uneven 0.69-1.03; 576 .. 768 0.93-1.02; prefix blocks as above;
  //     rows of at most 8 blocks 1.04-1.18 beyond 256.
  //     Other shapes: pipelined, except at d 64 where all ping-pong
  //     workgroups (two groups of wavefronts per query block) start at once and their rows are long: from
  //     16 tiles at block 128 (144 workgroups: 14 tiles 37 us against 35 pipelined, 36 tiles 65 against
  //     76, 144 tiles 199 against 269) and 24 at block 64 (512 workgroups: 8 tiles 30 against 25, 26
  //     tiles 45 and 48, 128 tiles 130 against 177).  Lists hide their lengths: an eighth of the blocks is
  //     assumed (fixed budgets keep a quarter, the threshold alone a few per cent).
  // The ping-pong kernel addresses K tiles by 32-bit byte offsets inside a slab: slabs of 4 GiB and
  // more take the wide and the lock-step kernel.  The tests can force the lock-step (1), the ping-pong (2) or the wide
  // kernel (4) where the shape has it (asa_test_force_fwd_kernel).
  const bool fits32 = (uint64_t)a.Nb * BLK * (uint64_t)a.tk.sL * 2u < 0xFFFFFFFFull;
  const bool pooled = a.Nbg > 0, dense = a.row_ptr == nullptr;
  if (pooled && (!fits32 || a.Nb + a.Nbg > kMaxNb || a.tk.sL != D)) return hipErrorNotSupported;
  // What the parameters of the rule say about lists that come from it (any others are served as well, at another speed):
  // rows of about one length; a few rows much longer than the rest, in the units of the comparison above
  const bool prefix = !dense && pb.n_prefix_blocks > 0;
  const bool even_rows = dense || (pb.m_min == pb.m_max && !prefix);
  const bool long_rows = prefix && (int64_t)a.Nb * 512 * 2 > (int64_t)total * pb.m_min * 3;
  constexpr bool kPingPongShape = BLK == 128 && D == 128, kSmallTile = BLK == 64 && D == 64;
  FwdArgs b = a;
  b.select = 0;
  if constexpr (!kPingPongShape) {
    if constexpr (BLK == 64) {
      if (small_shape_wide(pb, dense, pooled)) {
        b.Nb = (a.L + 127) / 128;
        return launch_wide<128, D, 4, false>(b, st);
      }
    }
    if (pooled) {
      if constexpr (D == 64)
        if (small_shape_ping_pong(pb, dense)) return launch_ping_pong<BLK, D, true>(b, grid, st);
      return pipe_in_two(pb, dense, a.Nbg) ? launch_pipe<BLK, D, true, 2>(b, grid, st) : launch_pipe<BLK, D, true, 1>(b, grid, st);
    }
    if (small_shape_pipe(pb, dense))
      return pipe_in_two(pb, dense, 0) ? launch_pipe<BLK, D, false, 2>(b, grid, st) : launch_pipe<BLK, D, false, 1>(b, grid, st);
  } else {
    // Rounds of ping-pong workgroups (one per compute unit); a round of the wide kernel takes as long as two of them.
    const int rounds = (total + 255) / 256, forced = forced_fwd_kernel();
    constexpr int kMinTiles = 18;
    if (pooled) {
      const bool pays = a.Nb <= 8 ? rounds > 1 : rounds > 3 || (rounds == 2 && even_rows);
      const bool wide = forced == 4 || (forced == 0 && pays && !long_rows);
      return wide ? launch_wide<BLK, D, 2, true>(b, st) : launch_ping_pong<BLK, D, true>(b, grid, st);
    }
    if (forced == 4) return dense ? launch_wide<BLK, D, 4, false>(b, st) : launch_wide<BLK, D, 2, false>(b, st);
    if (fits32 && forced == 2) return launch_ping_pong<BLK, D, false>(b, grid, st);
    // Up to three quarters of a workgroup per compute unit: two groups of wavefronts per row, pipelined, take the place of the
    // lock-step kernel where rows have more than two blocks.  Where the host knows the lengths one kernel is launched, not two.
    // Lock-step (with what ping-pong's empty launch costs) and this, us: 37 blocks, 1 head, 4 / 11 tiles 20.5 / 44.5 and 16.1 / 30.1,
    // 4 heads 21 / 45 and 17 / 33, prefix rows among short ones 127 and 87; 62 blocks, 6 tiles 30 and 21; 13 blocks, 2 tiles 10.8 and
    // 11.8, 4 tiles 17.1 and 15.9; no lists, 12 heads, 4, 7, 13 blocks: 17.5, 26, 45 and 16.5, 22, 35.  (256 workgroups, two of
    // whose wavefronts share every SIMD then: 31 and 27, ping-pong's rows 54 and 53.)
    const bool few = forced == 0 && total <= 192 && (dense ? a.Nb : std::min(a.Nb, pb.m_max + pb.n_prefix_blocks)) > 2;
    if (few && (a.Nb < kMinTiles || (!dense && even_rows && pb.m_min < kMinTiles))) return launch_pipe<BLK, D, false, 2>(b, grid, st);
    if (few && even_rows && fits32) return launch_ping_pong<BLK, D, false>(b, grid, st);
    if (forced == 0 && dense) {
      const bool filled = 2 * ((a.n_slabs * ((a.L + 255) / 256) + 255) / 256) <= rounds;
      const bool wide = a.Nb >= 48 ? filled || rounds > 7 : filled && a.Nb >= 8 && (a.Nb < 24 || rounds > 2);
      if (wide) return launch_wide<BLK, D, 4, false>(b, st);
      if (fits32 && a.Nb >= kMinTiles) return launch_ping_pong<BLK, D, false>(b, grid, st);
    } else if (forced == 0) {
      const bool wide = !long_rows && (rounds > 7 || (rounds % 2 == 0 && even_rows));
      if (a.Nb >= kMinTiles && (wide || fits32)) {
        b.select = 1;
        b.select_min_tiles = kMinTiles;
        const hipError_t e = wide ? launch_wide<BLK, D, 2, false>(b, st) : launch_ping_pong<BLK, D, false>(b, grid, st);
        if (e != hipSuccess) return e;
        b.select = -1;
        return few ? launch_pipe<BLK, D, false, 2>(b, grid, st) : launch_lock_step<BLK, D, false>(b, grid, st);
      }
    }
    timing_begin(st);
    return launch_lock_step<BLK, D, false>(b, grid, st);
  }
  // The lock-step kernel reads V's rows or their transposed copy.  Block 64 / d 64: 1.25 ms, or 1.20 ms +
  // 0.035 for the copy (48 heads of 17 776 tokens).  Mixed shapes: the rows cost more per tile, the copy costs
  // the same whatever the length of the rows; equal at about 3 500 keys per row (block 64 / d 128: 16 tiles
  // 43 and 48 us, 79 tiles 170 and 166; block 128 / d 64: 20 tiles 109 and 118, 79 tiles 311 and 303).
  if constexpr (!kPingPongShape) {
    const bool copy_v = kSmallTile || a.L >= 3584;
    if (copy_v) {
      const hipError_t e = launch_transpose(a.v, a.tv, a.H, a.L, a.Lpad, BLK, D, a.n_slabs, a.vt, st);
      if (e != hipSuccess) return e;
    }
    timing_begin(st);
    if constexpr (kSmallTile) return launch_lock_step<BLK, D, true>(b, grid, st);
    else return copy_v ? launch_lock_step<BLK, D, true>(b, grid, st) : launch_lock_step<BLK, D, false>(b, grid, st);
  }
}

hipError_t launch_fwd(const Problem &pb, const void *q, const void *k, const void *v, const void *vt,
                      const int32_t *row_ptr, const int32_t *col_idx, void *o, void *o_lo,
                      float *lse, const int32_t *order, hipStream_t st, const GlobalTokens *gt) {
  FwdArgs a;
  a.order = order;
  a.kg = gt ? gt->kg : nullptr;
  a.vgt = gt ? reinterpret_cast<const bf16 *>(gt->vgt) : nullptr;
  a.Lg = gt ? gt->Lg : 0;
  a.Nbg = gt ? gt->Nbg : 0;
  a.bias_log2 = gt ? log2f((float)gt->n) : 0.f;
  a.q = q; a.k = k; a.v = v; a.vg = gt ? gt->vg : nullptr; a.vt = reinterpret_cast<const bf16 *>(vt);
  a.row_ptr = row_ptr; a.col_idx = col_idx; a.o = o; a.o_lo = o_lo; a.lse = lse;
  a.tq = pb.q; a.tk = pb.k; a.tv = pb.v; a.to = pb.o;
  a.H = pb.H; a.L = pb.L; a.Lpad = pb.Lpad; a.Nb = pb.Nb; a.n_slabs = pb.n_slabs;
  a.scale_log2e = pb.scale * 1.44269504088896340736f;
  a.select = 0;
  a.select_min_tiles = 0;
  if (pb.block == 128 && pb.d == 128) return launch_fwd_t<128, 128>(a, pb, st);
  if (pb.block == 128 && pb.d == 64) return launch_fwd_t<128, 64>(a, pb, st);
  if (pb.block == 64 && pb.d == 128) return launch_fwd_t<64, 128>(a, pb, st);
  if (pb.block == 64 && pb.d == 64) return launch_fwd_t<64, 64>(a, pb, st);
  return hipErrorInvalidValue;
}

}  // namespace asa
