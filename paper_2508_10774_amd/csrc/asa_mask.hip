// Mask generation for gfx950: block importance map (Alg. 2 -> Alg. 1 of the paper's appendix),
// the threshold rule (Alg. 3 steps 6-11) and the CSR / CSC index lists that drive the
// block-sparse attention kernels.
#include <type_traits>
#include <utility>

#include "asa_common.hpp"
#include "asa_tiles.hpp"

namespace asa {

// ---------------------------------------------------------------------------------------
// Probe: P_imp[i][j] = max over sampled rows of block i and sampled keys of block j of the
// soft-max (over ALL sampled keys of the slab) of scale * Qs Ks^T.
//
// Alg. 1 of the paper, reorganised for 64-wide wavefronts.  A workgroup of 4 wavefronts owns 8
// query blocks, two per wavefront, and sweeps one of the four shares of its slab's key blocks.  The sampled key rows (Alg. 2
// steps 1-3) are gathered from K by direct global->LDS loads, 4 key blocks (64 rows) per
// chunk, double-buffered and shared by all wavefronts.  One chain of 32x32x16
// bf16 MFMAs gives a 32 x 32 logit tile: 2 key blocks x 16 samples on the M axis, 2 query
// blocks x 16 samples on the N axis.  The rows of the A operand are ordered so that lane half h
// holds, for ONE sampled query, all 16 samples of key block j0 + h: the block-row maximum
// Rt[query][j] of Alg. 1 is then a lane-local maximum, and the running reference / denominator of
// the row is kept lane-locally over the key blocks of that parity and merged across the two
// halves once, at the end.  No cross-lane traffic inside the
// sweep.  Rt (unscaled logits) and each wavefront's (reference, denominator) pair go to a
// workspace in global memory; finish_rule_kernel merges the pairs of a sampled row, turns Rt
// into probabilities, max-pools over the sampled rows and applies the rule to the row.
// ---------------------------------------------------------------------------------------
struct ProbeArgs {
  const void *q, *k;
  float *p_imp;
  float *rt;         // workspace [query group][pair][Nb rounded up to 8][32]: block-row maxima
  float *stat_r;     // workspace [query group][share][pair][32]: reference exponent of the share's keys
  double *stat_l;    //           and the denominator relative to 2^reference
  TensorView tq, tk;
  int H, L, Nb, n_slabs, block, ks;
  int64_t chunk_bytes;   // from a chunk's first token to the next one's
  int n_full_chunks; // chunks with no token >= L (none if a chunk's rows span 4 GiB or more: 32-bit offsets)
  int n_valid_last;  // sampled tokens of the last block that lie below L
  float c2;          // scale * log2(e)
  float rest;        // ln(2) * what the rounding of c2 left out
  float s_bound;     // kMaxExactExponent / c2
  uint32_t offs[kMaxSamples / 4];   // sample positions inside a block (below 128), a byte each
  const uint8_t *table;   // per-block sample positions [slab][Nb][ks] (TAB kernels), else null
};

constexpr int kProbeQBlocks = 8;   // query blocks per workgroup
constexpr int kProbeKBlocks = 4;   // key blocks per LDS chunk: two pairs, one 32 x 32 logit tile per wavefront each
constexpr int kProbePairs = kProbeQBlocks / 2;
constexpr int kProbePad = 8;       // the rows of block maxima are this many key blocks long, rounded up
// The key blocks of a slab are cut into four shares, each with a reference and a denominator of its own: the first and the second
// half of the even chunks and of the odd ones, one workgroup per share.  The cut is the same whatever the size of the call, so a head's
// map is too: a share's numerators and denominator are rounded relative to the share's own reference.  (Contiguous ranges, as many as
// the chip holds at once: 2 % of a map's entries differed in the last bits with the number of heads.  Two of them instead of four shares,
// us for the whole mask: 12 heads of 256 blocks, d = 128, 90.7 and 91.8; 24 heads of 313, d = 64, 190 and 187; 1 head of 256, 47 and 38.)
constexpr int kProbeShares = 4;

// The exponent of 2 of a raw logit s is s * c2 with c2 = scale * log2(e), rounded to fp32.  What the
// rounding leaves out multiplies exp2(s * c2) by 1 + s * rest.  That is used up to this exponent (logits
// beyond it are themselves rounded by more than that).
constexpr float kMaxExactExponent = 8192.f;

// chunk-position swizzle of the sampled-key rows in LDS (16 rows read together differ in row
// bits 0..2 and 4; at D = 64 a row is half the banks and parity picks the half)
template <int D>
__device__ __forceinline__ int probe_swz(int row) {
  return D == 128 ? ((row & 7) | (((row >> 4) & 1) << 3)) : (((row >> 1) & 3) | (((row >> 4) & 1) << 2));
}

// Bound: the vector ALU.  An entry costs an exponential (8 cycles of 64 lanes), a multiply-add, an addition and half a
// maximum (10), 576 cycles per wavefront and chunk, beside 512 (d = 128) or 256 matrix cycles; with what a chunk costs
// as a whole the vector ALU is busy 87 % of the cycles at d = 64 (48 heads, Nb = 278) and 70 % at d = 128 (12 heads,
// Nb = 256).  So the products of the next chunk stand between the vector instructions of this one, and one wavefront
// takes whole chunks (against 8 wavefronts that share chunks of twice the size and run products and vector work one behind the
// other: 75 -> 66 us at d = 128, 252 -> 220 us at d = 64).  Three wavefronts per SIMD: two (256 registers), with chunks of
// 4 or of 8 key blocks, are 3 % slower for the whole mask.
// TAB: the sample positions differ from block to block and come from a table (seeded random
// sampling) instead of one offset vector for all blocks.
template <int D, bool TAB>
__global__ __launch_bounds__(256, 3) void probe_kernel(ProbeArgs a) {
  constexpr int ROWS = kProbeKBlocks * 16;          // sampled rows per chunk
  constexpr int CH = D / 8;                         // 16-byte chunks per row
  constexpr int DMA_PER_WAVE = ROWS * CH / 64 / kProbePairs;  // 1 KB per wave instruction
  constexpr int NT = kProbeKBlocks / 2;             // logit tiles per chunk
  __shared__ __align__(1024) bf16 Kc[2][ROWS * D];

  const int n_groups = (a.Nb + kProbeQBlocks - 1) / kProbeQBlocks;
  const int item = xcd_contiguous_work(blockIdx.x, a.n_slabs * n_groups * kProbeShares);
  if (item < 0) return;
  const int work = item / kProbeShares, share = item % kProbeShares;   // (slab, query group)
  const int slab = work / n_groups;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int pair = wave;          // which two query blocks
  const int i_base = (work - slab * n_groups) * kProbeQBlocks;
  const int i0 = i_base + 2 * pair;
  const int hl = lane >> 5;  // operand k-half on loads, key-block parity on results
  const int n = lane & 31;   // A row on loads; query column on results
  const int nb_pad = (a.Nb + kProbePad - 1) / kProbePad * kProbePad;
  float *rt = a.rt + ((int64_t)work * kProbePairs + pair) * nb_pad * 32;

  const bf16 *qs = slab_ptr(a.q, a.tq, slab, a.H);
  const bf16 *ks = slab_ptr(a.k, a.tk, slab, a.H);

  // TAB: this slab's table in LDS, 16 entries to a block whatever ks, so that the entries of a lane's rows are constant distances
  // apart (with as many entries as samples the sweep spilled registers for the indexes and their masks; 48 heads of 278 blocks, d = 128,
  // seeded mask 445 -> 391 us).  Positions ascend inside a block, so the samples of the last block that lie below L are a prefix.
  __shared__ uint8_t tab[TAB ? kMaxNb * kMaxSamples : 1];
  int n_valid_last = a.n_valid_last;
  if (TAB) {
    const uint8_t *g = a.table + (int64_t)slab * a.Nb * a.ks;
    const int u = min(tid % kMaxSamples, a.ks - 1);          // (slots beyond the last sample repeat it)
#pragma unroll 4
    for (int t = tid; t < a.Nb * kMaxSamples; t += 256) tab[t] = g[t / kMaxSamples * a.ks + u];
    __syncthreads();
    n_valid_last = 0;
    for (int u = 0; u < a.ks; ++u)
      if ((a.Nb - 1) * a.block + tab[(a.Nb - 1) * kMaxSamples + u] < a.L) ++n_valid_last;
  }
  auto offset_of = [&](int blk, int u) {
    if (TAB) return (int)tab[blk * kMaxSamples + u];      // (any value for blocks past the last one: they start at or past L)
    // (from scalar registers: an indexed read of the kernel's arguments is a load from memory, which all that follows would wait for)
    const uint32_t lo = u & 4 ? a.offs[1] : a.offs[0], hi = u & 4 ? a.offs[3] : a.offs[2];
    return (int)(((u & 8 ? hi : lo) >> (8 * (u & 3))) & 255u);
  };
  auto valid_in_block = [&](int blk) {
    return blk >= a.Nb ? 0 : (blk == a.Nb - 1 ? n_valid_last : a.ks);
  };

  // B operand: column n = sampled query (n & 15) of query block i0 + (n >> 4)
  const int q_blk = i0 + (n >> 4);
  const bool q_ok = (n & 15) < valid_in_block(q_blk);
  bf16x8 qreg[D / 16];
  {
    const int64_t qpos = q_ok ? (int64_t)q_blk * a.block + offset_of(q_blk, n & 15) : 0;
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
      qreg[s] = *reinterpret_cast<const bf16x8 *>(qs + qpos * a.tq.sL + 16 * s + 8 * hl);
  }

  // producer: my share of a chunk of sampled key rows (row r of a chunk = key block r / 16,
  // sample r % 16)
  const uint32_t lds_at = ASA_LDS_ADDR_OF(Kc);
  // (addresses of a chunk come from its number by scalar arithmetic, at each use: pointers that run along
  // would be kept in vector registers)
  auto opaque = [](int chunk) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(chunk));
#endif
    return chunk;
  };
  auto lds_of = [&](int i, int buf) { return lds_at + (uint32_t)(buf * ROWS * D * 2 + (wave * DMA_PER_WAVE + i) * 1024); };
  auto row_of = [&](int i, int l) { return (wave * DMA_PER_WAVE + i) * (64 / CH) + l / CH; };
  auto pos_of = [&](int i, int l) { return ((l % CH) ^ probe_swz<D>(row_of(i, l))) * 8; };   // swizzled 16-byte position
  auto fetch = [&](int chunk, int buf) __attribute__((always_inline)) {
    int l = lane;
#if defined(__HIP_DEVICE_COMPILE__)
    if (!TAB) asm volatile("" : "+v"(l));   // (rare: nothing of it is to be kept in registers across the sweep)
#endif
#pragma unroll
    for (int i = 0; i < DMA_PER_WAVE; ++i) {
      const int row = row_of(i, l), blk = chunk * kProbeKBlocks + row / 16;
      const int tok = blk * a.block + offset_of(blk, row % 16);
      const uint32_t at = tok < a.L ? tok : 0;   // padded samples: any valid row, masked out below
      lds_dma16_v(reinterpret_cast<const char *>(ks) + (uint64_t)at * (uint32_t)(a.tk.sL * 2) + 2 * pos_of(i, l), lds_of(i, buf));
    }
  };

  // The common case of that, with all address arithmetic taken out of the sweep: one offset
  // vector for all blocks and a chunk that lies wholly below L.  Per lane a byte offset inside
  // the chunk, per chunk one wave-uniform base.
  uint32_t dma_off0[DMA_PER_WAVE];   // bytes from the first token of the chunk
#pragma unroll
  for (int i = 0; i < DMA_PER_WAVE; ++i) {
    const uint32_t tok = (row_of(i, lane) / 16) * a.block + (TAB ? 0 : offset_of(0, row_of(i, lane) % 16));
    dma_off0[i] = (tok * (uint32_t)a.tk.sL + (uint32_t)pos_of(i, lane)) * 2;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(dma_off0[i]));      // (else kept as the low half of a 64-bit product)
#endif
  }
  auto fetch_any = [&](int chunk, int buf) __attribute__((always_inline)) {
    if (!TAB && chunk < a.n_full_chunks) {
      const char *base = reinterpret_cast<const char *>(ks) + opaque(chunk) * a.chunk_bytes;   // wave-uniform
#pragma unroll
      for (int i = 0; i < DMA_PER_WAVE; ++i) lds_dma16_sv(base, dma_off0[i], lds_of(i, buf));
    } else {
      fetch(chunk, buf);
    }
  };

  // consumer: A row r = 8g + 4h + j is sample 4g + j of key block j0 + h
  const int a_row = ((n >> 2) & 1) * 16 + 4 * (n >> 3) + (n & 3);   // row inside a pair of key blocks
  const int a_swz = probe_swz<D>(a_row);
  // my fragment s of the first pair of key blocks of a chunk in buffer 0 (LDS address); the
  // second pair and the other buffer are constant distances away
  uint32_t a_at[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) a_at[s] = lds_at + (uint32_t)((a_row * D + (((2 * s + hl) ^ a_swz) * 8)) * 2);
  const uint32_t rt_off = hl * 32 + n;       // where my block-row maxima of a chunk's first pair go (floats)

  float rt_pend[NT];     // block-row maxima of the chunk just swept
  float Rr = -INFINITY;  // reference exponent of my query over the key blocks of parity hl (an integer)
  double lt = 0.0;       // running denominator over the same keys, relative to 2^Rr
  const float c2 = a.c2;
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // One turn of the sweep, a software pipeline inside each wavefront: the products of chunk t + 1 (out of
  // LDS buffer BUF, a compile-time constant: every LDS address is a per-lane register plus an
  // immediate) and between them, slot by slot, the maxima and exponentials of chunk t.
  // The exponentials are taken relative to the power of two at or below the running maximum's, brought up
  // to date first (no branch for it): one fp64 update per 32 keys, and neither the reference nor a
  // change of it is rounded (at or below: no numerator underflows that would not underflow relative
  // to the maximum).  finish_rule_kernel forms the numerators from the same product s * c2; the rest of
  // the rounded c2 is put right there per entry and here per chunk.
  constexpr int kNE = NT * (D / 16);              // products of a chunk
  // LDS operands read this many products ahead (d = 128: one more spills registers in the sweep; 12 heads, whole mask, 90.9 and 89.9 us)
  constexpr int kRing = D == 128 ? 3 : 4, kDepth = kRing - 1;
  constexpr int kMaxSlots = kNE / 4;              // slots that form the maxima; the exponentials fill the others
  auto turn = [&](int chunk, auto buf_tag, auto mul_tag, auto vec_tag, f32x16 (&cur)[NT], f32x16 (&nxt)[NT])
      __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf_tag)::value;
    constexpr bool kMul = decltype(mul_tag)::value, kVec = decltype(vec_tag)::value;
    bf16x8 ring[kRing];
    auto read = [&](auto e_tag) __attribute__((always_inline)) {
      constexpr int e = decltype(e_tag)::value, sb = e / (D / 16), s = e % (D / 16);
      ring[e % kRing] = lds_read<bf16x8>(a_at[s] + (uint32_t)((BUF * ROWS + sb * 32) * D * 2));
    };
    if constexpr (kMul)
      [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
        (read(std::integral_constant<int, E>{}), ...);
      }(std::make_integer_sequence<int, kDepth>{});
    if (kVec && (a.ks < kMaxSamples || (chunk + 1) * kProbeKBlocks >= a.Nb)) {
      // register i of lane half hl is sample i of key block j0 + hl; samples past L (only in
      // the last block), past the last block, or in sample slots >= k are masked out
#pragma unroll
      for (int sb = 0; sb < NT; ++sb) {
        const int nv = valid_in_block(chunk * kProbeKBlocks + 2 * sb + hl);
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (i >= nv) cur[sb][i] = -INFINITY;
      }
    }
    float mraw[NT], sum[NT], mnew = -INFINITY, bias = 0.f;
    int shift = 0;
#pragma unroll
    for (int sb = 0; sb < NT; ++sb) mraw[sb] = -INFINITY, sum[sb] = 0.f;
    __builtin_amdgcn_sched_barrier(0);
    [&]<int... E>(std::integer_sequence<int, E...>) __attribute__((always_inline)) {
      ([&]() __attribute__((always_inline)) {
        constexpr int e = E;
        if constexpr (kMul) {
          constexpr int sb = e / (D / 16), s = e % (D / 16);
          if constexpr (e + kDepth < kNE) read(std::integral_constant<int, e + kDepth>{});
          nxt[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[e % kRing], qreg[s], s == 0 ? zero16 : nxt[sb], 0, 0, 0);
        }
        if constexpr (kVec && e < kMaxSlots) {
          constexpr int i0 = e * 16 / kMaxSlots, i1 = (e + 1) * 16 / kMaxSlots;
#pragma unroll
          for (int i = i0; i < i1; ++i)
#pragma unroll
            for (int sb = 0; sb < NT; ++sb) mraw[sb] = fmaxf(mraw[sb], cur[sb][i]);
          if constexpr (e == kMaxSlots - 1) {
#pragma unroll
            for (int sb = 0; sb < NT; ++sb) {
              rt_pend[sb] = mraw[sb];                    // block-row maximum, Alg. 1 step 12 (unscaled)
              mnew = fmaxf(mnew, mraw[sb]);
            }
            // Alg. 1 steps 12-15 with the exponentials exp(scale * (s - reference)) as one fused multiply-add
            // and one exp2 each
            const float r_new = fmaxf(Rr, floorf(mnew * c2));
            bias = (r_new == -INFINITY) ? 0.f : -r_new;     // (no key has been seen yet: all sums stay 0)
            shift = (int)fmaxf(Rr - r_new, -2000.f);        // (-inf - x and -inf - -inf: the old sum is 0)
            Rr = r_new;
          }
        }
        if constexpr (kVec && e >= kMaxSlots) {
          // element x of the chunk: tile x % NT, register x / NT; summed one slot after its exponential
          constexpr int n_slots = kNE - kMaxSlots, f = e - kMaxSlots, all = 16 * NT;
          constexpr int x0 = f * all / n_slots, x1 = (f + 1) * all / n_slots;
          constexpr int y0 = f == 0 ? 0 : (f - 1) * all / n_slots, y1 = f == n_slots - 1 ? all : x0;
#pragma unroll
          for (int x = x0; x < x1; ++x) cur[x % NT][x / NT] = fast_exp2(fmaf(cur[x % NT][x / NT], c2, bias));
#pragma unroll
          for (int x = y0; x < y1; ++x) sum[x % NT] += cur[x % NT][x / NT];
        }
        __builtin_amdgcn_sched_barrier(0);
      }(), ...);
    }(std::make_integer_sequence<int, kNE>{});
    if constexpr (kVec)
      lt = fma((double)(sum[0] + sum[1]), fma((double)__builtin_amdgcn_fmed3f(mnew, -a.s_bound, a.s_bound), (double)a.rest, 1.0),
               __builtin_amdgcn_ldexp(lt, shift));
  };

  // The block-row maxima of a chunk are stored at the start of the turn after its own, just before
  // loads are requested: the wait for those loads at the top of the turn after that also
  // waits for the stores (one counter), and a store issued in the middle of a turn was not yet
  // acknowledged at its end.
  auto store_rt = [&](int chunk) __attribute__((always_inline)) {
    float *rt_c = rt + (int64_t)opaque(chunk) * kProbeKBlocks * 32;
#pragma unroll
    for (int sb = 0; sb < NT; ++sb) rt_c[rt_off + sb * 64] = rt_pend[sb];
  };
  // my chunks: every other one from c0 on
  constexpr int kStep = 2;
  const int n_chunks = (a.Nb + kProbeKBlocks - 1) / kProbeKBlocks, per_half = (n_chunks + 3) / 4 * 2;
  const int c0 = share / 2 * per_half + share % 2, c1 = min(n_chunks, (share / 2 + 1) * per_half);
  f32x16 s0[NT], s1[NT];
  using Yes = std::true_type;
  using No = std::false_type;
  using Buf0 = std::integral_constant<int, 0>;
  using Buf1 = std::integral_constant<int, 1>;
  // the loads of a chunk have landed (everyone's), and nobody reads the other buffer any more
  auto landed = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
  };
  if (c0 < c1) {
    fetch_any(c0, 0);
    landed();
    if (c0 + kStep < c1) fetch_any(c0 + kStep, 1);
    turn(c0, Buf0{}, Yes{}, No{}, s1, s0);       // the products of my first chunk
    for (int chunk = c0;; chunk += 2 * kStep) {
      // s0: products of `chunk`, whose successor is in buffer 1
      if (chunk + kStep >= c1) {
        if (chunk > c0) store_rt(chunk - kStep);
        turn(chunk, Buf1{}, No{}, Yes{}, s0, s1);
        store_rt(chunk);
        break;
      }
      landed();
      if (chunk > c0) store_rt(chunk - kStep);
      if (chunk + 2 * kStep < c1) fetch_any(chunk + 2 * kStep, 0);
      turn(chunk, Buf1{}, Yes{}, Yes{}, s0, s1);
      if (chunk + 2 * kStep >= c1) {
        store_rt(chunk);
        turn(chunk + kStep, Buf0{}, No{}, Yes{}, s1, s0);
        store_rt(chunk + kStep);
        break;
      }
      landed();
      store_rt(chunk);
      if (chunk + 3 * kStep < c1) fetch_any(chunk + 3 * kStep, 1);
      turn(chunk + kStep, Buf0{}, Yes{}, Yes{}, s1, s0);
    }
  }
  // merge the two parities of each query; the pair (reference, denominator) of my share of the
  // keys goes to the workspace (the kernel that follows merges the shares)
  {
    const float Ro = __shfl_xor(Rr, 32, 64);
    const double lo = __shfl_xor(lt, 32, 64);
    const float Rall = fmaxf(Rr, Ro);
    const double lall = __builtin_amdgcn_ldexp(lt, (int)fmaxf(Rr - Rall, -2000.f)) +
                        __builtin_amdgcn_ldexp(lo, (int)fmaxf(Ro - Rall, -2000.f));
    if (hl == 0) {
      a.stat_r[((int64_t)item * kProbePairs + pair) * 32 + n] = Rall;
      a.stat_l[((int64_t)item * kProbePairs + pair) * 32 + n] = lall;
    }
  }
}

static size_t probe_groups(const Problem &pb) {
  return (size_t)pb.n_slabs * ((pb.Nb + kProbeQBlocks - 1) / kProbeQBlocks);
}
static size_t probe_rt_bytes(const Problem &pb) {
  const size_t nb_pad = (pb.Nb + kProbePad - 1) / kProbePad * kProbePad;
  return (probe_groups(pb) * kProbePairs * nb_pad * 32 * sizeof(float) + 255) & ~(size_t)255;
}
static size_t probe_items(const Problem &pb) { return probe_groups(pb) * kProbeShares; }
size_t probe_workspace_bytes(const Problem &pb) {
  // block-row maxima, then the per-wavefront soft-max statistics (fp64 denominators first)
  return probe_rt_bytes(pb) + probe_items(pb) * kProbePairs * 32 * (sizeof(double) + sizeof(float));
}

static void fill_probe_args(const Problem &pb, const void *q, const void *k, float *p_imp,
                            void *workspace, const uint8_t *table, ProbeArgs *a) {
  a->table = table;
  a->q = q; a->k = k; a->p_imp = p_imp;
  unsigned char *ws = reinterpret_cast<unsigned char *>(workspace);
  a->rt = reinterpret_cast<float *>(ws);
  a->stat_l = reinterpret_cast<double *>(ws + probe_rt_bytes(pb));
  a->stat_r = reinterpret_cast<float *>(ws + probe_rt_bytes(pb) + probe_items(pb) * kProbePairs * 32 * sizeof(double));
  a->tq = pb.q; a->tk = pb.k;
  a->H = pb.H; a->L = pb.L; a->Nb = pb.Nb; a->n_slabs = pb.n_slabs; a->block = pb.block; a->ks = pb.ks;
  a->chunk_bytes = (int64_t)kProbeKBlocks * pb.block * pb.k.sL * 2;
  a->n_full_chunks = a->chunk_bytes >= ((int64_t)1 << 32) ? 0 : pb.L / (kProbeKBlocks * pb.block);
  a->c2 = pb.scale * 1.44269504088896340736f;
  a->rest = (float)(((double)pb.scale * 1.44269504088896340736 - (double)a->c2) * 0.69314718055994530942);
  a->s_bound = fminf(kMaxExactExponent / a->c2, 3.0e38f);   // (finite: the -inf of a tile without keys is bounded too)
  for (int u = 0; u < kMaxSamples; u += 4)
    a->offs[u / 4] = (uint32_t)pb.offs[u] | (uint32_t)pb.offs[u + 1] << 8 | (uint32_t)pb.offs[u + 2] << 16 | (uint32_t)pb.offs[u + 3] << 24;
  a->n_valid_last = 0;
  for (int u = 0; u < pb.ks; ++u)
    if ((int64_t)(pb.Nb - 1) * pb.block + pb.offs[u] < pb.L) ++a->n_valid_last;
}

hipError_t launch_probe(const Problem &pb, const void *q, const void *k, void *workspace,
                        hipStream_t st, const uint8_t *table) {
  ProbeArgs a;
  fill_probe_args(pb, q, k, nullptr, workspace, table, &a);
  const dim3 grid(xcd_grid((int)probe_items(pb))), block(64 * kProbePairs);
  if (pb.d == 128 && table) hipLaunchKernelGGL((probe_kernel<128, true>), grid, block, 0, st, a);
  else if (pb.d == 128) hipLaunchKernelGGL((probe_kernel<128, false>), grid, block, 0, st, a);
  else if (table) hipLaunchKernelGGL((probe_kernel<64, true>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((probe_kernel<64, false>), grid, block, 0, st, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Seeded random sampling (Alg. 3 step 2 made reproducible).  Philox-4x32 with 10 rounds
// (Salmon et al., SC'11) gives position j of block `blk` of slab `slab` the word
// Philox(counter = (j, blk, slab, 0), key = seed)[0]; the k positions with the smallest
// (word, j) are the block's sample, written in ascending position.  One wavefront per block.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t philox4x32_10_word0(uint32_t c0, uint32_t c1, uint32_t c2,
                                                        uint32_t c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n1 = (uint32_t)p1;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1, n3 = (uint32_t)p0;
    c0 = n0; c1 = n1; c2 = n2; c3 = n3;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c0;
}

__global__ __launch_bounds__(64) void sample_offsets_kernel(uint32_t seed_lo, uint32_t seed_hi,
                                                            int Nb, int b, int ks, uint8_t *table) {
  __shared__ uint64_t word[128];   // (philox word, position): distinct, so ranks are too
  __shared__ uint8_t chosen[128];
  const int blk = blockIdx.x, slab = blockIdx.y, lane = threadIdx.x;
  for (int j = lane; j < b; j += 64)
    word[j] = ((uint64_t)philox4x32_10_word0((uint32_t)j, (uint32_t)blk, (uint32_t)slab, 0u, seed_lo, seed_hi) << 32) | (uint32_t)j;
  __syncthreads();
  for (int j = lane; j < b; j += 64) {
    int rank = 0;
    for (int x = 0; x < b; ++x) rank += word[x] < word[j];
    chosen[j] = rank < ks;
  }
  __syncthreads();
  if (lane == 0) {
    uint8_t *out = table + ((int64_t)slab * Nb + blk) * ks;
    int n = 0;
    for (int j = 0; j < b; ++j)
      if (chosen[j]) out[n++] = (uint8_t)j;
  }
}

hipError_t launch_sample_offsets(const Problem &pb, uint64_t seed, uint8_t *table, hipStream_t st) {
  hipLaunchKernelGGL(sample_offsets_kernel, dim3(pb.Nb, pb.n_slabs), dim3(64), 0, st,
                     (uint32_t)seed, (uint32_t)(seed >> 32), pb.Nb, pb.block, pb.ks, table);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Threshold rule (Alg. 3 steps 6-11), one wavefront per row of the importance map.
// The row is sorted by (score descending, block index ascending) with a bitonic network on
// 64-bit keys (inverted order-preserving image of the fp32 score in the high word, the block
// index in the low word).  The keys live in registers, NPAD / 64 consecutive ranks per lane:
// network stages whose partners sit in the same lane are register compare-exchanges, the others
// fetch the partner lane's key through the cross-lane network (no LDS memory traffic: with the
// keys in LDS the kernel was bound by LDS bandwidth).  One lane then forms the fp64 running sums
// c_r in rank order -- the additions happen in exactly the sequence the algorithm states, so the
// decision is bit-identical to a sequential implementation -- then m* = #{r : c_r < tau * T},
// m = clamp(m*, m_min, m_max), keep rank < m.  A NaN score counts as 0.  Where m_min == m_max the m
// best keys are selected without sorting or summing.
// ---------------------------------------------------------------------------------------
struct RuleArgs {
  const float *scores;
  uint8_t *mask;
  int Nb, n_rows, m_min, m_max, n_prefix_blocks;
  float tau;
};

__device__ __forceinline__ uint32_t desc_key(float v) {
  v = (v == v) ? v + 0.0f : 0.0f;                 // NaN -> 0, -0 -> +0
  uint32_t u = __float_as_uint(v);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // ascending order-preserving image
  return ~u;                                       // larger score -> smaller key
}
__device__ __forceinline__ float key_score(uint32_t k) {
  uint32_t u = ~k;
  u = (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u;
  return __uint_as_float(u);
}

// The rule on one row whose Nb scores sit in the wavefront's registers as sort keys, score j in register j / 64 of lane
// j % 64 (key = order image of the score in the high word, block index in the low word; slots
// beyond Nb hold ~0).  cum: NPAD doubles of LDS owned by this wavefront.  Every step is
// wave-synchronous: no workgroup barrier.  Writes the row's Nb mask bytes to dst.
template <int NPAD>
__device__ __forceinline__ void rule_on_keys(unsigned long long (&key)[NPAD / 64], double *cum, int lane,
                                             int i, int Nb, float tau, int m_min, int m_max,
                                             int n_prefix_blocks, uint8_t *dst) {
  constexpr int E = NPAD / 64;               // keys per lane; rank of key r of a lane = lane * E + r
  if (m_min == m_max) {
    // A fixed budget: the running sums cannot change the outcome, the m_min smallest keys are kept.
    // The largest of them is found bit by bit (keys are distinct: the block index is part of them),
    // by counting the keys below a trial value with ballots.
    // A trial value with exactly m_min keys below it ends the search (adjacent scores part after a dozen bits or so, not 32), looked
    // for after every fourth bit; registers that hold padding only are not counted, a question only for the upper half of them.
    // (8 heads of 79 blocks of 64 tokens, this kernel in a mask: all 32 bits 7.0 us; both questions at every bit 7.5-8.1, each a branch of
    // the wavefront; so 6.6.)
    const int used = (Nb + 63) / 64;
    unsigned long long end = 0;              // the keys below it are kept
    uint32_t last = 0, parts = 0;            // score part of the m_min-th smallest key; of a value that parts the kept from the others
    for (uint32_t bits = 1u << 31; bits != 0 && parts == 0; bits >>= 4) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const uint32_t trial = last | bits >> x;
        int n = 0;
#pragma unroll
        for (int r = 0; r < E; ++r)
          if (r <= E / 2 || r < used) n += __popcll(__ballot((uint32_t)(key[r] >> 32) < trial));
        if (n < m_min) last = trial;
        if (n == m_min) parts = trial;
      }
    }
    if (parts != 0) {
      end = (unsigned long long)parts << 32;
    } else {
      // the m_min-th key has this score; of several with it the lower block indices (at most 1023) are in
      unsigned long long at = (unsigned long long)last << 32;
      for (int bit = 9; bit >= 0; --bit) {
        const unsigned long long trial = at | (1ull << bit);
        int n = 0;
#pragma unroll
        for (int r = 0; r < E; ++r)
          if (r <= E / 2 || r < used) n += __popcll(__ballot(key[r] < trial));
        if (n < m_min) at = trial;
      }
      end = at + 1;
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int j = (int)(key[r] & 0xffffffffu);
      if (j < Nb && j >= 0) dst[j] = (key[r] < end) || (i < n_prefix_blocks) || (j < n_prefix_blocks);
    }
    return;
  }
  // ascending bitonic network over e = lane * E + r: stage (k, jj) orders the pair (e, e ^ jj)
  // upwards where (e & k) == 0 and downwards elsewhere
  for (int k = 2; k <= NPAD; k <<= 1) {
    // partners in other lanes: lane ^ (jj / E), same register
    for (int jj = k >> 1; jj >= E; jj >>= 1) {
      const int dl = jj / E;
      const bool up = ((lane * E) & k) == 0;           // (k > jj >= E: decided by the lane)
      const bool keep_min = ((lane & dl) == 0) == up;
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const uint32_t lo = (uint32_t)key[r], hi = (uint32_t)(key[r] >> 32);
        const unsigned long long other =
            ((unsigned long long)(uint32_t)__shfl_xor((int)hi, dl, 64) << 32) | (uint32_t)__shfl_xor((int)lo, dl, 64);
        const bool other_smaller = other < key[r];
        key[r] = (other_smaller == keep_min) ? other : key[r];
      }
    }
    // partners in the same lane: registers r and r ^ jj
#pragma unroll
    for (int jj = E >> 1; jj > 0; jj >>= 1) {
      if (jj < k) {
#pragma unroll
        for (int r = 0; r < E; ++r) {
          if ((r & jj) == 0) {
            const bool up = ((lane * E + r) & k) == 0;
            const unsigned long long x = key[r], y = key[r ^ jj];
            const bool swap = (x > y) == up;
            key[r] = swap ? y : x;
            key[r ^ jj] = swap ? x : y;
          }
        }
      }
    }
  }
  // scores in rank order as fp64, zero-padded
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = lane * E + r;
    cum[e] = e < Nb ? (double)key_score((uint32_t)(key[r] >> 32)) : 0.0;
  }
  __builtin_amdgcn_wave_barrier();
  // Running sums in place: cum[r] becomes c_{r+1} = sum of the r+1 best scores.  Sequential on
  // purpose (see above): one lane, eight values fetched at a time so that only the additions
  // sit on the dependent chain.  Past the last score that is not zero the sum stays what it is
  // (many scores of a peaked row underflow to zero): the chain ends there.
  int n_sum = 0;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = lane * E + r;
    if (e < Nb && key_score((uint32_t)(key[r] >> 32)) != 0.f) n_sum = e + 1;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) n_sum = max(n_sum, __shfl_xor(n_sum, off, 64));
  n_sum = max(n_sum, 1);
  if (lane == 0) {
    double c = 0.0;
    for (int r0 = 0; r0 < n_sum; r0 += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = cum[r0 + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        c = c + v[u];
        v[u] = c;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) cum[r0 + u] = v[u];
    }
  }
  __builtin_amdgcn_wave_barrier();
  const double thr = (double)tau * cum[n_sum - 1];   // tau * T
  int inside = 0;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = lane * E + r;
    if (e < Nb) inside += ((e == 0 ? 0.0 : cum[min(e, n_sum) - 1]) < thr);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) inside += __shfl_xor(inside, off, 64);
  int m = inside;
  m = m < m_min ? m_min : m;
  m = m > m_max ? m_max : m;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = lane * E + r;
    if (e < Nb) {
      const int j = (int)(key[r] & 0xffffffffu);
      dst[j] = (e < m) || (i < n_prefix_blocks) || (j < n_prefix_blocks);
    }
  }
}

// Four rows per workgroup, one per wavefront, so that the sequential running sums of different
// rows run on different SIMDs.
template <int NPAD>
__global__ __launch_bounds__(256) void rule_kernel(RuleArgs a) {
  constexpr int E = NPAD / 64;
  __shared__ double cum_all[4][NPAD];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + wave;          // slab * Nb + i
  if (row >= a.n_rows) return;                     // whole wavefront; no workgroup barriers below
  const float *src = a.scores + (int64_t)row * a.Nb;
  unsigned long long key[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int j = lane + 64 * r;
    key[r] = j < a.Nb ? (((unsigned long long)desc_key(src[j]) << 32) | (unsigned)j)
                      : ~0ull;        // padding sorts last
  }
  rule_on_keys<NPAD>(key, cum_all[wave], lane, row % a.Nb, a.Nb, a.tau, a.m_min, a.m_max,
                     a.n_prefix_blocks, a.mask + (int64_t)row * a.Nb);
}

// ---------------------------------------------------------------------------------------
// Second half of the probe (Alg. 1, second loop) fused with the rule: one wavefront per query
// block.  It merges the soft-max statistics of the wavefronts that swept this block's sampled
// rows (the shares of the key blocks), turns the block-row maxima into
// probabilities, max-pools them over the sampled rows -- the row P_imp[i][:], written out if the
// caller wants it -- and applies the rule to that row while it is still in registers.
// ---------------------------------------------------------------------------------------
template <int NPAD>
__global__ __launch_bounds__(256) void finish_rule_kernel(ProbeArgs a, RuleArgs ra) {
  constexpr int E = NPAD / 64;
  __shared__ double cum_all[4][NPAD];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + wave;          // slab * Nb + i
  if (row >= ra.n_rows) return;
  const int slab = row / a.Nb, i = row - slab * a.Nb;
  const int n_groups = (a.Nb + kProbeQBlocks - 1) / kProbeQBlocks;
  const int nb_pad = (a.Nb + kProbePad - 1) / kProbePad * kProbePad;
  const int work = slab * n_groups + i / kProbeQBlocks;      // the query group that swept this block
  const int w = i % kProbeQBlocks, pr_ = w >> 1, qb = w & 1;  // its pair and position in the pair
  const float *rtq = a.rt + ((int64_t)work * kProbePairs + pr_) * nb_pad * 32 + qb * 16;
  // merge the shares
  // (the denominator is summed in fp64; its reciprocal is kept in two fp32 halves)
  // Lane u < 16 merges the shares of sampled row u; the 16 results are then handed to every
  // lane through scalar registers (all lanes doing all 16 rows cost 16 fp64 divisions a lane).
  float my_r = -INFINITY, my_inv = 0.f, my_inv_lo = 0.f, my_inv_rest = 0.f;
  {
    const int u = lane & 15;
    float pr[kProbeShares];
    double pl[kProbeShares];
#pragma unroll
    for (int x = 0; x < kProbeShares; ++x) {
      const int64_t at = (((int64_t)work * kProbeShares + x) * kProbePairs + pr_) * 32 + qb * 16 + u;
      pr[x] = a.stat_r[at];
      pl[x] = a.stat_l[at];
      my_r = fmaxf(my_r, pr[x]);
    }
    double l = 0.0;
#pragma unroll
    for (int x = 0; x < kProbeShares; ++x) l += __builtin_amdgcn_ldexp(pl[x], (int)fmaxf(pr[x] - my_r, -2000.f));
    const double inv = 1.0 / l;
    my_inv = (float)inv;
    my_inv_lo = (float)(inv - (double)my_inv);
    my_inv_rest = fabsf(my_r) < kMaxExactExponent ? my_inv * a.rest : 0.f;
  }
  float Rrow[16], Linv[16], Linv_lo[16], Linv_rest[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    Rrow[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_r), u));
    Linv[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_inv), u));
    Linv_lo[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_inv_lo), u));
    Linv_rest[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_inv_rest), u));
  }
  int rows_ok = a.ks;                       // sampled rows of this block that lie below L
  if (i == a.Nb - 1) {
    if (a.table) {
      rows_ok = 0;
      const uint8_t *t = a.table + ((int64_t)slab * a.Nb + i) * a.ks;
      for (int u = 0; u < a.ks; ++u) rows_ok += (int64_t)i * a.block + t[u] < a.L;
    } else {
      rows_ok = a.n_valid_last;
    }
  }
  float *out = a.p_imp ? a.p_imp + (int64_t)row * a.Nb : nullptr;
  unsigned long long key[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int j = lane + 64 * r;
    key[r] = ~0ull;                         // padding sorts last
    if (j < a.Nb) {
      const f32x4 *src = reinterpret_cast<const f32x4 *>(rtq + (int64_t)j * 32);
      const f32x4 r0 = src[0], r1 = src[1], r2 = src[2], r3 = src[3];
      const float rv[16] = {r0[0], r0[1], r0[2], r0[3], r1[0], r1[1], r1[2], r1[3],
                            r2[0], r2[1], r2[2], r2[3], r3[0], r3[1], r3[2], r3[3]};
      float best = 0.f;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if (u < rows_ok && rv[u] != -INFINITY) {
          // exp2(s * c2 - R) * (1 + s * rest) / denominator with one rounding of its own: the low parts enter
          // the sum before it
          const float e = fast_exp2(fmaf(rv[u], a.c2, -Rrow[u]));
          best = fmaxf(best, fmaf(e, Linv[u], e * fmaf(rv[u], Linv_rest[u], Linv_lo[u])));
        }
      }
      if (out) out[j] = best;
      key[r] = ((unsigned long long)desc_key(best) << 32) | (unsigned)j;
    }
  }
  if (ra.mask == nullptr) return;   // the caller only wanted the map (wave-uniform)
  rule_on_keys<NPAD>(key, cum_all[wave], lane, i, a.Nb, ra.tau, ra.m_min, ra.m_max, ra.n_prefix_blocks,
                     ra.mask + (int64_t)row * a.Nb);
}

// dst[s][i][j] = max of src[s][i g .. i g + g)[j g .. j g + g) (clipped at n_src): the importance
// map of blocks that are g times as large.  One thread per output element.
__global__ void pool_scores_kernel(const float *src, int n_src, float *dst, int n_dst, int g) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y, s = blockIdx.z;
  if (j >= n_dst) return;
  const float *in = src + (int64_t)s * n_src * n_src;
  float best = 0.f;
  for (int a = i * g; a < min(n_src, i * g + g); ++a)
    for (int b = j * g; b < min(n_src, j * g + g); ++b) best = fmaxf(best, in[(int64_t)a * n_src + b]);
  dst[((int64_t)s * n_dst + i) * n_dst + j] = best;
}
hipError_t launch_pool_scores(const float *src, int n_src, float *dst, int n_dst, int g, int n_slabs,
                              hipStream_t st) {
  hipLaunchKernelGGL(pool_scores_kernel, dim3((n_dst + 63) / 64, n_dst, n_slabs), dim3(64), 0, st, src,
                     n_src, dst, n_dst, g);
  return hipGetLastError();
}

hipError_t launch_finish_rule(const Problem &pb, void *workspace, float *p_imp, uint8_t *mask,
                              const uint8_t *table, hipStream_t st) {
  ProbeArgs a;
  fill_probe_args(pb, nullptr, nullptr, p_imp, workspace, table, &a);
  RuleArgs ra;
  ra.scores = nullptr; ra.mask = mask; ra.Nb = pb.Nb; ra.m_min = pb.m_min; ra.m_max = pb.m_max;
  ra.n_prefix_blocks = pb.n_prefix_blocks; ra.tau = pb.tau;
  ra.n_rows = pb.n_slabs * pb.Nb;
  const dim3 grid((ra.n_rows + 3) / 4), block(256);
  if (pb.Nb <= 64) hipLaunchKernelGGL(finish_rule_kernel<64>, grid, block, 0, st, a, ra);
  else if (pb.Nb <= 128) hipLaunchKernelGGL(finish_rule_kernel<128>, grid, block, 0, st, a, ra);
  else if (pb.Nb <= 256) hipLaunchKernelGGL(finish_rule_kernel<256>, grid, block, 0, st, a, ra);
  else if (pb.Nb <= 512) hipLaunchKernelGGL(finish_rule_kernel<512>, grid, block, 0, st, a, ra);
  else hipLaunchKernelGGL(finish_rule_kernel<1024>, grid, block, 0, st, a, ra);
  return hipGetLastError();
}

hipError_t launch_rule(const Problem &pb, const float *scores, uint8_t *mask, hipStream_t st) {
  RuleArgs a;
  a.scores = scores; a.mask = mask; a.Nb = pb.Nb; a.m_min = pb.m_min; a.m_max = pb.m_max;
  a.n_prefix_blocks = pb.n_prefix_blocks; a.tau = pb.tau;
  a.n_rows = pb.n_slabs * pb.Nb;
  const dim3 grid((a.n_rows + 3) / 4), block(256);
  // network size: power of two >= Nb
  if (pb.Nb <= 64) hipLaunchKernelGGL(rule_kernel<64>, grid, block, 0, st, a);
  else if (pb.Nb <= 128) hipLaunchKernelGGL(rule_kernel<128>, grid, block, 0, st, a);
  else if (pb.Nb <= 256) hipLaunchKernelGGL(rule_kernel<256>, grid, block, 0, st, a);
  else if (pb.Nb <= 512) hipLaunchKernelGGL(rule_kernel<512>, grid, block, 0, st, a);
  else hipLaunchKernelGGL(rule_kernel<1024>, grid, block, 0, st, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Index lists of a mask, by rows (CSR) and by columns (CSC), in three small fully parallel
// kernels: count (one workgroup per row i and column i), in-place scan of the counts, fill.
// ---------------------------------------------------------------------------------------
// blockIdx = (i, slab).  Wavefront 0 counts row i (coalesced), wavefront 1 counts column i.
__global__ __launch_bounds__(128) void csr_count_kernel(const uint8_t *mask, int Nb,
                                                        int32_t *row_ptr, int32_t *col_ptr) {
  const int i = blockIdx.x, slab = blockIdx.y;
  const uint8_t *m = mask + (int64_t)slab * Nb * Nb;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int32_t *ptr = wave == 0 ? row_ptr : col_ptr;
  if (ptr == nullptr) return;
  int n = 0;
  for (int x0 = 0; x0 < Nb; x0 += 64) {
    const int x = x0 + lane;
    const bool f = x < Nb && (wave == 0 ? m[(int64_t)i * Nb + x] : m[(int64_t)x * Nb + i]) != 0;
    n += __popcll(__ballot(f));
  }
  if (lane == 0) {
    ptr[(int64_t)slab * (Nb + 1) + i + 1] = n;
    if (i == 0) ptr[(int64_t)slab * (Nb + 1)] = 0;
  }
}

// blockIdx = (slab, 0: rows / 1: columns).  Inclusive scan of ptr[1..Nb] in place.
__global__ __launch_bounds__(256) void csr_scan_kernel(int Nb, int32_t *row_ptr, int32_t *col_ptr) {
  __shared__ int part[256];
  int32_t *ptr = blockIdx.y == 0 ? row_ptr : col_ptr;
  if (ptr == nullptr) return;
  ptr += (int64_t)blockIdx.x * (Nb + 1) + 1;
  const int tid = threadIdx.x;
  const int per = (Nb + 255) / 256;
  const int lo = tid * per;
  int sum = 0;
  for (int x = lo; x < lo + per && x < Nb; ++x) sum += ptr[x];
  part[tid] = sum;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    int v = tid >= off ? part[tid - off] : 0;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  int run = part[tid] - sum;   // exclusive prefix of my segment
  for (int x = lo; x < lo + per && x < Nb; ++x) {
    run += ptr[x];
    ptr[x] = run;
  }
}

// blockIdx = (i, slab).  Wavefront 0 writes the kept columns of row i, wavefront 1 the kept
// rows of column i, both ascending (ballot compaction, 64 entries per step).
__global__ __launch_bounds__(128) void csr_fill_kernel(const uint8_t *mask, int Nb,
                                                       const int32_t *row_ptr, int32_t *col_idx,
                                                       const int32_t *col_ptr, int32_t *row_idx) {
  const int i = blockIdx.x, slab = blockIdx.y;
  const uint8_t *m = mask + (int64_t)slab * Nb * Nb;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int32_t *ptr = wave == 0 ? row_ptr : col_ptr;
  int32_t *idx = wave == 0 ? col_idx : row_idx;
  if (ptr == nullptr) return;
  int o = ptr[(int64_t)slab * (Nb + 1) + i];
  idx += (int64_t)slab * Nb * Nb;
  for (int x0 = 0; x0 < Nb; x0 += 64) {
    const int x = x0 + lane;
    const bool f = x < Nb && (wave == 0 ? m[(int64_t)i * Nb + x] : m[(int64_t)x * Nb + i]) != 0;
    const unsigned long long b = __ballot(f);
    if (f) idx[o + __popcll(b & ((1ull << lane) - 1ull))] = x;
    o += __popcll(b);
  }
}

// The same in ONE kernel where a slab's mask fits in LDS: several workgroups per slab and direction.
// Each copies the whole mask into LDS, turns it into bits (pieces of 16 rows x 64 columns:
// lane r keeps the ballot of row r, or lane c gathers column c by shifts), counts with
// popcounts, scans the counts and fills its share of the lists, a wavefront per row or column,
// ascending, with coalesced stores.  Reading the mask again in every part costs less than a second
// launch and a trip through memory.  Bound: the latency of the copy and of the four steps behind it.
// Nb = 256, 12 slabs: 15 -> 13 us; Nb = 278, 48 slabs: 65 -> 24 us, against one thread per row or column that
// counts byte by byte out of LDS.  (Bytes straight from global memory instead of the copy: 22 and
// 48 us, bound by the address unit.)
// Up to 352 blocks (mask, bits and counts: 142 of 160 KB of LDS).  From 320 blocks on, with few slabs, the
// three launches above are faster than one copy of the whole mask per workgroup: 352 blocks, 1 .. 8 slabs, both
// directions 16.4 us against 20.3 .. 21.5, 12 slabs 20.9 and 22.0, 24 slabs 33 and 24; rows only, up to
// 32 slabs 16 .. 19 against 20 .. 23; 320 blocks, 8 slabs 16.5 and 17.3, rows only 16.0 and 16.2
constexpr int kCsrBitsMaxNb = 352;
// (48 slabs 21.2 and 18.7).
constexpr int kCsrThreeNb = 320, kCsrThreeSlabs = 12, kCsrThreeSlabsRows = 32;
constexpr int kCsrWords = (kCsrBitsMaxNb + 63) / 64;
__global__ __launch_bounds__(1024) void csr_bits_kernel(const uint8_t *mask, int Nb, int32_t *row_ptr,
                                                        int32_t *col_idx, int32_t *col_ptr,
                                                        int32_t *row_idx) {
  extern __shared__ __align__(16) unsigned char csr_smem[];        // the slab's mask, rows of Nb bytes
  __shared__ unsigned long long bits[kCsrBitsMaxNb * kCsrWords];   // [row or column][word]
  __shared__ int start[kCsrBitsMaxNb + 1];                         // counts, then exclusive offsets
  const int part = blockIdx.x, dir = blockIdx.y, slab = blockIdx.z, n_parts = gridDim.x;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int W = (Nb + 63) / 64;
  for (int x = tid; x < Nb; x += 1024) bits[x * W + W - 1] = 0;   // (its last quarters may have no rows)
  const uint8_t *m = mask + (int64_t)slab * Nb * Nb;
  if ((reinterpret_cast<uintptr_t>(m) & 3) == 0) {                 // four entries at a time
    const uint32_t *m4 = reinterpret_cast<const uint32_t *>(m);
    uint32_t *l4 = reinterpret_cast<uint32_t *>(csr_smem);
    const int n4 = Nb * Nb / 4;
#pragma unroll 8
    for (int t = tid; t < n4; t += 1024) l4[t] = m4[t];
    for (int t = 4 * n4 + tid; t < Nb * Nb; t += 1024) csr_smem[t] = m[t];
  } else {
#pragma unroll 8
    for (int t = tid; t < Nb * Nb; t += 1024) csr_smem[t] = m[t];
  }
  __syncthreads();
  // pieces of 16 rows x 64 columns
  for (int piece = wave; piece < W * ((Nb + 15) / 16); piece += 16) {
    const int r0 = (piece / W) * 16, c0 = (piece % W) * 64;
    const int n_rows = min(16, Nb - r0);
    const bool c_ok = c0 + lane < Nb;
    const unsigned char *src = csr_smem + r0 * Nb + c0 + (c_ok ? lane : 0);
    uint8_t b[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) b[x] = src[min(x, n_rows - 1) * Nb];
    if (dir == 0) {                              // lane x < 16: row r0 + x, columns c0 ..
      unsigned long long word = 0;
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const unsigned long long row = __ballot(c_ok && b[x] != 0);
        if (lane == x) word = row;
      }
      if (lane < n_rows) bits[(r0 + lane) * W + c0 / 64] = word;
    } else {                                     // lane: column c0 + lane, a quarter of its word of rows
      uint32_t quarter = 0;
#pragma unroll
      for (int x = 0; x < 16; ++x) quarter |= (uint32_t)(x < n_rows && b[x] != 0) << x;
      if (c_ok) reinterpret_cast<uint16_t *>(bits)[(c0 + lane) * W * 4 + r0 / 16] = (uint16_t)quarter;
    }
  }
  __syncthreads();
  for (int x = tid; x < Nb; x += 1024) {
    int n = 0;
    for (int w = 0; w < W; ++w) n += __popcll(bits[x * W + w]);
    start[x] = n;
  }
  __syncthreads();
  int32_t *ptr = (dir == 0 ? row_ptr : col_ptr) + (int64_t)slab * (Nb + 1);
  if (wave == 0) {                                 // exclusive scan of the counts
    int run = 0;
    for (int x0 = 0; x0 < Nb; x0 += 64) {
      const int x = x0 + lane;
      const int v = x < Nb ? start[x] : 0;
      int inc = v;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(inc, off, 64);
        if (lane >= off) inc += o;
      }
      if (x < Nb) {
        start[x] = run + inc - v;
        if (part == 0) ptr[x] = run + inc - v;
      }
      run += __shfl(inc, 63, 64);
    }
    if (part == 0 && lane == 0) ptr[Nb] = run;
  }
  __syncthreads();
  int32_t *idx = (dir == 0 ? col_idx : row_idx) + (int64_t)slab * Nb * Nb;
  for (int i = part * 16 + wave; i < Nb; i += 16 * n_parts) {
    int o = start[i];
    for (int w = 0; w < W; ++w) {
      const unsigned long long b = bits[i * W + w];
      if ((b >> lane) & 1) idx[o + __popcll(b & ((1ull << lane) - 1ull))] = 64 * w + lane;
      o += __popcll(b);
    }
  }
}

hipError_t launch_csr(const Problem &pb, const uint8_t *mask, int32_t *row_ptr, int32_t *col_idx,
                      int32_t *col_ptr, int32_t *row_idx, hipStream_t st) {
  const int few = col_ptr ? kCsrThreeSlabs : kCsrThreeSlabsRows;
  if (pb.Nb < kCsrThreeNb || (pb.Nb <= kCsrBitsMaxNb && pb.n_slabs > few)) {
    // as many parts as keep one workgroup per compute unit, at most one per 16 rows
    const int n_dir = col_ptr ? 2 : 1;
    const int most = (pb.Nb + 15) / 16;
    int parts = 256 / (n_dir * pb.n_slabs);
    parts = parts < 1 ? 1 : (parts > most ? most : parts);
    hipError_t e0 = set_dynamic_lds_once(reinterpret_cast<const void *>(&csr_bits_kernel),
                                         kCsrBitsMaxNb * kCsrBitsMaxNb);
    if (e0 != hipSuccess) return e0;
    hipLaunchKernelGGL(csr_bits_kernel, dim3(parts, n_dir, pb.n_slabs), dim3(1024), pb.Nb * pb.Nb, st, mask,
                       pb.Nb, row_ptr, col_idx, col_ptr, row_idx);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(csr_count_kernel, dim3(pb.Nb, pb.n_slabs), dim3(128), 0, st, mask, pb.Nb,
                     row_ptr, col_ptr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(csr_scan_kernel, dim3(pb.n_slabs, 2), dim3(256), 0, st, pb.Nb, row_ptr,
                     col_ptr);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(csr_fill_kernel, dim3(pb.Nb, pb.n_slabs), dim3(128), 0, st, mask, pb.Nb,
                     row_ptr, col_idx, col_ptr, row_idx);
  return hipGetLastError();
}

}  // namespace asa
