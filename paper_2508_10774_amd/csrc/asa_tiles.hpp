// MFMA operand orderings, LDS swizzles and direct global->LDS tile copies shared by the
// forward and backward attention kernels (device code only).
#pragma once

#include "asa_common.hpp"

namespace asa {

// Row r of an MFMA A operand / accumulator splits as r = 8g + 4h + j (g<4, h<2, j<4); lane
// half h holds accumulator register 4g + j.
//
// kappa: which key of a 32-key group is loaded as A row r of S^T = K Q^T.  Chosen so that
// lane half h, registers 8t..8t+7 hold keys 16t + 8h + 0..7: exactly the 8 consecutive k
// slots that the B operand of the following 16-deep P^T step wants from that lane.
__device__ __forceinline__ int kappa(int r) {
  int g = r >> 3, h = (r >> 2) & 1, j = r & 3;
  return 16 * (g >> 1) + 8 * h + 4 * (g & 1) + j;
}
// rho: which channel of a 32-channel group is loaded as A row r of O^T = V^T P^T, chosen so
// that lane half h ends up with 16 consecutive channels 16h + (4g + j) of its query.
__device__ __forceinline__ int rho(int r) {
  int g = r >> 3, h = (r >> 2) & 1, j = r & 3;
  return 16 * h + 4 * g + j;
}

// LDS tiles are filled by direct global->LDS loads, which write 64 lanes x 16 B contiguously:
// rows cannot be padded, so 16-byte chunks are XOR-swizzled instead.  A K row holds D/8 chunks
// and is read by 16 lanes with 16 different rows (kappa) and one chunk index: chunk c of row r
// lives at position c ^ (r mod chunks).  A V^T row holds 8 chunks (128 B, half the banks) and is
// read through rho, whose 16 rows differ in row bits 0..2 and 4: position c ^ f(r) with f built
// from bits 1, 2, 4 separates the 8 rows of equal parity, parity itself picks the bank half.
template <int D>
__device__ __forceinline__ int k_swz(int row) {
  // D = 128: a row is all 64 banks, 16 rows need 16 positions; D = 64: a row is half the banks,
  // parity picks the half and the 8 rows of equal parity need 8 positions
  return D == 128 ? (row & 15) : ((row >> 1) & 7);
}
__device__ __forceinline__ int v_swz(int row) { return ((row >> 1) & 3) | (((row >> 4) & 1) << 2); }

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

// Swizzle of a row tile that is read both row-wise (16 lanes, 16 rows, one 16-byte chunk) and
// through the transposing LDS read (16 lanes: 4 consecutive rows x four 8-byte pieces).  With
// D = 128 the row's low two bits go to the chunk's high two bits, so that the 4 consecutive rows
// of a transposing read fall into 4 different quarters of the banks; any bijection of row mod 16
// serves the row-wise reads.  With D = 64 the k_swz pattern already serves both.
template <int D>
__device__ __forceinline__ int t_swz(int row) {
  return D == 128 ? (((row & 3) << 2) | ((row >> 2) & 3)) : ((row >> 1) & 7);
}
// byte offset, in a t_swz row tile, of the 8-byte piece "row r, columns d4 .. d4 + 3" (d4 % 4 == 0)
template <int D>
__device__ __forceinline__ uint32_t tr_piece(int r, int d4) {
  return (uint32_t)((r * D + (((d4 >> 3) ^ t_swz<D>(r)) << 3) + (d4 & 4)) * 2);
}
// read of a T at an absolute LDS byte address
template <typename T>
__device__ __forceinline__ T lds_read(uint32_t addr) {
  return *reinterpret_cast<const __attribute__((address_space(3))) T *>((uintptr_t)addr);
}
// ds_read_b64_tr_b16: inside each group of 16 lanes, lane i receives as element j (j = 0..3) the
// 16-bit element i % 4 of the 8 bytes that lane 4 j + i / 4 of the group addressed.
__device__ __forceinline__ bf16x4 lds_read_tr16(const lds_char *p) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)p);
#else
  return bf16x4{};
#endif
}

// One direct global->LDS load: every lane fetches 16 bytes and the wavefront's 64 x 16 B land contiguously
// at the (wave-uniform) LDS address; counted by vmcnt.  The address is split into a wave-uniform 64-bit
// base (scalar registers) and a 32-bit per-lane byte offset: stepping to another tile then costs scalar adds only and the
// per-lane offsets stay 32 bits wide.  The compiler does not see this load: the caller waits
// with an explicit vmcnt before reading the LDS image, and a kernel that uses this form uses
// it for all of its direct loads (M0 is written here).
// lds_byte_addr is the wave-uniform LDS address (lds_addr_of() of the LDS array + offset).
// The load takes its base from a scalar copy made in front of it: a vector memory instruction must not
// read a scalar register within 5 wait states of the vector instruction (v_readfirstlane, v_readlane of a
// spilled register) that wrote it; the hardware does not check, the compiler does not look in here, and a
// scalar move may read it at once.  The copy also is the wait state between M0 and the load.
// FORCE = false leaves the operands as the compiler has them (it must then know them to be
// uniform, or the assembler rejects the instruction).
template <bool FORCE = true>
__device__ __forceinline__ void lds_dma16_sv(const void *uniform_base, uint32_t lane_off,
                                             uint32_t lds_byte_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  uint64_t base_copy;
  if (!FORCE) {
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
                 : "=&s"(base_copy) : "v"(lane_off), "s"(uniform_base), "s"(lds_byte_addr) : "memory");
    return;
  }
  // (readfirstlane costs nothing where the compiler already knows the value to be uniform and
  // puts it into scalar registers where it does not)
  const uint64_t b = reinterpret_cast<uint64_t>(uniform_base);
  // (the builtin returns a signed int: widen through uint32_t, or the low half sign-extends
  // into the high one)
  const uint64_t bu = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b) |
                      ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32);
  asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
               : "=&s"(base_copy)
               : "v"(lane_off), "s"(bu), "s"((uint32_t)__builtin_amdgcn_readfirstlane(lds_byte_addr)) : "memory");
#endif
}
// The same from a 64-bit address per lane.
__device__ __forceinline__ void lds_dma16_v(const void *lane_addr, uint32_t lds_byte_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               : : "v"(lane_addr), "s"((uint32_t)__builtin_amdgcn_readfirstlane(lds_byte_addr)) : "memory");
#endif
}
// The same for several loads in a row that share M0 and the base: lds_dma_begin sets M0 and returns the scalar copy of the
// base, lds_dma16_next<X> loads with X bytes added to the global AND to the LDS address (X < 4096).  Nothing else may write
// M0 in between (tests/test_asm_hazards.py looks).
__device__ __forceinline__ uint64_t lds_dma_begin(const void *uniform_base, uint32_t lds_byte_addr) {
  uint64_t base_copy = 0;
#if defined(__HIP_DEVICE_COMPILE__)
  const uint64_t b = reinterpret_cast<uint64_t>(uniform_base);
  const uint64_t bu = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b) |
                      ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32);
  asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 %0, %1"
               : "=&s"(base_copy)
               : "s"(bu), "s"((uint32_t)__builtin_amdgcn_readfirstlane(lds_byte_addr)) : "memory");
#endif
  return base_copy;
}
template <int X>
__device__ __forceinline__ void lds_dma16_next(uint64_t base_copy, uint32_t lane_off) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(lane_off), "s"(base_copy), "n"(X) : "memory");
#endif
}
// The same with 4 bytes per lane.
__device__ __forceinline__ void lds_dma4_sv(const void *uniform_base, uint32_t lane_off, uint32_t lds_byte_addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  uint64_t base_copy;
  const uint64_t b = reinterpret_cast<uint64_t>(uniform_base);
  const uint64_t bu = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b) |
                      ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32);
  asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dword %1, %0"
               : "=&s"(base_copy)
               : "v"(lane_off), "s"(bu), "s"((uint32_t)__builtin_amdgcn_readfirstlane(lds_byte_addr)) : "memory");
#endif
}
// LDS byte address of an object that the compiler knows to live in LDS (apply it to the
// __shared__ array itself, not to a pointer that travelled through generic address space)
#define ASA_LDS_ADDR_OF(shared_array) ((uint32_t)(uintptr_t)(::asa::lds_void *)(shared_array))

// The compiler places no wait states around a written-out MFMA (tests/test_asm_hazards.py walks the
// assembly).  settle_acc in front of a loop and behind it keeps what the compiler does with the
// accumulators (zeros, copies, reads) away from the loop's MFMAs: 2 states after a vector instruction has
// written an operand, 19 before one reads a result.
template <int N>
__device__ __forceinline__ void settle_acc(f32x16 (&acc)[N]) {
  static_assert(N == 2 || N == 4, "D = 64, 128");
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (N == 2) asm volatile("s_nop 15\n\ts_nop 3" : "+a"(acc[0]), "+a"(acc[1]));
  else asm volatile("s_nop 15\n\ts_nop 3" : "+a"(acc[0]), "+a"(acc[1]), "+a"(acc[2]), "+a"(acc[3]));
#endif
}

// ---------------------------------------------------------------------------------------
// Cooperative tile copies global -> LDS for a workgroup of WAVES wavefronts.  Per-lane byte
// offsets are computed once (init); every copy then costs only a wave-uniform base pointer.
// ---------------------------------------------------------------------------------------

// ROWS x D bf16 tile of a row-major [L][*] tensor (row pitch sL elements), rows past L - 1
// re-read row L - 1 (they are masked by the caller).  LDS image: unpadded rows, k_swz swizzle.
template <int ROWS, int D, int WAVES>
struct RowTileCopy {
  static constexpr int kChunks = D / 8;                       // 16-byte chunks per row
  static constexpr int kInstr = ROWS * kChunks / 64 / WAVES;  // wave instructions per copy
  uint32_t off[kInstr];
  int wave, lane;
  int64_t pitch_bytes;

  __device__ __forceinline__ void init(int wave_, int lane_, int64_t sL) {
    wave = wave_; lane = lane_; pitch_bytes = sL * 2;
#pragma unroll
    for (int i = 0; i < kInstr; ++i) {
      const int row = (wave * kInstr + i) * (64 / kChunks) + lane / kChunks;
      const int pos = lane % kChunks;
      off[i] = (uint32_t)(row * pitch_bytes + ((pos ^ k_swz<D>(row)) * 16));
    }
  }
  // row of the tile that instruction i of this lane copies; byte offset of its 1 KB LDS chunk
  __device__ __forceinline__ int row_of(int i) const {
    return (wave * kInstr + i) * (64 / kChunks) + lane / kChunks;
  }
  __device__ __forceinline__ uint32_t lds_chunk(int i) const { return (wave * kInstr + i) * 1024; }
  // copy the ROWS complete rows that start at byte address `base` to the LDS byte address `stage`
  __device__ __forceinline__ void issue_at(uint32_t stage, const char *base) const {
#pragma unroll
    for (int i = 0; i < kInstr; ++i) lds_dma16_sv(base, off[i], stage + (wave * kInstr + i) * 1024);
  }
  // the same for a tile whose rows past `lim` (relative to the tile) re-read row `lim`.
  // lim < 0 (the whole tile lies past the last row) moves the base back to that row first:
  // the per-lane offsets are unsigned and must not go negative.
  __device__ __forceinline__ void issue_at_ragged(uint32_t stage, const char *base, int lim) const {
    if (lim < 0) {
      base += (int64_t)lim * pitch_bytes;
      lim = 0;
    }
#pragma unroll
    for (int i = 0; i < kInstr; ++i) {
      const int row = (wave * kInstr + i) * (64 / kChunks) + lane / kChunks;
      const uint32_t o = row > lim ? off[i] - (uint32_t)(row - lim) * (uint32_t)pitch_bytes : off[i];
      lds_dma16_sv(base, o, stage + (wave * kInstr + i) * 1024);
    }
  }
};

// D x 64 slice (columns [col0, col0 + 64)) of a transposed tile stored as [D][BLK] bf16.
// LDS image: [D][64], v_swz swizzle.
template <int BLK, int D, int WAVES>
struct ColTileCopy {
  static constexpr int kInstr = D * 8 / 64 / WAVES;
  uint32_t off[kInstr];
  int wave;

  __device__ __forceinline__ void init(int wave_, int lane) {
    wave = wave_;
#pragma unroll
    for (int i = 0; i < kInstr; ++i) {
      const int row = (wave * kInstr + i) * 8 + lane / 8;
      off[i] = (uint32_t)((row * BLK + (((lane % 8) ^ v_swz(row)) * 8)) * 2);
    }
  }
  __device__ __forceinline__ void issue_at(uint32_t stage, const char *base) const {
#pragma unroll
    for (int i = 0; i < kInstr; ++i) lds_dma16_sv(base, off[i], stage + (wave * kInstr + i) * 1024);
  }
  template <bool FORCE = true>
  __device__ __forceinline__ void issue_one_at(int i, uint32_t stage, const char *base) const {
    lds_dma16_sv<FORCE>(base, off[i], stage + (wave * kInstr + i) * 1024);
  }
};

// ROWS x D row tile with the t_swz swizzle, copied by WAVES wavefronts one instruction at a time, so
// that a kernel can place the copies between other work.  Tiles start at multiples of ROWS; the one
// that holds the last row L - 1 re-reads that row where it reaches past it (a second set of
// per-lane offsets, chosen without a branch).  A tile wholly past L - 1 is replaced by
// the one that holds it: the caller masks such rows anyway.
template <int ROWS, int D, int WAVES>
struct TrTileCopy {
  static constexpr int kChunks = D / 8;                       // 16-byte chunks per row
  static constexpr int kInstr = ROWS * kChunks / 64 / WAVES;  // wave instructions per copy
  static_assert(kInstr * 64 * WAVES == ROWS * kChunks, "whole instructions per wavefront");
  uint32_t off[kInstr], off_last[kInstr];
  uint32_t lds0;                                              // LDS distance of my first instruction

  static __device__ __forceinline__ int last_row0(int L) { return (L - 1) / ROWS * ROWS; }
  __device__ __forceinline__ void init(int wave, int lane, int64_t sL, int L) {
    const uint32_t pitch = (uint32_t)(sL * 2);
    lds0 = (uint32_t)(wave * kInstr * 1024);
#pragma unroll
    for (int i = 0; i < kInstr; ++i) {
      const int row = (wave * kInstr + i) * (64 / kChunks) + lane / kChunks;
      const int row_c = min(row, L - 1 - last_row0(L));
      const uint32_t chunk = (uint32_t)(((lane % kChunks) ^ t_swz<D>(row)) * 16);
      off[i] = (uint32_t)row * pitch + chunk;
      off_last[i] = (uint32_t)row_c * pitch + chunk;
    }
  }
  // last (wave-uniform): this is the tile that holds row L - 1
  __device__ __forceinline__ void issue_one(int i, uint32_t stage, const char *base, bool last) const {
    lds_dma16_sv(base, last ? off_last[i] : off[i], stage + lds0 + i * 1024);
  }
};

// The same for a walk that goes tile by tile through blocks, with as few instructions per tile as it takes (a wavefront
// issues one per ~5 cycles, scalar ones too): the base runs along by one addition, a wavefront's kInstr loads of a tile
// have M0 and the base in common (start / load<i>), and the tile that holds row L - 1 changes the per-lane offsets where it
// is entered and left, in a branch that is otherwise not taken (watch), instead of choosing between two sets each time.
// Load i adds 1024 i to the LDS and to the global address alike: the per-lane offsets are less by that.  (Not below zero: a load's
// rows are 1024 / (2 D) apart from the next one's, at 2 D bytes or more each.  In the tile that holds the last row they
// come closer: there the base is less by 1024 (kInstr - 1) instead.)
template <int ROWS, int D, int WAVES>
struct RunningTileCopy {
  static constexpr int kChunks = D / 8;                       // 16-byte chunks per row
  static constexpr int kInstr = ROWS * kChunks / 64 / WAVES;  // wave instructions per copy
  static_assert(kInstr * 64 * WAVES == ROWS * kChunks && kInstr * 1024 <= 4096, "whole instructions per wavefront, 12-bit distances");
  uint32_t off[kInstr], to_last[kInstr];
  uint32_t lds0;                                              // LDS distance of my first instruction
  uint32_t pitch;
  const char *slab, *base;                                    // (wave-uniform)

  static __device__ __forceinline__ int last_row0(int L) { return (L - 1) / ROWS * ROWS; }
  __device__ __forceinline__ void init(int wave, int lane, const void *slab_rows, int64_t sL, int L) {
    slab = base = reinterpret_cast<const char *>(slab_rows);
    pitch = (uint32_t)(sL * 2);
    lds0 = (uint32_t)(wave * kInstr * 1024);
#pragma unroll
    for (int i = 0; i < kInstr; ++i) {
      const int row = (wave * kInstr + i) * (64 / kChunks) + lane / kChunks;
      const int row_c = min(row, L - 1 - last_row0(L));
      off[i] = (uint32_t)row * pitch + (uint32_t)(((lane % kChunks) ^ t_swz<D>(row)) * 16) - 1024u * i;
      to_last[i] = (uint32_t)(row_c - row) * pitch + 1024u * (kInstr - 1);
    }
  }
  __device__ __forceinline__ void block(int row0) { base = slab + (uint64_t)(uint32_t)row0 * pitch; }
  __device__ __forceinline__ void step() { base += (uint32_t)ROWS * pitch; }
  // the tile that holds row L - 1, or one wholly past it, which is replaced by the former
  __device__ __forceinline__ void at_last(int L) { base = slab + (uint64_t)(uint32_t)last_row0(L) * pitch - 1024 * (kInstr - 1); }
  __device__ __forceinline__ void turn(bool into_last) {
#pragma unroll
    for (int i = 0; i < kInstr; ++i) off[i] += into_last ? to_last[i] : 0u - to_last[i];
  }
  __device__ __forceinline__ uint64_t start(uint32_t stage) const { return lds_dma_begin(base, stage + lds0); }
  template <int I>
  __device__ __forceinline__ void load(uint64_t started) const { lds_dma16_next<I * 1024>(started, off[I]); }
};
// Which branch of one or more such walks a tile takes.  watch: a tile whose first row is at or past it has something to do.
struct LastTileWatch {
  int last_row0, watch;
  bool inside;
  __device__ __forceinline__ void init(int last) { last_row0 = watch = last; inside = false; }
  template <typename... C>
  __device__ __forceinline__ void tile(int row0, int L, C &...x) {
    if (__builtin_expect(row0 < watch, 1)) return;
    const bool now = row0 >= last_row0;
    if (now != inside) {
      (x.turn(now), ...);
      inside = now;
      watch = now ? 0 : last_row0;
    }
    if (now) (x.at_last(L), ...);
  }
};

}  // namespace asa
