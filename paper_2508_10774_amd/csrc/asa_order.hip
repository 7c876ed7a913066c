// Order in which the workgroups of the attention kernels take their work items.
//
// The selection rule gives every query block its own number of key blocks (Alg. 3 step 9 of the
// paper), and the columns of the mask differ even more (31..220 query blocks at 25 % density on
// video-like inputs).  A long item that starts late ends the kernel late.  Each XCD keeps its
// contiguous share of the (slab, block) items (its workgroups share an L2) but works through it
// longest list first (lists of one length in their natural order: neighbours share key blocks).  One
// workgroup per XCD share.  A share whose lists all have one length (a fixed budget per row) keeps
// its natural order and skips the sort.
#include "asa_common.hpp"

namespace asa {

constexpr int kOrderMax = 2048;   // items per XCD share that the sort handles
constexpr int kOrderWaves = 16;

// A stable counting sort.  Lengths are 0 .. Nb <= 1024; a wavefront owns 128 consecutive items, finds
// the rank of each among its lanes of equal length with one ballot per bit of the length, and counts
// its items per length in a histogram of its own; one thread per length then turns the histograms
// into start positions.  Five workgroup barriers in all (a bitonic network has 66 steps with one
// each: 1668 uneven items 23 us -> 10 us, 384 items 14 us -> 7 us).  blockIdx.y: which of the two lists (rows or columns).
struct OrderArgs {
  const int32_t *ptr[2];
  int32_t *order[2];
  int Nb, total;
};
__global__ __launch_bounds__(1024) void length_order_kernel(OrderArgs a) {
  __shared__ uint16_t hist[kOrderWaves][kMaxNb + 8];   // [wavefront][length]
  __shared__ int wave_sum[kOrderWaves];
  const int32_t *ptr = a.ptr[blockIdx.y];
  int32_t *order = a.order[blockIdx.y];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int share = (a.total + kNumXcd - 1) / kNumXcd;
  const int first = blockIdx.x * share;
  const int count = max(0, min(share, a.total - first));
  const int n_waves = (count + 127) / 128;       // wavefronts that have items
  uint32_t *h32 = reinterpret_cast<uint32_t *>(&hist[0][0]);
  for (int t = tid; t < n_waves * (kMaxNb + 8) / 2; t += 1024) h32[t] = 0;
  // (two steps of 64 items: items 128 wave .. 128 wave + 127 of the share)
  int len[2], rank[2];
  int uneven = 0, len0 = 0;
  if (count > 0) {
    const int slab = first / a.Nb, b = first - slab * a.Nb;
    len0 = ptr[slab * (a.Nb + 1) + b + 1] - ptr[slab * (a.Nb + 1) + b];
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int t = 128 * wave + 64 * u + lane;
    len[u] = 0;
    if (t < count) {
      const int item = first + t, slab = item / a.Nb, b = item - slab * a.Nb;
      len[u] = ptr[slab * (a.Nb + 1) + b + 1] - ptr[slab * (a.Nb + 1) + b];
      len[u] = min(max(len[u], 0), kMaxNb);
      uneven |= len[u] != len0;
    }
  }
  if (!__syncthreads_or(uneven)) {               // all lists of one length: the natural order
    for (int t = tid; t < count; t += 1024) order[first + t] = first + t;
    return;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const bool ok = 128 * wave + 64 * u + lane < count;
    unsigned long long same = __ballot(ok);
#pragma unroll
    for (int bit = 0; bit < 11; ++bit) {
      const unsigned long long set = __ballot((len[u] >> bit) & 1);
      same &= ((len[u] >> bit) & 1) ? set : ~set;
    }
    if (ok) {
      const int before = hist[wave][len[u]];     // (of the first step: the wavefront runs in step)
      rank[u] = before + __popcll(same & ((1ull << lane) - 1ull));
      __builtin_amdgcn_wave_barrier();
      if ((same >> lane) == 1) hist[wave][len[u]] = (uint16_t)(before + __popcll(same));
    }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // thread t: length kMaxNb - t (longest first), the last thread also length 0
  int mine = 0;
  for (int x = 0; x < (tid == 1023 ? 2 : 1); ++x) {
    const int l = kMaxNb - tid - x;
    for (int w = 0; w < n_waves; ++w) {          // exclusive over the wavefronts, in place
      const int n = hist[w][l];
      hist[w][l] = (uint16_t)mine;
      mine += n;
    }
  }
  int inc = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(inc, off, 64);
    if (lane >= off) inc += o;
  }
  if (lane == 63) wave_sum[wave] = inc;
  __syncthreads();
  int base = inc - mine;
  for (int w = 0; w < wave; ++w) base += wave_sum[w];
  for (int x = 0; x < (tid == 1023 ? 2 : 1); ++x)
    for (int w = 0; w < n_waves; ++w) hist[w][kMaxNb - tid - x] += (uint16_t)base;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int t = 128 * wave + 64 * u + lane;
    if (t < count) order[first + hist[wave][len[u]] + rank[u]] = first + t;
  }
}

// Shares of at most 64 items: one wavefront, every lane compares its item with all others.
__global__ __launch_bounds__(64) void length_order_small_kernel(OrderArgs a) {
  const int32_t *ptr = a.ptr[blockIdx.y];
  int32_t *order = a.order[blockIdx.y];
  const int lane = threadIdx.x;
  const int share = (a.total + kNumXcd - 1) / kNumXcd;
  const int first = blockIdx.x * share;
  const int count = max(0, min(share, a.total - first));
  int len = -1;
  if (lane < count) {
    const int item = first + lane, slab = item / a.Nb, b = item - slab * a.Nb;
    len = ptr[slab * (a.Nb + 1) + b + 1] - ptr[slab * (a.Nb + 1) + b];
  }
  int rank = 0;
  for (int x = 0; x < count; ++x) {
    const int other = __builtin_amdgcn_readlane(len, x);
    rank += (other > len) || (other == len && x < lane);
  }
  if (lane < count) order[first + rank] = first + lane;
}

// Up to one workgroup per compute unit all of them start at once, in whatever order: the launch
// would cost its 3-5 us for nothing.
bool length_order_wanted(int total) { return total > 256 && (total + kNumXcd - 1) / kNumXcd <= kOrderMax; }

hipError_t launch_length_order(const int32_t *ptr, int Nb, int total, int32_t *order, hipStream_t st,
                               const int32_t *ptr2, int32_t *order2) {
  OrderArgs a;
  a.ptr[0] = ptr; a.ptr[1] = ptr2;
  a.order[0] = order; a.order[1] = order2;
  a.Nb = Nb; a.total = total;
  const dim3 grid(kNumXcd, ptr2 ? 2 : 1);
  if ((total + kNumXcd - 1) / kNumXcd <= 64)
    hipLaunchKernelGGL(length_order_small_kernel, grid, dim3(64), 0, st, a);
  else
    hipLaunchKernelGGL(length_order_kernel, grid, dim3(1024), 0, st, a);
  return hipGetLastError();
}

}  // namespace asa
