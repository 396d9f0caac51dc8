// Single-pass prefix sums over blocks (decoupled look-back), as a device
// function for kernels that scan values they compute themselves: a parallel
// filter of Alg. 1 (Sec. 2.2) is then one launch that tests its elements, ranks
// them and places them.
#pragma once

#include "pc_common.hpp"

namespace pc {

constexpr int kScanItems = 4;
constexpr int kScanTile = kBlock * kScanItems;  // 1024

template <class T>
__device__ T block_exclusive_scan(T v, T &total) {
  constexpr int kNW = kBlock / kWave;  // waves per block
  __shared__ T sw[kNW + 1];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  T x = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    T y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  if (lane == kWave - 1) sw[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    T acc = 0;
    for (int w = 0; w < kNW; ++w) {
      T t = sw[w];
      sw[w] = acc;
      acc += t;
    }
    sw[kNW] = acc;
  }
  __syncthreads();
  T r = x - v + sw[wid];
  total = sw[kNW];
  __syncthreads();
  return r;
}

// A block takes the next ticket (so every block it waits for has started) and
// clears its share of the next scan's status array on the way.
__device__ __forceinline__ int scan_ticket(int *ticket, unsigned long long *st_next, int *ticket_next, int cap) {
  __shared__ int sbid;
  if (threadIdx.x == 0) sbid = atomicAdd(ticket, 1);
  __syncthreads();
  const int bid = sbid;
  for (int j = bid * kBlock + threadIdx.x; j < cap; j += gridDim.x * kBlock) st_next[j] = 0ull;
  if (bid == 0 && threadIdx.x == 0) *ticket_next = 0;
  return bid;
}

// Sum of the totals of the blocks before `bid`; called by every thread of the
// block with the block's own total. The block publishes its total (flag 1),
// one wavefront adds the totals of the blocks before it, 64 at a time, until
// it meets a published prefix (flag 2), and publishes the block's own prefix.
// A look-back that waits beyond kSpinLimit windows gives up with the part it
// has (every output position then stays at or below its true value) and
// raises the error flag. Totals are below 2^62.
constexpr unsigned long long kStValue = (1ull << 62) - 1;
constexpr int kSpinLimit = 1 << 22;

template <class T>
__device__ __forceinline__ T scan_look_back(unsigned long long *st, int bid, T tot, int *err) {
  __shared__ T sprefix;
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    T prefix = 0;
    if (bid == 0) {
      if (lane == 0)
        __hip_atomic_store(&st[0], (2ull << 62) | (unsigned long long)tot, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    } else {
      if (lane == 0)
        __hip_atomic_store(&st[bid], (1ull << 62) | (unsigned long long)tot, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      int top = bid - 1;  // the nearest block not yet added
      int spins = 0;
      while (true) {
        const int idx = top - lane;
        const unsigned long long w =
            idx >= 0 ? __hip_atomic_load(&st[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (2ull << 62);
        const unsigned long long pm = __ballot((w >> 62) == 2ull);
        const int fp = pm ? __ffsll((long long)pm) - 1 : kWave;  // nearest published prefix
        const unsigned long long need = fp >= kWave - 1 ? ~0ull : ((2ull << fp) - 1ull);
        if (__ballot((w >> 62) == 0ull) & need) {
          // a block in the window has not published yet
          if (++spins > kSpinLimit) {
            if (lane == 0) atomicExch(err, 1);
            break;
          }
          continue;
        }
        T add = lane <= fp ? (T)(w & kStValue) : (T)0;
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) add += __shfl_xor(add, o, kWave);
        prefix += add;
        if (fp < kWave) break;
        top -= kWave;
      }
      if (lane == 0)
        __hip_atomic_store(&st[bid], (2ull << 62) | (unsigned long long)(prefix + tot), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) sprefix = prefix;
  }
  __syncthreads();
  return sprefix;
}

// A filter F: len() elements, value(i) of each (0: not taken; their sum below
// 2^62), emit(i, prefix, value) for every element, total(sum) once at the end.
// total() may change what len() reads: it runs in the block of the last
// elements, after every block that has elements has read it, and a block that
// reads a smaller length later has none.
template <class F>
__global__ __launch_bounds__(kBlock) void k_filter_lb(F f, unsigned long long *st, int *ticket,
                                                      unsigned long long *st_next, int *ticket_next, int cap,
                                                      int *err) {
  const int bid = scan_ticket(ticket, st_next, ticket_next, cap);
  const int len = f.len();
  // blocks past the device length have nothing to do (the grid is sized for
  // the host's bound); the last live block writes the total
  const int live = len > 0 ? (len + kScanTile - 1) / kScanTile : 1;
  if (bid >= live) return;  // uniform per block
  const long long base = (long long)bid * kScanTile + threadIdx.x * kScanItems;
  unsigned long long v[kScanItems], s = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    const long long i = base + j;
    v[j] = i < len ? f.value((int)i) : 0ull;
    s += v[j];
  }
  unsigned long long tot;
  const unsigned long long ex = block_exclusive_scan<unsigned long long>(s, tot);
  const unsigned long long prefix = scan_look_back<unsigned long long>(st, bid, tot, err);
  unsigned long long run = ex + prefix;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    const long long i = base + j;
    if (i < len) f.emit((int)i, run, v[j]);
    run += v[j];
  }
  if (bid == live - 1 && threadIdx.x == 0) f.total(prefix + tot);
}

// short filters: one block walks the tiles in order
template <class F>
__global__ __launch_bounds__(kBlock) void k_filter_one(F f) {
  const int len = f.len();
  unsigned long long carry = 0;
  for (int b0 = 0; b0 < len; b0 += kScanTile) {
    unsigned long long v[kScanItems], s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
      const int i = b0 + threadIdx.x * kScanItems + j;
      v[j] = i < len ? f.value(i) : 0ull;
      s += v[j];
    }
    unsigned long long tot;
    unsigned long long run = carry + block_exclusive_scan<unsigned long long>(s, tot);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
      const int i = b0 + threadIdx.x * kScanItems + j;
      if (i < len) f.emit(i, run, v[j]);
      run += v[j];
    }
    carry += tot;
  }
  __syncthreads();
  if (threadIdx.x == 0) f.total(carry);
}

// clears both status arrays and the tickets of new memory
void scan_ws_prepare(ScanWs &ws, hipStream_t s);

constexpr int kSingleScan = 4 * kScanTile;

// `nmax`: the host's bound of len()
template <class F>
void launch_filter(const F &f, int nmax, ScanWs &ws, hipStream_t s) {
  const int nb = (nmax + kScanTile - 1) / kScanTile;
  if (nmax <= kSingleScan || nb > ws.cap) {
    // (the workspace is sized for the longest scan; one block is slow but safe)
    k_filter_one<F><<<1, kBlock, 0, s>>>(f);
    return;
  }
  scan_ws_prepare(ws, s);
  const int a = ws.turn;
  ws.turn ^= 1;
  k_filter_lb<F><<<nb, kBlock, 0, s>>>(f, ws.st[a], ws.ticket + a, ws.st[a ^ 1], ws.ticket + (a ^ 1), ws.cap, ws.err);
}

}  // namespace pc
