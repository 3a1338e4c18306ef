// The state's entries in ascending label order (hi, lo), for sorted export:
// tiles sorted in LDS, then merged pairwise.  Labels are distinct, so the
// order is total and no pass has ties to keep.
//
// What is sorted are 32-bit entry indices; labels are read through them (from
// L2 for the sizes at which latency counts) and never moved, so the passes
// need two index arrays and nothing else, and the state stays in place.  The
// last pass writes labels and amplitudes in order.  Each merge pass reads and
// writes an index and reads a label per entry; up to 2^18 entries a pass is
// its chain of round trips (search, indices, labels, ranks: 15 us), not its
// bytes.  100003 entries of 80-qubit labels: tiles 46 us, five merges 91; the
// sorted export as a whole 0.33 ms, where sorting the copied arrays on the host
// took 11.4, and at 2^20 entries 1.4 against 151.
#include <hip/hip_runtime.h>

#include "sim_internal.h"

namespace sparsesim {
namespace {

constexpr uint32_t kThreads = 1024, kItems = 4, kTile = kThreads * kItems;

template <bool WIDE>
struct Keys {
  uint64_t lo[kTile];
  uint64_t hi[WIDE ? kTile : 1];
};

template <bool WIDE>
__device__ __forceinline__ bool less(uint64_t alo, uint64_t ahi, uint64_t blo, uint64_t bhi) {
  return WIDE ? (ahi != bhi ? ahi < bhi : alo < blo) : alo < blo;
}

// How many of the keys [b, b + m[j]) of k are below (lo[j], hi[j]), for a
// thread's entries together: `steps` halvings (2^steps > every m), no branch
// but the one around the low words, which are read only where the high ones
// are equal (the searches are bound by LDS reads and their latency).  n: keys
// of the tile; a round of kThreads entries past them is left out.
template <bool WIDE>
__device__ __forceinline__ void rank_in(const Keys<WIDE>& k, const uint32_t (&b)[kItems], const uint32_t (&m)[kItems],
                                        const uint64_t (&lo)[kItems], const uint64_t (&hi)[kItems], uint32_t steps,
                                        uint32_t n, uint32_t (&r)[kItems]) {
#pragma unroll
  for (uint32_t j = 0; j < kItems; ++j) r[j] = 0;
  for (uint32_t h = 1u << (steps - 1); h; h >>= 1) {
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) {
      if (j * kThreads >= n) break;
      const bool in = r[j] + h <= m[j];
      const uint32_t p = b[j] + (in ? r[j] + h - 1 : 0u);
      bool below;
      if (WIDE) {
        const uint64_t x = k.hi[p];
        below = x < hi[j];
        if (x == hi[j]) below = k.lo[p] < lo[j];
      } else {
        below = k.lo[p] < lo[j];
      }
      r[j] += in && below ? h : 0u;
    }
  }
}

// Entry `from` to place `to` of the result: its index, or all of it.
template <bool WIDE>
__device__ __forceinline__ void emit(const Buf& in, const Buf& out, uint32_t* dst, uint64_t to, uint32_t from,
                                     uint64_t lo, uint64_t hi) {
  if (dst) {
    dst[to] = from;
    return;
  }
  out.key_lo[to] = lo;
  if (WIDE) out.key_hi[to] = hi;
  out.amp[to] = in.amp[from];
}

// Each tile of kTile entries in order, by merging runs of doubling length in
// LDS: an entry's place in the merged run is its own place plus its rank among
// the other run's keys.
template <bool WIDE>
__global__ __launch_bounds__(1024) void k_sort_tiles(Buf in, Buf out, uint64_t n, uint32_t* dst) {
  __shared__ Keys<WIDE> k;
  __shared__ uint16_t s_idx[kTile];
  const uint64_t base = (uint64_t)blockIdx.x * kTile;
  const uint32_t m = (uint32_t)(n - base < kTile ? n - base : kTile);
#pragma unroll
  for (uint32_t j = 0; j < kItems; ++j) {
    const uint32_t p = j * kThreads + threadIdx.x;
    if (p < m) {
      k.lo[p] = in.key_lo[base + p];
      if (WIDE) k.hi[p] = in.key_hi[base + p];
      s_idx[p] = (uint16_t)p;
    }
  }
  __syncthreads();
  for (uint32_t w = 1; w < m; w <<= 1) {
    uint64_t lo[kItems], hi[kItems];
    uint32_t q[kItems], len[kItems], r[kItems];
    uint16_t id[kItems];
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) {
      const uint32_t p = j * kThreads + threadIdx.x;   // (keys at and past m are read but never ranked)
      lo[j] = k.lo[p];
      hi[j] = WIDE ? k.hi[p] : 0ull;
      id[j] = s_idx[p];
      q[j] = p ^ w;                                     // in the other run of the pair
      q[j] &= ~(w - 1);
      len[j] = p >= m || q[j] >= m ? 0u : (m - q[j] < w ? m - q[j] : w);
    }
    rank_in<WIDE>(k, q, len, lo, hi, 32 - __clz(w), m, r);
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) {
      const uint32_t p = j * kThreads + threadIdx.x;
      if (p >= m) continue;
      const uint32_t to = (p & ~(2 * w - 1)) + (p & (w - 1)) + r[j];
      k.lo[to] = lo[j];
      if (WIDE) k.hi[to] = hi[j];
      s_idx[to] = id[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (uint32_t j = 0; j < kItems; ++j) {
    const uint32_t p = j * kThreads + threadIdx.x;
    if (p < m) emit<WIDE>(in, out, dst, base + p, (uint32_t)base + s_idx[p], k.lo[p], WIDE ? k.hi[p] : 0ull);
  }
}

// How many of the first d entries of the merge of runs a (na entries) and b
// (nb) come from a: 64 candidates a step, by one wave (two or three steps of
// memory latency where halving takes sixteen).
template <bool WIDE>
__device__ __forceinline__ uint32_t split_at(const Buf& in, const uint32_t* a, uint32_t na, const uint32_t* b,
                                             uint32_t nb, uint32_t d) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t l = d > nb ? d - nb : 0u, h = d < na ? d : na;   // the answer is in [l, h]
  while (l < h) {
    const uint32_t step = (h - l + 63) / 64, i = l + lane * step;
    bool below = false;   // entry i of a comes before entry d - 1 - i of b
    if (i < h) {
      const uint32_t x = a[i], y = b[d - 1 - i];
      below = less<WIDE>(in.key_lo[x], WIDE ? in.key_hi[x] : 0ull, in.key_lo[y], WIDE ? in.key_hi[y] : 0ull);
    }
    const uint32_t c = (uint32_t)__popcll(__ballot(below));   // true for a prefix of the candidates
    if (c == 0) break;
    const uint32_t next = l + c * step;
    l += (c - 1) * step + 1;
    if (next < h) h = next;
  }
  return l;
}

// Runs of w entries (a multiple of kTile) merged in pairs, kTile outputs a
// block.
template <bool WIDE>
__global__ __launch_bounds__(1024) void k_sort_merge(Buf in, Buf out, uint64_t n, uint64_t w,
                                                     const uint32_t* __restrict__ src, uint32_t* dst) {
  __shared__ Keys<WIDE> k;
  __shared__ uint32_t s_cut[2];
  const uint64_t base = (uint64_t)blockIdx.x * kTile;
  const uint32_t m = (uint32_t)(n - base < kTile ? n - base : kTile);
  const uint64_t a0 = base & ~(2 * w - 1), b0 = a0 + w < n ? a0 + w : n;   // w is a power of two
  const uint32_t na = (uint32_t)(b0 - a0), nb = (uint32_t)(n - b0 < w ? n - b0 : w), d0 = (uint32_t)(base - a0);
  const uint32_t wave = threadIdx.x >> 6;
  if (wave < 2) {
    const uint32_t c = split_at<WIDE>(in, src + a0, na, src + b0, nb, wave ? d0 + m : d0);
    if ((threadIdx.x & 63) == 0) s_cut[wave] = c;
  }
  __syncthreads();
  const uint32_t i0 = s_cut[0], ma = s_cut[1] - i0;
  const uint32_t* a = src + a0 + i0;
  const uint32_t* b = src + b0 + (d0 - i0);
  uint32_t id[kItems];
  uint64_t lo[kItems], hi[kItems];
#pragma unroll
  for (uint32_t j = 0; j < kItems; ++j) {
    const uint32_t p = j * kThreads + threadIdx.x;
    id[j] = p < m ? (p < ma ? a[p] : b[p - ma]) : 0u;
  }
#pragma unroll
  for (uint32_t j = 0; j < kItems; ++j) {
    const uint32_t p = j * kThreads + threadIdx.x;
    lo[j] = hi[j] = 0;
    if (p >= m) continue;
    lo[j] = k.lo[p] = in.key_lo[id[j]];
    if (WIDE) hi[j] = k.hi[p] = in.key_hi[id[j]];
  }
  __syncthreads();
  uint32_t q[kItems], len[kItems], r[kItems];
#pragma unroll
  for (uint32_t j = 0; j < kItems; ++j) {
    const uint32_t p = j * kThreads + threadIdx.x;
    q[j] = p < ma && ma < m ? ma : 0u;
    len[j] = p >= m ? 0u : (p < ma ? m - ma : ma);
  }
  rank_in<WIDE>(k, q, len, lo, hi, 32 - __clz(kTile), m, r);
#pragma unroll
  for (uint32_t j = 0; j < kItems; ++j) {
    const uint32_t p = j * kThreads + threadIdx.x;
    if (p < m) emit<WIDE>(in, out, dst, base + (p < ma ? p : p - ma) + r[j], id[j], lo[j], hi[j]);
  }
}

template <bool WIDE>
void sort_state(hipStream_t st, Buf in, Buf out, uint64_t n, uint32_t* idx) {
  const int tiles = (int)((n + kTile - 1) / kTile);
  int passes = 0;
  for (uint64_t w = kTile; w < n; w <<= 1) ++passes;
  // The last pass writes `out`, so it reads idx; the passes before alternate
  // with the room of the labels of `out`.
  uint32_t* alt = reinterpret_cast<uint32_t*>(out.key_lo);
  auto dst_of = [&](int p) -> uint32_t* { return p == passes ? nullptr : ((passes - p) & 1) ? idx : alt; };
  hipLaunchKernelGGL(k_sort_tiles<WIDE>, dim3(tiles), dim3(kThreads), 0, st, in, out, n, dst_of(0));
  uint64_t w = kTile;
  for (int p = 1; p <= passes; ++p, w <<= 1)
    hipLaunchKernelGGL(k_sort_merge<WIDE>, dim3(tiles), dim3(kThreads), 0, st, in, out, n, w, dst_of(p - 1), dst_of(p));
}

}  // namespace

void launch_sort_state(hipStream_t st, bool wide, Buf in, Buf out, uint64_t n, uint32_t* idx) {
  if (wide) sort_state<true>(st, in, out, n, idx);
  else sort_state<false>(st, in, out, n, idx);
}

}  // namespace sparsesim
