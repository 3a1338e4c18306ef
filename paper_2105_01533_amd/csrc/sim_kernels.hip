// HIP kernels of libsparsesim for gfx950 (wave64).
//
// The state is a structure-of-arrays list of (label, amplitude) pairs.  Every
// kernel reads the live entry count from device memory, so the host never has
// to know it to launch work.  Kernels that change the entry count (branching
// gates, measurement) are "chunked": block b owns the contiguous entry range
// [b*chunk, (b+1)*chunk) with chunk fixed per kernel (chunk_len), counts what it
// will emit, a one-block scan turns the counts into output offsets, and the
// write kernel emits in entry order.  Output order is therefore a fixed
// function of the input order: runs are deterministic and no floating-point
// value is ever accumulated with atomics.
//
// Arithmetic is fixed so that results match a plain sequential evaluation:
// complex products are (a.re*b.re - a.im*b.im, a.re*b.im + a.im*b.re), sums of
// two products are evaluated left to right, |a|^2 = re*re + im*im, and the
// library is compiled with -ffp-contract=off.
#include <algorithm>

#include "entry_ops.h"
#include "u2_lds.h"

namespace sparsesim {
namespace {

using ent::cadd;
using ent::cmul;
using ent::hash_label;
using ent::sel2;
using ent::survives;

// Entries per block of a chunked launch of nb blocks: `per`, or an even split
// when nb blocks of `per` do not cover n.  The host sizes the grid from its
// bound on n (at least n), so block ranges, and every sum grouped by block,
// depend on n alone and not on where the host last read the count.
__device__ __forceinline__ uint64_t chunk_len(uint64_t n, uint64_t nb, uint64_t per) {
  const uint64_t even = (n + nb - 1) / nb;
  return even > per ? even : per;
}

__device__ __forceinline__ void chunk_range(uint64_t n, uint64_t per, uint64_t& begin, uint64_t& end) {
  const uint64_t chunk = chunk_len(n, gridDim.x, per);
  begin = (uint64_t)blockIdx.x * chunk;
  end = begin + chunk < n ? begin + chunk : n;
  if (begin > end) begin = end;
}

// Exclusive prefix over the block of per-thread counts e in {0,1,2}, in
// thread order.  Returns the thread's offset; *total gets the block sum.
// Every thread of the block must call it.
__device__ __forceinline__ uint32_t block_prefix012(uint32_t e, uint32_t* s_wave, uint32_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint64_t b1 = __ballot(e >= 1), b2 = __ballot(e >= 2);
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const uint32_t pre = __popcll(b1 & lt) + __popcll(b2 & lt);
  if (lane == 0) s_wave[wid] = __popcll(b1) + __popcll(b2);
  __syncthreads();
  uint32_t woff = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    const uint32_t x = s_wave[w];
    woff += w < wid ? x : 0u;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return woff + pre;
}

// Sum over the block in a fixed order (deterministic): a butterfly within
// each wave, then the waves' sums in wave order.  sh needs one slot per wave.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ double2 wave_sum(double2 v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double x = __shfl_xor(v.x, o), y = __shfl_xor(v.y, o);
    v = make_double2(v.x + x, v.y + y);
  }
  return v;
}
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* sh) {
  const int nw = blockDim.x >> 6;
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  T r = sh[0];
  for (int w = 1; w < nw; ++w) r = r + sh[w];
  __syncthreads();
  return r;
}

__device__ __forceinline__ double2 operator+(double2 a, double2 b) { return cadd(a, b); }

// ---------------------------------------------------------------------------
__global__ void k_set_basis(Buf b, uint64_t* nnz, uint64_t lo, uint64_t hi) {
  b.key_lo[0] = lo;
  if (b.key_hi) b.key_hi[0] = hi;
  b.amp[0] = make_double2(1.0, 0.0);
  *nnz = 1;
}

__global__ void k_fill(uint64_t* __restrict__ p, uint64_t v, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// ---------------------------------------------------------------------------
// Fused phase/permutation pass (Sec. 3.2): each label takes every gate of the
// run in order, G_n o ... o G_1, entirely in registers; one read and one
// write of the entry per run.  Gate descriptors are wave-uniform.
template <bool WIDE, int ITEMS>
__global__ __launch_bounds__(256) void k_mono(Buf b, const uint64_t* __restrict__ nnz_p,
                                              const MonoDesc* __restrict__ g, uint32_t ng, uint32_t rf,
                                              uint32_t bpe, Ctl* ctl) {
  const uint64_t n = *nnz_p;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    atomicAdd((unsigned long long*)&ctl->updates, (unsigned long long)(n * ng));
    atomicAdd((unsigned long long*)&ctl->mono_bytes, (unsigned long long)(n * bpe));
    atomicAdd((unsigned long long*)&ctl->mono_updates, (unsigned long long)(n * ng));
  }
  const bool run_phase = rf & kRunPhase, run_flip = rf & kRunFlip;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * ITEMS;
  for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x * ITEMS; base < n; base += stride) {
    uint64_t lo[ITEMS], hi[ITEMS];
    double2 a[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint64_t idx = base + (uint64_t)i * blockDim.x + threadIdx.x;
      const bool ok = idx < n;
      lo[i] = ok ? b.key_lo[idx] : 0ull;
      hi[i] = (WIDE && ok) ? b.key_hi[idx] : 0ull;
      a[i] = make_double2(0.0, 0.0);
      if (ok && run_phase) a[i] = b.amp[idx];
    }
    for (uint32_t j = 0; j < ng; ++j) {
      const MonoDesc d = g[j];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) ent::mono_step(d, WIDE, lo[i], hi[i], a[i]);
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint64_t idx = base + (uint64_t)i * blockDim.x + threadIdx.x;
      if (idx < n) {
        if (run_flip) {
          b.key_lo[idx] = lo[i];
          if (WIDE) b.key_hi[idx] = hi[i];
        }
        if (run_phase) b.amp[idx] = a[i];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Hash index: open addressing with linear probing over a power-of-two table
// of 32-bit slots, claimed with CAS: the entry's index in the low bits the
// state needs, a fingerprint of its label in the rest.  Labels are unique, so
// an insert never meets its own label.  The table is sized in the kernels, from
// the entry count on the device: the host knows only a bound, several times
// the count between two reads, and a table sized for the bound spreads the
// probes over that much more memory and costs that much more to empty
// (40-qubit Trotter step, 2,500 gates: 85 -> 76 ms).
//
// The workspace holds two tables.  A gate builds and probes one and empties
// what the gate before left in the other, so no launch is spent on it, and the
// gate's own write can index its outputs for the next one.
struct Geom {
  uint32_t mask, bits;   // slots - 1; index bits of a slot
};
__device__ __forceinline__ Geom index_geom(const IndexTab& t, uint64_t n) {
  const uint64_t want = (uint64_t)((double)n * t.inv_load) + 2;
  uint64_t slots = want <= 64 ? 64ull : 1ull << (64 - __clzll(want - 1));
  if (slots > t.max_slots) slots = t.max_slots;
  // n < 2^bits, so a slot in use is never all ones (the empty slot).
  return {(uint32_t)(slots - 1), n ? 64u - __clzll(n) : 1u};
}

// Index entry i (label lo/hi).
struct Claim {
  uint32_t slot, val;
  bool wanted;
};
__device__ __forceinline__ Claim index_claim(const Geom& gm, uint64_t lo, uint64_t hi, uint32_t i, bool wanted) {
  const uint64_t h = hash_label(lo, hi);
  return {(uint32_t)h & gm.mask, (uint32_t)((h >> 32) >> gm.bits) << gm.bits | i, wanted};
}
// The claim's remaining tries after one that found slot content old.
__device__ __forceinline__ uint32_t index_settle(uint32_t* slots, const Geom& gm, Claim c, uint32_t old) {
  uint32_t tries = 1;
  while (old != kFreeSlot && tries <= gm.mask) {
    c.slot = (c.slot + 1) & gm.mask;
    old = atomicCAS(&slots[c.slot], kFreeSlot, c.val);
    ++tries;
  }
  return tries;
}
__device__ __forceinline__ uint32_t index_insert(uint32_t* slots, const Geom& gm, uint64_t lo, uint64_t hi,
                                                 uint32_t i) {
  const Claim c = index_claim(gm, lo, hi, i, true);
  return index_settle(slots, gm, c, atomicCAS(&slots[c.slot], kFreeSlot, c.val));
}

// Empty what the last build left in a table: by all threads of the grid, 16
// bytes a store (the slots in use are a power of two, at least 64).
__device__ __forceinline__ void index_empty(uint32_t* slots, const TabCtl* tc) {
  const uint32_t mask = tc->mask;
  if (!mask || tc->nopair) return;
  const uint64_t n4 = ((uint64_t)mask + 1) / 4;
  uint4* __restrict__ p = reinterpret_cast<uint4*>(slots);
  const uint4 e = make_uint4(kFreeSlot, kFreeSlot, kFreeSlot, kFreeSlot);
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n4; k += (uint64_t)gridDim.x * blockDim.x)
    p[k] = e;
}

__global__ __launch_bounds__(256) void k_index_empty(IndexTab t) {
  index_empty(t.slots, t.tc);
  index_empty(t.other, t.tc_other);
}

// Imported labels are distinct: all of them into the table, where two equal
// ones meet (the later one's tries pass every slot that the earlier one's
// did, so they reach it).  One random CAS per entry and few compares (26 G/s):
// 100003 labels in 16 us; sorting them on the host took 12 ms.
template <bool WIDE>
__global__ __launch_bounds__(256) void k_import_check(Buf b, uint64_t n, IndexTab t, uint64_t* nnz_out) {
  const Geom gm = index_geom(t, n);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    t.tc->mask = gm.mask;
    t.tc->bits = gm.bits;
    t.tc->nopair = 0;
    *nnz_out = n;
  }
  const uint32_t idx_mask = (1u << gm.bits) - 1u;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t lo = b.key_lo[i], hi = WIDE ? b.key_hi[i] : 0ull;
    Claim c = index_claim(gm, lo, hi, (uint32_t)i, true);
    for (uint64_t p = 0; p <= gm.mask; ++p) {
      const uint32_t v = atomicCAS(&t.slots[c.slot], kFreeSlot, c.val);
      if (v == kFreeSlot) break;
      if (!((v ^ c.val) & ~idx_mask)) {
        const uint32_t j = v & idx_mask;
        if (b.key_lo[j] == lo && (!WIDE || b.key_hi[j] == hi)) {
          t.tc->dup = 1;
          break;
        }
      }
      c.slot = (c.slot + 1) & gm.mask;
    }
  }
}

// The label of the entry before or after this thread's (the wave holds 64
// consecutive entries; i < n).
template <bool WIDE>
__device__ __forceinline__ bool next_to(const Buf& b, uint64_t n, uint64_t i, uint64_t lo, uint64_t hi, uint64_t qlo,
                                        uint64_t qhi, bool after, bool inside) {
  const int lane = threadIdx.x & 63;
  uint64_t l = after ? __shfl_down(lo, 1) : __shfl_up(lo, 1);
  uint64_t h = WIDE ? (after ? __shfl_down(hi, 1) : __shfl_up(hi, 1)) : 0ull;
  const bool edge = lane == (after ? 63 : 0);
  const bool there = after ? i + 1 < n : i > 0 && i < n;
  if (edge && inside) return false;
  if (edge && there) {
    l = b.key_lo[after ? i + 1 : i - 1];
    if (WIDE) h = b.key_hi[after ? i + 1 : i - 1];
  }
  return there && l == qlo && (!WIDE || h == qhi);
}

// Block sums of two per-thread counters added to dst[0], dst[1] by thread 0
// (one atomic pair per block); nothing when dst is null (counting off).
__device__ __forceinline__ void add_counters(unsigned long long* dst, uint32_t a, uint32_t b) {
  __shared__ uint32_t sh_a[16], sh_b[16];
  if (!dst) return;   // uniform: a kernel argument
  const uint32_t x = block_sum(a, sh_a), y = block_sum(b, sh_b);
  if (threadIdx.x == 0) {
    if (x) atomicAdd(dst, (unsigned long long)x);
    if (y) atomicAdd(dst + 1, (unsigned long long)y);
  }
}

// A held run's gates in LDS, loaded all at once: read one by one from memory,
// each costs the latency of its first touch (0.5 us or more).
struct RunLds {
  MonoDesc g[kHeldMax];
  __device__ __forceinline__ void load(const MonoDesc* __restrict__ src, uint32_t ng) {
    uint4* dst = reinterpret_cast<uint4*>(g);
    const uint4* s4 = reinterpret_cast<const uint4*>(src);
    for (uint32_t k = threadIdx.x; k < ng * (sizeof(MonoDesc) / 16); k += blockDim.x) dst[k] = s4[k];
    __syncthreads();
  }
};

// Index build, with the short phase/permutation run before the gate applied
// on the way (MONO: the run's gates in order on each entry, as k_mono, in the
// same pass over the labels).  Only the entries a partner look-up can ask for
// are indexed: those under the op's controls with the pivot bit clear (the
// look-ups come from their partners, whose pivot bit is set) whose partner is
// not the entry next to them in the wave (the two outputs of a pair are written
// next to each other, and the look-ups look there first).  Bound by the CAS
// rate, 26 G/s whatever the scope or the table's size (a plain random store
// runs at 77 G/s, a load at 55-75 G/s): indexing every entry, so that the
// single pass could look up both partners of a pair and the partner pass go,
// was slower at every size (2^20 entries of 24 bytes: 33 + 17 + 51 us against
// 75 + 148).
template <bool WIDE, bool MONO>
__global__ __launch_bounds__(256) void k_index_build(Buf b, const uint64_t* __restrict__ nnz_p, IndexTab t, U2Desc d,
                                                     unsigned long long* count, const MonoDesc* __restrict__ g,
                                                     uint32_t ng, uint32_t rf, Ctl* ctl) {
  __shared__ RunLds sg;
  const uint64_t n = *nnz_p;
  const Geom gm = index_geom(t, n);
  if (MONO) sg.load(g, ng);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    t.tc->mask = gm.mask;
    t.tc->bits = gm.bits;
    t.tc->nopair = 0;
    if (MONO) atomicAdd((unsigned long long*)&ctl->updates, (unsigned long long)(n * ng));
  }
  uint32_t inserts = 0, cas = 0;
  for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x; base < n; base += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t i = base + threadIdx.x;
    const bool ok = i < n;
    uint64_t lo = 0, hi = 0;
    if (ok) {
      lo = b.key_lo[i];
      hi = WIDE ? b.key_hi[i] : 0ull;
      if (MONO) {
        double2 a = make_double2(0.0, 0.0);
        if (rf & kRunPhase) a = b.amp[i];
        for (uint32_t j = 0; j < ng; ++j) ent::mono_step(sg.g[j], WIDE, lo, hi, a);
        if (rf & kRunFlip) {
          b.key_lo[i] = lo;
          if (WIDE) b.key_hi[i] = hi;
        }
        if (rf & kRunPhase) b.amp[i] = a;
      }
    }
    // Every lane takes part in the neighbours' shuffles (only those inside
    // the wave: other waves' labels may be before or after the run).
    const uint64_t qlo = lo ^ d.x_lo, qhi = WIDE ? hi ^ d.x_hi : 0ull;
    const bool before = next_to<WIDE>(b, n, i, lo, hi, qlo, qhi, false, true);
    const bool after = next_to<WIDE>(b, n, i, lo, hi, qlo, qhi, true, true);
    if (!ok || !ent::ctrl_ok(d, lo, hi, WIDE) || ent::pivot_set(d, lo, hi, WIDE)) continue;
    ++inserts;
    if (!(before || after) || count) cas += index_insert(t.slots, gm, lo, hi, (uint32_t)i);
  }
  add_counters(count, inserts, cas);
}

// The index of label lo/hi among the indexed entries, or kNoPartner.
template <bool WIDE>
__device__ __forceinline__ uint32_t find_label(const Buf& b, const uint32_t* __restrict__ slots, const Geom& gm,
                                               uint64_t n, uint64_t lo, uint64_t hi, uint32_t& steps) {
  const uint64_t h = hash_label(lo, hi);
  const uint32_t fp = (uint32_t)((h >> 32) >> gm.bits);
  const uint32_t idx_mask = (1u << gm.bits) - 1u;
  uint32_t slot = (uint32_t)h & gm.mask;
  for (uint64_t p = 0; p <= gm.mask; ++p) {
    const uint32_t v = slots[slot];
    ++steps;
    if (v == kFreeSlot) return kNoPartner;
    if ((uint32_t)((uint64_t)v >> gm.bits) == fp) {
      const uint32_t j = v & idx_mask;
      if (j < n && b.key_lo[j] == lo && (!WIDE || b.key_hi[j] == hi)) return j;
    }
    slot = (slot + 1) & gm.mask;
  }
  return kNoPartner;
}

// Partner look-up (Sec. 3.1: at most one per label): each entry under the
// controls with the pivot bit set finds label ^ x, next to itself or among the
// indexed entries; when found, it records its partner and marks it (a pivot-0
// entry has at most one such partner, so the marks never collide).  The pass
// also forms the AND and OR of all labels, from which the gate's write knows
// qubits that are the same in every entry, and empties the other table.
template <bool WIDE>
__global__ __launch_bounds__(1024) void k_u2_probe(Buf b, const uint64_t* __restrict__ nnz_p, IndexTab t, U2Desc d,
                                                   uint32_t* __restrict__ partner, uint32_t epoch,
                                                   unsigned long long* count) {
  __shared__ uint64_t s_m[4][16];
  const uint64_t n = *nnz_p;
  const Geom gm{t.tc->mask, t.tc->bits};
  const bool nopair = t.tc->nopair != 0;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (blockIdx.x == 0 && threadIdx.x < kLabelCells) {   // for the next gate's pass
    LabelCell& c = t.labels_other[threadIdx.x];
    c.and_lo = c.and_hi = ~0ull;
    c.or_lo = c.or_hi = 0;
  }
  uint32_t lookups = 0, steps = 0;
  uint64_t m[4] = {~0ull, ~0ull, 0, 0};   // AND and OR of the labels
  for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x; base < n; base += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t i = base + threadIdx.x;
    const bool ok = i < n;
    uint64_t lo = 0, hi = 0;
    if (ok) {
      lo = b.key_lo[i];
      hi = WIDE ? b.key_hi[i] : 0ull;
      m[0] &= lo;
      m[2] |= lo;
      if (WIDE) {
        m[1] &= hi;
        m[3] |= hi;
      }
    }
    if (nopair) continue;   // uniform
    const uint64_t qlo = lo ^ d.x_lo, qhi = WIDE ? hi ^ d.x_hi : 0ull;
    const bool before = next_to<WIDE>(b, n, i, lo, hi, qlo, qhi, false, false);
    const bool after = next_to<WIDE>(b, n, i, lo, hi, qlo, qhi, true, false);
    if (!ok || !ent::ctrl_ok(d, lo, hi, WIDE) || !ent::pivot_set(d, lo, hi, WIDE)) continue;
    ++lookups;
    uint32_t j = before ? (uint32_t)i - 1u : after ? (uint32_t)i + 1u : kNoPartner;
    if (j == kNoPartner || count) j = find_label<WIDE>(b, t.slots, gm, n, qlo, qhi, steps);
    partner[i] = j;
    if (j != kNoPartner) partner[j] = kHasPartner | epoch;
  }
  index_empty(t.other, t.tc_other);
  if ((uint64_t)blockIdx.x * blockDim.x < n) {   // uniform: the block saw an entry
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      m[0] &= __shfl_xor(m[0], o);
      m[2] |= __shfl_xor(m[2], o);
      if (WIDE) {
        m[1] &= __shfl_xor(m[1], o);
        m[3] |= __shfl_xor(m[3], o);
      }
    }
    if (lane == 0)
      for (int k = 0; k < 4; ++k) s_m[k][wid] = m[k];
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
        m[0] &= s_m[0][w];
        m[1] &= s_m[1][w];
        m[2] |= s_m[2][w];
        m[3] |= s_m[3][w];
      }
      LabelCell& c = t.labels[blockIdx.x % kLabelCells];
      atomicAnd((unsigned long long*)&c.and_lo, (unsigned long long)m[0]);
      atomicOr((unsigned long long*)&c.or_lo, (unsigned long long)m[2]);
      if (WIDE) {
        atomicAnd((unsigned long long*)&c.and_hi, (unsigned long long)m[1]);
        atomicOr((unsigned long long*)&c.or_hi, (unsigned long long)m[3]);
      }
    }
    __syncthreads();
  }
  add_counters(count, lookups, steps);
}

// Whether entry (lo, hi) has a partner, from its word of the partner array,
// and the partner's index if the entry's own pivot bit is set.
template <bool WIDE>
__device__ __forceinline__ uint32_t partner_of(const U2Desc& d, uint64_t lo, uint64_t hi, uint32_t word,
                                               uint32_t epoch) {
  if (!ent::ctrl_ok(d, lo, hi, WIDE)) return kNoPartner;
  if (ent::pivot_set(d, lo, hi, WIDE)) return word;
  return word == (kHasPartner | epoch) ? 0u : kNoPartner;
}

// The count, write and single-pass kernels take partner == null for a gate
// whose partner mask touches a qubit that is the same in every entry: then no
// entry has a partner, and no index is built or probed.
template <bool WIDE>
__device__ __forceinline__ bool pivot_set(const U2Desc& d, uint64_t lo, uint64_t hi) {
  return ent::pivot_set(d, lo, hi, WIDE);
}

using ent::U2Out;
template <bool WIDE>
__device__ __forceinline__ U2Out u2_eval(const Buf& b, const U2Desc& d, uint64_t lo, uint64_t hi, double2 a,
                                         uint32_t j) {
  return ent::u2_eval(d, WIDE, b.amp, lo, hi, a, j);
}

template <bool WIDE>
__global__ __launch_bounds__(256) void k_u2_count(Buf b, const uint64_t* __restrict__ nnz_p, U2Desc d,
                                                  const uint32_t* __restrict__ partner, uint32_t epoch,
                                                  uint32_t* __restrict__ tot, Ctl* ctl) {
  __shared__ uint32_t sh[256];
  __shared__ double2 shm[4];   // one slot per wave
  const uint64_t n = *nnz_p;
  uint64_t begin, end;
  chunk_range(n, kTwoPassChunk, begin, end);
  uint32_t emit = 0, dropped = 0;
  double mass = 0.0;
  for (uint64_t i = begin + threadIdx.x; i < end; i += blockDim.x) {
    const uint64_t lo = b.key_lo[i];
    const uint64_t hi = WIDE ? b.key_hi[i] : 0ull;
    const uint32_t j = partner ? partner_of<WIDE>(d, lo, hi, partner[i], epoch) : kNoPartner;
    const U2Out r = u2_eval<WIDE>(b, d, lo, hi, b.amp[i], j);
    if (r.mode == 0) {
      const bool k = survives(r.o0, d.eps);
      emit += k ? 1u : 0u;
      dropped += k ? 0u : 1u;
      mass += ent::dropped_mass(r.o0, k);
    } else if (r.mode == 1) {
      const bool k0 = survives(r.o0, d.eps), k1 = survives(r.o1, d.eps);
      emit += (k0 ? 1u : 0u) + (k1 ? 1u : 0u);
      dropped += (k0 ? 0u : 1u) + (k1 ? 0u : 1u);
      mass += ent::dropped_mass(r.o0, k0) + ent::dropped_mass(r.o1, k1);
    }
  }
  emit = block_sum(emit, sh);
  dropped = block_sum(dropped, sh);
  mass = block_sum(make_double2(mass, 0.0), shm).x;
  if (threadIdx.x == 0) {
    tot[blockIdx.x] = emit;
    if (dropped) {
      atomicAdd((unsigned long long*)&ctl->st_pruned, (unsigned long long)dropped);
      atomicAdd(&ctl->st_mass, mass);
    }
    if (blockIdx.x == 0) {
      atomicAdd((unsigned long long*)&ctl->st_updates, (unsigned long long)n);
      atomicAdd((unsigned long long*)&ctl->pass_bytes[0], (unsigned long long)(n * (WIDE ? 32u : 24u)));
    }
  }
}

// One block: exclusive scan of per-block counts in place; the total becomes
// the entry count of the output buffer.  The count pass's staged counters
// are committed if the total fits cap (otherwise the gate is rejected and
// they are discarded).
__global__ __launch_bounds__(1024) void k_scan(uint32_t* __restrict__ tot, int nb, uint64_t* nnz_out, Ctl* ctl,
                                               uint32_t entry_bytes, uint64_t cap) {
  __shared__ uint32_t sh[1024];
  const int per = (nb + blockDim.x - 1) / blockDim.x;
  const int first = threadIdx.x * per;
  uint32_t s = 0;
  for (int k = 0; k < per; ++k)
    if (first + k < nb) s += tot[first + k];
  sh[threadIdx.x] = s;
  __syncthreads();
  // Hillis-Steele inclusive scan over thread sums.
  for (unsigned off = 1; off < blockDim.x; off <<= 1) {
    const uint32_t x = threadIdx.x >= off ? sh[threadIdx.x - off] : 0u;
    __syncthreads();
    sh[threadIdx.x] += x;
    __syncthreads();
  }
  uint32_t run = sh[threadIdx.x] - s;
  for (int k = 0; k < per; ++k) {
    if (first + k < nb) {
      const uint32_t x = tot[first + k];
      tot[first + k] = run;
      run += x;
    }
  }
  if (threadIdx.x == blockDim.x - 1) {
    const uint64_t total = sh[threadIdx.x];
    *nnz_out = total;
    if (total <= cap) {
      if (total > ctl->peak) ctl->peak = total;
      ctl->pass_bytes[1] += total * entry_bytes;   // the write pass's output
      ctl->updates += ctl->st_updates;
      ctl->pruned += ctl->st_pruned;
      ctl->pruned_mass += ctl->st_mass;
    }
    ctl->st_updates = 0;
    ctl->st_pruned = 0;
    ctl->st_mass = 0.0;
  }
}

template <bool WIDE>
__global__ __launch_bounds__(256) void k_u2_write(Buf in, Buf out, const uint64_t* __restrict__ nnz_p,
                                                  const uint32_t* __restrict__ partner, uint32_t epoch,
                                                  const uint32_t* __restrict__ off, U2Desc d, Ctl* ctl) {
  __shared__ uint32_t s_wave[16];
  const uint64_t n = *nnz_p;
  if (blockIdx.x == 0 && threadIdx.x == 0)
    atomicAdd((unsigned long long*)&ctl->pass_bytes[1], (unsigned long long)(n * (WIDE ? 32u : 24u)));
  uint64_t begin, end;
  chunk_range(n, kTwoPassChunk, begin, end);
  uint64_t base = off[blockIdx.x];
  for (uint64_t tile = begin; tile < end; tile += blockDim.x) {
    const uint64_t i = tile + threadIdx.x;
    uint32_t e = 0;
    bool k0 = false, k1 = false;
    U2Out r;
    uint64_t lo = 0, hi = 0;
    r.mode = 2;
    if (i < end) {
      lo = in.key_lo[i];
      hi = WIDE ? in.key_hi[i] : 0ull;
      const uint32_t j = partner ? partner_of<WIDE>(d, lo, hi, partner[i], epoch) : kNoPartner;
      r = u2_eval<WIDE>(in, d, lo, hi, in.amp[i], j);
      if (r.mode == 0) {
        k0 = survives(r.o0, d.eps);
      } else if (r.mode == 1) {
        k0 = survives(r.o0, d.eps);
        k1 = survives(r.o1, d.eps);
      }
      e = (k0 ? 1u : 0u) + (k1 ? 1u : 0u);
    }
    uint32_t tile_total;
    uint64_t pos = base + block_prefix012(e, s_wave, &tile_total);
    if (r.mode == 0) {
      if (k0) {
        out.key_lo[pos] = lo;
        if (WIDE) out.key_hi[pos] = hi;
        out.amp[pos] = r.o0;
      }
    } else if (r.mode == 1) {
      const bool v = pivot_set<WIDE>(d, lo, hi);
      const uint64_t lo0 = v ? lo ^ d.x_lo : lo, hi0 = v ? hi ^ d.x_hi : hi;
      if (k0) {
        out.key_lo[pos] = lo0;
        if (WIDE) out.key_hi[pos] = hi0;
        out.amp[pos] = r.o0;
        ++pos;
      }
      if (k1) {
        out.key_lo[pos] = lo0 ^ d.x_lo;
        if (WIDE) out.key_hi[pos] = hi0 ^ d.x_hi;
        out.amp[pos] = r.o1;
      }
    }
    base += tile_total;
  }
}

// Single-pass branching gate: a block evaluates one tile of T ITEMS entries
// (Eq. 2 with T_eps, the results held in registers) and finds where its
// outputs go by a chained scan over the tiles: it publishes its tile's output
// count, adds its predecessors' counts back to the first published inclusive
// prefix, publishes its own inclusive prefix, writes, and takes the next tile.
// Tile numbers come from a counter in the order blocks ask for them, so a tile
// waited on always belongs to a block already running, whatever else runs on
// the device: each die starts its share of a grid by itself, and one filled with
// another handle's waiting blocks could keep a tile numbered by its block from
// ever starting.  The wait is bounded even so (a block that gives up sets error
// bit 2 and its outputs are wrong, but the kernel ends).  A
// status word packs (epoch, flag, count) and is read and written atomically at
// device scope, so no fence is needed; the epoch tells this launch's words from
// those of earlier launches.  Output order is input order, as in the two-pass
// form.
//
// What bounds it below a few million entries is the counter: atomics on one
// address complete one every 11.5 ns across the chip, so a tile costs that
// much whatever its size.  Hence blocks of 1024 threads, the tiles counted from
// the entry count on the device, and a block past them leaving before it takes
// a number.  With a number for each
// 512-entry tile of the bound this pass took 51 us at 2^20 entries of 24 bytes
// (1 us per 40 tiles), now 22 us.  Two counters alternate between launches,
// each reset by the launch that uses the other.
//
// The tile is 256 entries up to 2^16 entries, 512 up to 2^17, 1024 up to 2^18
// (up to 256 tiles: one a CU), 2048 up to 2^19, 4096 beyond (fewer numbers; 2^20
// entries of 24 bytes: 22 us against 31 with 1024).  The two small tiles take 5 %
// off a 40-qubit Trotter step (55.0 -> 52.5 ms) though each of up to 256 tiles
// waits for its number; numbered by block they would take 1 to 3 % more off.
//
// A gate whose outputs may not fit (seq != 0) writes nothing at or past cap,
// and if they did not fit reports an empty output and marks Ctl::over; `in`
// keeps the state.  The counters are staged by launch parity for that reason.
//
// NEXT: the short run up to the next branching gate is applied to the outputs
// and the outputs are indexed for that gate, which saves both a pass of their
// own (the table is sized for twice the entries, the most there can be).
// Nothing is indexed if the next gate's partner mask meets a qubit that is the
// same in every output.
constexpr uint64_t kStAgg = 1ull << 32, kStPrefix = 2ull << 32;
constexpr uint32_t kSpinMax = 1u << 22;
constexpr int kU2Threads = 1024, kU2Waves = kU2Threads / 64;

__device__ __forceinline__ uint64_t st_word(uint32_t epoch, uint64_t flag, uint32_t v) {
  return ((uint64_t)epoch << 34) | flag | v;
}

// The sum of the output counts of the tiles before `tile`, by one wave: lane l
// reads the status of tile - 1 - l and of the three tiles 64, 128 and 192
// before that in one round trip, and counts are added back to the nearest
// published inclusive prefix (positions before tile 0 count as a prefix of 0).
__device__ __forceinline__ uint32_t look_back(uint64_t* status, uint32_t tile, uint32_t epoch, uint32_t* error) {
  const int lane = threadIdx.x & 63;
  constexpr int kW = 4;
  uint32_t excl = 0, spins = 0;
  int64_t hi = (int64_t)tile - 1;
  while (hi >= 0) {
    uint64_t v[kW];
#pragma unroll
    for (int w = 0; w < kW; ++w) {
      const int64_t j = hi - lane - 64 * w;
      v[w] = st_word(epoch, kStPrefix, 0);
      if (j >= 0) v[w] = __hip_atomic_load(&status[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    bool wait = false, done = false;
#pragma unroll
    for (int w = 0; w < kW; ++w) {
      if (wait || done) continue;   // uniform
      const bool ready = (uint32_t)(v[w] >> 34) == epoch;
      const uint64_t pmask = __ballot(ready && (v[w] & kStPrefix));
      const uint64_t nready = __ballot(!ready);
      const int first = pmask ? __builtin_ctzll(pmask) : 63;   // nearest prefix in the window, else all 64
      const uint64_t need = first == 63 ? ~0ull : ((2ull << first) - 1);
      if (nready & need) {
        wait = true;
        continue;
      }
      excl += wave_sum(lane <= first ? (uint32_t)v[w] : 0u);
      done = pmask != 0;
      hi -= 64;
    }
    if (done) break;
    if (wait) {
      if (++spins > kSpinMax) {
        if (lane == 0) atomicOr(error, 2u);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  return excl;
}

// The last launch's staged counters join the state's (unless its outputs did
// not fit) and start over.  A wave's work, a cell a lane: one round trip.
__device__ __forceinline__ void commit_staged(Ctl* ctl, uint32_t p) {
  const uint32_t lane = threadIdx.x & 63;
  uint64_t updates = 0;
  uint32_t pruned = 0;
  double mass = 0.0;
  const bool fits = !ctl->over;
  if (lane < kStageCells) {
    StageCell& c = ctl->fst[p][lane];
    updates = c.updates;
    pruned = (uint32_t)c.pruned;   // at most two per entry of one gate
    mass = c.mass;
    c.updates = c.pruned = 0;
    c.mass = 0.0;
  }
  pruned = wave_sum(pruned);
  mass = wave_sum(make_double2(mass, 0.0)).x;
  if (lane != 0 || !fits) return;
  atomicAdd((unsigned long long*)&ctl->updates, (unsigned long long)updates);   // cell 0 holds them
  ctl->pruned += pruned;
  ctl->pruned_mass += mass;
}

// Whether the next gate's partner mask meets a qubit that is the same in every
// output of gate d and stays so over the run: those the same in every input
// but the partner mask's; a flip keeps its target only if its controls are.
// Every lane of the wave calls it.
__device__ __forceinline__ bool known_apart(const NextGate& nx, const U2Desc& d, const MonoDesc* run) {
  if (!nx.labels) return false;
  static_assert(kLabelCells == 32, "a cell per lane of half a wave");
  const LabelCell c = nx.labels[threadIdx.x & 31];
  uint64_t m[4] = {c.and_lo, c.and_hi, c.or_lo, c.or_hi};
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) {
    m[0] &= __shfl_xor(m[0], o);
    m[1] &= __shfl_xor(m[1], o);
    m[2] |= __shfl_xor(m[2], o);
    m[3] |= __shfl_xor(m[3], o);
  }
  uint64_t lo = ~(m[0] ^ m[2]) & ~d.x_lo, hi = ~(m[1] ^ m[3]) & ~d.x_hi;
  for (uint32_t k = 0; k < nx.run.ng; ++k) {
    const MonoDesc& g = run[k];
    if (!(g.flags & kFlip) || !((g.ctrl_lo & ~lo) | (g.ctrl_hi & ~hi))) continue;
    const uint64_t b = 1ull << (g.target & 63);
    if (g.target < 64) lo &= ~b;
    else hi &= ~b;
  }
  return ((nx.d.x_lo & lo) | (nx.d.x_hi & hi)) != 0;
}

struct U2Smem {
  uint32_t cnt[4 * kU2Waves];   // outputs by item and wave, then their exclusive prefix
  uint32_t drop[kU2Waves];
  double mass[kU2Waves];
  uint32_t tile, excl;
  bool apart;
  RunLds run;
};

// T: threads that take part (the others have left), ITEMS entries each.
template <bool WIDE, int T, int ITEMS, bool NEXT>
__device__ __forceinline__ void u2_tiles(const Buf& in, const Buf& out, uint64_t n, const uint32_t* __restrict__ partner,
                                         const U2Desc& d, Ctl* ctl, const TabCtl* tc, uint64_t* status, uint32_t par,
                                         uint32_t epoch, uint64_t* nnz_out, uint64_t cap, uint32_t seq,
                                         const NextGate& nx, U2Smem& sm) {
  constexpr int kItems = ITEMS;
  constexpr uint32_t kTile = T * ITEMS;
  constexpr int kW = T / 64;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t tiles = (uint32_t)((n + kTile - 1) / kTile);
  const Geom ng = NEXT ? index_geom(nx.tab, 2 * n <= cap ? 2 * n : cap) : Geom{0, 0};
  if (blockIdx.x >= tiles) {
    if (blockIdx.x == 0 && wid == 2) commit_staged(ctl, par ^ 1u);
    if (blockIdx.x == 0 && threadIdx.x == 0) {   // an empty state: nobody takes a number
      ctl->ticket[par ^ 1u] = 0;
      if (NEXT) nx.tab.tc->mask = 0, nx.tab.tc->nopair = 1;
      *nnz_out = 0;
    }
    return;
  }
  if (tc && tc->nopair) partner = nullptr;
  if (threadIdx.x == 0) sm.tile = atomicAdd(&ctl->ticket[par], 1u);
  if (NEXT) sm.run.load(nx.run.g, nx.run.ng);
  else __syncthreads();
  if (NEXT) {
    if (wid == 1) {
      const bool y = known_apart(nx, d, sm.run.g);
      if (lane == 0) sm.apart = y;
    }
    __syncthreads();
  }
  const bool apart = NEXT && sm.apart;
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (uint32_t tile = sm.tile; tile < tiles;) {
    // (before the tile's count is published: no later tile can have marked Ctl::over)
    if (tile == 0 && wid == 2) commit_staged(ctl, par ^ 1u);
    const uint64_t begin = (uint64_t)tile * kTile;
    U2Out r[kItems];
    uint64_t lo[kItems], hi[kItems];
    double2 a[kItems];
    uint32_t j[kItems], pre[kItems];
    bool k0[kItems], k1[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const uint64_t i = begin + (uint64_t)k * T + threadIdx.x;
      lo[k] = hi[k] = 0;
      a[k] = make_double2(0.0, 0.0);
      j[k] = kNoPartner;
      if (i < n) {
        if (partner) j[k] = partner[i];
        lo[k] = in.key_lo[i];
        hi[k] = WIDE ? in.key_hi[i] : 0ull;
        a[k] = in.amp[i];
      }
    }
    double2 aj[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      aj[k] = make_double2(0.0, 0.0);
      if (partner) j[k] = partner_of<WIDE>(d, lo[k], hi[k], j[k], epoch);
      if (j[k] != kNoPartner && pivot_set<WIDE>(d, lo[k], hi[k])) aj[k] = in.amp[j[k]];
    }
    uint32_t dropped = 0;
    double mass = 0.0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const uint64_t i = begin + (uint64_t)k * T + threadIdx.x;
      r[k] = ent::u2_eval(d, WIDE, lo[k], hi[k], a[k], j[k] != kNoPartner, aj[k]);
      if (i >= n) r[k].mode = 2;
      k0[k] = k1[k] = false;
      if (r[k].mode != 2) {
        k0[k] = survives(r[k].o0, d.eps);
        dropped += k0[k] ? 0u : 1u;
        mass += ent::dropped_mass(r[k].o0, k0[k]);
      }
      if (r[k].mode == 1) {
        k1[k] = survives(r[k].o1, d.eps);
        dropped += k1[k] ? 0u : 1u;
        mass += ent::dropped_mass(r[k].o1, k1[k]);
      }
      // A thread emits k0 + k1 entries.
      const uint64_t b0 = __ballot(k0[k]), b1 = __ballot(k1[k]);
      pre[k] = __popcll(b0 & lt) + __popcll(b1 & lt);
      if (lane == 0) sm.cnt[k * kW + wid] = __popcll(b0) + __popcll(b1);
    }
    const bool drops = __ballot(dropped != 0) != 0;   // uniform in the wave
    uint32_t wd = 0;
    double wm = 0.0;
    if (drops) {
      wd = wave_sum(dropped);
      wm = wave_sum(make_double2(mass, 0.0)).x;
    }
    if (lane == 0) {
      sm.drop[wid] = wd;
      sm.mass[wid] = wm;
    }
    __syncthreads();
    if (wid == 0) {
      // Offsets within the tile (items in order, waves in order within an item),
      // then the tiles before it.
      static_assert(kItems * kW <= 64, "one lane per item and wave");
      const uint32_t x = lane < kItems * kW ? sm.cnt[lane] : 0u;
      uint32_t incl = x;
#pragma unroll
      for (int o = 1; o < kItems * kW; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
      }
      const uint32_t run = __shfl(incl, kItems * kW - 1);
      if (lane < kItems * kW) sm.cnt[lane] = incl - x;
      if (lane == 0) {
        __hip_atomic_store(&status[tile], st_word(epoch, tile == 0 ? kStPrefix : kStAgg, run), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        if (tile == 0) {
          ctl->ticket[par ^ 1u] = 0;   // for the next launch
          ctl->fst[par][0].updates = n;
          if (NEXT) {
            nx.tab.tc->mask = ng.mask;
            nx.tab.tc->bits = ng.bits;
            nx.tab.tc->nopair = apart;
          }
        }
      }
      const uint32_t excl = look_back(status, tile, epoch, &ctl->error);
      if (lane == 0) {
        if (tile != 0)
          __hip_atomic_store(&status[tile], st_word(epoch, kStPrefix, excl + run), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        sm.excl = excl;
        if (tile == tiles - 1) {
          const uint32_t eb = WIDE ? 32u : 24u;
          const uint64_t total = (uint64_t)excl + run;
          if (total <= cap) {
            *nnz_out = total;
            if (total > ctl->peak) ctl->peak = total;
            atomicAdd((unsigned long long*)&ctl->pass_bytes[1], (unsigned long long)((n + total) * eb));
            if (NEXT && nx.run.ng)
              atomicAdd((unsigned long long*)&ctl->updates, (unsigned long long)(total * nx.run.ng));
          } else {
            *nnz_out = 0;
            ctl->over = seq;
            ctl->over_n = n;
            __hip_atomic_store(ctl->over_seen, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          }
        }
      }
    } else if (wid == 1) {
      const uint32_t td = wave_sum(lane < kW ? sm.drop[lane] : 0u);
      const double tm = wave_sum(make_double2(lane < kW ? sm.mass[lane] : 0.0, 0.0)).x;
      if (lane == 0 && td) {
        StageCell& c = ctl->fst[par][tile % kStageCells];
        atomicAdd((unsigned long long*)&c.pruned, (unsigned long long)td);
        atomicAdd(&c.mass, tm);
      }
    }
    __syncthreads();
    const uint64_t base = sm.excl;
    Claim claim[NEXT ? 2 * kItems : 1];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const uint64_t p = base + sm.cnt[k * kW + wid] + pre[k];
      const bool flipped = r[k].mode == 1 && pivot_set<WIDE>(d, lo[k], hi[k]);
      uint64_t l0 = flipped ? lo[k] ^ d.x_lo : lo[k], h0 = flipped ? hi[k] ^ d.x_hi : hi[k];
      uint64_t l1 = l0 ^ d.x_lo, h1 = h0 ^ d.x_hi;
      double2 a0 = r[k].o0, a1 = r[k].o1;
      const uint64_t p1 = p + (k0[k] ? 1u : 0u);
      const bool w0 = k0[k] && p < cap, w1 = k1[k] && p1 < cap;
      if (NEXT) {
        for (uint32_t q = 0; q < nx.run.ng; ++q) {
          const MonoDesc g = sm.run.g[q];
          ent::mono_step(g, WIDE, l0, h0, a0);
          ent::mono_step(g, WIDE, l1, h1, a1);
        }
        // Partners written next to each other need no index (see k_u2_probe).
        const bool index = !apart && !(k0[k] && k1[k] && (l0 ^ l1) == nx.d.x_lo && (!WIDE || (h0 ^ h1) == nx.d.x_hi));
        claim[2 * k] = index_claim(ng, l0, h0, (uint32_t)p,
                                   index && w0 && ent::ctrl_ok(nx.d, l0, h0, WIDE) &&
                                       !ent::pivot_set(nx.d, l0, h0, WIDE));
        claim[2 * k + 1] = index_claim(ng, l1, h1, (uint32_t)p1,
                                       index && w1 && ent::ctrl_ok(nx.d, l1, h1, WIDE) &&
                                           !ent::pivot_set(nx.d, l1, h1, WIDE));
      }
      if (w0) {
        out.key_lo[p] = l0;
        if (WIDE) out.key_hi[p] = h0;
        out.amp[p] = a0;
      }
      if (w1) {
        out.key_lo[p1] = l1;
        if (WIDE) out.key_hi[p1] = h1;
        out.amp[p1] = a1;
      }
    }
    if (NEXT && !apart) {
      // All first tries in flight together.
      uint32_t old[2 * kItems];
#pragma unroll
      for (int k = 0; k < 2 * kItems; ++k) {
        old[k] = kFreeSlot;
        if (claim[k].wanted) old[k] = atomicCAS(&nx.tab.slots[claim[k].slot], kFreeSlot, claim[k].val);
      }
#pragma unroll
      for (int k = 0; k < 2 * kItems; ++k) index_settle(nx.tab.slots, ng, claim[k], old[k]);
    }
    if (tiles <= gridDim.x) break;   // a tile for each block: no more to take
    if (threadIdx.x == 0) sm.tile = atomicAdd(&ctl->ticket[par], 1u);
    __syncthreads();
    tile = sm.tile;
  }
}

// One code path per tile size, chosen by the entry count on the device (the
// bound may be many times it): a small state's time is mostly latency, the
// fetch of the kernel's code part of it, so each path is no longer than it
// has to be (one path of four entries a thread for all sizes: 13 against 9 us
// at 31,000 entries).
template <bool WIDE, bool NEXT>
__global__ __launch_bounds__(kU2Threads) void k_u2_fused(Buf in, Buf out, const uint64_t* __restrict__ nnz_p,
                                                         const uint32_t* __restrict__ partner, U2Desc d, Ctl* ctl,
                                                         const TabCtl* tc, uint64_t* status, uint32_t par,
                                                         uint32_t epoch, uint64_t* nnz_out, uint64_t cap,
                                                         uint32_t seq, NextGate nx) {
  __shared__ U2Smem sm;
  const uint64_t n = *nnz_p;
#define SPARSESIM_U2_TILES(T, I) \
  u2_tiles<WIDE, T, I, NEXT>(in, out, n, partner, d, ctl, tc, status, par, epoch, nnz_out, cap, seq, nx, sm)
  if (n <= 256u * 256) {
    if (threadIdx.x >= 256) return;
    SPARSESIM_U2_TILES(256, 1);
  } else if (n <= 256u * 512) {
    if (threadIdx.x >= 512) return;
    SPARSESIM_U2_TILES(512, 1);
  } else if (n <= 256u * kU2Threads) {
    SPARSESIM_U2_TILES(kU2Threads, 1);
  } else if (n <= 512u * kU2Threads) {
    SPARSESIM_U2_TILES(kU2Threads, 2);
  } else {
    SPARSESIM_U2_TILES(kU2Threads, 4);
  }
#undef SPARSESIM_U2_TILES
}

__global__ void k_u2_restore(Ctl* ctl, int cur) {
  ctl->nnz[cur] = ctl->over_n;
  ctl->over = 0;
  ctl->error = 0;
  for (int p = 0; p < 2; ++p)
    for (StageCell& c : ctl->fst[p]) {
      c.updates = c.pruned = 0;
      c.mass = 0.0;
    }
}

__global__ void k_u2_tickets(Ctl* ctl) {
  for (int p = 0; p < 2; ++p) ctl->ticket[p] = ctl->lds_ticket[p] = 0;
}

// ---------------------------------------------------------------------------
// What a thread counted over the gates of a launch; waves add theirs up by
// shuffles, then one atomic a counter (block sums through LDS were no faster).
struct BlockCount {
  uint32_t dropped = 0, ix[4] = {};
  double mass = 0.0;
};
__device__ __forceinline__ void add_counts(const BlockCount& c, Ctl* ctl) {
  const uint32_t dropped = lds::wave_u(c.dropped);
  const double mass = lds::wave_d(c.mass);
  uint32_t ix[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) ix[q] = lds::wave_u(c.ix[q]);
  if (threadIdx.x & 63) return;
  if (dropped) {
    atomicAdd((unsigned long long*)&ctl->pruned, (unsigned long long)dropped);
    atomicAdd(&ctl->pruned_mass, mass);
  }
  for (int q = 0; q < 4; ++q)
    if (ix[q]) atomicAdd((unsigned long long*)&ctl->ix[q], (unsigned long long)ix[q]);
}

// Branching gates on a state of at most kChainMax entries in one block, the
// state and its partner index in LDS from gate to gate: same outputs, order and
// counters as the index-build / probe / single-pass kernels.  A launch runs a
// chain of gates with the short runs between them: a launch costs the host 6
// us and the GPU two or three with nothing to do, and a gate on a few entries
// over memory is little more than its chain of round trips (8 us).  A 12-qubit
// circuit's 10 gates with runs between them: 17 launches and 120 us of kernels;
// in one launch over memory 84 us, over LDS 27.  What bounds it is one CU's
// instruction issue, so waves without entries skip theirs: 4 us a gate up to
// 512 entries, 6 at 2048, where the kernels over many CUs take 14 to 16 and
// their launches 20.
struct ChainSmem {
  uint64_t lo[2 * kChainMax], hi[2 * kChainMax];   // a gate's inputs, then its outputs
  double2 amp[2 * kChainMax];
  uint32_t tab[2 * kChainMax];
  uint16_t par[kChainMax];
  MonoDesc g_run[kChainOps];
  ChainStep step[kChainSteps];
  uint32_t wave[kChainMax / 64];
};
static_assert(sizeof(ChainSmem) <= 160 * 1024, "LDS of a block");
constexpr uint16_t kNobody = 0xffff;   // in ChainSmem::par

// One gate on the n <= ITEMS * 1024 entries in sm, preceded by the run at run;
// returns the number of outputs.
template <bool WIDE, int ITEMS>
__device__ __forceinline__ uint32_t u2_resident(ChainSmem& sm, uint32_t n, const U2Desc& d, const MonoDesc* run,
                                                uint32_t ng, BlockCount& cnt) {
  constexpr uint32_t kWaves = 16;
  const uint32_t lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t kMask = (n <= 32 ? 64u : 2u << (32 - __clz(n - 1))) - 1u;   // at least two slots an entry
  uint64_t lo[ITEMS], hi[ITEMS];
  double2 a[ITEMS];
  bool under[ITEMS], piv[ITEMS];
  for (uint32_t k = threadIdx.x; k <= kMask; k += 1024) sm.tab[k] = 0u;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint32_t i = k * 1024 + threadIdx.x;
    under[k] = piv[k] = false;
    lo[k] = hi[k] = 0;
    a[k] = make_double2(0.0, 0.0);
    if (k * 1024 + wid * 64 >= n) continue;   // uniform: a wave without entries
    if (i < n) {
      lo[k] = sm.lo[i];
      hi[k] = WIDE ? sm.hi[i] : 0ull;
      a[k] = sm.amp[i];
      for (uint32_t q = 0; q < ng; ++q) ent::mono_step(run[q], WIDE, lo[k], hi[k], a[k]);
      if (ng) {
        sm.lo[i] = lo[k];
        if (WIDE) sm.hi[i] = hi[k];
        sm.amp[i] = a[k];
      }
      sm.par[i] = kNobody;
      under[k] = ent::ctrl_ok(d, lo[k], hi[k], WIDE);
      piv[k] = ent::pivot_set(d, lo[k], hi[k], WIDE);
    }
  }
  __syncthreads();
  // Index the pivot-clear entries under the controls; the others under them
  // look up label ^ x, which makes the two each other's partner.
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (!under[k] || piv[k]) continue;
    const uint32_t i = k * 1024 + threadIdx.x;
    const uint32_t h = lds::hash<WIDE>(lo[k], hi[k]);
    const uint32_t val = (h >> lds::kIdxBits) << lds::kIdxBits | (i + 1u);
    ++cnt.ix[0];
    for (uint32_t p = 0; p <= kMask; ++p) {
      ++cnt.ix[1];
      if (atomicCAS(&sm.tab[(h + p) & kMask], 0u, val) == 0u) break;
    }
  }
  __syncthreads();
  uint32_t j[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    j[k] = kNobody;
    if (!under[k] || !piv[k]) continue;
    const uint64_t qlo = lo[k] ^ d.x_lo, qhi = WIDE ? hi[k] ^ d.x_hi : 0ull;
    const uint32_t h = lds::hash<WIDE>(qlo, qhi);
    const uint32_t fp = h >> lds::kIdxBits;
    ++cnt.ix[2];
    for (uint32_t p = 0; p <= kMask; ++p) {
      const uint32_t v = sm.tab[(h + p) & kMask];
      ++cnt.ix[3];
      if (v == 0u) break;
      const uint32_t c = (v & lds::kIdxMask) - 1u;
      if ((v >> lds::kIdxBits) == fp && sm.lo[c] == qlo && (!WIDE || sm.hi[c] == qhi)) {
        j[k] = c;
        sm.par[c] = 0;   // (it is somebody's)
        break;
      }
    }
  }
  __syncthreads();
  U2Out r[ITEMS];
  bool k0[ITEMS], k1[ITEMS];
  uint64_t b0[ITEMS], b1[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint32_t i = k * 1024 + threadIdx.x;
    k0[k] = k1[k] = false;
    b0[k] = b1[k] = 0;
    r[k].mode = 2;
    uint32_t kept = 0;
    if (k * 1024 + wid * 64 < n) {
      if (i < n) {
        if (under[k] && !piv[k]) j[k] = sm.par[i];
        double2 aj = make_double2(0.0, 0.0);
        if (piv[k] && j[k] != kNobody) aj = sm.amp[j[k]];
        r[k] = ent::u2_eval(d, WIDE, lo[k], hi[k], a[k], j[k] != kNobody, aj);
        k0[k] = r[k].mode != 2 && survives(r[k].o0, d.eps);
        k1[k] = r[k].mode == 1 && survives(r[k].o1, d.eps);
        if (r[k].mode != 2 && !k0[k]) {
          ++cnt.dropped;
          cnt.mass += ent::dropped_mass(r[k].o0, false);
        }
        if (r[k].mode == 1 && !k1[k]) {
          ++cnt.dropped;
          cnt.mass += ent::dropped_mass(r[k].o1, false);
        }
      }
      b0[k] = __ballot(k0[k]);
      b1[k] = __ballot(k1[k]);
      kept = __popcll(b0[k]) + __popcll(b1[k]);
    }
    if (lane == 0) sm.wave[k * kWaves + wid] = kept;
  }
  __syncthreads();   // (the inputs have been read)
  // Every wave scans the waves' counts; its own offset is the sum before it.
  uint32_t incl = lane < ITEMS * kWaves ? sm.wave[lane] : 0u;
#pragma unroll
  for (int o = 1; o < ITEMS * (int)kWaves; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= (uint32_t)o) incl += y;
  }
  const uint32_t total = __builtin_amdgcn_readlane(incl, ITEMS * kWaves - 1);
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (k * 1024 + wid * 64 >= n) continue;
    const uint32_t w = k * kWaves + wid;
    uint32_t p = (w ? __builtin_amdgcn_readlane(incl, w - 1) : 0u) + __popcll(b0[k] & lt) + __popcll(b1[k] & lt);
    const bool flipped = r[k].mode == 1 && piv[k];
    const uint64_t lo0 = flipped ? lo[k] ^ d.x_lo : lo[k], hi0 = flipped ? hi[k] ^ d.x_hi : hi[k];
    if (k0[k]) {
      sm.lo[p] = lo0;
      if (WIDE) sm.hi[p] = hi0;
      sm.amp[p] = r[k].o0;
      ++p;
    }
    if (k1[k]) {
      sm.lo[p] = lo0 ^ d.x_lo;
      if (WIDE) sm.hi[p] = hi0 ^ d.x_hi;
      sm.amp[p] = r[k].o1;
    }
  }
  __syncthreads();
  return total;
}

template <bool WIDE>
__global__ __launch_bounds__(1024) void k_u2_chain(Buf in, Buf out, uint64_t* nnz, int cur, Chain chain, Ctl* ctl) {
  const int cur0 = cur;
  __shared__ ChainSmem sm;
  auto count = [](uint64_t* p, uint64_t v) {
    if (v) atomicAdd((unsigned long long*)p, (unsigned long long)v);
  };
  constexpr uint32_t kEntry = WIDE ? 32u : 24u;
  const uint64_t n0 = nnz[cur];
  uint32_t n = __builtin_amdgcn_readfirstlane((uint32_t)(n0 > kChainMax ? kChainMax + 1 : n0));
  if (n > kChainMax) {   // the host launches this kernel only below the bound
    if (threadIdx.x == 0) atomicOr(&ctl->error, 4u);
    return;
  }
  // The chain into LDS: its steps (from the kernel arguments), its runs' gates and the state.
  {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(chain.s);
    uint32_t* dst = reinterpret_cast<uint32_t*>(sm.step);
    for (uint32_t k = threadIdx.x; k < chain.n * (uint32_t)(sizeof(ChainStep) / 4); k += 1024) dst[k] = src[k];
    const uint4* g4 = reinterpret_cast<const uint4*>(chain.ops);
    uint4* d4 = reinterpret_cast<uint4*>(sm.g_run);
    for (uint32_t k = threadIdx.x; k < chain.n_ops * (uint32_t)(sizeof(MonoDesc) / 16); k += 1024) d4[k] = g4[k];
  }
  for (uint32_t i = threadIdx.x; i < n; i += 1024) {
    sm.lo[i] = in.key_lo[i];
    if (WIDE) sm.hi[i] = in.key_hi[i];
    sm.amp[i] = in.amp[i];
  }
  __syncthreads();
  BlockCount cnt;
  uint64_t updates = 0, bytes = 0, peak = 0;
  uint32_t op = 0, tail = 0;   // tail: gates of a run after the last branching gate
#pragma unroll 1
  for (uint32_t k = 0; k < chain.n; ++k) {
    const ChainStep& st = sm.step[k];
    const uint32_t ng = __builtin_amdgcn_readfirstlane(st.ng), gate = __builtin_amdgcn_readfirstlane(st.gate);
    updates += (uint64_t)n * (ng + gate);
    if (!gate) {
      tail = ng;
      break;
    }
    const MonoDesc* run = sm.g_run + op;
    op += ng;
    uint32_t m;
    if (n <= 1024) {
      m = u2_resident<WIDE, 1>(sm, n, st.d, run, ng, cnt);
    } else if (n <= kChainMax) {
      m = u2_resident<WIDE, 2>(sm, n, st.d, run, ng, cnt);
    } else {   // (as above: the host's bound rules it out)
      if (threadIdx.x == 0) atomicOr(&ctl->error, 4u);
      break;
    }
    bytes += (uint64_t)(n + m) * kEntry;
    n = m;
    if (n > peak) peak = n;
    cur ^= 1;
  }
  const Buf to = cur == cur0 ? in : out;
  for (uint32_t i = threadIdx.x; i < n; i += 1024) {
    uint64_t lo = sm.lo[i], hi = WIDE ? sm.hi[i] : 0ull;
    double2 a = sm.amp[i];
    for (uint32_t q = 0; q < tail; ++q) ent::mono_step(sm.g_run[op + q], WIDE, lo, hi, a);
    to.key_lo[i] = lo;
    if (WIDE) to.key_hi[i] = hi;
    to.amp[i] = a;
  }
  add_counts(cnt, ctl);
  if (threadIdx.x == 0) {
    nnz[cur] = n;
    count(&ctl->updates, updates);
    count(&ctl->pass_bytes[4], bytes);
    if (peak > ctl->peak) ctl->peak = peak;
  }
}

// A branching gate on a state of at most kLdsU2Max entries in one launch: every
// block reads all labels (from L2), indexes those with the pivot bit clear in
// its own LDS and looks the others' partners up there, so that it knows the
// partners of its own 1024 entries without waiting for the other blocks; it
// evaluates these and writes their outputs after those of the blocks before it
// (look_back; blocks are numbered from a counter as in the single pass, while
// their label loads are on the way).  m: a run of at most kLdsRun gates before the gate, applied to
// whatever is read (the state's buffer keeps the entries before the run).
// Outputs, order and counters (an entry's insert or look-up counts in its own
// block) as the three kernels' of the global index, which at these sizes are
// their launches (three of 5 to 7 us and 20 us of host time) and round trips;
// one block with the index in LDS took 22 us at 4096 entries and 45 at 8192, this
// 16 and 28: the probes of one CU's LDS by all entries.
struct LdsTileSmem {
  uint32_t tab[2 * kLdsU2Max];
  uint64_t lo[1024], hi[1024];   // the block's own labels
  uint32_t has[1024];            // whether an own entry with the pivot bit clear has a partner
  MonoDesc run[kLdsRun];
  uint32_t wave[16], before, tile;
};
template <bool WIDE>
__global__ __launch_bounds__(1024) void k_u2_lds_tiles(Buf in, Buf out, const uint64_t* __restrict__ nnz_in,
                                                       uint64_t* nnz_out, U2Desc d, MonoRun m, uint64_t* status,
                                                       uint32_t par, uint32_t epoch, Ctl* ctl) {
  __shared__ LdsTileSmem sm;
  auto count = [](uint64_t* p, uint64_t v) {
    if (v) atomicAdd((unsigned long long*)p, (unsigned long long)v);
  };
  constexpr uint32_t kEntry = WIDE ? 32u : 24u;
  const uint64_t n0 = *nnz_in;
  if (n0 > kLdsU2Max) {   // the host launches this kernel only below the bound
    if (threadIdx.x == 0) {
      atomicOr(&ctl->error, 4u);
      ctl->lds_ticket[par ^ 1u] = 0;
    }
    return;
  }
  const uint32_t n = (uint32_t)n0, blocks = n ? (n + 1023) / 1024 : 1u;
  if (blockIdx.x >= blocks) return;
  uint32_t ticket = 0;
  if (threadIdx.x == 0) ticket = atomicAdd(&ctl->lds_ticket[par], 1u);
  const uint32_t lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t kMask = (n <= 32 ? 64u : 2u << (32 - __clz(n - 1))) - 1u;   // at least two slots an entry
  for (uint32_t k = threadIdx.x; k < m.ng * (uint32_t)(sizeof(MonoDesc) / 16); k += 1024)
    reinterpret_cast<uint4*>(sm.run)[k] = reinterpret_cast<const uint4*>(m.g)[k];
  for (uint32_t k = threadIdx.x; k <= kMask; k += 1024) sm.tab[k] = 0u;
  const bool flips = m.run_flags & kRunFlip;
  constexpr uint32_t kRounds = kLdsU2Max / 1024;
  uint64_t l[kRounds], h2[kRounds];   // the thread's label of each 1024
#pragma unroll
  for (uint32_t k = 0; k < kRounds; ++k) {
    const uint32_t i = k * 1024 + threadIdx.x;
    l[k] = i < n ? in.key_lo[i] : 0ull;
    h2[k] = WIDE && i < n ? in.key_hi[i] : 0ull;
  }
  if (threadIdx.x == 0) sm.tile = ticket;
  __syncthreads();
  const uint32_t b = __builtin_amdgcn_readfirstlane(sm.tile), own = b * 1024 + threadIdx.x;
  if (b >= blocks) return;   // (uniform; the counter starts from zero, see launch_u2_tickets)
  if (b == 0 && threadIdx.x == 0) ctl->lds_ticket[par ^ 1u] = 0;   // for the next launch
  double2 a = make_double2(0.0, 0.0);
  uint64_t lo = 0, hi = 0;            // of its own entry
  if (own < n) {
    a = in.amp[own];
    lo = in.key_lo[own];
    hi = WIDE ? in.key_hi[own] : 0ull;
    for (uint32_t q = 0; q < m.ng; ++q) ent::mono_step(sm.run[q], WIDE, lo, hi, a);
    sm.lo[threadIdx.x] = lo;
    if (WIDE) sm.hi[threadIdx.x] = hi;
    sm.has[threadIdx.x] = 0u;
  }
  uint32_t inserts = 0, cas = 0, lookups = 0, steps = 0;
#pragma unroll
  for (uint32_t k = 0; k < kRounds; ++k) {
    const uint32_t i = k * 1024 + threadIdx.x;
    if (k * 1024 + wid * 64 >= n) break;   // uniform
    if (flips) {
      for (uint32_t q = 0; q < m.ng; ++q)
        if (sm.run[q].flags & kFlip) {
          const uint64_t f = ent::ctrl_ok(sm.run[q], l[k], h2[k], WIDE) ? 1ull << (sm.run[q].target & 63) : 0ull;
          if (WIDE && sm.run[q].target >= 64) h2[k] ^= f;
          else l[k] ^= f;
        }
    }
    if (i >= n || !ent::ctrl_ok(d, l[k], h2[k], WIDE) || ent::pivot_set(d, l[k], h2[k], WIDE)) continue;
    const uint32_t h = lds::hash<WIDE>(l[k], h2[k]);
    const uint32_t val = (h >> lds::kIdxBits) << lds::kIdxBits | (i + 1u);
    uint32_t p = 0;
    while (atomicCAS(&sm.tab[(h + p) & kMask], 0u, val) != 0u && p < kMask) ++p;
    if (k == b) {
      ++inserts;
      cas += p + 1;
    }
  }
  __syncthreads();
  // Each entry under the controls with the pivot bit set looks up label ^ x: a
  // partner among the block's own entries learns of it.
  const bool under = own < n && ent::ctrl_ok(d, lo, hi, WIDE), piv = ent::pivot_set(d, lo, hi, WIDE);
#pragma unroll
  for (uint32_t k = 0; k < kRounds; ++k) {
    const uint32_t i = k * 1024 + threadIdx.x;
    if (k * 1024 + wid * 64 >= n) break;   // uniform
    if (i >= n || !ent::ctrl_ok(d, l[k], h2[k], WIDE) || !ent::pivot_set(d, l[k], h2[k], WIDE)) continue;
    const uint64_t qlo = l[k] ^ d.x_lo, qhi = WIDE ? h2[k] ^ d.x_hi : 0ull;
    const uint32_t h = lds::hash<WIDE>(qlo, qhi);
    const uint32_t fp = h >> lds::kIdxBits;
    for (uint32_t p = 0; p <= kMask; ++p) {
      const uint32_t v = sm.tab[(h + p) & kMask];
      if (v == 0u) break;
      const uint32_t mine = (v & lds::kIdxMask) - 1u - b * 1024;
      if ((v >> lds::kIdxBits) == fp && mine < 1024 && sm.lo[mine] == qlo && (!WIDE || sm.hi[mine] == qhi)) {
        sm.has[mine] = 1u;
        break;
      }
    }
  }
  // The own entry, if it emits the pair, takes its partner's amplitude from
  // wherever it is.
  bool has = false;
  double2 aj = make_double2(0.0, 0.0);
  if (under && piv) {
    const uint64_t qlo = lo ^ d.x_lo, qhi = WIDE ? hi ^ d.x_hi : 0ull;
    const uint32_t h = lds::hash<WIDE>(qlo, qhi);
    const uint32_t fp = h >> lds::kIdxBits;
    ++lookups;
    for (uint32_t p = 0; p <= kMask; ++p) {
      const uint32_t v = sm.tab[(h + p) & kMask];
      ++steps;
      if (v == 0u) break;
      if ((v >> lds::kIdxBits) != fp) continue;
      const uint32_t c = (v & lds::kIdxMask) - 1u;
      uint64_t cl = in.key_lo[c], ch = WIDE ? in.key_hi[c] : 0ull;
      aj = in.amp[c];
      for (uint32_t q = 0; q < m.ng; ++q) ent::mono_step(sm.run[q], WIDE, cl, ch, aj);
      has = cl == qlo && (!WIDE || ch == qhi);
      if (has) break;
    }
  }
  __syncthreads();
  if (under && !piv) has = sm.has[threadIdx.x] != 0u;
  U2Out r = ent::u2_eval(d, WIDE, lo, hi, a, has, aj);
  if (own >= n) r.mode = 2;
  const bool k0 = r.mode != 2 && survives(r.o0, d.eps), k1 = r.mode == 1 && survives(r.o1, d.eps);
  const uint32_t dropped = (r.mode != 2 && !k0 ? 1u : 0u) + (r.mode == 1 && !k1 ? 1u : 0u);
  const double mass = (r.mode != 2 ? ent::dropped_mass(r.o0, k0) : 0.0) + (r.mode == 1 ? ent::dropped_mass(r.o1, k1) : 0.0);
  const uint64_t b0 = __ballot(k0), b1 = __ballot(k1), lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  if (lane == 0) sm.wave[wid] = __popcll(b0) + __popcll(b1);
  __syncthreads();
  uint32_t incl = lane < 16 ? sm.wave[lane] : 0u;
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= (uint32_t)o) incl += y;
  }
  const uint32_t total = __builtin_amdgcn_readlane(incl, 15);
  if (wid == 0) {
    if (lane == 0)
      __hip_atomic_store(&status[b], st_word(epoch, b == 0 ? kStPrefix : kStAgg, total), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t before = look_back(status, b, epoch, &ctl->error);
    if (lane == 0) sm.before = before;
  }
  __syncthreads();
  uint32_t p = sm.before + (wid ? __builtin_amdgcn_readlane(incl, wid - 1) : 0u) + __popcll(b0 & lt) + __popcll(b1 & lt);
  const bool flipped = r.mode == 1 && piv;
  const uint64_t lo0 = flipped ? lo ^ d.x_lo : lo, hi0 = flipped ? hi ^ d.x_hi : hi;
  if (k0) {
    out.key_lo[p] = lo0;
    if (WIDE) out.key_hi[p] = hi0;
    out.amp[p] = r.o0;
    ++p;
  }
  if (k1) {
    out.key_lo[p] = lo0 ^ d.x_lo;
    if (WIDE) out.key_hi[p] = hi0 ^ d.x_hi;
    out.amp[p] = r.o1;
  }
  BlockCount cnt;
  cnt.dropped = dropped;
  cnt.mass = mass;
  cnt.ix[0] = inserts;
  cnt.ix[1] = cas;
  cnt.ix[2] = lookups;
  cnt.ix[3] = steps;
  add_counts(cnt, ctl);
  if (threadIdx.x == 0 && b == blocks - 1) {
    const uint64_t n_out = sm.before + total;
    *nnz_out = n_out;
    if (n_out > ctl->peak) ctl->peak = n_out;
    count(&ctl->updates, (uint64_t)n * (m.ng + 1));
    count(&ctl->pass_bytes[4], (n + n_out) * kEntry);
  }
}

// ---------------------------------------------------------------------------
// Measurement (Born rule): per-block sums of |a|^2 split by the measured bit,
// a one-block decision, then an ordered compaction that scales the survivors.
template <bool WIDE>
__global__ __launch_bounds__(256) void k_measure_reduce(Buf b, const uint64_t* __restrict__ nnz_p, uint32_t q,
                                                        double2* __restrict__ part, uint32_t* __restrict__ cnt1) {
  __shared__ double2 shd[256];
  __shared__ uint32_t shu[256];
  const uint64_t n = *nnz_p;
  uint64_t begin, end;
  chunk_range(n, meas_chunk(n), begin, end);
  double p0 = 0.0, p1 = 0.0;
  uint32_t c1 = 0;
  const bool qhi = WIDE && q >= 64;
  for (uint64_t i = begin + threadIdx.x; i < end; i += blockDim.x) {
    const uint64_t w = qhi ? b.key_hi[i] : b.key_lo[i];
    const double2 a = b.amp[i];
    const double p = a.x * a.x + a.y * a.y;
    if ((w >> (q & 63)) & 1ull) {
      p1 += p;
      ++c1;
    } else {
      p0 += p;
    }
  }
  const double2 s = block_sum(make_double2(p0, p1), shd);
  const uint32_t c = block_sum(c1, shu);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = s;
    cnt1[blockIdx.x] = c;
  }
}

__global__ __launch_bounds__(1024) void k_measure_decide(const double2* __restrict__ part,
                                                         const uint32_t* __restrict__ cnt1,
                                                         uint32_t* __restrict__ off, int nb,
                                                         const uint64_t* __restrict__ nnz_in, uint64_t* nnz_out,
                                                         double u, int32_t forced, MeasRec* rec, int32_t* outcome,
                                                         Ctl* ctl, uint32_t entry_bytes,
                                                         const uint32_t* __restrict__ in_off) {
  __shared__ double2 shd[1024];
  __shared__ uint32_t shu[1024];
  __shared__ int s_o;
  // Every load is issued before any sum needs it (a rolled loop would wait on
  // each in turn); the sums keep the per-thread order k, k + 1024, ...
  constexpr int kPer = kMaxBlocks / 1024;
  const uint64_t n = *nnz_in;
  double2 pv[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int k = threadIdx.x + 1024 * i;
    pv[i] = make_double2(0.0, 0.0);
    if (k < nb) pv[i] = part[k];
  }
  // Per-block kept counts need each block's input length: its uniform chunk,
  // or (in_off given) the range the previous measurement's write block
  // produced.  Thread t owns blocks [t per, (t + 1) per).
  const uint64_t chunk = chunk_len(n, nb, meas_chunk(n));
  const int per = (nb + 1023) / 1024;
  const int first = threadIdx.x * per;
  uint32_t c1[kPer], len[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int bidx = first + i;
    c1[i] = len[i] = 0;
    if (i < per && bidx < nb) {
      c1[i] = cnt1[bidx];
      if (in_off) {
        len[i] = (uint32_t)((bidx + 1 < nb ? (uint64_t)in_off[bidx + 1] : n) - in_off[bidx]);
      } else {
        uint64_t bb = (uint64_t)bidx * chunk, be = bb + chunk < n ? bb + chunk : n;
        if (bb > be) bb = be;
        len[i] = (uint32_t)(be - bb);
      }
    }
  }
  double2 acc = make_double2(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < kPer; ++i) acc = cadd(acc, pv[i]);
  const double2 P = block_sum(acc, shd);
  if (threadIdx.x == 0) {
    const double tot = P.x + P.y;
    int o = forced >= 0 ? forced : (u < P.x / tot ? 0 : 1);
    const double po = o ? P.y : P.x;
    double scale = 1.0 / sqrt(po);
    if (!(tot > 0.0) || !(po > 0.0)) {
      atomicOr(&ctl->error, 1u);
      o = -1;
      scale = 0.0;
    }
    rec->p0 = P.x;
    rec->p1 = P.y;
    rec->scale = scale;
    rec->outcome = o;
    *outcome = o;
    s_o = o;
  }
  __syncthreads();
  const int o = s_o;
  // Output counts per block for the chosen outcome, then exclusive scan.
  uint32_t kept_b[kPer];
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    kept_b[i] = o == 1 ? c1[i] : (o == 0 ? len[i] - c1[i] : 0u);
    s += kept_b[i];
  }
  // Inclusive scan of the per-thread counts: within each wave by shuffles,
  // then the preceding waves' totals.
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t incl = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(incl, d);
    if (lane >= d) incl += y;
  }
  if (lane == 63) shu[wid] = incl;
  __syncthreads();
  uint32_t kept_total = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
    if (w < wid) incl += shu[w];
    kept_total += shu[w];
  }
  uint32_t run = incl - s;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int bidx = first + i;
    if (i < per && bidx < nb) {
      off[bidx] = run;
      run += kept_b[i];
    }
  }
  if (threadIdx.x == blockDim.x - 1) {
    const uint64_t kept = kept_total;
    *nnz_out = kept;
    // reduce: the label word holding the qubit and the amplitude of every
    // entry (none when the previous write formed the sums)
    if (!in_off) ctl->pass_bytes[2] += n * 24u;
    // write: that label word of every entry, the rest of each kept entry, and the kept entries written
    ctl->pass_bytes[3] += n * 8u + kept * (2u * entry_bytes - 8u);
  }
}

// Ordered compaction of the entries with the measured outcome, scaled.  The
// block's input range is its uniform chunk, or (in_off given) the range the
// previous measurement's write block produced.  With q_next >= 0 the block
// also forms the next measurement's sums over the entries it writes, in the
// same form as the reduce kernel (its output range is then that
// measurement's input range for this block).
template <bool WIDE>
__global__ __launch_bounds__(256) void k_measure_write(Buf in, Buf out, const uint64_t* __restrict__ nnz_p,
                                                       uint32_t q, const MeasRec* __restrict__ rec,
                                                       const uint32_t* __restrict__ off,
                                                       const uint32_t* __restrict__ in_off, int32_t q_next,
                                                       double2* __restrict__ part_next,
                                                       uint32_t* __restrict__ cnt1_next) {
  __shared__ uint32_t s_wave[16];
  __shared__ double2 shd[256];
  __shared__ uint32_t shu[256];
  const uint64_t n = *nnz_p;
  uint64_t begin, end;
  if (in_off) {
    begin = in_off[blockIdx.x];
    end = blockIdx.x + 1 < gridDim.x ? in_off[blockIdx.x + 1] : n;
  } else {
    chunk_range(n, meas_chunk(n), begin, end);
  }
  const int o = rec->outcome;
  const double scale = rec->scale;
  uint64_t base = off[blockIdx.x];
  const bool qhi = WIDE && q >= 64;
  const bool nhi = WIDE && q_next >= 64;
  double p0 = 0.0, p1 = 0.0;
  uint32_t c1 = 0;
  for (uint64_t tile = begin; tile < end; tile += blockDim.x) {
    const uint64_t i = tile + threadIdx.x;
    bool keep = false;
    uint64_t lo = 0, hi = 0;
    if (i < end && o >= 0) {
      lo = in.key_lo[i];
      hi = WIDE ? in.key_hi[i] : 0ull;
      const uint64_t w = qhi ? hi : lo;
      keep = (int)((w >> (q & 63)) & 1ull) == o;
    }
    uint32_t tile_total;
    const uint64_t pos = base + block_prefix012(keep ? 1u : 0u, s_wave, &tile_total);
    if (keep) {
      const double2 a = in.amp[i];
      const double2 v = make_double2(a.x * scale, a.y * scale);
      out.key_lo[pos] = lo;
      if (WIDE) out.key_hi[pos] = hi;
      out.amp[pos] = v;
      if (q_next >= 0) {
        const double p = v.x * v.x + v.y * v.y;
        if ((((nhi ? hi : lo) >> (q_next & 63)) & 1ull) != 0) {
          p1 += p;
          ++c1;
        } else {
          p0 += p;
        }
      }
    }
    base += tile_total;
  }
  if (q_next >= 0) {
    const double2 sum = block_sum(make_double2(p0, p1), shd);
    const uint32_t c = block_sum(c1, shu);
    if (threadIdx.x == 0) {
      part_next[blockIdx.x] = sum;
      cnt1_next[blockIdx.x] = c;
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers.
void launch_set_basis(hipStream_t st, Buf b, uint64_t* nnz, uint64_t lo, uint64_t hi) {
  hipLaunchKernelGGL(k_set_basis, dim3(1), dim3(1), 0, st, b, nnz, lo, hi);
}

void launch_fill(hipStream_t st, uint64_t* p, uint64_t v, uint64_t n) {
  const uint64_t blocks = (n + 255) / 256;
  const int grid = (int)(blocks < 16384 ? (blocks ? blocks : 1) : 16384);
  hipLaunchKernelGGL(k_fill, dim3(grid), dim3(256), 0, st, p, v, n);
}

void launch_mono(hipStream_t st, bool wide, Buf b, const uint64_t* nnz, const MonoDesc* g, uint32_t ng,
                 uint32_t run_flags, uint32_t bytes_per_entry, Ctl* ctl, int grid, int block) {
  if (wide)
    hipLaunchKernelGGL((k_mono<true, 4>), dim3(grid), dim3(block), 0, st, b, nnz, g, ng, run_flags, bytes_per_entry,
                       ctl);
  else
    hipLaunchKernelGGL((k_mono<false, 4>), dim3(grid), dim3(block), 0, st, b, nnz, g, ng, run_flags, bytes_per_entry,
                       ctl);
}

void launch_index_build(hipStream_t st, bool wide, Buf b, const uint64_t* nnz, const IndexTab& t, const U2Desc& d,
                        bool counting, const MonoRun& m, Ctl* ctl, uint64_t ub) {
  auto* count = counting ? reinterpret_cast<unsigned long long*>(&ctl->ix[0]) : nullptr;
  const int grid = (int)std::max<uint64_t>(1, std::min<uint64_t>((ub + 255) / 256, 4096));
#define SPARSESIM_BUILD(W, M)                                                                                  \
  hipLaunchKernelGGL((k_index_build<W, M>), dim3(grid), dim3(256), 0, st, b, nnz, t, d, count, m.g, m.ng, \
                     m.run_flags, ctl)
  if (wide) {
    if (m.ng) SPARSESIM_BUILD(true, true);
    else SPARSESIM_BUILD(true, false);
  } else {
    if (m.ng) SPARSESIM_BUILD(false, true);
    else SPARSESIM_BUILD(false, false);
  }
#undef SPARSESIM_BUILD
}

void launch_u2_probe(hipStream_t st, bool wide, Buf b, const uint64_t* nnz, const IndexTab& t, const U2Desc& d,
                     uint32_t* partner, uint32_t epoch, bool counting, Ctl* ctl, uint64_t ub) {
  auto* count = counting ? reinterpret_cast<unsigned long long*>(&ctl->ix[2]) : nullptr;
  // Two blocks a CU, whatever the bound: blocks that find no entries cost their launch.
  const int block = ub <= 1ull << 16 ? 256 : 1024;
  const int grid = (int)std::max<uint64_t>(1, std::min<uint64_t>((ub + block - 1) / block, 512));
  if (wide)
    hipLaunchKernelGGL(k_u2_probe<true>, dim3(grid), dim3(block), 0, st, b, nnz, t, d, partner, epoch, count);
  else
    hipLaunchKernelGGL(k_u2_probe<false>, dim3(grid), dim3(block), 0, st, b, nnz, t, d, partner, epoch, count);
}

void launch_import_check(hipStream_t st, bool wide, Buf b, uint64_t n, const IndexTab& t, uint64_t* nnz_out) {
  const int grid = (int)std::max<uint64_t>(1, std::min<uint64_t>((n + 255) / 256, 2048));
  if (wide) hipLaunchKernelGGL(k_import_check<true>, dim3(grid), dim3(256), 0, st, b, n, t, nnz_out);
  else hipLaunchKernelGGL(k_import_check<false>, dim3(grid), dim3(256), 0, st, b, n, t, nnz_out);
}

void launch_index_empty(hipStream_t st, const IndexTab& t) {
  hipLaunchKernelGGL(k_index_empty, dim3(1024), dim3(256), 0, st, t);
}

void launch_u2_count(hipStream_t st, bool wide, Buf b, const uint64_t* nnz, const U2Desc& d, const uint32_t* partner,
                     uint32_t epoch, uint32_t* tot, Ctl* ctl, int grid, int block) {
  if (wide)
    hipLaunchKernelGGL(k_u2_count<true>, dim3(grid), dim3(block), 0, st, b, nnz, d, partner, epoch, tot, ctl);
  else
    hipLaunchKernelGGL(k_u2_count<false>, dim3(grid), dim3(block), 0, st, b, nnz, d, partner, epoch, tot, ctl);
}

void launch_scan(hipStream_t st, uint32_t* tot, int nblocks, uint64_t* nnz_out, Ctl* ctl, uint32_t entry_bytes,
                 uint64_t cap) {
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, st, tot, nblocks, nnz_out, ctl, entry_bytes, cap);
}

void launch_u2_write(hipStream_t st, bool wide, Buf in, Buf out, const uint64_t* nnz, const uint32_t* partner,
                     uint32_t epoch, const uint32_t* off, const U2Desc& d, Ctl* ctl, int grid, int block) {
  if (wide)
    hipLaunchKernelGGL(k_u2_write<true>, dim3(grid), dim3(block), 0, st, in, out, nnz, partner, epoch, off, d, ctl);
  else
    hipLaunchKernelGGL(k_u2_write<false>, dim3(grid), dim3(block), 0, st, in, out, nnz, partner, epoch, off, d, ctl);
}

void launch_u2_fused(hipStream_t st, bool wide, Buf in, Buf out, const uint64_t* nnz, const uint32_t* partner,
                     const U2Desc& d, Ctl* ctl, const TabCtl* tc, uint64_t* status, uint32_t par, uint32_t epoch,
                     uint64_t* nnz_out, uint64_t cap, uint32_t seq, const NextGate& next, uint64_t ub) {
  // A block fills a CU (16 waves of up to 128 registers): more would only wait for a place.
  const int grid = (int)std::max<uint64_t>(1, std::min<uint64_t>((ub + 255) / 256, 256));
#define SPARSESIM_U2F(W, N)                                                                                       \
  hipLaunchKernelGGL((k_u2_fused<W, N>), dim3(grid), dim3(kU2Threads), 0, st, in, out, nnz, partner, d, ctl, tc, \
                     status, par, epoch, nnz_out, cap, seq, next)
  if (wide) {
    if (next.tab.slots) SPARSESIM_U2F(true, true);
    else SPARSESIM_U2F(true, false);
  } else {
    if (next.tab.slots) SPARSESIM_U2F(false, true);
    else SPARSESIM_U2F(false, false);
  }
#undef SPARSESIM_U2F
}

void launch_u2_restore(hipStream_t st, Ctl* ctl, int cur) {
  hipLaunchKernelGGL(k_u2_restore, dim3(1), dim3(1), 0, st, ctl, cur);
}

void launch_u2_tickets(hipStream_t st, Ctl* ctl) { hipLaunchKernelGGL(k_u2_tickets, dim3(1), dim3(1), 0, st, ctl); }

void launch_u2_chain(hipStream_t st, bool wide, Buf in, Buf out, uint64_t* nnz, int cur, const Chain& chain,
                     Ctl* ctl) {
  if (wide)
    hipLaunchKernelGGL(k_u2_chain<true>, dim3(1), dim3(lds::kThreads), 0, st, in, out, nnz, cur, chain, ctl);
  else
    hipLaunchKernelGGL(k_u2_chain<false>, dim3(1), dim3(lds::kThreads), 0, st, in, out, nnz, cur, chain, ctl);
}

void launch_u2_lds_tiles(hipStream_t st, bool wide, Buf in, Buf out, const uint64_t* nnz_in, uint64_t* nnz_out,
                         const U2Desc& d, const MonoRun& m, uint64_t* status, uint32_t par, uint32_t epoch, Ctl* ctl,
                         uint64_t ub) {
  const int grid = (int)std::max<uint64_t>(1, (ub + 1023) / 1024);
  if (wide)
    hipLaunchKernelGGL(k_u2_lds_tiles<true>, dim3(grid), dim3(1024), 0, st, in, out, nnz_in, nnz_out, d, m, status,
                       par, epoch, ctl);
  else
    hipLaunchKernelGGL(k_u2_lds_tiles<false>, dim3(grid), dim3(1024), 0, st, in, out, nnz_in, nnz_out, d, m, status,
                       par, epoch, ctl);
}

void launch_measure_reduce(hipStream_t st, bool wide, Buf b, const uint64_t* nnz, uint32_t q, BlockScratch s,
                           int grid, int block) {
  if (wide)
    hipLaunchKernelGGL(k_measure_reduce<true>, dim3(grid), dim3(block), 0, st, b, nnz, q, s.part, s.cnt1);
  else
    hipLaunchKernelGGL(k_measure_reduce<false>, dim3(grid), dim3(block), 0, st, b, nnz, q, s.part, s.cnt1);
}

void launch_measure_decide(hipStream_t st, const double2* part, const uint32_t* cnt1, uint32_t* off, int nblocks,
                           const uint64_t* nnz_in, uint64_t* nnz_out, double u, int32_t forced, MeasRec* rec,
                           int32_t* outcome, Ctl* ctl, uint32_t entry_bytes, const uint32_t* in_off) {
  hipLaunchKernelGGL(k_measure_decide, dim3(1), dim3(1024), 0, st, part, cnt1, off, nblocks, nnz_in, nnz_out, u,
                     forced, rec, outcome, ctl, entry_bytes, in_off);
}

void launch_measure_write(hipStream_t st, bool wide, Buf in, Buf out, const uint64_t* nnz, uint32_t q,
                          const MeasRec* rec, const uint32_t* off, const uint32_t* in_off, int32_t q_next,
                          double2* part_next, uint32_t* cnt1_next, int grid) {
  if (wide)
    hipLaunchKernelGGL(k_measure_write<true>, dim3(grid), dim3(256), 0, st, in, out, nnz, q, rec, off, in_off, q_next,
                       part_next, cnt1_next);
  else
    hipLaunchKernelGGL(k_measure_write<false>, dim3(grid), dim3(256), 0, st, in, out, nnz, q, rec, off, in_off,
                       q_next, part_next, cnt1_next);
}

}  // namespace sparsesim

// ---------------------------------------------------------------------------
// Plain streaming copy (bandwidth reference for hardware byte counters).
namespace sparsesim {
namespace {
__global__ __launch_bounds__(256) void k_copy16(uint4* __restrict__ dst, const uint4* __restrict__ src, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}
}  // namespace

void launch_copy16(hipStream_t st, void* dst, const void* src, uint64_t n16) {
  hipLaunchKernelGGL(k_copy16, dim3(8192), dim3(256), 0, st, static_cast<uint4*>(dst), static_cast<const uint4*>(src),
                     n16);
}
}  // namespace sparsesim
