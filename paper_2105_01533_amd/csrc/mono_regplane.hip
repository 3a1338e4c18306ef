// Register-plane fused phase/permutation pass for gfx950 (Sec. 3.2): the
// label bit-planes of a 2048-entry tile stay in VGPRs for the whole run and
// gates address them by index through the GPR indexing mode (see
// regplane_tile.h).  Phases accumulate exactly, as in the bit-sliced form:
// eighth turns in bit-sliced counters, other angles as 64-bit turn fractions,
// one complex multiply per amplitude at the end of the run.
#include <mutex>

#include "batch_units.h"
#include "regplane_tile.h"

namespace sparsesim {
namespace {

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// The empty asm statement names the highest plane register (rp::kVmax) as
// clobbered, which makes the kernel's VGPR count reach it; the compiler
// itself is held below v80 (amdgpu_num_vgpr), so it never allocates a
// reserved register.
template <bool TURNS>
__global__ __launch_bounds__(64, 2) __attribute__((amdgpu_num_vgpr(40))) void k_mono_rp(
    Buf b, const uint64_t* __restrict__ nnz_p, const RpBlock* __restrict__ prog, uint32_t nblk, BsRun run,
    Ctl* ctl) {
  static_assert(rp::kVmax == 230, "the clobber below names the highest plane register");
  asm volatile("" ::: "v230");
  extern __shared__ uint64_t rp_acc[];
  __shared__ uint64_t s_table[256];   // the subset sums of eight turn fractions
  const uint64_t n = *nnz_p;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    atomicAdd((unsigned long long*)&ctl->updates, (unsigned long long)(n * run.n_gates));
    atomicAdd((unsigned long long*)&ctl->mono_updates, (unsigned long long)(n * run.n_gates));
    atomicAdd((unsigned long long*)&ctl->mono_bytes, (unsigned long long)(n * run.bytes_per_entry));
  }
  // One tile per block (the grid covers the largest entry count the host
  // allows for; blocks past the live count do nothing).
  const uint64_t base = (uint64_t)blockIdx.x * 2048;
  if (base >= n) return;
  const uint32_t lim = (uint32_t)(n - base < 2048 ? n - base : 2048);
  rp::rp_tile<TURNS>([&] { return rp::RpArgs{b, run}; }, base, lim, prog, nblk, blockIdx.x < 64, rp_acc,
                     s_table);   // (eight waves an XCD)
}

// The fused runs of a batched tick: unit u is a tile of the state of item
// find_item(u), with that item's program.  Waves of different programs must
// not share a SIMD (see launch_mono_rp): the AGPRs named here make the wave's
// share of the registers more than half of a SIMD's, so that one fits (the build
// fails if it is not: check_regplane_alloc).  The
// tick's fused runs were the latency of the LDS-plane tile, 70 ns a gate; the
// register planes take 26 (2048 entries, 24 qubits): 45 us a tick of 24 requests
// instead of 135.
__global__ __launch_bounds__(64, 1) __attribute__((amdgpu_num_vgpr(40))) void kb_mono_rp(
    const BTick* __restrict__ hdr, const BItem* __restrict__ items, const uint32_t* __restrict__ units) {
  asm volatile("" ::: "v230");
  asm volatile("" ::: "a63");
  extern __shared__ uint64_t rp_acc[];
  __shared__ uint64_t s_table[256];
  const int n = (int)hdr->n_rp;
  if (n == 0) return;
  const BItem* rp = items + hdr->n_mono + hdr->n_u2 + hdr->n_meas + hdr->n_u2s;
  const uint32_t* u0 = units + hdr->rp_u0;
  const uint32_t u = blockIdx.x;   // a tile a block
  if (u >= u0[n]) return;
  const int i = __builtin_amdgcn_readfirstlane(find_item(u0, n, u));
  // The item by scalar loads, anew for each `item()` (see RpArgs).
  uint64_t at = reinterpret_cast<uint64_t>(rp + i);
  auto item = [&] {
    asm volatile("" : "+s"(at));
    return (const __attribute__((address_space(4))) BItem*)at;
  };
  auto get = [&] {
    const auto* p = item();
    rp::RpArgs r;
    r.b.key_lo = p->in.key_lo;
    r.b.key_hi = p->in.key_hi;
    r.b.amp = p->in.amp;
    r.run.n_planes = p->run.n_planes;
    r.run.words_read = p->run.words_read;
    r.run.words_write = p->run.words_write;
    r.run.has_phase = p->run.has_phase;
    r.run.has_turns = p->run.has_turns;
    r.run.g_omega = p->run.g_omega;
    r.run.g_turn = p->run.g_turn;
    return r;
  };
  const auto* p = item();
  const uint32_t tile = u - u0[i];
  const uint64_t base = (uint64_t)tile * 2048, nnz = p->nnz;
  const uint32_t lim = (uint32_t)(nnz - base < 2048 ? nnz - base : 2048);
  rp::rp_tile<true>(get, base, lim, p->prog, p->ngroups, tile < 8, rp_acc, s_table);   // (a wave an XCD)
}
#pragma clang diagnostic pop

}  // namespace

namespace {

// Register-plane passes of this process never run at the same time on one
// device: waves of two passes with different programs sharing a SIMD gave
// results that depended on the pairing (the GPR-indexed plane accesses),
// while waves of one pass -- one program -- reproduce the LDS-plane pass bit
// for bit.  Each launch records an event on its stream; a launch from another
// stream first waits for it.  (Skipped on a stream under graph capture, where
// the ordering is the graph's.)  The event is made once per device, at
// set-up, so launches allocate nothing.
struct RpOrder {
  std::mutex mu;
  hipEvent_t ev = nullptr;
  hipStream_t last = nullptr;
};

RpOrder& rp_order() {
  static RpOrder orders[64];
  int dev = 0;
  (void)hipGetDevice(&dev);
  return orders[dev & 63];
}

}  // namespace

hipError_t mono_rp_init() {
  RpOrder& o = rp_order();
  std::lock_guard<std::mutex> lk(o.mu);
  if (o.ev) return hipSuccess;
  return hipEventCreateWithFlags(&o.ev, hipEventDisableTiming);
}

namespace {

template <class Launch>
void in_order(hipStream_t st, Launch&& launch) {
  RpOrder& o = rp_order();
  std::lock_guard<std::mutex> lk(o.mu);
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  (void)hipStreamIsCapturing(st, &cs);
  const bool ordered = cs == hipStreamCaptureStatusNone;
  if (ordered && o.ev && o.last != st) (void)hipStreamWaitEvent(st, o.ev, 0);
  launch();
  if (ordered && o.ev && hipEventRecord(o.ev, st) == hipSuccess) o.last = st;
}

}  // namespace

void launch_mono_rp(hipStream_t st, Buf b, const uint64_t* nnz, const RpBlock* p, uint32_t nblk, const BsRun& run,
                    Ctl* ctl, int grid) {
  in_order(st, [&] {
    if (run.has_turns)
      hipLaunchKernelGGL(k_mono_rp<true>, dim3(grid), dim3(64), rp::kTurnAccBytes, st, b, nnz, p, nblk, run, ctl);
    else
      hipLaunchKernelGGL(k_mono_rp<false>, dim3(grid), dim3(64), 0, st, b, nnz, p, nblk, run, ctl);
  });
}

void launch_batch_mono_rp(hipStream_t st, const BTick* hdr, const BItem* items, const uint32_t* units, uint32_t tiles) {
  in_order(st, [&] { hipLaunchKernelGGL(kb_mono_rp, dim3(tiles), dim3(64), rp::kTurnAccBytes, st, hdr, items, units); });
}

}  // namespace sparsesim
