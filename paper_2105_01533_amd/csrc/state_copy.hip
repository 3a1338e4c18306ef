// Copy of a device state (structure of arrays) to host records, shared by
// state export (sim_export_state) and the server's result copies, and of host
// records to a device state (sim_import_state).
//
// A device-to-host copy into pageable memory goes through the runtime's own
// staging and serialises across host threads; here each call borrows a pinned
// staging buffer, copies a chunk of the state into it at DMA speed and
// interleaves the chunk into the caller's (lo, hi) key records and amplitudes.
// Several threads can do this at once (the server copies the states of
// several finished requests in parallel).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

#include "host_pool.h"
#include "sim_internal.h"

namespace sparsesim {

namespace {

constexpr size_t kStageBytes = 16u << 20;
// Staging buffers kept when no copy uses them (as many as the host pool has
// threads; beyond, a buffer lasts one call).  An allocation takes longer than
// most copies.
constexpr size_t kStagesKept = HostPool::kMaxThreads;

struct StagePool {
  std::mutex mu;
  std::vector<char*> free;
  StagePool() { free.reserve(kStagesKept); }
  static StagePool& get() {
    static auto* pool = new StagePool;   // (never destroyed: copies may run until the process ends)
    return *pool;
  }
};

}  // namespace

hipError_t CopyStage::take() {
  StagePool& pool = StagePool::get();
  {
    std::lock_guard<std::mutex> lk(pool.mu);
    if (!pool.free.empty()) {
      p = pool.free.back();
      pool.free.pop_back();
      return hipSuccess;
    }
  }
  void* m = nullptr;
  const hipError_t e = hipHostMalloc(&m, kStageBytes, hipHostMallocDefault);
  if (e == hipSuccess) p = static_cast<char*>(m);
  return e;
}

CopyStage::~CopyStage() {
  if (!p) return;
  if (in_flight) (void)hipStreamSynchronize(st);
  StagePool& pool = StagePool::get();
  {
    std::lock_guard<std::mutex> lk(pool.mu);
    if (pool.free.size() < kStagesKept) {
      pool.free.push_back(p);
      return;
    }
  }
  (void)hipHostFree(p);
}

namespace {

// Chunks of the state through the staging buffer; emit(b, m, s_lo, s_hi,
// s_amp, pb, pe) writes entries [pb, pe) of the chunk that starts at entry b.
template <class Emit>
hipError_t staged_copy(const uint64_t* lo, const uint64_t* hi, const double2* amp, uint64_t n, hipStream_t st,
                       size_t part, Emit&& emit) {
  if (!n) return hipSuccess;
  CopyStage own(st);
  hipError_t e = own.take();
  if (e != hipSuccess) return e;
  char* const stage = own.p;
  const size_t per_entry = hi ? 32 : 24;
  const uint64_t chunk = kStageBytes / per_entry;
  for (uint64_t b = 0; b < n; b += chunk) {
    const uint64_t m = std::min<uint64_t>(chunk, n - b);
    auto* s_lo = reinterpret_cast<const uint64_t*>(stage);
    auto* s_hi = reinterpret_cast<const uint64_t*>(stage + 8 * m);
    auto* s_amp = reinterpret_cast<const double2*>(stage + (hi ? 16 : 8) * m);
    e = hipMemcpyAsync(stage, lo + b, 8 * m, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && hi) e = hipMemcpyAsync(stage + 8 * m, hi + b, 8 * m, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipMemcpyAsync(const_cast<double2*>(s_amp), amp + b, 16 * m, hipMemcpyDeviceToHost, st);
    const hipError_t done = hipStreamSynchronize(st);   // (also after an error: the stage is used again)
    if (e == hipSuccess) e = done;
    if (e != hipSuccess) return e;
    // On the host thread pool (on this thread alone when it is itself one of
    // the pool's tasks).
    parallel_parts(m, part, [&](size_t pb, size_t pe, size_t) { emit(b, s_lo, hi ? s_hi : nullptr, s_amp, pb, pe); });
  }
  return hipSuccess;
}

}  // namespace

hipError_t copy_state_to_host(const uint64_t* lo, const uint64_t* hi, const double2* amp, uint64_t n, sim_key* keys,
                              sim_c64* amps, hipStream_t st) {
  return staged_copy(lo, hi, amp, n, st, kCopyPart,
                     [&](uint64_t b, const uint64_t* s_lo, const uint64_t* s_hi, const double2* s_amp, size_t pb, size_t pe) {
                       for (size_t k = pb; k < pe; ++k) keys[b + k] = sim_key{s_lo[k], s_hi ? s_hi[k] : 0};
                       std::memcpy(amps + b + pb, s_amp + pb, 16 * (pe - pb));
                     });
}

hipError_t copy_state_to_host_soa(const uint64_t* lo, const uint64_t* hi, const double2* amp, uint64_t n,
                                  uint64_t* key_lo, uint64_t* key_hi, sim_c64* amps, hipStream_t st,
                                  size_t part) {
  return staged_copy(lo, hi, amp, n, st, part,
                     [&](uint64_t b, const uint64_t* s_lo, const uint64_t* s_hi, const double2* s_amp, size_t pb, size_t pe) {
                       std::memcpy(key_lo + b + pb, s_lo + pb, 8 * (pe - pb));
                       if (key_hi) {
                         if (s_hi) std::memcpy(key_hi + b + pb, s_hi + pb, 8 * (pe - pb));
                         else std::memset(key_hi + b + pb, 0, 8 * (pe - pb));
                       }
                       std::memcpy(amps + b + pb, s_amp + pb, 16 * (pe - pb));
                     });
}

hipError_t copy_state_to_device(const uint64_t* lo, const uint64_t* hi, size_t stride, const sim_c64* amps, uint64_t n,
                                uint64_t out_lo, uint64_t out_hi, Buf b, bool wide, CopyStage& own, LabelCell* seen) {
  *seen = LabelCell{~0ull, ~0ull, 0, 0};
  if (!n) return hipSuccess;
  hipError_t e = own.take();
  if (e != hipSuccess) return e;
  char* const stage = own.p;
  const hipStream_t st = own.st;
  const size_t per_entry = wide ? 32 : 24;
  const uint64_t chunk = kStageBytes / per_entry;
  for (uint64_t c = 0; c < n; c += chunk) {
    const uint64_t m = std::min<uint64_t>(chunk, n - c);
    auto* s_lo = reinterpret_cast<uint64_t*>(stage);
    auto* s_hi = reinterpret_cast<uint64_t*>(stage + 8 * m);
    char* s_amp = stage + (wide ? 16 : 8) * m;
    LabelCell part[HostPool::kMaxThreads];
    for (LabelCell& p : part) p = LabelCell{~0ull, ~0ull, 0, 0};
    parallel_parts(m, kCopyPart, [&](size_t pb, size_t pe, size_t t) {
      LabelCell v{~0ull, ~0ull, 0, 0};
      for (size_t k = pb; k < pe; ++k) {
        const sim_key q{lo[(c + k) * stride], hi ? hi[(c + k) * stride] : 0};
        v.and_lo &= q.lo;
        v.and_hi &= q.hi;
        v.or_lo |= q.lo;
        v.or_hi |= q.hi;
        s_lo[k] = q.lo;
        if (wide) s_hi[k] = q.hi;
      }
      std::memcpy(s_amp + 16 * pb, amps + c + pb, 16 * (pe - pb));
      part[t] = v;
    });
    for (const LabelCell& p : part) {
      seen->and_lo &= p.and_lo;
      seen->and_hi &= p.and_hi;
      seen->or_lo |= p.or_lo;
      seen->or_hi |= p.or_hi;
    }
    if ((seen->or_lo & out_lo) || (seen->or_hi & out_hi)) return hipSuccess;
    own.in_flight = true;
    e = hipMemcpyAsync(b.key_lo + c, s_lo, 8 * m, hipMemcpyHostToDevice, st);
    if (e == hipSuccess && wide) e = hipMemcpyAsync(b.key_hi + c, s_hi, 8 * m, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(b.amp + c, s_amp, 16 * m, hipMemcpyHostToDevice, st);
    // The stage is used again by the next chunk; after the last one the caller waits.
    const hipError_t done = c + m < n || e != hipSuccess ? hipStreamSynchronize(st) : hipSuccess;
    if (e == hipSuccess) e = done;
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace sparsesim
