// Host check of the blocks the register-plane kernel reads
// (RunCompiler::encode_program): random programs of segments, as the scheduler
// writes them, are packed into blocks and both are run on random bit planes --
// the segments by their definition, the blocks slot by slot from where their
// headers say the handlers start -- and must agree.  Built and run by
// test_rp_blocks.py; prints "OK" on success.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../paper_2105_01533_amd/csrc/run_compiler.h"

using namespace sparsesim;

namespace {

uint64_t sm_state;
uint64_t next_u64() {
  uint64_t z = (sm_state += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
uint32_t below(uint32_t n) { return (uint32_t)(next_u64() % n); }

// One 32-entry word per register: v80.. = accumulators P, Q0, Q1, R0..R2,
// v100 + q = plane q, as the kernel numbers them from v80.
struct Machine {
  uint32_t v[256] = {};
  std::vector<uint32_t> log;   // the data words of general eighth-turn segments, in order
  uint64_t turns[32] = {};     // per entry
  void turn(uint32_t x, uint64_t tau) {
    for (int j = 0; j < 32; ++j)
      if ((x >> j) & 1u) turns[j] += tau;
  }
  void t(uint32_t x) {         // weight-1 add
    const uint32_t c = v[3] & x;
    v[3] ^= x;
    v[5] ^= v[4] & c;
    v[4] ^= c;
  }
  void s(uint32_t x) {         // weight-2 add
    v[2] ^= v[1] & x;
    v[1] ^= x;
  }
};

void run_segments(Machine& m, const std::vector<RpRec>& p, uint32_t nq) {
  auto plane = [&](uint32_t q) -> uint32_t& { return m.v[kRpPlane0 + (q & 0xff)]; };
  for (size_t pc = 0; pc < p.size();) {
    const uint32_t sh = p[pc].w[0] & 0xff, cnt = p[pc].w[0] >> 8;
    const size_t len = sh == kRpTB || sh == kRpTG ? 3 * (size_t)cnt : cnt;
    if (sh == kRpTB || sh == kRpTG) {
      for (uint32_t i = 0; i < 4 * cnt; ++i) {
        const RpRec* g = &p[pc + 1 + 3 * (i / 4)];
        const uint32_t w = g[0].w[i % 4];
        uint64_t tau;
        std::memcpy(&tau, &g[1 + (i % 4) / 2].w[2 * (i % 2)], 8);
        m.turn(sh == kRpTB ? plane(w) : plane(w) & plane(w >> 8) & plane(w >> 16) & plane(w >> 24), tau);
      }
      pc += 1 + len;
      continue;
    }
    for (size_t r = 0; r < len; ++r)
      for (int u = 0; u < 4; ++u) {
        const uint32_t w = p[pc + 1 + r].w[u];
        if (sh >= kRpF1 && sh <= kRpF3) {
          uint32_t c = ~0u;
          for (uint32_t k = 1; k <= sh; ++k) c &= plane(w >> (8 * k));
          if ((w & 0xff) != nq + 1) plane(w) ^= c;
        } else if (sh > kRpOB) {
          const uint32_t k = sh - kRpOB, x = plane(w);
          if (k & 1) m.t(x);
          if (k & 2) m.s(x);
          if (k & 4) m.v[0] ^= x;
        } else {
          m.log.push_back(w);
        }
      }
    pc += 1 + len;
  }
}

bool run_blocks(Machine& m, const std::vector<RpBlock>& p, uint32_t nq) {
  auto plane = [&](uint32_t q) -> uint32_t& { return m.v[kRpPlane0 + (q & 0xff)]; };
  static const uint32_t slots[6] = {0, 15, 10, 7, 7, 15}, code[6] = {0, 16, 24, 32, 88, 16};
  for (size_t pc = 0; pc < p.size();) {
    const RpBlock& b = p[pc++];
    const uint32_t sh = b.w[0] / kRpStride, off = b.w[0] % kRpStride;
    auto half = [&](uint32_t h) { return (b.w[h / 2] >> (16 * (h & 1))) & 0xffffu; };
    auto src = [&](uint32_t f) -> uint32_t { return m.v[f & 0xff]; };
    if (sh == kBlkExit) {
      if (off) return false;
      if (b.w[1] == kRpEnd) return pc == p.size();
      if (b.w[1] == kRpOG) {
        for (uint32_t i = 0; i < 4 * b.w[2]; ++i) m.log.push_back(p[pc + i / 16].w[i % 16]);
        pc += (b.w[2] + 3) / 4;
        continue;
      }
      if (b.w[1] == kRpTC && 8 * b.w[2] > rp_capture_planes(nq)) return false;
      for (uint32_t g = 0; g < b.w[2]; ++g, ++pc)
        for (uint32_t u = 0; u < (b.w[1] == kRpTC ? 8u : 4u); ++u) {
          uint64_t tau;
          std::memcpy(&tau, &p[pc].w[b.w[1] == kRpTC ? 2 * u : 4 + 2 * u], 8);
          const uint32_t w = p[pc].w[u];
          if (b.w[1] == kRpTC) {
            m.turn(plane(nq + 3 + 8 * g + u), tau);
            plane(nq + 3 + 8 * g + u) = 0;
          } else {
            m.turn(b.w[1] == kRpTB ? plane(w) : plane(w) & plane(w >> 8) & plane(w >> 16) & plane(w >> 24), tau);
          }
        }
      continue;
    }
    if (sh > kBlkS || off % code[sh] || off / code[sh] >= slots[sh]) return false;
    for (uint32_t j = off / code[sh]; j < slots[sh]; ++j) {
      if (sh <= kBlkF3) {
        const uint32_t h = (sh == kBlkF3 ? 4 : 2) + (sh + 1) * j;
        uint32_t c = ~0u;
        for (uint32_t k = 0; k < sh; ++k) {
          if ((half(h + k) & 0xf000) != kRpSrc) return false;
          c &= src(half(h + k));
        }
        if ((half(h + sh) & 0xf000) != kRpSrcDst) return false;
        m.v[half(h + sh) & 0xff] ^= c;
      } else if (sh == kBlkT) {
        for (uint32_t k = 0; k < 4; ++k) m.t(src(half(4 + 4 * j + k)));
      } else {
        m.s(src(b.w[1 + j]));
      }
    }
  }
  return false;   // no END
}

}  // namespace

int main(int argc, char** argv) {
  const int cases = argc > 1 ? atoi(argv[1]) : 300;
  const uint32_t nqs[] = {3, 24, 64, 100, 115, 122, 128};
  for (int c = 0; c < cases; ++c) {
    sm_state = 0xB10Cull * (c + 1);
    const uint32_t nq = nqs[c % 7], scratch = nq + 1, zero = nq + 2;
    const uint32_t pad = scratch | zero << 8 | zero << 16 | zero << 24;
    std::vector<RpRec> p;
    const uint32_t segs = below(60);
    for (uint32_t s = 0; s < segs; ++s) {
      const uint32_t kinds[] = {kRpF1, kRpF2, kRpF3, kRpF1, kRpF2, kRpOG, kRpTB, kRpTG, kRpOB};
      uint32_t sh = kinds[below(9)];
      if (sh == kRpOB) sh += 1 + below(7);
      const uint32_t n = 1 + below(below(4) ? 9 : 90);   // ops (groups for turns)
      const bool turn = sh == kRpTB || sh == kRpTG;
      const uint32_t recs = turn ? n : sh == kRpOG ? (n + 1) / 2 : (n + 3) / 4;
      p.push_back(RpRec{{sh | recs << 8, 0, 0, 0}});
      for (uint32_t r = 0; r < (turn ? 3 * recs : recs); ++r) {
        RpRec q;
        for (uint32_t u = 0; u < 4; ++u) {
          if (sh >= kRpF1 && sh <= kRpF3) {
            uint32_t f[4];   // target and controls, all different; unused controls all-ones
            for (int k = 0; k < 4; ++k) {
              f[k] = below(nq);
              for (int l = 0; l < k; ++l)
                if (f[l] == f[k]) f[k] = nq;
              if (k > (int)sh) f[k] = nq;
            }
            q.w[u] = 4 * r + u < n ? f[0] | f[1] << 8 | f[2] << 16 | f[3] << 24 : pad;
          } else if (sh > kRpOB) {
            q.w[u] = 4 * r + u < n ? below(nq) : zero;
          } else {
            q.w[u] = (uint32_t)next_u64();
          }
        }
        if (turn && r % 3 == 0) {   // cond words of a group
          for (uint32_t u = 0; u < 4; ++u) {
            const uint32_t k = sh == kRpTB ? 1 : 1 + below(4);
            uint32_t f[4] = {nq, nq, nq, nq};
            for (uint32_t i = 0; i < k && i < nq; ++i) f[i] = (7 * i + below(nq / 4 + 1)) % nq;
            q.w[u] = sh == kRpTB ? f[0] : f[0] | f[1] << 8 | f[2] << 16 | f[3] << 24;
            if (r + 3 >= 3 * recs && u > 1) q.w[u] = zero | zero << 8 | zero << 16 | zero << 24;   // padding
          }
        }
        p.push_back(q);
      }
    }
    std::vector<RpBlock> blocks;
    RunCompiler::encode_program(p, nq, blocks);
    Machine a;
    for (uint32_t q = 0; q < nq; ++q) a.v[kRpPlane0 + q] = (uint32_t)next_u64();
    a.v[kRpPlane0 + nq] = ~0u;
    Machine b = a;
    run_segments(a, p, nq);
    if (!run_blocks(b, blocks, nq)) return printf("case %d: malformed block\n", c), 1;
    if (std::memcmp(a.v, b.v, sizeof a.v) || std::memcmp(a.turns, b.turns, sizeof a.turns) || a.log != b.log) return printf("case %d: results differ\n", c), 1;
  }
  printf("OK cases=%d\n", cases);
  return 0;
}
