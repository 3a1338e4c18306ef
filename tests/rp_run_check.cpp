// Host check of a run's register-plane program as the engines build it
// (RunCompiler::compile and program: the run cut into parts, each scheduled and
// packed by itself, one END block): random gate lists are compiled with parts
// of a few ops, the blocks run on random bit planes, and the result must be
// that of the run's bit-sliced ops one by one; and no program may take more
// blocks than rp_blocks_bound, by which the server sizes its runs.  Built and
// run by test_rp_run.py; prints "OK" on success.
#define main rp_block_check_main
#include "rp_block_check.cpp"
#undef main

#include <algorithm>
#include <cmath>

namespace {

// The eighths and turns an entry has gained.
uint32_t eighths(const Machine& m, int j) {
  auto bit = [&](int r) { return (m.v[r] >> j) & 1u; };
  return (bit(3) + 2 * bit(4) + 4 * bit(5) + 2 * (bit(1) + 2 * bit(2)) + 4 * bit(0)) & 7u;
}

// The whole program: general eighth-turn segments here, the rest block by block.
bool run_program(Machine& m, const std::vector<RpBlock>& p, uint32_t nq) {
  auto plane = [&](uint32_t q) { return m.v[kRpPlane0 + (q & 0xff)]; };
  const RpBlock end{};
  for (size_t pc = 0; pc < p.size();) {
    const RpBlock& b = p[pc];
    const bool exit = b.w[0] == kBlkExit * kRpStride;
    if (exit && b.w[1] == kRpEnd) return pc + 1 == p.size();
    const size_t data = !exit ? 0 : b.w[1] == kRpOG ? (b.w[2] + 3) / 4 : b.w[2];
    if (pc + 1 + data >= p.size()) return false;
    if (exit && b.w[1] == kRpOG) {
      for (uint32_t i = 0; i < 2 * b.w[2]; ++i) {
        const uint32_t* w = &p[pc + 1 + i / 8].w[2 * (i % 8)];
        const uint32_t x = plane(w[0]) & plane(w[0] >> 8) & plane(w[0] >> 16) & plane(w[0] >> 24);
        if (w[1] & 1) m.t(x);
        if (w[1] & 2) m.s(x);
        if (w[1] & 4) m.v[0] ^= x;
      }
    } else {
      std::vector<RpBlock> one(p.begin() + (long)pc, p.begin() + (long)(pc + 1 + data));
      one.push_back(end);
      if (!run_blocks(m, one, nq)) return false;
    }
    pc += 1 + data;
  }
  return false;
}

sim_gate random_gate(uint32_t nq, uint32_t kind, uint32_t nc) {
  sim_gate g{};
  g.op = SIM_OP_MONO;
  g.forced = -1;
  g.target = below(nq);
  for (uint32_t k = 0; k < nc;) {
    const uint32_t q = below(nq);
    uint64_t& w = q < 64 ? g.ctrl.lo : g.ctrl.hi;
    if (q == g.target || ((w >> (q & 63)) & 1ull)) continue;
    w |= 1ull << (q & 63);
    ++k;
  }
  const double h = M_SQRT1_2, re[8] = {1, h, 0, -h, -1, -h, 0, h}, im[8] = {0, h, 1, h, 0, -h, -1, -h};
  g.m[0].re = g.m[1].re = 1.0;
  if (kind & 1u) g.flip = 1;
  if (kind & 2u) {   // eighth turns
    const uint32_t a = below(8), b = below(8);
    g.m[0] = sim_c64{re[a], im[a]};
    g.m[1] = sim_c64{re[b], im[b]};
  } else if (kind & 4u) {   // any angles
    const double a = (double)(next_u64() >> 11) * 0x1p-53, b = (double)(next_u64() >> 11) * 0x1p-53;
    g.m[0] = sim_c64{std::cos(a), std::sin(a)};
    g.m[1] = sim_c64{std::cos(b), -std::sin(b)};
  }
  return g;
}

}  // namespace

int main(int argc, char** argv) {
  const int cases = argc > 1 ? atoi(argv[1]) : 300;
  const uint32_t nqs[] = {4, 24, 64, 65, 100, 113, 120, 121, 125, 128};
  double most = 0;
  for (int c = 0; c < cases; ++c) {
    sm_state = 0x5EEDull * (c + 1);
    const uint32_t nq = nqs[c % 10], len = 1 + below(c % 3 ? 300 : 6);
    const uint32_t only_kind = 1 + below(12), only_ctrl = below(8);   // (7 and 3 or fewer: all gates so)
    RunCompiler rc;
    rc.schedule_part = 1 + below(40);
    rc.compile_part = 16;
    for (uint32_t i = 0; i < len; ++i) {
      const uint32_t kind = only_kind <= 7 ? only_kind : 1 + below(7), nc = only_ctrl <= 3 ? only_ctrl : below(4);
      rc.descs.push_back(mono_desc(random_gate(nq, kind, std::min(nc, nq - 1))));
    }
    rc.compile(nq);
    BsRun br{};
    if (!rc.run_params(0, len, SIM_MONO_BITSLICE, 0, &br)) return printf("case %d: not bit-sliced\n", c), 1;
    std::vector<RpBlock> blocks;
    rc.program(0, len, blocks, &br);
    if (blocks.size() > RunCompiler::rp_blocks_bound(len, nq))
      return printf("case %d (nq %u, %u gates): %zu blocks, the bound is %zu\n", c, nq, len, blocks.size(),
                    RunCompiler::rp_blocks_bound(len, nq)), 1;
    most = std::max(most, (double)blocks.size() / (double)RunCompiler::rp_blocks_bound(len, nq));
    Machine got;
    for (uint32_t q = 0; q < nq; ++q) got.v[kRpPlane0 + q] = (uint32_t)next_u64();
    got.v[kRpPlane0 + nq] = ~0u;
    Machine ref = got;
    BsRun plain{};
    (void)rc.run_params(0, len, SIM_MONO_BITSLICE, 0, &plain);
    for (const BsOp& o : rc.ops) {
      uint32_t x = ~0u;
      for (int k = 0; k < o.nctrl; ++k) x &= ref.v[kRpPlane0 + o.ctrl[k]];
      if (o.op == kBsFlip) {
        ref.v[kRpPlane0 + o.target] ^= x;
        continue;
      }
      if (o.cmode) x &= ref.v[kRpPlane0 + o.target];
      if (o.op == kBsTurn) {
        ref.turn(x, o.arg);
      } else {
        if (o.arg & 1) ref.t(x);
        if (o.arg & 2) ref.s(x);
        if (o.arg & 4) ref.v[0] ^= x;
      }
    }
    if (!run_program(got, blocks, nq)) return printf("case %d (nq %u, %u gates): malformed program\n", c, nq, len), 1;
    for (uint32_t q = 0; q < nq; ++q)
      if (got.v[kRpPlane0 + q] != ref.v[kRpPlane0 + q]) return printf("case %d: plane %u differs\n", c, q), 1;
    for (int j = 0; j < 32; ++j)
      if (((eighths(got, j) + br.g_omega) & 7u) != ((eighths(ref, j) + plain.g_omega) & 7u) ||
          got.turns[j] + br.g_turn != ref.turns[j] + plain.g_turn)
        return printf("case %d: phases differ\n", c), 1;
  }
  printf("OK cases=%d, at most %.2f of the bound\n", cases, most);
  return 0;
}
