// CPU checks of the kernel that keeps two copies of a lattice in LDS: its pass
// (whole_slots, whole_pass_slots) against the oracle for one to five quads a
// thread and sides of every remainder mod 8, the species a test of the stop
// condition sees (species_bits), and the windows between those tests
// (pair_window), whose cost is bounded for a stop after any MCS.
#include "escg_lds.hpp"
#include "escg_whole.hpp"
#include <vector>
#include <cstdlib>
emu_dim3 threadIdx, blockDim, blockIdx, gridDim;
using namespace escg;
extern "C" void orc_o2_run(uint32_t L, uint32_t S, const uint8_t *D, double ex, double sel, double rep,
  uint64_t seed, uint32_t replica, int rounds, int nbhd, const double *P, uint32_t mcs0, uint32_t n_mcs, uint8_t *grid, uint32_t *counts);
extern "C" void orc_thresholds(double ex, double sel, double rep, uint32_t *T1, uint32_t *T2);
extern "C" void orc_circulant_matrix(uint32_t S, uint32_t kmask, uint8_t *D);

template <class Fn> static void threads(uint32_t n, Fn &&fn) {
  blockDim.x = n;
  for (threadIdx.x = 0; threadIdx.x < n; ++threadIdx.x) fn();
  blockDim.x = 1; threadIdx.x = 0;
}

template <int SP, int kSlots>
static int run_case(uint32_t L, uint32_t S, bool moore, const double *r, uint32_t nt) {
  std::vector<uint8_t> D(S * S);
  orc_circulant_matrix(S, S < 5 ? 0b10 : 0b1010, D.data());
  uint32_t dom[32] = {0};
  for (uint32_t a = 1; a <= S; ++a) for (uint32_t b = 1; b <= S; ++b) if (D[(a-1)*S+(b-1)]) dom[a] |= 1u << b;
  uint32_t T1, T2; orc_thresholds(r[0], r[1], r[2], &T1, &T2);
  static LdsTables<SP> TB;
  setup_tables(TB, dom, moore);
  const auto qc = make_quad_ctx(TB, T1, T2);
  const WholeGeom G = whole_geom(L);
  const uint32_t size = L * G.LS, nw = L * G.Q(), n = 5;
  // a spare word on either side of the copies: a window that left them shows
  std::vector<uint64_t> sm(2 * size / 8 + 2, 0x1F1F1F1F1F1F1F1Full);
  uint8_t *src = reinterpret_cast<uint8_t *>(sm.data() + 1), *dst = src + size;
  std::fill(sm.begin() + 1, sm.end() - 1, 0);
  std::vector<uint8_t> g(L * L); srand(L + S); for (auto &v : g) v = rand() % (S + 1);
  threads(64, [&] { whole_load(src, g.data(), G); });
  const uint64_t seed = 7 + L; const uint32_t rep = 3, mcs0 = 11, k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  uint32_t s = 0;
  for (uint32_t t = mcs0; t < mcs0 + n; ++t) {
    const Words off = philox(0u, t, kTagOffset << 8, rep, k0, k1);
    for (uint32_t p = 0; p < 4; ++p) {
      threads(nt, [&] {
        WholeSlots<kSlots> W = whole_slots<kSlots>(G, nt);
        Words rf = philox(W.c0[0], t, (kTagPass << 8) | p, rep, k0, k1); QuadSel sf = quad_sel(rf, qc);
        const PassIndex nx = p < 3 ? PassIndex{t, p + 1} : PassIndex{t + 1, 0};
        whole_pass_slots<kSlots>(src, dst, s, G, W, off.w[p], PassIndex{t, p}, nx, rep, k0, k1, qc, rf, sf);
      });
      std::swap(src, dst);
      s = off.w[p] & 1u;
    }
  }
  std::vector<uint8_t> out(L * L, 0xEE), ref = g;
  for (uint32_t i = 0; i < nw; ++i) whole_store_word(src, s, i / G.Q(), i % G.Q(), out.data(), G);
  std::vector<uint32_t> rc((n + 1) * (S + 1));
  orc_o2_run(L, S, D.data(), r[0], r[1], r[2], seed, rep, kPhiloxRounds, moore ? 8 : 4, nullptr, mcs0, n, ref.data(), rc.data());
  uint32_t seen = 0, want = 0;
  for (uint32_t i = 0; i < nw; ++i) seen |= species_fold<SP == 8>(species_bits<SP == 8>(reinterpret_cast<const uint2 *>(src)[i]));
  for (uint8_t v : ref) want |= 1u << v;
  const bool ok = out == ref && ((seen ^ want) & ~1u) == 0 && sm.front() == 0x1F1F1F1F1F1F1F1Full && sm.back() == sm.front();
  if (!ok) printf("MISMATCH L=%u S=%u slots=%d threads=%u\n", L, S, kSlots, nt);
  return !ok;
}

template <int SP>
static int run_slots(uint32_t L, uint32_t S, bool moore, const double *r, uint32_t nt) {
  switch (((L >> 1) * ((L + 7) / 8) + nt - 1) / nt) {
  case 1: return run_case<SP, 1>(L, S, moore, r, nt);
  case 2: return run_case<SP, 2>(L, S, moore, r, nt);
  case 3: return run_case<SP, 3>(L, S, moore, r, nt);
  case 4: return run_case<SP, 4>(L, S, moore, r, nt);
  case 5: return run_case<SP, 5>(L, S, moore, r, nt);
  default: printf("NO SLOTS L=%u threads=%u\n", L, nt); return 1;
  }
}

// A run that stops after MCS `stop` as the kernel goes through it: MCS run and
// tests made.
static int window_case(uint32_t stop) {
  uint32_t t = 0, run = 0, tests = 1; bool replay = false;
  for (;;) {
    const uint32_t n = replay ? 1 : pair_window(t);
    t += n; run += n; ++tests;
    if (t < stop) continue;
    if (n == 1) break;
    t -= n; replay = true;
  }
  const bool ok = t == stop && run <= stop + stop / 8 && tests <= 137 + stop / 32 + 32 && (stop > 128 || run == stop);
  if (!ok) printf("WINDOWS stop=%u run=%u tests=%u\n", stop, run, tests);
  return !ok;
}

int main() {
  blockDim.x = 1; threadIdx.x = 0;
  // L, threads: one to five quads a thread, last slots full, partly and not
  const uint32_t Ls[][2] = {{2, 64}, {8, 64}, {14, 64}, {22, 64}, {24, 64}, {26, 64}, {32, 64}, {34, 64}, {36, 64},
    {38, 64}, {40, 64}, {42, 64}, {44, 64}, {46, 64}, {48, 64}, {50, 64}, {66, 128}, {68, 128}, {70, 128}, {278, 1024}, {280, 1024}};
  const uint32_t Ss[] = {3, 5, 7, 13, 31};
  const double rates[][3] = {{0.5, 1, 1}, {13.1, 1, 1}, {0, 1, 1}};
  int bad = 0, cases = 0;
  for (const auto &x : Ls) for (int k = 0; k < 2; ++k) {
    const uint32_t S = Ss[cases % 5]; const bool moore = cases % 3 == 2;
    bad += (S <= 7 ? run_slots<8>(x[0], S, moore, rates[cases % 3], x[1]) : run_slots<32>(x[0], S, moore, rates[cases % 3], x[1])) != 0;
    cases++;
  }
  for (uint32_t stop = 1; stop < 4000; ++stop, ++cases) bad += window_case(stop);
  printf("%d/%d pair cases ok\n", cases - bad, cases);
  return bad != 0;
}
