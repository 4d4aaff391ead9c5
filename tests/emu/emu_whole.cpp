// CPU check of the small-lattice kernel's phases (whole_load, whole_pass,
// counting sums, whole_store_word) against the oracle, for sides of every
// remainder mod 8 from the smallest to the largest.
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

template <int SP>
static int run_case(uint32_t L, uint32_t S, bool moore, const double *r) {
  int bad = 0;
  std::vector<uint8_t> D(S * S);
  orc_circulant_matrix(S, S < 5 ? 0b10 : 0b1010, D.data());
  if (S == 2) { D[1] = 1; D[2] = 1; }
  uint32_t dom[32] = {0};
  for (uint32_t a = 1; a <= S; ++a) for (uint32_t b = 1; b <= S; ++b) if (D[(a-1)*S+(b-1)]) dom[a] |= 1u << b;
  uint32_t T1, T2; orc_thresholds(r[0], r[1], r[2], &T1, &T2);
  static LdsTables<SP> TB;
  setup_tables(TB, dom, moore);
  const auto qc = make_quad_ctx(TB, T1, T2);
  const WholeGeom G = whole_geom(L);
  const uint32_t size = L * G.LS, nw = L * G.Q(), n = 6, nt = ((L >> 1) * G.Q() + 63) / 64 * 64;
  std::vector<uint64_t> sm(3 * size / 8, 0);
  uint8_t *cur = reinterpret_cast<uint8_t *>(sm.data()), *p1 = cur + size, *p2 = cur + 2 * size;
  std::vector<uint8_t> g(L * L); srand(L + S); for (auto &v : g) v = rand() % (S + 1);
  std::vector<uint32_t> cnt((n + 1) * (S + 1), 0), rc(cnt);
  threads(64, [&] { whole_load(cur, g.data(), G); });
  const uint64_t seed = 7 + L; const uint32_t rep = 3, mcs0 = 11, k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  uint32_t s = 0;
  auto count = [&](uint32_t row) {
    const uint32_t ns = count_states(S);
    if (SP == 32) {
      std::vector<uint32_t> h(32 * kCountSlots + 4, 0); uint32_t *hp = h.data(); while ((uintptr_t)hp & 15) ++hp;
      for (uint32_t st = 0; st < 3; ++st) threads(64, [&] { whole_hist(cur, nw, st, hp); });
      std::vector<uint32_t> c(32, 0);
      for (uint32_t l = 0; l < 64; ++l) c[l >> 1] += patch_hist_half(hp, l);
      c[0] -= size - L * L;
      for (uint32_t v = 0; v <= S; ++v) cnt[row * (S + 1) + v] = c[v];
      return;
    }
    uint32_t T[8] = {0}; // the wave's sums, as pair_sums_count takes them apart
    threads(64, [&] {
      uint32_t q4[2] = {0}, q6[3] = {0}, q8[4] = {0}, *q = ns == 4 ? q4 : ns == 6 ? q6 : q8;
      for (uint32_t st = 0; st < 3; ++st)
        if (ns == 4) whole_word_sums<4>(cur, nw, st, q4); else if (ns == 6) whole_word_sums<6>(cur, nw, st, q6); else whole_word_sums<8>(cur, nw, st, q8);
      for (uint32_t k = 0; k < ns - 1; ++k) T[k] += (k & 1) ? q[k / 2] >> 16 : k + 2 == ns ? q[k / 2] : q[k / 2] & 0xFFFF;
    });
    for (uint32_t k = 0; k < ns - 1; ++k) if (T[k] > 0xFFFF) { bad++; printf("SUM OVER 16 BITS\n"); }
    for (uint32_t v = 0; v <= S; ++v) {
      uint32_t t3[3], t5[5], t7[7]; for (int k = 0; k < 7; ++k) { if (k < 3) t3[k] = T[k]; if (k < 5) t5[k] = T[k]; t7[k] = T[k]; }
      cnt[row * (S + 1) + v] = ns == 4 ? count_species<4>(v, t3, L * L) : ns == 6 ? count_species<6>(v, t5, L * L) : count_species<8>(v, t7, L * L);
    }
  };
  count(0);
  for (uint32_t t = 0; t < n; ++t) {
    const Words off = philox(0u, mcs0 + t, kTagOffset << 8, rep, k0, k1);
    for (uint32_t p = 0; p < 4; ++p) {
      const uint8_t *src = p == 0 ? cur : (p & 1) ? p1 : p2; uint8_t *dst = (p & 1) ? p2 : p1;
      threads(nt, [&] {
        PatchList<1> T; const WholeQuad W = whole_quad(G, T);
        Words rf = philox(W.c0, mcs0 + t, (kTagPass << 8) | p, rep, k0, k1); QuadSel sf = quad_sel(rf, qc);
        whole_pass(src, dst, s, G, W, T, G.part() != 0, off.w[p], mcs0 + t, (kTagPass << 8) | (p + 1), rep, k0, k1, qc, rf, sf);
      });
      s = off.w[p] & 1u;
    }
    uint8_t *x = p2; p2 = p1; p1 = cur; cur = x;
    count(t + 1);
  }
  std::vector<uint8_t> out(L * L, 0xEE), ref = g;
  for (uint32_t i = 0; i < nw; ++i) whole_store_word(cur, s, i / G.Q(), i % G.Q(), out.data(), G);
  orc_o2_run(L, S, D.data(), r[0], r[1], r[2], seed, rep, kPhiloxRounds, moore ? 8 : 4, nullptr, mcs0, n, ref.data(), rc.data());
  if (out != ref) { bad++; printf("MISMATCH L=%u S=%u\n", L, S); }
  if (cnt != rc) { bad++; printf("COUNT MISMATCH L=%u S=%u\n", L, S); }
  return bad;
}

int main() {
  blockDim.x = 1; threadIdx.x = 0;
  const uint32_t Ls[] = {2, 4, 6, 8, 10, 12, 14, 16, 18, 30, 64, 66, 68, 70, 82, 88}, Ss[] = {3, 5, 7, 13, 2, 31, 1};
  const double rates[][3] = {{0.5, 1, 1}, {13.1, 1, 1}, {0, 1, 1}};
  int bad = 0, cases = 0;
  for (bool moore : {false, true}) for (uint32_t L : Ls) for (int k = 0; k < 2; ++k) {
    const uint32_t S = Ss[(cases * 3 + k) % 7];
    bad += (S <= 7 ? run_case<8>(L, S, moore, rates[cases % 3]) : run_case<32>(L, S, moore, rates[cases % 3])) != 0;
    cases++;
  }
  printf("%d/%d whole cases ok\n", cases - bad, cases);
  return bad != 0;
}
