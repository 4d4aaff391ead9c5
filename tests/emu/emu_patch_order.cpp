// CPU check that a run of up to K MCS on patches needs no order among them:
// the patches of a lattice are loaded, run and stored one after the other, in
// two orders, from one copy of the lattice to another, and give the oracle's
// bytes.  (In place they do not: a patch would load what its neighbour stored.)
#include "escg_lds.hpp"
#include "escg_patch.hpp"
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

struct C { uint32_t L, PY, PX, K, n; };

static int run_case(const C &c) {
  const uint32_t S = 3, L = c.L, seed = 99 + L, rep = 2, mcs0 = 5;
  std::vector<uint8_t> D(S * S);
  orc_circulant_matrix(S, 0b10, D.data());
  uint32_t dom[32] = {0};
  for (uint32_t a = 1; a <= S; ++a) for (uint32_t b = 1; b <= S; ++b) if (D[(a-1)*S+(b-1)]) dom[a] |= 1u << b;
  uint32_t T1, T2; orc_thresholds(0.5, 1, 1, &T1, &T2);
  static LdsTables<8> TB;
  setup_tables(TB, dom, false);
  const auto qc = make_quad_ctx(TB, T1, T2);
  PatchGeom G{};
  G.L = L; G.PY = c.PY; G.PX = c.PX; G.K = c.K; G.HQ = (4 * c.K + 1 + 7) / 8;
  G.set_cuts();
  const uint32_t T = c.PY * c.PX, nb = patch_buffer_bytes(G);
  std::vector<uint8_t> g(L * L); srand(L); for (auto &v : g) v = rand() % (S + 1);
  const auto run = [&](const uint8_t *from, uint8_t *to, bool backwards) {
    for (uint32_t i = 0; i < T; ++i) {
      const Patch P = patch_of(G, backwards ? T - 1 - i : i);
      const uint32_t bd = ((P.RH / 2) * P.NJ + 63) / 64 * 64;
      std::vector<uint64_t> sm(nb / 4 + 8, 0);
      uint8_t *src = reinterpret_cast<uint8_t *>(sm.data()) + 8, *dst = src + nb;
      uint32_t s = 0;
      threads(bd, [&] { patch_load(src, from, G, P); });
      for (uint32_t t = mcs0; t < mcs0 + c.n; ++t) {
        const Words off = philox(0u, t, kTagOffset << 8, rep, seed, 0);
        for (uint32_t p = 0; p < 4; ++p) {
          threads(bd, [&] {
            const PatchList<1> Q = patch_list<1>(G, P, bd);
            Words rf = philox(Q.c0[0], t, (kTagPass << 8) | p, rep, seed, 0); QuadSel sf = quad_sel(rf, qc);
            const PassIndex ix{t, p}, nx{t, p + 1};
            if (P.seam != ~0u) patch_pass<true>(src, dst, s, P, Q, off.w[p], ix, nx, rep, seed, 0, qc, rf, sf);
            else patch_pass<false>(src, dst, s, P, Q, off.w[p], ix, nx, rep, seed, 0, qc, rf, sf);
          });
          std::swap(src, dst);
          s = off.w[p] & 1u;
        }
      }
      threads(bd, [&] { patch_store(src, s, to, G, P, bd); });
    }
  };
  std::vector<uint8_t> ref = g, place = g;
  std::vector<uint32_t> rc((c.n + 1) * (S + 1));
  orc_o2_run(L, S, D.data(), 0.5, 1, 1, seed, rep, kPhiloxRounds, 4, nullptr, mcs0, c.n, ref.data(), rc.data());
  int bad = 0;
  for (bool backwards : {false, true}) {
    std::vector<uint8_t> out(L * L, 0xEE);
    run(g.data(), out.data(), backwards);
    if (out != ref) { bad++; printf("MISMATCH L=%u n=%u\n", L, c.n); }
  }
  run(place.data(), place.data(), false);
  if (place == ref) { bad++; printf("IN PLACE EQUAL L=%u\n", L); }
  return bad;
}

int main() {
  blockDim.x = 1; threadIdx.x = 0;
  const C cs[] = {{72, 3, 2, 1, 1}, {74, 4, 2, 1, 1}, {100, 3, 2, 3, 1}, {100, 3, 2, 3, 3}, {98, 2, 2, 2, 2}, {126, 3, 1, 5, 4}, {96, 5, 4, 2, 2}};
  int bad = 0, cases = 0;
  for (const C &c : cs) { bad += run_case(c) != 0; cases++; }
  printf("%d/%d order cases ok\n", cases - bad, cases);
  return bad != 0;
}
