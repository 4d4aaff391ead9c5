// CPU check of the patch kernel's phases (patch_load, patch_pass, counts,
// patch_publish, patch_gather, patch_store) against the oracle: even sides of
// every remainder mod 8, uneven cuts, one to five MCS between exchanges, both
// count layouts, probabilities, both neighbourhoods.
#include "escg_lds.hpp"
#include "escg_patch.hpp"
#include <vector>
#include <cstdlib>
#include <algorithm>
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

// One pass of a whole workgroup (threads one after another: a pass reads one
// copy of the region and writes the other).
template <int kSlots, class Ctx>
static void wg_pass(const uint8_t *src, uint8_t *dst, uint32_t s, const PatchGeom &G, const Patch &P, uint32_t bd,
                    uint32_t w, uint32_t t, uint32_t p, uint32_t rep, uint32_t k0, uint32_t k1, const Ctx &qc) {
  threads(bd, [&] {
    const PatchList<kSlots> T = patch_list<kSlots>(G, P, bd);
    Words rf = philox(T.c0[0], t, (kTagPass << 8) | p, rep, k0, k1);
    QuadSel sf = quad_sel(rf, qc);
    const PassIndex ix{t, p}, nx{t, p + 1};
    if (P.seam != ~0u) patch_pass<true>(src, dst, s, P, T, w, ix, nx, rep, k0, k1, qc, rf, sf);
    else patch_pass<false>(src, dst, s, P, T, w, ix, nx, rep, k0, k1, qc, rf, sf);
  });
}

static int words = 0;  // patches counted by the counting wave's sums
struct C { uint32_t L, PY, PX, K, S; };

template <bool kProb, int SP>
static int run_case(const C &c, bool moore, const double *r, int ci) {
  int bad = 0;
  const uint32_t S = c.S, L = c.L;
  std::vector<uint8_t> D(S * S);
  orc_circulant_matrix(S, S == 3 ? 0b10 : 0b1010, D.data());
  if (S == 2) { D[1] = 1; D[2] = 1; }
  uint32_t dom[32] = {0};
  for (uint32_t a = 1; a <= S; ++a) for (uint32_t b = 1; b <= S; ++b) if (D[(a-1)*S+(b-1)]) dom[a] |= 1u << b;
  uint32_t T1, T2; orc_thresholds(r[0], r[1], r[2], &T1, &T2);
  std::vector<double> Pr(S * S, 0.0);
  std::vector<uint32_t> ab(2 * SP * SP, 0u);
  for (uint32_t i = 0; i < S * S; ++i) Pr[i] = D[i] ? 0.25 + 0.05 * (i % 11) : 0.0;
  for (uint32_t x = 1; x <= S; ++x) for (uint32_t y = 1; y <= S; ++y) if (x != y) {
    const uint32_t R = T2 - T1, A = (uint32_t)(Pr[(x-1)*S+y-1] * R);
    ab[x * SP + y] = A;
    ab[SP * SP + x * SP + y] = A + (uint32_t)(Pr[(y-1)*S+x-1] * (double)(R - A));
  }
  PatchGeom G{};
  G.L = L; G.PY = c.PY; G.PX = c.PX; G.K = c.K; G.HQ = (4 * c.K + 1 + 7) / 8;
  G.set_cuts();
  const uint32_t T = c.PY * c.PX;
  uint32_t TQmax = 0, THmax = 0, THmin = ~0u, TQmin = ~0u;
  for (uint32_t i = 0; i < T; ++i) { const Patch P = patch_of(G, i);
    TQmax = std::max(TQmax, P.TQ); THmax = std::max(THmax, P.TH); THmin = std::min(THmin, P.TH); TQmin = std::min(TQmin, P.TQ); }
  if (THmin < G.HR() || TQmin < G.HQ || (G.part() && TQmin < 2 * G.HQ + 1)) { printf("BAD CASE L=%u\n", L); return 1; }
  G.slot_words = patch_slot_words(THmax, TQmax, G.HR(), G.HQ);
  const uint32_t nb = patch_buffer_bytes(G), cdw = patch_count_dwords(SP == 8);
  static LdsTables<SP> TB;
  setup_tables(TB, dom, moore, kProb ? ab.data() : nullptr);
  const auto qc = make_quad_ctx<kProb>(TB, T1, T2);
  std::vector<uint8_t> g(L * L); srand(L + S * 7 + T1 + ci);
  for (auto &v : g) v = rand() % (S + 1);
  std::vector<std::vector<uint64_t>> sm(T, std::vector<uint64_t>(nb / 4 + 8, 0));
  std::vector<uint64_t> exch(2 * (size_t)T * G.slot_words, 0);
  for (size_t i = exch.size() / 2; i < exch.size(); ++i) exch[i] = 0x8080808080808080ull;
  uint32_t abort_word = 0;
  auto bufs = [&](uint32_t t, int b) { return reinterpret_cast<uint8_t *>(sm[t].data()) + 8 + (size_t)b * nb; };
  for (uint32_t t = 0; t < T; ++t) { const Patch P = patch_of(G, t); threads(64, [&] { patch_load(bufs(t, 0), g.data(), G, P); }); }
  { // the sweep's quads and its load and store give the same regions
    const uint32_t RH = 2 * G.row_cut(1) + 2 * G.HR();
    std::vector<uint8_t> out(L * L, 0xEE);
    for (uint32_t t = 0; t < T; ++t) {
      const Patch P = patch_of(G, t);
      const uint32_t bd = ((RH / 2) * P.NJ + 3 * 64 - 1) / (3 * 64) * 64;
      std::vector<uint64_t> tmp(nb / 4 + 8, 0);
      uint8_t *buf = reinterpret_cast<uint8_t *>(tmp.data()) + 8;
      std::vector<SweepQuads<3>> W(bd);
      threads(bd, [&] { sweep_column(G, P, RH, bd, W[threadIdx.x]); sweep_load(buf, g.data(), G, P, W[threadIdx.x]);
        const PatchList<3> T3 = patch_list<3>(G, P, bd);
        for (int i = 0; i < 3; ++i) if (W[threadIdx.x].row[i] < P.RH / 2 && (T3.pa[i] != W[threadIdx.x].T.pa[i] || T3.c0[i] != W[threadIdx.x].T.c0[i] || T3.part[i] != W[threadIdx.x].T.part[i]) && threadIdx.x + i * bd < (P.RH / 2) * P.NJ) { bad++; printf("SWEEP QUAD L=%u\n", L); } });
      for (uint32_t r = 0; r < P.RH; ++r) if (std::memcmp(buf + r * P.LS, bufs(t, 0) + r * P.LS, 8 * P.NJ)) { bad++; printf("SWEEP LOAD L=%u row %u\n", L, r); break; }
      threads(bd, [&] { sweep_store(buf, 0, out.data(), G, P, W[threadIdx.x]); });
    }
    if (out != g) { bad++; printf("SWEEP STORE L=%u\n", L); }
  }
  const uint64_t seed = 99 + L; const uint32_t rep = 2, mcs0 = 5, n = 2 * c.K + 3;
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  std::vector<uint32_t> cnt((n + 1) * (S + 1), 0);
  int cur = 0; uint32_t s = 0;
  auto count = [&](uint32_t row) {
    for (uint32_t t = 0; t < T; ++t) {
      const Patch P = patch_of(G, t);
      const uint32_t gap = P.seam != ~0u ? P.TH * (8 - 2 * G.part()) : 0u, sites = P.TH * 8 * P.TQ - gap;
      std::vector<uint32_t> part(cdw + 4, 0), sc(64, 0);
      uint32_t *pp = part.data(); while ((uintptr_t)pp & 15) ++pp;
      const uint32_t ns = count_states(S), bd = (row & 1) ? 64 : std::max(P.TQ, 5u);
      threads(bd, [&] { const PatchCount K = patch_count_plan(G, P);
        if (SP == 32) patch_count_hist(bufs(t, cur), K, P.TH, pp);
        else if (ns == 4) patch_count_sums<4>(bufs(t, cur), K, P.TH, pp);
        else if (ns == 6) patch_count_sums<6>(bufs(t, cur), K, P.TH, pp);
        else patch_count_sums<8>(bufs(t, cur), K, P.TH, pp); });
      if (SP == 8 && P.TH * P.TQ <= 64 * kCountWords && (row & 1)) { // the counting wave's sums instead
        std::fill(pp, pp + cdw, 0u);
        threads(64, [&] { const PatchCounted w = patch_read_words(bufs(t, cur), patch_words(G, P));
          uint32_t q4[2] = {0}, q6[3] = {0}, q8[4] = {0}, *q = ns == 4 ? q4 : ns == 6 ? q6 : q8;
          if (ns == 4) { patch_word_sums<4, 0>(w, q4); patch_word_sums<4, 1>(w, q4); }
          else if (ns == 6) { patch_word_sums<6, 0>(w, q6); patch_word_sums<6, 1>(w, q6); }
          else { patch_word_sums<8, 0>(w, q8); patch_word_sums<8, 1>(w, q8); }
          for (uint32_t k = 0; k < ns - 1; ++k) pp[k * kCountSlots] += (k & 1) ? q[k / 2] >> 16 : k + 2 == ns ? q[k / 2] : q[k / 2] & 0xFFFF; });
        words++;
      }
      if (SP == 32) {
        for (uint32_t l = 0; l < 64; ++l) sc[l >> 1] += patch_hist_half(pp, l);
        sc[0] -= gap;
      } else {
        uint32_t T8[8] = {0};
        for (uint32_t l = 0; l < 64; ++l) T8[l >> 3] += count_slot_sum(pp, l, ns - 1);
        for (uint32_t l = 0; l <= S; ++l) {
          if (ns == 4) { uint32_t t3[3] = {T8[0], T8[1], T8[2]}; sc[l] = count_species<4>(l, t3, sites); }
          else if (ns == 6) { uint32_t t5[5] = {T8[0], T8[1], T8[2], T8[3], T8[4]}; sc[l] = count_species<6>(l, t5, sites); }
          else { uint32_t t7[7]; for (int q = 0; q < 7; ++q) t7[q] = T8[q]; sc[l] = count_species<8>(l, t7, sites); }
        }
      }
      for (uint32_t q = 0; q < cdw; ++q) if (pp[q]) { bad++; printf("SLOT NOT CLEARED\n"); break; }
      for (uint32_t q = 0; q <= S; ++q) cnt[row * (S + 1) + q] += sc[q];
    }
  };
  count(0);
  for (uint32_t t0 = 0, e = 1; t0 < n; ++e) {
    const uint32_t m1 = std::min(G.K, n - t0);
    for (uint32_t m = 0; m < m1; ++m) {
      const uint32_t mt = mcs0 + t0 + m;
      const Words off = philox(0u, mt, kTagOffset << 8, rep, k0, k1);
      for (uint32_t p = 0; p < 4; ++p) {
        for (uint32_t t = 0; t < T; ++t) {
          const Patch P = patch_of(G, t);
          const uint32_t nq = (P.RH / 2) * P.NJ;
          const int sl = 1 + (ci + t) % 3;
          const uint32_t bd = (nq + 64 * sl - 1) / (64 * sl) * 64;
          if (sl == 1) wg_pass<1>(bufs(t, cur), bufs(t, cur ^ 1), s, G, P, bd, off.w[p], mt, p, rep, k0, k1, qc);
          else if (sl == 2) wg_pass<2>(bufs(t, cur), bufs(t, cur ^ 1), s, G, P, bd, off.w[p], mt, p, rep, k0, k1, qc);
          else wg_pass<3>(bufs(t, cur), bufs(t, cur ^ 1), s, G, P, bd, off.w[p], mt, p, rep, k0, k1, qc);
        }
        cur ^= 1; s = off.w[p] & 1u;
      }
      count(t0 + m + 1);
    }
    t0 += m1;
    if (t0 == n) break;
    const uint32_t tag = exch_tag(e);
    uint64_t *area = exch.data() + (size_t)exch_slot(e) * T * G.slot_words;
    const uint32_t bd = 64 + 64 * (ci % 4);
    for (int fresh = 0; fresh < 2; ++fresh) {
      // nothing published yet for this exchange: every word must read stale
      for (uint32_t t = 0; t < T; ++t) {
        const Patch P = patch_of(G, t);
        std::vector<uint64_t> tmp; uint8_t *to = bufs(t, cur);
        if (!fresh) { tmp = sm[t]; to = reinterpret_cast<uint8_t *>(tmp.data()) + 8 + (size_t)cur * nb; }
        threads(bd, [&] {
          const PatchHalo H = patch_halo(G, P);
          const uint32_t st = patch_gather(to, area, H, G, P, tag, &abort_word, fresh ? 64 : 32, [] {});
          if (st != (fresh || threadIdx.x >= H.n ? 0u : 2u)) { bad++; if (bad < 9) printf("GATHER %u L=%u fresh=%d\n", st, L, fresh); }
        });
      }
      if (!fresh)
        for (uint32_t t = 0; t < T; ++t) {
          const Patch P = patch_of(G, t);
          threads(bd, [&] { patch_publish(bufs(t, cur), area + (size_t)t * G.slot_words, patch_halo(G, P), G, P, tag); });
        }
    }
  }
  std::vector<uint8_t> out(L * L, 0xEE), ref = g;
  for (uint32_t t = 0; t < T; ++t) { const Patch P = patch_of(G, t); threads(64, [&] { patch_store(bufs(t, cur), s, out.data(), G, P, 64); }); }
  std::vector<uint32_t> rc((n + 1) * (S + 1), 0);
  orc_o2_run(L, S, D.data(), r[0], r[1], r[2], seed, rep, kPhiloxRounds, moore ? 8 : 4, kProb ? Pr.data() : nullptr, mcs0, n, ref.data(), rc.data());
  if (out != ref) { bad++; size_t d = 0; for (size_t i = 0; i < out.size(); ++i) d += out[i] != ref[i];
    printf("MISMATCH L=%u PY=%u PX=%u K=%u S=%u moore=%d: %zu sites\n", L, c.PY, c.PX, c.K, S, moore, d); }
  if (cnt != rc) { bad++; printf("COUNT MISMATCH L=%u PY=%u PX=%u K=%u S=%u\n", L, c.PY, c.PX, c.K, S); }
  return bad;
}

int main() {
  blockDim.x = 1; threadIdx.x = 0;
  const C cs[] = {{72, 3, 2, 1, 3}, {74, 4, 2, 1, 5}, {76, 2, 3, 1, 2}, {78, 3, 1, 1, 7}, {80, 3, 3, 2, 3}, {98, 2, 2, 2, 8},
                  {100, 3, 2, 3, 4}, {102, 4, 1, 3, 6}, {130, 1, 1, 1, 3}, {126, 3, 1, 5, 13}, {104, 2, 3, 4, 3}, {84, 2, 2, 1, 31},
                  {90, 1, 1, 3, 5}, {96, 5, 4, 2, 1}};
  const double rates[][3] = {{0.5, 1, 1}, {13.1, 1, 1}, {0, 1, 1}};
  int bad = 0, cases = 0, ci = 0;
  for (bool moore : {false, true}) for (const C &c : cs) {
    const double *r = rates[ci % 3];
    const bool prob = ci % 4 == 3 && c.S > 2;
    int b = c.S <= 7 ? (prob ? run_case<true, 8>(c, moore, r, ci) : run_case<false, 8>(c, moore, r, ci))
                     : (prob ? run_case<true, 32>(c, moore, r, ci) : run_case<false, 32>(c, moore, r, ci));
    cases++; ci++; bad += b != 0;
  }
  if (!words) printf("NO COUNTING WAVE\n");
  printf("%d/%d patch cases ok\n", cases - bad, cases);
  return bad != 0 || !words;
}
