// escg_whole.hpp -- a small lattice whole in one workgroup's LDS, one quad per
// thread.
//
// What bounds it: latency.  With at most one quad per thread (L <= 88, one to
// two waves a SIMD) a pass is one chain of row reads, rule lookup, stores and
// a barrier, whatever the lattice holds.  So, as in the patch kernel
// (escg_patch.hpp: the two copies of the lattice and their shifts, the row's
// partial quad and its gap, the counting wave): a pass reads one copy and
// writes another with aligned stores and one barrier, the next pass's draws
// and selector lookups run in the shadow of the rows', and a wave of its own
// counts the species and tests the stop condition while the next MCS runs.
// Three copies: an MCS's four passes go from the first to the second and then
// to and fro between the other two, so the state that is being counted, and
// is the result if it meets the stop condition, outlives them.
// The lattice wraps inside the copies: the column past a row's last quad is
// its first one's, the row below the last is row 0.
// Measured at L = 64, one copy updated in place with the counts closed before
// the next MCS / this kernel: 2.9 / 1.45 us per MCS.
#pragma once

#include "escg_patch.hpp"

namespace escg {

struct WholeGeom {
    uint32_t L, LS; // side, LDS row stride 8 ceil(L / 8)
    __host__ __device__ uint32_t Q() const { return LS >> 3; }
    __host__ __device__ uint32_t part() const { return (L >> 1) & 3u; }
};

__host__ __device__ inline WholeGeom whole_geom(uint32_t L)
{
    return WholeGeom{L, (L + 7) & ~7u};
}

// A thread's quad, fixed for the run; threads past the last quad repeat it.
struct WholeQuad {
    uint32_t c0;         // Philox counter word
    uint32_t pa;         // LDS offset of the top row for oy = 0
    uint32_t pd;         // of the bottom row for oy = 1 (wrapped)
    uint32_t left, right; // offsets from a row's word to the dword before it
                          // and after it (wrapped)
};

// The quad's list entry for patch_swap as well: its selectors and whether it
// is the row's partial quad.
__device__ inline WholeQuad whole_quad(const WholeGeom &G, PatchList<1> &T)
{
    const uint32_t Q = G.Q(), Lb = G.L >> 1, nq = Lb * Q;
    const uint32_t q = min((uint32_t)threadIdx.x, nq - 1u);
    const uint32_t row = q / Q, col = q - row * Q;
    WholeQuad W;
    W.c0 = q;
    W.pa = 2 * row * G.LS + 8 * col;
    W.pd = row + 1 == Lb ? 8 * col : W.pa + 2 * G.LS;
    W.left = col == 0 ? G.LS - 4 : 0u - 4u;
    W.right = col + 1 == Q ? 8 - G.LS : 8u;
    patch_swap_selectors(G.part(), T);
    T.part[0] = G.part() && col + 1 == Q;
    return W;
}

// One pass from `src` (shift s) to `dst` (shift ox) with offsets w; (rf, sf),
// `ctr` and `t`: as patch_pass (one quad per thread), ctr and t being those
// of the pass that follows.
template <class Ctx>
__device__ __forceinline__ void whole_pass(const uint8_t *src, uint8_t *dst,
                                           uint32_t s, const WholeGeom &G,
                                           const WholeQuad &W,
                                           const PatchList<1> &T, bool seam,
                                           uint32_t w, uint32_t t,
                                           uint32_t ctr, uint32_t replica,
                                           uint32_t k0, uint32_t k1,
                                           const Ctx &qc, Words &rf,
                                           QuadSel &sf)
{
    const uint32_t ox = w & 1u;
    const bool oy = w & 2u, back = ox < s;
    const uint32_t pa = W.pa + (oy ? G.LS : 0u);
    const uint32_t pc = oy ? W.pd : W.pa + G.LS;
    const uint32_t sh = (ox - s) & 3u, side = back ? W.left : W.right;
    const uint2 ra = *reinterpret_cast<const uint2 *>(src + pa);
    const uint2 rc = *reinterpret_cast<const uint2 *>(src + pc);
    const uint32_t xa = *reinterpret_cast<const uint32_t *>(src + (pa + side));
    const uint32_t xc = *reinterpret_cast<const uint32_t *>(src + (pc + side));
    const Words rn = philox(W.c0, t, ctr, replica, k0, k1);
    const QuadSel qn = quad_sel(rn, qc);
    // the three dwords the window is cut from: side word first or last
    const uint32_t d0 = back ? xa : ra.x, d1 = back ? ra.x : ra.y,
                   d2 = back ? ra.y : xa;
    const uint32_t e0 = back ? xc : rc.x, e1 = back ? rc.x : rc.y,
                   e2 = back ? rc.y : xc;
    uint32_t a0 = __builtin_amdgcn_alignbyte(d1, d0, sh);
    uint32_t a1 = __builtin_amdgcn_alignbyte(d2, d1, sh);
    uint32_t c0 = __builtin_amdgcn_alignbyte(e1, e0, sh);
    uint32_t c1 = __builtin_amdgcn_alignbyte(e2, e1, sh);
    if (seam && ox) {
        patch_swap(a0, a1, T, 0);
        patch_swap(c0, c1, T, 0);
    }
    quad_update_sel(a0, a1, c0, c1, rf, sf, qc);
    if (seam && ox) {
        patch_swap(a0, a1, T, 0);
        patch_swap(c0, c1, T, 0);
    }
    *reinterpret_cast<uint2 *>(dst + pa) = make_uint2(a0, a1);
    *reinterpret_cast<uint2 *>(dst + pc) = make_uint2(c0, c1);
    rf = rn;
    sf = qn;
}

// Several quads a thread (larger lattices, two copies): quad tid + i *
// threads in row-major order, i < kSlots = ceil(quads / threads).  Threads
// past the last quad repeat it; a wave with no quad in the last slot skips it.
constexpr int kWholeSlots = 5; // at most (L = 280 has 4900 quads)

template <int kSlots>
struct WholeSlots {
    bool full;            // the wave has quads in the last slot (uniform)
    uint32_t pa[kSlots];  // LDS offset of the top row for oy = 0
    uint32_t pd[kSlots];  // of the bottom row for oy = 1 (wrapped)
    uint32_t side[kSlots]; // offsets to the dwords before (low half) and
                           // after (high half) a row's word, wrapped
    uint32_t c0[kSlots];  // Philox counter word
    PatchList<1> swap;    // selectors of the partial quad
};

template <int kSlots>
__device__ inline WholeSlots<kSlots> whole_slots(const WholeGeom &G,
                                                 uint32_t threads)
{
    const uint32_t Q = G.Q(), Lb = G.L >> 1, nq = Lb * Q;
    WholeSlots<kSlots> W;
    W.full = (threadIdx.x & ~63u) + (kSlots - 1) * threads < nq;
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kSlots; ++i) {
        const uint32_t q = min(threadIdx.x + i * threads, nq - 1u);
        const uint32_t row = q / Q, col = q - row * Q;
        W.pa[i] = 2 * row * G.LS + 8 * col;
        W.pd[i] = row + 1 == Lb ? 8 * col : W.pa[i] + 2 * G.LS;
        const uint32_t left = col == 0 ? G.LS - 4 : 0u - 4u;
        const uint32_t right = col + 1 == Q ? 8 - G.LS : 8u;
        W.side[i] = (left & 0xFFFFu) | right << 16;
        W.c0[i] = q;
    }
    patch_swap_selectors(G.part(), W.swap);
    return W;
}

// One pass from `src` (shift kSrcOdd) to `dst` (shift kOdd), slot by slot as
// patch_pass_slots.
template <bool kOdd, bool kSrcOdd, int kSlots, class Ctx>
__device__ __forceinline__ void whole_pass_slots(
    const uint8_t *src, uint8_t *dst, const WholeGeom &G,
    WholeSlots<kSlots> &W, bool oy, PassIndex ix, PassIndex nx,
    uint32_t replica, uint32_t k0, uint32_t k1, const Ctx &qc, Words &rf,
    QuadSel &sf)
{
    const bool seam = kOdd && G.part() != 0;
    const auto draw = [&](uint32_t i, PassIndex at) {
        return philox(W.c0[i], at.t, (kTagPass << 8) | at.p, replica, k0, k1);
    };
    const auto top = [&](uint32_t i) { return W.pa[i] + (oy ? G.LS : 0u); };
    const auto bottom = [&](uint32_t i) {
        return oy ? W.pd[i] : W.pa[i] + G.LS;
    };
    const auto load = [&](uint32_t i) {
        return load_window<kOdd, kSrcOdd>(src, top(i), bottom(i),
                                          (int16_t)W.side[i],
                                          (int32_t)W.side[i] >> 16);
    };
    const auto update = [&](uint32_t i, QuadRows &q, const Words &r,
                            const QuadSel &qs) {
        if (seam) {
            W.swap.part[0] = (int32_t)W.side[i] >> 16 != 8;
            patch_swap(q.a0, q.a1, W.swap, 0);
            patch_swap(q.c0, q.c1, W.swap, 0);
        }
        quad_update_sel(q.a0, q.a1, q.c0, q.c1, r, qs, qc);
        if (seam) {
            patch_swap(q.a0, q.a1, W.swap, 0);
            patch_swap(q.c0, q.c1, W.swap, 0);
        }
        *reinterpret_cast<uint2 *>(dst + top(i)) = make_uint2(q.a0, q.a1);
        *reinterpret_cast<uint2 *>(dst + bottom(i)) = make_uint2(q.c0, q.c1);
    };
    Words r[kSlots + 1];
    QuadSel qs[kSlots + 1];
    r[0] = rf;
    qs[0] = sf;
    constexpr uint32_t n = kSlots == 1 ? 1 : kSlots - 1; // common slots
#pragma unroll
    for (uint32_t i = 0; i < n; ++i) {
        QuadRows q = load(i);
        r[i + 1] = i + 1 == n ? draw(0, nx) : draw(i + 1, ix);
        qs[i + 1] = quad_sel(r[i + 1], qc);
        if (kSlots > 1 || W.full)
            update(i, q, r[i], qs[i]);
    }
    if (kSlots > 1 && W.full) {
        QuadRows q = load(kSlots - 1);
        const Words w = draw(kSlots - 1, ix);
        update(kSlots - 1, q, w, quad_sel(w, qc));
    }
    rf = r[n];
    sf = qs[n];
}

// The pass with offsets w from (src, shift s).
template <int kSlots, class Ctx>
__device__ __forceinline__ void whole_pass_slots(
    const uint8_t *src, uint8_t *dst, uint32_t s, const WholeGeom &G,
    WholeSlots<kSlots> &W, uint32_t w, PassIndex ix, PassIndex nx,
    uint32_t replica, uint32_t k0, uint32_t k1, const Ctx &qc, Words &rf,
    QuadSel &sf)
{
    const bool oy = w & 2u;
#define ESCG_PASS(O, S)                                                       \
    whole_pass_slots<O, S, kSlots>(src, dst, G, W, oy, ix, nx, replica, k0,   \
                                   k1, qc, rf, sf)
    if (w & 1u)
        s ? ESCG_PASS(true, true) : ESCG_PASS(true, false);
    else
        s ? ESCG_PASS(false, true) : ESCG_PASS(false, false);
#undef ESCG_PASS
}

// MCS from the test of the stop condition after MCS t to the next one.  A
// species that is extinct stays extinct, so a condition that holds at a test
// has held since some MCS after the last test: the job goes back to the state
// of that test (kept in its lattice's place in global memory) and tests after
// every MCS.  Up to t = 128 every MCS is tested and no state is kept: a test
// takes 0.3 to 0.5 us of an MCS's 2 to 10 (pair_stop), the copy of the state
// 2.8 at L = 206.  So a stop up to 128 costs no MCS more, one past it at most an
// eighth.
// Batches that stop after 25 MCS (64 of L = 256, 512 of L = 192, 16 of L = 8),
// us: first test after 32 MCS 1048, 3177, 349; in-place kernel, which tests
// after every MCS, 775, 2463, 225; now 639, 2470, 194.
__host__ __device__ inline uint32_t pair_window(uint32_t t)
{
    return t < 128u ? 1u : min(32u, t / 8u);
}

// Loads the lattice (shift 0) into `buf`, which holds zeros.
__device__ inline void whole_load(uint8_t *buf, const uint8_t *g,
                                  const WholeGeom &G)
{
    const uint32_t L = G.L;
    if ((L & 3u) == 0) {
        const uint32_t dwr = L >> 2;
        const uint32_t *g32 = reinterpret_cast<const uint32_t *>(g);
        for (uint32_t i = threadIdx.x; i < L * dwr; i += blockDim.x)
            *reinterpret_cast<uint32_t *>(buf + (i / dwr) * G.LS +
                                          4 * (i % dwr)) = g32[i];
    } else {
        const uint32_t hr = L >> 1;
        const uint16_t *g16 = reinterpret_cast<const uint16_t *>(g);
        for (uint32_t i = threadIdx.x; i < L * hr; i += blockDim.x)
            *reinterpret_cast<uint16_t *>(buf + (i / hr) * G.LS +
                                          2 * (i % hr)) = g16[i];
    }
}

// Writes the columns of quad j, row r of a copy `buf` of shift s to the
// lattice: with shift 1 the word is one column ahead, so its first column is
// the last byte of the word before (of the row's last word for j = 0).
__device__ __forceinline__ void whole_store_word(const uint8_t *buf,
                                                 uint32_t s, uint32_t r,
                                                 uint32_t j, uint8_t *g,
                                                 const WholeGeom &G)
{
    const uint8_t *row = buf + r * G.LS;
    uint2 v = *reinterpret_cast<const uint2 *>(row + 8 * j);
    if (s) {
        const uint32_t y = row[j == 0 ? G.LS - 1 : 8 * j - 1];
        v.y = __builtin_amdgcn_alignbyte(v.y, v.x, 3);
        v.x = (v.x << 8) | y;
    }
    const uint32_t nb = G.part() && j + 1 == G.Q() ? G.part() : 4u;
    store_quad_row(g + (size_t)r * G.L + 8 * j, v, nb, G.L);
}

// The counting wave: words lane + 64 k of the lattice, kWholeStage of them a
// lane in each of three stages.
constexpr uint32_t kWholeStage = 6;

__device__ __forceinline__ uint2 whole_word(const uint8_t *buf, uint32_t n,
                                            uint32_t k)
{
    const uint32_t i = (threadIdx.x & 63u) + 64 * k;
    return 64 * k < n && i < n
               ? *reinterpret_cast<const uint2 *>(buf + 8 * i)
               : make_uint2(0u, 0u);
}

// Adds the linear sums of a lane's words of `stage` to `pair` (two 16-bit
// sums a dword, as patch_word_sums; n words in all; over a wave they stay
// below 64 * 18 * 8 * 7 < 2^16).
template <int NS>
__device__ __forceinline__ void whole_word_sums(const uint8_t *buf, uint32_t n,
                                                uint32_t stage,
                                                uint32_t (&pair)[NS / 2])
{
    constexpr int NP = (NS - 2) / 2;
    static_assert(kWholeStage <= 7, "a nibble holds 7 words' counts");
    uint32_t sv = 0, cp[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k)
        cp[k] = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWholeStage; ++w) {
        const uint2 v = whole_word(buf, n, stage * kWholeStage + w);
        sv += v.x + v.y;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const uint64_t t = pair_code_table(k);
            const uint32_t hi = (uint32_t)(t >> 32), lo = (uint32_t)t;
            cp[k] += perm(hi, lo, v.x) + perm(hi, lo, v.y);
        }
    }
#pragma unroll
    for (int k = 0; k < NP; ++k)
        pair[k] += __builtin_amdgcn_udot8(cp[k], 0x01010101u, 0u, false) |
                   __builtin_amdgcn_udot8(cp[k], 0x10101010u, 0u, false) << 16;
    pair[NP] = __builtin_amdgcn_udot4(sv, 0x01010101u, pair[NP], false);
}

// Adds a lane's words of `stage` to the histogram (S > 7; gap bytes count as
// zeros).
__device__ __forceinline__ void whole_hist(const uint8_t *buf, uint32_t n,
                                           uint32_t stage, uint32_t *hist)
{
    uint32_t *const h = hist + (threadIdx.x & (kCountSlots - 1));
    for (uint32_t w = 0; w < kWholeStage; ++w) {
        const uint32_t i =
            (threadIdx.x & 63u) + 64 * (stage * kWholeStage + w);
        if (i < n)
            patch_hist_word(*reinterpret_cast<const uint2 *>(buf + 8 * i), h);
    }
}

} // namespace escg
