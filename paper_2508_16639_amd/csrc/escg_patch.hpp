// escg_patch.hpp -- phases of the patch kernel: a lattice of any even side
// cut into uneven patches, several MCS between two halo exchanges.
//
// What bounds it.  Up to a few thousand sites per compute unit an MCS is not
// bound by work but by latency: four dependent passes (row read, rule
// lookup, store, barrier) and the round trip of the halo exchange, 1.5 to
// 2 us through memory.  So a patch keeps a halo of 4 K rows above and below
// and of HQ quads (8 columns each, 8 HQ > 4 K) left and right, runs K MCS on
// its region redundantly and exchanges halos once per K MCS.
//
// Cuts.  Block rows are cut into PY parts and quad columns (a quad: the four
// blocks of one Philox call, 8 columns; ceil(L / 8) of them per row) into PX
// parts, each as even as possible, so any even L gets patches of equal size
// up to one block row and one quad.  When L % 8 != 0 the row's last quad has
// only `part` = 1..3 blocks.  It takes 8 bytes in LDS like any other, the
// bytes past its columns (its gap) being 0: an update of two equal sites
// changes nothing, so the gap stays 0 through blocks that do not exist.  Only
// in a pass with odd column offset its window needs care: the first column
// of the next quad belongs into its last block instead of behind the gap, so
// two bytes of the window change places before and after the update
// (patch_pass, kOdd).  The quads are numbered from `rot` on, so that the
// partial quad lies inside patch column 0, never in a halo.
//
// Two buffers.  A pass reads one copy of the region and writes the other, in
// which its own windows are 8-byte aligned: with column offset ox, byte b of
// a row holds column b + ox (the copy's shift).  Every store is then one
// aligned 8-byte word per row, a pass needs one barrier, and the species
// counts of an MCS read the copy that the next pass reads, beside that pass.
// Blocks move information by one cell per pass, so after n passes the cells
// within n of the region's edge are stale (as are the few that a pass does
// not cover); 4 K rows and 8 HQ >= 4 K + 1 columns (one more for the shift)
// keep the interior exact.  With shift 1 a patch counts, publishes and
// receives the columns one to the right of its own: all patches have the
// same shift, so those domains tile the lattice as well.
//
// Measured, us per MCS with counts, before / now.  L % 8 == 0, before: equal
// tiles, an exchange every MCS: L = 200 4.1 / 1.9, 512 3.6 / 1.9, 1600 7.2 /
// 4.2, 3200 8.6 / 8.1; S = 8 with probabilities at 400: 6.9 / 2.9.  L % 8 != 0,
// before: the lattice in one LDS or a launch per MCS: 300 40 / 2.1, 500 26 /
// 2.1.  Up to L = 1000 or so latency is left (0.3 us a pass, 1 us an
// exchange), from 2000 on vector issue: 22.1 lane-instructions per site update
// at L = 3200 (15 of them the update itself, the halo's share most of the
// rest), 72 % of the issue slots.
#pragma once

#include "escg_tile.hpp"

namespace escg {

struct PatchGeom {
    uint32_t L, PY, PX;
    uint32_t K;          // MCS between halo exchanges
    uint32_t HQ;         // halo quads left and right, 8 HQ >= 4 K + 1
    uint32_t rot;        // global quad of rotated quad 0
    uint32_t slot_words; // 64-bit words of one patch's exchange slot
    uint32_t rq, rr, cq, cr; // Lb / PY, Lb % PY, Q / PX, Q % PX (set_cuts)

    __host__ __device__ uint32_t Lb() const { return L >> 1; }
    __host__ __device__ uint32_t Q() const { return ((L >> 1) + 3) >> 2; }
    // blocks of the row's last quad (0: four)
    __host__ __device__ uint32_t part() const { return (L >> 1) & 3u; }
    __host__ __device__ uint32_t HR() const { return 4 * K; }
    // the first parts of a cut are one longer than the others
    __host__ __device__ uint32_t row_cut(uint32_t i) const // block rows
    {
        return i * rq + (i < rr ? i : rr);
    }
    __host__ __device__ uint32_t col_cut(uint32_t j) const // rotated quads
    {
        return j * cq + (j < cr ? j : cr);
    }
    // after L, PY and PX: the cuts, and the partial quad into the middle of
    // patch column 0
    __host__ __device__ void set_cuts()
    {
        rq = Lb() / PY;
        rr = Lb() % PY;
        cq = Q() / PX;
        cr = Q() % PX;
        rot = part() ? (2 * Q() - 1 - col_cut(1) / 2) % Q() : 0u;
    }
};

// One patch (wave-uniform).
struct Patch {
    uint32_t py, px;
    uint32_t b0, TH; // first block row, interior rows
    uint32_t c0, TQ; // first rotated quad, interior quads
    uint32_t RH, NJ; // region rows and quads per row
    uint32_t LS;     // LDS row stride: 8 NJ and one spare word (always 0)
    uint32_t seam;   // region quad column of the partial quad, or ~0
};

__host__ __device__ inline Patch patch_at(const PatchGeom &G, uint32_t py,
                                          uint32_t px)
{
    Patch P;
    P.py = py;
    P.px = px;
    P.b0 = G.row_cut(P.py);
    P.TH = 2 * (G.row_cut(P.py + 1) - P.b0);
    P.c0 = G.col_cut(P.px);
    P.TQ = G.col_cut(P.px + 1) - P.c0;
    P.RH = P.TH + 2 * G.HR();
    P.NJ = P.TQ + 2 * G.HQ;
    P.LS = 8 * P.NJ + 8;
    P.seam = ~0u;
    if (G.part()) { // G.rot < Q: the partial quad's rotated number
        const uint32_t at = G.Q() - 1 - G.rot;
        if (at >= P.c0 && at < P.c0 + P.TQ)
            P.seam = G.HQ + at - P.c0;
    }
    return P;
}

__host__ __device__ inline Patch patch_of(const PatchGeom &G, uint32_t idx)
{
    return patch_at(G, idx / G.PX, idx % G.PX);
}

// Bytes of one copy of the largest region: a spare word before the first row
// (read as the column before a quad), one after each row and a spare row.
__host__ __device__ inline uint32_t patch_buffer_bytes(const PatchGeom &G)
{
    const uint32_t TH = 2 * G.row_cut(1), TQ = G.col_cut(1);
    return (TH + 2 * G.HR() + 1) * (8 * (TQ + 2 * G.HQ) + 8) + 8;
}

// The first 2 nb columns of a quad's row at s, the other bytes 0 (rows of
// side L are 4-byte aligned when L % 4 == 0, where nb is 2 or 4, and 2-byte
// otherwise).
__device__ __forceinline__ uint2 load_quad_row(const uint8_t *s, uint32_t nb,
                                               uint32_t L)
{
    uint2 v = make_uint2(0u, 0u);
    if ((L & 3u) == 0) {
        const uint32_t *s4 = reinterpret_cast<const uint32_t *>(s);
        v.x = s4[0];
        if (nb > 2)
            v.y = s4[1];
    } else {
        const uint16_t *s2 = reinterpret_cast<const uint16_t *>(s);
        v.x = s2[0];
        if (nb > 1)
            v.x |= (uint32_t)s2[1] << 16;
        if (nb > 2)
            v.y = s2[2];
        if (nb > 3)
            v.y |= (uint32_t)s2[3] << 16;
    }
    return v;
}

// Loads the region (shift 0) into `buf` from the global lattice (4-byte
// aligned, so rows are 4-byte aligned when L % 4 == 0 and 2-byte otherwise);
// gap bytes become 0.  (row, quad) advance with a carry: one division a
// thread, and the loop's loads can be in flight together.
__device__ inline void patch_load(uint8_t *buf, const uint8_t *g,
                                  const PatchGeom &G, const Patch &P)
{
    const uint32_t L = G.L, Q = G.Q(), HR = G.HR();
    const uint32_t r0 = (2 * P.b0 + 4 * L - HR % L) % L;
    const uint32_t qa = (G.rot + P.c0 + 4 * Q - G.HQ) % Q;
    const uint32_t last = G.part() ? G.part() : 4u;
    uint32_t r = threadIdx.x / P.NJ, j = threadIdx.x - r * P.NJ;
    const uint32_t dr = blockDim.x / P.NJ, dj = blockDim.x - dr * P.NJ;
    const uint32_t n = P.RH * P.NJ;
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        uint32_t gr = r0 + r; // < L + RH, and RH <= 3 L
        gr = min(gr, gr - L);
        gr = min(gr, gr - L);
        gr = min(gr, gr - L);
        uint32_t q = qa + j; // NJ <= 3 Q
        q = min(q, q - Q);
        q = min(q, q - Q);
        q = min(q, q - Q);
        const uint32_t nb = q == Q - 1 ? last : 4u;
        *reinterpret_cast<uint2 *>(buf + r * P.LS + 8 * j) =
            load_quad_row(g + (size_t)gr * L + 8 * q, nb, L);
        j += dj;
        r += dr;
        if (j >= P.NJ) {
            j -= P.NJ;
            ++r;
        }
    }
}

// Stores the first 2 nb columns of a quad's row v to d (rows of side L are
// 4-byte aligned when L % 4 == 0, where nb is 2 or 4, and 2-byte otherwise).
__device__ __forceinline__ void store_quad_row(uint8_t *d, uint2 v,
                                               uint32_t nb, uint32_t L)
{
    if ((L & 3u) == 0) {
        uint32_t *d4 = reinterpret_cast<uint32_t *>(d);
        d4[0] = v.x;
        if (nb > 2)
            d4[1] = v.y;
    } else {
        uint16_t *d2 = reinterpret_cast<uint16_t *>(d);
        d2[0] = (uint16_t)v.x;
        if (nb > 1)
            d2[1] = (uint16_t)(v.x >> 16);
        if (nb > 2)
            d2[2] = (uint16_t)v.y;
        if (nb > 3)
            d2[3] = (uint16_t)(v.y >> 16);
    }
}

// Stores the interior columns from the copy `buf` of shift s: column 8 j of
// the region is byte 8 j - s (the column before a quad's first byte is the
// last byte of the quad before it, the partial one included).
__device__ inline void patch_store(const uint8_t *buf, uint32_t s, uint8_t *g,
                                   const PatchGeom &G, const Patch &P,
                                   uint32_t threads)
{
    const uint32_t L = G.L, Q = G.Q(), HR = G.HR();
    const uint32_t last = G.part() ? G.part() : 4u;
    uint32_t r = threadIdx.x / P.TQ, j = threadIdx.x - r * P.TQ;
    const uint32_t dr = threads / P.TQ, dj = threads - dr * P.TQ;
    for (uint32_t i = threadIdx.x; i < P.TH * P.TQ; i += threads) {
        uint32_t q = G.rot + P.c0 + j;
        q = min(q, q - Q);
        const uint32_t nb = q == Q - 1 ? last : 4u;
        const uint8_t *p = buf + (HR + r) * P.LS + 8 * (G.HQ + j);
        uint2 v = *reinterpret_cast<const uint2 *>(p);
        if (s) {
            const uint32_t y = p[-1];
            v.y = __builtin_amdgcn_alignbyte(v.y, v.x, 3);
            v.x = (v.x << 8) | y;
        }
        store_quad_row(g + (size_t)(2 * P.b0 + r) * L + 8 * q, v, nb, L);
        j += dj;
        r += dr;
        if (j >= P.TQ) {
            j -= P.TQ;
            ++r;
        }
    }
}

// A thread's quads, fixed for the run: quad tid + i * threads in row-major
// order over (region block row, quad column), i < kSlots.  Lanes past the
// last quad repeat it (they store the same bytes), so that a pass needs no
// lane masks; a wave with no quad in the last slot skips it.  A pass with
// row offset 1 updates the last block row too, with the spare row below the
// region: both rows are stale then in any case.
template <int kSlots>
struct PatchList {
    uint32_t pa[kSlots]; // LDS offset of the top row for oy = 0
    uint32_t c0[kSlots]; // Philox counter word
    bool part[kSlots];   // the row's partial quad
    uint32_t n;          // slots this wave fills (uniform)
    uint32_t sa, sb;     // selectors that swap two bytes of its odd window
};

// Byte 7 of a partial quad's window changes places with byte 2 part - 1.
template <int kSlots>
__device__ inline void patch_swap_selectors(uint32_t part,
                                            PatchList<kSlots> &T)
{
    T.sa = part == 1 ? 0x03020700u : part == 2 ? 0x07020100u : 0x03020100u;
    T.sb = part == 1 ? 0x01060504u : part == 2 ? 0x03060504u : 0x05060704u;
}

template <int kSlots>
__device__ inline PatchList<kSlots> patch_list(const PatchGeom &G,
                                               const Patch &P,
                                               uint32_t threads)
{
    const uint32_t Q = G.Q(), Lb = G.Lb();
    const uint32_t by = (P.b0 + 4 * Lb - (G.HR() >> 1) % Lb) % Lb;
    const uint32_t qa = (G.rot + P.c0 + 4 * Q - G.HQ) % Q;
    const uint32_t nq = (P.RH >> 1) * P.NJ;
    PatchList<kSlots> T;
    patch_swap_selectors(G.part(), T);
    T.n = 0;
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kSlots; ++i) {
        const uint32_t first = (threadIdx.x & ~63u) + i * threads;
        T.n += first < nq ? 1u : 0u;
        const uint32_t q = min(threadIdx.x + i * threads, nq - 1u);
        const uint32_t row = q / P.NJ, col = q - row * P.NJ;
        T.pa[i] = 2 * row * P.LS + 8 * col;
        T.c0[i] = ((by + row) % Lb) * Q + (qa + col) % Q;
        T.part[i] = col == P.seam;
    }
    T.n = __builtin_amdgcn_readfirstlane(T.n);
    return T;
}

// Where a pass stands in the run: MCS index and pass, for the counter words.
struct PassIndex {
    uint32_t t, p;
};

// The partial quad's odd window, before and after its update.
template <int kSlots>
__device__ __forceinline__ void patch_swap(uint32_t &x0, uint32_t &x1,
                                           const PatchList<kSlots> &T, int i)
{
    const uint32_t y0 = perm(x1, x0, T.sa), y1 = perm(x1, x0, T.sb);
    x0 = T.part[i] ? y0 : x0;
    x1 = T.part[i] ? y1 : x1;
}

// One quad per thread (small regions, bound by latency): one pass of the
// region from `src` (shift s) to `dst` (shift ox), straight-line code for
// every offset and shift.  A window starts ox - s = -1, 0 or 1 bytes from the
// aligned word, so it is cut from three dwords with a uniform byte shift;
// four versions of the pass, one per (ox, s), measured 25 % slower, since the
// compiler joins their ends and with them puts the selector lookups off
// until just before the barrier.  (rf, sf): Philox words and selector pairs,
// computed during the pass before; the pass leaves those of pass `nx`, drawn
// while its rows are on their way from LDS.
template <bool kSeam, class Ctx>
__device__ __forceinline__ void patch_pass(const uint8_t *src, uint8_t *dst,
                                           uint32_t s, const Patch &P,
                                           const PatchList<1> &T, uint32_t w,
                                           PassIndex, PassIndex nx,
                                           uint32_t replica, uint32_t k0,
                                           uint32_t k1, const Ctx &qc,
                                           Words &rf, QuadSel &sf)
{
    const uint32_t ox = w & 1u, pa = T.pa[0] + ((w & 2u) ? P.LS : 0u);
    const uint32_t sh = (ox - s) & 3u; // 3: one byte left
    const uint8_t *qa = src + pa - (sh & 2u) * 2u, *qb = qa + P.LS;
    uint32_t d[3], e[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        d[k] = reinterpret_cast<const uint32_t *>(qa)[k];
        e[k] = reinterpret_cast<const uint32_t *>(qb)[k];
    }
    const Words rn =
        philox(T.c0[0], nx.t, (kTagPass << 8) | nx.p, replica, k0, k1);
    const QuadSel qn = quad_sel(rn, qc);
    uint32_t a0 = __builtin_amdgcn_alignbyte(d[1], d[0], sh);
    uint32_t a1 = __builtin_amdgcn_alignbyte(d[2], d[1], sh);
    uint32_t c0 = __builtin_amdgcn_alignbyte(e[1], e[0], sh);
    uint32_t c1 = __builtin_amdgcn_alignbyte(e[2], e[1], sh);
    if (kSeam && ox) {
        patch_swap(a0, a1, T, 0);
        patch_swap(c0, c1, T, 0);
    }
    quad_update_sel(a0, a1, c0, c1, rf, sf, qc);
    if (kSeam && ox) {
        patch_swap(a0, a1, T, 0);
        patch_swap(c0, c1, T, 0);
    }
    *reinterpret_cast<uint2 *>(dst + pa) = make_uint2(a0, a1);
    *reinterpret_cast<uint2 *>(dst + pa + P.LS) = make_uint2(c0, c1);
    rf = rn;
    sf = qn;
}

// The window of a quad whose aligned word is at `pa` (top row) and `pc`, from
// a copy of shift kSrcOdd, for a pass with column offset kOdd: aligned, or one
// byte to the right or left of the aligned word; right / left: offsets to the
// byte after and to the dword before the word.
template <bool kOdd, bool kSrcOdd>
__device__ __forceinline__ QuadRows load_window(const uint8_t *src,
                                                uint32_t pa, uint32_t pc,
                                                int32_t left = -4,
                                                int32_t right = 8)
{
    const uint2 ra = *reinterpret_cast<const uint2 *>(src + pa);
    const uint2 rc = *reinterpret_cast<const uint2 *>(src + pc);
    if (kOdd == kSrcOdd)
        return QuadRows{ra.x, ra.y, rc.x, rc.y};
    if (kOdd) {
        const uint32_t xa = src[(int32_t)pa + right],
                       xc = src[(int32_t)pc + right];
        return QuadRows{__builtin_amdgcn_alignbyte(ra.y, ra.x, 1),
                        __builtin_amdgcn_alignbyte(xa, ra.y, 1),
                        __builtin_amdgcn_alignbyte(rc.y, rc.x, 1),
                        __builtin_amdgcn_alignbyte(xc, rc.y, 1)};
    }
    const uint32_t xa =
        *reinterpret_cast<const uint32_t *>(src + ((int32_t)pa + left));
    const uint32_t xc =
        *reinterpret_cast<const uint32_t *>(src + ((int32_t)pc + left));
    return QuadRows{__builtin_amdgcn_alignbyte(ra.x, xa, 3),
                    __builtin_amdgcn_alignbyte(ra.y, ra.x, 3),
                    __builtin_amdgcn_alignbyte(rc.x, xc, 3),
                    __builtin_amdgcn_alignbyte(rc.y, rc.x, 3)};
}

// Several quads per thread: the pass for one (ox, s), which needs fewer LDS
// reads and no byte shift when ox = s; dy: oy * LS.  Every wave runs the
// first kSlots - 1 slots (a wave with fewer repeats its last quad), so that
// they are straight-line code, each slot's draws made before the slot before
// it is updated and the next pass's first ones before the last of them; the
// last slot is one block of its own for the waves that fill it.  (With a test
// per slot the draws handed from slot to slot cost 13 v_mov of 76
// instructions a quad, 3 % of the time at L = 3200.)
template <bool kOdd, bool kSrcOdd, bool kSeam, int kSlots, class Ctx>
__device__ __forceinline__ void patch_pass_slots(
    const uint8_t *src, uint8_t *dst, uint32_t LS, uint32_t dy,
    const PatchList<kSlots> &T, PassIndex ix, PassIndex nx, uint32_t replica,
    uint32_t k0, uint32_t k1, const Ctx &qc, Words &rf, QuadSel &sf)
{
    const auto draw = [&](uint32_t i, PassIndex at) {
        return philox(T.c0[i], at.t, (kTagPass << 8) | at.p, replica, k0, k1);
    };
    const auto update = [&](uint32_t i, QuadRows &q, const Words &r,
                            const QuadSel &qs) {
        if (kOdd && kSeam) {
            patch_swap(q.a0, q.a1, T, i);
            patch_swap(q.c0, q.c1, T, i);
        }
        quad_update_sel(q.a0, q.a1, q.c0, q.c1, r, qs, qc);
        if (kOdd && kSeam) {
            patch_swap(q.a0, q.a1, T, i);
            patch_swap(q.c0, q.c1, T, i);
        }
        const uint32_t pa = T.pa[i] + dy;
        *reinterpret_cast<uint2 *>(dst + pa) = make_uint2(q.a0, q.a1);
        *reinterpret_cast<uint2 *>(dst + pa + LS) = make_uint2(q.c0, q.c1);
    };
    Words r[kSlots];
    QuadSel qs[kSlots];
    r[0] = rf;
    qs[0] = sf;
#pragma unroll
    for (uint32_t i = 0; i + 1 < (uint32_t)kSlots; ++i) {
        const uint32_t pa = T.pa[i] + dy;
        QuadRows q = load_window<kOdd, kSrcOdd>(src, pa, pa + LS);
        const bool last = i + 2 == (uint32_t)kSlots;
        r[i + 1] = last ? draw(0, nx) : draw(i + 1, ix);
        qs[i + 1] = quad_sel(r[i + 1], qc);
        update(i, q, r[i], qs[i]);
    }
    if (T.n == (uint32_t)kSlots) {
        const uint32_t i = kSlots - 1, pa = T.pa[i] + dy;
        QuadRows q = load_window<kOdd, kSrcOdd>(src, pa, pa + LS);
        const Words w = draw(i, ix);
        update(i, q, w, quad_sel(w, qc));
    }
    rf = r[kSlots - 1];
    sf = qs[kSlots - 1];
}

template <bool kSeam, int kSlots, class Ctx>
__device__ __forceinline__ void patch_pass(const uint8_t *src, uint8_t *dst,
                                           uint32_t s, const Patch &P,
                                           const PatchList<kSlots> &T,
                                           uint32_t w, PassIndex ix,
                                           PassIndex nx, uint32_t replica,
                                           uint32_t k0, uint32_t k1,
                                           const Ctx &qc, Words &rf,
                                           QuadSel &sf)
{
    const uint32_t dy = (w & 2u) ? P.LS : 0u;
#define ESCG_PASS(O, S)                                                       \
    patch_pass_slots<O, S, kSeam, kSlots>(src, dst, P.LS, dy, T, ix, nx,      \
                                          replica, k0, k1, qc, rf, sf)
    if (w & 1u)
        s ? ESCG_PASS(true, true) : ESCG_PASS(true, false);
    else
        s ? ESCG_PASS(false, true) : ESCG_PASS(false, false);
#undef ESCG_PASS
}

// ---------------------------------------------------------------------------
// One patch after the other in a workgroup (patch sweep): a thread's quads,
// by their region block row and column, stay the same while the patch column
// does, so a patch costs some hundred instructions a wave besides its passes
// (with patch_list and patch_load for each patch, 800: as many as one MCS).
// Every region has the rows of the tallest, RH; a shorter patch's last rows
// only feed each other.
// ---------------------------------------------------------------------------
template <int kSlots>
struct SweepQuads {
    PatchList<kSlots> T;
    uint32_t row[kSlots], col[kSlots];
};

template <int kSlots>
__device__ inline void sweep_column(const PatchGeom &G, const Patch &P,
                                    uint32_t RH, uint32_t threads,
                                    SweepQuads<kSlots> &W)
{
    const uint32_t nq = (RH >> 1) * P.NJ;
    patch_swap_selectors(G.part(), W.T);
    W.T.n = 0;
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kSlots; ++i) {
        const uint32_t first = (threadIdx.x & ~63u) + i * threads;
        W.T.n += first < nq ? 1u : 0u;
        const uint32_t q = min(threadIdx.x + i * threads, nq - 1u);
        W.row[i] = q / P.NJ;
        W.col[i] = q - W.row[i] * P.NJ;
        W.T.pa[i] = 2 * W.row[i] * P.LS + 8 * W.col[i];
        W.T.part[i] = W.col[i] == P.seam;
    }
    W.T.n = __builtin_amdgcn_readfirstlane(W.T.n);
}

// Counter words of the patch's quads, and its region into `buf` (shift 0).
template <int kSlots>
__device__ __forceinline__ void sweep_load(uint8_t *buf, const uint8_t *g,
                                           const PatchGeom &G, const Patch &P,
                                           SweepQuads<kSlots> &W)
{
    const uint32_t L = G.L, Q = G.Q(), Lb = G.Lb(), hb = G.HR() >> 1;
    const uint32_t by = P.b0 >= hb ? P.b0 - hb : P.b0 + Lb - hb;
    uint32_t qa = G.rot + P.c0 + Q - G.HQ; // < 3 Q
    qa = min(qa, qa - Q);
    qa = min(qa, qa - Q);
    const uint32_t last = G.part() ? G.part() : 4u;
    uint2 v[kSlots][2];
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kSlots; ++i) {
        uint32_t b = by + W.row[i], q = qa + W.col[i];
        b = min(b, b - Lb); // by < Lb, row < 2 Lb; quads alike
        b = min(b, b - Lb);
        q = min(q, q - Q);
        q = min(q, q - Q);
        W.T.c0[i] = b * Q + q;
        const uint32_t nb = q == Q - 1 ? last : 4u;
        const uint8_t *s = g + (size_t)(2 * b) * L + 8 * q;
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h, s += L)
            v[i][h] = load_quad_row(s, nb, L);
    }
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kSlots; ++i) {
        *reinterpret_cast<uint2 *>(buf + W.T.pa[i]) = v[i][0];
        *reinterpret_cast<uint2 *>(buf + W.T.pa[i] + P.LS) = v[i][1];
    }
}

// Stores the interior from the copy `buf` of shift s (as patch_store).
template <int kSlots>
__device__ __forceinline__ void sweep_store(const uint8_t *buf, uint32_t s,
                                            uint8_t *g, const PatchGeom &G,
                                            const Patch &P,
                                            const SweepQuads<kSlots> &W)
{
    const uint32_t L = G.L, Q = G.Q(), hb = G.HR() >> 1;
    const uint32_t last = G.part() ? G.part() : 4u;
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kSlots; ++i) {
        const uint32_t b = W.row[i] - hb, j = W.col[i] - G.HQ;
        if (b >= P.TH >> 1 || j >= P.TQ) // unsigned: the halo too
            continue;
        uint32_t q = G.rot + P.c0 + j;
        q = min(q, q - Q);
        const uint32_t nb = q == Q - 1 ? last : 4u;
        uint8_t *d = g + (size_t)(2 * (P.b0 + b)) * L + 8 * q;
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h, d += L) {
            const uint8_t *p = buf + W.T.pa[i] + h * P.LS;
            uint2 v = *reinterpret_cast<const uint2 *>(p);
            if (s) {
                const uint32_t y = p[-1];
                v.y = __builtin_amdgcn_alignbyte(v.y, v.x, 3);
                v.x = (v.x << 8) | y;
            }
            store_quad_row(d, v, nb, L);
        }
    }
}

// ---------------------------------------------------------------------------
// Halo exchange: 64-bit words, every byte carrying the exchange's tag in bit
// 7 (exch_tag; slots and tags as in the tiled kernel, e counting exchanges).
// A slot holds the interior's HR top rows, its HR bottom rows, its HQ left
// and its HQ right quad columns.
// ---------------------------------------------------------------------------
__host__ __device__ inline uint32_t patch_slot_words(uint32_t TH, uint32_t TQ,
                                                     uint32_t HR, uint32_t HQ)
{
    return 2 * HR * TQ + 2 * TH * HQ;
}

__device__ __forceinline__ void xstore64(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t xload64(const uint64_t *p)
{
    return __hip_atomic_load(const_cast<uint64_t *>(p), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

// Word i of the patch's slot: its LDS offset.
__device__ inline uint32_t patch_strip_word(const PatchGeom &G,
                                            const Patch &P, uint32_t i)
{
    const uint32_t HR = G.HR(), HQ = G.HQ, rows = 2 * HR * P.TQ;
    uint32_t r, j;
    if (i < rows) {
        r = i / P.TQ;
        j = HQ + i - r * P.TQ;
        r = r < HR ? HR + r : P.TH + r - HR;
    } else {
        const uint32_t k = i - rows, side = P.TH * HQ;
        const uint32_t q = k < side ? k : k - side;
        r = q / HQ;
        j = (k < side ? HQ : P.TQ) + q - r * HQ;
        r += HR;
    }
    return r * P.LS + 8 * j;
}

// Halo word i of the region: its source (64-bit word of exchange slot 0 of
// the whole lattice) and its LDS offset.
struct PatchHaloWord {
    uint32_t src, dst;
};

__device__ inline uint32_t patch_halo_count(const PatchGeom &G,
                                            const Patch &P)
{
    return 2 * G.HR() * P.NJ + 2 * P.TH * G.HQ;
}

__device__ inline PatchHaloWord patch_halo_word(const PatchGeom &G,
                                                const Patch &P, uint32_t i)
{
    const uint32_t HR = G.HR(), HQ = G.HQ, rows = 2 * HR * P.NJ;
    const uint32_t up = (P.py + G.PY - 1) % G.PY, dn = (P.py + 1) % G.PY;
    const uint32_t lf = (P.px + G.PX - 1) % G.PX, rt = (P.px + 1) % G.PX;
    PatchHaloWord w;
    if (i < rows) { // rows above and below the interior
        uint32_t r = i / P.NJ;
        const uint32_t j = i - r * P.NJ;
        const bool above = r < HR;
        const uint32_t y = above ? up : dn;
        const uint32_t x = j < HQ ? lf : (j < HQ + P.TQ ? P.px : rt);
        const uint32_t xq = G.col_cut(x + 1) - G.col_cut(x);
        const uint32_t col = j < HQ            ? xq - HQ + j
                             : j < HQ + P.TQ ? j - HQ
                                               : j - HQ - P.TQ;
        w.dst = (above ? r : P.TH + r) * P.LS + 8 * j;
        r = above ? HR + r : r - HR; // bottom strip above, top strip below
        w.src = (y * G.PX + x) * G.slot_words + r * xq + col;
    } else { // the quads left and right of it
        const uint32_t k = i - rows, side = P.TH * HQ;
        const bool left = k < side;
        const uint32_t q = left ? k : k - side;
        const uint32_t r = q / HQ, c = q - r * HQ;
        const uint32_t x = left ? lf : rt;
        const uint32_t xq = G.col_cut(x + 1) - G.col_cut(x);
        w.dst = (HR + r) * P.LS + 8 * (left ? c : HQ + P.TQ + c);
        w.src = (P.py * G.PX + x) * G.slot_words + 2 * HR * xq +
                (left ? side : 0u) + q;
    }
    return w;
}

// A thread's first kHaloWords words of the strips it publishes and of the
// halo it gathers, fixed for the run (later ones, if any, are mapped on the
// fly, at some hundred instructions a word).
constexpr uint32_t kHaloWords = 2;

struct PatchHalo {
    uint32_t ns, n; // words of the slot, of the halo
    uint32_t strip[kHaloWords];
    PatchHaloWord w[kHaloWords];
};

__device__ inline PatchHalo patch_halo(const PatchGeom &G, const Patch &P)
{
    PatchHalo H;
    H.ns = patch_slot_words(P.TH, P.TQ, G.HR(), G.HQ);
    H.n = patch_halo_count(G, P);
#pragma unroll
    for (uint32_t k = 0; k < kHaloWords; ++k) {
        const uint32_t i = threadIdx.x + k * blockDim.x;
        H.strip[k] = patch_strip_word(G, P, i < H.ns ? i : 0u);
        H.w[k] = patch_halo_word(G, P, i < H.n ? i : 0u);
    }
    return H;
}

// Writes the interior's strips from `buf`, tagged, into the patch's slot.
__device__ inline void patch_publish(const uint8_t *buf, uint64_t *slot,
                                     const PatchHalo &H, const PatchGeom &G,
                                     const Patch &P, uint32_t tag)
{
    const uint64_t tag2 = ((uint64_t)tag << 32) | tag;
#pragma unroll
    for (uint32_t k = 0; k < kHaloWords; ++k) {
        const uint32_t i = threadIdx.x + k * blockDim.x;
        if (i < H.ns)
            xstore64(slot + i, tag2 | *reinterpret_cast<const uint64_t *>(
                                          buf + H.strip[k]));
    }
    for (uint32_t i = threadIdx.x + kHaloWords * blockDim.x; i < H.ns;
         i += blockDim.x)
        xstore64(slot + i, tag2 | *reinterpret_cast<const uint64_t *>(
                                      buf + patch_strip_word(G, P, i)));
}

// Rebuilds the halo in `buf` from exchange slot `area` (of the whole
// lattice) once its words carry `tag`; between() runs after the first loads
// are issued (every thread calls it once).  0, or 1 if another workgroup
// raised the abort word, or 2 after spin_limit polls.  A thread's two words
// are polled together.  (Two to four loads of a word in flight, one behind
// the other, measured 9 to 14 % slower on a whole MCS at L = 512, 16 x 16
// patches of K = 3, than one; a pause before the first load 1 to 7 %.)
template <class Fn>
__device__ inline uint32_t patch_gather(uint8_t *buf, const uint64_t *area,
                                        const PatchHalo &H,
                                        const PatchGeom &G, const Patch &P,
                                        uint32_t tag, const uint32_t *abort,
                                        uint32_t spin_limit, Fn &&between)
{
    const uint64_t tag2 = ((uint64_t)tag << 32) | tag;
    const uint64_t bits = 0x8000000080ull; // the tag bits that are tested
    uint64_t v[kHaloWords];
    bool need[kHaloWords];
#pragma unroll
    for (uint32_t k = 0; k < kHaloWords; ++k) {
        need[k] = threadIdx.x + k * blockDim.x < H.n;
        if (need[k])
            v[k] = xload64(area + H.w[k].src);
    }
    between();
    for (uint32_t spins = 0;;) {
#pragma unroll
        for (uint32_t k = 0; k < kHaloWords; ++k)
            if (need[k] && ((v[k] ^ tag2) & bits) == 0) {
                *reinterpret_cast<uint64_t *>(buf + H.w[k].dst) =
                    v[k] & 0x7F7F7F7F7F7F7F7Full;
                need[k] = false;
            }
        if (!need[0] && !need[1])
            break;
#pragma unroll
        for (uint32_t k = 0; k < kHaloWords; ++k)
            if (need[k])
                v[k] = xload64(area + H.w[k].src);
        if ((++spins & 63u) == 0) {
            if (xload(abort))
                return 1;
            if (spins > spin_limit)
                return 2;
        }
    }
    static_assert(kHaloWords == 2, "the loop above tests two words");
    for (uint32_t i = threadIdx.x + kHaloWords * blockDim.x; i < H.n;
         i += blockDim.x) {
        const PatchHaloWord w = patch_halo_word(G, P, i);
        uint64_t x = xload64(area + w.src);
        for (uint32_t spins = 0; (x ^ tag2) & bits;) {
            if ((++spins & 63u) == 0) {
                if (xload(abort))
                    return 1;
                if (spins > spin_limit)
                    return 2;
            }
            __builtin_amdgcn_s_sleep(1);
            x = xload64(area + w.src);
        }
        *reinterpret_cast<uint64_t *>(buf + w.dst) =
            x & 0x7F7F7F7F7F7F7F7Full;
    }
    return 0;
}

// ---------------------------------------------------------------------------
// Species counts of the interior (gap bytes are 0: they only show in the
// count of empty sites, which is taken as the rest)
// ---------------------------------------------------------------------------

// A thread's share of the interior's words, fixed for the run: one quad
// column and the rows r0, r0 + rstep, ... .
struct PatchCount {
    uint32_t p0, pstep; // LDS offset of the first word, step
    uint32_t r0, rstep;
};

__device__ inline PatchCount patch_count_plan(const PatchGeom &G,
                                              const Patch &P)
{
    PatchCount C;
    C.rstep = blockDim.x / P.TQ; // >= 1: TQ <= blockDim
    C.r0 = threadIdx.x / P.TQ;
    const uint32_t j = threadIdx.x - C.r0 * P.TQ;
    if (C.r0 >= C.rstep)
        C.r0 = P.TH; // none
    C.p0 = (G.HR() + C.r0) * P.LS + 8 * (G.HQ + j);
    C.pstep = C.rstep * P.LS;
    return C;
}

// S <= 7: NS - 1 linear sums (as tile_count_sums) into slots
// part[q * kCountSlots + lane % kCountSlots].
template <int NS>
__device__ __forceinline__ void patch_count_sums(const uint8_t *buf,
                                                 const PatchCount &C,
                                                 uint32_t TH, uint32_t *part)
{
    constexpr int NP = (NS - 2) / 2;
    if (C.r0 >= TH)
        return;
    uint32_t n[NS - 1];
#pragma unroll
    for (int q = 0; q < NS - 1; ++q)
        n[q] = 0;
    const uint8_t *p = buf + C.p0;
    uint32_t r = C.r0;
    while (r < TH) {
        uint32_t sv = 0, cp[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k)
            cp[k] = 0;
        for (uint32_t g = 0; g < 7 && r < TH; ++g) {
            const uint2 v = *reinterpret_cast<const uint2 *>(p);
            sv += v.x + v.y;
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const uint64_t t = pair_code_table(k);
                const uint32_t hi = (uint32_t)(t >> 32), lo = (uint32_t)t;
                cp[k] += perm(hi, lo, v.x) + perm(hi, lo, v.y);
            }
            r += C.rstep;
            p += C.pstep;
        }
        n[NS - 2] = __builtin_amdgcn_udot4(sv, 0x01010101u, n[NS - 2], false);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            n[2 * k] = __builtin_amdgcn_udot8(cp[k], 0x01010101u, n[2 * k],
                                              false);
            n[2 * k + 1] = __builtin_amdgcn_udot8(cp[k], 0x10101010u,
                                                  n[2 * k + 1], false);
        }
    }
    uint32_t *slot = part + (threadIdx.x & (kCountSlots - 1));
#pragma unroll
    for (int q = 0; q < NS - 1; ++q)
        atomicAdd(slot + q * kCountSlots, n[q]);
}

__device__ __forceinline__ void patch_hist_word(uint2 v, uint32_t *slot)
{
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        atomicAdd(slot + ((v.x >> (8 * k)) & 31u) * kCountSlots, 1u);
        atomicAdd(slot + ((v.y >> (8 * k)) & 31u) * kCountSlots, 1u);
    }
}

// S > 7: a histogram with kCountSlots slots per value,
// part[value * kCountSlots + lane % kCountSlots]; a wave's 64 adds meet two
// to a bank whatever the values are.
__device__ __forceinline__ void patch_count_hist(const uint8_t *buf,
                                                 const PatchCount &C,
                                                 uint32_t TH, uint32_t *part)
{
    uint32_t *slot = part + (threadIdx.x & (kCountSlots - 1));
    const uint8_t *p = buf + C.p0;
    for (uint32_t r = C.r0; r < TH; r += C.rstep, p += C.pstep) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        patch_hist_word(v, slot);
    }
}

// Counting wave.  With a small interior one wave beside those that update
// quads counts: it reads the interior's words, at most kCountWords a lane in
// two stages, while the next MCS's first pass reads them too, and adds them
// up during the passes after, so that no updating wave spends an instruction
// on counts.
constexpr uint32_t kCountStage = 7; // a nibble holds 7 words' counts
constexpr uint32_t kCountWords = 2 * kCountStage;

// LDS offsets of the counting wave's words (those past the interior: none).
struct PatchWords {
    uint32_t n; // words of the interior
    uint32_t at[kCountWords];
};

__device__ inline PatchWords patch_words(const PatchGeom &G, const Patch &P)
{
    PatchWords W;
    W.n = P.TH * P.TQ;
#pragma unroll
    for (uint32_t k = 0; k < kCountWords; ++k) {
        const uint32_t i = (threadIdx.x & 63u) + 64u * k;
        const uint32_t r = i / P.TQ, j = i - r * P.TQ;
        W.at[k] = i < W.n ? (G.HR() + r) * P.LS + 8 * (G.HQ + j) : ~0u;
    }
    return W;
}

struct PatchCounted {
    uint2 v[kCountWords];
};

__device__ __forceinline__ PatchCounted patch_read_words(const uint8_t *buf,
                                                         const PatchWords &W)
{
    PatchCounted c;
#pragma unroll
    for (uint32_t k = 0; k < kCountWords; ++k) {
        c.v[k] = make_uint2(0u, 0u);
        if (64u * k < W.n && W.at[k] != ~0u)
            c.v[k] = *reinterpret_cast<const uint2 *>(buf + W.at[k]);
    }
    return c;
}

// Adds a lane's NS - 1 linear sums of its words of `stage` to `pair`, two
// sums in a dword (over a wave each stays below 64 * 14 * 8 * 7 < 2^16).
template <int NS, uint32_t stage>
__device__ __forceinline__ void patch_word_sums(const PatchCounted &c,
                                                uint32_t (&pair)[NS / 2])
{
    constexpr int NP = (NS - 2) / 2;
    uint32_t sv = 0, cp[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k)
        cp[k] = 0;
#pragma unroll
    for (uint32_t w = stage * kCountStage; w < (stage + 1) * kCountStage;
         ++w) {
        sv += c.v[w].x + c.v[w].y;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const uint64_t t = pair_code_table(k);
            const uint32_t hi = (uint32_t)(t >> 32), lo = (uint32_t)t;
            cp[k] += perm(hi, lo, c.v[w].x) + perm(hi, lo, c.v[w].y);
        }
    }
#pragma unroll
    for (int k = 0; k < NP; ++k)
        pair[k] += __builtin_amdgcn_udot8(cp[k], 0x01010101u, 0u, false) |
                   __builtin_amdgcn_udot8(cp[k], 0x10101010u, 0u, false) << 16;
    pair[NP] = __builtin_amdgcn_udot4(sv, 0x01010101u, pair[NP], false);
}

// Dwords of one MCS's count slots.
__host__ __device__ inline uint32_t patch_count_dwords(bool packed)
{
    return (packed ? 8u : 32u) * kCountSlots;
}

// Flush of a histogram, lane l of a wave: the sum of half (l & 1) of the
// slots of value l / 2, which it clears.
__device__ __forceinline__ uint32_t patch_hist_half(uint32_t *part,
                                                    uint32_t lane)
{
    uint4 *p = reinterpret_cast<uint4 *>(part + lane * (kCountSlots / 2));
    uint32_t c = 0;
#pragma unroll
    for (uint32_t k = 0; k < kCountSlots / 8; ++k) {
        const uint4 x = p[k];
        c += x.x + x.y + x.z + x.w;
        p[k] = make_uint4(0u, 0u, 0u, 0u);
    }
    return c;
}

// The count of value l / 2 in lanes l (all 64 lanes of one wave), the slots
// cleared; gap: the interior's gap bytes, which count as zeros.
__device__ __forceinline__ uint32_t patch_hist_sum(uint32_t *part,
                                                   uint32_t lane,
                                                   uint32_t gap)
{
    uint32_t c = patch_hist_half(part, lane);
    c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xB1, 0xF, 0xF,
                                               true);
    return lane < 2 ? c - gap : c;
}

// Adds the counts in the slots of one MCS (cleared) to row[0..S]; called by
// all 64 lanes of one wave.  sites: the interior's sites; gap: its gap bytes
// (histogram only).
template <bool kPacked>
__device__ inline void patch_count_flush(uint32_t *part, uint32_t S,
                                         uint32_t sites, uint32_t gap,
                                         uint32_t *row)
{
    if constexpr (kPacked) {
        tile_count_flush(part, S, sites, row);
    } else {
        const uint32_t lane = threadIdx.x & 63u, s = lane >> 1;
        const uint32_t c = patch_hist_sum(part, lane, gap);
        if ((lane & 1u) == 0 && s <= S && c)
            atomicAdd(row + s, c);
    }
}

} // namespace escg
