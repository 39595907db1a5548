// gpp_fwd_tile.h -- the forward work of one wave tile (one or several G'
// columns x 64 consecutive G rows), shared by the plain forward and the
// persistent batched kernel so both run the same arithmetic.  See
// gpp_fwd.hip for the derivation.
#pragma once

#include <type_traits>

#include "gpp_device.h"
#include "gpp_fwd_shape.h"

namespace gpp {

// Column tiles per block of the tile walk: blocks of Q tiles of C columns go
// through all g-tiles, so that the block's aqsmtemp columns (Q * C * 16 bytes
// per band: 2 MB at 128 two-column tiles and 512 bands, half an XCD's L2) stay
// in the L2 while the g-tiles' aqsntemp rows stream past, each row fetched
// once per block.  Q is GPP_FWD_COL_BLOCK, at most twice that many columns.
// Measured with band chunks of 512 on MI355X, nfreq 3: Q = 128 took the
// HBM-side traffic of the 1024-band forward from 45.3 GB (Q = 64) to 39.1 GB
// and its time, the 512-band one's and the 64-state batched workload's down by
// 0.4-0.9 %; Q = 160 and 192 (2.5 and 3 MB) thrashed the L2 (85 and 98 GB) and
// ran slower.  At 512 bands x 32768 rows x 1638 columns, nfreq 2 (three
// columns), 128 and 85 tiles: 24.6 and 22.1 ms.  One-column tiles at 128 and
// 256: 73.0 and 72.0 ms there at nfreq 7, but 40.8 and 41.3 at 900 x 17000 x
// 900, nfreq 8.  With one frequency the rows stream by about twice as fast,
// and where their pitch is a multiple of 256 KB, so that every band meets in
// the same sets of the caches, half the tiles are better: 128 and 64 tiles 15.6
// and 14.6 ms there, 3.90 and 3.67 at 16384 rows x 819 columns; but 17.1 and
// 17.3 at 700 x 24000 x 2000, 1.68 and 1.69 at 300 x 12000 x 900.
#ifndef GPP_FWD_COL_BLOCK
#define GPP_FWD_COL_BLOCK 128
#endif
template <int NW, int C>
__device__ __forceinline__ int col_block(int ng)
{
    if (NW == 1 && ng % 16384 == 0) return GPP_FWD_COL_BLOCK / 2;
    return C > 2 ? 2 * GPP_FWD_COL_BLOCK / C : GPP_FWD_COL_BLOCK;
}

// (g-tile, column tile, band chunk) of a tile index, a bijection on
// [0, gtiles * npt * nchunk).  Within a block of Q column tiles the walk
// takes band chunk by band chunk, each through all g-tiles.  The results
// are wave-uniform and made scalar explicitly, since the divisions run on
// the vector unit and a column index left in vector registers would turn
// the tile's aqsmtemp loads into vector loads.
template <typename Int>
__device__ __forceinline__ void tile_coords_in(Int tile, int Q, int npt, int gtiles, int nchunk, int &gt,
                                               int &pt, int &ck)
{
    const Int per = (Int)Q * (Int)gtiles * (Int)nchunk;
    const int c = (int)(tile / per);
    Int r = tile - (Int)c * per;
    const int c0 = c * Q;
    const int qc = npt - c0 < Q ? npt - c0 : Q;  // the last block may be short
    const Int per_chunk = (Int)qc * (Int)gtiles;
    ck = (int)(r / per_chunk);
    r -= (Int)ck * per_chunk;
    gt = (int)(r / (Int)qc);
    pt = c0 + (int)(r - (Int)gt * (Int)qc);
}
// In 32 bits wherever a block of tiles and the tile index fit (a 64-bit
// division costs about a hundred instructions, three of them as much as the
// band loop of a few bands).
__device__ __forceinline__ void tile_coords(long tile, int Q, int npt, int gtiles, int nchunk, int &gt,
                                            int &pt, int &ck)
{
    if (tile < (1L << 31) && (long)Q * gtiles * nchunk < (1L << 31))
        tile_coords_in<uint32_t>((uint32_t)tile, Q, npt, gtiles, nchunk, gt, pt, ck);
    else
        tile_coords_in<long>(tile, Q, npt, gtiles, nchunk, gt, pt, ck);
    gt = __builtin_amdgcn_readfirstlane(gt);
    pt = __builtin_amdgcn_readfirstlane(pt);
    ck = __builtin_amdgcn_readfirstlane(ck);
}

// an conj(am) for a lane's aqsntemp value and a wave-uniform aqsmtemp
// value; the sign sits on the uniform factor, so it folds into an operand
// modifier instead of costing a vector instruction.
__device__ __forceinline__ cplx qm_of(cplx an, cplx am) {
    const double nai = -am.im;
    return cmake(fma(an.re, am.re, an.im * am.im), fma(an.im, am.re, an.re * nai));
}

// One Coulomb-hole term with denominator d and reciprocal r: P1 += r x qm
// and P2 += r qm where d > thr (branch A).  The compare writes the wave's
// execution mask (v_cmpx) around the accumulation, so a masked term adds
// nothing and no select is spent; the mask goes back to all 64 lanes, which
// every caller has active (the tile bodies run whole waves).
__device__ __forceinline__ void ch_term(double d, double thr, double r, double x, cplx qm,
                                        cplx &P1, cplx &P2) {
    double rx;
    // Not volatile: the block touches no memory and restores exec, and a
    // volatile block would count as a possible store, which keeps the
    // compiler from turning later wave-uniform loads into scalar loads.
    asm("v_cmpx_gt_f64_e32 vcc, %[d], %[thr]\n\t"
        "v_mul_f64 %[rx], %[r], %[x]\n\t"
        "v_fma_f64 %[p2r], %[r], %[qr], %[p2r]\n\t"
        "v_fma_f64 %[p2i], %[r], %[qi], %[p2i]\n\t"
        "v_fma_f64 %[p1r], %[rx], %[qr], %[p1r]\n\t"
        "v_fma_f64 %[p1i], %[rx], %[qi], %[p1i]\n\t"
        "s_mov_b64 exec, -1"
        : [rx] "=&v"(rx), [p1r] "+v"(P1.re), [p1i] "+v"(P1.im), [p2r] "+v"(P2.re),
          [p2i] "+v"(P2.im)
        : [d] "v"(d), [thr] "v"(thr), [r] "v"(r), [x] "s"(x), [qr] "v"(qm.re), [qi] "v"(qm.im)
        : "vcc");
}

// What BU consecutive bands bring into a group: a lane's aqsntemp values and
// the frequencies x (wave-uniform).  Bands at or beyond nb repeat the last
// one.
template <int NW, int BU>
struct BandGroup {
    cplx an[BU];
    double xs[BU * NW];
    // An empty use of the values: whatever was asked for up to them has
    // arrived here (loads return in order), so that a loop behind this point
    // does not start every round with a wait for its own loads.  Not volatile
    // (see ch_term).
    __device__ __forceinline__ void arrived() {
#pragma unroll
        for (int u = 0; u < BU; ++u) asm("" : "+v"(an[u].re), "+v"(an[u].im));
#pragma unroll
        for (int k = 0; k < BU * NW; ++k) asm("" : "+s"(xs[k]));
    }
    __device__ __forceinline__ void load_first(int n, int nb, int ng, gptr<double2> aqsn,
                                               uint32_t goff, gptr<double> wx) {
#pragma unroll
        for (int u = 0; u < BU; ++u) {
            const int m = n + u < nb ? n + u : nb - 1;
            an[u] = load_row_elem(aqsn + (size_t)m * ng, ng, goff);
#pragma unroll
            for (int w = 0; w < NW; ++w)
                xs[u * NW + w] = Walker{(uint64_t)(wx + (size_t)w * nb + m)}.real(0);
        }
    }
};

// Coulomb-hole sums of NC columns over the whole groups of BU bands in
// [n, n_hi), the first of them loaded in `cur`; returns the first
// band left over.  The BU*NW*NC denominators of a group share one batch
// inversion; they go in unclamped: every one is at least (Im om)^2.  Where
// a lane has a column with (Im om)^2 below kMinUnclampedWi2 the wave takes the
// NARROW form, whose denominators are at least kLimitTwo, which changes no term
// that ch_term keeps (thr is at least that), and whose reciprocals get a Newton
// step each: as good as one by one (200 bands x 8192 rows x 400 columns, all om
// real, nfreq 1, 3, 5 and 8: 500, 1231, 2001 and 3155 us with a batch and then
// each by itself in one loop for all waves, 418, 976, 1588 and 2465 so).
// Loads run ahead of their use, so that no wait sits in front of a group's
// arithmetic: the frequencies of the next group are asked for together with
// this group's aqsmtemp values, which are needed only after the reciprocals;
// the next group's aqsntemp rows are asked for once this group's have gone
// into the products.  aqsntemp[n][g] is read through a buffer descriptor of
// the row (scalar registers) plus the lane's 32-bit byte offset, so the
// address arithmetic stays on the scalar unit.
// Measured on MI355X against loads waited for in front of each group's
// arithmetic, one chain for the inversion and addresses formed per load: 512
// bands x 32768 rows x 1638 columns 33.1 -> 31.7 ms (3.97e10 -> 4.1e10
// wave-terms per second; a register-only loop of the same instructions
// reaches 4.3e10 at the part's power limit), 256 states of 32-128 bands
// 10.7 -> 10.2 ms; of that the running addresses 2.0 and 2.6 %.
template <int NW, int BU, int NC, bool NARROW>
__device__ __forceinline__ int ch_bands(int n, int n_hi, int nb, int ng, gptr<double2> aqsn,
                                        uint32_t goff, gptr<double2> aqsm, const int (&pc)[NC],
                                        gptr<double> wx, const double (&a)[NC],
                                        const double (&wi2)[NC], const double (&thr)[NC],
                                        BandGroup<NW, BU> &cur,
                                        cplx (&P1)[NC][NW], cplx (&P2)[NC][NW])
{
    constexpr int KB = BU * NW;  // terms of one column
    constexpr int K = NC * KB;
    int left = (n_hi - n) / BU;
    if (left <= 0) return n;
    n += left * BU;
    cplx (&an)[BU] = cur.an;
    double (&xs)[KB] = cur.xs;
    const uint32_t row_bytes = (uint32_t)ng * (uint32_t)sizeof(double2);
    const long step = (long)BU * row_bytes;
    uint64_t rows = (uint64_t)(aqsn + (size_t)(n - left * BU) * ng);
    Walker am_at[NC], x_at[NW];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        am_at[c].start((uint64_t)(aqsm + pc[c] + (size_t)(n - left * BU) * ng));
    // the last group asks for its own frequencies and rows again
    int more = left > 1 ? BU : 0;  // bands to the next group
#pragma unroll
    for (int w = 0; w < NW; ++w)
        x_at[w].start((uint64_t)(wx + (size_t)w * nb + (n - left * BU) + more));
    cur.arrived();
    for (;;) {
        cplx am[NC][BU];
        double xn[KB];
#pragma unroll
        for (int u = 0; u < BU; ++u) {
#pragma unroll
            for (int c = 0; c < NC; ++c) am[c][u] = am_at[c].complex(u * row_bytes);
#pragma unroll
            for (int w = 0; w < NW; ++w) xn[u * NW + w] = x_at[w].real(u);
        }
        rows += more ? step : 0;
        more = left > 2 ? BU : 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) am_at[c].advance(step);
#pragma unroll
        for (int w = 0; w < NW; ++w) x_at[w].advance(more * (long)sizeof(double));
        double d[K], r[K];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                const double dr = xs[k] - a[c];
                d[c * KB + k] = fma(dr, dr, wi2[c]);
                if constexpr (NARROW) d[c * KB + k] = fmax(d[c * KB + k], kLimitTwo);
            }
        }
        double c[K];
        const double all = batch_prefix<K>(d, c);
        batch_back<K>(d, c, all, r);
        if (__builtin_expect(batch_misses(all, 0) != 0, 0)) one_by_one<K>(d, r);
        if constexpr (NARROW) refine_in_turn<K>(d, r);
        cplx qm[NC][BU];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int u = 0; u < BU; ++u) qm[c][u] = qm_of(an[u], am[c][u]);
#pragma unroll
        for (int u = 0; u < BU; ++u) an[u] = load_elem_at(rows, u * row_bytes, goff);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int u = 0; u < BU; ++u)
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const int k = u * NW + w;
                    ch_term(d[c * KB + k], thr[c], r[c * KB + k], xs[k], qm[c][u], P1[c][w],
                            P2[c][w]);
                }
        if (--left == 0) return n;
#pragma unroll
        for (int k = 0; k < KB; ++k) xs[k] = xn[k];
    }
}

// One occupied band's values for NC columns.
template <int NW, int NC>
struct OccupiedBand {
    cplx an, am[NC];
    double x[NW];
    __device__ __forceinline__ void load(int n, int nb, int ng, gptr<double2> aqsn, uint32_t goff,
                                         gptr<double2> aqsm, const int (&pc)[NC],
                                         gptr<double> wx) {
        an = load_row_elem(aqsn + (size_t)n * ng, ng, goff);
#pragma unroll
        for (int c = 0; c < NC; ++c)
            am[c] = Walker{(uint64_t)(aqsm + pc[c] + (size_t)n * ng)}.complex(0);
#pragma unroll
        for (int w = 0; w < NW; ++w) x[w] = Walker{(uint64_t)(wx + (size_t)w * nb + n)}.real(0);
    }
};

// Both sums over an occupied band's terms K0 .. K0+G-1 (term k: column k / NW,
// frequency k % NW) of one lane: the Coulomb-hole terms over e om / 2 in HX, the
// screened-exchange ones over e om in SX.  With d = x - om, s = x + om,
// r = 1/|d|^2 and rs = 1/|s|^2 these are
//   hole      A:  1/d = conj(d) r = (Re d, Im om) r
//   exchange  A:  om/(d s) = om conj(s) rs / d,
//             B:  -1/(2 s) = -conj(s) rs / 2
// where om conj(s) = (fma(Re om, Re s, (Im om)^2), Im om x).  With BATCH one
// batch inversion, of |d|^2 |s|^2, gives every r and rs of the group, each
// refined by a Newton step of its own; `over` collects the lanes whose product
// left the range.  Otherwise each is inverted by itself, which keeps rs finite
// on an exact pole, and branch C is looked for.  Branch A's term is multiplied by
// r and rs in turn: r rs alone is below the smallest double from |x| = 1e80 on.
// The compare d > thr is the execution mask of the hole's sums and, inverted, of
// branch B's value.
template <int NW, int NC, int K0, int G, bool BATCH>
__device__ __forceinline__ void occupied_terms(const OccupiedBand<NW, NC> &band,
                                               const cplx (&om)[NC], const double (&wi2)[NC],
                                               const double (&thr)[NC], uint64_t &over,
                                               cplx (&HX)[NC][NW], cplx (&SX)[NC][NW])
{
    double d[G], r[G], rs[G];
    {
        double pr[G], ws[G], q[G], c[G];
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int i = (K0 + k) / NW;
            const double x = band.x[(K0 + k) % NW];
            const double dr = x - om[i].re, sp = x + om[i].re;
            d[k] = fma(dr, dr, wi2[i]);  // |x - om|^2, the branch's wdiffr
            ws[k] = fma(sp, sp, wi2[i]);  // |x + om|^2
            pr[k] = d[k] * ws[k];
        }
        if constexpr (BATCH) {
            const double all = batch_prefix<G>(pr, c);
            over |= batch_misses(all, 0);
            batch_back<G>(pr, c, all, q);
#pragma unroll
            for (int k = 0; k < G; ++k) {
                r[k] = q[k] * ws[k];
                rs[k] = q[k] * d[k];
            }
            refine<G>(d, r);
            refine<G>(ws, rs);
        } else {
            one_by_one<G>(d, r);
            one_by_one<G>(ws, rs);
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const int i = (K0 + k) / NW;
                const double wtr = fma(om[i].re, om[i].re, wi2[i]);
                if (!(d[k] > thr[i] || branch_b_holds(wtr, d[k]))) rs[k] = 0.0;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int i = (K0 + k) / NW, w = (K0 + k) % NW;
        const cplx qm = qm_of(band.an, band.am[i]);
        const double x = band.x[w], a = om[i].re, b = om[i].im;
        const double sp = x + a;
        const cplx h = cmake(r[k] * (x - a), r[k] * b);  // 1/d
        asm("v_cmpx_gt_f64_e32 vcc, %[d], %[thr]\n\t"
            "v_fma_f64 %[xr], %[hr], %[qr], %[xr]\n\t"
            "v_fma_f64 %[xi], %[hr], %[qi], %[xi]\n\t"
            "v_fma_f64 %[xr], -%[hi], %[qi], %[xr]\n\t"
            "v_fma_f64 %[xi], %[hi], %[qr], %[xi]\n\t"
            "s_mov_b64 exec, -1"
            : [xr] "+v"(HX[i][w].re), [xi] "+v"(HX[i][w].im)
            : [d] "v"(d[k]), [thr] "v"(thr[i]), [hr] "v"(h.re), [hi] "v"(h.im),
              [qr] "v"(qm.re), [qi] "v"(qm.im)
            : "vcc");
        cplx t = cmul(cmake(fma(a, sp, wi2[i]), b * x), h);
        asm("v_cmpx_ngt_f64_e32 vcc, %[d], %[thr]\n\t"
            "v_mul_f64 %[tr], -0.5, %[sp]\n\t"
            "v_mul_f64 %[ti], 0.5, %[b]\n\t"
            "s_mov_b64 exec, -1"
            : [tr] "+v"(t.re), [ti] "+v"(t.im)
            : [d] "v"(d[k]), [thr] "v"(thr[i]), [sp] "v"(sp), [b] "v"(b)
            : "vcc");
        cmac(SX[i][w], qm, cscale(rs[k], t));
    }
}

// Terms K0, K0 + 1, ... of a band in groups of at most G, one group's registers
// at a time.
template <int NW, int NC, int K0, int G, bool BATCH>
__device__ __forceinline__ void occupied_groups(const OccupiedBand<NW, NC> &band,
                                                const cplx (&om)[NC], const double (&wi2)[NC],
                                                const double (&thr)[NC], uint64_t &over,
                                                cplx (&HX)[NC][NW], cplx (&SX)[NC][NW])
{
    constexpr int left = NC * NW - K0;
    occupied_terms<NW, NC, K0, (left < G ? left : G), BATCH>(band, om, wi2, thr, over, HX, SX);
    if constexpr (left > G) {
        __builtin_amdgcn_sched_barrier(0);
        occupied_groups<NW, NC, K0 + G, G, BATCH>(band, om, wi2, thr, over, HX, SX);
    }
}

// The sums of one form; returns the lanes whose batch left its range.
template <int NW, int NC, int G, bool BATCH>
__device__ __forceinline__ uint64_t occupied_sums(int n0, int n1, int nb, int ng,
                                                  gptr<double2> aqsn, uint32_t goff,
                                                  gptr<double2> aqsm, const int (&pc)[NC],
                                                  gptr<double> wx, const cplx (&om)[NC],
                                                  const double (&wi2)[NC], const double (&thr)[NC],
                                                  cplx (&HX)[NC][NW], cplx (&SX)[NC][NW])
{
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int w = 0; w < NW; ++w) HX[c][w] = SX[c][w] = cmake(0.0, 0.0);
    uint64_t over = 0;
    OccupiedBand<NW, NC> cur;
    cur.load(n0, nb, ng, aqsn, goff, aqsm, pc, wx);
    for (int n = n0; n < n1; ++n) {
        OccupiedBand<NW, NC> next;  // loads while this band computes
        next.load(n + 1 < n1 ? n + 1 : n, nb, ng, aqsn, goff, aqsm, pc, wx);
        occupied_groups<NW, NC, 0, G, BATCH>(cur, om, wi2, thr, over, HX, SX);
        cur = next;
    }
    return over;
}

// Both sums over the occupied bands n0 <= n < n1 (all below nvband).  The batch
// needs denominators of at least 2^-60 (a product of G <= 6 pairs is then in its
// range) and waves where no lane's threshold lets branch C occur; `narrow`
// waves, those with a nearly vanishing om, and those whose batch overflowed take
// the sums term by term, in a loop of their own (a branch inside the common one
// costs it 12 to 100 spilled registers).
// One loop for both sums because every value but the last products is common:
// 150 occupied bands of 200, 4096 rows x 200 columns, nfreq 1, 2, 3, 4 and 8, took
// 303, 504, 696, 768 and 1528 us with the hole's terms in the hot loop and their
// reciprocals from its batch, 230, 419, 584, 671 and 1271 so; all of om real,
// nfreq 3 and 8, 1004 and 2295 against 681 and 1545.
template <int NW, int NC>
__device__ __forceinline__ void occupied_bands(int n0, int n1, int nb, int ng, gptr<double2> aqsn,
                                               uint32_t goff, gptr<double2> aqsm,
                                               const int (&pc)[NC], gptr<double> wx,
                                               const cplx (&om)[NC], const double (&wi2)[NC],
                                               const double (&thr)[NC], uint64_t narrow,
                                               cplx (&HX)[NC][NW], cplx (&SX)[NC][NW])
{
    constexpr int K = NC * NW;
    constexpr int groups = (K + kOccTerms - 1) / kOccTerms, G = (K + groups - 1) / groups;
    static_assert(G <= 6, "the 2^-60 lane bound keeps products of 6 pairs in the batch's range");
    bool below = false;
#pragma unroll
    for (int c = 0; c < NC; ++c)  // d <= thr off branch A, and rounding is monotone
        below = below || !branch_b_holds(fma(om[c].re, om[c].re, wi2[c]), thr[c]);
    uint64_t alone = narrow | __builtin_amdgcn_ballot_w64(below);
    if (alone == 0)
        alone = occupied_sums<NW, NC, G, true>(n0, n1, nb, ng, aqsn, goff, aqsm, pc, wx, om, wi2, thr,
                                               HX, SX);
    if (__builtin_expect(alone != 0, 0))
        occupied_sums<NW, NC, 1, false>(n0, n1, nb, ng, aqsn, goff, aqsm, pc, wx, om, wi2, thr, HX,
                                        SX);
}

// Where a tile's sums go.  hole() takes the lanes' Coulomb-hole parts (2 NW
// values per lane) of the unoccupied bands, occupied() those of the occupied
// ones and their screened-exchange parts; either may be called or not, at most
// once, hole() first.
//
// A row of 4 NW wave totals in LDS, achtemp re, im, asxtemp re, im per
// frequency, so that no total stays in registers over the band loop.  With
// KEEP values of the lane that the tile needs only at its end wait in LDS as
// well (`kept`, KEEP x 64 doubles): under the 128-VGPR cap of the 16-wave
// workgroups the compiler would spill them to memory, whose way back is a
// visible part of a short tile's time.
template <int NW, int KEEP = 0>
struct RowSink {
    static constexpr int kKeep = KEEP;
    double *row;
    int lane;
    double *kept;
    __device__ __forceinline__ void keep(int i, double v) const { kept[i * kWave + lane] = v; }
    __device__ __forceinline__ double fetch(int i) const { return kept[i * kWave + lane]; }
    __device__ __forceinline__ void hole(const double (&v)[2 * NW]) const {
        wave_totals<2 * NW>(v, lane, [&](int i, double t) { row[i + (i & ~1)] = t; });
    }
    // each total is added by the lane that wrote hole()'s
    __device__ __forceinline__ void occupied(const double (&v)[2 * NW],
                                             const double (&x)[2 * NW]) const {
        wave_totals<2 * NW>(v, lane, [&](int i, double t) { row[i + (i & ~1)] += t; });
        wave_totals<2 * NW>(x, lane, [&](int i, double t) { row[i + (i & ~1) + 2] = t; });
    }
};
// Running sums of a persistent wave, in scalar registers.
template <int NW>
struct RunningSink {
    static constexpr int kKeep = 0;
    cplx ach[NW], asx[NW];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int w = 0; w < NW; ++w) ach[w] = asx[w] = cmake(0.0, 0.0);
    }
    __device__ __forceinline__ void hole(const double (&v)[2 * NW]) { add(ach, v); }
    __device__ __forceinline__ void occupied(const double (&v)[2 * NW],
                                             const double (&x)[2 * NW]) {
        add(ach, v);
        add(asx, x);
    }
    __device__ __forceinline__ void add(cplx (&to)[NW], const double (&v)[2 * NW]) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            to[w].re = to_uniform(to[w].re + wave_sum(v[2 * w]));
            to[w].im = to_uniform(to[w].im + wave_sum(v[2 * w + 1]));
        }
    }
};

// NC consecutive G' columns p0 .. p0+NC-1 of one 64-row tile per wave,
// bands n_lo <= n < n_hi: each aqsntemp element a lane loads serves all of
// them, which divides the vector-memory traffic of the hot loop by NC.
// Columns at or beyond np repeat p0 and their contribution is dropped.  The
// sums go to the sink, the exchange ones only where the bands hold occupied
// ones.  All 64 lanes of the wave must call it together (wave reductions and
// full execution masks inside); lane l takes row g = gt*64 + l.
template <int NW, int BU, int NC, typename Sink>
__device__ __forceinline__ void fwd_tile_body(int nb, int nv, int n_lo, int n_hi, int ng, int np,
                                              int p0, int gt, int lane, gptr<double2> aqsm,
                                              gptr<double2> aqsn, gptr<double2> ieps,
                                              gptr<double2> wt, gptr<double> vcoul,
                                              gptr<double> wx, Sink &sink)
{
    const int g = gt * kWave + lane;
    const bool valid = g < ng;
    const int gc = valid ? g : ng - 1;  // clamped, contribution zeroed

    int pc[NC];
    cplx om[NC], ev[NC];
    double a[NC], wi2[NC], thr[NC];
    const uint32_t goff = (uint32_t)gc * (uint32_t)sizeof(double2);
    // every column's loads before the first value is used, also e, which the
    // sums need only at the end: one wait for all of them
    const double v = valid ? vcoul[gc] : 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        pc[c] = p0 + c < np ? p0 + c : p0;
        om[c] = cload(wt + (size_t)pc[c] * ng + gc);
        ev[c] = cload(ieps + (size_t)pc[c] * ng + gc);
    }
    bool wide_all = true;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        ev[c] = cscale(p0 + c < np ? v : 0.0, ev[c]);
        a[c] = om[c].re;
        wi2[c] = om[c].im * om[c].im;
        thr[c] = branch_a_threshold(fma(a[c], a[c], wi2[c]));
        wide_all = wide_all && wi2[c] >= kMinUnclampedWi2;
    }
    const uint64_t narrow = __builtin_amdgcn_ballot_w64(!wide_all);

    if constexpr (Sink::kKeep > 0) {
        static_assert(Sink::kKeep == 3 * NC, "three values per column");
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            sink.keep(3 * c, ev[c].re);
            sink.keep(3 * c + 1, ev[c].im);
            sink.keep(3 * c + 2, om[c].im);
        }
    }

    // occupied bands come last, so that neither part holds the other's sums in
    // registers (first, 32 x 512 x 64 with two of them took 1 us more)
    const int occ_hi = nv < n_hi ? nv : n_hi;
    if (occ_hi < n_hi) {
        // Coulomb hole of the unoccupied bands, whole groups, then band by band
        cplx P1[NC][NW], P2[NC][NW];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int w = 0; w < NW; ++w) P1[c][w] = P2[c][w] = cmake(0.0, 0.0);
        const int n0 = occ_hi > n_lo ? occ_hi : n_lo;
        const auto hole = [&](auto narrow_form) {
            constexpr bool NARROW = decltype(narrow_form)::value;
            BandGroup<NW, BU> first;
            first.load_first(n0, nb, ng, aqsn, goff, wx);
            const int n = ch_bands<NW, BU, NC, NARROW>(n0, n_hi, nb, ng, aqsn, goff, aqsm, pc, wx, a,
                                                       wi2, thr, first, P1, P2);
            if constexpr (BU > 1) {
                if (n < n_hi) {
                    BandGroup<NW, 1> rest;
                    rest.load_first(n, nb, ng, aqsn, goff, wx);
                    ch_bands<NW, 1, NC, NARROW>(n, n_hi, nb, ng, aqsn, goff, aqsm, pc, wx, a, wi2,
                                                thr, rest, P1, P2);
                }
            }
        };
        if (__builtin_expect(narrow != 0, 0)) hole(std::true_type());
        else hole(std::false_type());
        if constexpr (Sink::kKeep > 0) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                ev[c] = cmake(sink.fetch(3 * c), sink.fetch(3 * c + 1));
                om[c] = cmake(a[c], sink.fetch(3 * c + 2));
            }
        }
        double v2[2 * NW];
#pragma unroll
        for (int k = 0; k < 2 * NW; ++k) v2[k] = 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double wtr = fma(a[c], a[c], wi2[c]);
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                // S = om P1 - wtr P2
                cplx S = cmul(om[c], P1[c][w]);
                S.re = fma(-wtr, P2[c][w].re, S.re);
                S.im = fma(-wtr, P2[c][w].im, S.im);
                const cplx t = cscale(0.5, cmul(ev[c], S));
                v2[2 * w] += t.re;
                v2[2 * w + 1] += t.im;
            }
        }
        sink.hole(v2);
    }

    if (occ_hi > n_lo) {
        cplx HX[NC][NW], SX[NC][NW];
        occupied_bands<NW, NC>(n_lo, occ_hi, nb, ng, aqsn, goff, aqsm, pc, wx, om, wi2, thr, narrow,
                               HX, SX);
        double v2[2 * NW], x2[2 * NW];
#pragma unroll
        for (int k = 0; k < 2 * NW; ++k) v2[k] = x2[k] = 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (Sink::kKeep > 0)
                ev[c] = cmake(sink.fetch(3 * c), sink.fetch(3 * c + 1));
            const cplx evom = cmul(ev[c], om[c]);
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const cplx h = cmul(evom, HX[c][w]), x = cmul(evom, SX[c][w]);
                v2[2 * w] = fma(0.5, h.re, v2[2 * w]);
                v2[2 * w + 1] = fma(0.5, h.im, v2[2 * w + 1]);
                x2[2 * w] += x.re;
                x2[2 * w + 1] += x.im;
            }
        }
        sink.occupied(v2, x2);
    }
}

}  // namespace gpp
