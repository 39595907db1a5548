// gpp_bwd.hip -- adjoint of the GPP reduction on gfx950 (fp64, no MFMA).
//
// Loss L = sum_w Re(conj(ga[w]) achtemp[w] + conj(gs[w]) asxtemp[w]); the
// gradient of a complex input z is dL/dRe z + i dL/dIm z (no derivative
// through the branch).  Nothing is stored by the forward: every term's
// wdiff, reciprocal and branch are recomputed here.
//
// Per (n, p, g), with u_w = conj(1/(x_w - om)) for branch-A terms (else 0)
// and the exchange quantities of occupied bands (ssx = e sigma,
// d ssx/d om = e delta):
//   K  = sum_w ga_w/2 u_w            L  = sum_w x_w ga_w/2 u_w^2
//   KS = sum_w gs_w conj(sigma_w)    LS = sum_w gs_w conj(delta_w)
//   Z  = conj(om) K + KS             W  = L + LS
// the gradients are
//   dI_eps[p][g]    = vcoul[g]         sum_n conj(M) Z
//   dwtilde[p][g]   = vcoul[g] conj(e) sum_n conj(M) W
//   daqsntemp[n][g] = sum_p vcoul[g] conj(e) aqsmtemp[n][p] Z
//   daqsmtemp[n][p] = sum_g vcoul[g] e aqsntemp[n][g] conj(Z)
// with M = aqsntemp[n][g] conj(aqsmtemp[n][p]).
//
// Kernels.  bwd_pairs (lane = g, wave-uniform p, bands serial) writes
// dwtilde and dI_eps.  K and L are linear in ga/2, so over unoccupied bands
// the lane never forms them: it keeps four sums per frequency over the bands,
// weighted by conj(M),
//   A2_w = sum_n conj(M) r,           B1_w = sum_n conj(M) x r,
//   B2_w = sum_n conj(M) x r^2,       B3_w = sum_n conj(M) x (x - Re om) r^2
// (r the reciprocal of |x - om|^2 on branch-A terms, which add nothing
// otherwise) and applies ga/2 once at the end: with u = (x - om) r and, on
// branch A, |x - om|^2 r = 1,
//   sum_n conj(M) K = sum_w ga_w/2 (B1_w - om A2_w),
//   sum_n conj(M) L = sum_w ga_w/2 (B1_w - 2 (Im om)^2 B2_w - 2i Im om B3_w).
// B1 - om A2 cancels by |om| / |x - om|, up to 500 on branch A, so from five
// frequencies on the sums are A2 and
//   C1_w = sum_n conj(M) (x - Re om) r,
//   D1_w = sum_n conj(M) x r (1 - 2 (Im om)^2 r),  B3_w as above, with
//   sum_n conj(M) K = sum_w ga_w/2 (C1_w - i Im om A2_w),
//   sum_n conj(M) L = sum_w ga_w/2 (D1_w - 2i Im om B3_w).
// (dI_eps at |om| / |x - om| = 450, nfreq 5 to 8, in 2^-53 of the sum of |term|:
// up to 1000 with B1, up to 14 so; two operations per term more: whole adjoint,
// bands x rows x columns, 128 x 8192 x 400 at nfreq 5 and 8 2.66 -> 2.78 and
// 3.97 -> 4.19 ms.)
// Occupied bands, and up to four frequencies the bands left over of the
// groups, form K and L per band.
// bwd_bands (lane = g; a workgroup of four waves owns kBandTile bands and
// 256 consecutive rows, 64 per wave, and walks a range of G' columns)
// forms vcoul conj(e) Z per term, adds aqsmtemp[n][p] times it into
// daqsntemp (registers), and takes aqsntemp[n][g] conj(vcoul conj(e) Z) =
// vcoul e aqsntemp conj(Z) as the term of daqsmtemp[n][p]: those terms go
// through a per-wave LDS slab (8 lanes per row, then a DPP sum over the 8),
// are added over the workgroup's four waves and written as one partial per
// 256-row block; reduce_am sums the partials in a fixed order and zero-fills
// columns >= ngpown.  No atomics: results are bitwise reproducible.
//
// What bounds it.  Large grids: the fp64 vector ALU at the clock the part
// holds (256 bands x 16384 rows x 819 columns, nfreq 3: pairs kernel 6.8 ->
// 6.7 ms, 0.92 of the issue slots at 1.98 GHz; bands kernel 7.5 -> 6.7 ms, 0.75
// -> 0.87 at 2.05 GHz, since it needs x and gh only and its loads run ahead;
// whole adjoint timed in turn 14.00 -> 13.36 ms on one box, 14.95 -> 13.50 on
// another).  Short grids: the number of waves and the longest workgroup, hence
// the forms below (512 rows x 32 bands x 64 columns: 142 us in four-band
// workgroups, 37 now; 3001 x 101 x 150, nfreq 5: 631 and 351).
#include "gpp_bwd_shape.h"
#include "gpp_device.h"
#include "gpp_fwd_tile.h"
#include "gpp_internal.h"

namespace gpp {

constexpr int kBwdWaves = 4;
constexpr int kBwdThreads = kBwdWaves * kWave;
constexpr int kRowsPerBlock = kBwdWaves * kWave;  // g rows per workgroup (both kernels)
// Bands per batch-inverted group of the pairs kernel's band sums (at most 12
// denominators) and the minimum waves per SIMD the compiler must allow (a
// register cap; the four sums take 16 VGPRs per frequency), for nfreq 1 to 8.
#ifndef GPP_BWD_PAIRS_GROUP
#define GPP_BWD_PAIRS_GROUP 4, 3, 2, 2, 1, 1, 1, 1
#endif
constexpr int kPairsGroup[8] = {GPP_BWD_PAIRS_GROUP};
constexpr int pairs_group(int nw) { return kPairsGroup[nw - 1]; }
// Which four sums the pairs kernel keeps: A2, C1, D1, B3 from five frequencies
// on, A2, B1, B2, B3 below (two operations per term fewer).
constexpr bool pairs_many(int nw) { return nw >= 5; }
static_assert(pairs_group(5) == 1 && pairs_group(6) == 1 && pairs_group(7) == 1 &&
                  pairs_group(8) == 1,
              "with more than four frequencies no bands are left over of the groups");
#ifndef GPP_BWD_PAIRS_WAVES
#define GPP_BWD_PAIRS_WAVES 4, 4, 4, 3, 3, 3, 2, 2
#endif
constexpr int kPairsWaves[8] = {GPP_BWD_PAIRS_WAVES};
constexpr int pairs_waves(int nw) { return kPairsWaves[nw - 1]; }
constexpr int kOctet = 8;                          // lanes that share one row sum, and slab rows
// The same cap of the bands kernel without and with the daqsmtemp sums.
// Bands per bands-kernel workgroup: four, so that the daqsmtemp slab of two
// columns fills the 8 rows an octet of lanes reduces.  Measured on MI355X at
// the adjoint workload's sizes against three bands at 5 and 4 waves: the
// kernel with daqsmtemp 4.5 % faster at nfreq 3 (at 4 waves, with four bands,
// it spilled and ran 28 % slower), without daqsmtemp 3 % faster at nfreq 3
// and 2-2.5x faster at nfreq 4 and 8, where three bands at 5 waves spilled.
#ifndef GPP_BWD_BANDS_WAVES
#define GPP_BWD_BANDS_WAVES 4
#endif
#ifndef GPP_BWD_BANDS_AM_WAVES
#define GPP_BWD_BANDS_AM_WAVES 3
#endif
#ifndef GPP_BWD_BAND_TILE
#define GPP_BWD_BAND_TILE 4
#endif
constexpr int kBandTile = GPP_BWD_BAND_TILE;       // bands per bands-kernel workgroup
// Bands-kernel p-range split (see bwd_geometry): resident bands waves of the
// MI355X (256 CUs x 4 SIMDs x GPP_BWD_BANDS_WAVES), rounds of them to aim
// at, and the shortest segment.
#ifndef GPP_BWD_BANDS_ROUNDS
#define GPP_BWD_BANDS_ROUNDS 16
#endif
constexpr long kBandsCUs = 256;
constexpr long kBandsWaveSlots = kBandsCUs * 4 * GPP_BWD_BANDS_WAVES;
constexpr int kBandsRounds = GPP_BWD_BANDS_ROUNDS;
constexpr int kMinSegCols = 64;
// Bands per batch-inverted group of the bands kernel: the largest divisor
// of the band tile whose group holds at most 12 denominators.
constexpr int bands_group(int nw, int bt)
{
    for (int g = bt; g > 1; --g)
        if (bt % g == 0 && g * nw <= 12) return g;
    return 1;
}
// Short grids of the bands kernel (fewer than kBandsShortBelow waves of the
// long form) take kShortTile bands per workgroup and kShortRanges waves per
// row tile, each on its own part of the column segment; or one band per
// workgroup where that still makes at most one workgroup per compute unit
// (whole adjoint of 32 bands x 512 rows x 64 columns, nfreq 3: 32.1 -> 24.4 us
// without occupied bands, 43 -> 40.9 with two).
constexpr int kTinyTile = 1;
constexpr int kShortTile = 2;
constexpr int kShortRanges = 4;
#ifndef GPP_BWD_SHORT_BELOW
#define GPP_BWD_SHORT_BELOW 8192
#endif
constexpr long kBandsShortBelow = GPP_BWD_SHORT_BELOW;
// An occupied band costs about three others (its exchange terms, and single
// reciprocals), so a tile of them outlasts the rest: they take a tile each
// where there are at most kSingleOccupied, or the short form runs at most
// kSingleBlocks workgroups.  More of them fill the GPU by themselves, and
// share a pair's constants better in whole tiles.  Whole adjoint, rows x
// bands x columns (occupied, nfreq), shared and single tiles: 512 x 32 x 64
// (2, 3) 63.7 and 43.0 us, 1024 x 64 x 102 (32, 5) 202 and 151, 2048 x 64 x 102
// (2, 3) 121.8 and 102.4, 8192 x 256 x 409 (4, 5) 5300 and 5120, 6000 x 200 x
// 300 (12, 8) 4110 and 3770; but 3001 x 101 x 150 (20, 5) 489 and 500, 8192 x
// 256 x 409 (40, 3) 4720 and 4850.
constexpr int kSingleOccupied = 12;
constexpr long kSingleBlocks = 1024;
// daqsmtemp sums of the bands kernel: the slab holds the terms of 8 / BT G'
// columns (BT rows each); every kAmCols columns the row tiles' sums are added
// and written.
constexpr int kAmCols = 16;

// The upstream gradient scaled for the kernels, gh = ga/2 (wave-uniform; the
// halving is exact, so x gh rounds as x ga / 2 does).
__device__ __forceinline__ cplx half_of(const double2 *__restrict__ ga, int w)
{
    const cplx g = cload(ga + w);
    return cmake(0.5 * g.re, 0.5 * g.im);
}

struct PairState {
    double a, b, wi2, wtr, thr;
    double b2, wi2x2;  // 2 Im om and 2 (Im om)^2
    bool wide;  // (Im om)^2 >= kMinUnclampedWi2: batch inversion allowed
    cplx om, e, ve;  // ve = vcoul[g] e (0 for rows beyond ncouls)
};

// One band of one lane with frequencies x (wave-uniform): its Z = conj(om) K
// [+ KS] and, with WANT_W, W = L [+ LS]; OCC adds the exchange parts.  With
// d = x - om, s = x + om, u = conj(1/d) and y = conj(1/s) those are, from ssx =
// e sigma and d ssx/d om = e delta,
//   A:  conj(sigma) = conj(om)^2 u y,   conj(delta) = 2 conj(om) (x u y)^2
//   B:  conj(sigma) = -conj(om) y / 2,  conj(delta) = -x y^2 / 2
// and so, with m = conj(om) u on branch A, -1/2 on B and l = 2 x u on A, 1 on B,
//   conj(sigma) = conj(om) m y,         conj(delta) = x l m y^2
// without a divide: u = d r and y = s rs, where r = 1/|d|^2 (0 off branch A) and
// rs = 1/|s|^2 (0 on branch C).  Selecting m and l in place of sigma and delta:
// 100 occupied bands of 128, 4096 rows x 200 columns, nfreq 1, 3 and 8, 614 -> 560,
// 1353 -> 1191 and 3305 -> 2876 us for the whole adjoint.
// The reciprocals come one by one: delta takes their squares, and those of a
// batch inversion (one Newton step, shared error) raised the dwtilde error of
// a problem with few bands from 3.8e-16 to 1.7e-15.
template <int NW, bool OCC, bool WANT_W>
__device__ __forceinline__ void band_zw(const double (&x)[NW], const double2 *__restrict__ ga,
                                        const double2 *__restrict__ gs, const PairState &ps,
                                        cplx &Z, cplx &W)
{
    const double a = ps.a, b = ps.b, wi2 = ps.wi2;
    cplx K = cmake(0.0, 0.0), L = cmake(0.0, 0.0), KS = K, LS = K;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const double dr = x[w] - a, sp = x[w] + a;
        const double d = fma(dr, dr, wi2), r = rcp_nr2(d);
        const bool isA = d > ps.thr;
        const double rm = isA ? r : 0.0;
        const cplx u = cmake(dr * rm, -b * rm);
        const cplx gh = half_of(ga, w);
        cmac(K, gh, u);
        if (WANT_W) cmac(L, cscale(x[w], gh), cmul(u, u));
        if constexpr (OCC) {
            const double rs = rcp_nr2(fma(sp, sp, wi2));
            const double rsm = isA || branch_b_holds(ps.wtr, d) ? rs : 0.0;
            const cplx y = cmake(sp * rsm, b * rsm);
            cplx m = cmul(cmake(a, -b), u);
            m.re = isA ? m.re : -0.5;
            const cplx my = cmul(m, y), g = cload(gs + w);
            cmac(KS, g, my);
            if constexpr (WANT_W) {
                cplx l = cscale(2.0 * x[w], u);
                l.re = isA ? l.re : 1.0;
                cmac(LS, cscale(x[w], g), cmul(cmul(my, y), l));
            }
            // one term at a time: six and more at once take 40 registers more
            if constexpr (NW > 5 && WANT_W) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (OCC) {
        K = cadd(K, KS);
        L = cadd(L, LS);
    }
    Z = cmul(cmake(a, -b), K);
    W = L;
}

__device__ __forceinline__ PairState make_pair(cplx om, cplx e, double v)
{
    PairState s;
    s.om = om;
    s.e = e;
    s.a = om.re;
    s.b = om.im;
    s.wi2 = s.b * s.b;
    s.b2 = 2.0 * s.b;
    s.wi2x2 = 2.0 * s.wi2;
    s.wtr = fma(s.a, s.a, s.wi2);
    s.thr = branch_a_threshold(s.wtr);
    s.wide = s.wi2 >= kMinUnclampedWi2;
    s.ve = cscale(v, e);
    return s;
}

// One branch-A term of the pairs kernel's band sums, up to four frequencies:
// A2 += cM r, B1 += cM x r, B2 += cM x r^2, B3 += cM x dr r^2 (dr = x - Re om),
// with the compare d > thr as the execution mask (a term off branch A adds
// nothing, whatever its reciprocal), all 64 lanes active before and after.
__device__ __forceinline__ void pairs_term(double d, double thr, double r, double x, double dr,
                                           cplx cm, cplx &A2, cplx &B1, cplx &B2, cplx &B3)
{
    double xr, xr2, xdr2;
    asm("v_cmpx_gt_f64_e32 vcc, %[d], %[thr]\n\t"
        "v_mul_f64 %[xr], %[r], %[x]\n\t"
        "v_fma_f64 %[a2r], %[r], %[cr], %[a2r]\n\t"
        "v_fma_f64 %[a2i], %[r], %[ci], %[a2i]\n\t"
        "v_mul_f64 %[xr2], %[xr], %[r]\n\t"
        "v_fma_f64 %[b1r], %[xr], %[cr], %[b1r]\n\t"
        "v_fma_f64 %[b1i], %[xr], %[ci], %[b1i]\n\t"
        "v_mul_f64 %[xdr2], %[xr2], %[dr]\n\t"
        "v_fma_f64 %[b2r], %[xr2], %[cr], %[b2r]\n\t"
        "v_fma_f64 %[b2i], %[xr2], %[ci], %[b2i]\n\t"
        "v_fma_f64 %[b3r], %[xdr2], %[cr], %[b3r]\n\t"
        "v_fma_f64 %[b3i], %[xdr2], %[ci], %[b3i]\n\t"
        "s_mov_b64 exec, -1"
        : [xr] "=&v"(xr), [xr2] "=&v"(xr2), [xdr2] "=&v"(xdr2),
          [a2r] "+v"(A2.re), [a2i] "+v"(A2.im), [b1r] "+v"(B1.re), [b1i] "+v"(B1.im),
          [b2r] "+v"(B2.re), [b2i] "+v"(B2.im), [b3r] "+v"(B3.re), [b3i] "+v"(B3.im)
        : [d] "v"(d), [thr] "v"(thr), [r] "v"(r), [x] "s"(x), [dr] "v"(dr), [cr] "v"(cm.re),
          [ci] "v"(cm.im)
        : "vcc");
}
// The same from five frequencies on: A2 += cM r, C1 += cM dr r,
// D1 += cM x r (1 - wi2x2 r), B3 += cM x dr r^2, wi2x2 = 2 (Im om)^2.
__device__ __forceinline__ void pairs_term_many(double d, double thr, double r, double x, double dr,
                                                double wi2x2, cplx cm, cplx &A2, cplx &C1,
                                                cplx &D1, cplx &B3)
{
    double xr, yr, t;
    asm("v_cmpx_gt_f64_e32 vcc, %[d], %[thr]\n\t"
        "v_mul_f64 %[xr], %[r], %[x]\n\t"
        "v_mul_f64 %[yr], %[r], %[dr]\n\t"
        "v_fma_f64 %[t], -%[wi2x2], %[r], 1.0\n\t"
        "v_fma_f64 %[a2r], %[r], %[cr], %[a2r]\n\t"
        "v_fma_f64 %[a2i], %[r], %[ci], %[a2i]\n\t"
        "v_mul_f64 %[t], %[xr], %[t]\n\t"
        "v_fma_f64 %[c1r], %[yr], %[cr], %[c1r]\n\t"
        "v_fma_f64 %[c1i], %[yr], %[ci], %[c1i]\n\t"
        "v_mul_f64 %[xr], %[xr], %[yr]\n\t"
        "v_fma_f64 %[d1r], %[t], %[cr], %[d1r]\n\t"
        "v_fma_f64 %[d1i], %[t], %[ci], %[d1i]\n\t"
        "v_fma_f64 %[b3r], %[xr], %[cr], %[b3r]\n\t"
        "v_fma_f64 %[b3i], %[xr], %[ci], %[b3i]\n\t"
        "s_mov_b64 exec, -1"
        : [xr] "=&v"(xr), [yr] "=&v"(yr), [t] "=&v"(t),
          [a2r] "+v"(A2.re), [a2i] "+v"(A2.im), [c1r] "+v"(C1.re), [c1i] "+v"(C1.im),
          [d1r] "+v"(D1.re), [d1i] "+v"(D1.im), [b3r] "+v"(B3.re), [b3i] "+v"(B3.im)
        : [d] "v"(d), [thr] "v"(thr), [r] "v"(r), [x] "s"(x), [dr] "v"(dr), [wi2x2] "v"(wi2x2),
          [cr] "v"(cm.re), [ci] "v"(cm.im)
        : "vcc");
}

// The band sums of one lane over the whole groups of G unoccupied bands in
// [n, end): one batch inversion over a group's G*NW denominators, then
// pairs_term per term; returns the first band left over.  Loads run ahead
// and addresses run along as in the forward's loop (ch_bands).
template <int NW, int G>
__device__ __forceinline__ int pairs_bands(int n, int end, int nb, int ng, gptr<double2> aqsn,
                                           uint32_t goff, gptr<double2> am_col, gptr<double> wx,
                                           const PairState &ps, cplx (&S1)[NW], cplx (&S2)[NW],
                                           cplx (&S3)[NW], cplx (&S4)[NW])
{
    constexpr int Kt = G * NW;
    static_assert(Kt <= 12, "a group holds at most 12 denominators");
    int left = (end - n) / G;
    if (left <= 0) return n;
    const uint64_t narrow = __builtin_amdgcn_ballot_w64(!ps.wide);
    const uint32_t row_bytes = (uint32_t)ng * (uint32_t)sizeof(double2);
    const long step = (long)G * row_bytes;
    BandGroup<NW, G> cur;
    cur.load_first(n, nb, ng, aqsn, goff, wx);
    uint64_t rows = (uint64_t)(aqsn + (size_t)n * ng);
    Walker am_at, x_at[NW];
    am_at.start((uint64_t)(am_col + (size_t)n * ng));
    int more = left > 1 ? G : 0;  // bands to the next group; the last repeats
#pragma unroll
    for (int w = 0; w < NW; ++w) x_at[w].start((uint64_t)(wx + (size_t)w * nb + n + more));
    n += left * G;
    cur.arrived();
    for (;;) {
        cplx am[G];
        double xn[Kt];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            am[u] = am_at.complex(u * row_bytes);
#pragma unroll
            for (int w = 0; w < NW; ++w) xn[u * NW + w] = x_at[w].real(u);
        }
        rows += more ? step : 0;
        more = left > 2 ? G : 0;
        am_at.advance(step);
#pragma unroll
        for (int w = 0; w < NW; ++w) x_at[w].advance(more * (long)sizeof(double));
        double drs[Kt], d[Kt], c[Kt], r[Kt];
#pragma unroll
        for (int k = 0; k < Kt; ++k) {
            drs[k] = cur.xs[k] - ps.a;
            d[k] = fma(drs[k], drs[k], ps.wi2);  // unclamped: see batch_prefix
        }
        const double all = batch_prefix<Kt>(d, c);
        batch_back<Kt>(d, c, all, r);
        if (__builtin_expect(batch_misses(all, narrow) != 0, 0)) one_by_one<Kt>(d, r);
        cplx cM[G];
#pragma unroll
        for (int u = 0; u < G; ++u) cM[u] = cmul_conj(am[u], cur.an[u]);  // conj(an) am
#pragma unroll
        for (int u = 0; u < G; ++u) cur.an[u] = load_elem_at(rows, u * row_bytes, goff);
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int k = u * NW + w;
                if constexpr (pairs_many(NW))
                    pairs_term_many(d[k], ps.thr, r[k], cur.xs[k], drs[k], ps.wi2x2, cM[u], S1[w],
                                    S2[w], S3[w], S4[w]);
                else
                    pairs_term(d[k], ps.thr, r[k], cur.xs[k], drs[k], cM[u], S1[w], S2[w], S3[w],
                               S4[w]);
            }
        if (--left == 0) return n;
#pragma unroll
        for (int k = 0; k < Kt; ++k) cur.xs[k] = xn[k];
    }
}

// Bands [n, end) of one lane, band by band (OCC: occupied ones):
// Ge += conj(M) Z and Gw += conj(M) W.  The next band's values load while this
// one computes.
template <int NW, bool OCC>
__device__ __forceinline__ void pairs_per_band(int n, int end, int nb, int ng, gptr<double2> aqsn,
                                               gptr<double2> am_col, gptr<double> wx,
                                               const double2 *__restrict__ ga,
                                               const double2 *__restrict__ gs,
                                               const PairState &ps, uint32_t goff, cplx &Ge,
                                               cplx &Gw)
{
    if (n >= end) return;
    const int pc[1] = {0};
    OccupiedBand<NW, 1> cur;
    cur.load(n, nb, ng, aqsn, goff, am_col, pc, wx);
    for (; n < end; ++n) {
        OccupiedBand<NW, 1> next;
        next.load(n + 1 < end ? n + 1 : n, nb, ng, aqsn, goff, am_col, pc, wx);
        cplx Z, W;
        band_zw<NW, OCC, true>(cur.x, ga, gs, ps, Z, W);
        const cplx cM = cmul_conj(cur.am[0], cur.an);  // conj(M) = conj(an) am
        cmac(Ge, cM, Z);
        cmac(Gw, cM, W);
        cur = next;
    }
}

// ---- pairs kernel: dwtilde and dI_eps -------------------------------------
// Workgroup = 256 rows (one 64-row tile per wave) x one G' column p, p
// fastest, so concurrently resident workgroups share one row block.  With
// SHARE, for grids that leave SIMDs without a wave, a workgroup's four waves
// share one 64-row tile's bands instead and the first of them adds their
// gradients.
template <int NW, bool SHARE>
__global__ void __launch_bounds__(kBwdThreads)
__attribute__((amdgpu_waves_per_eu(pairs_waves(NW))))
bwd_pairs(int nb, int nv, int ng, int np, long nblocks, const double2 *__restrict__ aqsm,
          const double2 *__restrict__ aqsn, const double2 *__restrict__ ieps,
          const double2 *__restrict__ wt, const double *__restrict__ vcoul,
          const double *__restrict__ wx, const double2 *__restrict__ ga,
          const double2 *__restrict__ gs, double2 *__restrict__ grad_wt,
          double2 *__restrict__ grad_ieps)
{
    constexpr int S = SHARE ? kBwdWaves : 1;  // waves per tile
    constexpr int G = pairs_group(NW);
    __shared__ double2 part[SHARE ? S - 1 : 1][2][SHARE ? kWave : 1];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const long blk = xcd_remap(blockIdx.x, gridDim.x);
    if (blk >= nblocks) return;  // the whole workgroup leaves together
    const int gb = (int)(blk / np);
    const int p = (int)(blk - (long)gb * np);
    const int g = (SHARE ? gb : gb * kBwdWaves + wid) * kWave + lane;
    const bool valid = g < ng;
    const int gc = valid ? g : ng - 1;
    const double v = valid ? vcoul[gc] : 0.0;
    const cplx om = cload(wt + (size_t)p * ng + gc), e = cload(ieps + (size_t)p * ng + gc);
    const PairState ps = make_pair(om, e, v);
    const double2 *am_col = aqsm + p;
    const uint32_t goff = (uint32_t)gc * (uint32_t)sizeof(double2);

    // the wave's bands: its shares of the occupied ones and of the groups
    const int nocc = nv < nb ? nv : nb, k = SHARE ? wid : 0;
    const int end = share_first_band(nb, nocc, G, k + 1, S);

    cplx Ge = cmake(0.0, 0.0), Gw = cmake(0.0, 0.0);
    pairs_per_band<NW, true>(share_begin(nocc, k, S), share_begin(nocc, k + 1, S), nb, ng,
                             as_global(aqsn), as_global(am_col), as_global(wx), ga, gs, ps, goff,
                             Ge, Gw);
    // A2, B1, B2, B3, or A2, C1, D1, B3 (pairs_many)
    cplx S1[NW], S2[NW], S3[NW], S4[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) S1[w] = S2[w] = S3[w] = S4[w] = cmake(0.0, 0.0);
    int n = share_first_band(nb, nocc, G, k, S);
    n = pairs_bands<NW, G>(n, end, nb, ng, as_global(aqsn), goff, as_global(am_col),
                           as_global(wx), ps, S1, S2, S3, S4);
    if constexpr (G > 1)
        pairs_per_band<NW, false>(n, end, nb, ng, as_global(aqsn), as_global(am_col),
                                  as_global(wx), ga, gs, ps, goff, Ge, Gw);
    // sum_n conj(M) K and sum_n conj(M) L from the band sums
    cplx SK = cmake(0.0, 0.0), SL = cmake(0.0, 0.0);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const cplx h = half_of(ga, w);
        cplx k, l;
        if constexpr (pairs_many(NW)) {
            // C1 - i (Im om) A2 and D1 - 2i (Im om) B3
            k = cmake(fma(ps.b, S1[w].im, S2[w].re), fma(-ps.b, S1[w].re, S2[w].im));
            l = cmake(fma(ps.b2, S4[w].im, S3[w].re), fma(-ps.b2, S4[w].re, S3[w].im));
        } else {
            // B1 - om A2 and B1 - 2 (Im om)^2 B2 - 2i (Im om) B3
            k = cadd(S2[w], cmul(cmake(-ps.a, -ps.b), S1[w]));
            l = cmake(fma(ps.b2, S4[w].im, fma(-ps.wi2x2, S3[w].re, S2[w].re)),
                      fma(-ps.b2, S4[w].re, fma(-ps.wi2x2, S3[w].im, S2[w].im)));
        }
        cmac(SK, h, k);
        cmac(SL, h, l);
    }
    cmac(Ge, cmake(ps.om.re, -ps.om.im), SK);
    Gw = cadd(Gw, SL);

    if constexpr (SHARE) {
        if (wid > 0) {
            part[wid - 1][0][lane] = make_double2(Ge.re, Ge.im);
            part[wid - 1][1][lane] = make_double2(Gw.re, Gw.im);
        }
        __syncthreads();
        if (wid > 0) return;
#pragma unroll
        for (int i = 0; i < S - 1; ++i) {
            const double2 pe = part[i][0][lane], pw = part[i][1][lane];
            Ge = cadd(Ge, cmake(pe.x, pe.y));
            Gw = cadd(Gw, cmake(pw.x, pw.y));
        }
    }
    if (valid) {
        const size_t idx = (size_t)p * ng + g;
        if (grad_ieps) {
            const cplx r = cscale(v, Ge);
            grad_ieps[idx] = make_double2(r.re, r.im);
        }
        if (grad_wt) {
            const cplx r = cscale(v, cmul(cmake(ps.e.re, -ps.e.im), Gw));
            grad_wt[idx] = make_double2(r.re, r.im);
        }
    }
}

// ---- bands kernel: daqsntemp and the daqsmtemp partials -------------------
// LDS of the daqsmtemp sums of four waves (the row tiles of 256 rows): each
// wave's slab of per-lane terms (8 rows: BT bands x 8 / BT columns) and the
// waves' row sums of up to kAmCols columns.  A row is 8 entries (128 bytes)
// longer than the wave, see am_column_done.
template <int BT>
struct AmStage {
    double2 slab[kBwdWaves][kOctet][kWave + kOctet];
    double2 red[kBwdWaves][BT * kAmCols];
};

// Where a wave's daqsmtemp terms go.  `first` is the first column whose sums
// wait in red.
template <int BT>
struct AmCtx {
    AmStage<BT> *st;
    double2 *part;  // am_part: [256-row block][nb][np]
    int wid, lane, gblk, n0, n_end, nb, np, first;
};

// This lane's daqsmtemp term of band u at column p: an conj(vcoul conj(e) Z).
template <int BT>
__device__ __forceinline__ void am_put(AmCtx<BT> &a, int p, int u, cplx an, cplx vz)
{
    constexpr int C = kOctet / BT;
    const cplx t = cmul_conj(an, vz);
    a.st->slab[a.wid][((p - a.first) % C) * BT + u][a.lane] = make_double2(t.re, t.im);
}

// After column p: when the slab is full (8 / BT columns) or p is the last of
// the columns up to `end`, add each slab row over the wave (lane (tj, tk) adds
// the entries tk, tk + 8, ..., tk + 56 of row tj, then the octet adds its 8
// sums) into red.  An octet thus reads 128 contiguous bytes at a time, and
// the row length shifts row tj by tj * 128 bytes, so that the two octets the
// LDS serves per clock fall in different halves of its banks: measured on
// gfx950 (gpp_mb_lds patterns 2 and 1), such a 16-byte read takes 4 LDS
// cycles with no bank conflict, against 8 cycles (4 of them conflict stalls)
// when each lane reads 8 consecutive entries.  With the shift in the row
// length the eight reads share one address register.
template <int BT>
__device__ __forceinline__ void am_column_done(AmCtx<BT> &a, int p, int end)
{
    constexpr int C = kOctet / BT;
    const int c = (p - a.first) % C;
    if (c + 1 < C && p + 1 < end) return;
    const int rows = (c + 1) * BT;
    wave_lds_sync();
    const int tj = a.lane >> 3, tk = a.lane & (kOctet - 1);
    double sr = 0.0, si = 0.0;
    if (tj < rows) {
#pragma unroll
        for (int i = 0; i < kOctet; ++i) {
            const double2 v = a.st->slab[a.wid][tj][tk + kOctet * i];
            sr += v.x;
            si += v.y;
        }
    }
    sr = octet_sum(sr);
    si = octet_sum(si);
    if (tk == 0 && tj < rows) a.st->red[a.wid][(p - c - a.first) * BT + tj] = make_double2(sr, si);
    wave_lds_sync();
}

// Adds the row tiles' sums of the columns [a.first, end) and writes them;
// every wave of the workgroup calls it.
template <int BT>
__device__ __forceinline__ void am_flush(AmCtx<BT> &a, int end)
{
    __syncthreads();
    const int rows = end > a.first ? (end - a.first) * BT : 0;
    const int t = threadIdx.x % kBwdThreads;
    if (t < 2 * rows) {
        const int j = t >> 1, comp = t & 1;
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < kBwdWaves; ++k) {
            const double2 v = a.st->red[k][j];
            s += comp ? v.y : v.x;
        }
        const int col = a.first + j / BT, n = a.n0 + j % BT;
        if (n < a.n_end)
            reinterpret_cast<double *>(a.part + ((size_t)a.gblk * a.nb + n) * a.np + col)[comp] = s;
    }
    __syncthreads();
}

// x - a again where the first one, before the inversion, has left the
// registers (held over it, 12 of them made the four-band kernels spill; formed
// again, whole adjoint of 256 bands x 16384 rows x 819 columns, nfreq 3, 14.01
// and 14.02 ms without and with it).
__device__ __forceinline__ double subtract_again(double x, double a)
{
    double y;
    asm("v_add_f64 %0, %1, -%2" : "=v"(y) : "s"(x), "v"(a));
    return y;
}

// Fast form of a wave's columns [p_lo, p_hi): every band n0 .. n0+BT-1 is
// unoccupied and below nb.  With r_w the masked reciprocal of |x_w - om|^2,
//   vcoul conj(e) Z = vcoul conj(e om) sum_w gh_w (x_w - om) r_w.
// With y_w = x_w - Re om, rounded once (x_w and Re om in separate sums would
// cancel by |om| / |x - om|, up to 500 on branch A), it is up to four
// frequencies (FACTOR) the sum of (y_w c1_w + c2_w) r_w with the constants
// c1_w = gh_w vcoul conj(e om) and c2_w = -i Im om c1_w of a pair: two FMAs per
// term for the factor, two for the sum, and per column six products per
// frequency.  With more, whose constants would spill, vcoul conj(e om)
// (S - i Im om R) with S = sum_w gh_w (y_w r_w) and R = sum_w gh_w r_w.
// Either way the loop needs x and gh only, in scalar registers: x gh itself,
// 12 complex values per column at nfreq 3 from the scalar cache, took 15
// scalar loads with their waits per column against 4 here.  256 bands x 8192
// rows x 409 columns, whole adjoint at nfreq 1, 2, 4: 1977 -> 1806, 2740 ->
// 2647, 4452 -> 4252 us (FACTOR at 5, 6 and 8 instead ran 6-20 % slower than
// before).  The frequencies of the band tile stay in scalar registers where
// HOLD.
template <int NW, int BT, bool AM>
struct BandsFast {
    static constexpr int G = bands_group(NW, BT);
    static constexpr int Kt = G * NW;
    static constexpr bool FACTOR = NW <= 4 && BT > 1;
    static constexpr bool HOLD = NW * BT <= 20;
    double xs[BT * NW];
    cplx gh[NW];
    cplx om_next, e_next;

    __device__ __forceinline__ void frequencies(int n, int nb, gptr<double> wx)
    {
#pragma unroll
        for (int u = 0; u < BT; ++u)
#pragma unroll
            for (int w = 0; w < NW; ++w) xs[u * NW + w] = wx[(size_t)w * nb + n + u];
    }
    __device__ __forceinline__ void start(int nb, int ng, int n0, int gc, int p,
                                          gptr<double2> ieps, gptr<double2> wt, gptr<double> wx,
                                          const double2 *__restrict__ ga)
    {
        om_next = cload(wt + (size_t)p * ng + gc);
        e_next = cload(ieps + (size_t)p * ng + gc);
        if (HOLD) frequencies(n0, nb, wx);
#pragma unroll
        for (int w = 0; w < NW; ++w) gh[w] = half_of(ga, w);
    }
    // Columns [p, end) of the wave's [.., p_hi).
    __device__ __forceinline__ void columns(int p, int end, int p_hi, int nb, int ng, int n0,
                                            int gc, double vc, gptr<double2> aqsm,
                                            gptr<double2> ieps, gptr<double2> wt,
                                            gptr<double> wx, const cplx (&an)[BT],
                                            AmCtx<BT> &amc, cplx (&acc)[BT])
    {
        const uint32_t row_bytes = (uint32_t)ng * (uint32_t)sizeof(double2);
        Walker am_at;
        am_at.start((uint64_t)(aqsm + (size_t)n0 * ng + p));
        for (; p < end; ++p) {
            // om and e of the next column are loaded one iteration ahead, so
            // their latency overlaps this column's arithmetic
            const cplx om = om_next, e = e_next;
            const int pn = p + 1 < p_hi ? p + 1 : p;
            om_next = cload(wt + (size_t)pn * ng + gc);
            e_next = cload(ieps + (size_t)pn * ng + gc);
            cplx am[BT];
#pragma unroll
            for (int u = 0; u < BT; ++u) am[u] = am_at.complex(u * row_bytes);
            am_at.advance(sizeof(double2));
            if (!HOLD) frequencies(opaque_uniform(n0), nb, wx);
            const double a = om.re, b = om.im;
            const double wi2 = b * b;
            const double wtr = fma(a, a, wi2);
            const double thr = branch_a_threshold(wtr);
            const uint64_t narrow = __builtin_amdgcn_ballot_w64(!(wi2 >= kMinUnclampedWi2));
            const cplx vce = cmake(vc * e.re, -(vc * e.im));  // vcoul conj(e)
            const cplx vcw = cmul(vce, cmake(a, -b));         // vcoul conj(e om)
            cplx c1[FACTOR ? NW : 1], c2[FACTOR ? NW : 1];
            if constexpr (FACTOR) {
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    c1[w] = cmul(gh[w], vcw);
                    c2[w] = cmake(b * c1[w].im, -b * c1[w].re);
                }
            }
#pragma unroll
            for (int u0 = 0; u0 < BT; u0 += G) {
                double d[Kt], c[Kt], r[Kt];
#pragma unroll
                for (int k = 0; k < Kt; ++k) {
                    const double dr = xs[u0 * NW + k] - a;
                    d[k] = fma(dr, dr, wi2);  // unclamped: see batch_prefix
                }
                const double all = batch_prefix<Kt>(d, c);
                batch_back<Kt>(d, c, all, r);
                if (__builtin_expect(batch_misses(all, narrow) != 0, 0)) one_by_one<Kt>(d, r);
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    // the first frequency starts the sums through a select,
                    // the others add under an execution mask written by the
                    // compare (all lanes are active here)
                    const int k0 = u * NW;
                    const double r0 = mask_keep(d[k0] > thr, r[k0]);
                    const double y0 = subtract_again(xs[u0 * NW + k0], a);
                    cplx vz;
                    if constexpr (FACTOR) {
                        vz = cmake(r0 * fma(y0, c1[0].re, c2[0].re),
                                   r0 * fma(y0, c1[0].im, c2[0].im));
#pragma unroll
                        for (int w = 1; w < NW; ++w) {
                            double y;
                            cplx f;
                            asm("v_cmpx_gt_f64_e32 vcc, %[d], %[thr]\n\t"
                                "v_add_f64 %[y], %[x], -%[a]\n\t"
                                "v_fma_f64 %[fr], %[y], %[c1r], %[c2r]\n\t"
                                "v_fma_f64 %[fi], %[y], %[c1i], %[c2i]\n\t"
                                "v_fma_f64 %[zr], %[r], %[fr], %[zr]\n\t"
                                "v_fma_f64 %[zi], %[r], %[fi], %[zi]\n\t"
                                "s_mov_b64 exec, -1"
                                : [y] "=&v"(y), [fr] "=&v"(f.re), [fi] "=&v"(f.im),
                                  [zr] "+v"(vz.re), [zi] "+v"(vz.im)
                                : [d] "v"(d[k0 + w]), [thr] "v"(thr), [r] "v"(r[k0 + w]),
                                  [x] "s"(xs[u0 * NW + k0 + w]), [a] "v"(a), [c1r] "v"(c1[w].re),
                                  [c1i] "v"(c1[w].im), [c2r] "v"(c2[w].re), [c2i] "v"(c2[w].im)
                                : "vcc");
                        }
                    } else {
                        cplx S = cscale(r0 * y0, gh[0]), R = cscale(r0, gh[0]);
#pragma unroll
                        for (int w = 1; w < NW; ++w) {
                            double ry;
                            asm("v_cmpx_gt_f64_e32 vcc, %[d], %[thr]\n\t"
                                "v_add_f64 %[ry], %[x], -%[a]\n\t"
                                "v_mul_f64 %[ry], %[r], %[ry]\n\t"
                                "v_fma_f64 %[rr], %[r], %[gr], %[rr]\n\t"
                                "v_fma_f64 %[ri], %[r], %[gi], %[ri]\n\t"
                                "v_fma_f64 %[sr], %[ry], %[gr], %[sr]\n\t"
                                "v_fma_f64 %[si], %[ry], %[gi], %[si]\n\t"
                                "s_mov_b64 exec, -1"
                                : [ry] "=&v"(ry), [sr] "+v"(S.re), [si] "+v"(S.im),
                                  [rr] "+v"(R.re), [ri] "+v"(R.im)
                                : [d] "v"(d[k0 + w]), [thr] "v"(thr), [r] "v"(r[k0 + w]),
                                  [x] "s"(xs[u0 * NW + k0 + w]), [a] "v"(a), [gr] "s"(gh[w].re),
                                  [gi] "s"(gh[w].im)
                                : "vcc");
                        }
                        // S - i Im om R
                        vz = cmul(vcw, cmake(fma(b, R.im, S.re), fma(-b, R.re, S.im)));
                    }
                    cmac(acc[u0 + u], am[u0 + u], vz);
                    if constexpr (AM) am_put(amc, p, u0 + u, an[u0 + u], vz);
                }
                // one group's reciprocal chain at a time (register pressure)
                if (G < BT) __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (AM) am_column_done(amc, p, end);
        }
    }
};

// Generic form of a wave's columns: occupied bands (exchange terms) and a
// ragged last tile, band by band.
template <int NW, int BT, bool AM>
struct BandsGeneric {
    double xs[BT][NW];
    uint32_t row_off[BT];  // of the bands' aqsmtemp rows; past nb the last row again
    cplx om_next, e_next;

    __device__ __forceinline__ void start(int nb, int ng, int n0, int gc, int p,
                                          gptr<double2> ieps, gptr<double2> wt, gptr<double> wx)
    {
        om_next = cload(wt + (size_t)p * ng + gc);
        e_next = cload(ieps + (size_t)p * ng + gc);
#pragma unroll
        for (int u = 0; u < BT; ++u) {
            const int n = n0 + u < nb ? n0 + u : nb - 1;
            row_off[u] = (uint32_t)(n - n0) * (uint32_t)ng * (uint32_t)sizeof(double2);
#pragma unroll
            for (int w = 0; w < NW; ++w) xs[u][w] = wx[(size_t)w * nb + n];
        }
    }
    // Columns [p, end) of the wave's [.., p_hi).
    __device__ __forceinline__ void columns(int p, int end, int p_hi, int n_end, int nv, int ng,
                                            int n0, int gc, double vc, gptr<double2> aqsm,
                                            gptr<double2> ieps, gptr<double2> wt,
                                            const double2 *__restrict__ ga,
                                            const double2 *__restrict__ gs,
                                            const cplx (&an)[BT], AmCtx<BT> &amc,
                                            cplx (&acc)[BT])
    {
        Walker am_at;
        am_at.start((uint64_t)(aqsm + (size_t)n0 * ng + p));
        for (; p < end; ++p) {
            const cplx om = om_next, e = e_next;
            const int pn = p + 1 < p_hi ? p + 1 : p;
            om_next = cload(wt + (size_t)pn * ng + gc);
            e_next = cload(ieps + (size_t)pn * ng + gc);
            cplx am[BT];
#pragma unroll
            for (int u = 0; u < BT; ++u) am[u] = am_at.complex(row_off[u]);
            am_at.advance(sizeof(double2));
            const PairState ps = make_pair(om, e, vc);
            const cplx vce = cmake(ps.ve.re, -ps.ve.im);  // vcoul conj(e)
#pragma unroll
            for (int u = 0; u < BT; ++u) {
                cplx vz = cmake(0.0, 0.0);
                if (n0 + u < n_end) {  // wave-uniform, like the next
                    cplx Z, W;
                    if (n0 + u < nv) band_zw<NW, true, false>(xs[u], ga, gs, ps, Z, W);
                    else band_zw<NW, false, false>(xs[u], ga, gs, ps, Z, W);
                    vz = cmul(vce, Z);
                    cmac(acc[u], am[u], vz);
                }
                if constexpr (AM) am_put(amc, p, u, an[u], vz);
            }
            if constexpr (AM) am_column_done(amc, p, end);
        }
    }
};

// Workgroup = BT bands x 256 rows (four 64-row tiles) x one segment of the G'
// range, which PW waves per row tile share; band tile fastest (neighbouring
// workgroups share the rows of wtilde/I_eps), then row block, then segment.
// One segment writes daqsntemp itself, several write partial sums (grad_an
// may be NULL: daqsmtemp only).  With AM, also the daqsmtemp partials of the
// workgroup's bands, rows and columns.  The columns go in steps of kAmCols
// per wave, the same number for every wave, since a step ends with a barrier.
template <int NW, int BT, int PW, bool AM>
__global__ void __launch_bounds__(kBwdThreads * PW)
__attribute__((amdgpu_waves_per_eu(PW > 1 ? 4 : AM ? GPP_BWD_BANDS_AM_WAVES
                                                   : GPP_BWD_BANDS_WAVES)))
bwd_bands(int nb, int nv, int ng, int np, long nwg, int nbt, int single, int ngb, int nps,
          const double2 *__restrict__ aqsm, const double2 *__restrict__ aqsn,
          const double2 *__restrict__ ieps, const double2 *__restrict__ wt,
          const double *__restrict__ vcoul, const double *__restrict__ wx,
          const double2 *__restrict__ ga, const double2 *__restrict__ gs,
          double2 *__restrict__ grad_an, double2 *__restrict__ am_part)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wid = wave % kBwdWaves, range = wave / kBwdWaves;
    const long wg = xcd_remap(blockIdx.x, gridDim.x);
    if (wg >= nwg) return;  // the whole workgroup leaves together
    const long per_seg = (long)ngb * nbt;
    const int seg = __builtin_amdgcn_readfirstlane((int)(wg / per_seg));
    const long in_seg = wg - (long)seg * per_seg;
    const int gblk = __builtin_amdgcn_readfirstlane((int)(in_seg / nbt));
    // the first `single` tiles hold one (occupied) band, the others BT
    const int tile = __builtin_amdgcn_readfirstlane((int)(in_seg - (long)gblk * nbt));
    const int n0 = tile < single ? tile : single + (tile - single) * BT;
    const int n_end = tile < single ? tile + 1 : nb;
    double2 *const dst = grad_an ? grad_an + (size_t)seg * nb * ng : nullptr;
    const int g = gblk * kRowsPerBlock + wid * kWave + lane;
    const bool valid = g < ng;
    const int gc = valid ? g : ng - 1;

    // the wave's columns: range `range` of the segment's
    const int seg_lo = __builtin_amdgcn_readfirstlane((int)((long)np * seg / nps));
    const int seg_hi = __builtin_amdgcn_readfirstlane((int)((long)np * (seg + 1) / nps));
    const int per = (seg_hi - seg_lo + PW - 1) / PW;
    const int lo_r = seg_lo + range * per;
    const int p_lo = lo_r < seg_hi ? lo_r : seg_hi;
    const int p_hi = p_lo + per < seg_hi ? p_lo + per : seg_hi;

    // LDS: the daqsmtemp stages of the PW ranges; afterwards the ranges'
    // daqsntemp sums
    constexpr size_t stage_bytes = AM ? sizeof(AmStage<BT>) * PW : 0;
    constexpr size_t sums_bytes = sizeof(double2) * (PW - 1) * kBwdWaves * BT * kWave;
    constexpr size_t lds_bytes = stage_bytes > sums_bytes ? stage_bytes : sums_bytes;
    __shared__ __align__(16) unsigned char lds[lds_bytes > 0 ? lds_bytes : 16];

    AmCtx<BT> amc;
    amc.st = AM ? reinterpret_cast<AmStage<BT> *>(lds) + range : nullptr;
    amc.part = am_part;
    amc.wid = wid;
    amc.lane = lane;
    amc.gblk = gblk;
    amc.n0 = n0;
    amc.n_end = n_end;
    amc.nb = nb;
    amc.np = np;

    cplx an[BT];
#pragma unroll
    for (int u = 0; u < BT; ++u) {
        an[u] = cmake(0.0, 0.0);
        if (AM && n0 + u < nb) an[u] = cload(aqsn + (size_t)(n0 + u) * ng + gc);
    }
    cplx acc[BT];
#pragma unroll
    for (int u = 0; u < BT; ++u) acc[u] = cmake(0.0, 0.0);
    const int step = AM ? kAmCols : per;
    const double vc = valid ? vcoul[gc] : 0.0;
    if (n0 >= nv && n0 + BT <= nb) {
        BandsFast<NW, BT, AM> f;
        f.start(nb, ng, n0, gc, p_lo < np ? p_lo : np - 1, as_global(ieps), as_global(wt),
                as_global(wx), ga);
        for (int at = 0; at < per; at += step) {
            const int p = p_lo + at < p_hi ? p_lo + at : p_hi;
            const int end = p + step < p_hi ? p + step : p_hi;
            amc.first = p;
            f.columns(p, end, p_hi, nb, ng, n0, gc, vc, as_global(aqsm), as_global(ieps),
                      as_global(wt), as_global(wx), an, amc, acc);
            if constexpr (AM) am_flush(amc, end);
        }
    } else {
        BandsGeneric<NW, BT, AM> f;
        f.start(nb, ng, n0, gc, p_lo < np ? p_lo : np - 1, as_global(ieps), as_global(wt),
                as_global(wx));
        for (int at = 0; at < per; at += step) {
            const int p = p_lo + at < p_hi ? p_lo + at : p_hi;
            const int end = p + step < p_hi ? p + step : p_hi;
            amc.first = p;
            f.columns(p, end, p_hi, n_end, nv, ng, n0, gc, vc, as_global(aqsm), as_global(ieps),
                      as_global(wt), ga, gs, an, amc, acc);
            if constexpr (AM) am_flush(amc, end);
        }
    }
    if constexpr (PW > 1) {
        // the ranges' sums into range 0's, in order
        double2 *const sums = reinterpret_cast<double2 *>(lds);
        __syncthreads();
        if (range > 0) {
#pragma unroll
            for (int u = 0; u < BT; ++u)
                sums[(((range - 1) * kBwdWaves + wid) * BT + u) * kWave + lane] =
                    make_double2(acc[u].re, acc[u].im);
        }
        __syncthreads();
        if (range > 0) return;
#pragma unroll
        for (int k = 0; k < PW - 1; ++k)
#pragma unroll
            for (int u = 0; u < BT; ++u) {
                const double2 v = sums[((k * kBwdWaves + wid) * BT + u) * kWave + lane];
                acc[u] = cadd(acc[u], cmake(v.x, v.y));
            }
    }
    if (dst && valid) {
#pragma unroll
        for (int u = 0; u < BT; ++u) {
            const int n = n0 + u;
            if (n < n_end) dst[(size_t)n * ng + g] = make_double2(acc[u].re, acc[u].im);
        }
    }
}

// daqsmtemp[n][p] = sum over row blocks of the partials (p < np), 0 for
// columns np..ncouls-1.  One thread per output element, fixed order.  The
// nb * np sums come first in the grid and the zero columns after them, so
// that the workgroups which read run together instead of one in twenty
// across the whole grid.
__global__ void reduce_am(int nb, int ng, int np, int ngb, const double2 *__restrict__ part,
                          double2 *__restrict__ grad_am)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long nsum = (long)nb * np;
    if (i < nsum) {
        const int n = (int)(i / np), col = (int)(i - (long)n * np);
        double re = 0.0, im = 0.0;
        // unrolled so that eight loads are in flight; the additions keep
        // their order
#pragma unroll 8
        for (int b = 0; b < ngb; ++b) {
            const double2 v = part[((size_t)b * nb + n) * np + col];
            re += v.x;
            im += v.y;
        }
        grad_am[(size_t)n * ng + col] = make_double2(re, im);
        return;
    }
    const long j = i - nsum, nz = ng - np;
    if (nz <= 0 || j >= (long)nb * nz) return;
    const int n = (int)(j / nz);
    grad_am[(size_t)n * ng + np + (j - (long)n * nz)] = make_double2(0.0, 0.0);
}

// daqsntemp = sum of the nps segment partials, in segment order.
__global__ void reduce_an(long nbg, int nps, const double2 *__restrict__ part,
                          double2 *__restrict__ grad_an)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nbg) return;
    double re = 0.0, im = 0.0;
#pragma unroll 4
    for (int s = 0; s < nps; ++s) {
        const double2 v = part[(size_t)s * nbg + i];
        re += v.x;
        im += v.y;
    }
    grad_an[i] = make_double2(re, im);
}

__global__ void fill_zero_n(double2 *a, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = make_double2(0.0, 0.0);
}

// Whether a pairs workgroup's four waves share one tile: where that is less
// work on the fullest compute unit, a tile's fixed part (set-up, gradients)
// counting as kPairsTileBands bands; at most 1/64 less counts as equal.
// Whole adjoint, rows x bands x columns (nfreq), apart and shared: 512 x 32 x
// 64 (3) 41.4 and 37.4 us, 1400 x 64 x 102 (5) 118.5 and 107.9, 3001 x 101 x
// 150 (5) 354 and 338; but 3072 x 64 x 102 (3) 128.2 and 130.2, 2048 x 16 x 102
// (3) 60.2 and 62.0.
constexpr int kPairsTileBands = 3;
static bool pairs_share(long gtiles, int ngb, int np, int nb)
{
    const auto cost = [](long blocks, double bands) {
        return (double)((blocks + kBandsCUs - 1) / kBandsCUs) * (bands + kPairsTileBands);
    };
    return cost(gtiles * np, (double)nb / kBwdWaves) < cost((long)ngb * np, nb) * (1 - 1.0 / 64);
}

BwdGeometry bwd_geometry(const Dims32 &d)
{
    BwdGeometry geo{};
    geo.gh_elems = d.nw;
    geo.xgh_elems = (size_t)d.nw * d.nb;
    if (d.nb > 0 && d.ng > 0 && d.np > 0) {
        geo.ngb = (d.ng + kRowsPerBlock - 1) / kRowsPerBlock;
        const long gtiles = (d.ng + kWave - 1) / kWave;
        geo.share_pairs = pairs_share(gtiles, geo.ngb, d.np, d.nb);
        geo.pair_blocks = (geo.share_pairs ? gtiles : geo.ngb) * d.np;
        geo.nbt = (d.nb + kBandTile - 1) / kBandTile;
        geo.ngt = geo.ngb * kBwdWaves;
        // Split the p loop into segments when one pass has too few waves:
        // every wave walks its whole p range, so the last partial round of
        // a short grid leaves most SIMDs idle.  Aim at kBandsRounds rounds
        // of the MI355X's resident bands waves, each segment at least
        // kMinSegCols columns long.
        const long per_seg = (long)geo.ngt * geo.nbt;
        const long want = (long)kBandsRounds * kBandsWaveSlots;
        long nps = (want + per_seg - 1) / per_seg;
        const long max_nps = d.np / kMinSegCols > 1 ? d.np / kMinSegCols : 1;
        geo.nps = (int)(nps < max_nps ? nps : max_nps);
        geo.band_tiles = per_seg * geo.nps;
        geo.short_bands = geo.band_tiles < kBandsShortBelow;
        const long per_band = (long)geo.ngb * geo.nps;
        geo.tile_bands = !geo.short_bands                  ? kBandTile
                         : per_band * d.nb <= kBandsCUs ? kTinyTile
                                                           : kShortTile;
        const int nocc = d.nv < d.nb ? d.nv : d.nb, bt = geo.tile_bands;
        const bool few = geo.short_bands && per_band * ((d.nb + bt - 1) / bt) <= kSingleBlocks;
        geo.single = nocc <= kSingleOccupied || few ? nocc : 0;
        geo.nbt = geo.single + (d.nb - geo.single + bt - 1) / bt;
        geo.band_blocks = (long)geo.ngb * geo.nbt * geo.nps;
        geo.am_part_elems = (size_t)geo.ngb * d.nb * d.np;
        geo.an_part_elems = geo.nps > 1 ? (size_t)geo.nps * d.nb * d.ng : 0;
    }
    // complex elements, each 16 bytes; sections 256-byte aligned
    auto up = [](size_t e) { return (e * sizeof(double2) + 255) / 256 * 256; };
    geo.workspace_bytes = up(geo.gh_elems) + up(geo.xgh_elems) + up(geo.am_part_elems) +
                          up(geo.an_part_elems);
    if (geo.workspace_bytes == 0) geo.workspace_bytes = 256;
    return geo;
}

template <int NW>
static hipError_t launch_bwd_nw(const Dims32 &d, const BwdGeometry &geo, const DevInputs &in,
                                const double2 *ga, const double2 *gs, const BwdOutputs &out,
                                char *ws, hipStream_t st)
{
    auto up = [](size_t e) { return (e * sizeof(double2) + 255) / 256 * 256; };
    // the first two sections (once the scaled upstream gradient) lie unused:
    // the workspace keeps its size
    char *const after = ws + up(geo.gh_elems) + up(geo.xgh_elems);
    double2 *am_part = reinterpret_cast<double2 *>(after);
    double2 *an_part = reinterpret_cast<double2 *>(after + up(geo.am_part_elems));
    hipError_t e;
    if (out.grad_wt || out.grad_ieps) {
        const auto kernel = geo.share_pairs ? bwd_pairs<NW, true> : bwd_pairs<NW, false>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)geo.pair_blocks), dim3(kBwdThreads), 0, st,
                           d.nb, d.nv, d.ng, d.np, geo.pair_blocks, in.aqsm, in.aqsn, in.ieps,
                           in.wt, in.vcoul, in.wx, ga, gs, out.grad_wt, out.grad_ieps);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (out.grad_an || out.grad_am) {
        double2 *an_dst = !out.grad_an ? nullptr : (geo.nps > 1 ? an_part : out.grad_an);
        const dim3 grid((unsigned)geo.band_blocks);
        const dim3 block(kBwdThreads * (geo.short_bands ? kShortRanges : 1));
        double2 *const am_dst = out.grad_am ? am_part : nullptr;
        const auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, 0, st, d.nb, d.nv, d.ng, d.np, geo.band_blocks,
                               geo.nbt, geo.single, geo.ngb, geo.nps, in.aqsm, in.aqsn, in.ieps, in.wt,
                               in.vcoul, in.wx, ga, gs, an_dst, am_dst);
            return hipGetLastError();
        };
        if (geo.tile_bands == kTinyTile)
            e = out.grad_am ? launch(bwd_bands<NW, kTinyTile, kShortRanges, true>)
                            : launch(bwd_bands<NW, kTinyTile, kShortRanges, false>);
        else if (geo.short_bands)
            e = out.grad_am ? launch(bwd_bands<NW, kShortTile, kShortRanges, true>)
                            : launch(bwd_bands<NW, kShortTile, kShortRanges, false>);
        else
            e = out.grad_am ? launch(bwd_bands<NW, kBandTile, 1, true>)
                            : launch(bwd_bands<NW, kBandTile, 1, false>);
        if (e != hipSuccess) return e;
        if (out.grad_an && geo.nps > 1) {
            const long nbg = (long)d.nb * d.ng;
            hipLaunchKernelGGL(reduce_an, dim3((unsigned)((nbg + 255) / 256)), dim3(256), 0, st,
                               nbg, geo.nps, an_part, out.grad_an);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    if (out.grad_am) {
        const long n = (long)d.nb * d.ng;
        hipLaunchKernelGGL(reduce_am, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d.nb,
                           d.ng, d.np, geo.ngb, am_part, out.grad_am);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_bwd(const Dims32 &d, const DevInputs &in, const double2 *ga,
                      const double2 *gs, const BwdOutputs &out, void *workspace, hipStream_t st)
{
    const BwdGeometry geo = bwd_geometry(d);
    if (geo.pair_blocks == 0) {
        // an empty sum: every requested gradient is zero
        const long npg = (long)d.np * d.ng, nbg = (long)d.nb * d.ng;
        double2 *outs[4] = {out.grad_wt, out.grad_ieps, out.grad_an, out.grad_am};
        const long lens[4] = {npg, npg, nbg, nbg};
        for (int k = 0; k < 4; ++k) {
            if (!outs[k] || lens[k] == 0) continue;
            hipLaunchKernelGGL(fill_zero_n, dim3((unsigned)((lens[k] + 255) / 256)), dim3(256), 0,
                               st, outs[k], lens[k]);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    char *ws = static_cast<char *>(workspace);
    switch (d.nw) {
    case 1: return launch_bwd_nw<1>(d, geo, in, ga, gs, out, ws, st);
    case 2: return launch_bwd_nw<2>(d, geo, in, ga, gs, out, ws, st);
    case 3: return launch_bwd_nw<3>(d, geo, in, ga, gs, out, ws, st);
    case 4: return launch_bwd_nw<4>(d, geo, in, ga, gs, out, ws, st);
    case 5: return launch_bwd_nw<5>(d, geo, in, ga, gs, out, ws, st);
    case 6: return launch_bwd_nw<6>(d, geo, in, ga, gs, out, ws, st);
    case 7: return launch_bwd_nw<7>(d, geo, in, ga, gs, out, ws, st);
    case 8: return launch_bwd_nw<8>(d, geo, in, ga, gs, out, ws, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace gpp
