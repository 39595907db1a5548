// gpp_fwd_shape.h -- tile shape of the forward tile kernels per frequency
// count, shared by the plain forward, the batched flat grid and the
// batched plan's tile counts (host and device code).
#pragma once

namespace gpp {

// G' columns per wave tile, and bands per batch-inverted group, so that a group holds
// columns x bands x nfreq <= 12 denominators.  More columns let each
// aqsntemp load serve more terms; the accumulators (columns x nfreq x 4
// doubles) bound how many fit.  Pairs (columns, bands) for nfreq = 1..8;
// nfreq 3 takes GPP_FWD_COLS x GPP_FWD_BANDS.  Measured on MI355X at 512
// bands, 32768 rows, 1638 columns: nfreq 1 with 2 x 2 15.4 ms, 4 x 2 15.5, 3 x 4
// 15.3, 2 x 4 16.5 and 3 x 2 14.1, whose longer group of the short grids' form
// needs scratch, though (128 x 2000 x 100: 34.7 us against 27.7); nfreq 2 with
// 3 x 2 22.6 ms, 2 x 3 23.4, 2 x 2 23.2, 3 x 1 23.6; nfreq 5 and 6 with 2-band
// groups 20 % and 15 % faster than 1-band ones; nfreq 4 with 1 x 2 faster than
// 1 x 3 or 2 x 1.
#ifndef GPP_FWD_COLS
#define GPP_FWD_COLS 2
#endif
#ifndef GPP_FWD_BANDS
#define GPP_FWD_BANDS 2
#endif
#ifndef GPP_FWD_SHAPE
#define GPP_FWD_SHAPE 2, 2, 3, 2, GPP_FWD_COLS, GPP_FWD_BANDS, 1, 2, 1, 2, 1, 2, 1, 1, 1, 1
#endif
constexpr int kFwdShape[16] = {GPP_FWD_SHAPE};
constexpr int fwd_cols(int nw) { return kFwdShape[2 * (nw - 1)]; }
constexpr int fwd_bands(int nw) { return kFwdShape[2 * (nw - 1) + 1]; }
constexpr bool fwd_shapes_fit()
{
    for (int nw = 1; nw <= 8; ++nw)
        if (fwd_cols(nw) < 1 || fwd_bands(nw) < 1 || fwd_cols(nw) * fwd_bands(nw) * nw > 12)
            return false;
    return true;
}
static_assert(fwd_shapes_fit(), "a forward tile's batch inversion holds at most 12 denominators");
// Minimum waves per SIMD (a VGPR cap) of the forward tile kernels for
// nfreq = 1..8.  nfreq 2 capped at 168 VGPRs (3 waves; 8 of them spilled, outside
// the hot loop) against 176 (2 waves): 23.0 and 24.3 ms at 512 bands x 32768 rows
// x 1638 columns, 2.77 and 2.86 at 300 x 12000 x 900.  nfreq 4 capped at 96 (5
// waves; 12 spilled) against 100 (4): equal there, 5.24 and 5.32 ms at 300 x 12000
// x 900.  At 3 (154), 7 (120) and 8 (128) the cap is what the compiler takes
// without it (times equal to 1 %); it keeps a change from crossing the line.
// nfreq 1 capped for 6 waves and nfreq 6 for 4 ran 0.9 % and 16 % slower.
#ifndef GPP_FWD_MIN_WAVES
#define GPP_FWD_MIN_WAVES 1, 3, 3, 5, 1, 1, 4, 4
#endif
constexpr int kFwdMinWaves[8] = {GPP_FWD_MIN_WAVES};
constexpr int fwd_min_waves(int nw) { return kFwdMinWaves[nw - 1]; }

// Band chunks of the plain forward's tiles.  The waves an XCD holds at
// once start and end together, so a value one tile reads comes back to the
// next tiles only after a whole tile's band loop of other traffic (about
// 8 KB per band for the resident tiles of one XCD); splitting the band
// loop into chunks of at most GPP_FWD_CHUNK_BANDS bands keeps that inside
// the XCD's 4 MB L2.  Every chunk of a tile adds its own partial sums (the
// sums are linear in the bands), so chunks cost their own set-up, exchange
// sums and partial row.  0 turns chunking off.  Chunks hold whole band
// groups except the last.
#ifndef GPP_FWD_CHUNK_BANDS
#define GPP_FWD_CHUNK_BANDS 512
#endif
inline void fwd_band_chunks(int nb, int nw, int &nchunk, int &chunk_bands)
{
    nchunk = 1;
    chunk_bands = nb;
    if (GPP_FWD_CHUNK_BANDS <= 0 || nb <= GPP_FWD_CHUNK_BANDS) return;
    const int bu = fwd_bands(nw);
    const int want = (nb + GPP_FWD_CHUNK_BANDS - 1) / GPP_FWD_CHUNK_BANDS;
    int cb = (nb + want - 1) / want;
    cb = (cb + bu - 1) / bu * bu;
    chunk_bands = cb;
    nchunk = (nb + cb - 1) / cb;
}

// Above kSplitBelow tiles but with few workgroups per compute unit, the
// last of them leave much of the GPU idle: finer band chunks even that out,
// until a tile's fixed part (set-up, epilogue: worth kTileBands bands) costs
// more.  The chunk count in [1, kMaxFineChunks] with the least work on the
// fullest compute unit, at most 1/64 less than with fewer chunks counting as
// equal.  Measured at 128 bands x 4096 rows x 204 columns, nfreq 3 (1632
// workgroups of 4 tiles): 156.0 us in one chunk, 150.8 in two, 165.4 in
// four; 64 x 2048 x 102 at nfreq 5 (816): 47.3, 45.8 and 50.6.
constexpr int kTileBands = 7;
constexpr int kMaxFineChunks = 4;
inline int fwd_fine_chunks(long tiles, int bands, int cus)
{
    int best = 1;
    double least = 0.0;
    for (int m = 1; m <= kMaxFineChunks; ++m) {
        const long per_cu = ((tiles * m + 3) / 4 + cus - 1) / cus;
        const double cost = (double)per_cu * ((double)bands / m + kTileBands);
        if (m == 1 || cost < least * (1.0 - 1.0 / 64)) {
            best = m;
            least = cost;
        }
    }
    return best;
}

// Terms of an occupied band that share a batch inversion, at most: one group's
// values must fit beside both sums' accumulators.  With 4 in place of 3, 200
// bands x 8192 rows x 400 columns (2 occupied) at nfreq 4 took 1093 us against
// 1051, and with 150 occupied bands at 4096 x 200, nfreq 8, 1321 against 1271; 2
// measured as 3.
constexpr int kOccTerms = 3;

// The most partial rows a grid with finer chunks makes (16895 tiles in two, at
// 486 bands and more), and the most tiles a call has at any frequency count (one
// column each).
constexpr long kFineRows = 8448;
inline long fwd_most_tiles(long gtiles, int np, int nb)
{
    const int chunks = GPP_FWD_CHUNK_BANDS > 0 ? (nb - 1) / GPP_FWD_CHUNK_BANDS + 1 : 1;
    return gtiles * np * chunks;
}

// The split form of the forward's tile kernel, for grids of fewer than
// kSplitBelow tiles (gpp_fwd.hip).  Bands per batch-inverted group there: a
// 16-wave workgroup holds its waves to 128 VGPRs.
#ifndef GPP_FWD_SPLIT_BELOW
#define GPP_FWD_SPLIT_BELOW 2048
#endif
constexpr long kSplitBelow = GPP_FWD_SPLIT_BELOW;
#ifndef GPP_FWD_SPLIT_BANDS
#define GPP_FWD_SPLIT_BANDS 4, 1, 1, 2, 2, 1, 1, 1
#endif
constexpr int kSplitBands[8] = {GPP_FWD_SPLIT_BANDS};
constexpr int split_bands(int nw) { return kSplitBands[nw - 1]; }
// An occupied band's cost in unoccupied ones, by which the split form deals
// bands out to waves (3 and 6 measured slower at 61 x 777 x 38 and 100 x 600 x
// 40).
constexpr int kOccupiedCost = 4;

}  // namespace gpp
