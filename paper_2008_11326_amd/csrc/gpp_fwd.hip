// gpp_fwd.hip -- forward GPP reduction on gfx950 (fp64 vector ALU, no MFMA).
//
// Work decomposition.  A wave owns one to three G' columns (by the frequency
// count) and 64 consecutive G rows g (one per lane) and walks every
// band n sequentially, as in the band-inner loop order of Sec. III v4
// (bands serial per thread keeps the g-fastest arrays coalesced and reads
// wtilde/I_eps once); each aqsntemp[n][g] a lane loads serves all
// of them.  Within a wave p and n are uniform, so aqsmtemp[n][p] and
// wx_array[w][n] are scalar loads; the frequencies are register-blocked
// (all NW in one pass, none of v5's recompute).
//
// Per lane, e = I_eps[p][g] and vcoul[g] are constant over the band loop,
// so they multiply once at the end.  For a branch-A term,
//   om / (x - om) = (x om - |om|^2) / |x - om|^2 = r (x om - wtr),
// so with Qm = aqsntemp[n][g] conj(aqsmtemp[n][p]) the lane accumulates
//   P1[w] += (r x) Qm,  P2[w] += r Qm
// and ends with  achtemp += vcoul/2 * e * (om P1 - wtr P2).  The branch-A
// test is one compare against a per-(p,g) threshold that reproduces the
// specification exactly (gpp_device.h).  r = 1/wdiffr needs no IEEE divide
// (the v1 idea); the reciprocals of a group of BU bands, all columns and
// frequencies, come from a single hardware reciprocal by batch inversion
// (gpp_device.h: unclamped denominators, a lane test on (Im om)^2 for the
// product's range), and the branch-A test is the execution mask around
// each term's four fused multiply-adds, so a masked term adds nothing and
// costs no select.  Occupied bands (n < nvband) run after the others, both
// their terms from batch inversions of |x - om|^2 |x + om|^2 instead of complex
// divides (gpp_fwd_tile.h).  Above 512 bands each tile's band loop is split into
// chunks, each a tile of its own.
//
// What bounds it.  Large grids: the fp64 vector ALU at the clock the part
// holds under that load (1024 bands x 65536 rows x 3276 columns, nfreq 3:
// 260.0 ms before and 250.3 ms after the loop's loads moved ahead of their
// use, its addresses to the scalar unit and its reciprocal chain into two
// halves; 12.6 instructions per term in 0.89-0.91 of the issue slots, 0.85
// before).  Short grids: launches, first loads and too few waves, hence the
// split form, in which 2, 4 or 8 waves of a 16-wave workgroup share a tile's
// bands (512 rows x 32 bands x 64 columns, nfreq 3: 24.1 us with four waves of
// a tile each and two reduction stages, 10.6 so).
//
// Each workgroup writes one partial per output into the workspace; one or two
// reduction kernels then sum the partials in a fixed order (the separate
// reduction kernel of Sec. II-A), so results are bitwise reproducible.
#include "gpp_device.h"
#include "gpp_fwd_tile.h"
#include "gpp_internal.h"

namespace gpp {

constexpr int kFwdWaves = 4;      // waves per workgroup of the long form
constexpr int kSplitWaves = 16;   // and of the split form
constexpr long kCUs = 256;        // compute units of the MI355X
constexpr int kRedThreads = 256;  // first reduction stage
constexpr long kRedBlocks = 512;
constexpr int kFinalThreads = 1024;

// G' columns per wave tile and bands per batch-inverted group (K = columns
// x bands x nfreq reciprocals from one hardware reciprocal) come from
// fwd_cols and fwd_bands, and a cap on VGPRs through a minimum number of
// waves per SIMD from fwd_min_waves (gpp_fwd_shape.h), all chosen by
// measurement on MI355X.  At nfreq 3, two columns per wave let each
// aqsntemp load serve both: 159 VGPRs (3 waves per SIMD) with 2-band groups,
// 2.8-3.1 % faster than one column with 3-band groups (4 waves); three
// columns with 1-band groups at 3 waves measured 6 % slower and four at 2
// waves 10 % slower, two with 1-band groups at 4 waves 7 % slower.

// Bands [n_lo, n_hi) of a tile's band chunk for one of 2^shift waves that
// share the tile.  An occupied band counts as kOccupiedCost others; the cuts
// between unoccupied bands fall on whole groups of BU.
template <int BU>
__device__ __forceinline__ int split_at(int k, int shift, int lo, int occ, int hi)
{
    const int cost = hi - lo + (kOccupiedCost - 1) * occ;
    const int at = (int)(((long)cost * k) >> shift);
    if (at >= cost) return hi;
    if (at < kOccupiedCost * occ) return lo + at / kOccupiedCost;
    return lo + occ + (at - kOccupiedCost * occ) / BU * BU;
}

// WAVES waves per workgroup, 2^shift of them on one tile (its bands split
// between them), one partial row per workgroup.  Long grids run 4 waves and
// shift 0; short ones the split form, 16 waves (fwd_geometry).
template <int NW, int BU, int C, int WAVES, int MIN_WAVES>
__global__ void __launch_bounds__(WAVES * kWave) __attribute__((amdgpu_waves_per_eu(MIN_WAVES)))
fwd_tiles(int nb, int nv, int ng, int np, long ntiles, int nchunk, int chunk_bands, int shift,
          const double2 *__restrict__ aqsm, const double2 *__restrict__ aqsn,
          const double2 *__restrict__ ieps, const double2 *__restrict__ wt,
          const double *__restrict__ vcoul, const double *__restrict__ wx,
          double *__restrict__ partials)
{
    constexpr int kKeep = WAVES > kFwdWaves ? 3 * C : 0;  // split form: see RowSink
    __shared__ double red[WAVES][4 * NW];
    __shared__ double kept[WAVES][kKeep > 0 ? kKeep * kWave : 1];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const long wave = (long)xcd_remap(blockIdx.x, gridDim.x) * WAVES + wid;
    const long tile = WAVES > kFwdWaves ? wave >> shift : wave;

    clear_row<4 * NW>(red[wid], lane);  // the tile may write only some of it
    if (tile < ntiles) {
        // consecutive tiles share a g-tile (and so the same aqsntemp rows)
        const int npt = (np + C - 1) / C;  // column tiles per g-tile
        int gt, pt, ck;
        tile_coords(tile, col_block<NW, C>(ng), npt, (ng + kWave - 1) / kWave, nchunk, gt, pt, ck);
        int n_lo = ck * chunk_bands;
        int n_hi = nb - n_lo < chunk_bands ? nb : n_lo + chunk_bands;
        if (WAVES > kFwdWaves) {
            const int k = (int)wave & ((1 << shift) - 1);
            const int occ = nv < n_hi ? (nv > n_lo ? nv - n_lo : 0) : n_hi - n_lo;
            const int lo = n_lo, hi = n_hi;
            // wave-uniform, and told so: the divisions run on the vector unit
            n_lo = __builtin_amdgcn_readfirstlane(split_at<BU>(k, shift, lo, occ, hi));
            n_hi = __builtin_amdgcn_readfirstlane(split_at<BU>(k + 1, shift, lo, occ, hi));
        }
        RowSink<NW, kKeep> sink{red[wid], lane, kept[wid]};
        if (n_lo < n_hi)
            fwd_tile_body<NW, BU, C>(nb, nv, n_lo, n_hi, ng, np, C * pt, gt, lane, as_global(aqsm),
                                     as_global(aqsn), as_global(ieps), as_global(wt),
                                     as_global(vcoul), as_global(wx), sink);
    }

    // the workgroup's row, the waves' rows added in a fixed order; row layout
    // [4 w + 0..3] = achtemp[w].re, .im, asxtemp[w].re, .im
    __syncthreads();
    if (threadIdx.x < 4 * NW) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) s += red[k][threadIdx.x];
        partials[(size_t)blockIdx.x * 4 * NW + threadIdx.x] = s;
    }
}

// Quasiparticle quantities from the final sums fin[4 w + 0..3] = achtemp[w]
// re, im, asxtemp[w] re, im, for nfreq odd and at least 3 (the caller
// checks): Sigma(E_w) = achtemp[w] - asxtemp[w] (asxtemp is the unsigned
// exchange sum), dSigma/dE at the middle frequency m by the central
// difference of its neighbours, Z = 1/(1 - Re dSigma/dE) and the linearised
// quasiparticle energy E + Z (Re Sigma(E) - V_xc).  out = Sigma re, im,
// dSigma/dE re, im, Z, E_qp.
template <int NW>
__device__ inline void qp_epilogue(const double *fin, const QpArgs &qp)
{
    if constexpr (NW >= 3 && NW % 2 == 1) {
        constexpr int m = (NW - 1) / 2;
        const double sr = fin[4 * m] - fin[4 * m + 2], si = fin[4 * m + 1] - fin[4 * m + 3];
        const double hi_r = fin[4 * (m + 1)] - fin[4 * (m + 1) + 2];
        const double hi_i = fin[4 * (m + 1) + 1] - fin[4 * (m + 1) + 3];
        const double lo_r = fin[4 * (m - 1)] - fin[4 * (m - 1) + 2];
        const double lo_i = fin[4 * (m - 1) + 1] - fin[4 * (m - 1) + 3];
        const double span = 2.0 * qp.step;
        const double dr = (hi_r - lo_r) / span, di = (hi_i - lo_i) / span;
        const double z = 1.0 / (1.0 - dr);
        qp.out[0] = sr;
        qp.out[1] = si;
        qp.out[2] = dr;
        qp.out[3] = di;
        qp.out[4] = z;
        qp.out[5] = qp.energy + z * (sr - qp.vxc);
    }
}

// Column sums of the partial rows: block b adds rows [b*chunk, (b+1)*chunk)
// into one row of `out`.  With FINAL, one block adds all of them and writes
// achtemp/asxtemp instead, and with qp.out set also the quasiparticle
// quantities (qp_epilogue).
template <int NW, int T, bool FINAL>
__global__ void __launch_bounds__(T)
reduce_rows(const double *__restrict__ in, long nrows, long chunk, double *__restrict__ out,
            double2 *__restrict__ ach, double2 *__restrict__ asx, QpArgs qp)
{
    constexpr int W = 4 * NW;
    __shared__ double lds[T];
    const long lo = (long)blockIdx.x * chunk;
    const long hi = lo + chunk < nrows ? lo + chunk : nrows;
    const double s = column_sums<W, T>(in, lo, hi, lds);
    if constexpr (!FINAL) {
        if (threadIdx.x < W) out[(size_t)blockIdx.x * W + threadIdx.x] = s;
        return;
    }
    __syncthreads();  // lds is read above, written below
    if (threadIdx.x < W) {
        const int w = threadIdx.x / 4, c = threadIdx.x % 4;
        double *dst = reinterpret_cast<double *>(c < 2 ? ach + w : asx + w);
        dst[c & 1] = s;
        lds[threadIdx.x] = s;
    }
    if (qp.out) {  // uniform: a kernel argument
        __syncthreads();
        if (threadIdx.x == 0) qp_epilogue<NW>(lds, qp);
    }
}

// Zero outputs of an empty sum (and its quasiparticle quantities: Sigma = 0,
// Z = 1, E_qp = E - V_xc).
template <int NW>
__global__ void fill_zero(double2 *a, double2 *b, QpArgs qp)
{
    __shared__ double fin[4 * NW];
    int i = threadIdx.x;
    if (i < NW) {
        a[i] = make_double2(0.0, 0.0);
        b[i] = make_double2(0.0, 0.0);
    }
    if (i < 4 * NW) fin[i] = 0.0;
    if (qp.out) {
        __syncthreads();
        if (i == 0) qp_epilogue<NW>(fin, qp);
    }
}

static hipError_t launch_fill_zero(int nw, double2 *a, double2 *b, const QpArgs &qp,
                                   hipStream_t st)
{
    switch (nw) {
#define GPP_Z(N)                                                                      \
    case N: hipLaunchKernelGGL(fill_zero<N>, dim3(1), dim3(64), 0, st, a, b, qp); break;
        GPP_Z(1) GPP_Z(2) GPP_Z(3) GPP_Z(4) GPP_Z(5) GPP_Z(6) GPP_Z(7) GPP_Z(8)
#undef GPP_Z
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Partial rows that one workgroup of kFinalThreads adds by itself: up to 24
// loads per thread.  More rows go through a first stage of kRedBlocks
// workgroups, whose launch costs as much as about that many loads.
static bool one_stage(int nw, long rows) { return rows * 4 * nw <= 24L * kFinalThreads; }

FwdGeometry fwd_geometry(const Dims32 &d)
{
    FwdGeometry geo{};
    if (d.nb == 0 || d.ng == 0 || d.np == 0) return geo;
    const long gtiles = (d.ng + kWave - 1) / kWave;
    const int cols = fwd_cols(d.nw);
    fwd_band_chunks(d.nb, d.nw, geo.nchunk, geo.chunk_bands);
    geo.ntiles = gtiles * ((d.np + cols - 1) / cols) * geo.nchunk;
    if (geo.ntiles >= kSplitBelow) {
        const int m = fwd_fine_chunks(geo.ntiles, geo.chunk_bands, kCUs);
        if (m > 1) {
            const int bu = fwd_bands(d.nw);
            const long tiles = geo.ntiles / geo.nchunk;
            geo.chunk_bands = ((geo.chunk_bands + m - 1) / m + bu - 1) / bu * bu;
            geo.nchunk = (d.nb + geo.chunk_bands - 1) / geo.chunk_bands;
            geo.ntiles = tiles * geo.nchunk;
        }
    }
    geo.waves = kFwdWaves;
    geo.nblocks = (geo.ntiles + kFwdWaves - 1) / kFwdWaves;
    const long long_rows = geo.nblocks;
    if (geo.ntiles < kSplitBelow) {
        // the split form: enough waves per tile to fill the GPU
        geo.waves = kSplitWaves;
        while (geo.shift < 3 && (geo.ntiles << geo.shift) < kSplitWaves * kCUs) ++geo.shift;
        geo.nblocks = ((geo.ntiles << geo.shift) + kSplitWaves - 1) / kSplitWaves;
    }
    const bool one = one_stage(d.nw, geo.nblocks);
    geo.red_blocks = one ? 0 : geo.nblocks < kRedBlocks ? geo.nblocks : kRedBlocks;
    geo.red_chunk = one ? 0 : (geo.nblocks + geo.red_blocks - 1) / geo.red_blocks;
    // sized for the long form and its first stage: 2^3 waves per tile and 16
    // per workgroup make at most twice its rows, and then no first stage.
    // Where finer band chunks may be chosen, at least for the most rows they
    // make at any size, so that a smaller call never needs more than a larger
    // one and one buffer serves every state of a program.
    const size_t row = 4 * sizeof(double) * d.nw;
    const long stage_rows = long_rows < kRedBlocks ? long_rows : kRedBlocks;
    long rows = long_rows + stage_rows;
    if (fwd_most_tiles(gtiles, d.np, d.nb) >= kSplitBelow && rows < kFineRows + kRedBlocks)
        rows = kFineRows + kRedBlocks;
    geo.workspace_bytes = (size_t)rows * row;
    return geo;
}

template <int NW>
static hipError_t launch_reduce_nw(const double *partials, long rows, long red_blocks,
                                   long red_chunk, double *stage, double2 *ach, double2 *asx,
                                   hipStream_t st, const QpArgs &qp)
{
    if (red_blocks > 0) {
        hipLaunchKernelGGL((reduce_rows<NW, kRedThreads, false>), dim3((unsigned)red_blocks),
                           dim3(kRedThreads), 0, st, partials, rows, red_chunk, stage, nullptr,
                           nullptr, QpArgs());
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        partials = stage;
        rows = red_blocks;
    }
    hipLaunchKernelGGL((reduce_rows<NW, kFinalThreads, true>), dim3(1), dim3(kFinalThreads), 0, st,
                       partials, rows, rows, nullptr, ach, asx, qp);
    return hipGetLastError();
}

template <int NW>
static hipError_t launch_fwd_nw(const Dims32 &d, const FwdGeometry &geo, const DevInputs &in,
                                double2 *ach, double2 *asx, double *ws, hipStream_t st,
                                const QpArgs &qp)
{
    double *partials = ws;
    double *stage = ws + (size_t)geo.nblocks * 4 * NW;
    const dim3 grid((unsigned)geo.nblocks), block((unsigned)(geo.waves * kWave));
    if (geo.waves == kFwdWaves)
        hipLaunchKernelGGL((fwd_tiles<NW, fwd_bands(NW), fwd_cols(NW), kFwdWaves,
                                      fwd_min_waves(NW)>),
                           grid, block, 0, st, d.nb, d.nv, d.ng, d.np, geo.ntiles, geo.nchunk,
                           geo.chunk_bands, 0, in.aqsm, in.aqsn, in.ieps, in.wt, in.vcoul, in.wx,
                           partials);
    else
        hipLaunchKernelGGL((fwd_tiles<NW, split_bands(NW), fwd_cols(NW), kSplitWaves,
                                      kSplitWaves / 4>),
                           grid, block, 0, st, d.nb, d.nv, d.ng, d.np, geo.ntiles, geo.nchunk,
                           geo.chunk_bands, geo.shift, in.aqsm, in.aqsn, in.ieps, in.wt, in.vcoul,
                           in.wx, partials);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_reduce_nw<NW>(partials, geo.nblocks, geo.red_blocks, geo.red_chunk, stage, ach,
                                asx, st, qp);
}

size_t reduce_stage_bytes(int nw, long nrows)
{
    const long blocks = nrows < kRedBlocks ? nrows : kRedBlocks;
    return (size_t)blocks * 4 * sizeof(double) * nw;
}

hipError_t launch_reduce_partials(int nw, const double *partials, long nrows, double *stage,
                                  double2 *ach, double2 *asx, hipStream_t st)
{
    if (nrows <= 0) return launch_fill_zero(nw, ach, asx, QpArgs(), st);
    const long blocks = one_stage(nw, nrows) ? 0 : nrows < kRedBlocks ? nrows : kRedBlocks;
    const long chunk = blocks ? (nrows + blocks - 1) / blocks : 0;
    switch (nw) {
    case 1: return launch_reduce_nw<1>(partials, nrows, blocks, chunk, stage, ach, asx, st, QpArgs());
    case 2: return launch_reduce_nw<2>(partials, nrows, blocks, chunk, stage, ach, asx, st, QpArgs());
    case 3: return launch_reduce_nw<3>(partials, nrows, blocks, chunk, stage, ach, asx, st, QpArgs());
    case 4: return launch_reduce_nw<4>(partials, nrows, blocks, chunk, stage, ach, asx, st, QpArgs());
    case 5: return launch_reduce_nw<5>(partials, nrows, blocks, chunk, stage, ach, asx, st, QpArgs());
    case 6: return launch_reduce_nw<6>(partials, nrows, blocks, chunk, stage, ach, asx, st, QpArgs());
    case 7: return launch_reduce_nw<7>(partials, nrows, blocks, chunk, stage, ach, asx, st, QpArgs());
    case 8: return launch_reduce_nw<8>(partials, nrows, blocks, chunk, stage, ach, asx, st, QpArgs());
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fwd(const Dims32 &d, const DevInputs &in, double2 *ach, double2 *asx,
                      void *workspace, hipStream_t st, const QpArgs &qp)
{
    const FwdGeometry geo = fwd_geometry(d);
    if (geo.nblocks == 0) return launch_fill_zero(d.nw, ach, asx, qp, st);
    double *ws = static_cast<double *>(workspace);
    switch (d.nw) {
    case 1: return launch_fwd_nw<1>(d, geo, in, ach, asx, ws, st, qp);
    case 2: return launch_fwd_nw<2>(d, geo, in, ach, asx, ws, st, qp);
    case 3: return launch_fwd_nw<3>(d, geo, in, ach, asx, ws, st, qp);
    case 4: return launch_fwd_nw<4>(d, geo, in, ach, asx, ws, st, qp);
    case 5: return launch_fwd_nw<5>(d, geo, in, ach, asx, ws, st, qp);
    case 6: return launch_fwd_nw<6>(d, geo, in, ach, asx, ws, st, qp);
    case 7: return launch_fwd_nw<7>(d, geo, in, ach, asx, ws, st, qp);
    case 8: return launch_fwd_nw<8>(d, geo, in, ach, asx, ws, st, qp);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace gpp
