// gpp_device.h -- device helpers shared by the GPP kernels (gfx950, fp64).
//
// Branch specification (Sec. III v2 three-way branch, v3 squared compares;
// the |delw| test is cross-multiplied so no divide is needed):
//   dr = x - Re om;  wi2 = (Im om)^2;  wdiffr = fma(dr, dr, wi2);
//   wtr = fma(Re om, Re om, wi2)
//   A: wdiffr > kLimitTwo && wtr < fl(kLimitOne * wdiffr)
//   B: !A && wtr > fl(kTolZero * wdiffr)
//   C: otherwise
// Every quantity in a branch decision is computed with exactly these
// roundings; only term *values* may use other (faithful) evaluations.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gpp {

constexpr double kLimitTwo = 0.25;
constexpr double kLimitOne = 250000.0;
constexpr double kTolZero = 1e-12;
// kLimitOne * kLimitTwo, exact.  For wtr below it, A <=> wdiffr > kLimitTwo:
// rounding is monotone, so wdiffr > 1/4 gives fl(kLimitOne*wdiffr) >= 62500.
constexpr double kFastWtr = 62500.0;
// Smallest (Im om)^2 for which the batch inversion may take the CH
// denominators unclamped: every |x - om|^2 >= (Im om)^2 >= 2^-60, so a
// product of up to 12 of them stays >= 2^-720, far from underflow.
constexpr double kMinUnclampedWi2 = 0x1p-60;

constexpr int kWave = 64;

struct cplx {
    double re, im;
};

// Global-memory pointer types: pointers read from memory (not kernel
// arguments) keep their address space this way, so loads through them
// compile to global or scalar loads rather than flat ones.
template <typename T>
using gptr = const __attribute__((address_space(1))) T *;

template <typename T>
__device__ __forceinline__ gptr<T> as_global(const T *p) {
    return (gptr<T>)p;
}

// A running wave-uniform address (scalar registers) of read-only data.  Its
// loads are scalar loads whatever else the kernel writes (constant address
// space); the empty asm in advance() keeps the compiler from folding the
// running addresses of a loop back into one index, whose products and sums
// per load then stand in front of every load.
struct Walker {
    uint64_t at;
    __device__ __forceinline__ void start(uint64_t a) {
        at = (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32 |
             (unsigned)__builtin_amdgcn_readfirstlane((int)a);
    }
    __device__ __forceinline__ void advance(long bytes) {
        at += bytes;
        asm("" : "+s"(at));
    }
    // the real value `i` doubles further on
    __device__ __forceinline__ double real(int i) const {
        return ((const __attribute__((address_space(4))) double *)at)[i];
    }
    // the complex value `bytes` further on
    __device__ __forceinline__ cplx complex(uint32_t bytes) const {
        typedef double pair __attribute__((ext_vector_type(2)));
        const pair v = *(const __attribute__((address_space(4))) pair *)(at + bytes);
        return {v.x, v.y};
    }
};

__device__ __forceinline__ cplx cmake(double re, double im) { return {re, im}; }
__device__ __forceinline__ cplx cload(const double2 *p) {
    double2 v = *p;
    return {v.x, v.y};
}
// The same wave-uniform integer, opaque to the optimiser: loads indexed by
// it cannot be hoisted out of the loop that calls this.  Used where
// wave-uniform values would otherwise be hoisted into more scalar registers
// than exist (and spilled into vector lanes); reloading them each iteration
// goes through the scalar cache instead.  The base pointer stays visible,
// so the loads remain scalar loads.
__device__ __forceinline__ int opaque_uniform(int v) {
    asm volatile("" : "+s"(v));
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ cplx cload(gptr<double2> p) {
    return {p->x, p->y};  // member reads: one 16-byte load after vectorising
}
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
    return {fma(a.re, b.re, -a.im * b.im), fma(a.re, b.im, a.im * b.re)};
}
// a * conj(b)
__device__ __forceinline__ cplx cmul_conj(cplx a, cplx b) {
    return {fma(a.re, b.re, a.im * b.im), fma(a.im, b.re, -a.re * b.im)};
}
__device__ __forceinline__ cplx cscale(double s, cplx a) { return {s * a.re, s * a.im}; }
// acc += a * b
__device__ __forceinline__ void cmac(cplx &acc, cplx a, cplx b) {
    acc.re = fma(a.re, b.re, fma(-a.im, b.im, acc.re));
    acc.im = fma(a.re, b.im, fma(a.im, b.re, acc.im));
}

// 1/d for normal d: the hardware estimate refined by two Newton-Raphson
// steps r <- r + r (1 - d r).  Each step squares the relative error; two
// steps from the estimate end within about one ulp.  Not for 0, inf,
// denormal inputs (callers only use it where d > 1/4).
__device__ __forceinline__ double rcp_nr2(double d) {
    double r = __builtin_amdgcn_rcp(d);
    double e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    return r;
}

// Newton steps after the hardware estimate for the batch product.  The
// estimate is good to 2^-24.4; one step leaves a relative error below
// 2.2e-15 (2^-48.7, measured over normal inputs with exponents -720..1000, the
// range of a product of 12 denominators of at least 2^-60 or of 6 pairs of
// them), which is shared by the K reciprocals
// of the batch.  That is far inside the 1e-12 bar on every output, and saves
// two fused multiply-adds per batch.
#ifndef GPP_BATCH_NEWTON
#define GPP_BATCH_NEWTON 1
#endif
// 1/d for normal d with GPP_BATCH_NEWTON Newton-Raphson steps from the
// hardware estimate.
__device__ __forceinline__ double rcp_batch(double d) {
    double r = __builtin_amdgcn_rcp(d);
#pragma unroll
    for (int i = 0; i < GPP_BATCH_NEWTON; ++i) {
        const double e = fma(-d, r, 1.0);
        r = fma(r, e, r);
    }
    return r;
}

// Batch inversion: r[k] = 1/d[k] for K positive values from one reciprocal
// of their product.  The values go in two halves, each with its own prefix
// products c[k]; with R = 1 / (product of all), R times the other half's
// product is the reciprocal of a half's product, and walking a half back,
// r[k] = R c[k-1] and R <- R d[k].  Two halves cost the same 3(K-1)
// multiplies as one run over all K, with half the serial chain.  Each r[k]
// carries the error of R plus at most 2K roundings.  The batch path needs
// every d[k] >= 2^-60, or 2^-120 with at most 6 of them (so that no product
// leaves the normal range at the bottom; callers keep lanes without that bound
// out of it, or pass batch_ok = false) and a total product below 2^1000 (an
// overflowed prefix stays infinite, so this also covers the prefixes).
// batch_prefix forms the prefix products and returns the total, batch_back the
// r[k]; where a lane of the wave fails one of the bounds (batch_misses, one
// scalar test), every lane inverts one by one instead (one_by_one); a zero there
// gives an infinite or NaN reciprocal, which callers mask.
template <int K>
__device__ __forceinline__ double batch_prefix(const double (&d)[K], double (&c)[K]) {
    static_assert(K <= 12, "the 2^-60 lane bound keeps products of at most 12 factors normal");
    constexpr int H = (K + 1) / 2;  // the first half's length
    c[0] = d[0];
    if constexpr (K > 1) c[H] = d[H];
#pragma unroll
    for (int k = 1; k < H; ++k) {  // one step of each half
        c[k] = c[k - 1] * d[k];
        if (H + k < K) c[H + k] = c[H + k - 1] * d[H + k];
    }
    return K > 1 ? c[H - 1] * c[K - 1] : c[0];
}
template <int K>
__device__ __forceinline__ void batch_back(const double (&d)[K], const double (&c)[K], double all,
                                           double (&r)[K]) {
    constexpr int H = (K + 1) / 2;
    const double R = rcp_batch(all);
    double ra = K > 1 ? R * c[K - 1] : R, rb = R * c[H - 1];
#pragma unroll
    for (int k = H - 1; k > 0; --k) {
        if (H + k < K) {
            r[H + k] = rb * c[H + k - 1];
            rb = rb * d[H + k];
        }
        r[k] = ra * c[k - 1];
        ra = ra * d[k];
    }
    r[0] = ra;
    if constexpr (K > 1) r[H] = rb;
}
// The lanes whose batch of product `all` may not be used; narrow = the lanes
// (as a wave mask) with a denominator that may be below 2^-60.
__device__ __forceinline__ uint64_t batch_misses(double all, uint64_t narrow) {
    return __builtin_amdgcn_ballot_w64(!(all < 0x1p1000)) | narrow;
}
template <int K>
__device__ __forceinline__ void one_by_one(const double (&d)[K], double (&r)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) r[k] = rcp_nr2(d[k]);
}
// One Newton step on each reciprocal: of the batch's error, up to 2e-15, one
// rounding is left.
template <int K>
__device__ __forceinline__ void refine(const double (&d)[K], double (&r)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) r[k] = fma(fma(-d[k], r[k], 1.0), r[k], r[k]);
}
// The same one after the other, with one register pair for all of them.
template <int K>
__device__ __forceinline__ void refine_in_turn(const double (&d)[K], double (&r)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double e;
        asm("v_fma_f64 %[e], -%[d], %[r], 1.0\n\t"
            "v_fma_f64 %[r], %[e], %[r], %[r]"
            : [e] "=&v"(e), [r] "+v"(r[k])
            : [d] "v"(d[k]));
    }
}
template <int K>
__device__ __forceinline__ void batch_reciprocal(const double (&d)[K], double (&r)[K],
                                                 bool batch_ok = true) {
    double c[K];
    const double all = batch_prefix<K>(d, c);
    batch_back<K>(d, c, all, r);
    if (__builtin_expect(batch_misses(all, __builtin_amdgcn_ballot_w64(!batch_ok)) != 0, 0))
        one_by_one<K>(d, r);
}

// keep ? v : (a value of magnitude below 2^-1042) with one 32-bit select:
// only the high word (sign, exponent, top mantissa bits) is cleared, which
// leaves a denormal made of v's low word.  Added to any accumulator above
// 2^-990 in magnitude it changes nothing, so sums are the same as with an
// exact zero unless the whole sum is below ~2^-1000.
__device__ __forceinline__ double mask_keep(bool keep, double v) {
    const int lo = __double2loint(v);
    const int hi = keep ? __double2hiint(v) : 0;
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double next_up(double t) {
    return __longlong_as_double(__double_as_longlong(t) + 1);  // t > 0
}
__device__ __forceinline__ double next_down(double t) {
    return __longlong_as_double(__double_as_longlong(t) - 1);  // t > 0
}

// Per-(p,g) threshold thr with  A <=> wdiffr > thr,  bit-exact with the
// specification for every wdiffr >= 0.  fl(kLimitOne * d) is monotone in
// d, so {d : wtr < fl(kLimitOne * d)} = {d >= T}; A is then
// d > kLimitTwo && d >= T, i.e. d > max(kLimitTwo, pred(T)).
__device__ inline double threshold_search(double wtr) {
#pragma clang fp contract(off)
    if (wtr < kFastWtr) return kLimitTwo;
    if (!(wtr <= 1.0e300)) return __builtin_inf();  // NaN/huge: never A
    double t = wtr * 4.0e-6;                          // ~ wtr / kLimitOne
    for (int i = 0; i < 64 && !(kLimitOne * t > wtr); ++i) t = next_up(t);
    for (int i = 0; i < 64 && (kLimitOne * next_down(t) > wtr); ++i) t = next_down(t);
    double p = next_down(t);
    return p > kLimitTwo ? p : kLimitTwo;
}
// The search only where a lane of the wave needs it (one scalar branch).
__device__ __forceinline__ double branch_a_threshold(double wtr) {
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(wtr < kFastWtr)) != 0, 0))
        return threshold_search(wtr);
    return kLimitTwo;
}

__device__ inline bool branch_b_holds(double wtr, double wdiffr) {
#pragma clang fp contract(off)
    return wtr > kTolZero * wdiffr;
}

// Lane exchange inside a row of 16 lanes (DPP), both halves of a double.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    // every source lane of the controls used here exists, so no lane keeps
    // an old value (bound_ctrl only matters for lanes outside the row)
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Sum over each aligned group of 8 lanes; every lane of the group gets it.
__device__ __forceinline__ double octet_sum(double v)
{
    v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]: lane ^ 1
    v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]: lane ^ 2
    v += dpp_f64<0x141>(v);  // row_half_mirror: lane i <-> 7 - i within 8
    return v;
}
// Sum over each row of 16 lanes; every lane of the row gets it.
__device__ __forceinline__ double row_sum(double v)
{
    v = octet_sum(v);
    return v + dpp_f64<0x140>(v);  // row_mirror: lane i <-> 15 - i within 16
}

// a + b after a's upper 32 lanes and b's lower 32 have changed places: lanes
// 0-31 get the two halves of a added up, lanes 32-63 those of b.
__device__ __forceinline__ double add_halves(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// The same between a's odd rows of 16 lanes and b's even ones: rows 0 and 2
// get a's rows 0 + 1 and 2 + 3, rows 1 and 3 those of b.
__device__ __forceinline__ double add_rows(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// Wave total of v in every lane.
__device__ __forceinline__ double wave_sum(double v) {
    v = add_halves(v, v);
    return row_sum(add_rows(v, v));
}

// Wave totals of M values (M even): calls put(i, total of v[i]) for each, on
// one lane each.  The first two steps fold two values into one register
// instead of exchanging each value with itself (permlane swaps), so that
// only M/4 registers go through the row sums: 63 vector instructions for 12
// values, against 18 per value one at a time, or 6 LDS round trips each with
// __shfl_xor.  Row q of register j ends up with value 4 j + {0, 2, 1, 3}[q].
template <int M, typename F>
__device__ __forceinline__ void wave_totals(const double (&v)[M], int lane, F put) {
    static_assert(M % 2 == 0, "values go in pairs");
    constexpr int H = M / 2, R = (H + 1) / 2;
    double h[H];
#pragma unroll
    for (int k = 0; k < H; ++k) h[k] = add_halves(v[2 * k], v[2 * k + 1]);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const double t = row_sum(add_rows(h[2 * j], h[2 * j + 1 < H ? 2 * j + 1 : 2 * j]));
        const int q = lane / 16;
        const int i = 4 * j + (q == 1 ? 2 : q == 2 ? 1 : q);
        if (lane % 16 == 0 && i < M) put(i, t);
    }
}

// Order this wave's LDS writes before its later LDS reads (and the reverse)
// when lanes exchange data through LDS without a workgroup barrier.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Zeroes a wave's row of W <= 64 values in LDS; any lane may write them next.
template <int W>
__device__ __forceinline__ void clear_row(double *row, int lane)
{
    if (lane < W) row[lane] = 0.0;
    wave_lds_sync();
}

// A wave-uniform value moved into scalar registers (the value of lane 0).
__device__ __forceinline__ double to_uniform(double t) {
    const int lo = __builtin_amdgcn_readfirstlane(__double2loint(t));
    const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(t));
    return __hiloint2double(hi, lo);
}

// Element at byte offset `off` of a complex row of `len` elements whose
// base is wave-uniform: a raw buffer load with the row in a scalar buffer
// descriptor (gfx9 descriptor word 3 = 0x00020000) and the offset in a
// vector register.  Offsets at or beyond the row length read as zero.
__device__ __forceinline__ cplx load_row_elem(gptr<double2> row, int len, uint32_t off) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(const double2 *)row, (short)0, len * (int)sizeof(double2), 0x00020000);
    const double2 v = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    return {v.x, v.y};
}

// The same for the row `row_off` bytes further on (a scalar register) than
// the 64-bit row address `at`.  The callers' offsets are those of existing
// elements, so the descriptor sets no bound.
__device__ __forceinline__ cplx load_elem_at(uint64_t at, uint32_t row_off, uint32_t off) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)at, (short)0, -1,
                                                                        0x00020000);
    const double2 v = __builtin_bit_cast(
        double2, __builtin_amdgcn_raw_buffer_load_b128(rs, off, row_off, 0));
    return {v.x, v.y};
}

// Map a hardware workgroup id to a logical one so that each of the 8 XCDs
// (which receive workgroups round-robin) walks a contiguous logical range
// and its private L2 sees neighbouring tiles.  A bijection on [0, n).
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t n) {
    const uint32_t kXcd = 8;
    uint32_t x = b % kXcd, i = b / kXcd, per = n / kXcd, rem = n % kXcd;
    return x * per + (x < rem ? x : rem) + i;
}

// Column sums of the rows [lo, hi) of W doubles by a workgroup of T threads,
// in a fixed order: thread t adds column t % W of every (T / W)-th row, eight
// loads in flight, then the T / W row lanes are added through LDS (T doubles)
// in two steps.  Thread t < W returns column t's sum.
template <int W, int T>
__device__ __forceinline__ double column_sums(const double *__restrict__ rows, long lo, long hi,
                                              double *lds)
{
    constexpr int R = T / W, G = R < 8 ? R : 8;
    static_assert(R >= 1, "a row lane per column at least");
    const int t = threadIdx.x;
    double s = 0.0;
    if (t < R * W) {
        constexpr long step = R * W;
        const long end = hi * W;
        long i = lo * W + t;
        double a[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = 0.0;
        for (; i + 7 * step < end; i += 8 * step) {
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] += rows[i + k * step];
        }
#pragma unroll
        for (int k = 0; k < 7; ++k)
            if (i + k * step < end) a[k] += rows[i + k * step];
        s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
        lds[t] = s;
    }
    __syncthreads();
    if (t < G * W) {
        s = lds[t];
        for (int k = t + G * W; k < R * W; k += G * W) s += lds[k];
    }
    __syncthreads();
    if (t < G * W) lds[t] = s;
    __syncthreads();
    if (t < W) {
#pragma unroll
        for (int k = 1; k < G; ++k) s += lds[t + k * W];
    }
    return s;
}

}  // namespace gpp
