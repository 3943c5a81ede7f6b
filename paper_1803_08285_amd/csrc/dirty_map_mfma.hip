// Dirty map on the matrix cores (float32 path, antipodal seeds).
//
// Same definition as dirty_map.hip,
//   X(k,p) = sum_t w(t,k) gamma(t,p) Re[C(t,k) e^{2 pi i f_k tau(t,p)}],
// evaluated per 64-bin strip (absolute bins k_s .. k_s + 63) as a dense
// contraction.  With the strip centre f_c = f0 + (k_s + 31.5) df, the bin
// offsets s_j = (j - 31.5) / 31.5 in [-1, 1] and eta = 2 pi 31.5 df tau,
//   e^{2 pi i f_j tau} = e^{2 pi i f_c tau} e^{i s_j eta}
//                      = e^{2 pi i f_c tau} sum_m eps_m i^m J_m(eta) T_m(s_j)
// (Jacobi-Anger expansion; J_m Bessel functions, T_m Chebyshev polynomials,
// eps_0 = 1, eps_m = 2).  Truncated after M = 5 terms the error is below
// 2 (eta/2)^5 / 5! <= 1e-6 for |eta| <= 0.29, i.e. df <= 1/32 Hz with any
// baseline on the Earth (|tau| <= 2 R / c); larger df use the recurrence kernel.
// So for bin j of the strip and the antipodal pair (p, p'),
//   X(j,p) = P_r - P_i,  X(j,p') = P_r + P_i,
//   P_r(j,p) = sum_{m,t} [T_m(s_j) y_re(t,j)] Re U_m(t,p),
//   P_i(j,p) = sum_{m,t} [T_m(s_j) y_im(t,j)] Im U_m(t,p),
//   U_m = gamma e^{2 pi i f_c tau} eps_m i^m J_m(eta)      (U_m(p') = conj U_m(p)),
// two real GEMMs with K = (m, t).  The prep measures max |tau| of the seeds on
// the device and the kernel picks the cheapest form the bound allows, per
// launch: where |eta| <= 0.07 (baselines up to ~3400 km at df = 1/32 Hz) four
// terms suffice (the dropped remainder is below 2 (eta/2)^4 / 4! <= 1.3e-7) and
// m = 2 needs no split (|2 J_2| <= 1.2e-3); where |eta| <= 0.17 five terms with
// m = 2 unsplit (|2 J_2| <= 7.3e-3, single roundings below 3.6e-6 of the
// scale).  Operands are float16 on
// v_mfma_f32_32x32x16_f16 with float32 accumulation; the leading terms
// m = 0, 1, 2 are split hi + lo (x = hi + lo + O(2^-21 x)) and take three
// products each (hi.hi + hi.lo + lo.hi), m = 3, 4 one product.  Power-of-two
// scales keep every operand, lo halves included, in the float16 normal range
// (the matrix cores flush float16 subnormals): 2^e_j per bin on the data side
// (its largest |y| lands in [2^13, 2^14)), 2^12 on the pixel side, and 2^g_m
// per term.
//
// Data-side operands A (per strip, 16-segment chunk, component, part, 32-bin
// block, lane: the operand layout of the instruction) are prepared once per
// call, and with them the Bessel amplitudes, which depend on the seed alone,
// once per (segment, pixel pair).  The pixel-side operands
// B are generated by each wave for its 32 pixel pairs and 16 segments (one
// lane = one pixel x 8 segments) from those amplitudes and the strip's
// phasor, term by term, so the matrix cores work on term m while the vector
// units build term m + 1.  The workgroup copies the strip's next A chunk from
// global memory straight into LDS while it contracts the current one.  The
// maps and the A fragments are written with streaming (nontemporal) stores.
// On request the epilogue also writes the float64 sum of each strip's band
// columns per pixel (the broadband map without reading X back); with no X
// (a broadband-only call) those sums are all it writes.
#include "seed_rows.h"
#include "sgwb_internal.h"

namespace sgwb {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kXmS = 64;       // bins per strip
constexpr int kXmParts = 8;    // m0h m0l m1h m1l m2h m3 m4 m2l: a four-term form needs the first six
constexpr int kXmWaves = 4;    // waves per workgroup
constexpr int kXmPairs = 32 * kXmWaves;  // pixel pairs per workgroup
constexpr int kXmFrags = 2 * kXmParts * 2;  // component x part x bin block
// place of term m's part in that order
__host__ __device__ constexpr int xm_part(int m, bool lo) { return m < 2 ? 2 * m + lo : m == 2 ? (lo ? 7 : 4) : m + 2; }
// per-term scale exponents 2^g_m (B side) and 2^-g_m (A side)
__host__ __device__ constexpr int xm_g(int m) { return m == 0 ? 0 : m == 1 ? 2 : m == 2 ? 5 : m == 3 ? 9 : 14; }
constexpr int kXmBShift = 12;  // common scale 2^12 of the pixel-side operands

// The float32 value itself, hidden from the optimiser: a float16 split must
// take hi and lo from one rounded float32 value, and the backend otherwise
// folds "(half)(a * b)" into one fused multiply-convert that rounds the exact
// product, which differs from the rounded product at float16 ties.
__device__ __forceinline__ float rounded(float x)
{
    asm volatile("" : "+v"(x));
    return x;
}


// Fixed-point reduction of the phase (xm_phase).
constexpr double kXmTurns = 1.5 * 1048576.0;  // 1.5 2^20: last place 2^-32
constexpr double kXmMaxTurns = 524288.0;      // 2^19

// Host check that a matrix-core form can apply: |eta| <= kXmEtaMax (where
// 2 (eta/2)^5 / 120 <= 1e-6) for every delay of a baseline on the Earth
// (|tau| <= 2 R / c, i.e. df <= 0.0344 Hz); tile indices in 32 bits.
bool xm_eligible(const MapArgs &a)
{
    const double eta_max = kTwoPi * 31.5 * a.df * 2.0 * kEarthRadius / kLightSpeed;
    if (a.nside <= 0 || !(eta_max <= kXmEtaMax)) return false;
    const int64_t nstrips = (a.k0 + a.nf - 1) / kXmS - a.k0 / kXmS + 1;
    const int64_t npblocks = (a.npix / 2 + kXmPairs - 1) / kXmPairs;
    return nstrips * npblocks <= 0x7fffffff;
}

// Real data whose delays are tiny (the overlap terms of a day's consecutive
// segments: differences of a few 1e-4 s) take strips of twice the width, the
// second 64 bins in the place of the second component: the pixel-side operands,
// most of the vector work, then serve 128 bins.  Three terms are enough where
// |eta| <= 0.01 over those (the dropped 2 J_3 is below 4.2e-8, the single
// rounding of 2 J_2 <= 2.5e-5 below 1.3e-8).  Measured, the overlap diagonal of
// 4101 bins at nside 32 (the whole call): 875 us, with 64-bin strips 1022 us.
constexpr double kXmEtaWide = 0.01;
constexpr double kXmWideScale = 63.5 / 31.5;  // eta of 128 bins over eta of 64
constexpr int kXmWideS = 2 * kXmS;

constexpr int kTmaxParts = 2048;  // partial maxima of |tau|
// Form record of a call (float64 words): [0] largest |tau|, [1] form code,
// then the partial maxima and the spot check's per-workgroup flags.
constexpr int kXmRecWords = 2 + kTmaxParts + kSymParts;

static size_t up256_(size_t n) { return (n + 255) / 256 * 256; }

size_t xm_workspace_bytes(int64_t k0, int32_t nt, int32_t nf, int32_t npix)
{
    const int64_t nstrips = (k0 + nf - 1) / kXmS - k0 / kXmS + 1;
    const int64_t nchunks = (nt + kXmT - 1) / kXmT;
    const size_t frags = (size_t)nstrips * nchunks * kXmFrags * 64 * sizeof(uint4);
    const size_t scales = (size_t)nstrips * kXmS * sizeof(int);
    const size_t tmax = kXmRecWords * sizeof(double);
    const size_t items = (size_t)nt * (npix / 2);
    return up256_(frags) + up256_(scales) + up256_(tmax) + up256_(items * sizeof(float4)) + up256_(items * sizeof(float));
}

constexpr int kXmPrepThreads = 1024;

// Largest |tau| of a block's share of the seeds (block b of n), without atomics;
// xm_tmax_final_kernel takes the largest of the blocks' (a maximum is exact in
// any order).
__device__ __forceinline__ void xm_tmax_block(const double *__restrict__ tau, int64_t n, int64_t b, int64_t nb,
                                              double *__restrict__ part, double *red)
{
    // four independent maxima per thread, so that their loads go out together
    double m[4] = {0.0, 0.0, 0.0, 0.0};
    const int64_t stride = nb * kXmPrepThreads;
    int64_t i = b * kXmPrepThreads + threadIdx.x;
    for (; i + 3 * stride < n; i += 4 * stride) {
#pragma unroll
        for (int u = 0; u < 4; ++u) m[u] = fmax(m[u], fabs(tau[i + u * stride]));
    }
    for (; i < n; i += stride) m[0] = fmax(m[0], fabs(tau[i]));
    red[threadIdx.x] = fmax(fmax(m[0], m[1]), fmax(m[2], m[3]));
    __syncthreads();
    for (int st = kXmPrepThreads / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + st]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[b] = red[0];
}

constexpr int kSymThreads = 1024;

// Spot check of the antipodal symmetry that the pairing relies on: for the
// first, middle and last segment and every northern pixel p,
// gamma(t, a(p)) == gamma(t, p) and tau(t, a(p)) == -tau(t, p) exactly (the
// geometry kernel writes them so; a NaN fails too).  One flag per workgroup.
__global__ __launch_bounds__(kSymThreads) void xm_symcheck_kernel(const float *__restrict__ gamma,
                                                          const double *__restrict__ tau, int32_t nt, int64_t npix,
                                                          int64_t nside, double *__restrict__ flags)
{
    const int bad = __syncthreads_or(antipodal_mismatch(gamma, tau, nt, npix, nside, blockIdx.x, kSymParts));
    if (threadIdx.x == 0) flags[blockIdx.x] = bad ? 1.0 : 0.0;
}

hipError_t launch_antipodal_check(const float *gamma, const double *tau, int32_t nt, int64_t npix, int64_t nside,
                                  double *flags, hipStream_t s)
{
    hipLaunchKernelGGL(xm_symcheck_kernel, dim3(kSymParts), dim3(kSymThreads), 0, s, gamma, tau, nt, npix, nside, flags);
    return hipGetLastError();
}

// The call's form, chosen once on the device: the largest |tau| of the seeds
// (from the partial maxima) against the expansion bounds, or rejected when the
// spot check failed or a delay exceeds the call's bound.  rec[0] = max |tau|,
// rec[1] = SGWB_XFORM_* code (SGWB_XFORM_VALU: no matrix-core form is accurate
// enough, a gated vector-unit launch computes the map).
__global__ __launch_bounds__(256) void xm_tmax_final_kernel(const double *__restrict__ part, int nparts,
                                                            const double *__restrict__ flags, double eta_scale,
                                                            double tau_limit, int32_t unit_c,
                                                            double *__restrict__ rec)
{
    __shared__ double red[256];
    double m = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 256) m = fmax(m, part[i]);
    red[threadIdx.x] = m;
    const int bad = __syncthreads_or((int)threadIdx.x < kSymParts && flags[threadIdx.x] != 0.0);
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + st]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double tm = red[0], eta = eta_scale * tm;
        int form;
        if (bad || !(tm <= tau_limit * (1.0 + 1e-9))) form = kXFormRejected;
        else if (unit_c && eta * kXmWideScale <= kXmEtaWide) form = kXFormWide;
        else if (eta <= kXmEtaFour) form = SGWB_XFORM_MFMA4;
        else if (eta <= kXmEtaM2) form = SGWB_XFORM_MFMA5;
        else if (eta <= kXmEtaMax) form = SGWB_XFORM_MFMA5S;
        else form = SGWB_XFORM_VALU;
        rec[0] = tm;
        rec[1] = (double)form;
    }
}

// Per-bin scale exponent: max_t |y| * 2^e in [2^13, 2^14).  One workgroup per
// strip: lane l takes bin l of the strip, wave w the segments w, w + 16, ...;
// the waves' maxima meet in LDS (a maximum is exact in any order).
constexpr int kXmScaleWaves = 16;

__device__ __forceinline__ void xm_scale_strip(const XmArgs &x, int64_t strip, const float2 *__restrict__ C,
                                               const float *__restrict__ w, int *__restrict__ e_out,
                                               float (*red)[64])
{
    static_assert(kXmS == 64, "one lane per bin of the strip");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t i = strip * kXmS + lane;  // strip-local bin index over all strips
    const int64_t c = (x.strip_first * kXmS + i) - x.a.k0;  // column in C
    float mx = 0.0f;
    if (c >= 0 && c < x.a.nf) {
        // Eight segments a pass, so that their loads go out together: with one,
        // the few workgroups of a sub-band wait out 56 memory latencies in a row.
        // (Rows past the last read it again.)
        constexpr int kBatch = 8;
        for (int t0 = wv; t0 < x.a.nt; t0 += kXmScaleWaves * kBatch) {
            float2 cv[kBatch];
            float wt[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int64_t off = (int64_t)min(t0 + u * kXmScaleWaves, x.a.nt - 1) * x.a.ldc + c;
                cv[u] = x.a.unit_c ? make_float2(1.0f, 0.0f) : C[off];
                wt[u] = w[off];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                mx = fmaxf(mx, fmaxf(fabsf(wt[u] * cv[u].x), fabsf(wt[u] * cv[u].y)));
        }
    }
    red[wv][lane] = mx;
    __syncthreads();
    if (wv != 0) return;
#pragma unroll
    for (int k = 1; k < kXmScaleWaves; ++k) mx = fmaxf(mx, red[k][lane]);
    int e = 0;
    if (mx > 0.0f) {
        int ex;
        frexpf(mx, &ex);  // mx in [2^(ex-1), 2^ex)
        e = 14 - ex;
    }
    e_out[i] = e;
}

// First preparation launch of a call, kXmPrepThreads a workgroup: the strips'
// scales, the antipodal spot check and the largest |tau|, none of which needs
// another; a call with prepared seeds, or seeds alone, has only its part.  (As
// launches of their own they took 20, 5 and 7 us of a 6272-bin sub-band's call at
// nside 16, none of which fills the chip.)
__global__ __launch_bounds__(kXmPrepThreads) void xm_prep_kernel(XmArgs x, const float2 *__restrict__ C,
                                                                 const float *__restrict__ w, int *__restrict__ e_out,
                                                                 const float *__restrict__ gamma,
                                                                 const double *__restrict__ tau,
                                                                 double *__restrict__ flags, double *__restrict__ part,
                                                                 int64_t nscale, int64_t nsym, int64_t ntmax)
{
    static_assert(64 * kXmScaleWaves == kXmPrepThreads, "one workgroup a strip");
    __shared__ double red[kXmPrepThreads];
    int64_t b = blockIdx.x;
    if (b < nscale) {
        xm_scale_strip(x, b, C, w, e_out, reinterpret_cast<float(*)[64]>(red));
    } else if ((b -= nscale) < nsym) {
        const int bad = __syncthreads_or(antipodal_mismatch(gamma, tau, x.a.nt, x.a.npix, x.a.nside, b, kSymParts));
        if (threadIdx.x == 0) flags[b] = bad ? 1.0 : 0.0;
    } else {
        xm_tmax_block(tau, (int64_t)x.a.nt * x.a.npix, b - nsym, ntmax, part, red);
    }
}

__device__ __forceinline__ float cheb(int m, float s)
{
    const float s2 = s * s;
    switch (m) {
    case 0: return 1.0f;
    case 1: return s;
    case 2: return 2.0f * s2 - 1.0f;
    case 3: return s * (4.0f * s2 - 3.0f);
    default: return fmaf(8.0f * s2, s2 - 1.0f, 1.0f);
    }
}

// 128-bin strips of the call (real data).
__device__ __forceinline__ int64_t xm_wide_strips(const XmArgs &x)
{
    return (x.a.k0 + x.a.nf - 1) / kXmWideS - x.a.k0 / kXmWideS + 1;
}

// A fragments: [strip][chunk][comp][part][jb][lane] of uint4 (8 x f16, k = 8 (lane/32) + e),
// the parts that the call's form reads (none, if it is not a matrix-core form).
// Bound by what it writes: 48 of the 64 bytes per segment, bin and component
// in the four-term form.
__device__ __forceinline__ void xm_afrag(const XmArgs &x, int64_t block, const float2 *__restrict__ C,
                                         const float *__restrict__ w, const int *__restrict__ e_in,
                                         const double *__restrict__ rec, uint4 *__restrict__ A)
{
#pragma clang fp contract(off)  // hi and lo from the same rounded float32 value
    const int form = (int)rec[1];
    const bool wide = form == kXFormWide;
    if (!wide && form != SGWB_XFORM_MFMA4 && form != SGWB_XFORM_MFMA5 && form != SGWB_XFORM_MFMA5S) return;
    const int64_t gid = block * 256 + threadIdx.x;
    const int64_t total = (wide ? xm_wide_strips(x) : x.nstrips) * x.nchunks * 4 * 64;
    if (gid >= total) return;
    const int lane = (int)(gid & 63);
    const int cj = (int)((gid >> 6) & 3);  // comp * 2 + jb
    const int64_t sc = gid >> 8;           // strip * nchunks + chunk
    const int64_t strip = sc / x.nchunks, chunk = sc % x.nchunks;
    const int comp = cj >> 1, jb = cj & 1;
    if (!wide && comp && x.a.unit_c) return;  // real data: the second component is never read
    const int j = (wide ? comp * kXmS : 0) + jb * 32 + (lane & 31);
    const int64_t c = wide ? (x.a.k0 / kXmWideS + strip) * kXmWideS + j - x.a.k0
                           : (x.strip_first + strip) * kXmS + j - x.a.k0;
    const bool inside = c >= 0 && c < x.a.nf;
    const int half = lane >> 5, t0 = (int)chunk_row(x.a.nt, chunk) + half * half_row(x.a.nt);
    const float scale = inside ? ldexpf(1.0f, e_in[c + x.a.k0 - x.strip_first * kXmS]) : 0.0f;
    const float s = wide ? ((float)j - 63.5f) * (1.0f / 63.5f) : ((float)j - 31.5f) * (1.0f / 31.5f);
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int t = t0 + e;
        float v = 0.0f;
        if (inside && slot_is_new(x.a.nt, chunk, half, e)) {
            const int64_t off = (int64_t)t * x.a.ldc + c;
            const float2 cv = x.a.unit_c ? make_float2(1.0f, 0.0f) : C[off];
            v = w[off] * (comp && !wide ? cv.y : cv.x) * scale;
        }
        y[e] = v;
    }
    // streaming stores: 1.2-1.6 GB at the full band, read back only by the main kernel
    u32x4 *out = reinterpret_cast<u32x4 *>(A) + (sc * kXmFrags + comp * kXmParts * 2 + jb) * 64 + lane;
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        if ((m == 4 && form == SGWB_XFORM_MFMA4) || (m == 3 && wide)) break;
        const float tm = cheb(m, s) * ldexpf(1.0f, -xm_g(m));
        h8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = rounded(y[e] * tm);
            hi[e] = (_Float16)v;
            lo[e] = (_Float16)(v - (float)hi[e]);
        }
        __builtin_nontemporal_store(__builtin_bit_cast(u32x4, hi), out + 2 * xm_part(m, false) * 64);
        if (m < 2 || (m == 2 && form == SGWB_XFORM_MFMA5S))
            __builtin_nontemporal_store(__builtin_bit_cast(u32x4, lo), out + 2 * xm_part(m, true) * 64);
    }
}

// Per-item values shared by all terms: the strip-centre phasor e^{2 pi i f_c tau}
// = c + i s and the signed amplitudes a_m = gamma eps_m J_m(eta) 2^(g_m + kXmBShift)
// (a_2 stored negated, so that term 2 needs no sign of its own).
struct XmItem {
    float c, s;
    float a[5];
};

// The phase x = f_c tau (in turns, ~70 at most on the Earth at 1.7 kHz) is reduced in
// one float64 operation: x + 1.5 2^20, rounded to that value's last place of
// 2^-32 turns (7e-10 rad at most), has x's fraction in its low 32 bits, as a signed
// integer u in units of 2^-32 turns (for |x| < 2^19; calls whose frequencies go
// beyond that are XmArgs::ext and pass the fraction of x).
// e^{2 pi i u} then comes from the half angle h = pi u 2^-32,
// |h| <= pi/2, as cos 2h = 1 - 2 sin^2 h, sin 2h = 2 sin h cos h, with
// near-minimax polynomials for sin h (odd, degree 9) and cos h (even, degree
// 10), fitted on |h| <= pi/2 by reweighted least squares on Chebyshev nodes
// (largest error 7e-9 and 2e-10 before float32 rounding); no quadrant
// selects.  (The float64 product, its rint, the difference and the conversion
// from float64 that this takes the place of were four instructions of 18, each
// as dear as two of the others.)
// eps_m J_m(eta) 2^(g_m + kXmBShift) are Horner series in
// eta^2 (|eta| <= 0.3; the dropped terms are below 2e-8 of J_0 ~ 1).  The common factor
// 2^kXmBShift keeps the float16 lo halves of the pixel-side operands in the
// normal range (the matrix cores flush float16 subnormals).
__device__ __forceinline__ void xm_phase(double ta, double fc, XmItem &it)
{
    const int32_t u = (int32_t)(uint32_t)__double_as_longlong(fma(fc, ta, kXmTurns));
    const float h = (float)u * (3.14159265358979324f / 4294967296.0f), h2 = h * h;
    const float sh =
        h * fmaf(h2, fmaf(h2, fmaf(h2, fmaf(h2, 2.60522491e-6f, -1.98090753e-4f), 8.33305106e-3f), -1.66666580e-1f),
                 9.99999996e-1f);
    const float ch =
        fmaf(h2, fmaf(h2, fmaf(h2, fmaf(h2, fmaf(h2, -2.60514952e-7f, 2.47601613e-5f), -1.38883614e-3f),
                                   4.16666363e-2f), -4.99999994e-1f), 1.0f);
    const float sh2 = sh + sh;
    it.c = fmaf(-sh2, sh, 1.0f);
    it.s = sh2 * ch;
}

// The amplitudes depend on the seed alone (eta is the same for every strip),
// so a prep kernel evaluates them once per (segment, pixel pair) and the
// strips read them back.
__device__ __forceinline__ void xm_amps(float g, double ta, float eta_scale, float (&a)[5])
{
    const float x = (float)ta * eta_scale, x2 = x * x;
    const float gb = g * (float)(1 << kXmBShift);
    const float gx = gb * x, gx2 = gx * x, gx3 = gx2 * x, gx4 = gx3 * x;
    // eps_m J_m(x) 2^g_m: J0 = 1 - x^2/4 + x^4/64 - x^6/2304, 2^2 * 2 J1 = 4x (1 - x^2/8 + x^4/192),
    // 2^5 * 2 J2 = 8x^2 (1 - x^2/12 + x^4/384), 2^9 * 2 J3 = (64/3) x^3 (1 - x^2/16),
    // 2^14 * 2 J4 = (256/3) x^4 (1 - x^2/20)
    a[0] = gb * fmaf(x2, fmaf(x2, fmaf(x2, -1.0f / 2304.0f, 1.0f / 64.0f), -0.25f), 1.0f);
    a[1] = gx * fmaf(x2, fmaf(x2, 4.0f / 192.0f, -0.5f), 4.0f);
    a[2] = gx2 * fmaf(x2, fmaf(x2, -8.0f / 384.0f, 8.0f / 12.0f), -8.0f);  // negated
    a[3] = gx3 * fmaf(x2, -64.0f / 48.0f, 64.0f / 3.0f);
    a[4] = gx4 * fmaf(x2, -256.0f / 60.0f, 256.0f / 3.0f);
}

// amp[t][q] = (a_0, a_1, a_2, a_3), amp4[t][q] = a_4 for segment t and pixel
// pair q (the pair's first pixel carries the seeds).
__device__ __forceinline__ void xm_amp(const XmArgs &x, int64_t block, const float *__restrict__ gamma,
                                       const double *__restrict__ tau, const double *__restrict__ rec,
                                       float4 *__restrict__ amp, float *__restrict__ amp4)
{
    const int64_t npairs = x.a.npix / 2;
    const int64_t i = block * 256 + threadIdx.x;
    if (i >= (int64_t)x.a.nt * npairs) return;
    const int64_t t = i / npairs, q = i - t * npairs;
    const int64_t off = t * x.a.npix + q;
    float a[5];
    const bool wide = (int)rec[1] == kXFormWide;
    xm_amps(gamma[off], tau[off], (float)(wide ? x.eta_scale * kXmWideScale : x.eta_scale), a);
    amp[i] = make_float4(a[0], a[1], a[2], a[3]);
    if (!wide) amp4[i] = a[4];
}

// Second preparation launch, once the form is known: nfrag workgroups of data-side
// fragments, the rest amplitudes.
__global__ __launch_bounds__(256) void xm_operands_kernel(XmArgs x, const float2 *__restrict__ C,
                                                          const float *__restrict__ w, const int *__restrict__ e_in,
                                                          const float *__restrict__ gamma,
                                                          const double *__restrict__ tau,
                                                          const double *__restrict__ rec, uint4 *__restrict__ A,
                                                          float4 *__restrict__ amp, float *__restrict__ amp4,
                                                          int64_t nfrag)
{
    if (blockIdx.x < nfrag) xm_afrag(x, blockIdx.x, C, w, e_in, rec, A);
    else xm_amp(x, blockIdx.x - nfrag, gamma, tau, rec, amp, amp4);
}

// Split a float32 value into float16 hi + lo with plain float32 arithmetic: hi
// keeps the leading 11 significant bits (truncation, exact in float16 in the
// scaled range), lo = v - hi is exact in float32 and rounded once to float16, so
// hi + lo = v (1 + O(2^-21)).
__device__ __forceinline__ void split_f16(float v, float &hi, float &lo)
{
    hi = __uint_as_float(__float_as_uint(v) & 0xFFFFE000u);
    lo = v - hi;
}

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

// Two float32 values rounded (to nearest even) into one register of float16.
__device__ __forceinline__ uint32_t pack_f16(float a, float b)
{
    h2 r;
    r.x = (_Float16)a;
    r.y = (_Float16)b;
    return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ f32x16 mfma16(const uint4 &a, const uint4 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// Pixel-side operands of term M, Re U_m and Im U_m = a_m i^m (c + i s):
//   m = 0, 4: (a c, a s); m = 1: (-a s, a c); m = 2: (a' c, a' s), a' = -a_2; m = 3: (a s, -a c);
// then the matrix products with the strip's data-side operands.
// Data-side fragments of term M for this lane (hi and, split, lo parts of
// both components and bin blocks), read from LDS ahead of their use.
struct XmFrags {
    uint4 h[2][2], l[2][2];
};

template <int M, bool SPLIT, int NA>
__device__ __forceinline__ XmFrags xm_frags(const uint4 (*As)[64], int lane)
{
    XmFrags fr;
#pragma unroll
    for (int comp = 0; comp < NA; ++comp)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const int f = comp * kXmParts * 2 + jb;
            fr.h[comp][jb] = As[f + 2 * xm_part(M, false)][lane];
            if (SPLIT) fr.l[comp][jb] = As[f + 2 * xm_part(M, true)][lane];
        }
    return fr;
}

template <int M, bool SPLIT, int NC, int NA>
__device__ __forceinline__ void xm_term(const XmItem (&items)[8], const XmFrags &fr, f32x16 (&acc)[2][2])
{
    // hi and lo must come from the same rounded float32 product
#pragma clang fp contract(off)
    constexpr bool ODD = (M & 1) != 0;
    uint32_t bh[2][4], bl[2][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float v[2][2];  // [comp][item of the pair]
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const XmItem &u = items[2 * q + e];
            const float xr = ODD ? u.s : u.c, xi = ODD ? u.c : u.s;
            v[0][e] = (M == 1 ? -u.a[M] : u.a[M]) * xr;
            v[1][e] = (M == 3 ? -u.a[M] : u.a[M]) * xi;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (SPLIT) {
                float h0, l0, h1, l1;
                split_f16(v[c][0], h0, l0);
                split_f16(v[c][1], h1, l1);
                bh[c][q] = pack_f16(h0, h1);
                bl[c][q] = pack_f16(l0, l1);
            } else {
                bh[c][q] = pack_f16(v[c][0], v[c][1]);
            }
        }
    }
    uint4 h4[2], l4[2];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        h4[c] = make_uint4(bh[c][0], bh[c][1], bh[c][2], bh[c][3]);
        if (SPLIT) l4[c] = make_uint4(bl[c][0], bl[c][1], bl[c][2], bl[c][3]);
    }
#pragma unroll
    for (int comp = 0; comp < NA; ++comp) {
        const int u = comp < NC ? comp : 0;  // both halves of a wide strip share their operand
        if (SPLIT) {
            acc[comp][0] = mfma16(fr.l[comp][0], h4[u], acc[comp][0]);
            acc[comp][1] = mfma16(fr.l[comp][1], h4[u], acc[comp][1]);
            acc[comp][1] = mfma16(fr.h[comp][1], l4[u], acc[comp][1]);
            acc[comp][0] = mfma16(fr.h[comp][0], l4[u], acc[comp][0]);
        }
        acc[comp][0] = mfma16(fr.h[comp][0], h4[u], acc[comp][0]);
        acc[comp][1] = mfma16(fr.h[comp][1], h4[u], acc[comp][1]);
    }
}

// One chunk of data-side fragments (up to kXmFrags x 64 uint4, 32 KiB: the 24 KiB
// that a four-term form reads, half of either for real data) from global memory
// straight into LDS: each wave moves 64 consecutive uint4 per instruction (lane
// l to slot l of the wave's base).
constexpr int kVmcnt0 = 0x0F70;  // s_waitcnt vmcnt(0), expcnt and lgkmcnt left at their maxima

// Global-memory view of a pointer.  The multi-job kernel reads its pointers
// out of a job table, so the compiler cannot tell them from LDS pointers and
// would use flat instructions, which count against the LDS counter as well
// and must wait for the direct copies into LDS; through this view every
// access is a plain global one.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T *gmem(T *p)
{
    return (__attribute__((address_space(1))) T *)p;
}

template <class T>
__device__ __forceinline__ __attribute__((address_space(3))) T *lds_ptr(T *p)
{
    return (__attribute__((address_space(3))) T *)p;
}

// A view of `bytes` bytes of global memory at a wave-uniform address; its users
// stay inside it.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_view(const void *p, int64_t bytes)
{
    const uint64_t a = (uint64_t)(uintptr_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    const uint64_t n = bytes < 0 ? 0 : (uint64_t)bytes > 0xffffffffull ? 0xffffffffull : (uint64_t)bytes;
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)hi << 32) | lo), 0,
                                             __builtin_amdgcn_readfirstlane((int)(uint32_t)n), 0x00020000);
}

// With real data (NA = 1) only the first component's half is copied: the
// second component's operands are zero and never read.
template <int NA, int NT>
__device__ __forceinline__ void stage_frags(const uint4 *__restrict__ src, uint4 *dst)
{
    constexpr int rows = NT <= 4 ? 12 : 16;  // of a component's 16
    static_assert(rows % kXmWaves == 0, "one row of 64 uint4 per wave and instruction");
    const auto view = buffer_view(src, kXmFrags * 64 * (int64_t)sizeof(uint4));
    const uint32_t off = threadIdx.x * 16u;
    const int w0 = __builtin_amdgcn_readfirstlane(threadIdx.x) & ~63;
#pragma unroll
    for (int c = 0; c < NA; ++c)
#pragma unroll
        for (int r = c * 16; r < c * 16 + rows; r += kXmWaves)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(view, lds_ptr(dst + r * 64 + w0), 16, off, r * 1024, 0, 0);
}

// One tile: 128 pixel pairs (block pblock) x one strip (index strip_rel within
// the call's strips).  Called by all threads of the workgroup.  NC = 1 for
// real data (C = 1): the imaginary component, identically zero, is skipped.
template <int NC, int NT, bool SPLIT2, bool EXT>
__device__ __forceinline__ void xm_tile_n(const XmArgs &x, int64_t strip_rel, int64_t pblock,
                                        const uint4 *__restrict__ A, const int *__restrict__ e_in,
                                        const float4 *__restrict__ amp, const float *__restrict__ amp4,
                                        const double *__restrict__ tau, float *__restrict__ X, uint4 (*As0)[64],
                                        uint4 (*As1)[64])
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t npairs = x.a.npix / 2;
    constexpr bool WIDE = NT == 3;
    constexpr int NA = NC == 2 || WIDE ? 2 : 1;  // components, or halves of a wide strip
    const int64_t strip = (WIDE ? x.a.k0 / kXmWideS : x.strip_first) + strip_rel;
    const int64_t p = pblock * kXmPairs + wv * 32 + (lane & 31);
    const bool pvalid = p < npairs;
    const int64_t pc = pvalid ? p : 0;
    const double fc = x.a.f0 + (WIDE ? (double)(strip * kXmWideS) + 63.5 : (double)(strip * kXmS) + 31.5) * x.a.df;  // strip centre
    const double fm = EXT ? 1.0 : fc;
    const uint4 *Ast = A + strip_rel * x.nchunks * kXmFrags * 64;

    f32x16 acc[2][2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[c][jb][r] = 0.0f;

    // the barrier orders this tile's first copy into LDS after the previous tile's reads
    __syncthreads();

    // Seeds (delays and amplitudes) of this lane's 8 segments, loaded one chunk
    // ahead through buffer views: the chunk's first row is the view's base, the
    // row within a half a scalar offset and the lane's place a vector offset
    // that never changes, so a load costs no vector instruction for its address
    // (64-bit row addresses took 40 per chunk, 16 of them quarter-rate).  Every
    // row lies inside the day (seed_rows.h): a view's range check need not take
    // the scalar offset into account.  (Scalar offsets that also repeat the last
    // row of a day of fewer than eight segments made the full band 1.5 % slower;
    // such a day is EXT.)  A row of delays and one of amplitudes have the same
    // number of bytes.
    f32x4 aN[8];
    float a4N[8];
    double tN[8];
    const uint32_t row = (uint32_t)npairs * 16u;
    const uint32_t aoff = (uint32_t)(lane >> 5) * (uint32_t)half_row(x.a.nt) * row + (uint32_t)pc * 16u;
    const uint32_t toff = aoff - (uint32_t)pc * 8u, a4off = aoff >> 2;
    auto load_seeds = [&](int64_t ch) {
        const int64_t first = chunk_row(x.a.nt, ch), left = x.a.nt - first;  // the window's first row, rows to the end
        if constexpr (EXT) {  // a chunk's rows may span more than 32 bits of bytes, or be fewer than eight
            const int t0 = (int)first + (lane >> 5) * half_row(x.a.nt);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int t = t0 + slot_row(x.a.nt, e);
                const int64_t q = (int64_t)t * npairs + pc;
                aN[e] = gmem(reinterpret_cast<const f32x4 *>(amp))[q];
                if (NT == 5) a4N[e] = gmem(amp4)[q];
                tN[e] = gmem(tau)[(int64_t)t * x.a.npix + pc];
            }
            return;
        }
        const auto va = buffer_view(amp + first * npairs, left * row);
        const auto vt = buffer_view(tau + first * x.a.npix, left * row);
        const auto v4 = buffer_view(amp4 + first * npairs, left * (row >> 2));
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            aN[e] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(va, aoff, e * row, 0));
            if (NT == 5)
                a4N[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(v4, a4off, e * (row >> 2), 0));
            tN[e] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(vt, toff, e * row, 0));
        }
    };
    load_seeds(0);
    stage_frags<NA, NT>(Ast, &As0[0][0]);
    // chunk 0's seeds and operands have landed: the loop starts with nothing in flight
    __builtin_amdgcn_s_waitcnt(kVmcnt0);
    __syncthreads();

    XmItem items[8];
    // One chunk: its operands are in Acur; the next chunk's go straight into
    // Anext (its readers finished at the previous barrier) while the chunk's
    // products run.  The two buffers are distinct LDS variables, so reads of
    // one need not be ordered after the copy into the other.
    auto step = [&](int64_t ch, const uint4 (*Acur)[64], uint4 (*Anext)[64]) {
        const bool more = ch + 1 < x.nchunks;
        // the first term's fragments are read from LDS while the items are computed
        XmFrags fa = xm_frags<NT - 1, false, NA>(Acur, lane);
        if constexpr (EXT) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                tN[e] = fma(fc, tN[e], -rint(fc * tN[e]));  // the phase's fraction
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            xm_phase(tN[e], fm, items[e]);
            items[e].a[0] = aN[e].x;
            items[e].a[1] = aN[e].y;
            items[e].a[2] = aN[e].z;
            items[e].a[3] = aN[e].w;
            items[e].a[4] = NT == 5 ? a4N[e] : 0.0f;
        }
        // issued after the seeds are consumed, so no wait for them holds the copy up
        if (more) stage_frags<NA, NT>(Ast + (ch + 1) * kXmFrags * 64, &Anext[0][0]);
        // unconditional (the last chunk reloads its own seeds, unused): a
        // conditional load would be joined by register copies that wait for it
        load_seeds(more ? ch + 1 : ch);
        // the scheduler would move these loads to the chunk's end, where their
        // whole latency is waited for
        __builtin_amdgcn_sched_barrier(0);
        // a wave in its products goes before one in its vector phase
        __builtin_amdgcn_s_setprio(1);
        // smallest terms first: fixed order; each term's fragments are read
        // one term ahead
        if constexpr (NT == 5) {
            const XmFrags f3 = xm_frags<3, false, NA>(Acur, lane);
            xm_term<4, false, NC, NA>(items, fa, acc);
            fa = f3;
        }
        if constexpr (!WIDE) {
            const XmFrags f2 = xm_frags<2, SPLIT2, NA>(Acur, lane);
            xm_term<3, false, NC, NA>(items, fa, acc);
            fa = f2;
        }
        const XmFrags f1 = xm_frags<1, true, NA>(Acur, lane);
        xm_term<2, SPLIT2, NC, NA>(items, fa, acc);
        const XmFrags f0 = xm_frags<0, true, NA>(Acur, lane);
        xm_term<1, true, NC, NA>(items, f1, acc);
        xm_term<0, true, NC, NA>(items, f0, acc);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_s_waitcnt(kVmcnt0);  // the copy into Anext (and the seeds) have landed
        __syncthreads();
    };
    for (int64_t ch = 0; ch < x.nchunks; ch += 2) {
        step(ch, As0, As1);
        if (ch + 1 < x.nchunks) step(ch + 1, As1, As0);
    }

    if (!pvalid) return;  // lanes l and l ^ 32 hold the same pair: both leave or both stay
    const int64_t pB = antipode_north(ring_of_north(p, x.a.nside), x.a.npix);
    const int64_t col0 = strip * (WIDE ? kXmWideS : kXmS) - x.a.k0;
    double sa = 0.0, sb = 0.0;  // this lane's share of the strip's broadband sums
    if constexpr (NC == 1) {
        // Real data are the neighbour terms that are added into a map.
        // Read-modify-write of the map: the loads of 64 bins (32 in a wide strip,
        // whose sums leave room for no more) are issued before any is used (one
        // wait instead of two round trips per output): the scale exponents and
        // the old values, at a clamped row.
        constexpr int NB = WIDE ? 1 : 2;  // blocks of 32 bins a batch
#pragma unroll
        for (int b = 0; b < 2 * NA; b += NB) {
            int ex[NB][16];
            float olda[NB][16], oldb[NB][16];
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = (b + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    const int64_t c = col0 + j, cc = c < 0 ? 0 : (c >= x.a.nf ? x.a.nf - 1 : c);
                    ex[i][r] = gmem(e_in)[cc + x.a.k0 - x.strip_first * kXmS];
                    auto row = gmem(X + cc * (int64_t)x.a.npix);
                    olda[i][r] = row[p];
                    oldb[i][r] = row[pB];
                }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = (b + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    const int64_t c = col0 + j;
                    if (c < 0 || c >= x.a.nf) continue;
                    const float v = acc[(b + i) >> 1][(b + i) & 1][r] * ldexpf(1.0f, -ex[i][r] - kXmBShift);
                    auto row = gmem(X + c * (int64_t)x.a.npix);
                    row[p] = olda[i][r] + v;
                    row[pB] = oldb[i][r] + v;
                }
        }
    } else {
        // write-only: streaming stores (the map is not read back here), or
        // none at all for a broadband-only call.  Batching the exponent loads
        // here as above measured 1.5 % slower, so they stay one per output.
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = jb * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                const int64_t c = col0 + j;
                if (c < 0 || c >= x.a.nf) continue;
                const float inv = ldexpf(1.0f, -gmem(e_in)[strip_rel * kXmS + j] - kXmBShift);
                const float pi = acc[1][jb][r];
                const float xa = (acc[0][jb][r] - pi) * inv, xb = (acc[0][jb][r] + pi) * inv;
                if (X) {
                    auto row = gmem(X + c * (int64_t)x.a.npix);
                    __builtin_nontemporal_store(xa, &row[p]);
                    __builtin_nontemporal_store(xb, &row[pB]);
                }
                if (c >= x.a.band_lo && c < x.a.band_hi) {
                    sa += (double)xa;
                    sb += (double)xb;
                }
            }
    }
    if (x.a.band_part) {
        // lower half-wave's 32 bins, then the upper half's: one fixed order
        const double oa = __shfl_xor(sa, 32), ob = __shfl_xor(sb, 32);
        if (lane < 32) {
            auto part = gmem(x.a.band_part + strip_rel * (int64_t)x.a.npix);
            part[p] = sa + oa;
            part[pB] = sb + ob;
        }
    }
}

int64_t xm_band_rows(const MapArgs &a)
{
    const int64_t first = a.k0 / kXmS;
    return (a.k0 + a.nf - 1) / kXmS - first + 1;
}

// A tile of a call whose seeds were rejected: NaN in every output it owns
// (the map rows and, if requested, the strip's broadband sums), so that a
// wrong promise about the seeds cannot pass as a map.
__device__ __forceinline__ void xm_tile_reject(const XmArgs &x, int64_t strip_rel, int64_t pblock,
                                               float *__restrict__ X)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t npairs = x.a.npix / 2;
    const int64_t p = pblock * kXmPairs + wv * 32 + (lane & 31);
    if (p >= npairs) return;
    const int64_t pB = antipode_north(ring_of_north(p, x.a.nside), x.a.npix);
    const int64_t col0 = (x.strip_first + strip_rel) * kXmS - x.a.k0;
    const float nan = __builtin_nanf("");
    for (int jj = 0; X && jj < 32; ++jj) {
        const int64_t c = col0 + (lane >> 5) * 32 + jj;
        if (c < 0 || c >= x.a.nf) continue;
        auto row = gmem(X + c * (int64_t)x.a.npix);
        row[p] = nan;
        row[pB] = nan;
    }
    if (x.a.band_part && lane < 32) {
        auto part = gmem(x.a.band_part + strip_rel * (int64_t)x.a.npix);
        part[p] = (double)nan;
        part[pB] = (double)nan;
    }
}

// The form the prep chose for the call (uniform per launch: the same decision
// for every tile, sub-band and schedule).  SGWB_XFORM_VALU: a gated
// vector-unit launch computes the map, these workgroups have nothing to do.
template <int NC, bool EXT>
__device__ __forceinline__ void xm_tile(const XmArgs &x, int64_t strip_rel, int64_t pblock,
                                        const uint4 *__restrict__ A, const int *__restrict__ e_in,
                                        const double *__restrict__ rec, const float4 *__restrict__ amp,
                                        const float *__restrict__ amp4, const double *__restrict__ tau,
                                        float *__restrict__ X, uint4 (*As0)[64], uint4 (*As1)[64])
{
    const int form = (int)gmem(rec)[1];
    if (NC == 1 && form == kXFormWide)
        xm_tile_n<1, 3, false, EXT>(x, strip_rel, pblock, A, e_in, amp, amp4, tau, X, As0, As1);
    else if (form == SGWB_XFORM_MFMA4)
        xm_tile_n<NC, 4, false, EXT>(x, strip_rel, pblock, A, e_in, amp, amp4, tau, X, As0, As1);
    else if (form == SGWB_XFORM_MFMA5)
        xm_tile_n<NC, 5, false, EXT>(x, strip_rel, pblock, A, e_in, amp, amp4, tau, X, As0, As1);
    else if (form == SGWB_XFORM_MFMA5S)
        xm_tile_n<NC, 5, true, EXT>(x, strip_rel, pblock, A, e_in, amp, amp4, tau, X, As0, As1);
    else if (form == kXFormRejected)
        xm_tile_reject(x, strip_rel, pblock, X);
}

// Workgroups are dealt round-robin to the 8 XCDs (L2 domains) of the chip in
// launch order.  Tile T of n goes to the workgroups of XCD T's eighth: XCD x
// takes the x-th contiguous range of tiles, so the workgroups that run together
// on one XCD work on neighbouring tiles.  A bijection for any n.
constexpr int kXcds = 8;

// Order of the (strip, pixel block) tiles: blocks of kXmPB pixel blocks, all
// strips inside a block, pixel blocks fastest.  The ~64 workgroups resident on
// one XCD then cover 16 strips x 4 pixel blocks and share, chunk by chunk, the
// seeds of 4 pixel blocks (49 KB each) and the data operands of 16 strips
// (24-32 KB each) through that XCD's L2.  A bijection for any strip and block
// counts.  Measured with 2 / 4 / 8 / 16 pixel blocks: the full band at nside 32
// 14.9 / 14.9 / 15.3 / 18.6 ms, at nside 64 (X and Gam) 60.0 / 57.8 / 58.7 ms / -,
// 6272 bins at nside 16 620 / 618 / 629 / 635 us.
constexpr uint32_t kXmPB = 4;
__device__ __forceinline__ void xm_tile_coords(uint32_t T, uint32_t nstrips, uint32_t npb, uint32_t &strip,
                                               uint32_t &pb)
{
    const uint32_t fb = npb / kXmPB, full = fb * kXmPB * nstrips;
    if (T < full) {
        const uint32_t per = kXmPB * nstrips, b = T / per, r = T - b * per;
        strip = r / kXmPB;
        pb = b * kXmPB + (r - strip * kXmPB);
    } else {
        const uint32_t rem = npb - fb * kXmPB, r = T - full;
        strip = r / rem;
        pb = fb * kXmPB + (r - strip * rem);
    }
}
__device__ __forceinline__ int64_t xcd_range_begin(int64_t x, int64_t n)
{
    const int64_t q = n / kXcds, r = n % kXcds;
    return x * q + (x < r ? x : r);
}

__device__ __forceinline__ int64_t xcd_tile(int64_t L, int64_t n)
{
    return xcd_range_begin(L % kXcds, n) + L / kXcds;
}

// Bound by the matrix products (43 % of a SIMD's cycles at nside 64) and the vector
// work that builds their pixel-side operands (57 %), and on the full band by the
// package's power cap.  Four waves a workgroup, so that two workgroups share a compute unit
// and one's vector phase runs beside the other's products (eight waves of one
// workgroup meet at every chunk's barrier in the same phase), and so that the
// last round of tiles is half as long.  Measured, a day at 1/32 Hz, whole calls: 98
// strips at nside 16 with their Fisher diagonal 744 -> 633 us, at nside 32 the
// overlap diagonal of 4101 bins 1210 -> 1008 us and the full band 16.04 -> 15.45 ms, against
// one eight-wave workgroup with 64-bit seed addresses, every part copied and the
// phase reduced by four float64 instructions (eight waves with the other changes:
// 725 and 1164 us).  With what came since (strips of 128 bins for the overlap
// terms, one preparation launch, the tile order): 618 us, 834 us, 14.9 ms.
template <int NC, bool EXT>
__global__ __launch_bounds__(64 * kXmWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void xm_main_kernel(
    XmArgs x, int64_t npblocks, const uint4 *__restrict__ A, const int *__restrict__ e_in,
    const double *__restrict__ tmax, const float4 *__restrict__ amp, const float *__restrict__ amp4,
    const double *__restrict__ tau, float *__restrict__ X)
{
    __shared__ uint4 As0[kXmFrags][64], As1[kXmFrags][64];  // 2 x 32 KB
    uint32_t sr, pb;
    int64_t nstrips = x.nstrips;
    if (NC == 1 && (int)gmem(tmax)[1] == kXFormWide) {
        nstrips = xm_wide_strips(x);
        if (blockIdx.x >= nstrips * npblocks) return;
    }
    xm_tile_coords((uint32_t)xcd_tile(blockIdx.x, nstrips * npblocks), (uint32_t)nstrips, (uint32_t)npblocks, sr, pb);
    xm_tile<NC, EXT>(x, sr, pb, A, e_in, tmax, amp, amp4, tau, X, As0, As1);
}

// Multi-job form: one launch over the tiles of all jobs, one workgroup per tile.
// Every XCD takes the x-th eighth of every job (each job in the blocked order
// above), so jobs of different cost (number of terms, segments) load the XCDs
// evenly; XCD x works through its ranges job after job.  Launched with
// 8 sum_j ceil(n_j / 8) workgroups: the few slots past an XCD's share exit.
// (A persistent loop over tiles was measured slower: its state pushed the
// kernel to the register limit.)  A tile's result does not depend on which
// workgroup computes it.  No job is XmArgs::ext (a plan launches those job by
// job).
__global__ __launch_bounds__(64 * kXmWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void xm_batched_kernel(
    const XmJob *__restrict__ jobs, int32_t njobs)
{
    __shared__ uint4 As0[kXmFrags][64], As1[kXmFrags][64];
    const int64_t xcd = blockIdx.x % kXcds;
    int64_t slot = blockIdx.x / kXcds;
    int j = 0;
    int64_t tile = -1;
    for (; j < njobs; ++j) {
        const int64_t n = jobs[j].x.nstrips * jobs[j].npblocks;
        const int64_t lo = xcd_range_begin(xcd, n), cnt = xcd_range_begin(xcd + 1, n) - lo;
        if (slot < cnt) {
            tile = lo + slot;
            break;
        }
        slot -= cnt;
    }
    if (tile < 0) return;  // padding slot: this XCD's share is done
    j = __builtin_amdgcn_readfirstlane(j);  // uniform
    uint32_t sr, pb;
    xm_tile_coords((uint32_t)tile, (uint32_t)jobs[j].x.nstrips, (uint32_t)jobs[j].npblocks, sr, pb);
    xm_tile<2, false>(jobs[j].x, sr, pb, jobs[j].A, jobs[j].e, jobs[j].tmax, jobs[j].amp, jobs[j].amp4, jobs[j].tau, jobs[j].X,
            As0, As1);
}

void fill_xmjob(XmJob *j, const MapArgs &a, const float *C, const float *w, const float *gamma, const double *tau,
                float *X, void *work)
{
    XmArgs &x = j->x;
    x.a = a;
    x.strip_first = a.k0 / kXmS;
    x.nstrips = (a.k0 + a.nf - 1) / kXmS - x.strip_first + 1;
    x.nchunks = (a.nt + kXmT - 1) / kXmT;
    x.eta_scale = kTwoPi * 31.5 * a.df;
    const double fmax = std::max(std::fabs(a.f0 + a.df * (double)(a.k0 - kXmS)),
                                 std::fabs(a.f0 + a.df * (double)(a.k0 + a.nf + kXmS)));
    // delays reach 2 R / c, the overlap terms' differences of two 4 R / c
    x.ext = !(fmax * 4.0 * kEarthRadius / kLightSpeed < kXmMaxTurns) ||
            (int64_t)(a.npix / 2) * 16 * kXmT > 0xffffffffll || a.nt < kXmHalf;
    const size_t frag_bytes = (size_t)x.nstrips * x.nchunks * kXmFrags * 64 * sizeof(uint4);
    j->A = reinterpret_cast<uint4 *>(work);
    j->e = reinterpret_cast<int *>(reinterpret_cast<char *>(work) + (frag_bytes + 255) / 256 * 256);
    const size_t scale_bytes = (size_t)x.nstrips * kXmS * sizeof(int);
    char *tm = reinterpret_cast<char *>(work) + up256_(frag_bytes) + up256_(scale_bytes);
    j->tmax = reinterpret_cast<double *>(tm);
    const size_t items = (size_t)a.nt * (a.npix / 2);
    j->amp = reinterpret_cast<float4 *>(tm + up256_(kXmRecWords * sizeof(double)));
    j->amp4 = reinterpret_cast<float *>(reinterpret_cast<char *>(j->amp) + up256_(items * sizeof(float4)));
    j->C = C;
    j->w = w;
    j->gamma = gamma;
    j->tau = tau;
    j->X = X;
    j->npblocks = (a.npix / 2 + kXmPairs - 1) / kXmPairs;
    j->tile_begin = 0;
}

int64_t xmjob_tiles(const XmJob &j) { return j.x.nstrips * j.npblocks; }

// Preparation of a call: of its data (per-bin scales and the A fragments), of its
// seeds (the form record and the Bessel amplitudes, which depend on the seeds
// and the frequency spacing alone), or of both.
static hipError_t launch_xm_prep_parts(const XmJob &j, bool data, bool seeds, hipStream_t s)
{
    const float2 *Cc = reinterpret_cast<const float2 *>(j.C);
    const int64_t n = (int64_t)j.x.a.nt * j.x.a.npix;
    const int64_t nscale = data ? j.x.nstrips : 0, nsym = seeds ? kSymParts : 0;
    const int64_t ntmax = seeds ? std::min<int64_t>(kTmaxParts, (n + 4 * kXmPrepThreads - 1) / (4 * kXmPrepThreads)) : 0;
    double *part = j.tmax + 2, *flags = j.tmax + 2 + kTmaxParts;
    auto prep = [&](int64_t scale, int64_t sym, int64_t tmax) {
        hipLaunchKernelGGL(xm_prep_kernel, dim3((unsigned)(scale + sym + tmax)), dim3(kXmPrepThreads), 0, s, j.x, Cc,
                           j.w, const_cast<int *>(j.e), j.gamma, j.tau, flags, part, scale, sym, tmax);
    };
    if (!data || !seeds || fits_launch(nscale + nsym + ntmax, kXmPrepThreads)) {
        prep(nscale, nsym, ntmax);
    } else {
        prep(nscale, 0, 0);
        prep(0, nsym, ntmax);
    }
    if (seeds)
        hipLaunchKernelGGL(xm_tmax_final_kernel, dim3(1), dim3(256), 0, s, part, (int)ntmax, flags, j.x.eta_scale,
                           j.x.a.tau_limit, j.x.a.unit_c, j.tmax);
    const int64_t nfrag = data ? j.x.nstrips * j.x.nchunks : 0;  // 4 x 64 threads each
    const int64_t namp = seeds ? ((int64_t)j.x.a.nt * (j.x.a.npix / 2) + 255) / 256 : 0;
    auto operands = [&](int64_t frag, int64_t amp) {
        hipLaunchKernelGGL(xm_operands_kernel, dim3((unsigned)(frag + amp)), dim3(256), 0, s, j.x, Cc, j.w, j.e,
                           j.gamma, j.tau, j.tmax, const_cast<uint4 *>(j.A), j.amp, j.amp4, frag);
    };
    if (!data || !seeds || fits_launch(nfrag + namp, 256)) {
        operands(nfrag, namp);
    } else {
        operands(nfrag, 0);
        operands(0, namp);
    }
    return hipGetLastError();
}

hipError_t launch_xm_prep(const XmJob &j, hipStream_t s) { return launch_xm_prep_parts(j, true, true, s); }

size_t xm_seed_bytes(int32_t nt, int32_t npix)
{
    const size_t items = (size_t)nt * (npix / 2);
    return up256_(kXmRecWords * sizeof(double)) + up256_(items * sizeof(float4)) + up256_(items * sizeof(float));
}

// Point a job's seed-side products at a caller's buffer of xm_seed_bytes().
static void use_seed_buffer(XmJob *j, void *seeds)
{
    const size_t items = (size_t)j->x.a.nt * (j->x.a.npix / 2);
    char *p = reinterpret_cast<char *>(seeds);
    j->tmax = reinterpret_cast<double *>(p);
    j->amp = reinterpret_cast<float4 *>(p + up256_(kXmRecWords * sizeof(double)));
    j->amp4 = reinterpret_cast<float *>(reinterpret_cast<char *>(j->amp) + up256_(items * sizeof(float4)));
}

hipError_t launch_xm_seed_products(const MapArgs &a, const float *gamma, const double *tau, void *seeds,
                                   hipStream_t s)
{
    XmJob j;
    fill_xmjob(&j, a, nullptr, nullptr, gamma, tau, nullptr, nullptr);
    use_seed_buffer(&j, seeds);
    return launch_xm_prep_parts(j, false, true, s);
}

hipError_t launch_xm_batched(const XmJob *jobs_dev, int32_t njobs, int64_t grid, hipStream_t s)
{
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(xm_batched_kernel, dim3((unsigned)grid), dim3(64 * kXmWaves), 0, s, jobs_dev, njobs);
    return hipGetLastError();
}

int64_t xm_batched_grid(const XmJob *jobs, int32_t njobs)
{
    int64_t per_xcd = 0;
    for (int32_t j = 0; j < njobs; ++j) per_xcd += (xmjob_tiles(jobs[j]) + kXcds - 1) / kXcds;
    return per_xcd * kXcds;
}

hipError_t launch_xm_main(const XmJob &j, hipStream_t s)
{
    const int64_t ntiles = xmjob_tiles(j);
    if (ntiles > 0x7fffffff) return hipErrorInvalidValue;
    if (ntiles == 0) return hipSuccess;
    const auto kernel = j.x.a.unit_c ? (j.x.ext ? xm_main_kernel<1, true> : xm_main_kernel<1, false>)
                                     : (j.x.ext ? xm_main_kernel<2, true> : xm_main_kernel<2, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)ntiles), dim3(64 * kXmWaves), 0, s, j.x, j.npblocks, j.A, j.e, j.tmax,
                       j.amp, j.amp4, j.tau, j.X);
    return hipGetLastError();
}

hipError_t launch_dirty_map_mfma(const MapArgs &a, const float *C, const float *w, const float *gamma,
                                 const double *tau, float *X, void *work, hipStream_t s, const double **form_rec,
                                 const void *seeds)
{
    XmJob j;
    fill_xmjob(&j, a, C, w, gamma, tau, X, work);
    if (seeds) use_seed_buffer(&j, const_cast<void *>(seeds));
    if (form_rec) *form_rec = j.tmax;
    hipError_t err = launch_xm_prep_parts(j, true, !seeds, s);
    if (err != hipSuccess) return err;
    return launch_xm_main(j, s);
}

}  // namespace sgwb
