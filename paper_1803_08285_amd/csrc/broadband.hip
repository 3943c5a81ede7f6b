// Broadband dirty map with the sum over the band's bins taken first (Sec. V:
// the broadband map is the sum of the narrowband maps over a band; Eq.
// eq_dirtymap written per bin).  Exchanging the sums over bins and segments,
//   Xbb(p) = sum_t gamma(t,p) Re[ e^{2 pi i f_c tau} Y_t(tau) ],  tau = tau(t,p),
//   Y_t(tau) = sum_{k in band} y(t,k) e^{2 pi i (f_k - f_c) tau},  y = w C,
// with f_c the band's centre.  Y_t is a trigonometric polynomial in tau whose
// frequencies lie within F = (nb - 1) df / 2 of zero, so it is smooth on the
// scale 1 / F: one table per segment on a uniform delay grid, read with
// 4-point Lagrange interpolation, replaces the per-bin phase of every
// (segment, bin, pixel) term by one interpolation per (segment, pixel).
//
// Kernels: the tables (float64: Y_t by Horner's rule at the few Chebyshev nodes
// that determine it, its Chebyshev series evaluated at the grid's nodes; or
// Horner's rule at every grid node), and the map pass (antipodal seeds: a pixel
// pair a thread, the tables through LDS, or for few pixels or long tables a run of
// the segments a wave; any seeds: one pixel a thread), one chunk of segments a
// workgroup row, float64 partial sums added in a fixed order by the band finish
// kernel.
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "broadband.h"

namespace sgwb {

// The delay grid: nodes tau_j = (j - m - 1) h, j = 0 .. 2m + 2, so that every
// |tau| <= m h has the four nodes j - 1 .. j + 2 around it.
//
// Spacing.  The interpolation error of 4 nodes is at most
// max|Y''''| max_x |(x+1) x (x-1) (x-2)| h^4 / 4! <= (2 pi F h)^4 (9/16) / 24 sum_k |y(t,k)|;
// 2 pi F h = kBbPhaseStep = 0.03 keeps it below 1.9e-8 of sum_k |y(t,k)|.
constexpr double kBbPhaseStep = 0.03;
constexpr int32_t kBbMaxHalf = 1 << 20;  // m: at most 2^21 + 3 nodes per table
constexpr int kBbNodes = 64;  // table nodes per workgroup (one wave)
constexpr int kBbBatch = 2;  // segments whose loads the map pass issues together
constexpr int kBbRunBatch = 4;  // the same where a run is split over the waves

bool bb_grid(int32_t nb, double df, double bound, BbGrid *g)
{
    if (!(bound > 0.0) || !isfinite(bound) || nb < 1) return false;
    const double F = 0.5 * (nb - 1) * df;
    // a single bin (F = 0) makes Y_t constant: any spacing is exact
    const double h = F > 0.0 ? kBbPhaseStep / (2.0 * kPi * F) : bound;
    const double m = ceil(bound / h);
    if (!(m <= kBbMaxHalf)) return false;
    g->m = (int32_t)(m < 1.0 ? 1.0 : m);
    g->G = 2 * g->m + 3;
    g->h = h;
    g->bound = bound;
    return true;
}

static size_t up256_(size_t n) { return (n + 255) / 256 * 256; }

// Workspace: T [nt][G] float2 | the map pass's partial sums [segment
// chunks][npix] | the Fisher band weights' scratch (v, then its partial sums)
// | the antipodal spot check's flags.
struct BbLayout {
    size_t t, part, gam, flags, total;
};
static BbLayout bb_layout(int32_t nt, int32_t npix, const BbGrid &g)
{
    const size_t ntb = kBandTChunks;
    BbLayout L;
    L.t = 0;
    L.part = L.t + up256_((size_t)nt * g.G * sizeof(float2));
    L.gam = L.part + up256_(ntb * (size_t)npix * sizeof(double));
    L.flags = L.gam + up256_(band_gamma_scratch_bytes(nt, npix));
    L.total = L.flags + up256_(kSymParts * sizeof(double));
    return L;
}

size_t bb_workspace_bytes(int32_t nt, int32_t npix, int32_t nb, const BbGrid &g)
{
    (void)nb;
    return bb_layout(nt, npix, g).total;
}

// T[t][j] = sum_k y(t,k) e^{2 pi i (k - kc) df tau_j}, kc = (nb - 1) / 2,
// y(t,k) = w[t][klo + k] C[t][klo + k]: with omega = e^{2 pi i df tau_j},
// T = omega^{-kc} sum_k y(t,k) omega^k, the sum by Horner's rule from the top
// bin down (|omega| = 1, so rounding errors do not grow with the power), all
// in float64; omega and omega^{-kc} from phases reduced in float64.  One wave
// a workgroup (blockIdx.x the segment, blockIdx.y a block of 64 nodes), its y
// staged through LDS 64 bins at a time (every lane then reads the same bin).
__global__ __launch_bounds__(kBbNodes) void bb_table_kernel(const float *__restrict__ C, const float *__restrict__ w,
                                                            int64_t ldc, int32_t klo, int32_t nb, int32_t G,
                                                            int32_t m, double dfh, float2 *__restrict__ T)
{
    __shared__ double2 ys[kBbNodes];
    const int32_t t = blockIdx.x, j = blockIdx.y * kBbNodes + threadIdx.x;
    const double node = (double)(j - m - 1);  // tau_j / h
    double turns = dfh * node;
    turns -= rint(turns);
    double os, oc;
    sincospi(2.0 * turns, &os, &oc);
    const int64_t row = (int64_t)t * ldc + klo;
    double ar = 0.0, ai = 0.0;
    for (int32_t kb = (nb - 1) / kBbNodes * kBbNodes; kb >= 0; kb -= kBbNodes) {
        const int32_t k = kb + (int32_t)threadIdx.x;
        double2 yv = make_double2(0.0, 0.0);
        if (k < nb) {
            const double wv = (double)w[row + k];
            yv = make_double2(wv * (double)C[2 * (row + k)], wv * (double)C[2 * (row + k) + 1]);
        }
        __syncthreads();  // the previous block's reads are done
        ys[threadIdx.x] = yv;
        __syncthreads();
        // bins past the band were staged as zeros: above the top bin they keep
        // the sum at exactly zero, so every block runs the full count
#pragma unroll 16
        for (int i = kBbNodes - 1; i >= 0; --i) {
            const double2 y = ys[i];
            const double nr = fma(ar, oc, fma(-ai, os, y.x));
            const double ni = fma(ar, os, fma(ai, oc, y.y));
            ar = nr;
            ai = ni;
        }
    }
    double back = 0.5 * (nb - 1) * dfh * node;  // omega^{-kc}
    back -= rint(back);
    double bs, bc;
    sincospi(-2.0 * back, &bs, &bc);
    if (j < G) T[(int64_t)t * G + j] = make_float2((float)(ar * bc - ai * bs), (float)(ar * bs + ai * bc));
}

// Y_t has frequencies within F of zero, so on the grid's span |tau| <= (m + 1) h
// it is determined to float64 rounding by N = Z / 2 + O(20) Chebyshev nodes,
// Z = 2 pi F (m + 1) h = kBbPhaseStep (m + 1): the interpolant's error is at
// most 4 sum_{n >= N} |J_n(Z)| <= about 4 (Z / 2)^N / N! of sum_k |y(t,k)| (kept
// below 1e-13).  The grid has ~67 nodes per unit of Z, so summing the band at
// the N nodes and evaluating the series at the grid's takes about a tenth of
// the operations (full day, 4096 bins, AB: N = 22 against G = 271).
constexpr int kBbChebMax = 512;  // N at most (the LDS arrays; larger N take the direct kernel)
constexpr int kBbTabThreads = 256;
constexpr int kBbStage = 512;  // bins per LDS stage, at most
constexpr int32_t kBbPrepNodes = 1024;  // grid nodes of a narrow band that one workgroup sums directly, at most

// The node count for a grid, 0 where the sums are taken at every grid node: no
// N of at most kBbChebMax, or the longest chain of recurrence steps is no
// shorter (the chains bound both forms while the segments do not fill the
// chip): nb bins over 256 / N threads a node and then N terms for every 256th
// grid node, one workgroup a segment (about 2048 run together), against nb
// bins, one wave per 64 nodes and segment (about 8192 run together).
static int32_t bb_cheb_nodes(int32_t nb, int32_t nt, const BbGrid &g)
{
    const double half = nb > 1 ? 0.5 * kBbPhaseStep * (g.m + 1) : 0.0;  // Z / 2
    double term = 4.0;  // 4 (Z / 2)^N / N!
    for (int32_t n = 1; n <= kBbChebMax; ++n) {
        term *= half / n;
        if (!(term <= 1e-13 && n > half)) continue;
        const double R = n < kBbTabThreads ? kBbTabThreads / n : (double)kBbTabThreads / n;
        const double nodes = nb / R + (double)n * ((g.G + kBbTabThreads - 1) / kBbTabThreads);
        const double every = (double)nb * std::max(1.0, (double)nt * ((g.G + kBbNodes - 1) / kBbNodes) / 8192.0);
        return nodes * std::max(1.0, nt / 2048.0) < every ? n : 0;
    }
    return 0;
}

// Everything a query needs before its map pass, in one launch.  Workgroup t <
// nt: T[t][j] as bb_table_kernel defines it, and, with v, segment t's band
// weight.  The last kSymParts workgroups, with flags: the antipodal spot check.
//
// The tables through Chebyshev nodes (N > 0).  Node sums: thread (n, r) of R =
// 256 / ceil(N / 2) takes the nodes x_n = cos(pi (n + 1/2) / N) and x_{N-1-n} =
// -x_n, whose omega are conjugate, and the bins k = r mod R, by Horner's rule in
// omega^R from the top bin down (|omega| = 1), the band staged through LDS as y =
// w C in float64, the next stage's loads in flight; the R partial sums are turned
// by omega^(r - kc) and added in a fixed order.  Then the series' coefficients
// (cosine sums of the node values) and Clenshaw's recurrence at the grid's nodes,
// two mirror images a thread (x and -x share the sums of the even and of the odd
// terms).  Bound by the float64 FMAs of the node sums (4 per bin and node), the
// LDS reads beside them (16 bytes per bin and two nodes) and the read of the
// band.  Full day, 4096 bins, AB: 38 us (one node a thread 46 us, the direct
// sums over all 271 nodes 267 us); AC, 1531 bins: 25 against 26 and 101 us.  N =
// 0: a band of at most kBbStage bins, staged once, Horner's rule at every grid
// node.
__global__ __launch_bounds__(kBbTabThreads) void bb_prep_kernel(
    const float *__restrict__ C, const float *__restrict__ w, int64_t ldc, int32_t klo, int32_t nb, int32_t G,
    int32_t m, double dfh, int32_t N, float2 *__restrict__ T, const float *__restrict__ H, double *__restrict__ v,
    const float *__restrict__ gamma, const double *__restrict__ tau, int32_t nt, int64_t npix, int64_t nside,
    double *__restrict__ flags)
{
    __shared__ double2 stage[kBbStage];
    extern __shared__ double dyn[];
    double *const ct = dyn;                                            // cos(pi i / (2 N)), i < 4 N
    double2 *const node = reinterpret_cast<double2 *>(dyn + 4 * N);    // node values
    double2 *const coef = reinterpret_cast<double2 *>(dyn + 6 * N);    // series coefficients
    const int tid = threadIdx.x;
    const int32_t t = blockIdx.x;
    if (t >= nt) {
        const int part = t - nt;
        const int bad = __syncthreads_or(antipodal_mismatch(gamma, tau, nt, npix, nside, part, kSymParts));
        if (tid == 0) flags[part] = bad ? 1.0 : 0.0;
        return;
    }
    const int64_t row = (int64_t)t * ldc + klo;
    const double kc = 0.5 * (nb - 1);
    auto bin = [&](int32_t k) {
        if (k >= nb) return make_double2(0.0, 0.0);
        const double wv = (double)w[row + k];
        return make_double2(wv * (double)C[2 * (row + k)], wv * (double)C[2 * (row + k) + 1]);
    };
    // threads per node pair, bins per stage (per for every residue r); the first
    // (top) stage's values are under way before anything else
    const int32_t half = (N + 1) / 2;
    const int32_t R = N > 0 ? kBbTabThreads / half : 1, per = kBbStage / R, sb = per * R;
    int32_t kb = N > 0 ? (nb - 1) / sb * sb : 0;
    double2 y0 = bin(kb + tid), y1 = bin(kb + tid + kBbTabThreads);
    if (v) {
        const double sum = band_weight<kBbTabThreads>(w + (int64_t)t * ldc, H, klo, klo + nb,
                                                      reinterpret_cast<double *>(stage));
        if (tid == 0) v[t] = sum;
    }
    if (N == 0) {
        __syncthreads();  // the weight's sums are read
        stage[tid] = y0;
        stage[tid + kBbTabThreads] = y1;
        __syncthreads();
        for (int32_t j = tid; j < G; j += kBbTabThreads) {
            const double at = dfh * (double)(j - m - 1);  // df tau_j
            double turns = at - rint(at), back = kc * at;
            back -= rint(back);
            double os, oc, bs, bc;
            sincospi(2.0 * turns, &os, &oc);
            sincospi(-2.0 * back, &bs, &bc);
            double ar = 0.0, ai = 0.0;
            for (int32_t k = nb - 1; k >= 0; --k) {
                const double2 y = stage[k];
                const double nr = fma(ar, oc, fma(-ai, os, y.x));
                const double ni = fma(ar, os, fma(ai, oc, y.y));
                ar = nr;
                ai = ni;
            }
            T[(int64_t)t * G + j] = make_float2((float)(ar * bc - ai * bs), (float)(ar * bs + ai * bc));
        }
        return;
    }
    for (int32_t i = tid; i < 4 * N; i += kBbTabThreads) ct[i] = cospi(0.5 * i / N);
    __syncthreads();
    {
        const int32_t r = tid / half, n = tid - r * half;
        const bool active = r < R;
        const double turns = dfh * (m + 1) * ct[2 * n + 1];  // df tau_n
        double step = R * turns;
        step -= rint(step);
        double os, oc;
        sincospi(2.0 * step, &os, &oc);
        double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0;  // at x_n and at -x_n
        for (; kb >= 0; kb -= sb) {
            __syncthreads();  // the previous stage's reads are done
            stage[tid] = y0;
            stage[tid + kBbTabThreads] = y1;  // past sb: not read
            __syncthreads();
            const int32_t top = min(per - 1, (nb - 1 - kb) / R);  // bins past the band are zeros
            if (kb > 0) {
                y0 = bin(kb - sb + tid);
                y1 = bin(kb - sb + tid + kBbTabThreads);
            }
            if (active) {
#pragma unroll 4
                for (int32_t q = top; q >= 0; --q) {
                    const double2 y = stage[q * R + r];
                    const double nr = fma(ar, oc, fma(-ai, os, y.x));
                    const double ni = fma(ar, os, fma(ai, oc, y.y));
                    const double mr = fma(br, oc, fma(bi, os, y.x));
                    const double mi = fma(br, -os, fma(bi, oc, y.y));
                    ar = nr;
                    ai = ni;
                    br = mr;
                    bi = mi;
                }
            }
        }
        double back = (r - kc) * turns;  // omega^(r - kc)
        back -= rint(back);
        double bs, bc;
        sincospi(2.0 * back, &bs, &bc);
        __syncthreads();
        // partial sums [node][r]: node n and, behind, node N - 1 - n
        if (active) {
            stage[n * R + r] = make_double2(ar * bc - ai * bs, ar * bs + ai * bc);
            stage[(half + n) * R + r] = make_double2(br * bc + bi * bs, bi * bc - br * bs);
        }
        __syncthreads();
        // up to eight lanes a node: every u-th partial sum, then a butterfly
        int32_t u = 8;
        while (u > 1 && 2 * half * u > kBbTabThreads) u >>= 1;
        for (int32_t e = tid; e < 2 * half * u; e += kBbTabThreads) {
            const int32_t q = e / u;
            double2 a = make_double2(0.0, 0.0);
            for (int32_t i = e % u; i < R; i += u) {
                a.x += stage[q * R + i].x;
                a.y += stage[q * R + i].y;
            }
            for (int32_t h = u / 2; h > 0; h >>= 1) {
                a.x += __shfl_xor(a.x, h);
                a.y += __shfl_xor(a.y, h);
            }
            if (e % u == 0) node[q < half ? q : N - 1 - (q - half)] = a;
        }
        __syncthreads();
    }
    // a_k = (2 - [k = 0]) / N sum_n Y_n cos(pi k (2 n + 1) / (2 N))
    for (int32_t e = tid; e < 2 * N; e += kBbTabThreads) {
        const int32_t k = e >> 1, part = e & 1;
        const double *val = reinterpret_cast<const double *>(node) + part;
        double a = 0.0;
        int32_t i = k;
        for (int32_t n = 0; n < N; ++n) {
            a = fma(val[2 * n], ct[i], a);
            i += 2 * k;
            if (i >= 4 * N) i -= 4 * N;
        }
        reinterpret_cast<double *>(coef)[e] = a * ((k ? 2.0 : 1.0) / N);
    }
    if (tid == 0) coef[N] = make_double2(0.0, 0.0);  // an odd N's last pair
    __syncthreads();
    float2 *Tc = T + (int64_t)t * G + (m + 1);  // the centre node
    for (int32_t j = tid; j <= m + 1; j += kBbTabThreads) {
        const double x = (double)j / (m + 1), y2 = 2.0 * (2.0 * x * x - 1.0);
        // the even terms sum a_2k T_k(y) and the odd ones sum a_{2k+1} T_{2k+1}(x), by
        // the same recurrence
        double e1r = 0.0, e1i = 0.0, e2r = 0.0, e2i = 0.0, o1r = 0.0, o1i = 0.0, o2r = 0.0, o2i = 0.0;
#pragma unroll 2
        for (int32_t k = (N - 1) / 2; k >= 0; --k) {
            const double2 ae = coef[2 * k], ao = coef[2 * k + 1];
            const double er = fma(y2, e1r, ae.x - e2r), ei = fma(y2, e1i, ae.y - e2i);
            const double dr = fma(y2, o1r, ao.x - o2r), di = fma(y2, o1i, ao.y - o2i);
            e2r = e1r;
            e2i = e1i;
            e1r = er;
            e1i = ei;
            o2r = o1r;
            o2i = o1i;
            o1r = dr;
            o1i = di;
        }
        const double er = fma(-0.5 * y2, e2r, e1r), ei = fma(-0.5 * y2, e2i, e1i);  // b_0 - y b_1
        const double dr = x * (o1r - o2r), di = x * (o1i - o2i);                     // b_0 T_1 - b_1 T_{-1}
        Tc[j] = make_float2((float)(er + dr), (float)(ei + di));
        Tc[-j] = make_float2((float)(er - dr), (float)(ei - di));
    }
}

// part[blockIdx.y][p] = sum over this chunk's segments t of
// gamma(t,p) Re[e^{2 pi i f_c tau} Y_t(tau)], Y_t from its table by 4-point
// Lagrange interpolation; a seed with |tau| beyond the grid's bound (or not a
// number) makes its pixel's sum NaN.  With v (GB), gpart[blockIdx.y][p] =
// sum_t v[t] gamma(t,p)^2 as band_gamma_kernel sums it (same chunks, same
// order, same arithmetic), from the gamma values this pass reads anyway.
template <bool GB>
__global__ __launch_bounds__(256) void bb_map_kernel(const float *__restrict__ gamma, const double *__restrict__ tau,
                                                     int32_t nt, int32_t npix, const float2 *__restrict__ T,
                                                     int32_t G, int32_t m, double h, double bound, double fc,
                                                     int32_t per, double *__restrict__ part,
                                                     const double *__restrict__ v, double *__restrict__ gpart)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    double acc = 0.0, gacc = 0.0;  // sums of the chunk's runs so far
    const double inv_h = 1.0 / h, origin = (double)(m + 1);
    const double jmax = (double)(2 * m);
    bool bad = false;
    // segments kBbBatch at a time: their seed loads, then their table reads, are
    // issued together (segments past t1 repeat t1 - 1 with weight zero; no
    // branch, so that the compiler keeps the loads ahead of the arithmetic)
    for (int sl = 0; sl < kBandSlices; ++sl) {
        const BandSlice run = band_slice(blockIdx.y, sl, per, nt);
        const int32_t t1 = run.end;
        double sum = 0.0, gsum = 0.0;
        for (int32_t tq = run.begin; tq < t1; tq += kBbBatch) {
            double ta[kBbBatch];
            float g[kBbBatch];
#pragma unroll
            for (int e = 0; e < kBbBatch; ++e) {
                const int64_t o = (int64_t)min(tq + e, t1 - 1) * npix + p;
                ta[e] = tau[o];
                g[e] = gamma[o];
            }
            float2 a[kBbBatch][4];
            float x[kBbBatch];
#pragma unroll
            for (int e = 0; e < kBbBatch; ++e) {
                const double u = fma(ta[e], inv_h, origin);
                const double jd = fmin(fmax(floor(u), 1.0), jmax);  // NaN and out-of-range delays stay inside the table
                x[e] = (float)(u - jd);
                const float2 *row = T + (int64_t)min(tq + e, t1 - 1) * G + ((int32_t)jd - 1);
#pragma unroll
                for (int i = 0; i < 4; ++i) a[e][i] = row[i];
            }
#pragma unroll
            for (int e = 0; e < kBbBatch; ++e) {
                const bool valid = tq + e < t1;
                bad |= valid && !(fabs(ta[e]) <= bound);
                // Lagrange weights of the nodes at -1, 0, 1, 2
                const float xe = x[e], xp = xe + 1.0f, xm = xe - 1.0f, xm2 = xe - 2.0f;
                const float l0 = -(1.0f / 6.0f) * xe * xm * xm2;
                const float l1 = 0.5f * xp * xm * xm2;
                const float l2 = -0.5f * xp * xe * xm2;
                const float l3 = (1.0f / 6.0f) * xp * xe * xm;
                const float yr = fmaf(l0, a[e][0].x, fmaf(l1, a[e][1].x, fmaf(l2, a[e][2].x, l3 * a[e][3].x)));
                const float yi = fmaf(l0, a[e][0].y, fmaf(l1, a[e][1].y, fmaf(l2, a[e][2].y, l3 * a[e][3].y)));
                // carrier e^{2 pi i f_c tau}: the phase reduced in float64
                const double turns = fc * ta[e];
                const float r = (float)(turns - rint(turns));
                float sn, cs;
                sincospif(2.0f * r, &sn, &cs);
                sum = fma(valid ? (double)g[e] : 0.0, (double)fmaf(cs, yr, -sn * yi), sum);
                if (GB) {
                    const double gd = (double)g[e];
                    const double ga = fma(v[min(tq + e, t1 - 1)], gd * gd, gsum);
                    gsum = valid ? ga : gsum;
                }
            }
        }
        acc += sum;
        gacc += gsum;
    }
    part[(int64_t)blockIdx.y * npix + p] = bad ? (double)__builtin_nanf("") : acc;
    if (GB) gpart[(int64_t)blockIdx.y * npix + p] = gacc;
}

// A pixel pair's terms.  Antipodal seeds have gamma(t,pB) = gamma(t,p) and
// tau(t,pB) = -tau(t,p), and the delay grid is symmetric about zero, so one
// read of p's seeds serves both pixels: with u = |tau| / h, jd = floor(u) and
// x = u - jd, the nodes of +|tau| are jd - 1 .. jd + 2 counted from the centre,
// those of -|tau| their mirror images with the same weights, and the carriers
// are conjugate.
struct BbAt {
    int32_t j;  // jd, in [0, m - 1] whatever the delay (NaN included)
    float x;
    float cs, sn;  // carrier e^{2 pi i f_c |tau|}
};

// What bb_at needs of the grid and the carrier.
struct BbScale {
    double inv_h, fc4;  // intervals per second, quarter turns per second
    int32_t jmax;       // the last interval
    // intervals or quarter turns beyond the fixed-point forms (2^20 intervals,
    // 2^21 quarter turns: at 40 ms frequencies above 1.2e7 Hz)
    int32_t far;
};

// Cell and phase in fixed point: adding 2^20 to u leaves its integer part in the
// high word and its fraction, to 2^-32, in the low one; adding 1.5 2^22 to the
// quarter turns leaves the quadrant in the low word's two top bits and the
// fraction, to 2^-30 (7e-10 rad at most), below.  One float64 operation each
// where product, floor or rint, difference and conversions took six and nine
// (a full day, nside 128, 4096 bins: the call 296 -> 286 us).
__device__ __forceinline__ BbAt bb_at(double ta, const BbScale &c)
{
    BbAt r;
    const double at = fabs(ta);
    uint32_t turn;  // the phase in units of 2^-30 quarter turns, mod 4
    if (!c.far) {
        const uint64_t b = (uint64_t)__double_as_longlong(fma(at, c.inv_h, 1048576.0));
        const int32_t j = (int32_t)(b >> 32) & 0xfffff;
        r.j = min(j, c.jmax);
        r.x = fmaf((float)(uint32_t)b, 1.0f / 4294967296.0f, (float)(j - r.j));
        turn = (uint32_t)__double_as_longlong(fma(c.fc4, at, 6291456.0));
    } else {
        const double u = at * c.inv_h, jd = fmin(floor(u), (double)c.jmax);
        r.j = (int32_t)jd;
        r.x = (float)(u - jd);
        const double x4 = c.fc4 * at, whole = 4.0 * rint(0.25 * x4);
        turn = (uint32_t)__double_as_longlong(fma(c.fc4, at, -whole) + 6291456.0);
    }
    // to the nearest quarter turn; sine and cosine by their series on |theta| <=
    // pi / 4 (truncation below 2e-9), turned by the quadrant.  (A half-angle
    // form without the quadrant was 4 % faster, but its rounding took the maps'
    // error from 8.4e-8 to 1.4e-7.)
    const uint32_t k = (turn + 0x20000000u) >> 30;
    const float th = (float)(int32_t)(turn << 2) * (1.57079632679489662f / 4294967296.0f), t2 = th * th;
    const float s =
        th * fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, 2.75573192e-6f, -1.98412698e-4f), 8.33333333e-3f), -1.66666667e-1f),
                  1.0f);
    const float c0 =
        fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, -2.75573192e-7f, 2.48015873e-5f), -1.38888889e-3f),
                               4.16666667e-2f), -0.5f), 1.0f);
    const float cr = (k & 1) ? s : c0, sr = (k & 1) ? c0 : s;
    r.cs = __uint_as_float(__float_as_uint(cr) ^ (((k + 1) & 2) << 30));
    r.sn = __uint_as_float(__float_as_uint(sr) ^ ((k & 2) << 30));
    return r;
}

// Re[e^{2 pi i f_c tau} Y(tau)] at tau and at -tau (x, y) from the four nodes
// (Y(+tau_j), Y(-tau_j)) around |tau|.
__device__ __forceinline__ float2 bb_pair_value(const float4 (&e)[4], const BbAt &at, bool negative)
{
    // Lagrange weights of the nodes at -1, 0, 1, 2
    const float x = at.x, xp = x + 1.0f, xm = x - 1.0f, xm2 = x - 2.0f;
    const float outer = (1.0f / 6.0f) * x * xm, inner = 0.5f * xp * xm2;
    const float l0 = -outer * xm2, l1 = inner * xm, l2 = -inner * x, l3 = outer * xp;
    const float pr = fmaf(l0, e[0].x, fmaf(l1, e[1].x, fmaf(l2, e[2].x, l3 * e[3].x)));
    const float pi = fmaf(l0, e[0].y, fmaf(l1, e[1].y, fmaf(l2, e[2].y, l3 * e[3].y)));
    const float mr = fmaf(l0, e[0].z, fmaf(l1, e[1].z, fmaf(l2, e[2].z, l3 * e[3].z)));
    const float mi = fmaf(l0, e[0].w, fmaf(l1, e[1].w, fmaf(l2, e[2].w, l3 * e[3].w)));
    const float p = fmaf(at.cs, pr, -at.sn * pi), q = fmaf(at.cs, mr, at.sn * mi);
    return negative ? make_float2(q, p) : make_float2(p, q);
}

// The chunk's sums of a pixel pair.  The antipodal promise is spot-checked
// (flags, one per part of the check): a failed check makes both maps NaN.
template <bool GB>
__device__ __forceinline__ void bb_store_pair(int64_t p, int64_t npix, int64_t nside, const double *__restrict__ flags,
                                              bool bad, double a, double b, double g, double *__restrict__ part,
                                              double *__restrict__ gpart)
{
    bool broken = false;
    for (int i = 0; i < kSymParts; ++i) broken |= flags[i] != 0.0;
    const double nan = (double)__builtin_nanf("");
    const int64_t pB = antipode_north(ring_of_north(p, nside), npix);
    double *row = part + (int64_t)blockIdx.y * npix;
    row[p] = bad || broken ? nan : a;
    row[pB] = bad || broken ? nan : b;
    if (GB) {
        double *grow = gpart + (int64_t)blockIdx.y * npix;
        grow[p] = broken ? nan : g;
        grow[pB] = broken ? nan : g;
    }
}

// Few pixels: the four waves of a workgroup take a run each of the chunk's
// segments (band_slice) for the same 64 pixel pairs, reading the tables where
// they are; bound by the latency of the segments in series, hence the split.
template <bool GB>
__global__ __launch_bounds__(256) void bb_map_pair_kernel(const float *__restrict__ gamma,
                                                          const double *__restrict__ tau, int32_t nt, int32_t npix,
                                                          int64_t nside, const float2 *__restrict__ T, int32_t G,
                                                          int32_t m, double bound, BbScale scale, int32_t per,
                                                          const double *__restrict__ flags, double *__restrict__ part,
                                                          const double *__restrict__ v, double *__restrict__ gpart)
{
    __shared__ double red[3][kBandSlices][64];
    __shared__ int redbad[kBandSlices][64];
    const int lane = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int64_t p = (int64_t)blockIdx.x * 64 + lane, npairs = npix / 2, pc = p < npairs ? p : npairs - 1;
    const BandSlice run = band_slice(blockIdx.y, sl, per, nt);
    double accA = 0.0, accB = 0.0, gacc = 0.0;
    bool bad = false;
    for (int32_t tq = run.begin; tq < run.end; tq += kBbRunBatch) {
        double ta[kBbRunBatch];
        float g[kBbRunBatch];
#pragma unroll
        for (int e = 0; e < kBbRunBatch; ++e) {
            const int64_t o = (int64_t)min(tq + e, run.end - 1) * npix + pc;
            ta[e] = tau[o];
            g[e] = gamma[o];
        }
        BbAt at[kBbRunBatch];
        float4 n[kBbRunBatch][4];
#pragma unroll
        for (int e = 0; e < kBbRunBatch; ++e) {
            at[e] = bb_at(ta[e], scale);
            const float2 *row = T + (int64_t)min(tq + e, run.end - 1) * G + (m + 1);  // the centre node
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float2 a = row[at[e].j - 1 + i], b = row[-(at[e].j - 1 + i)];
                n[e][i] = make_float4(a.x, a.y, b.x, b.y);
            }
        }
#pragma unroll
        for (int e = 0; e < kBbRunBatch; ++e) {
            const bool valid = e == 0 || tq + e < run.end;  // a segment past the run repeats its last
            bad |= !(fabs(ta[e]) <= bound);
            const float2 val = bb_pair_value(n[e], at[e], ta[e] < 0.0);
            const double wg = valid ? (double)g[e] : 0.0;
            accA = fma(wg, (double)val.x, accA);
            accB = fma(wg, (double)val.y, accB);
            if (GB) {  // (not a product with zero: the weight or the seed may be infinite)
                const double gd = (double)g[e], ga = fma(v[min(tq + e, run.end - 1)], gd * gd, gacc);
                gacc = valid ? ga : gacc;
            }
        }
    }
    red[0][sl][lane] = accA;
    red[1][sl][lane] = accB;
    red[2][sl][lane] = gacc;
    redbad[sl][lane] = bad;
    __syncthreads();
    if (sl != 0 || p >= npairs) return;
#pragma unroll
    for (int k = 1; k < kBandSlices; ++k) {
        accA += red[0][k][lane];
        accB += red[1][k][lane];
        gacc += red[2][k][lane];
        bad |= redbad[k][lane] != 0;
    }
    bb_store_pair<GB>(p, npix, nside, flags, bad, accA, accB, gacc, part, gpart);
}

// Many pixels: one pixel pair a thread over the chunk's runs in turn, the
// segments' tables staged through LDS, kBbBatch at a time and double-buffered,
// as (Y(+tau_j), Y(-tau_j)) per node counted from the centre (index j + 1 for
// j = -1 .. m + 1), so a pair's four nodes are four 16-byte reads.  K: staged
// entries per thread.  Bound by the seeds' 12 bytes a pair and segment, with
// ~85 vector instructions close behind.  Full day, nside 128, 4096 bins, AB: the
// pass ~230 us (221 us at the copy rate), 348 us with the nodes read from global
// memory by each pair.
constexpr int kBbMapThreads = 512;
constexpr int64_t kBbLdsPairs = 6144;

template <bool GB, int K>
__global__ __launch_bounds__(kBbMapThreads) void bb_map_pair_lds_kernel(
    const float *__restrict__ gamma, const double *__restrict__ tau, int32_t nt, int32_t npix, int64_t nside,
    const float2 *__restrict__ T, int32_t G, int32_t m, double bound, BbScale scale, int32_t per,
    const double *__restrict__ flags, double *__restrict__ part, const double *__restrict__ v,
    double *__restrict__ gpart)
{
    extern __shared__ float4 tab[];  // [2][kBbBatch][m + 3]
    const int32_t E = m + 3;
    const int64_t p = (int64_t)blockIdx.x * kBbMapThreads + threadIdx.x;
    const int64_t npairs = npix / 2, pc = p < npairs ? p : npairs - 1;
    double totA = 0.0, totB = 0.0, totG = 0.0, accA = 0.0, accB = 0.0, gacc = 0.0;
    bool bad = false;

    // the batches of the chunk's runs, in order (uniform over the workgroup)
    int sl = 0;
    BandSlice run = band_slice(blockIdx.y, 0, per, nt);
    int32_t tq = run.begin;
    auto settle = [&]() {  // to the next batch; false past the last
        while (tq >= run.end) {
            if (++sl >= kBandSlices) return false;
            run = band_slice(blockIdx.y, sl, per, nt);
            tq = run.begin;
        }
        return true;
    };
    double ta[kBbBatch];
    float g[kBbBatch];
    float4 st[K];
    auto fetch = [&]() {
#pragma unroll
        for (int e = 0; e < kBbBatch; ++e) {
            const int64_t o = (int64_t)min(tq + e, run.end - 1) * npix + pc;
            ta[e] = tau[o];
            g[e] = gamma[o];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t i = min((int32_t)threadIdx.x + k * kBbMapThreads, kBbBatch * E - 1);
            const int32_t e = i >= E ? 1 : 0, j = i - e * E - 1;
            const float2 *row = T + (int64_t)min(tq + e, run.end - 1) * G + (m + 1);
            const float2 a = row[j], b = row[-j];
            st[k] = make_float4(a.x, a.y, b.x, b.y);
        }
    };
    static_assert(kBbBatch == 2, "the staging index splits two segments");
    auto put = [&](float4 *buf) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t i = (int32_t)threadIdx.x + k * kBbMapThreads;
            if (i < kBbBatch * E) buf[i] = st[k];
        }
    };
    bool more = settle();
    if (more) {
        fetch();
        put(tab);
    }
    __syncthreads();
    int cur = 0;
    while (more) {
        double tc[kBbBatch];
        float gc[kBbBatch];
#pragma unroll
        for (int e = 0; e < kBbBatch; ++e) {
            tc[e] = ta[e];
            gc[e] = g[e];
        }
        const int32_t t0 = tq, t1 = run.end;
        const int sl0 = sl;
        tq += kBbBatch;
        more = settle();
        if (more) fetch();
        const float4 *buf = tab + cur * kBbBatch * E;
#pragma unroll
        for (int e = 0; e < kBbBatch; ++e) {
            const bool valid = e == 0 || t0 + e < t1;  // a segment past the run repeats its last
            const BbAt at = bb_at(tc[e], scale);
            float4 n[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) n[i] = buf[e * E + at.j + i];
            bad |= !(fabs(tc[e]) <= bound);
            const float2 val = bb_pair_value(n, at, tc[e] < 0.0);
            const double gd = (double)gc[e], wg = valid ? gd : 0.0;
            accA = fma(wg, (double)val.x, accA);
            accB = fma(wg, (double)val.y, accB);
            if (GB) {  // (not a product with zero: the weight or the seed may be infinite)
                const double ga = fma(v[min(t0 + e, t1 - 1)], gd * gd, gacc);
                gacc = valid ? ga : gacc;
            }
        }
        if (!more || sl != sl0) {  // the run is done
            totA += accA;
            totB += accB;
            totG += gacc;
            accA = accB = gacc = 0.0;
        }
        cur ^= 1;
        if (more) put(tab + cur * kBbBatch * E);
        __syncthreads();
    }
    if (p >= npairs) return;
    bb_store_pair<GB>(p, npix, nside, flags, bad, totA, totB, totG, part, gpart);
}

template <bool GB>
static hipError_t launch_bb_map_pair(const float *gamma, const double *tau, int32_t nt, int32_t npix, int64_t nside,
                                     const float2 *T, const BbGrid &g, double fc, int32_t nchunks, int32_t per,
                                     const double *flags, double *part, const double *v, double *gpart, hipStream_t s)
{
    const int64_t npairs = npix / 2;
    BbScale scale;
    scale.inv_h = 1.0 / g.h;
    scale.fc4 = 4.0 * fc;
    scale.jmax = g.m - 1;
    scale.far = g.m > (1 << 20) - 2 || !(std::fabs(scale.fc4) * g.bound < 2097152.0 - 1.0);
    const int32_t entries = kBbBatch * (g.m + 3), k = (entries + kBbMapThreads - 1) / kBbMapThreads;
    // The LDS form from kBbLdsPairs pixel pairs on, while the tables fit in 64 KB
    // (at most 1021 intervals of |tau|).  Measured, full day, AB, 1531 bins, call
    // (LDS / split form): nside 8 44.2 / 35.1, 16 45.8 / 37.6, 32 54.6 / 54.8, 64
    // 105 / 143, 128 331 / 492 us; AC alike.
    if (npairs >= kBbLdsPairs && k <= 4) {
        const dim3 grid((unsigned)((npairs + kBbMapThreads - 1) / kBbMapThreads), (unsigned)nchunks);
        const size_t lds = 2 * (size_t)entries * sizeof(float4);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, grid, dim3(kBbMapThreads), lds, s, gamma, tau, nt, npix, nside, T, g.G, g.m,
                               g.bound, scale, per, flags, part, v, gpart);
        };
        if (k == 1)
            go(bb_map_pair_lds_kernel<GB, 1>);
        else if (k == 2)
            go(bb_map_pair_lds_kernel<GB, 2>);
        else
            go(bb_map_pair_lds_kernel<GB, 4>);
    } else {
        hipLaunchKernelGGL(bb_map_pair_kernel<GB>, dim3((unsigned)((npairs + 63) / 64), (unsigned)nchunks), dim3(256),
                           0, s, gamma, tau, nt, npix, nside, T, g.G, g.m, g.bound, scale, per, flags, part, v,
                           gpart);
    }
    return hipGetLastError();
}

hipError_t launch_broadband_table_maps(const float *C, const float *w, int64_t ldc, int32_t nt, int32_t klo,
                                       int32_t khi, double f0, double df, int64_t k0, const float *H,
                                       const float *gamma, const double *tau, int32_t npix, int64_t nside,
                                       const BbGrid &g, float *Xbb, float *Gbb, void *work, hipStream_t s)
{
    const int32_t nb = khi - klo;
    const BbLayout L = bb_layout(nt, npix, g);
    char *ws = reinterpret_cast<char *>(work);
    double *v = reinterpret_cast<double *>(ws + L.gam), *gpart = v + nt;
    const int32_t nchunks = band_gamma_chunks(npix), per = (nt + nchunks - 1) / nchunks;
    if (!Xbb) {  // Gbb alone: the weight-side kernels by themselves
        return launch_band_gamma(w, ldc, nt, H, klo, khi, gamma, npix, v, Gbb, s);
    }
    float2 *T = reinterpret_cast<float2 *>(ws + L.t);
    double *part = reinterpret_cast<double *>(ws + L.part);
    double *flags = nside > 0 ? reinterpret_cast<double *>(ws + L.flags) : nullptr;
    const int32_t N = bb_cheb_nodes(nb, nt, g);
    hipError_t e;
    if (N > 0 || (nb <= kBbStage && g.G <= kBbPrepNodes)) {
        hipLaunchKernelGGL(bb_prep_kernel, dim3((unsigned)(nt + (flags ? kSymParts : 0))), dim3(kBbTabThreads),
                           (8 * N + 2) * sizeof(double), s, C, w, ldc, klo, nb, g.G, g.m, df * g.h, N, T, H,
                           Gbb ? v : (double *)nullptr, gamma, tau, nt, (int64_t)npix, nside, flags);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    } else {  // many nodes: one wave per segment and 64 of them
        hipLaunchKernelGGL(bb_table_kernel, dim3((unsigned)nt, (unsigned)((g.G + kBbNodes - 1) / kBbNodes)),
                           dim3(kBbNodes), 0, s, C, w, ldc, klo, nb, g.G, g.m, df * g.h, T);
        e = hipGetLastError();
        if (e == hipSuccess && Gbb) e = launch_band_weights(w, ldc, nt, H, klo, khi, v, s);
        if (e == hipSuccess && flags) e = launch_antipodal_check(gamma, tau, nt, npix, nside, flags, s);
        if (e != hipSuccess) return e;
    }
    // the band's centre: absolute bin k0 + klo + (nb - 1) / 2
    const double fc = f0 + ((double)(k0 + klo) + 0.5 * (nb - 1)) * df;
    if (nside > 0) {  // antipodal seeds: each thread a pixel pair
        e = Gbb ? launch_bb_map_pair<true>(gamma, tau, nt, npix, nside, T, g, fc, nchunks, per, flags, part, v, gpart, s)
                : launch_bb_map_pair<false>(gamma, tau, nt, npix, nside, T, g, fc, nchunks, per, flags, part, nullptr,
                                            nullptr, s);
        if (e != hipSuccess) return e;
        return launch_band_partial_finish(part, nchunks, npix, Xbb, s, gpart, Gbb);
    }
    const dim3 grid((unsigned)((npix + 255) / 256), (unsigned)nchunks);
    if (Gbb)
        hipLaunchKernelGGL(bb_map_kernel<true>, grid, dim3(256), 0, s, gamma, tau, nt, npix, (const float2 *)T, g.G,
                           g.m, g.h, g.bound, fc, per, part, (const double *)v, gpart);
    else
        hipLaunchKernelGGL(bb_map_kernel<false>, grid, dim3(256), 0, s, gamma, tau, nt, npix, (const float2 *)T, g.G,
                           g.m, g.h, g.bound, fc, per, part, (const double *)nullptr, (double *)nullptr);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_band_partial_finish(part, nchunks, npix, Xbb, s, gpart, Gbb);
}


}  // namespace sgwb
