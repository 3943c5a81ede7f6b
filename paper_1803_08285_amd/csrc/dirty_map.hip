// Narrowband dirty map X(k,p) = sum_t w(t,k) gamma(t,p) Re[C(t,k) e^{2 pi i f_k tau(t,p)}]
// (Eq. eq_dirtymap split per frequency bin as in Eq. eq:narrowband) on gfx950.
//
// Work decomposition
//   * A wave owns 64 pixel columns (one per lane) and one strip of S consecutive
//     frequency bins that starts at an absolute bin k = 0 mod S (S = 64 in
//     float32, 32 in float64).
//   * Short days: a workgroup's four waves walk the whole day for neighbouring
//     columns, and each writes its sums.  Longer days (dm_slices) are split: four
//     or eight waves take a share of the segments each (consecutive ones) for the
//     same columns, so that a small map still fills the chip; their sums meet in
//     LDS and are added in wave order.
//   * The weighted CSD y(t,k) = w(t,k) C(t,k) of the strip is staged in LDS, WTC
//     segments at a time per workgroup, or XTC per wave of a split day with the
//     next ones' loads in flight; every lane reads the same y (LDS broadcast).
//   * Per (t, pixel) the phase is reduced once per strip in float64,
//     frac(f_anchor tau), and turned into the anchor phasor z = gamma e^{i phi};
//     the remaining S-1 bins advance z by the rotor 1 + eps = e^{i 2 pi df tau},
//     z <- z + z eps (four FMAs), so no transcendental is evaluated per term.
//   * Antipodal pairing (HEALPix RING seeds from the geometry kernel): the
//     antipode p' of p has gamma(t,p') = gamma(t,p) and tau(t,p') = -tau(t,p),
//     so its phasor is conj(z).  With a = sum y_re z_re and b = sum y_im z_im,
//     X(k,p) = a - b and X(k,p') = a + b: one rotation serves two pixels.
//   * On request the strip's broadband sums (float64) are written beside the
//     map, from the values in hand.
//   * Fixed summation order over t, no atomics: bitwise reproducible, and the
//     absolute anchor grid makes a sub-band bitwise equal to the full band.
// Bound by the vector instructions: six FMAs per segment, bin and pixel pair
// (at one per lane and cycle and 64 lanes a compute unit, 1.5 of the 1.72 ms
// below); in float64 also by the LDS broadcasts, 16 bytes a bin; a day of a few
// segments by the map's write (one segment, nside 32, 6823 bins, 335 MB: 69 us).
// Measured, split against whole days: 240 segments, nside 32, 6823 bins of 0.25 Hz
// 1.72 against 2.04 ms; nside 8, 1024 bins 44 against 302 us; float64, nside 16,
// 1001 bins 141 against 263 us.
#include <algorithm>
#include <type_traits>

#include "sgwb_internal.h"

namespace sgwb {

template <typename T>
struct Cplx;
template <>
struct Cplx<float> {
    using type = float2;
};
template <>
struct Cplx<double> {
    using type = double2;
};

template <typename T>
struct StripTraits;
template <>
struct StripTraits<float> {
    static constexpr int S = 64;     // bins per anchor strip
    static constexpr int WTC = 32;   // segments per LDS stage of a workgroup (whole days)
    static constexpr int XTC = 8;    // and of a wave (split days)
    static constexpr int SLAB = 16;  // bins per round of the final sums
};
template <>
struct StripTraits<double> {
    static constexpr int S = 32;
    static constexpr int WTC = 16;
    static constexpr int XTC = 4;
    static constexpr int SLAB = 8;
};

constexpr int kDmCols = 64;       // pixel columns per wave
constexpr int kDmWaveLds = 8192;  // of a split day's wave: its stage, then its share of a round of the final sums

// Segment slices of a map: one (whole days), four or eight.  They depend on the
// segments and the pixel columns alone, so that a sub-band's rows are the whole
// band's.  Slices fill the chip where columns and bins are few, but their final
// sums cost the same for every day: some 85 (four) and 195 us (eight) for nside 32 and
// 6823 bins.  So a day is split where that was no slower for the widest band,
// measured at 1 to 6823 bins (paired, 64 / 6823 bins, whole / four / eight slices):
// nside 8, 16 segments 27/12/11 and 31/25/28 us; nside 16, 32 segments 46/16/12 and
// 101/92/113, 60 segments 80/24/16 and 175/139/165; nside 32, 32 segments 46/17/12
// and 305/319/417, 60 segments 80/24/17 and 533/490/609, 100 segments 128/35/23
// and 862/747/860; nside 64, 60 segments 84/29/33 and 1983/1982/2407.  Without
// pairs whole days hold more waves a unit: nside 32, 60 segments 751/760/855, 240
// segments 2961/2909/3092; nside 64, 100 segments of 1024 bins 748/758/818, 160
// 1181/1174/1231.  float64 gains earlier and takes the same rule.
inline int dm_slices(int32_t nt, int64_t ncol, bool pair)
{
    struct Row {
        int64_t cols;
        int32_t four, eight;  // segments from which the day is split
    };
    constexpr int32_t kNever = 0x7fffffff;
    const Row rows[] = {
        {1024, 16, 16},
        {4096, 32, 60},
        {16384, pair ? 48 : 80, pair ? 100 : kNever},
        {0x7fffffffffff, pair ? 80 : 160, kNever},
    };
    for (const Row &r : rows)
        if (ncol <= r.cols) return nt >= r.eight ? 8 : nt >= r.four ? 4 : 1;
    return 1;
}

// f(std::integral_constant<int, slices>)
template <typename F>
inline void dm_with_slices(int slices, const F &f)
{
    if (slices == 1) f(std::integral_constant<int, 1>());
    else if (slices == 4) f(std::integral_constant<int, 4>());
    else f(std::integral_constant<int, 8>());
}

// Waves per workgroup: four, or one a slice.
constexpr int dm_waves(int slices) { return slices > 4 ? slices : 4; }
// Its LDS: the whole-day tile's stage, or the waves' stages and the final sums.
template <typename T>
constexpr int dm_lds(int slices)
{
    return slices > 1 ? kDmWaveLds * slices
                      : StripTraits<T>::WTC * StripTraits<T>::S * (int)sizeof(typename Cplx<T>::type);
}
// Rotor 1 + eps = e^{i d} for the per-bin phase step d = 2 pi df tau:
// eps_re = cos d - 1, eps_im = sin d, each with full relative precision.
__device__ inline void rotor(float d, float *er, float *ei)
{
    const float d2 = d * d;
    if (fabsf(d) <= 0.25f) {
        // Taylor series; truncation error below 2e-9 relative for |d| <= 0.25.
        *er = -0.5f * d2 * (1.0f - d2 * (1.0f / 12.0f) * (1.0f - d2 * (1.0f / 30.0f)));
        *ei = d * (1.0f - d2 * (1.0f / 6.0f) * (1.0f - d2 * (1.0f / 20.0f)));
    } else {
        float sh, ch, s, c;
        sincosf(0.5f * d, &sh, &ch);
        sincosf(d, &s, &c);
        *er = -2.0f * sh * sh;
        *ei = s;
    }
}
__device__ inline void rotor(double d, double *er, double *ei)
{
    const double d2 = d * d;
    if (fabs(d) <= 0.25) {
        // Taylor series; the dropped terms are below 1e-18 relative
        *er = -0.5 * d2 * fma(d2, fma(d2, fma(d2, fma(d2, fma(d2, -1.0 / 239500800, 1.0 / 1814400), -1.0 / 20160),
                                              1.0 / 360), -1.0 / 12), 1.0);
        *ei = d * fma(d2, fma(d2, fma(d2, fma(d2, fma(d2, fma(d2, 1.0 / 6227020800, -1.0 / 39916800), 1.0 / 362880),
                                              -1.0 / 5040), 1.0 / 120), -1.0 / 6), 1.0);
    } else {
        double sh, ch, s, c;
        sincos(0.5 * d, &sh, &ch);
        sincos(d, &s, &c);
        *er = -2.0 * sh * sh;
        *ei = s;
    }
}

// Anchor phasor gamma e^{2 pi i x} for x = f tau cycles, given as x4 = 4 x.
// float64 reduction to the nearest quarter turn q (x4 - q in [-1/2, 1/2]),
// Taylor series for sin and cos on |theta| <= pi/4 (truncation below 3e-8),
// then a rotation by i^q.
__device__ inline void anchor4(float g, double x4, float *zr, float *zi)
{
    const double q = rint(x4);
    const float th = (float)(x4 - q) * 1.57079632679489662f;
    const int m = (int)q & 3;
    const float t2 = th * th;
    const float s =
        th * fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, 2.75573192e-6f, -1.98412698e-4f), 8.33333333e-3f),
                           -1.66666667e-1f),
                  1.0f);
    const float c =
        fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, 2.48015873e-5f, -1.38888889e-3f), 4.16666667e-2f), -0.5f), 1.0f);
    float cr = (m & 1) ? -s : c;
    float ci = (m & 1) ? c : s;
    if (m & 2) {
        cr = -cr;
        ci = -ci;
    }
    *zr = g * cr;
    *zi = g * ci;
}
__device__ inline void anchor4(double g, double x4, double *zr, double *zi)
{
    double x = 0.25 * x4;
    x -= rint(x);
    double s, c;
    sincospi(2.0 * x, &s, &c);
    *zr = g * c;
    *zi = g * s;
}

// Global-memory accesses.  The multi-job kernel reads its pointers out of a
// job table, so the compiler cannot tell them from LDS pointers and would use
// flat instructions, which count against the LDS counter as well; through
// these every access is a plain global one.
template <typename T>
__device__ inline __attribute__((address_space(1))) T *gmem(T *p)
{
    return (__attribute__((address_space(1))) T *)p;
}
template <typename C2>
__device__ inline C2 gload_c(const C2 *p, int64_t i)
{
    typedef decltype(p->x) R;
    typedef R v2 __attribute__((ext_vector_type(2)));
    const v2 v = ((const __attribute__((address_space(1))) v2 *)p)[i];
    C2 r;
    r.x = v.x;
    r.y = v.y;
    return r;
}

// Orders a wave's LDS accesses among its own lanes: they run in order, so only
// the compiler has to keep them so.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// z advanced by a bin: z <- z (1 + eps), and the bin's terms y z.
template <typename T, bool PAIR>
__device__ __forceinline__ void add_bin(T yr, T yi, T &zr, T &zi, T er, T ei, T &a, T &b)
{
    a = fma(yr, zr, a);
    if (PAIR) b = fma(yi, zi, b);
    else a = fma(-yi, zi, a);
    T nr = fma(zr, er, zr);
    nr = fma(-zi, ei, nr);
    T ni = fma(zi, er, zi);
    ni = fma(zr, ei, ni);
    zr = nr;
    zi = ni;
}

// One output of a column's strip (column c of the band, pixels col and colB).
template <typename T, bool PAIR>
__device__ __forceinline__ void put_bin(const MapArgs &a, T *__restrict__ X, int64_t c, int64_t col, int64_t colB,
                                        T va, T vb)
{
    auto row = gmem(X + c * (int64_t)a.npix);
    const T xa = va - vb, xb = va + vb;
    row[col] = a.accumulate ? row[col] + xa : xa;
    if (PAIR) row[colB] = a.accumulate ? row[colB] + xb : xb;
}

// The strip's bins [lo, hi) that lie in the band of the broadband sums, and a bin's
// share of them.
template <int S>
struct BandBins {
    int lo, hi;
    __device__ __forceinline__ BandBins(const MapArgs &a, int64_t c0)
        : lo((int)min(max((int64_t)a.band_lo - c0, (int64_t)0), (int64_t)S)),
          hi((int)min(max((int64_t)a.band_hi - c0, (int64_t)0), (int64_t)S))
    {
    }
    template <typename T>
    __device__ __forceinline__ void add(int j, T va, T vb, double &sa, double &sb) const
    {
        if (j < lo || j >= hi) return;
        sa += (double)(va - vb);
        sb += (double)(va + vb);
    }
};

// One tile of a map whose day is not split: 64 NW pixel columns (the coltile-th
// block) x one S-bin strip (absolute index strip), the strip's y staged by the
// whole workgroup of NW waves.
template <typename T, bool PAIR, int NW>
__device__ inline void dirty_map_whole_tile(const MapArgs &a, int64_t strip, int64_t coltile,
                                            const typename Cplx<T>::type *__restrict__ C, const T *__restrict__ w,
                                            const T *__restrict__ gamma, const double *__restrict__ tau,
                                            T *__restrict__ X, double *__restrict__ band_row, char *lds)
{
    using C2 = typename Cplx<T>::type;
    constexpr int S = StripTraits<T>::S;
    constexpr int WTC = StripTraits<T>::WTC;
    C2(*ys)[S] = reinterpret_cast<C2(*)[S]>(lds);

    const int64_t ncol = PAIR ? (int64_t)a.npix / 2 : (int64_t)a.npix;
    const int64_t col = coltile * (NW * kDmCols) + threadIdx.x;
    const bool active = col < ncol;
    const int64_t kabs0 = strip * S;                          // absolute first bin of the strip
    const int64_t c0 = kabs0 - a.k0;                           // its column in C (may be < 0)
    const double fa4 = 4.0 * (a.f0 + (double)kabs0 * a.df);   // anchor frequency, quarter turns
    const double two_pi_df = kTwoPi * a.df;

    T acc_a[S], acc_b[PAIR ? S : 1];
#pragma unroll
    for (int j = 0; j < S; ++j) acc_a[j] = T(0);
#pragma unroll
    for (int j = 0; j < (PAIR ? S : 1); ++j) acc_b[j] = T(0);

    const int64_t pcol = active ? col : 0;
    for (int tc = 0; tc < a.nt; tc += WTC) {
        const int tn = min(WTC, a.nt - tc);
        __syncthreads();
        for (int e = threadIdx.x; e < WTC * S; e += NW * 64) {
            const int tt = e / S, kk = e % S;
            const int64_t c = c0 + kk;
            C2 y;
            y.x = T(0);
            y.y = T(0);
            if (tt < tn && c >= 0 && c < a.nf) {
                const int64_t off = (int64_t)(tc + tt) * a.ldc + c;
                const T wv = gmem(w)[off];
                if (a.unit_c) {
                    y.x = wv;
                } else {
                    const C2 cv = gload_c(C, off);
                    y.x = wv * cv.x;
                    y.y = wv * cv.y;
                }
            }
            ys[tt][kk] = y;
        }
        __syncthreads();
        if (!active) continue;
        for (int tt = 0; tt < tn; ++tt) {
            const int64_t o = (int64_t)(tc + tt) * a.npix + pcol;
            const T g = gmem(gamma)[o];
            const double tv = gmem(tau)[o];
            T zr, zi, er, ei;
            anchor4(g, fa4 * tv, &zr, &zi);
            rotor((T)(two_pi_df * tv), &er, &ei);
#pragma unroll
            for (int j = 0; j < S; ++j)
                add_bin<T, PAIR>(ys[tt][j].x, ys[tt][j].y, zr, zi, er, ei, acc_a[j], acc_b[PAIR ? j : 0]);
        }
    }
    if (!active) return;
    int64_t colB = 0;
    if (PAIR) colB = antipode_north(ring_of_north(col, a.nside), a.npix);
#pragma unroll
    for (int j = 0; j < S; ++j) {
        const int64_t c = c0 + j;
        if (c < 0 || c >= a.nf) continue;
        put_bin<T, PAIR>(a, X, c, col, colB, acc_a[j], PAIR ? acc_b[PAIR ? j : 0] : T(0));
    }
    if (!band_row) return;
    double sa = 0.0, sb = 0.0;
    const BandBins<S> band(a, c0);
#pragma unroll
    for (int j = 0; j < S; ++j) band.add(j, acc_a[j], PAIR ? acc_b[PAIR ? j : 0] : T(0), sa, sb);
    gmem(band_row)[col] = sa;
    if (PAIR) gmem(band_row)[colB] = sb;
}

// One tile of a map whose day is split: 64 pixel columns (the coltile-th block) x one
// S-bin strip (absolute index strip), a slice of the segments for each of the
// workgroup's W waves.  Both tiles are called by every thread of the workgroup; lds
// is its dm_lds bytes of LDS.
template <typename T, bool PAIR, int W>
__device__ inline void dirty_map_split_tile(const MapArgs &a, int64_t strip, int64_t coltile,
                                      const typename Cplx<T>::type *__restrict__ C, const T *__restrict__ w,
                                      const T *__restrict__ gamma, const double *__restrict__ tau,
                                      T *__restrict__ X, double *__restrict__ band_row, char *lds)
{
    using C2 = typename Cplx<T>::type;
    constexpr int S = StripTraits<T>::S;
    constexpr int XTC = StripTraits<T>::XTC;
    constexpr int SLAB = StripTraits<T>::SLAB;
    constexpr int NLD = XTC * S / 64;  // staged values per lane
    constexpr int NA = PAIR ? 2 : 1;   // sums per bin
    static_assert(XTC * S * sizeof(C2) <= kDmWaveLds, "the waves' stages");
    static_assert(NA * SLAB * kDmCols * sizeof(T) <= kDmWaveLds, "a round of the final sums");
    static_assert(S % SLAB == 0 && SLAB % W == 0, "whole rounds");

    // The wave's number as a scalar makes its loops and row addresses scalar: without
    // pairs 7-15 % faster (240 segments, nside 32, 6823 bins 3.02 against 3.55 ms),
    // float64 5 %; the float32 pairs' tile is 1-3 % faster with it in a vector register
    // (1.71 against 1.73 ms).
    constexpr bool kScalarWave = !PAIR || sizeof(T) == 8;
    const int lane = threadIdx.x & 63;
    const int wv = kScalarWave ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : (int)threadIdx.x >> 6;
    const int64_t ncol = PAIR ? (int64_t)a.npix / 2 : (int64_t)a.npix;
    const int64_t col = coltile * kDmCols + lane;
    const bool active = col < ncol;
    const int64_t pcol = active ? col : 0;
    const int64_t kabs0 = strip * S;                          // absolute first bin of the strip
    const int64_t c0 = kabs0 - a.k0;                           // its column in C (may be < 0)
    const double fa4 = 4.0 * (a.f0 + (double)kabs0 * a.df);   // anchor frequency, quarter turns
    const double two_pi_df = kTwoPi * a.df;
    const int per = (a.nt + W - 1) / W;
    const int ta = min(wv * per, a.nt), tb = min(ta + per, a.nt);  // this wave's segments

    T acc_a[S], acc_b[PAIR ? S : 1];
#pragma unroll
    for (int j = 0; j < S; ++j) acc_a[j] = T(0);
#pragma unroll
    for (int j = 0; j < (PAIR ? S : 1); ++j) acc_b[j] = T(0);

    C2(*ys)[S] = reinterpret_cast<C2(*)[S]>(lds + wv * (XTC * S * sizeof(C2)));
    T wr[NLD];
    C2 cr[NLD];
    auto fetch = [&](int tc) {  // values past the slice or the band become zero
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int tt = (i * 64 + lane) / S;
            const int64_t c = c0 + (i * 64 + lane) % S;
            wr[i] = T(0);
            cr[i].x = cr[i].y = T(0);
            if (tc + tt < tb && c >= 0 && c < a.nf) {
                const int64_t off = (int64_t)(tc + tt) * a.ldc + c;
                wr[i] = gmem(w)[off];
                if (a.unit_c)
                    cr[i].x = T(1);
                else
                    cr[i] = gload_c(C, off);
            }
        }
    };
    __syncthreads();  // the previous tile's sums are read
    if (ta < tb) {
        fetch(ta);
        T gn = gmem(gamma)[(int64_t)ta * a.npix + pcol];
        double tn = gmem(tau)[(int64_t)ta * a.npix + pcol];
        for (int tc = ta; tc < tb; tc += XTC) {
            wave_fence();  // the wave's own stage: its reads precede these writes
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                C2 y;
                y.x = wr[i] * cr[i].x;
                y.y = a.unit_c ? T(0) : wr[i] * cr[i].y;
                ys[(i * 64 + lane) / S][(i * 64 + lane) % S] = y;
            }
            wave_fence();
            if (tc + XTC < tb) fetch(tc + XTC);
            const int nseg = min(XTC, tb - tc);
            for (int tt = 0; tt < nseg; ++tt) {
                const T g = gn;
                const double tv = tn;
                // the next segment's seeds (the last one's again at the end)
                const int64_t o = (int64_t)min(tc + tt + 1, tb - 1) * a.npix + pcol;
                gn = gmem(gamma)[o];
                tn = gmem(tau)[o];
                T zr, zi, er, ei;
                anchor4(g, fa4 * tv, &zr, &zi);
                rotor((T)(two_pi_df * tv), &er, &ei);
#pragma unroll
                for (int j = 0; j < S; ++j)
                    add_bin<T, PAIR>(ys[tt][j].x, ys[tt][j].y, zr, zi, er, ei, acc_a[j], acc_b[PAIR ? j : 0]);
            }
        }
    }
    int64_t colB = 0;
    if (PAIR && active) colB = antipode_north(ring_of_north(col, a.nside), a.npix);
    double sa = 0.0, sb = 0.0;  // this thread's share of the strip's broadband sums
    const BandBins<S> band(a, c0);
    // the slices' sums, SLAB bins a round: [slice][sum][bin][column], every thread
    // then adds them for its column and every W-th bin
    T(*sum)[NA][SLAB][kDmCols] = reinterpret_cast<T(*)[NA][SLAB][kDmCols]>(lds);
#pragma unroll
    for (int j0 = 0; j0 < S; j0 += SLAB) {
        __syncthreads();  // the stages, or the previous round, are read
#pragma unroll
        for (int j = 0; j < SLAB; ++j) {
            sum[wv][0][j][lane] = acc_a[j0 + j];
            if (PAIR) sum[wv][NA - 1][j][lane] = acc_b[PAIR ? j0 + j : 0];
        }
        __syncthreads();
        for (int j = wv; j < SLAB; j += W) {
            const int64_t c = c0 + j0 + j;
            if (!active || c < 0 || c >= a.nf) continue;
            T va = sum[0][0][j][lane], vb = PAIR ? sum[0][NA - 1][j][lane] : T(0);
#pragma unroll
            for (int k = 1; k < W; ++k) {
                va += sum[k][0][j][lane];
                if (PAIR) vb += sum[k][NA - 1][j][lane];
            }
            put_bin<T, PAIR>(a, X, c, col, colB, va, vb);
            if (band_row) band.add(j0 + j, va, vb, sa, sb);
        }
    }
    if (!band_row) return;
    __syncthreads();
    double(*bs)[2][kDmCols] = reinterpret_cast<double(*)[2][kDmCols]>(lds);
    bs[wv][0][lane] = sa;
    bs[wv][1][lane] = sb;
    __syncthreads();
    if (wv != 0 || !active) return;
#pragma unroll
    for (int k = 1; k < W; ++k) {
        sa += bs[k][0][lane];
        sb += bs[k][1][lane];
    }
    gmem(band_row)[col] = sa;
    if (PAIR) gmem(band_row)[colB] = sb;
}

// The broadband partial sums' row of a strip (a.band_part, one row per strip the
// call touches), or none.
__device__ inline double *band_row_of(const MapArgs &a, int64_t strip, int S)
{
    return a.band_part ? a.band_part + (strip - a.k0 / S) * (int64_t)a.npix : nullptr;
}

// Either kind of tile.
template <typename T, bool PAIR, int W>
__device__ __forceinline__ void dirty_map_tile(const MapArgs &a, int64_t strip, int64_t coltile,
                                               const typename Cplx<T>::type *__restrict__ C, const T *__restrict__ w,
                                               const T *__restrict__ gamma, const double *__restrict__ tau,
                                               T *__restrict__ X, char *lds)
{
    double *band_row = band_row_of(a, strip, StripTraits<T>::S);
    if constexpr (W == 1)
        dirty_map_whole_tile<T, PAIR, dm_waves(W)>(a, strip, coltile, C, w, gamma, tau, X, band_row, lds);
    else
        dirty_map_split_tile<T, PAIR, W>(a, strip, coltile, C, w, gamma, tau, X, band_row, lds);
}

// Waves per SIMD that the registers have to leave room for: the split tile's two
// sums a bin take half of them, its one sum a quarter.
constexpr int dm_occupancy(bool one_sum, int slices) { return slices == 1 ? 1 : one_sum ? 4 : 2; }

template <typename T, bool PAIR, int W>
__global__ __launch_bounds__(64 * dm_waves(W)) __attribute__((
    amdgpu_waves_per_eu(dm_occupancy(!PAIR && sizeof(T) == 4, W)))) void dirty_map_kernel(MapArgs a, int64_t strip0,
                                                         const typename Cplx<T>::type *__restrict__ C,
                                                         const T *__restrict__ w,
                                                         const T *__restrict__ gamma,
                                                         const double *__restrict__ tau,
                                                         T *__restrict__ X)
{
    __shared__ __attribute__((aligned(16))) char lds[dm_lds<T>(W)];
    dirty_map_tile<T, PAIR, W>(a, strip0 + (int64_t)blockIdx.y, blockIdx.x, C, w, gamma, tau, X, lds);
}

// The same tiles of paired float32 seeds where the matrix-core prep found no
// accurate form (gate).  Nearly every launch finds one and has nothing to do, so
// the tiles share kDmGated workgroups at most: one a tile took 46 us to leave at
// the full band of nside 32, these 5.
constexpr int64_t kDmGated = 8192;

template <int W>
__global__ __launch_bounds__(64 * dm_waves(W)) __attribute__((
    amdgpu_waves_per_eu(dm_occupancy(false, W)))) void dirty_map_gated_kernel(MapArgs a, int64_t strip0,
                                                                             int64_t ncoltiles, int64_t ntiles,
                                                                             const float2 *__restrict__ C,
                                                                             const float *__restrict__ w,
                                                                             const float *__restrict__ gamma,
                                                                             const double *__restrict__ tau,
                                                                             float *__restrict__ X,
                                                                             const double *__restrict__ gate)
{
    __shared__ __attribute__((aligned(16))) char lds[dm_lds<float>(W)];
    if ((int)gate[1] != SGWB_XFORM_VALU) return;
    for (int64_t g = blockIdx.x; g < ntiles; g += gridDim.x)
        dirty_map_tile<float, true, W>(a, strip0 + g / ncoltiles, g % ncoltiles, C, w, gamma, tau, X, lds);
}

// Multi-job form over the concatenated tile list of the jobs (each job: its column
// tiles fastest within a strip, or its strips fastest, as the plan chose).  Whole
// days: persistent, workgroup b takes tiles b, b + grid, b + 2 grid, ...  Split
// days: one workgroup a tile, from tile `first` on.  A tile's result does not depend on which workgroup
// computes it or when.  PAIR and the slices W are uniform over the jobs (the plan
// launches one table per pairing and slices).
template <bool PAIR, int W>
__global__ __launch_bounds__(64 * dm_waves(W)) __attribute__((
    amdgpu_waves_per_eu(dm_occupancy(!PAIR, W)))) void dirty_map_batched_kernel(const XJob *__restrict__ jobs,
                                                                               int32_t njobs, int64_t first,
                                                                               int64_t ntiles)
{
    __shared__ __attribute__((aligned(16))) char lds[dm_lds<float>(W)];
    for (int64_t g = first + blockIdx.x; g < ntiles; g += gridDim.x) {
        int j = 0;
        while (j + 1 < njobs && g >= jobs[j + 1].tile_begin) ++j;
        j = __builtin_amdgcn_readfirstlane(j);
        // read the job's fields as scalars (uniform over the workgroup)
        const MapArgs a = jobs[j].a;
        const int64_t local = g - jobs[j].tile_begin;
        const int64_t ncoltiles = jobs[j].ncoltiles, nstrips = jobs[j].nstrips;
        const int64_t strip0 = jobs[j].strip_first;
        int64_t strip, coltile;
        if (jobs[j].strip_major) {
            strip = strip0 + local / ncoltiles;
            coltile = local % ncoltiles;
        } else {
            coltile = local / nstrips;
            strip = strip0 + local % nstrips;
        }
        const float2 *C = reinterpret_cast<const float2 *>(jobs[j].C);
        dirty_map_tile<float, PAIR, W>(a, strip, coltile, C, jobs[j].w, jobs[j].gamma, jobs[j].tau, jobs[j].X,
                                           lds);
        if (W > 1) break;
    }
}

void fill_xjob(XJob *j, const MapArgs &a, const float *C, const float *w, const float *gamma, const double *tau,
               float *X, bool strip_major)
{
    constexpr int S = StripTraits<float>::S;
    j->a = a;
    j->C = C;
    j->w = w;
    j->gamma = gamma;
    j->tau = tau;
    j->X = X;
    j->strip_first = a.k0 / S;
    j->nstrips = (a.k0 + a.nf - 1) / S - j->strip_first + 1;
    const int64_t ncol = a.nside > 0 ? a.npix / 2 : a.npix;
    j->slices = dm_slices(a.nt, ncol, a.nside > 0);
    const int64_t cols = kDmCols * dm_waves(j->slices) / j->slices;  // per workgroup
    j->ncoltiles = (ncol + cols - 1) / cols;
    j->strip_major = strip_major ? 1 : 0;
    j->tile_begin = 0;
}

hipError_t launch_dirty_map_batched(const XJob *jobs_dev, int32_t njobs, int64_t ntiles, int64_t grid, bool pair,
                                    int32_t slices, hipStream_t s)
{
    decltype(&dirty_map_batched_kernel<true, 1>) kernel = nullptr;
    dm_with_slices(slices, [&](auto n) {
        constexpr int W = decltype(n)::value;
        kernel = pair ? dirty_map_batched_kernel<true, W> : dirty_map_batched_kernel<false, W>;
    });
    const int64_t step = slices > 1 ? 1 << 22 : ntiles;  // tiles a launch
    for (int64_t first = 0; first < ntiles; first += step) {
        const int64_t n = slices > 1 ? std::min(step, ntiles - first) : grid;
        hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(64 * dm_waves(slices)), 0, s, jobs_dev, njobs, first,
                           ntiles);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_dirty_map(const MapArgs &a, const T *C, const T *w, const T *gamma,
                            const double *tau, T *X, hipStream_t s)
{
    using C2 = typename Cplx<T>::type;
    constexpr int S = StripTraits<T>::S;
    const bool pair = a.nside > 0;
    const int64_t ncol = pair ? a.npix / 2 : a.npix;
    const int64_t strip_first = a.k0 / S;
    const int64_t strip_last = (a.k0 + a.nf - 1) / S;
    const int64_t nstrips = strip_last - strip_first + 1;
    const C2 *Cc = reinterpret_cast<const C2 *>(C);
    const int slices = dm_slices(a.nt, ncol, pair), waves = dm_waves(slices);
    const int64_t cols = kDmCols * waves / slices;  // per workgroup
    decltype(&dirty_map_kernel<T, true, 1>) kernel = nullptr;
    dm_with_slices(slices, [&](auto n) {
        constexpr int W = decltype(n)::value;
        kernel = pair ? dirty_map_kernel<T, true, W> : dirty_map_kernel<T, false, W>;
    });
    // grid.y is limited to 65535 strips per launch; larger bands are split.
    for (int64_t s0 = 0; s0 < nstrips; s0 += 65535) {
        const int64_t ns = nstrips - s0 < 65535 ? nstrips - s0 : 65535;
        dim3 grid((unsigned)((ncol + cols - 1) / cols), (unsigned)ns);
        hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, s, a, strip_first + s0, Cc, w, gamma, tau, X);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template hipError_t launch_dirty_map<float>(const MapArgs &, const float *, const float *,
                                            const float *, const double *, float *, hipStream_t);
template hipError_t launch_dirty_map<double>(const MapArgs &, const double *, const double *,
                                             const double *, const double *, double *, hipStream_t);

hipError_t launch_dirty_map_gated(const MapArgs &a, const float *C, const float *w, const float *gamma,
                                  const double *tau, float *X, hipStream_t s, const double *gate)
{
    if (a.nside <= 0) return hipErrorInvalidValue;
    XJob j;
    fill_xjob(&j, a, C, w, gamma, tau, X, true);
    decltype(&dirty_map_gated_kernel<1>) kernel = nullptr;
    dm_with_slices(j.slices, [&](auto n) { kernel = dirty_map_gated_kernel<decltype(n)::value>; });
    hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(kDmGated, xjob_tiles(j))), dim3(64 * dm_waves(j.slices)), 0, s, a,
                       j.strip_first, j.ncoltiles, xjob_tiles(j), reinterpret_cast<const float2 *>(C), w, gamma, tau,
                       X, gate);
    return hipGetLastError();
}

}  // namespace sgwb
