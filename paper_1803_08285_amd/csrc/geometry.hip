// ORF seed matrices gamma(t,p), tau(t,p) (Sec. III.D, Fig. 3) on gfx950.
//
// A workgroup takes 512 northern-half pixels q (two neighbours a lane, so that a
// lane stores 8 and 16 bytes) and a run of segments t.  In float64 a thread
// finds its HEALPix centres once, then for each segment rotates them from the
// celestial frame into the Earth-fixed frame of sidereal time t_k (the inverse
// of the Earth's rotation, equivalent to rotating the detector tensors forward;
// the run's sines and cosines are worked out once, in LDS), and evaluates
//   gamma = sum_A F^A_a F^A_b = 2 tr(P Da P Db) - tr(P Da) tr(P Db),
//   P = I - n n^T (projector transverse to the direction n),
//   tau   = n . (x_a - x_b) / c.
// The antipode a(q) gets gamma and -tau, so the stored seeds are exactly
// antipodally symmetric.  Bound by the float64 arithmetic (~50 instructions a
// direction and segment) beside the 12 bytes a seed that it writes.  Full day,
// nside 64 (530 MB): 114 us (4.6 TB/s); one pixel a lane 126 us, and one thread
// per direction and segment, centre and sidereal angle included, 250 us.
#include "sgwb_internal.h"

namespace sgwb {

constexpr int kGeoRun = 64;  // segments per workgroup, at most

template <typename G>
__global__ __launch_bounds__(256) void geometry_kernel(GeomArgs a, int32_t run, G *__restrict__ gamma,
                                                        double *__restrict__ tau)
{
    // the outputs are aligned to their element alone
    typedef G G2 __attribute__((ext_vector_type(2), aligned(sizeof(G))));
    typedef double D2 __attribute__((ext_vector_type(2), aligned(sizeof(double))));
    __shared__ double sc[kGeoRun][2];
    const int32_t t0 = blockIdx.y * run, nseg = min(run, a.nt - t0);
    if ((int)threadIdx.x < nseg) {
        const double tk = a.t0 + (double)(t0 + (int)threadIdx.x) * a.stride + a.half_dur;
        const double th = kTwoPi * tk / kSiderealDay;
        sincos(th, &sc[threadIdx.x][0], &sc[threadIdx.x][1]);
    }
    __syncthreads();
    const int64_t q = 2 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    if (q >= a.npix / 2) return;
    // rings start at multiples of four and hold a multiple of four pixels, so q
    // and q + 1 share a ring and their antipodes are consecutive too
    const RingPos r = ring_of_north(q, a.nside);
    const int64_t qa = antipode_north(r, a.npix);
    double nx[2], ny[2], nz[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        RingPos re = r;
        re.j += e;
        centre_north(re, a.nside, &nx[e], &ny[e], &nz[e]);
    }
    const double *A = a.DA, *B = a.DB;
    double trAB = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) trAB += A[i] * B[i];
    const double trA = A[0] + A[4] + A[8];
    const double trB = B[0] + B[4] + B[8];
    for (int32_t i = 0; i < nseg; ++i) {
        // Earth-fixed components of the celestial direction at sidereal angle
        // th: n_earth = R_z(-th) n.
        const double s = sc[i][0], c = sc[i][1];
        G2 gv;
        D2 dv;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const double ex = c * nx[e] + s * ny[e];
            const double ey = -s * nx[e] + c * ny[e];
            const double ez = nz[e];
            // u = Da n, v = Db n (symmetric tensors), alpha = n.Da.n, beta = n.Db.n
            const double ux = A[0] * ex + A[1] * ey + A[2] * ez;
            const double uy = A[3] * ex + A[4] * ey + A[5] * ez;
            const double uz = A[6] * ex + A[7] * ey + A[8] * ez;
            const double vx = B[0] * ex + B[1] * ey + B[2] * ez;
            const double vy = B[3] * ex + B[4] * ey + B[5] * ez;
            const double vz = B[6] * ex + B[7] * ey + B[8] * ez;
            const double alpha = ex * ux + ey * uy + ez * uz;
            const double beta = ex * vx + ey * vy + ez * vz;
            // tr(P Da P Db) = tr(Da Db) - 2 u.v + alpha beta ; tr(P D) = tr D - n.D.n
            const double tPAPB = trAB - 2.0 * (ux * vx + uy * vy + uz * vz) + alpha * beta;
            gv[e] = (G)(2.0 * tPAPB - (trA - alpha) * (trB - beta));
            dv[e] = (ex * a.dx[0] + ey * a.dx[1] + ez * a.dx[2]) / kLightSpeed;
        }
        const int64_t row = (int64_t)(t0 + i) * a.npix;
        *reinterpret_cast<G2 *>(gamma + row + q) = gv;
        *reinterpret_cast<G2 *>(gamma + row + qa) = gv;
        *reinterpret_cast<D2 *>(tau + row + q) = dv;
        *reinterpret_cast<D2 *>(tau + row + qa) = -dv;
    }
}

template <typename G>
hipError_t launch_geometry(const GeomArgs &a, G *gamma, double *tau, hipStream_t s)
{
    const int64_t nhalf = a.npix / 2;
    // runs of segments, halved until 1024 workgroups fill the chip: longer runs
    // share a centre's trigonometry, but at nside 32 runs that leave 512 / 1024 /
    // 4096 workgroups took 26 / 24 / 35 us (nside 64: 117 / 117 / 113)
    const int64_t blocks = (nhalf / 2 + 255) / 256;
    int32_t run = kGeoRun;
    while (run > 1 && blocks * ((a.nt + run - 1) / run) < 1024) run /= 2;
    dim3 grid((unsigned)blocks, (unsigned)((a.nt + run - 1) / run));
    hipLaunchKernelGGL(geometry_kernel<G>, grid, dim3(256), 0, s, a, run, gamma, tau);
    return hipGetLastError();
}
template hipError_t launch_geometry<float>(const GeomArgs &, float *, double *, hipStream_t);
template hipError_t launch_geometry<double>(const GeomArgs &, double *, double *, hipStream_t);

__global__ __launch_bounds__(256) void centres_kernel(int64_t nside, double *__restrict__ xyz,
                                                      int32_t *__restrict__ anti)
{
    const int64_t npix = 12 * nside * nside;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= npix / 2) return;
    const RingPos r = ring_of_north(q, nside);
    const int64_t qa = antipode_north(r, npix);
    if (xyz) {
        double x, y, z;
        centre_north(r, nside, &x, &y, &z);
        xyz[3 * q] = x;
        xyz[3 * q + 1] = y;
        xyz[3 * q + 2] = z;
        xyz[3 * qa] = -x;
        xyz[3 * qa + 1] = -y;
        xyz[3 * qa + 2] = -z;
    }
    if (anti) {
        anti[q] = (int32_t)qa;
        anti[qa] = (int32_t)q;
    }
}

hipError_t launch_centres(int64_t nside, double *xyz, int32_t *anti, hipStream_t s)
{
    const int64_t nhalf = 6 * nside * nside;
    hipLaunchKernelGGL(centres_kernel, dim3((unsigned)((nhalf + 255) / 256)), dim3(256), 0, s, nside,
                       xyz, anti);
    return hipGetLastError();
}

}  // namespace sgwb
