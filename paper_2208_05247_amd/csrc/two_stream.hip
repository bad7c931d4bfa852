// two_stream.hip -- clear-sky two-stream column that sets the flux entering
// the top of the ray tracer's domain (sec. 2.3, initialisation paragraph).
// C ABI declared in include/rt3d.h (rt3d_two_stream).
//
// One workgroup per column (a column is typically one g-point's clear-sky
// profile, a few hundred layers), or one lane per column where there are many
// of them or they are longer than the workgroup's LDS (lane_per_column).  FP64
// throughout.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "rt3d.h"

namespace {

constexpr double kKFloor = 1e-12;     // eigenvalue floor (conservative scattering)
constexpr double kResonance = 1e-5;   // |1 - k^2 mu0^2| below this: resonant layer
constexpr double kShift = 1e-5;       // relative mu0 shift around a resonance

struct LayerRT {
    double R, T;        // diffuse reflectance / transmittance (either face)
    double Rdir, Tdir;  // direct beam -> diffuse up at the top / down at the bottom
    double Tb;          // unscattered direct transmittance
};

// Direct-beam terms for the sun at cosine mu: particular solution
// (U, D) = (a, b) exp(-tau/mu) for unit direct horizontal flux at the top,
// plus the source-free solution that removes its diffuse flux entering at
// the top (-b) and at the bottom (-a exp(-tau/mu)), which the layer reflects
// and transmits with R and T.
__device__ void direct_terms(double tau, double w, double g, double g1, double g2, double k, double R, double T,
                             double mu, double* Rdir, double* Tdir) {
    const double g3 = 0.25 * (2.0 - 3.0 * mu * g);
    const double g4 = 1.0 - g3;
    const double d = 1.0 - k * k * mu * mu;
    const double a = w * (g3 * (1.0 - g1 * mu) - g2 * g4 * mu) / d;
    const double b = -w * (g4 * (1.0 + g1 * mu) + g2 * g3 * mu) / d;
    const double tb = exp(-tau / mu);
    *Rdir = a - R * b - T * a * tb;
    *Tdir = b * tb - T * b - R * a * tb;
}

// One homogeneous layer with PIFM coefficients.
__device__ LayerRT layer_rt(double tau, double w, double g, double mu0) {
    const double g1 = 0.25 * (8.0 - w * (5.0 + 3.0 * g));
    const double g2 = 0.75 * w * (1.0 - g);
    const double k = fmax(sqrt(fmax((g1 - g2) * (g1 + g2), 0.0)), kKFloor);
    // source-free solution: modes exp(+-k tau); E = exp(-k tau), X = 1 - E^2
    const double e = exp(-k * tau);
    const double x = -expm1(-2.0 * k * tau);
    const double den = k * (1.0 + e * e) + g1 * x;
    LayerRT L;
    L.R = g2 * x / den;
    L.T = 2.0 * k * e / den;
    if (fabs(1.0 - k * k * mu0 * mu0) < kResonance) {
        // singular particular solution, smooth result: mean of both sides
        // (error O(kShift^2) from the mean; just outside the window the
        // closed form loses about eps / kResonance to cancellation)
        double r1, t1, r2, t2;
        direct_terms(tau, w, g, g1, g2, k, L.R, L.T, mu0 * (1.0 - kShift), &r1, &t1);
        direct_terms(tau, w, g, g1, g2, k, L.R, L.T, mu0 * (1.0 + kShift), &r2, &t2);
        L.Rdir = 0.5 * (r1 + r2);
        L.Tdir = 0.5 * (t1 + t2);
    } else {
        direct_terms(tau, w, g, g1, g2, k, L.R, L.T, mu0, &L.Rdir, &L.Tdir);
    }
    L.Tb = exp(-tau / mu0);
    return L;
}

// Adding method per column.  Up sweep from the surface: rb = diffuse albedo
// of everything below a level, q = upward diffuse flux there produced by the
// direct beam below it; both are parked in flux_up / flux_dn_dif.  Down
// sweep: diffuse downward flux from multiple reflection between a layer and
// what lies below it, then up = rb * down + q overwrites the scratch.
__global__ void two_stream_kernel(int ncols, int nlay, const double* __restrict__ tau,
                                  const double* __restrict__ ssa, const double* __restrict__ asy,
                                  const double* __restrict__ albedo, double mu0, const double* __restrict__ flux_toa,
                                  double* __restrict__ S, double* __restrict__ D, double* __restrict__ U, int tod,
                                  double* __restrict__ tod_flux, float* __restrict__ tod_fd) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncols) return;
    const size_t lo = (size_t)c * nlay;
    const size_t vo = (size_t)c * (nlay + 1);
    double s = (flux_toa ? flux_toa[c] : 1.0) * mu0;
    S[vo] = s;
    for (int l = 0; l < nlay; ++l) {
        s *= exp(-tau[lo + l] / mu0);
        S[vo + l + 1] = s;
    }
    double rb = albedo[c];
    double q = rb * S[vo + nlay];
    U[vo + nlay] = rb;
    D[vo + nlay] = q;
    for (int l = nlay - 1; l >= 0; --l) {
        const LayerRT L = layer_rt(tau[lo + l], ssa[lo + l], asy[lo + l], mu0);
        const double m = 1.0 / (1.0 - L.R * rb);
        const double sl = S[vo + l];
        q = L.Rdir * sl + L.T * (q + rb * L.Tdir * sl) * m;
        rb = L.R + L.T * L.T * rb * m;
        U[vo + l] = rb;
        D[vo + l] = q;
    }
    // top of the atmosphere: no diffuse light comes down
    U[vo] = D[vo];
    D[vo] = 0.0;
    double dn = 0.0;
    for (int l = 0; l < nlay; ++l) {
        const LayerRT L = layer_rt(tau[lo + l], ssa[lo + l], asy[lo + l], mu0);
        const double rbn = U[vo + l + 1];
        const double qn = D[vo + l + 1];
        dn = (L.T * dn + L.Tdir * S[vo + l] + L.R * qn) / (1.0 - L.R * rbn);
        D[vo + l + 1] = dn;
        U[vo + l + 1] = rbn * dn + qn;
    }
    const double tot = S[vo + tod] + D[vo + tod];
    if (tod_flux) tod_flux[c] = tot;
    if (tod_fd) tod_fd[c] = tot > 0.0 ? (float)(D[vo + tod] / tot) : 0.0f;
}

// The same with a workgroup per column.  What is bound is the chain through the
// layers, so everything that does not depend on a neighbour is taken out of
// it: the layer coefficients are computed by all lanes at once (and once, not
// in both sweeps), the direct beam and the diffuse albedo run down and up at
// the same time in two waves, the only division of the albedo's recursion is
// kept (m = 1 / (1 - R rb), which the down sweep divides by again), and the
// fluxes q and dn are then linear recursions x <- A x + B, one FMA per layer,
// whose A and B are again computed by all lanes.  Per layer: 8 FP64 values in
// LDS.  112 columns x 160 layers: 304 us with a lane per column, 37 here.
constexpr int kMaxLayers = 1024;
constexpr int kColumnLanes = 128;

__global__ void __launch_bounds__(kColumnLanes)
two_stream_column_kernel(int nlay, const double* __restrict__ tau, const double* __restrict__ ssa,
                         const double* __restrict__ asy, const double* __restrict__ albedo, double mu0,
                         const double* __restrict__ flux_toa, double* __restrict__ S, double* __restrict__ D,
                         double* __restrict__ U, int tod, double* __restrict__ tod_flux, float* __restrict__ tod_fd) {
    extern __shared__ double sh[];
    double *sR = sh, *sT = sR + nlay, *sRdir = sT + nlay, *sTdir = sRdir + nlay, *sA = sTdir + nlay, *sB = sA + nlay;
    double *sS = sB + nlay, *sRb = sS + nlay + 1;  // nlay + 1 levels
    const int c = blockIdx.x, tid = threadIdx.x;
    const size_t lo = (size_t)c * nlay, vo = (size_t)c * (nlay + 1);
    for (int l = tid; l < nlay; l += kColumnLanes) {
        const LayerRT L = layer_rt(tau[lo + l], ssa[lo + l], asy[lo + l], mu0);
        sR[l] = L.R;
        sT[l] = L.T;
        sRdir[l] = L.Rdir;
        sTdir[l] = L.Tdir;
        sA[l] = L.Tb;
    }
    __syncthreads();
    const double alb = albedo[c];
    if (tid < 64) {  // direct beam, down (every lane the same; one stores)
        double s = (flux_toa ? flux_toa[c] : 1.0) * mu0;
        if (tid == 0) sS[0] = s;
#pragma unroll 4
        for (int l = 0; l < nlay; ++l) {
            s *= sA[l];
            if (tid == 0) sS[l + 1] = s;
        }
    } else {  // diffuse albedo of what lies below, up
        double rb = alb;
        if (tid == 64) sRb[nlay] = rb;
#pragma unroll 4
        for (int l = nlay - 1; l >= 0; --l) {
            const double R = sR[l], T = sT[l];
            const double m = 1.0 / (1.0 - R * rb);
            rb = R + T * T * rb * m;
            if (tid == 64) {
                sB[l] = m;
                sRb[l] = rb;
            }
        }
    }
    __syncthreads();
    // q, the upward flux the direct beam gives: q <- A q + B, up
    for (int l = tid; l < nlay; l += kColumnLanes) {
        const double m = sB[l], A = sT[l] * m;
        sA[l] = A;
        sB[l] = sRdir[l] * sS[l] + A * (sRb[l + 1] * sTdir[l] * sS[l]);
        sTdir[l] = sTdir[l] * sS[l] * m;  // what dn's B needs of them
        sR[l] = sR[l] * m;
    }
    __syncthreads();
    double* sQ = sRdir;  // q of levels 0 .. nlay-1 (Rdir is no longer needed)
    const double q_low = alb * sS[nlay];
    if (tid < 64) {
        double q = q_low;
#pragma unroll 4
        for (int l = nlay - 1; l >= 0; --l) {
            q = __builtin_fma(sA[l], q, sB[l]);
            if (tid == 0) sQ[l] = q;
        }
    }
    __syncthreads();
    // dn, the downward diffuse flux: dn <- A dn + B, down; none comes in at the top
    for (int l = tid; l < nlay; l += kColumnLanes) sB[l] = sTdir[l] + sR[l] * (l + 1 < nlay ? sQ[l + 1] : q_low);
    __syncthreads();
    double* sD = sT;  // dn of levels 1 .. nlay, at l - 1
    if (tid < 64) {
        double dn = 0.0;
#pragma unroll 4
        for (int l = 0; l < nlay; ++l) {
            dn = __builtin_fma(sA[l], dn, sB[l]);
            if (tid == 0) sD[l] = dn;
        }
    }
    __syncthreads();
    for (int l = tid; l <= nlay; l += kColumnLanes) {
        const double dn = l ? sD[l - 1] : 0.0, q = l < nlay ? sQ[l] : q_low;
        S[vo + l] = sS[l];
        D[vo + l] = dn;
        U[vo + l] = sRb[l] * dn + q;
        if (l == tod) {
            const double tot = sS[l] + dn;
            if (tod_flux) tod_flux[c] = tot;
            if (tod_fd) tod_fd[c] = tot > 0.0 ? (float)(dn / tot) : 0.0f;
        }
    }
}

// Which of the two.  A lane's sweeps take 2.3 us a layer, for up to 16384
// columns (a wave a CU) at the same time; a workgroup's 0.21, but its 64 lanes
// repeat one recursion: 0.12 ns a layer and column once the CUs are full, more
// beyond 256 layers, where its LDS lets few share a CU.  From 40000 to 60000
// columns on the lanes' columns no longer fit the caches.  Whole calls in us,
// lane / workgroup:
//   layers    4096 cols    8192       12288      16384      32768      49152      65536     262144
//      4      19 / 19    19 / 19       -        19 / 29       -          -       19 / 115   94 / 441
//     12      26 / 20    27 / 25    28 / 36     28 / 46    37 / 91    60 / 134  127 / 177  626 / 691
//     16      36 / 19    37 / 30    38 / 42     39 / 54    55 / 105  137 / 158  239 / 209 1036 / 815
//     24      53 / 21    54 / 39    56 / 55     58 / 71    88 / 139  212 / 206  354 / 272     -
//     48     111 / 37   112 / 67   117 / 94    124 / 123  188 / 238  418 / 350  696 / 462     -
//    100        -       243 / 129  251 / 188   260 / 234  361 / 451  796 / 668     -     6290 / 3457
//    200     470 / 135  482 / 246  495 / 352   521 / 457  934 / 878 1659 / 1302 2705 / 1720   -
//    400     935 / 317  953 / 591 1011 / 851  1081 / 1119 1934 / 2172 3302 / 3236 5409 / 4292 -
//    500    1182 / 503 1261 / 992 1325 / 1476 1416 / 1953 2625 / 3864 4482 / 5769 6712 / 7672 31552 / 30524
//   1024    2494 / 1864 2636 / 3699 2759 / 5535 2949 / 7359 5013 / 14671 8326 / 21982 12377 / 29235 62394 / 116449
// A launch has fewer than 2^32 lanes: 2^25 columns and more by lanes.
bool lane_per_column(int64_t cols, int64_t nlay) {
    if (nlay > kMaxLayers || cols * kColumnLanes >= (int64_t)1 << 32) return true;
    if (nlay <= 12) return cols > 8192;
    if (nlay <= 16) return cols > 10000 && cols <= 60000;
    if (nlay <= 24) return cols > 12288 && cols <= 49152;
    if (nlay <= 100) return cols > 16384 && cols <= 40960;
    if (nlay <= 352) return false;
    if (nlay <= 400) return cols > 16384 && cols <= 32768;
    return cols * nlay > 6000000 && (nlay > 480 || cols <= 57344);
}

}  // namespace

extern "C" {

rt3d_status rt3d_two_stream(int32_t n_cols, int32_t nlay, const double* tau, const double* ssa, const double* g,
                            const double* albedo, double mu0, const double* flux_toa, double* flux_dir,
                            double* flux_dn_dif, double* flux_up, int32_t tod_level, double* tod_flux,
                            float* tod_diffuse_fraction, void* stream) {
    if (n_cols < 1 || nlay < 1 || !tau || !ssa || !g || !albedo || !flux_dir || !flux_dn_dif || !flux_up)
        return RT3D_EINVAL;
    if (!(mu0 > 0.0 && mu0 <= 1.0)) return RT3D_EINVAL;
    if (tod_level < 0 || tod_level > nlay) return RT3D_EINVAL;
    if (lane_per_column(n_cols, nlay))
        hipLaunchKernelGGL(two_stream_kernel, dim3((unsigned)(((int64_t)n_cols + 63) / 64)), dim3(64), 0, (hipStream_t)stream,
                           n_cols, nlay, tau, ssa, g, albedo, mu0, flux_toa, flux_dir, flux_dn_dif, flux_up, tod_level,
                           tod_flux, tod_diffuse_fraction);
    else
        hipLaunchKernelGGL(two_stream_column_kernel, dim3((unsigned)n_cols), dim3(kColumnLanes),
                           sizeof(double) * (8 * (size_t)nlay + 2), (hipStream_t)stream, nlay, tau, ssa, g, albedo, mu0,
                           flux_toa, flux_dir, flux_dn_dif, flux_up, tod_level, tod_flux, tod_diffuse_fraction);
    return hipGetLastError() == hipSuccess ? RT3D_OK : RT3D_EDEVICE;
}

}  // extern "C"
