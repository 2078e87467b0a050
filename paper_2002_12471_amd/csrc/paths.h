// Device code that the kernels share: the order of work over the XCDs, and the
// per-path weights of the model (FP64: table build, binned rows, the exact
// training targets of the learned scatter term).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include "lmosem_int.h"

namespace lmo {

// workgroups are dealt to the 8 XCDs round-robin: the item that gives each
// XCD one contiguous run.  Each XCD's L2 starts a kernel empty, so what all
// eight read crosses the fabric eight times: kernels order their items so
// that a run shares its larger operand.
__device__ __forceinline__ int xcd_logical(int p, int n) {
    const int x = p % 8, m = n / 8, rem = n % 8;
    return x * m + min(x, rem) + p / 8;
}

// sum of n values, a power of two, in pairs: log2(n) roundings instead of n
template <int n>
__device__ __forceinline__ float pair_sum(float (&v)[n]) {
#pragma unroll
    for (int h = n / 2; h; h >>= 1)
#pragma unroll
        for (int k = 0; k < h; ++k) v[k] += v[k + h];
    return v[0];
}

// Klein-Nishina total cross-section in units of r_e^2.
__device__ __host__ inline double kn_total(double e) {
    double k = e / kMeC2;
    double l = log1p(2.0 * k);
    double k1 = 1.0 + k, k2 = 1.0 + 2.0 * k;
    return 2.0 * M_PI * (k1 / (k * k) * (2.0 * k1 / k2 - l / k) + l / (2.0 * k) - (1.0 + 3.0 * k) / (k2 * k2));
}

// What a path takes from its flight along (di, dj) pixels to a scatter towards
// (nx, ny): end energy E', Klein-Nishina shape, attenuation ratio at E'.
struct Flight {
    double ep, psi, rho;
};

__device__ inline Flight flight(const Geo &g, int di, int dj, double nx, double ny) {
    const double c = (di * nx + dj * ny) / sqrt((double)(di * di + dj * dj));
    const double t = 1.0 + g.kappa * (1.0 - c);
    const double P = 1.0 / t;
    const double ep = g.e0 * P;
    return {ep, P * P * (P + t - 1.0 + c * c), kn_total(ep) / g.sigma_kn_e0};
}

// Tables of what a path takes from its flight have an entry per pixel offset
// q -> s that the support's bounding box allows, or, where the support has fewer
// pairs than its box has offsets (a few pixels far apart), an entry per pair
// (s, q): never more flights than paths.  Entry offset_from(q) + offset_to(s).
__host__ __device__ inline bool offset_pairs(const Geo &g, const Box &b) {
    return (int64_t)g.n_p * g.n_q < (int64_t)(2 * b.w - 1) * (2 * b.h - 1);
}
__host__ __device__ inline int n_offsets(const Geo &g, const Box &b) {
    return offset_pairs(g, b) ? g.n_p * g.n_q : (2 * b.w - 1) * (2 * b.h - 1);
}
__device__ inline int offset_from(const Geo &g, const Box &b, const int *__restrict__ p_pix, int q) {
    const int i = p_pix[q] % g.nx - b.x, j = p_pix[q] / g.nx - b.y;
    return offset_pairs(g, b) ? q : (b.h - 1 - j) * (2 * b.w - 1) + b.w - 1 - i;
}
__device__ inline int offset_to(const Geo &g, const Box &b, const int *__restrict__ p_pix, int s) {
    const int i = p_pix[s] % g.nx - b.x, j = p_pix[s] / g.nx - b.y;
    return offset_pairs(g, b) ? s * g.n_q : j * (2 * b.w - 1) + i;
}
// the offset (di, dj) of an entry
__device__ inline int2 offset_at(const Geo &g, const Box &b, const int *__restrict__ p_pix, int entry) {
    if (offset_pairs(g, b)) {
        const int ps = p_pix[entry / g.n_q], pq = p_pix[entry % g.n_q];
        return make_int2(ps % g.nx - pq % g.nx, ps / g.nx - pq / g.nx);
    }
    const int w = 2 * b.w - 1;
    return make_int2(entry % w - (b.w - 1), entry / w - (b.h - 1));
}

// Weight w and end energy E' of the path from emission pixel q through path
// end s at angle a (s == q: the primary path).
struct PathW {
    double w, ep;
};

__device__ inline PathW path_weight(const Geo &g, const int *__restrict__ p_pix, const double *__restrict__ L,
                                    const double *__restrict__ Bt, double nx, double ny, int a, int q, int s) {
    if (s == q) return {exp(-L[(size_t)a * g.n_p + q]), g.e0};
    if (!g.scatter) return {0.0, g.e0};
    const int pq = p_pix[q], ps = p_pix[s];
    const int di = ps % g.nx - pq % g.nx, dj = ps / g.nx - pq / g.nx;
    const Flight f = flight(g, di, dj, nx, ny);
    return {Bt[(size_t)s * g.n_p + q] * f.psi / g.psi_bar * exp(-f.rho * L[(size_t)a * g.n_p + s]), f.ep};
}

}  // namespace lmo
