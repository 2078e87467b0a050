// Binned data: the binned alternative to list mode (Sec. 2.2).  Events are
// counted in bins (a, b, k): angle a, one of n_pos equal position bins over
// the detector, and energy bin [e_k, e_k+1).  The binned system row of a bin
// integrates the list-mode row over it,
//     H[(a,b,k)][q] = sum over paths from q of w * (mass of K over the
//                     position bin) * (mass of G over the energy bin),
// with every path weight in FP64 from the line integrals and scatter-point
// factors (the function the table build uses).  Binned OS-MLEM then runs on
// these rows with the kernels of the cached-row path (row means,
// backprojection of y / mean, update).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "lmosem_int.h"
#include "paths.h"

namespace lmo {

// mass of the truncated position response centred at us over [u0, u1]
__device__ inline double pos_mass(const Geo &g, double us, double u0, double u1) {
    const double s = g.sig_u;
    const double a = fmax(u0 - us, -3.0 * s), b = fmin(u1 - us, 3.0 * s);
    if (b <= a) return 0.0;
    const double gs = s * sqrt(M_PI / 2.0) * (erf(b / (M_SQRT2 * s)) - erf(a / (M_SQRT2 * s)));
    return (gs - exp(-4.5) * (b - a)) / g.zk;
}

// mass of the energy response centred at ep over [e0, e1]
__device__ inline double energy_mass(const Geo &g, double ep, double e0, double e1) {
    const double s2 = M_SQRT2 * g.sig_e;
    return 0.5 * (erf((e1 - ep) / s2) - erf((e0 - ep) / s2));
}

// H[row][q] for the bins listed in row_bin (flat id (a * n_pos + b) * n_e + k);
// one block row per bin, one thread per emission pixel; padding columns are 0.
__global__ __launch_bounds__(256) void k_binned_rows(Geo g, const int *__restrict__ p_pix,
                                                     const double *__restrict__ cs, const double *__restrict__ Ld,
                                                     const double *__restrict__ Bt, const int *__restrict__ s_sorted,
                                                     const double *__restrict__ us_sorted, int n_pos,
                                                     const double *__restrict__ edges, int n_e,
                                                     const int *__restrict__ row_bin, float *__restrict__ H) {
    const int row = blockIdx.y;
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= g.n_qpad) return;
    float *out = H + (size_t)row * g.n_qpad + q;
    if (q >= g.n_q) { *out = 0.0f; return; }
    const int bin = row_bin[row];
    const int a = bin / (n_pos * n_e), b = (bin / n_e) % n_pos, k = bin % n_e;
    const double width = 2.0 * g.half_len / n_pos;
    const double u0 = -g.half_len + b * width, u1 = u0 + width;
    const double e0 = edges[k], e1 = edges[k + 1];
    const double nx = cs[2 * a], ny = cs[2 * a + 1];
    const double *us = us_sorted + (size_t)a * g.n_p;
    const double reach = 3.0 * g.sig_u;
    int lo = 0, hi = g.n_p;   // first rank with us > u0 - reach
    while (lo < hi) { const int m = (lo + hi) >> 1; if (us[m] > u0 - reach) hi = m; else lo = m + 1; }
    double sum = 0.0;
    for (int r = lo; r < g.n_p && us[r] < u1 + reach; ++r) {
        const double pm = pos_mass(g, us[r], u0, u1);
        if (pm <= 0.0) continue;
        const PathW pw = path_weight(g, p_pix, Ld, Bt, nx, ny, a, q, s_sorted[(size_t)a * g.n_p + r]);
        if (pw.w > 0.0) sum += pw.w * pm * energy_mass(g, pw.ep, e0, e1);
    }
    *out = (float)sum;
}

// All bins of every angle at once.  A path end's position response spans at
// most W consecutive position bins, and path ends are ranked by position, so
// one thread per (angle, emission pixel) walks the ranks once, evaluating each
// path weight once (rather than once per bin that the path reaches), with W
// bins of accumulators that slide along the detector.
//
// What a path takes from its direction of flight at an angle (Klein-Nishina
// factor, attenuation ratio, mass of the energy response over each energy bin)
// depends on the pixel offset q -> s alone: it is evaluated once per (angle,
// offset), four times the area of the support's bounding box of them, instead of
// once per path, n_p n_q of them (whichever are fewer: offset_pairs).  A path then
// costs one exponential and 24 bytes from the L2, which bound it: 6.06 ms ->
// 1.04 ms for 120 angles x 1436 x 1436 paths.  What depends
// on the rank only comes precomputed as well (k_rank_terms), read as scalars.
template <int W>
__global__ void k_rank_terms(Geo g, Box box, const int *__restrict__ p_pix, const double *__restrict__ Ld,
                             const int *__restrict__ s_sorted, const double *__restrict__ us_sorted, int n_pos,
                             int *__restrict__ rb0, int *__restrict__ roff, double *__restrict__ rL,
                             double *__restrict__ rpm) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x, a = blockIdx.y;
    if (r >= g.n_p) return;
    const size_t o = (size_t)a * g.n_p + r;
    const double us = us_sorted[o];
    const double width = 2.0 * g.half_len / n_pos;
    const int b0 = min(max((int)floor((us - 3.0 * g.sig_u + g.half_len) / width), 0), n_pos - 1);
    rb0[o] = b0;
    const int s = s_sorted[o];
    roff[o] = offset_to(g, box, p_pix, s);
    rL[o] = Ld[(size_t)a * g.n_p + s];
    for (int i = 0; i < W; ++i) {
        const int b = b0 + i;
        const double u0 = -g.half_len + b * width, u1 = u0 + width;
        rpm[o * W + i] = b < n_pos ? pos_mass(g, us, u0, u1) : 0.0;
    }
}

// tab[angle - a0][1 + n_e][entry]: attenuation ratio, and Klein-Nishina factor
// times the energy-bin masses of a flight along the entry's offset (0 for no
// offset: the primary path, which the rows weigh by themselves)
__global__ __launch_bounds__(256) void k_direction_terms(Geo g, Box box, const int *__restrict__ p_pix,
                                                         const double *__restrict__ cs, int a0,
                                                         const double *__restrict__ edges, int n_e,
                                                         double *__restrict__ tab) {
    const int n = n_offsets(g, box);
    const int i = blockIdx.x * blockDim.x + threadIdx.x, a = a0 + blockIdx.y;
    if (i >= n) return;
    const int2 d = offset_at(g, box, p_pix, i);
    double *out = tab + (size_t)blockIdx.y * (1 + n_e) * n + i;
    if (d.x == 0 && d.y == 0) {
        for (int k = 0; k < 1 + n_e; ++k) out[(size_t)k * n] = 0.0;
        return;
    }
    const Flight fl = flight(g, d.x, d.y, cs[2 * a], cs[2 * a + 1]);
    out[0] = fl.rho;
    for (int k = 0; k < n_e; ++k)
        out[(size_t)(1 + k) * n] = fl.psi / g.psi_bar * energy_mass(g, fl.ep, edges[k], edges[k + 1]);
}

// One wave per (angle, 64 emission pixels); an XCD takes a run of angles, whose
// direction terms then stay in its L2.  The loads of
// the next kAhead ranks are on their way while the current ones are used.
template <int W, int KMAX>
__global__ __launch_bounds__(64) void k_binned_rows_all(Geo g, Box box, const int *__restrict__ p_pix,
                                                        const double *__restrict__ Ld, const double *__restrict__ Bt,
                                                        const int *__restrict__ s_sorted, const int *__restrict__ rb0,
                                                        const int *__restrict__ roff, const double *__restrict__ rL,
                                                        const double *__restrict__ rpm, int n_pos,
                                                        const double *__restrict__ edges, int n_e,
                                                        const double *__restrict__ tab, int a0, int n_a,
                                                        const int *__restrict__ angle_row0, float *__restrict__ H) {
    constexpr int kAhead = 4;
    const int item = xcd_logical(blockIdx.x, gridDim.x);
    const int n_qb = g.n_qpad / 64, al = item / n_qb, qb = item - al * n_qb, a = a0 + al;
    const int q = qb * 64 + threadIdx.x;   // n_qpad is a multiple of 64
    const bool active = q < g.n_q;
    const int qc = min(q, g.n_q - 1);
    const int n_off = n_offsets(g, box), from = offset_from(g, box, p_pix, qc);
    const double *ta = g.scatter ? tab + (size_t)al * (1 + n_e) * n_off : nullptr;
    // the primary path
    const double w0 = active ? exp(-Ld[(size_t)a * g.n_p + qc]) : 0.0;
    double em0[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) em0[k] = k < n_e ? energy_mass(g, g.e0, edges[k], edges[k + 1]) : 0.0;
    float *Hq = H + (size_t)angle_row0[a] * g.n_qpad + q;
    double acc[W][KMAX];
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int k = 0; k < KMAX; ++k) acc[i][k] = 0.0;
    int base = 0;
    // write the lowest bin of the window and slide it up by one bin
    auto shift = [&]() {
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
            if (k < n_e) Hq[(size_t)(base * n_e + k) * g.n_qpad] = (float)acc[0][k];
#pragma unroll
        for (int i = 0; i + 1 < W; ++i)
#pragma unroll
            for (int k = 0; k < KMAX; ++k) acc[i][k] = acc[i + 1][k];
#pragma unroll
        for (int k = 0; k < KMAX; ++k) acc[W - 1][k] = 0.0;
        ++base;
    };
    const size_t o = (size_t)a * g.n_p;
    struct Ranks {
        int s[kAhead];
        double B[kAhead], rho[kAhead], em[kAhead][KMAX];
    };
    auto load = [&](Ranks &x, int r0) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int r = min(r0 + u, g.n_p - 1);
            x.s[u] = s_sorted[o + r];
            if (!g.scatter) {
#pragma unroll
                for (int k = 0; k < KMAX; ++k) x.em[u][k] = 0.0;
                continue;
            }
            const double *td = ta + from + roff[o + r];
            x.B[u] = Bt[(size_t)x.s[u] * g.n_p + qc];
            x.rho[u] = td[0];
#pragma unroll
            for (int k = 0; k < KMAX; ++k) x.em[u][k] = td[(size_t)(1 + min(k, n_e - 1)) * n_off];
        }
    };
    auto use = [&](const Ranks &x, int r0) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int r = r0 + u;
            if (r >= g.n_p) break;
            const int b0 = rb0[o + r];
            while (base < b0) shift();
            const bool self = x.s[u] == qc;
            if (!g.scatter && __ballot(self) == 0) continue;
            double w = 0.0;
            if (g.scatter) w = active ? x.B[u] * exp(-x.rho[u] * rL[o + r]) : 0.0;
            w = self ? w0 : w;
            const double *pm = rpm + (o + r) * W;
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                const double we = w * (self ? em0[k] : x.em[u][k]);
#pragma unroll
                for (int i = 0; i < W; ++i) acc[i][k] = fma(we, pm[i], acc[i][k]);
            }
        }
    };
    Ranks x, y;
    load(x, 0);
    for (int r0 = 0; r0 < g.n_p; r0 += 2 * kAhead) {
        load(y, r0 + kAhead);
        use(x, r0);
        load(x, r0 + 2 * kAhead);
        use(y, r0 + kAhead);
    }
    while (base < n_pos) shift();
}

// counts[(a * n_pos + b) * n_e + k] += 1 per event inside a bin
__global__ void k_bin_events(Geo g, int64_t n, const int32_t *__restrict__ angle, const float *__restrict__ u_bin,
                             const float *__restrict__ energy, int n_pos, const double *__restrict__ edges, int n_e,
                             float *__restrict__ counts) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int a = angle[j];
    if (a < 0 || a >= g.n_angles) return;
    const float ub = u_bin[j];
    if (!(ub >= 0.0f) || !(ub < (float)g.n_bins)) return;
    const int b = min((int)((double)ub * n_pos / g.n_bins), n_pos - 1);
    const double e = (double)energy[j];
    if (!(e >= edges[0]) || !(e <= edges[n_e])) return;
    int k = 0;
    while (k + 1 < n_e && e >= edges[k + 1]) ++k;
    atomicAdd(counts + ((size_t)a * n_pos + b) * n_e + k, 1.0f);   // integer counts: exact in any order
}

__global__ void k_gather_counts(const float *__restrict__ counts, const int *__restrict__ row_bin, int n_rows,
                                float *__restrict__ y) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_rows) y[i] = counts[row_bin[i]];
}

// weights of the binned backprojection: y_i / mean_i (0 for a dead bin)
__global__ void k_count_weights(const float *__restrict__ y, const float *__restrict__ inv, int n_rows,
                                float *__restrict__ w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_rows) w[i] = y[i] * inv[i];
}

hipError_t launch_binned_rows(const Geo &g, const Tables &t, int n_pos, const double *edges_dev, int n_e,
                              const int *row_bin_dev, int n_rows, float *H, hipStream_t st) {
    if (n_rows <= 0) return hipSuccess;
    if (!t.Ld) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((g.n_qpad + 255) / 256), (unsigned)n_rows);
    hipLaunchKernelGGL(k_binned_rows, grid, dim3(256), 0, st, g, t.p_pix, t.cs, t.Ld, t.Bt, t.s_sorted, t.us_sorted,
                       n_pos, edges_dev, n_e, row_bin_dev, H);
    return hipGetLastError();
}

// scratch of the rows of every bin
struct RowScratch {
    int *rb0 = nullptr, *roff = nullptr;
    double *rL = nullptr, *rpm = nullptr, *tab = nullptr;
    int n_a = 0;   // angles whose direction terms fit
};

template <int W, int KMAX>
hipError_t launch_rows_all(const Geo &g, const Tables &t, int n_pos, const double *edges_dev, int n_e,
                           const int *angle_row0_dev, const RowScratch &w, float *H, hipStream_t st) {
    hipLaunchKernelGGL(k_rank_terms<W>, dim3((unsigned)((g.n_p + 255) / 256), (unsigned)g.n_angles), dim3(256), 0, st,
                       g, t.box, t.p_pix, t.Ld, t.s_sorted, t.us_sorted, n_pos, w.rb0, w.roff, w.rL, w.rpm);
    const int n_off = n_offsets(g, t.box);
    for (int a0 = 0; a0 < g.n_angles; a0 += w.n_a) {
        const int n_a = std::min(w.n_a, g.n_angles - a0);
        if (g.scatter)
            hipLaunchKernelGGL(k_direction_terms, dim3((unsigned)((n_off + 255) / 256), (unsigned)n_a), dim3(256), 0, st, g,
                               t.box, t.p_pix, t.cs, a0, edges_dev, n_e, w.tab);
        hipLaunchKernelGGL((k_binned_rows_all<W, KMAX>), dim3((unsigned)(g.n_qpad / 64 * n_a)), dim3(64), 0, st, g, t.box, t.p_pix,
                           t.Ld, t.Bt, t.s_sorted, w.rb0, w.roff, w.rL, w.rpm, n_pos, edges_dev, n_e, w.tab, a0, n_a,
                           angle_row0_dev, H);
    }
    return hipGetLastError();
}

// Rows of every bin, angle a's rows starting at angle_row0[a] in (position
// bin, energy bin) order.  hipErrorNotSupported when a position response
// spans more bins, or there are more energy bins, than the instantiated
// windows hold, or the scratch does not fit (the caller then lists the bins for
// k_binned_rows, which needs none).
hipError_t launch_binned_rows_all(const Geo &g, const Tables &t, int n_pos, const double *edges_dev, int n_e,
                                  const int *angle_row0_dev, float *H, Arena *arena, hipStream_t st) {
    if (!t.Ld) return hipErrorInvalidValue;
    const double width = 2.0 * g.half_len / n_pos;
    const int span = (int)ceil(6.0 * g.sig_u / width) + 2;   // bins a response can touch
    const int W = span <= 8 ? 8 : span <= 16 ? 16 : 0;
    if (W == 0 || n_e > (W == 8 ? 4 : 2)) return hipErrorNotSupported;
    RowScratch w;
    const size_t na_np = (size_t)g.n_angles * g.n_p;
    // direction terms of as many angles as 64 MB hold (all of them for supports
    // within 128 x 128: the chip is full with a few tens of angles)
    const size_t per = (size_t)n_offsets(g, t.box) * (1 + n_e) * sizeof(double);
    w.n_a = g.scatter ? (int)std::min<size_t>(g.n_angles, std::max<size_t>(1, (size_t(64) << 20) / per)) : g.n_angles;
    hipError_t e = dev_take(arena, &w.rb0, sizeof(int) * na_np);
    if (e == hipSuccess) e = dev_take(arena, &w.roff, sizeof(int) * na_np);
    if (e == hipSuccess) e = dev_take(arena, &w.rL, sizeof(double) * na_np);
    if (e == hipSuccess) e = dev_take(arena, &w.rpm, sizeof(double) * na_np * W);
    if (e == hipSuccess && g.scatter) e = dev_take(arena, &w.tab, per * w.n_a);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        e = hipErrorNotSupported;
    }
    if (e == hipSuccess) {
        // the fewest accumulators that hold the energy bins
        auto rows = W == 8 ? (n_e == 1 ? launch_rows_all<8, 1> : n_e == 2 ? launch_rows_all<8, 2> : launch_rows_all<8, 4>)
                           : (n_e == 1 ? launch_rows_all<16, 1> : launch_rows_all<16, 2>);
        e = rows(g, t, n_pos, edges_dev, n_e, angle_row0_dev, w, H, st);
    }
    // the scratch is released once the kernels are done
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    for (void *p : {(void *)w.rb0, (void *)w.roff, (void *)w.rL, (void *)w.rpm, (void *)w.tab}) dev_give(arena, p);
    return e;
}

hipError_t launch_bin_events(const Geo &g, const lmosem_events &ev, int n_pos, const double *edges_dev, int n_e,
                             float *counts, hipStream_t st) {
    if (ev.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_bin_events, dim3((unsigned)((ev.n + 255) / 256)), dim3(256), 0, st, g, ev.n, ev.angle,
                       ev.u_bin, ev.energy_kev, n_pos, edges_dev, n_e, counts);
    return hipGetLastError();
}

hipError_t launch_gather_counts(const float *counts, const int *row_bin, int n_rows, float *y, hipStream_t st) {
    if (n_rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_counts, dim3((n_rows + 255) / 256), dim3(256), 0, st, counts, row_bin, n_rows, y);
    return hipGetLastError();
}

hipError_t launch_count_weights(const float *y, const float *inv, int n_rows, float *w, hipStream_t st) {
    if (n_rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_count_weights, dim3((n_rows + 255) / 256), dim3(256), 0, st, y, inv, n_rows, w);
    return hipGetLastError();
}

}  // namespace lmo
