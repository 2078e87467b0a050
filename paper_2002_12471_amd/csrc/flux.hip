// Sub-iterations through directional flux: the per-event means (denominator
// of Eq. 8) and the backprojection (numerator of Eq. 7) of the exact model
// without a term per (event, emission pixel, path end).
//
// The scatter part of the model is, for event j of angle a,
//     sum_s K(u_j - u_s) sum_q f_q B(q, s) g_as(phi_qs; E_j),
//     g_as(phi; E) = Psi(c)/Psi_bar e^(-rho(c) L_a(s)) G(E; E'(c)),  c = cos(phi - theta_a),
// with phi_qs the direction of flight from q to s: for one scatter point
// everything behind B depends on the emission pixel only through phi_qs, and
// g is smooth in phi and in E.  So the sums are taken in stages,
//     I_s(n)    = sum_q f_q B(q, s) l_n(phi_qs)               directional flux (k_flux_spread)
//     S_as(k)   = sum_n I_s(n) g_as(phi_n; E_k)               spectra (k_flux_spectra)
//     mean_j    = sum_s K_js (P_as g0_j + sum_k l_k(E_j) S_as(k))   (k_flux_means)
// and the adjoint runs the same stages backwards (k_flux_adjoint: events to
// energy nodes, k_flux_fields: energy nodes to directions, k_flux_gather:
// directions to emission pixels).  l_n and l_k are eight-point interpolation
// weights on equispaced directions phi_n and energies E_k.  The primary path
// (P_as = f_s e^(-L_a(s)), energy factor g0_j) is carried exactly.
//
// The interpolated functions are Gaussians of the energy difference, so in a
// node's neighbourhood they run like exponentials e^(b x); the weights are
// exact for eight exponents b at Chebyshev points of the range met (and not
// for powers of x, whose remainder grows far out in the tails): for the
// energies after dividing out a Gaussian about the middle of the end
// energies, which leaves pure exponentials.  One path's relative error is at
// most 4.5e-7 in energy at any distance from its end energy; in direction
// flux_geometry evaluates it for the response, the Klein-Nishina factor and the
// attenuation at hand and takes as many nodes as keep it within 2e-7 up to
// three widths of the energy response, 2e-6 up to six and 6e-5 anywhere in the
// window, alternating in sign from path to path (term by term FP32 leaves up to
// 1e-6 of one path's code).  Against FP64, events whose mean is at least 1e-8 of
// the largest have 1.2 to 2e-7 rms, uniform and compact sources alike, and 2e-7
// term by term.
//
// Work per sub-iteration: n_p^2 pair visits (twice), angles x n_p x N x K
// multiply-adds on the matrix cores (twice), and eight multiply-adds per
// (event, path end) (twice), where the direct form evaluates an exponential
// per (event, path end, emission pixel).
#include <hip/hip_runtime.h>
#include <hipcub/device/device_scan.hpp>
#include <math.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "lmosem_int.h"
#include "paths.h"

namespace lmo {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSec = 12;    // direction intervals per sector (a workgroup's share of a pixel block's pairs)
constexpr int kTap = 8;     // interpolation points
constexpr int kStrip = 16;  // columns of a strip of the flux order

// interpolation weights at offset t (in node spacings, [0, 1) from the fourth
// node), exact for the fit's eight exponentials
__device__ __forceinline__ void fit_weights(const FluxFit &fit, double t, double (&w)[kTap]) {
    double x[kTap];
#pragma unroll
    for (int m = 0; m < kTap; ++m) x[m] = exp(fit.b[m] * t);
#pragma unroll
    for (int i = 0; i < kTap; ++i) {
        w[i] = 0.0;
#pragma unroll
        for (int m = 0; m < kTap; ++m) w[i] = fma(fit.v[i][m], x[m], w[i]);
    }
}

__device__ __forceinline__ int wrap(int n, int N) { return n < 0 ? n + N : (n >= N ? n - N : n); }

// ---------------------------------------------------------------- tables (once per attenuation map)

// node position (in node spacings, [0, N)) of the direction of offset (di, dj)
__device__ inline double node_pos(int di, int dj, int N) {
    double t = atan2((double)dj, (double)di) * (N / (2.0 * M_PI));
    if (t < 0.0) t += N;
    return t >= N ? 0.0 : t;
}

// the box offsets whose direction lies in node interval n, in index order:
// one block per interval
__global__ __launch_bounds__(256) void k_flux_offsets(int W, int Hh, int N, int cap, int *__restrict__ cnt,
                                                      int2 *__restrict__ off) {
    __shared__ int wsum[4];
    const int n = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int w2 = 2 * W - 1, total = w2 * (2 * Hh - 1);
    int have = 0;
    for (int i0 = 0; i0 < total; i0 += 256) {
        const int i = i0 + threadIdx.x;
        const int di = i % w2 - (W - 1), dj = i / w2 - (Hh - 1);
        const bool in = i < total && (di || dj) && (int)node_pos(di, dj, N) == n;
        const unsigned long long m = __ballot(in);
        if (lane == 0) wsum[wave] = __popcll(m);
        __syncthreads();
        int at = have + __popcll(m & ((1ull << lane) - 1));
        for (int w = 0; w < wave; ++w) at += wsum[w];
        if (in && at < cap) off[(size_t)n * cap + at] = make_int2(di, dj);
        have += wsum[0] + wsum[1] + wsum[2] + wsum[3];
        __syncthreads();
    }
    if (threadIdx.x == 0) cnt[n] = min(have, cap);
}

// Per pixel block (64 pixels of the flux order, one per lane) and node
// interval: the offsets that lead at least one of its pixels to another
// support pixel.  FILL = 0 counts them; FILL = 1 writes their records (box
// offset and the interpolation weights of their direction) and, per lane, the
// symmetric part of the pair factor, B(q, s) / mu(s) = pixel_cm^2 e^(-l) / (2 pi r)
// (0 where the lane's pixel has no partner), rounded from FP64.
template <int FILL>
__global__ __launch_bounds__(64) void k_flux_pairs(Geo g, FluxGeo fg, FluxFit fit, const int *__restrict__ sup,
                                                   const int *__restrict__ p_pix, const int *__restrict__ q_of_pix,
                                                   const float *__restrict__ mu, const double *__restrict__ Bt,
                                                   const int *__restrict__ cnt, const int2 *__restrict__ off, int cap,
                                                   int *__restrict__ beg, int *__restrict__ rec_off,
                                                   int *__restrict__ rec_n, float *__restrict__ rec_w, double *__restrict__ rec_w64,
                                                   float *__restrict__ sym) {
    const int n = blockIdx.x, b = blockIdx.y, lane = threadIdx.x;
    const int x = b * 64 + lane < g.n_p ? sup[b * 64 + lane] : -1;
    const int px = x >= 0 ? p_pix[x] : -1;
    const int xi = px >= 0 ? px % g.nx : -1, xj = px >= 0 ? px / g.nx : -1;
    int at = FILL ? beg[b * fg.N + n] : 0;
    for (int k = 0; k < cnt[n]; ++k) {
        const int2 d = off[(size_t)n * cap + k];
        const int yi = xi + d.x, yj = xj + d.y;
        const bool in = px >= 0 && yi >= 0 && yi < g.nx && yj >= 0 && yj < g.ny;
        const int y = in ? q_of_pix[yj * g.nx + yi] : -1;
        // a pair without an emission pixel carries nothing
        const bool use = y >= 0 && (x < g.n_q || y < g.n_q);
        if (__ballot(use) == 0) continue;
        if (FILL) {
            double v = 0.0;
            if (use)
                v = y < g.n_q ? Bt[(size_t)x * g.n_p + y] / (double)mu[px]
                              : Bt[(size_t)y * g.n_p + x] / (double)mu[p_pix[y]];
            sym[(size_t)at * 64 + lane] = (float)v;
            if (lane == 0) {
                rec_off[at] = d.y * fg.W + d.x;
                rec_n[at] = n;
                double w[kTap];
                fit_weights(fit, node_pos(d.x, d.y, fg.N) - n, w);
#pragma unroll
                for (int i = 0; i < kTap; ++i) {
                    rec_w[(size_t)at * kTap + i] = (float)w[i];
                    rec_w64[(size_t)at * kTap + i] = w[i];
                }
            }
        }
        ++at;
    }
    if (!FILL && lane == 0) beg[b * fg.N + n] = at;
}

// per (angle, direction node): Psi/Psi_bar, -rho log2 e, and the energy
// response at every energy node; one block per angle and 16 directions
__global__ __launch_bounds__(256) void k_flux_angles(Geo g, FluxGeo fg, const double *__restrict__ cs,
                                                     float *__restrict__ psi, float *__restrict__ rho,
                                                     float *__restrict__ G) {
    __shared__ double ep_s[16];
    const int a = blockIdx.y, n0 = blockIdx.x * 16;
    if (threadIdx.x < 16) {
        const int n = n0 + threadIdx.x;
        const double ph = 2.0 * M_PI * n / fg.N;
        const double c = cos(ph) * cs[2 * a] + sin(ph) * cs[2 * a + 1];
        const double t = 1.0 + g.kappa * (1.0 - c), P = 1.0 / t, ep = g.e0 * P;
        psi[(size_t)a * fg.N + n] = (float)(P * P * (P + t - 1.0 + c * c) / g.psi_bar);
        rho[(size_t)a * fg.N + n] = (float)(-kn_total(ep) / g.sigma_kn_e0 * 1.4426950408889634);
        ep_s[threadIdx.x] = ep;
    }
    __syncthreads();
    const double norm = 1.0 / (sqrt(2.0 * M_PI) * g.sig_e);
    for (int i = threadIdx.x; i < 16 * fg.K; i += 256) {
        const int n = i / fg.K, k = i - n * fg.K;
        const double e = fg.e_lo + (k - 3) * fg.h - ep_s[n];
        G[((size_t)a * fg.N + n0 + n) * fg.K + k] = (float)(norm * exp2(-g.c2 * e * e));
    }
}

// tables of the flux order (strips of kStrip columns, so that a block of 64
// pixels is compact in both directions): support index, box index, mu; per
// angle rank, primary weight and attenuation, and the order's index by rank
__global__ void k_flux_support(Geo g, FluxGeo fg, const int *__restrict__ sup, const int *__restrict__ p_pix,
                               const float *__restrict__ mu, int *__restrict__ pos, int *__restrict__ box,
                               float *__restrict__ mu_s, float *__restrict__ mu_box) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= g.n_p) return;
    const int pix = p_pix[sup[x]];
    pos[sup[x]] = x;
    box[x] = (pix / g.nx - fg.y0) * fg.W + (pix % g.nx - fg.x0);
    mu_s[x] = mu[pix];
    mu_box[box[x]] = mu[pix];
}

__global__ void k_flux_ranks(Geo g, const int *__restrict__ pos, const int *__restrict__ s_sorted,
                             const double *__restrict__ Ld, int *__restrict__ rank_of, int *__restrict__ x_of,
                             float *__restrict__ pw, float *__restrict__ pwr, float *__restrict__ Lx) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n_angles * g.n_p) return;
    const int a = i / g.n_p, s = s_sorted[i], x = pos[s];
    const size_t o = (size_t)a * g.n_p;
    const double L = Ld[o + s];
    const float w = (float)exp(-L);
    x_of[i] = x;
    pwr[i] = w;
    rank_of[o + x] = i - (int)o;
    pw[o + x] = w;
    Lx[o + x] = (float)L;
}

// ---------------------------------------------------------------- forward stages

// the estimate on the support's bounding box (0 off the emission set)
__global__ void k_flux_box(Geo g, FluxGeo fg, FluxTables ft, const float *__restrict__ f, float *__restrict__ fbox) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
    if (x >= g.n_p) return;
    const int q = ft.sup[x];
    fbox[(size_t)r * fg.nb + ft.box[x]] = q < g.n_q ? f[(size_t)r * g.n_qpad + q] : 0.0f;
}

// I_s(n): one workgroup per (block of 64 scatter points, sector of kSec node
// intervals); its eight waves share the sector's pairs evenly (a sector that
// looks across the object has four times the average, and would be the last to
// end by far).  Every lane visits the same offset, so its direction's weights
// are broadcasts and the eight sums of the current interval's nodes sit in
// registers, moving on by one node per interval; the pair factors stream in as
// written, one per lane.  The waves' nodes overlap and are added in LDS; a
// sector touches kSec + 7 nodes, so even and odd sectors write two separate
// copies (24 nodes each, the rest zero) that the next stage adds.
constexpr int kPairWaves = 8;   // waves of a workgroup of the pair stages
constexpr int kBatch = 8;       // pairs loaded together
constexpr int kChunk = 32;      // pairs whose records a wave holds
constexpr int kSecNodes = kSec + kTap - 1;

__global__ __launch_bounds__(64 * kPairWaves) void k_flux_spread(Geo g, FluxGeo fg, FluxTables ft,
                                                                 const int *__restrict__ beg_all,
                                                                 const int *__restrict__ rec_off,
                                                                 const float *__restrict__ rec_w,
                                                                 const float *__restrict__ sym,
                                                                 const float *__restrict__ fbox, float *__restrict__ I) {
    __shared__ float part[kPairWaves][kSecNodes][64];
    __shared__ __align__(16) float w_s[kPairWaves][kChunk][kTap];
    __shared__ int span[kPairWaves][2];   // nodes that a wave has written
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int sec = blockIdx.y, b = blockIdx.x, r = blockIdx.z;
    const int s = b * 64 + lane;
    const int lin = s < g.n_p ? ft.box[s] : 0;
    const float *__restrict__ fr = fbox + (size_t)r * fg.nb;
    const unsigned top = (unsigned)fg.nb - 1;
    const int bound = beg_all[b * fg.N + sec * kSec + min(lane, kSec)];   // lane i: first record of interval i
    const int first = __builtin_amdgcn_readlane(bound, 0), end = __builtin_amdgcn_readlane(bound, kSec);
    const int share = (end - first + kPairWaves - 1) / kPairWaves;
    const int e0 = min(first + wave * share, end), e1 = min(e0 + share, end);
    // the interval of the wave's first pair
    int k = __popcll(__ballot(lane > 0 && lane < kSec && bound <= e0));
    if (lane == 0) span[wave][0] = k;
    if (e0 < e1) {
        float acc[kTap];
#pragma unroll
        for (int i = 0; i < kTap; ++i) acc[i] = 0.0f;
        int next = __builtin_amdgcn_readlane(bound, k + 1);
        for (int c0 = e0; c0 < e1; c0 += kChunk) {
            // a lane fetches a pair's record: the box offset stays there, to be
            // read back as a scalar, and the weights go to LDS, to be read back
            // as a broadcast, so that the pair loop waits for no scalar load
            const int mine = min(c0 + (lane & (kChunk - 1)), e1 - 1);
            const int off = rec_off[mine];
            const f32x4 *src = reinterpret_cast<const f32x4 *>(rec_w + (size_t)mine * kTap);
            const f32x4 half = src[lane / kChunk];
            __builtin_amdgcn_wave_barrier();
            *reinterpret_cast<f32x4 *>(&w_s[wave][lane & (kChunk - 1)][4 * (lane / kChunk)]) = half;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (read back by the same wave only)
            __builtin_amdgcn_wave_barrier();
            const int n = min(kChunk, e1 - c0);
            const float *__restrict__ sy = sym + (size_t)c0 * 64 + lane;
#pragma unroll 2
            for (int u0 = 0; u0 < n; u0 += kBatch) {
                float y[kBatch], v[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int i = min(u0 + u, n - 1);
                    y[u] = sy[(size_t)i * 64];
                    v[u] = fr[min((unsigned)(lin + __builtin_amdgcn_readlane(off, i)), top)];
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    if (u0 + u < n) {
                        while (c0 + u0 + u >= next) {   // the lowest node is complete: on to the next interval
                            part[wave][k][lane] = acc[0];
#pragma unroll
                            for (int i = 0; i + 1 < kTap; ++i) acc[i] = acc[i + 1];
                            acc[kTap - 1] = 0.0f;
                            ++k;
                            next = __builtin_amdgcn_readlane(bound, k + 1);
                        }
                        const float p = y[u] != 0.0f ? y[u] * v[u] : 0.0f;
#pragma unroll
                        for (int i = 0; i < kTap; ++i) acc[i] = fmaf(w_s[wave][u0 + u][i], p, acc[i]);
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kTap; ++i) part[wave][k + i][lane] = acc[i];
    }
    if (lane == 0) span[wave][1] = e0 < e1 ? k + kTap : 0;
    __syncthreads();
    // directions of flight q -> s are opposite to the offsets s -> q
    const int n0 = sec * kSec - 3 + fg.N / 2;
    const float m = s < g.n_p ? ft.mu_s[s] : 0.0f;
    float *out = I + ((size_t)(r * 2 + (sec & 1)) * fg.N) * fg.np64 + s;
    for (int j = wave; j < 2 * kSec; j += kPairWaves) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < kPairWaves; ++w)
            if (j >= span[w][0] && j < span[w][1]) t += part[w][j][lane];
        out[(size_t)wrap(n0 + j, fg.N) * fg.np64] = m * t;
    }
}

// S_as(k) and P_as of a chunk of (realisation, angle) slots, in rank order:
// C[s][k] = sum_n A[s][n] G_a[n][k] on v_mfma_f32_16x16x4_f32 with
// A = I psi e^(-rho L) formed in the operand registers.  One workgroup: 32
// scatter points x NT tiles of 16 energy nodes, its eight waves an eighth of
// the directions each, added in LDS: one wave's share is a chain of loads from
// the L2, and a small problem has few workgroups.
constexpr int kSpecTiles = 6;   // most 16-node tiles of one workgroup
constexpr int kSpecWaves = 8;

template <int NT>
__global__ __launch_bounds__(64 * kSpecWaves) void k_flux_spectra(Geo g, FluxGeo fg, FluxTables ft,
                                                                  const int *__restrict__ alist, int n_list, int per,
                                                                  int slot0, const float *__restrict__ I, const float *__restrict__ f,
                                                                  float *__restrict__ S, float *__restrict__ SP) {
    __shared__ f32x4 red[kSpecWaves / 2][2 * NT][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = lane & 15, q = lane >> 4;
    // items: point tiles, all of a realisation's angles in turn (per: its slots here)
    const int n_s = (g.n_p + 31) / 32, item = xcd_logical(blockIdx.x, gridDim.x);
    const int grp = item / (n_s * per), tile_s = (item - grp * n_s * per) / per;
    const int s0 = tile_s * 32, ls = grp * per + (item - (grp * n_s + tile_s) * per), slot = slot0 + ls;
    const int r = slot / n_list, a = alist[slot - r * n_list];
    const int kb = blockIdx.y * 16 * NT, n_kt = min(NT, (fg.K - kb) / 16);
    const int *rank = ft.rank_of + (size_t)a * g.n_p;
    if (blockIdx.y == 0 && threadIdx.x < 32) {
        const int s = s0 + threadIdx.x;
        if (s < g.n_p) {
            const int p = ft.sup[s];
            SP[(size_t)ls * g.n_p + rank[s]] = p < g.n_q ? f[(size_t)r * g.n_qpad + p] * ft.pw[(size_t)a * g.n_p + s] : 0.0f;
        }
    }
    const float *I0 = I + (size_t)r * 2 * fg.N * fg.np64 + s0 + c, *I1 = I0 + (size_t)fg.N * fg.np64;
    const float *psi = ft.psi + (size_t)a * fg.N, *rho = ft.rho + (size_t)a * fg.N;
    const float *G = ft.G + (size_t)a * fg.N * fg.K + kb + c;
    float L[2];
    f32x4 acc[2][NT];
    int tile[NT];   // (a last part may have fewer tiles: the rest repeat its last and are dropped)
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) tile[kt] = 16 * min(kt, n_kt - 1);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        L[t] = ft.Lx[(size_t)a * g.n_p + min(s0 + 16 * t + c, g.n_p - 1)];
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) acc[t][kt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // N is a multiple of 48: groups of four directions go round the waves
    // three at a time, so that a wave has all operands of 12 in flight
    for (int n1 = wave * 12; n1 < fg.N; n1 += 12 * kSpecWaves) {
        float ps[3], rh[3], gv[3][NT], iv[3][2];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int n = n1 + 4 * j + q;
            ps[j] = psi[n];
            rh[j] = rho[n];
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) gv[j][kt] = G[(unsigned)(n * fg.K + tile[kt])];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const unsigned at = (unsigned)n * fg.np64 + 16 * t;   // np64 covers whole groups of 32
                iv[j][t] = I0[at] + I1[at];
            }
        }
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const float av = iv[j][t] * ps[j] * __builtin_amdgcn_exp2f(rh[j] * L[t]);
#pragma unroll
                for (int kt = 0; kt < NT; ++kt)
                    acc[t][kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, gv[j][kt], acc[t][kt], 0, 0, 0);
            }
    }
    if (wave >= kSpecWaves / 2) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) red[wave - kSpecWaves / 2][t * NT + kt][lane] = acc[t][kt];
    }
    __syncthreads();
    if (wave < kSpecWaves / 2) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) red[wave][t * NT + kt][lane] += acc[t][kt];
    }
    __syncthreads();
    for (int i = wave; i < 2 * NT; i += kSpecWaves) {
        const int t = i / NT, kt = i - t * NT;
        if (kt >= n_kt) continue;
        const f32x4 v = (red[0][i][lane] + red[1][i][lane]) + (red[2][i][lane] + red[3][i][lane]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int s = s0 + 16 * t + 4 * q + j;
            if (s < g.n_p) S[((size_t)ls * g.n_p + rank[s]) * fg.K + kb + 16 * kt + c] = v[j];
        }
    }
}

// position response (times Z_K): offset in FP64, response in FP32, as the
// term-by-term kernel evaluates it
__device__ __forceinline__ float response(double d, float inv2s2, float edge) {
    const float x = (float)d;
    return fmaxf(__expf(-x * x * inv2s2) - edge, 0.0f);
}

// Event means on the matrix cores.  Events come in blocks of 64 neighbours in
// position, ordered by energy within a block; a wave takes 16 of them:
// V[k][j] = sum_s S_as(k) K_js over the ends that any of them reaches and the
// 16-node tiles that their eight nodes touch, then mean_j = sum_k l_k(E_j) V[k][j].
// The spectra are the A operand, the responses, formed in registers (one per
// end and event), the B operand: a lane's sums then all belong to one event,
// its weights are read four nodes at a time from a row with zeros around the
// eight, and three additions end the sum.  16 events share each read of the
// spectra, and the energy order keeps a wave's nodes to two or three tiles.
//
// SPLIT waves share the ends of 16 events (kSplitEnds); the waves of a workgroup
// that work on the same ends read the same spectra.  It is bound by its vector
// instructions: 200k events of 12 to 20 ends in 15 us, where a branch per tile
// in the inner loop cost as much again.
constexpr int kMaxTiles = kFluxMaxK / 16;
constexpr int kEvRow = 28;   // floats of an event's row in LDS: head 8, zeros 4, weights 8, zeros 4

// minimum and maximum over 16 lanes
__device__ __forceinline__ int dpp(int x, const int ctrl) {
    switch (ctrl) {
        case 0: return __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xf, 0xf, false);    // lane ^ 1
        case 1: return __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xf, 0xf, false);    // lane ^ 2
        case 2: return __builtin_amdgcn_update_dpp(x, x, 0x141, 0xf, 0xf, false);   // 7 - lane of 8
        default: return __builtin_amdgcn_update_dpp(x, x, 0x140, 0xf, 0xf, false);  // 15 - lane of 16
    }
}

template <int SPLIT>
__global__ __launch_bounds__(256 * SPLIT) void k_flux_means(Geo g, FluxGeo fg, const FluxEvent *__restrict__ ev,
                                                    const FluxBlock *__restrict__ blk,
                                                    const double *__restrict__ us_sorted,
                                                    const int *__restrict__ alist, int n_list, int slot_base, int slot0,
                                                    int row0, int row_base, const float *__restrict__ S,
                                                    const float *__restrict__ SP, float *__restrict__ mean,
                                                    float *__restrict__ inv, unsigned long long *__restrict__ skipped) {
    static_assert(sizeof(FluxEvent) == 64 && kTap == 8, "four 16-byte pieces: head, ranks, weights");
    constexpr int WAVES = 4 * SPLIT;
    __shared__ __align__(16) float ev_s[WAVES][16][kEvRow];
    __shared__ double us_s[WAVES][64];
    __shared__ float pr_s[WAVES][64], sum_s[WAVES][16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = lane & 15, q = lane >> 4;
    const int item = xcd_logical(blockIdx.x, gridDim.x);   // (runs of slots: their spectra)
    const FluxBlock bk = blk[item];
    const int part = wave / 4, i0 = 16 * (wave % 4);   // the wave's share of the ends, its first event in the block
    const bool idle = i0 >= bk.n;
    if (SPLIT == 1 && idle) return;
    const int slot = bk.slot - slot_base, ls = slot - slot0, r = slot / n_list;
    const size_t ao = (size_t)alist[slot - r * n_list] * g.n_p;
    const double *us = us_sorted + ao;
    {
        const f32x4 *src = reinterpret_cast<const f32x4 *>(ev + (bk.row + min(i0 + (lane >> 2), bk.n - 1) - row0));
        const int piece = lane & 3;
        const f32x4 v = src[piece];
        float *row = ev_s[wave][lane >> 2];
        *reinterpret_cast<f32x4 *>(row + 4 * piece + (piece >= 2 ? 4 : 0)) = v;
        if (piece < 2) *reinterpret_cast<f32x4 *>(row + (piece ? 20 : 8)) = f32x4{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (read back by the same wave only)
        __builtin_amdgcn_wave_barrier();
    }
    const FluxEvent &e = *reinterpret_cast<const FluxEvent *>(ev_s[wave][c]);   // (its weights lie four floats on)
    const double u = e.u;
    const int et = e.et;
    // the wave's ranks and tiles (energies ascend)
    int r0 = e.r0, r1 = e.r1;
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        r0 = min(r0, dpp(r0, o));
        r1 = max(r1, dpp(r1, o));
    }
    r0 = __builtin_amdgcn_readfirstlane(r0);
    r1 = __builtin_amdgcn_readfirstlane(r1);
    const int t0 = __builtin_amdgcn_readlane(et, 0) >> 4, t1 = (__builtin_amdgcn_readlane(et, 15) + kTap - 1) >> 4;
    if (SPLIT > 1) {   // this wave's share
        const int per = ((r1 - r0 + SPLIT - 1) / SPLIT + 3) & ~3;
        r0 = min(r0 + part * per, r1);
        r1 = idle ? r0 : min(r0 + per, r1);
    }
    const float inv2s2 = (float)(1.0 / (2.0 * g.sig_u * g.sig_u));
    const float edge = expf(-4.5f);
    const float *Sr = S + (size_t)ls * g.n_p * fg.K, *Pr = SP + (size_t)ls * g.n_p;
    const unsigned K = fg.K, last = (unsigned)(r1 - 1) * K + c;
    float total = 0.0f, prim = 0.0f;   // of this lane's event and nodes
    // NT tiles from tb on (a compile-time count: no branch between a rank's loads
    // and products)
    auto tiles = [&](auto count, int tb) {
        constexpr int NT = decltype(count)::value;
        f32x4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        const float *Sc = Sr + 16 * tb;
        // path ends go to LDS 64 at a time, those past the wave's out of
        // reach; 16 ranks' spectra are read before the first is used
#pragma unroll 1
        for (int kc = r0; kc < r1; kc += 64) {
            const int kl = min(kc + lane, r1 - 1);
            const double ul = kc + lane < r1 ? us[kl] : 1e30;
            const float pl = tb == t0 ? Pr[kl] : 0.0f;   // (the primary paths once)
            __builtin_amdgcn_wave_barrier();
            us_s[wave][lane] = ul;
            pr_s[wave][lane] = pl;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (read back by the same wave only)
            __builtin_amdgcn_wave_barrier();
            const int n = min(64, r1 - kc);
            unsigned at = (unsigned)(kc + q) * K + c;
#pragma unroll 1
            for (int k0 = 0; k0 < n; k0 += 16) {
                float sv[4][NT];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned o = min(at, last);
                    at += 4 * K;
#pragma unroll
                    for (int t = 0; t < NT; ++t) sv[j][t] = Sc[o + 16 * t];
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = k0 + 4 * j + q;
                    const float kv = response(u - us_s[wave][k], inv2s2, edge);
                    prim = fmaf(kv, pr_s[wave][k], prim);
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(sv[j][t], kv, acc[t], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int d = 16 * (tb + t) + 4 * q - et;   // of the lane's first node in the event's eight
            const float *w = &ev_s[wave][c][12 + min(max(d, -4), kTap)];
#pragma unroll
            for (int v = 0; v < 4; ++v) total = fmaf(w[v], acc[t][v], total);
        }
    };
    for (int tb = t0; tb <= t1; tb += 3) {
        if (t1 - tb >= 2) tiles(std::integral_constant<int, 3>(), tb);
        else if (t1 - tb == 1) tiles(std::integral_constant<int, 2>(), tb);
        else tiles(std::integral_constant<int, 1>(), tb);
    }
    float s = fmaf(prim, e.g0, total);
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (SPLIT > 1) {
        if (lane < 16) sum_s[wave][c] = s;
        __syncthreads();
        if (part || idle) return;
#pragma unroll
        for (int p = 1; p < SPLIT; ++p) s += sum_s[wave + 4 * p][c];
    }
    int dead = 0;
    if (q == 0 && i0 + c < bk.n) {
        s *= fg.inv_zk;
        const int j = e.row - row_base;
        mean[j] = s;
        dead = !(s > 1e-30f);
        inv[bk.row + i0 + c - row_base] = dead ? 0.0f : 1.0f / s;   // (in record order, as the adjoint reads it)
    }
    const unsigned long long m = __ballot(dead);
    if (lane == 0 && m) atomicAdd(skipped, (unsigned long long)__popcll(m));
}

// primary paths only: LPE lanes per event, the primary weights formed here
template <int LPE>
__global__ __launch_bounds__(256) void k_flux_means_primary(Geo g, FluxGeo fg, FluxTables ft,
                                                            const FluxEvent *__restrict__ ev,
                                                            const double *__restrict__ us_sorted,
                                                            const int *__restrict__ s_sorted,
                                                            const int *__restrict__ alist, int n_list, int slot_base,
                                                            int j0, int j1, int row0, int row_base,
                                                            const float *__restrict__ f, float *__restrict__ mean,
                                                            float *__restrict__ inv,
                                                            unsigned long long *__restrict__ skipped) {
    const int sub = threadIdx.x % LPE;
    const int i = j0 + (blockIdx.x * 256 + threadIdx.x) / LPE;
    int dead = 0;
    if (i < j1) {
        const FluxEvent e = ev[i - row0];
        const int slot = e.slot - slot_base, r = slot / n_list;
        const size_t ao = (size_t)alist[slot - r * n_list] * g.n_p;
        const double *us = us_sorted + ao;
        const float inv2s2 = (float)(1.0 / (2.0 * g.sig_u * g.sig_u));
        const float edge = expf(-4.5f);
        const float *fr = f + (size_t)r * g.n_qpad;
        float s = 0.0f;
#pragma unroll 4
        for (int k = e.r0 + sub; k < e.r1; k += LPE) {
            const int p = s_sorted[ao + k];
            const float h = p < g.n_q ? fr[p] * ft.pwr[ao + k] : 0.0f;
            s = fmaf(response(e.u - us[k], inv2s2, edge), h, s);
        }
#pragma unroll
        for (int o = LPE / 2; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
        if (sub == 0) {
            s *= e.g0 * fg.inv_zk;
            const int j = e.row - row_base;
            mean[j] = s;
            dead = !(s > 1e-30f);
            inv[i - row_base] = dead ? 0.0f : 1.0f / s;   // (in record order)
        }
    }
    const unsigned long long m = __ballot(dead);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(skipped, (unsigned long long)__popcll(m));
}

// ---------------------------------------------------------------- adjoint stages

// first block in [lo, hi) whose last position is past v (FIRST: whose first
// position is at or past v), by 64-way steps: every lane of the wave takes
// part and gets the same answer
template <bool FIRST>
__device__ __forceinline__ int wave_search(const FluxBlock *blk, int lo, int hi, double v, int lane) {
    while (hi > lo) {
        const int step = (hi - lo + 63) / 64, at = min(lo + lane * step + step - 1, hi - 1);
        const unsigned long long m = __ballot(FIRST ? blk[at].u0 >= v : blk[at].u1 > v);
        if (m == 0) return hi;
        const int k = __ffsll((unsigned long long)m) - 1;
        hi = min(lo + k * step + step - 1, hi - 1);   // this one is past v; the answer is at most here
        lo = lo + k * step;
        if (step == 1) return hi;
    }
    return lo;
}

// R_as(k) = sum_j w_j K_js l_k(E_j) (and the primary's R0 = sum_j w_j K_js g0_j)
// of 16 path ends of one slot on the matrix cores: the workgroup's four waves
// walk the event blocks that reach any of its ends, every fourth block each,
// four events per product (A: responses of 16 ends to four events; B: the
// events' interpolation weights spread over a 16-node tile).  The events'
// energy order within a block makes those that touch a tile neighbours: per
// tile, one loop without branches over their groups of four.  (A tile test per
// group instead cost five scalar instructions and an LDS wait a product.)
// Every sum has one owner and a fixed order.  Rows are written in flux order.
template <int TILES>
__global__ __launch_bounds__(256) void k_flux_adjoint(Geo g, FluxGeo fg, FluxTables ft, const FluxEvent *__restrict__ ev,
                                                      const FluxBlock *__restrict__ blk,
                                                      const double *__restrict__ us_sorted,
                                                      const int *__restrict__ alist, const int *__restrict__ blk_beg,
                                                      int n_list, int slot0, int row_base,
                                                      const float *__restrict__ wgt, float *__restrict__ R,
                                                      float *__restrict__ R0) {
    constexpr int NT = TILES > 0 ? TILES : 1;
    constexpr int kRow = kTap + 3;   // a zero, the weights, a zero (odd: rows start at different banks)
    union Shared {
        struct {
            float w[4][TILES > 0 ? 64 : 1][kRow];   // weight times interpolation weights
            float kv[4][TILES > 0 ? 16 : 1][64];    // responses, [group of four events][lane]
            double u[4][64];
            float p[4][64];         // weight times the primary's energy response
            int et[4][64];
        } in;
        f32x4 red[3][NT][64];
    };
    __shared__ __align__(16) Shared sh;
    __shared__ float red0[4][16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 15, q = lane >> 4;
    const int item = xcd_logical(blockIdx.x, gridDim.x), n_k = (g.n_p + 15) / 16;   // (runs of slots: their events)
    const int ls = item / n_k, slot = slot0 + ls;
    const int r = slot / n_list, a = alist[slot - r * n_list];
    const double *us = us_sorted + (size_t)a * g.n_p;
    const int *x_of = ft.x_of + (size_t)a * g.n_p;
    const int k0 = (item - ls * n_k) * 16, rank = min(k0 + c, g.n_p - 1);
    const double my_u = us[rank], reach = 3.0 * g.sig_u;
    const int b0 = wave_search<false>(blk, blk_beg[slot], blk_beg[slot + 1], us[k0] - reach, lane);
    const int b1 = wave_search<true>(blk, b0, blk_beg[slot + 1], us[min(k0 + 15, g.n_p - 1)] + reach, lane);
    const float inv2s2 = (float)(1.0 / (2.0 * g.sig_u * g.sig_u));
    const float edge = expf(-4.5f);
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float r0 = 0.0f;
    if (TILES > 0) sh.in.w[wave][lane][0] = sh.in.w[wave][lane][kTap + 1] = 0.0f;
    // the next block's records and weights are on their way while the current
    // one is used, and the one's after it known
    FluxBlock bk = blk[min(b0 + wave, max(b1 - 1, 0))], next = bk;
    FluxEvent e;
    float y = 0.0f;
    auto load = [&](const FluxBlock &k) {
        const int at = k.row + min(lane, k.n - 1);
        e = ev[at];
        y = wgt[at - row_base];
    };
    if (b0 + wave < b1) {
        load(bk);
        next = blk[min(b0 + wave + 4, b1 - 1)];
    }
    for (int b = b0 + wave; b < b1; b += 4) {
        y = lane < bk.n ? y * fg.inv_zk : 0.0f;
        const int et = e.et, n = bk.n;
        __builtin_amdgcn_wave_barrier();
        sh.in.u[wave][lane] = e.u;
        sh.in.p[wave][lane] = y * e.g0;
        if (TILES > 0) {
#pragma unroll
            for (int i = 0; i < kTap; ++i) sh.in.w[wave][lane][1 + i] = y * e.w[i];
            sh.in.et[wave][lane] = e.et;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (read back by the same wave only)
        __builtin_amdgcn_wave_barrier();
        bk = next;
        if (b + 4 < b1) {
            load(bk);
            next = blk[min(b + 8, b1 - 1)];
        }
        const int groups = (n + 3) / 4;
#pragma unroll 4
        for (int k = 0; k < groups; ++k) {
            const int i = 4 * k + q;
            const float kv = response(sh.in.u[wave][i] - my_u, inv2s2, edge);
            r0 = fmaf(kv, sh.in.p[wave][i], r0);
            if (TILES > 0) sh.in.kv[wave][k][lane] = kv;
        }
        if (TILES > 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                // the events that touch the tile: neighbours (energies ascend)
                const unsigned long long m = __ballot(lane < n && et < 16 * (t + 1) && et + kTap > 16 * t);
                if (m == 0) continue;
                const int g1 = (63 - __clzll(m)) / 4;
#pragma unroll 4
                for (int k = (__ffsll(m) - 1) / 4; k <= g1; ++k) {
                    const int i = 4 * k + q;
                    const int d = 16 * t + c - sh.in.et[wave][i];
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(sh.in.kv[wave][k][lane],
                                                                  sh.in.w[wave][i][min(max(d, -1), kTap) + 1], acc[t], 0, 0, 0);
                }
            }
        }
    }
    r0 += __shfl_xor(r0, 16, 64);
    r0 += __shfl_xor(r0, 32, 64);
    if (lane < 16) red0[wave][c] = r0;
    __syncthreads();
    if (TILES > 0 && wave > 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t) sh.red[wave - 1][t][lane] = acc[t];
    }
    __syncthreads();
    if (wave) return;
    if (lane < 16 && k0 + c < g.n_p)
        R0[(size_t)ls * g.n_p + x_of[k0 + c]] = (red0[0][c] + red0[1][c]) + (red0[2][c] + red0[3][c]);
    if (TILES == 0) return;
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = (acc[t] + sh.red[0][t][lane]) + (sh.red[1][t][lane] + sh.red[2][t][lane]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int k = k0 + 4 * q + v;
        if (k >= g.n_p) continue;
        float *row = R + ((size_t)ls * g.n_p + x_of[k]) * fg.K + c;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (16 * t < fg.K) row[16 * t] = acc[t][v];
    }
}

// T_s(n) = mu(s) sum_a psi_a(n) e^(-rho_a(n) L_a(s)) sum_k G_a[n][k] R_as(k),
// over the chunk's angles of one realisation (added to the stored field from
// the second chunk on), and the primary paths' share of the backprojection.
// One workgroup: 32 directions x 32 scatter points, its eight waves every
// eighth angle each, added in LDS; the energy sum on the matrix cores with
// both operands read as float4 along k (lane group q takes k = 16 i + 4 q + v
// in step v).  T holds groups of four directions, [group][box pixel][4], group
// 0 directions -4 .. -1 and the last N .. N + 3, so that the next stage reads
// eight neighbours in two or three wide loads and without wrapping.
__host__ __device__ inline int field_groups(const FluxGeo &fg) { return fg.N / 4 + 2; }

constexpr int kFieldWaves = 8;

__global__ __launch_bounds__(64 * kFieldWaves) void k_flux_fields(Geo g, FluxGeo fg, FluxTables ft, const int *__restrict__ alist,
                                                     int n_list, int slot0, int n_slots, const float *__restrict__ R,
                                                     const float *__restrict__ R0, float *__restrict__ T,
                                                     float *__restrict__ pb) {
    __shared__ f32x4 red[kFieldWaves][4][64];   // [wave][direction tile * 2 + point tile]
    __shared__ float red0[kFieldWaves][32];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = lane & 15, q = lane >> 4;
    // items: point tiles, all directions in turn (they share the tile's rows of R)
    const int n_n = (fg.N + 31) / 32, n_s = (g.n_p + 31) / 32, item = xcd_logical(blockIdx.x, gridDim.x);
    const int z = item / (n_s * n_n), tile_s = (item - z * n_s * n_n) / n_n, tile_n = item - (z * n_s + tile_s) * n_n;
    const int n0 = tile_n * 32, s0 = tile_s * 32;
    const int s[2] = {min(s0 + c, g.n_p - 1), min(s0 + 16 + c, g.n_p - 1)};
    const int r = slot0 / n_list + z;
    const int a_lo = max(0, slot0 - r * n_list), a_hi = min(n_list, slot0 + n_slots - r * n_list);
    const bool two = n0 + 16 < fg.N;   // N is a multiple of 16
    f32x4 tot[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) tot[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
    float prim[2] = {0.0f, 0.0f};
    for (int ai = a_lo + wave; ai < a_hi; ai += kFieldWaves) {
        const int a = alist[ai], ls = r * n_list + ai - slot0;
        const float *R1 = R + ((size_t)ls * g.n_p + s[0]) * fg.K + 4 * q, *R2 = R + ((size_t)ls * g.n_p + s[1]) * fg.K + 4 * q;
        const float *G1 = ft.G + ((size_t)a * fg.N + n0 + c) * fg.K + 4 * q, *G2 = two ? G1 + (size_t)16 * fg.K : G1;
        float L[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            L[u] = ft.Lx[(size_t)a * g.n_p + s[u]];
            if (tile_n == 0) prim[u] = fmaf(ft.pw[(size_t)a * g.n_p + s[u]], R0[(size_t)ls * g.n_p + s[u]], prim[u]);
        }
        f32x4 acc[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 5
        for (int k = 0; k < fg.K; k += 16) {
            const f32x4 r1 = *reinterpret_cast<const f32x4 *>(R1 + k), r2 = *reinterpret_cast<const f32x4 *>(R2 + k);
            const f32x4 g1 = *reinterpret_cast<const f32x4 *>(G1 + k), g2 = *reinterpret_cast<const f32x4 *>(G2 + k);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(g1[v], r1[v], acc[0][0], 0, 0, 0);
                acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(g1[v], r2[v], acc[0][1], 0, 0, 0);
                acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(g2[v], r1[v], acc[1][0], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(g2[v], r2[v], acc[1][1], 0, 0, 0);
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t == 1 && !two) continue;
            const f32x4 ps = *reinterpret_cast<const f32x4 *>(ft.psi + (size_t)a * fg.N + n0 + 16 * t + 4 * q);
            const f32x4 rh = *reinterpret_cast<const f32x4 *>(ft.rho + (size_t)a * fg.N + n0 + 16 * t + 4 * q);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    tot[t][u][v] = fmaf(acc[t][u][v], ps[v] * __builtin_amdgcn_exp2f(rh[v] * L[u]), tot[t][u][v]);
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) red[wave][2 * t + u][lane] = tot[t][u];
    if (q == 0) {
        red0[wave][c] = prim[0];
        red0[wave][16 + c] = prim[1];
    }
    __syncthreads();
    const bool first = a_lo == 0;
    if (tile_n == 0 && threadIdx.x < 32 && s0 + threadIdx.x < g.n_p) {
        const int i = threadIdx.x, p = ft.sup[s0 + i];
        if (p < g.n_q) {
            float *o = pb + (size_t)r * (fg.N / kSec + 1) * g.n_qpad + p;
            const float v = ((red0[0][i] + red0[1][i]) + (red0[2][i] + red0[3][i])) +
                            ((red0[4][i] + red0[5][i]) + (red0[6][i] + red0[7][i]));
            *o = first ? v : *o + v;
        }
    }
    if (wave >= 4) return;
    // wave w finishes direction tile w / 2, point tile w % 2
    const int t = wave >> 1, x = s0 + 16 * (wave & 1) + c;
    if ((t == 1 && !two) || x >= g.n_p) return;
    const f32x4 v = ((red[0][wave][lane] + red[1][wave][lane]) + (red[2][wave][lane] + red[3][wave][lane])) +
                    ((red[4][wave][lane] + red[5][wave][lane]) + (red[6][wave][lane] + red[7][wave][lane]));
    const float m = ft.mu_s[x];
    f32x4 *Tr = reinterpret_cast<f32x4 *>(T) + (size_t)r * field_groups(fg) * fg.nb + ft.box[x];
    const int d = n0 / 4 + 4 * t + q;   // directions 4 d .. 4 d + 3: group d + 1
    f32x4 *o = Tr + (size_t)(d + 1) * fg.nb;
    f32x4 y = first ? f32x4{0.f, 0.f, 0.f, 0.f} : *o;
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = fmaf(m, v[i], y[i]);
    *o = y;
    if (d == 0) o[(size_t)(fg.N / 4) * fg.nb] = y;
    if (d == fg.N / 4 - 1) *Tr = y;
}

// b_q: one workgroup per (block of 64 emission pixels, sector), as
// k_flux_spread with the sums the other way round: the field's eight nodes
// around each offset's direction, read along the pixels.  Interval n takes
// directions n - 3 .. n + 4, values (n + 1) % 4 .. + 7 of the groups from
// (n + 1) / 4 on: three float4 loads and twelve weights (zeros around the
// eight).  Eight separate rows asked the vector cache for as many cycles but
// for three times the lines, which then had to come from the L2 again for the
// next offset.  The same lines serve neighbours in the pair order, so sixteen
// waves walk it together, two pairs each in turn: what they read at a time
// should fit the vector cache, and the misses still bound it.  135 us for 688k
// pair rows of 64 at 128x128, 19 us for 55k at 64x64 (eight waves of four: 162
// and 24, of two: 158 and 25; sixteen of four: 146 and 22, of one: 147 and 23; a
// run of its own for each wave: 176 and 27).  Each XCD takes a run of sectors,
// so that its L2 holds the few directions they read.
constexpr int kGroupTap = 12;
constexpr int kGatherWaves = 16;
constexpr int kGatherBatch = 2;   // pairs that a wave loads together

__global__ __launch_bounds__(64 * kGatherWaves) void k_flux_gather(Geo g, FluxGeo fg, FluxTables ft,
                                                                 const int *__restrict__ beg_all,
                                                                 const int *__restrict__ rec_off,
                                                                 const int *__restrict__ rec_n,
                                                                 const float *__restrict__ rec_w,
                                                                 const float *__restrict__ sym,
                                                                 const float *__restrict__ T, float *__restrict__ pb) {
    __shared__ float sum[kGatherWaves][64];
    __shared__ __align__(16) float w_s[kGatherWaves][kChunk][kGroupTap];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int item = xcd_logical(blockIdx.x, gridDim.x);
    const int sec = item / fg.n_blk, b = item - sec * fg.n_blk, r = blockIdx.y;
    const int x = b * 64 + lane;
    const int lin = x < g.n_p ? ft.box[x] : 0;
    const unsigned top = (unsigned)fg.nb - 1;
    const size_t nb = fg.nb;
    float acc = 0.0f;
    const int start = beg_all[b * fg.N + sec * kSec], end = beg_all[b * fg.N + (sec + 1) * kSec];
    const f32x4 *__restrict__ Tr = reinterpret_cast<const f32x4 *>(T) + (size_t)r * field_groups(fg) * nb;
    // kGatherBatch neighbours at a time go round the waves
    constexpr int kB = kGatherBatch;
    for (int c0 = start + kB * wave; c0 < end; c0 += kGatherWaves * kChunk) {
        const int l = lane & (kChunk - 1), mine = min(c0 + kB * kGatherWaves * (l / kB) + l % kB, end - 1);
        const int off = rec_off[mine], m1 = rec_n[mine] + 1;
        const f32x4 *src = reinterpret_cast<const f32x4 *>(rec_w + (size_t)mine * kTap);
        const f32x4 lo = src[0], hi = src[1];
        __builtin_amdgcn_wave_barrier();
        if (lane < kChunk) {
            float *w = w_s[wave][lane] + (m1 & 3);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w[i] = lo[i];
                w[4 + i] = hi[i];
            }
            // the four places around the eight
#pragma unroll
            for (int i = 0; i < 4; ++i) w_s[wave][lane][i < (m1 & 3) ? i : 8 + i] = 0.0f;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (read back by the same wave only)
        __builtin_amdgcn_wave_barrier();
        const float *__restrict__ sy = sym + (size_t)c0 * 64 + lane;
#pragma unroll 1
        for (int u0 = 0; u0 < kChunk; u0 += kB) {
            const int at0 = kGatherWaves * u0, left = end - c0 - at0;   // (records of this batch and after)
            if (left <= 0) break;
            float y[kB];
            f32x4 t[kB][3];
#pragma unroll
            for (int u = 0; u < kB; ++u) {
                const int m = __builtin_amdgcn_readlane(m1, u0 + u);
                y[u] = u < left ? sy[(size_t)(at0 + u) * 64] : 0.0f;
                const unsigned at = min((unsigned)(lin + __builtin_amdgcn_readlane(off, u0 + u)), top);
                const f32x4 *__restrict__ T0 = Tr + (size_t)(m >> 2) * nb;
                t[u][0] = T0[at];
                t[u][1] = (T0 + nb)[at];
                t[u][2] = (T0 + (m & 3 ? 2 * nb : nb))[at];   // (all eight in two groups: no third)
            }
#pragma unroll
            for (int u = 0; u < kB; ++u) {
                const float *wu = w_s[wave][u0 + u];
                float v = 0.0f;
#pragma unroll
                for (int j = 0; j < kGroupTap; ++j) v = fmaf(wu[j], t[u][j >> 2][j & 3], v);
                acc = y[u] != 0.0f ? fmaf(y[u], v, acc) : acc;
            }
        }
    }
    sum[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && x < g.n_p) {
        const int p = ft.sup[x];
        float v[kGatherWaves];
#pragma unroll
        for (int w = 0; w < kGatherWaves; ++w) v[w] = sum[w][lane];
        if (p < g.n_q) pb[((size_t)r * (fg.N / kSec + 1) + 1 + sec) * g.n_qpad + p] = pair_sum(v);
    }
}

// the primary paths' backprojection without scatter: per angle chunk of one
// realisation (added to the stored row from the second chunk on)
__global__ __launch_bounds__(256) void k_flux_primary_back(Geo g, FluxTables ft, const int *__restrict__ alist,
                                                           int n_list, int slot0, int n_slots,
                                                           const float *__restrict__ R0, float *__restrict__ pb) {
    __shared__ float part[4][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, x = blockIdx.x * 64 + lane;
    const int r = slot0 / n_list + blockIdx.y;
    const int a_lo = max(0, slot0 - r * n_list), a_hi = min(n_list, slot0 + n_slots - r * n_list);
    float s = 0.0f;
    if (x < g.n_p)
#pragma unroll 4
        for (int ai = a_lo + wave; ai < a_hi; ai += 4)
            s = fmaf(ft.pw[(size_t)alist[ai] * g.n_p + x], R0[(size_t)(r * n_list + ai - slot0) * g.n_p + x], s);
    part[wave][lane] = s;
    __syncthreads();
    if (wave || x >= g.n_p) return;
    const int p = ft.sup[x];
    if (p >= g.n_q) return;
    float *o = pb + (size_t)r * g.n_qpad + p;
    const float v = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
    *o = a_lo == 0 ? v : *o + v;
}

// the primary paths' backprojection b and f <- f b / sens at once (BACK: b
// itself), where one chunk holds every slot: without scatter a sub-iteration is
// a few short kernels, and this saves one of four (7.5 -> 3.7 us)
template <bool BACK>
__global__ __launch_bounds__(256) void k_flux_primary_update(Geo g, FluxTables ft, const int *__restrict__ alist,
                                                             int n_list, const float *__restrict__ R0,
                                                             const float *__restrict__ sens, float *__restrict__ f) {
    __shared__ float part[4][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, x = blockIdx.x * 64 + lane, r = blockIdx.y;
    float s = 0.0f;
    if (x < g.n_p)
#pragma unroll 4
        for (int ai = wave; ai < n_list; ai += 4)
            s = fmaf(ft.pw[(size_t)alist[ai] * g.n_p + x], R0[(size_t)(r * n_list + ai) * g.n_p + x], s);
    part[wave][lane] = s;
    __syncthreads();
    if (wave || x >= g.n_p) return;
    const int p = ft.sup[x];
    if (p >= g.n_q) return;
    const float b = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
    float *fp = f + (size_t)r * g.n_qpad + p;
    if (BACK) {
        *fp = b;
        return;
    }
    const float se = sens[p], v = *fp;
    *fp = se > 0.0f ? (v * b) / se : v;
}

// f <- f b / sens with b the sum of the realisation's partial rows (the
// primary's first), and the box copy of the new estimate; BACK: b itself.
// Summed in pairs: one row after the other left 3.0e-7 of the estimate after
// eight sub-iterations at 64x64, pairs 1.8e-7, at the same time (in FP64 1.2e-7,
// but 5 us a sub-iteration more).
template <bool BACK>
__global__ void k_flux_update(Geo g, FluxGeo fg, FluxTables ft, int rows, const float *__restrict__ pb,
                              const float *__restrict__ sens, float *__restrict__ f, float *__restrict__ fbox) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
    if (x >= g.n_p) return;
    const int q = ft.sup[x];
    if (q >= g.n_q) return;
    const float *p = pb + (size_t)r * rows * g.n_qpad + q;
    float b = 0.0f;
    for (int k0 = 0; k0 < rows; k0 += 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = k0 + k < rows ? p[(size_t)(k0 + k) * g.n_qpad] : 0.0f;
        b += pair_sum(v);
    }
    float *fp = f + (size_t)r * g.n_qpad + q;
    if (BACK) {
        *fp = b;
        return;
    }
    const float s = sens[q];
    float v = *fp;
    if (s > 0.0f) v = (v * b) / s;
    *fp = v;
    if (fg.N) fbox[(size_t)r * fg.nb + ft.box[x]] = v;
}

// the event records of the stages above, from the sorted events: one wave per
// block of 64 neighbours of one slot, their records ordered by energy node.
// blk_beg [slots + 1]: first block of each slot over all subsets' slots,
// slot_row their first rows; base[i] is the first slot of subset i (null: one
// list).  Blocks [b0, b0 + gridDim) go to ev[row - row0].
__global__ __launch_bounds__(64) void k_flux_events(Geo g, FluxGeo fg, FluxFit fit, int b0, int row0,
                                                    const int *__restrict__ slot_row, const int *__restrict__ blk_beg,
                                                    int n_slots, const int *__restrict__ base,
                                                    const int *__restrict__ ang, const float *__restrict__ su,
                                                    const float *__restrict__ se, const double *__restrict__ us_sorted,
                                                    FluxEvent *__restrict__ ev, FluxBlock *__restrict__ blk) {
    __shared__ int key[64];
    const int b = b0 + blockIdx.x, lane = threadIdx.x;
    int lo = 0, hi = n_slots;   // the last slot whose blocks begin at or before b
    while (hi - lo > 1) { const int m = (lo + hi) >> 1; if (blk_beg[m] <= b) lo = m; else hi = m; }
    const int first = slot_row[lo] + 64 * (b - blk_beg[lo]);
    const int n = min(64, slot_row[lo + 1] - first);
    const int row = first + min(lane, n - 1);
    FluxEvent e;
    const int a = ang[row];
    e.slot = lo - (base ? base[a % g.n_subsets] : 0);
    e.row = row;
    e.u = ((double)su[row] - 0.5 * g.n_bins) * g.bin_cm;
    const double en = (double)se[row] + g.e_c;
    // the node interval of the energy and the weights of its eight nodes
    const double t = (en - fg.e_lo) / fg.h;
    e.et = min(max((int)t, 0), max(fg.K - 8, 0));
    if (fg.N) {
        double w[kTap];
        fit_weights(fit, t - e.et, w);
        const double y = en - fg.e_mid;
#pragma unroll
        for (int i = 0; i < kTap; ++i) {
            const double yi = fg.e_lo + (e.et + i - 3) * fg.h - fg.e_mid;
            e.w[i] = (float)(w[i] * exp2(g.c2 * (yi * yi - y * y)));
        }
    }
    const double d0 = en - g.e0;
    e.g0 = (float)(exp2(-g.c2 * d0 * d0) / (sqrt(2.0 * M_PI) * g.sig_e));
    const double *us = us_sorted + (size_t)a * g.n_p;
    const double reach = 3.0 * g.sig_u;
    int l = 0, h = g.n_p;     // first rank with us > u - reach
    while (l < h) { const int m = (l + h) >> 1; if (us[m] > e.u - reach) h = m; else l = m + 1; }
    e.r0 = l;
    h = g.n_p;                // first rank with us >= u + reach
    while (l < h) { const int m = (l + h) >> 1; if (us[m] >= e.u + reach) h = m; else l = m + 1; }
    e.r1 = l;
    key[lane] = e.et;
    __syncthreads();
    int at = 0;
    for (int i = 0; i < n; ++i) at += key[i] < e.et || (key[i] == e.et && i < lane);
    if (lane < n) ev[first + at - row0] = e;
    const double u0 = __shfl(e.u, 0, 64), u1 = __shfl(e.u, n - 1, 64);
    if (lane == 0) blk[b] = FluxBlock{u0, u1, e.slot, first, n, 0};
}

// ---------------------------------------------------------------- sensitivity (once per attenuation map, FP64)
// sens_i(q) = T sum_{a in i} (e^(-L_a(q)) D_a(q) W(e0) + sum_s B(q, s) h_a(s, phi_qs)),
// h_a(s, phi) = Psi/Psi_bar e^(-rho L_a(s)) D_a(s) W(E'): the adjoint stages once
// more, with the window's acceptance in place of the events, in FP64 with the
// FP64 pair factors.  One path walk per (angle, pixel, path end) took 6.4 ms
// on brain64 (75 ms on brain128), most of it exp, log1p and erf; here these
// are evaluated per (angle, direction node, scatter point).

// per (angle, node): Psi/Psi_bar times the window's acceptance, and rho
__global__ void k_flux_sens_angles(Geo g, FluxGeo fg, const double *__restrict__ cs, double2 *__restrict__ tab) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n_angles * fg.N) return;
    const int a = i / fg.N, n = i - a * fg.N;
    const double ph = 2.0 * M_PI * n / fg.N;
    const double c = cos(ph) * cs[2 * a] + sin(ph) * cs[2 * a + 1];
    const double t = 1.0 + g.kappa * (1.0 - c), P = 1.0 / t, ep = g.e0 * P, s2 = M_SQRT2 * g.sig_e;
    const double win = 0.5 * (erf((g.win_hi - ep) / s2) - erf((g.win_lo - ep) / s2));
    tab[i] = make_double2(P * P * (P + t - 1.0 + c * c) / g.psi_bar * win, kn_total(ep) / g.sigma_kn_e0);
}

// U[n + 3][box][C] = mu(s) sum_{a in subset i0 + c} h_a(s, phi_n), direction
// rows -3 .. N + 3 as in the fields
template <int C>
__global__ __launch_bounds__(64) void k_flux_sens_fields(Geo g, FluxGeo fg, FluxTables ft, int i0,
                                                         const double2 *__restrict__ tab,
                                                         const double *__restrict__ Ld,
                                                         const double *__restrict__ D_sorted, double *__restrict__ U) {
    const int x = blockIdx.x * 64 + threadIdx.x, n = blockIdx.y;
    if (x >= g.n_p) return;
    const int s = ft.sup[x];
    double u[C];
#pragma unroll
    for (int c = 0; c < C; ++c) u[c] = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (i0 + c < g.n_subsets)
            for (int a = i0 + c; a < g.n_angles; a += g.n_subsets) {
                const size_t o = (size_t)a * g.n_p;
                const double2 h = tab[a * fg.N + n];
                u[c] += h.x * exp(-h.y * Ld[o + s]) * D_sorted[o + ft.rank_of[o + x]];
            }
    const double m = ft.mu_s[x];
    double *o = U + ((size_t)(n + 3) * fg.nb + ft.box[x]) * C;
    const ptrdiff_t turn = (ptrdiff_t)fg.N * fg.nb * C;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        o[c] = m * u[c];
        if (n < 4) o[c + turn] = m * u[c];
        if (n >= fg.N - 3) o[c - turn] = m * u[c];
    }
}

constexpr int kWaveSec = 3;   // intervals of one wave of the FP64 sensitivities

// part[sector][c][x] of C subsets: one wave per (pixel block, kWaveSec node
// intervals)
template <int C>
__global__ __launch_bounds__(64) void k_flux_sens_pairs(Geo g, FluxGeo fg, FluxTables ft,
                                                        const int *__restrict__ rec_off,
                                                        const double *__restrict__ rec_w,
                                                        const int *__restrict__ p_pix,
                                                        const int *__restrict__ q_of_pix,
                                                        const double *__restrict__ Bt, const double *__restrict__ U,
                                                        double *__restrict__ part) {
    const int b = blockIdx.x, sec = blockIdx.y, lane = threadIdx.x, x = b * 64 + lane;
    const int q = x < g.n_p ? ft.sup[x] : -1;
    const int lin = q >= 0 ? ft.box[x] : 0;
    const unsigned top = (unsigned)fg.nb - 1;
    double acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = 0.0;
    for (int k = 0; k < kWaveSec; ++k) {
        const int n = sec * kWaveSec + k;
        for (int e = ft.beg[b * fg.N + n]; e < ft.beg[b * fg.N + n + 1]; ++e) {
            const unsigned at = min((unsigned)(lin + rec_off[e]), top);
            const bool on = q >= 0 && q < g.n_q && ft.sym[(size_t)e * 64 + lane] != 0.0f;
            if (__ballot(on) == 0) continue;
            double B = 0.0;
            if (on) {
                const int j = (int)at / fg.W, i = (int)at - j * fg.W;
                const int s = q_of_pix[(j + fg.y0) * g.nx + i + fg.x0];
                B = Bt[(size_t)s * g.n_p + q] / (double)ft.mu_box[at];
            }
            double v[C];
#pragma unroll
            for (int c = 0; c < C; ++c) v[c] = 0.0;
#pragma unroll
            for (int i = 0; i < kTap; ++i) {
                const double w = rec_w[(size_t)e * kTap + i];
                const double *u = U + ((size_t)(n + i) * fg.nb + at) * C;
#pragma unroll
                for (int c = 0; c < C; ++c) v[c] = fma(w, u[c], v[c]);
            }
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = on ? fma(B, v[c], acc[c]) : acc[c];
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) part[((size_t)sec * C + c) * fg.np64 + x] = acc[c];
}

// sens of one of C subsets (blockIdx.y): the partial sums and the primary
// paths, kept in FP64 for the sum over subsets; four lanes per pixel
template <int C>
__global__ __launch_bounds__(256) void k_flux_sens_sum(Geo g, FluxGeo fg, FluxTables ft, int i0, int n_part,
                                                       const double *__restrict__ part, const double *__restrict__ Ld,
                                                       const double *__restrict__ D_sorted, float *__restrict__ sens,
                                                       double *__restrict__ sens64) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, x = blockIdx.x * 64 + lane, c = blockIdx.y, i = i0 + c;
    if (i >= g.n_subsets) return;
    const int q = x < g.n_p ? ft.sup[x] : g.n_q;
    double s = 0.0;
    if (q < g.n_q) {
        const double s2 = M_SQRT2 * g.sig_e;
        const double w0 = 0.5 * (erf((g.win_hi - g.e0) / s2) - erf((g.win_lo - g.e0) / s2));
        for (int k = w; k < n_part; k += 4) s += part[((size_t)k * C + c) * fg.np64 + x];
        for (int a = i + w * g.n_subsets; a < g.n_angles; a += 4 * g.n_subsets) {
            const size_t o = (size_t)a * g.n_p;
            s += exp(-Ld[o + q]) * D_sorted[o + ft.rank_of[o + x]] * w0;
        }
    }
    red[w][lane] = s;
    __syncthreads();
    if (w || q >= g.n_q) return;
    s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    sens64[(size_t)i * g.n_q + q] = s;
    sens[(size_t)i * g.n_qpad + q] = (float)(g.acq_time * s);
}

__global__ void k_flux_sens_total(Geo g, const double *__restrict__ sens64, float *__restrict__ sens_all) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= g.n_q) return;
    double s = 0.0;
    for (int i = 0; i < g.n_subsets; ++i) s += sens64[(size_t)i * g.n_q + q];
    sens_all[q] = (float)(g.acq_time * s);
}

template <int C>
static hipError_t sens_subsets(const Geo &g, const FluxGeo &fg, const Tables &t, const FluxTables &ft, const double *w64,
                               const double2 *tab, double *U, double *part, double *total, hipStream_t st) {
    const int n_part = fg.N / kWaveSec;
    for (int i0 = 0; i0 < g.n_subsets; i0 += C) {
        if (fg.N) {
            hipLaunchKernelGGL(k_flux_sens_fields<C>, dim3(fg.n_blk, fg.N), dim3(64), 0, st, g, fg, ft, i0, tab, t.Ld,
                               t.D_sorted, U);
            hipLaunchKernelGGL(k_flux_sens_pairs<C>, dim3(fg.n_blk, n_part), dim3(64), 0, st, g, fg, ft, ft.rec_off, w64,
                               t.p_pix, t.p_pix + g.n_p, t.Bt, U, part);
        }
        hipLaunchKernelGGL(k_flux_sens_sum<C>, dim3(fg.n_blk, C), dim3(256), 0, st, g, fg, ft, i0, n_part, part, t.Ld,
                           t.D_sorted, t.sens, total);
    }
    hipLaunchKernelGGL(k_flux_sens_total, dim3((g.n_q + 63) / 64), dim3(64), 0, st, g, total, t.sens_all);
    return hipGetLastError();
}

// t.sens and t.sens_all (allocated, zero beyond the emission set)
static hipError_t flux_sensitivity(const Geo &g, const FluxGeo &fg, const Tables &t, const FluxTables &ft,
                                   const double *w64, hipStream_t st) {
    const int C = g.n_subsets >= 8 ? 8 : g.n_subsets >= 4 ? 4 : g.n_subsets >= 2 ? 2 : 1;
    double2 *tab = nullptr;
    double *ws = nullptr;
    const size_t nU = fg.N ? (size_t)(fg.N + kTap - 1) * fg.nb * C : 0, nP = (size_t)(fg.N / kWaveSec) * C * fg.np64;
    hipError_t e = launch_fill(t.sens, (size_t)g.n_subsets * g.n_qpad, 0.0f, st);
    if (e == hipSuccess) e = launch_fill(t.sens_all, g.n_qpad, 0.0f, st);
    if (e == hipSuccess && fg.N) e = hipMalloc(&tab, sizeof(double2) * (size_t)g.n_angles * fg.N);
    if (e == hipSuccess) e = hipMalloc(&ws, sizeof(double) * (nU + nP + (size_t)g.n_subsets * g.n_q));
    if (e == hipSuccess) {
        if (fg.N)
            hipLaunchKernelGGL(k_flux_sens_angles, dim3((unsigned)(((size_t)g.n_angles * fg.N + 255) / 256)), dim3(256), 0, st,
                               g, fg, t.cs, tab);
        auto run = C == 8 ? sens_subsets<8> : C == 4 ? sens_subsets<4> : C == 2 ? sens_subsets<2> : sens_subsets<1>;
        e = run(g, fg, t, ft, w64, tab, ws, ws + nU, ws + nU + nP, st);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    hipFree(tab);
    hipFree(ws);
    return e;
}

// ---------------------------------------------------------------- host side
// weights exact for exponents at the Chebyshev points of [-b, b] (per node
// spacing): the inverse of their values at the nodes -3 .. 4, in extended
// precision
static void fit_exponentials(double b, FluxFit &fit) {
    b = std::max(b, 0.4);   // (closer exponents would lose digits, and gain nothing)
    long double A[kTap][2 * kTap];
    for (int m = 0; m < kTap; ++m) {
        fit.b[m] = b * cos((2 * m + 1) * M_PI / (2 * kTap));
        for (int i = 0; i < kTap; ++i) {
            A[m][i] = expl((long double)fit.b[m] * (i - 3));
            A[m][kTap + i] = m == i;
        }
    }
    for (int k = 0; k < kTap; ++k) {
        int p = k;
        for (int j = k + 1; j < kTap; ++j)
            if (fabsl(A[j][k]) > fabsl(A[p][k])) p = j;
        for (int i = 0; i < 2 * kTap; ++i) std::swap(A[k][i], A[p][i]);
        const long double d = A[k][k];
        for (int i = 0; i < 2 * kTap; ++i) A[k][i] /= d;
        for (int j = 0; j < kTap; ++j) {
            if (j == k) continue;
            const long double f = A[j][k];
            for (int i = 0; i < 2 * kTap; ++i) A[j][i] -= f * A[k][i];
        }
    }
    for (int i = 0; i < kTap; ++i)
        for (int m = 0; m < kTap; ++m) fit.v[i][m] = (double)A[i][kTap + m];
}

// Whether eight nodes of N hold the direction interpolation of every path, and
// with which exponents: one path's relative error half way between two nodes,
// over the directions, without attenuation and with e^-8 of it, at end energies
// off by 0, 3 and 6 widths of the response and at the window's ends, against
// what kDirectionErr allows for the distance.  The spacing that the response's
// steepest slope needs is only where the search starts: wide responses are
// bound by the curvature of E'(phi) and of the Klein-Nishina factor (at 25 %
// of 159 keV the slope alone asks for 48 nodes, which leave 1.4e-4 within three
// widths; 144 are taken, 6e-8).  The exponents fill 0.6 or 0.7 of the slope's range:
// the near tails carry the sums.
constexpr double kDirectionErr[3] = {2e-7, 2e-6, 6e-5};   // up to 3 widths, 6 widths, anywhere
constexpr double kLongest = 8.0;

static bool fit_directions(const Geo &g, double slope, int N, FluxFit &best) {
    constexpr int kDirs = 16, kShares = 2, kFar = 7;
    const double share[kShares] = {0.6, 0.7};
    FluxFit fit[kShares];
    double w[kShares][kTap], score[kShares] = {0.0, 0.0};
    for (int c = 0; c < kShares; ++c) {
        fit_exponentials(share[c] * slope * 2.0 * M_PI / N, fit[c]);
        for (int i = 0; i < kTap; ++i) {
            w[c][i] = 0.0;
            for (int m = 0; m < kTap; ++m) w[c][i] += fit[c].v[i][m] * exp(0.5 * fit[c].b[m]);
        }
    }
    const double c2 = 0.5 / (g.sig_e * g.sig_e);
    struct Path { double ep, psi, rho; };
    auto path = [&](double node) {
        const double c = cos(2.0 * M_PI * node / N), t = 1.0 + g.kappa * (1.0 - c), P = 1.0 / t;
        return Path{g.e0 * P, P * P * (P + t - 1.0 + c * c), kn_total(g.e0 * P) / g.sigma_kn_e0};
    };
    for (int d = 0; d < kDirs; ++d) {
        const int n = (int)lround(d * (0.5 * N) / (kDirs - 1) - 0.5);   // intervals from 0 to pi, both ends' included
        const Path at = path(n + 0.5);
        // the nodes' values over the exact one: without the energy response, at
        // either attenuation, and the energy response
        double f[2][kTap], ep[kTap];
        for (int i = 0; i < kTap; ++i) {
            const Path x = path(n + i - 3);
            ep[i] = x.ep;
            f[0][i] = x.psi / at.psi;
            f[1][i] = f[0][i] * exp((at.rho - x.rho) * kLongest);
        }
        const double far[kFar] = {0.0, -3.0 * g.sig_e, 3.0 * g.sig_e, -6.0 * g.sig_e, 6.0 * g.sig_e, g.win_lo - at.ep,
                                  g.win_hi - at.ep};
        for (int k = 0; k < kFar; ++k) {
            const double e = at.ep + far[k];
            if (k < kFar - 2 && (e < g.win_lo || e > g.win_hi)) continue;
            const double widths = fabs(far[k]) / g.sig_e;
            const double allowed = kDirectionErr[widths < 3.001 ? 0 : widths < 6.001 ? 1 : 2];
            double err[kShares][2];
            for (int c = 0; c < kShares; ++c) err[c][0] = err[c][1] = -1.0;
            for (int i = 0; i < kTap; ++i) {
                const double r = exp(c2 * (far[k] * far[k] - (e - ep[i]) * (e - ep[i])));
                for (int c = 0; c < kShares; ++c) {
                    err[c][0] += w[c][i] * f[0][i] * r;
                    err[c][1] += w[c][i] * f[1][i] * r;
                }
            }
            for (int c = 0; c < kShares; ++c)
                score[c] = std::max(score[c], std::max(fabs(err[c][0]), fabs(err[c][1])) / allowed);
        }
    }
    const int c = (int)(std::min_element(score, score + kShares) - score);
    best = fit[c];
    return score[c] <= 1.0;
}

// Pixels spread thinly over a box share few flights: a pair record then serves
// one or two lanes of its 64, and tables and pair stages cost more than the
// sums that they replace.  Refused are supports with more than kThinBox offsets a
// pixel (less than a 32nd of the box filled), before any work, and those whose
// records have more than kThinRecords times as many rows as there are pairs
// (solid shapes 1.2 to 2.5).  With the stages | without, us: 600 pixels spread over
// 200x203 (43 times), new map 5378 | 1504, forward of 500 events 317 | 153, of 25k
// 422 | 308; 2000 (25 times) 16411 | 9105, 856 | 405, 894 | 1050; but a ring of 724
// (11 times) 232 | 259, 25k events 279 | 780, 40 disks of 17 (10 times) 218 | 283,
// 275 | 811.
constexpr int kThinBox = 128, kThinRecords = 16;

bool flux_geometry(const Geo &g, const Box &box, const std::vector<int> &p_pix, FluxModel &fg, std::vector<int> &order) {
    const int x0 = box.x, y0 = box.y;
    fg.x0 = x0; fg.y0 = y0; fg.W = box.w; fg.Hh = box.h;
    fg.nb = fg.W * fg.Hh;
    // the flux order: strips of kStrip columns, row by row within a strip
    std::vector<int> at((size_t)fg.nb, -1);
    for (int p = 0; p < g.n_p; ++p) at[(size_t)(p_pix[p] / g.nx - y0) * fg.W + (p_pix[p] % g.nx - x0)] = p;
    order.clear();
    for (int i0 = 0; i0 < fg.W; i0 += kStrip)
        for (int j = 0; j < fg.Hh; ++j)
            for (int i = i0; i < std::min(fg.W, i0 + kStrip); ++i)
                if (at[(size_t)j * fg.W + i] >= 0) order.push_back(at[(size_t)j * fg.W + i]);
    fg.n_blk = (g.n_p + 63) / 64;
    fg.np64 = fg.n_blk * 64;
    fg.inv_zk = (float)(1.0 / g.zk);
    fg.e_lo = g.win_lo;
    fg.N = fg.K = 0;
    fg.h = 1.0;
    if (!g.scatter) return true;
    if ((int64_t)(2 * fg.W - 1) * (2 * fg.Hh - 1) > (int64_t)kThinBox * g.n_p) return false;
    // the steepest logarithmic slope over directions and window energies
    auto end_energy = [&](double ph) { return g.e0 / (1.0 + g.kappa * (1.0 - cos(ph))); };
    double slope = 0.0;
    for (int i = 0; i < 128; ++i) {
        const double ph = M_PI * i / 128, ep = end_energy(ph);
        const double far = std::max(fabs(g.win_lo - ep), fabs(g.win_hi - ep));
        slope = std::max(slope, far * ep * ep * g.kappa * sin(ph) / g.e0);
    }
    slope /= g.sig_e * g.sig_e;
    // direction nodes: slope x spacing at most 0.79 and what the error asks for, a
    // multiple of 48 (whole matrix tiles, an even number of sectors)
    const double n = std::max(2.0 * M_PI * slope / 0.79, 48.0);
    // energy nodes: largest exponent x spacing at most 0.70, eight nodes more
    // than intervals, a multiple of 16
    fg.e_mid = 0.5 * (g.e0 + end_energy(M_PI));
    const double b_e = 0.5 * (g.e0 - end_energy(M_PI)) / (g.sig_e * g.sig_e);
    const double k = (g.win_hi - g.win_lo) * b_e / 0.70 + 8.0;
    if (!(n <= kFluxMaxN) || !(k <= kFluxMaxK)) return false;
    fg.N = (int)ceil(n / 48.0) * 48;
    while (!fit_directions(g, slope, fg.N, fg.direction))
        if ((fg.N += 48) > kFluxMaxN) return false;
    fg.K = std::max(32, (int)ceil(k / 16.0) * 16);
    fg.h = (g.win_hi - g.win_lo) / (fg.K - 8);
    fit_exponentials(b_e * fg.h, fg.energy);
    return (int64_t)g.n_angles * fg.N * fg.K <= kFluxMaxG;
}

void free_flux(FluxTables &ft) {
    hipFree(ft.mem[0]);
    hipFree(ft.mem[1]);
    ft = FluxTables{};
}

namespace {

// arrays that share one allocation: sized with a null base, then placed
struct Slab {
    char *base = nullptr;
    size_t used = 0;
    template <class T>
    void add(T *&p, size_t n) {
        if (base) p = reinterpret_cast<T *>(base + used);
        used += (std::max<size_t>(n, 1) * sizeof(T) + 255) & ~size_t(255);
    }
};

template <class F>
hipError_t place(void *&mem, int64_t &held, int64_t room, F &&arrays) {
    Slab s;
    arrays(s);
    if (held + (int64_t)s.used > room) return hipErrorOutOfMemory;
    const hipError_t e = hipMalloc(&mem, s.used);
    if (e != hipSuccess) { mem = nullptr; return e; }
    held += (int64_t)s.used;
    s = Slab{static_cast<char *>(mem), 0};
    arrays(s);
    return hipSuccess;
}

}  // namespace

hipError_t build_flux(const Geo &g, const FluxModel &fm, const std::vector<int> &order, const Tables &t, FluxTables &ft,
                      bool sens, int64_t room, hipStream_t st, int64_t &bytes) {
    const FluxGeo &fg = fm;
    hipError_t e = hipSuccess;
    int *cnt = nullptr, *pos = nullptr;
    int2 *off = nullptr;
    double *w64 = nullptr;
    char *tmp = nullptr;
    void *scratch[2] = {nullptr, nullptr};   // for the build only
    int64_t held = 0, own = 0;
    auto done = [&](hipError_t err) {
        hipFree(scratch[0]);
        hipFree(scratch[1]);
        if (err != hipSuccess) { hipStreamSynchronize(st); free_flux(ft); }
        else bytes += held;
        return err;
    };
    const size_t na_np = (size_t)g.n_angles * g.n_p, an = g.scatter ? (size_t)g.n_angles * fg.N : 0;
    // offsets of one direction interval: the lattice points of a sector of
    // the box's diagonal, with room for the lattice lines along it
    const double diag = sqrt((double)fg.W * fg.W + (double)fg.Hh * fg.Hh);
    const int cap = (int)std::min(0.5 * diag * diag * 2.0 * M_PI / std::max(fg.N, 1) + 4.0 * diag + 64.0,
                                  4.0 * (double)fg.W * fg.Hh);
    const int nbin = fg.n_blk * fg.N;
    size_t tmp_bytes = 0;
    if (g.scatter && (e = hipcub::DeviceScan::ExclusiveSum(nullptr, tmp_bytes, ft.beg, ft.beg, nbin + 1, st)) != hipSuccess)
        return done(e);
    e = place(ft.mem[0], held, room, [&](Slab &s) {
        s.add(ft.sup, g.n_p);
        s.add(ft.box, g.n_p);
        s.add(ft.mu_s, g.n_p);
        s.add(ft.mu_box, fg.nb);
        s.add(ft.rank_of, na_np);
        s.add(ft.x_of, na_np);
        s.add(ft.pw, na_np);
        s.add(ft.pwr, na_np);
        s.add(ft.Lx, na_np);
        s.add(ft.psi, an);
        s.add(ft.rho, an);
        s.add(ft.G, an * fg.K);
        s.add(ft.beg, (size_t)nbin + 1);
    });
    if (e == hipSuccess)
        e = place(scratch[0], own, kNoLimit, [&](Slab &s) {
            s.add(pos, g.n_p);
            if (!g.scatter) return;
            s.add(cnt, fg.N);
            s.add(off, (size_t)fg.N * cap);
            s.add(tmp, tmp_bytes);
        });
    if (e != hipSuccess) return done(e);
    if ((e = hipMemcpyAsync(ft.sup, order.data(), sizeof(int) * g.n_p, hipMemcpyHostToDevice, st)) != hipSuccess) return done(e);
    hipLaunchKernelGGL(k_flux_support, dim3((g.n_p + 255) / 256), dim3(256), 0, st, g, fg, ft.sup, t.p_pix, t.mu, pos,
                       ft.box, ft.mu_s, ft.mu_box);
    hipLaunchKernelGGL(k_flux_ranks, dim3((unsigned)((na_np + 255) / 256)), dim3(256), 0, st, g, pos, t.s_sorted, t.Ld,
                       ft.rank_of, ft.x_of, ft.pw, ft.pwr, ft.Lx);
    if ((e = hipGetLastError()) != hipSuccess) return done(e);
    if (!g.scatter) {
        if (sens) e = flux_sensitivity(g, fg, t, ft, nullptr, st);
        return done(e == hipSuccess ? hipStreamSynchronize(st) : e);
    }
    hipLaunchKernelGGL(k_flux_angles, dim3(fg.N / 16, g.n_angles), dim3(256), 0, st, g, fg, t.cs, ft.psi, ft.rho, ft.G);
    hipLaunchKernelGGL(k_flux_offsets, dim3(fg.N), dim3(256), 0, st, fg.W, fg.Hh, fg.N, cap, cnt, off);
    const dim3 grid(fg.N, fg.n_blk);
    const int *q_of_pix = t.p_pix + g.n_p;
    hipLaunchKernelGGL(k_flux_pairs<0>, grid, dim3(64), 0, st, g, fg, fm.direction, ft.sup, t.p_pix, q_of_pix, t.mu, t.Bt, cnt, off,
                       cap, ft.beg, (int *)nullptr, (int *)nullptr, (float *)nullptr, (double *)nullptr, (float *)nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return done(e);
    if ((e = launch_fill(reinterpret_cast<float *>(ft.beg + nbin), 1, 0.0f, st)) != hipSuccess) return done(e);
    if ((e = hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, ft.beg, ft.beg, nbin + 1, st)) != hipSuccess) return done(e);
    int total = 0;
    if ((e = hipMemcpyAsync(&total, ft.beg + nbin, sizeof(int), hipMemcpyDeviceToHost, st)) != hipSuccess) return done(e);
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return done(e);
    if ((int64_t)total * 64 > (int64_t)kThinRecords * fg.np64 * fg.np64) return done(hipErrorNotSupported);
    e = place(ft.mem[1], held, room, [&](Slab &s) {
        s.add(ft.rec_off, total);
        s.add(ft.rec_n, total);
        s.add(ft.rec_w, (size_t)total * kTap);
        s.add(ft.sym, (size_t)total * 64);
    });
    if (e == hipSuccess) e = place(scratch[1], own, kNoLimit, [&](Slab &s) { s.add(w64, (size_t)total * kTap); });
    if (e != hipSuccess) return done(e);
    hipLaunchKernelGGL(k_flux_pairs<1>, grid, dim3(64), 0, st, g, fg, fm.direction, ft.sup, t.p_pix, q_of_pix, t.mu, t.Bt, cnt, off,
                       cap, ft.beg, ft.rec_off, ft.rec_n, ft.rec_w, w64, ft.sym);
    if ((e = hipGetLastError()) == hipSuccess && sens) e = flux_sensitivity(g, fg, t, ft, w64, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    return done(e);
}

// weights in the caller's event order -> record order (rows [0, n) of one list)
__global__ void k_flux_weights(const FluxEvent *__restrict__ ev, const int *__restrict__ orig, int n,
                               const float *__restrict__ src, float *__restrict__ dst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[orig[ev[i].row]];
}

hipError_t flux_weights(const FluxEvent *ev, const int *orig, int n, const float *src, float *dst, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_flux_weights, dim3((n + 255) / 256), dim3(256), 0, st, ev, orig, n, src, dst);
    return hipGetLastError();
}

static size_t up64(size_t n) { return (n + 63) & ~size_t(63); }
int flux_rows(const FluxGeo &fg) { return fg.N / kSec + 1; }
static size_t per_real(const Geo &g, const FluxGeo &fg) {
    return up64(fg.N ? fg.nb : 0) + up64((size_t)2 * fg.N * fg.np64) + up64(fg.N ? (size_t)4 * field_groups(fg) * fg.nb : 0) +
           up64((size_t)flux_rows(fg) * g.n_qpad);
}
static size_t per_slot(const Geo &g, const FluxGeo &fg) { return (size_t)g.n_p * (fg.K + 1); }

// Angles of one realisation that run together: all of the list, or as many
// as have spectra of 32 MB (a function of the geometry alone, so that a
// realisation's sums are the same in any batch and workspace).
int flux_angles(const Geo &g, const FluxGeo &fg, int n_list) {
    return (int)std::min<size_t>(n_list, std::max<size_t>(1, (size_t(8) << 20) / per_slot(g, fg)));
}

size_t flux_ws_floats(const Geo &g, const FluxGeo &fg, int n_real, int n_slots) {
    return n_real * per_real(g, fg) + (size_t)n_slots * per_slot(g, fg);
}

// realisations whose fields fit a workspace beside one chunk of angles (0: none)
int flux_group(const Geo &g, const FluxGeo &fg, size_t floats, int n_real, int n_list) {
    const size_t one = flux_angles(g, fg, n_list) * per_slot(g, fg);
    return (int)std::min<size_t>(n_real, (floats > one ? floats - one : 0) / per_real(g, fg));
}

// event records of blocks [b0, b1) of a set, at ev[row - row0]
hipError_t flux_events(const Geo &g, const FluxModel &fg, int b0, int b1, int row0, const int *slot_row,
                       const int *blk_beg, int n_slots, const int *base, const int *ang, const float *su,
                       const float *se, const Tables &t, FluxEvent *ev, FluxBlock *blk, hipStream_t st) {
    if (b1 <= b0) return hipSuccess;
    hipLaunchKernelGGL(k_flux_events, dim3(b1 - b0), dim3(64), 0, st, g, (const FluxGeo &)fg, fg.energy, b0, row0, slot_row,
                       blk_beg, n_slots, base, ang, su, se, t.us_sorted, ev, blk);
    return hipGetLastError();
}

namespace {

// the workspace of one group of realisations
struct Carve {
    float *fbox, *I, *T, *pb, *S, *SP;
    int slots;   // slots whose spectra fit
    Carve(const Geo &g, const FluxGeo &fg, float *ws, size_t floats, int n_real) {
        float *p = ws;
        auto take = [&](size_t per) { float *q = p; p += n_real * up64(per); return q; };
        fbox = take(fg.N ? fg.nb : 0);
        I = take((size_t)2 * fg.N * fg.np64);
        T = take(fg.N ? (size_t)4 * field_groups(fg) * fg.nb : 0);
        pb = take((size_t)flux_rows(fg) * g.n_qpad);
        const size_t used = (size_t)(p - ws), room = floats > used ? floats - used : 0;
        slots = (int)std::min<size_t>(room / per_slot(g, fg), 1 << 30);
        S = p;
        SP = p + (size_t)slots * g.n_p * fg.K;
    }
};

// Ends of an event from which two waves share them (a function of the geometry
// alone: a realisation's sums are the same in any batch).  With fewer, a wave's
// work is mostly its start and end; with more, halves take 15 -> 13 us at 64x64
// (25k events, few waves) and nothing at 128x128 (125k events, 49 and 50 us).
constexpr double kSplitEnds = 32.0;
constexpr int kSplit = 2;

// means of blocks [b0, b1), whose records begin at row row0
void launch_means(const FluxRun &p, int slot_base, int s0, int b0, int b1, int row0, const Carve &w, const float *f) {
    const Geo &g = *p.g;
    const FluxGeo &fg = *p.fg;
    // ends that an event reaches, about
    const double ends = g.n_p * 6.0 * g.sig_u / std::max(std::max(fg.W, fg.Hh) * g.dx, 6.0 * g.sig_u);
    if (fg.N) {
        const int split = ends >= kSplitEnds ? kSplit : 1;
        hipLaunchKernelGGL((split > 1 ? k_flux_means<kSplit> : k_flux_means<1>), dim3(b1 - b0), dim3(256 * split), 0, p.st, g,
                           fg, p.ev, p.blk + b0, p.t->us_sorted, p.alist, p.n_list, slot_base, s0, row0, p.row_base, w.S,
                           w.SP, p.mean, p.inv, p.skipped);
        return;
    }
    // lanes per event: about as many as it has ends
    const int lanes = ends < 48.0 ? 16 : ends < 160.0 ? 32 : 64;
    const int j0 = p.blk_rows(b0), j1 = p.blk_rows(b1);
    auto *kern = lanes == 16 ? k_flux_means_primary<16> : lanes == 32 ? k_flux_means_primary<32> : k_flux_means_primary<64>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(((size_t)(j1 - j0) * lanes + 255) / 256)), dim3(256), 0, p.st, g, fg, *p.ft, p.ev,
                       p.t->us_sorted, p.t->s_sorted, p.alist, p.n_list, slot_base, j0, j1, row0, p.row_base, f, p.mean,
                       p.inv, p.skipped);
}

}  // namespace

// row of a block's first event (the host's copy of the slots' first rows and blocks)
int FluxRun::blk_rows(int b) const {
    const int *k = std::upper_bound(blk_host, blk_host + n_real * n_list, b) - 1;   // the last slot at or before b
    const int s = (int)(k - blk_host);
    return std::min(slot_rows[s] + 64 * (b - blk_host[s]), slot_rows[s + 1]);
}

hipError_t flux_run(const FluxRun &p, bool adjoint, const FluxStage &stage) {
    const Geo &g = *p.g;
    const FluxGeo &fg = *p.fg;   // (without the fits: kernel arguments)
    const FluxTables &ft = *p.ft;
    const bool sc = fg.N > 0;
    // one group size for every subset of a set, also where their lists differ in
    // length: the box copy that one sub-iteration leaves has the next one's form
    const int grp = flux_group(g, fg, p.ws_floats, p.n_real, p.n_long), n_rows = flux_rows(fg);
    const int ca = flux_angles(g, fg, p.n_list);
    if (grp < 1) return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    for (int ra = 0; ra < p.n_real; ra += grp) {
        const int nr = std::min(grp, p.n_real - ra);
        const Carve w(g, fg, p.ws, p.ws_floats, nr);
        const int n_slots = nr * p.n_list, sb = ra * p.n_list;
        float *f = p.f + (size_t)ra * g.n_qpad;
        if (p.means && sc) {
            e = stage(0, [&] {
                // the box copy of the estimate: the previous sub-iteration's
                // update left it, unless the workspace served other sets or
                // other realisations of this one since
                if (p.box || grp < p.n_real)
                    hipLaunchKernelGGL(k_flux_box, dim3((g.n_p + 255) / 256, nr), dim3(256), 0, p.st, g, fg, ft, f, w.fbox);
                hipLaunchKernelGGL(k_flux_spread, dim3(fg.n_blk, fg.N / kSec, nr), dim3(64 * kPairWaves), 0, p.st, g, fg, ft, ft.beg,
                                   ft.rec_off, ft.rec_w, ft.sym, w.fbox, w.I);
                return hipGetLastError();
            });
            if (e != hipSuccess) return e;
        }
        // chunks of slots: whole realisations, or ca angles of one
        bool whole = false;   // a single chunk
        for (int s0 = 0, s1; s0 < n_slots; s0 = s1) {
            if (ca == p.n_list) s1 = std::min(n_slots, s0 + std::max(1, w.slots / p.n_list) * p.n_list);
            else s1 = std::min(s0 + ca, (s0 / p.n_list + 1) * p.n_list);
            const int ns = s1 - s0;
            if (ns > w.slots) return hipErrorInvalidValue;
            whole = ns == n_slots;
            if (p.means) {
                const int b0 = p.blk_host[sb + s0], b1 = p.blk_host[sb + s1];
                e = stage(0, [&] {
                    if (sc) {
                        // even parts of at most kSpecTiles tiles
                        const int kt = fg.K / 16, nz = (kt + kSpecTiles - 1) / kSpecTiles, nt = (kt + nz - 1) / nz;
                        hipLaunchKernelGGL(nt <= 4 ? k_flux_spectra<4> : nt == 5 ? k_flux_spectra<5> : k_flux_spectra<6>,
                                           dim3((g.n_p + 31) / 32 * ns, nz), dim3(64 * kSpecWaves), 0, p.st, g, fg, ft,
                                           p.alist, p.n_list, std::min(ns, p.n_list), s0, w.I, f, w.S, w.SP);
                    }
                    for (int a = b0, b; a < b1; a = b) {
                        b = p.fill ? std::min(b1, a + p.ev_cap / 64) : b1;
                        hipError_t fe = hipSuccess;
                        if (p.fill && (fe = p.fill(a, b)) != hipSuccess) return fe;
                        launch_means(p, sb, s0, a, b, p.fill ? p.blk_rows(a) : 0, w, f);
                    }
                    return hipGetLastError();
                });
                if (e != hipSuccess) return e;
            }
            if (!adjoint) continue;
            e = stage(1, [&] {
                const dim3 ag((g.n_p + 15) / 16 * ns);
                const int zr = (s1 - 1) / p.n_list - s0 / p.n_list + 1;
                // 16-node tiles of the energy nodes held in registers
                auto *adj = !sc ? k_flux_adjoint<0> : fg.K <= 96 ? k_flux_adjoint<6> : k_flux_adjoint<kMaxTiles>;
                hipLaunchKernelGGL(adj, ag, dim3(256), 0, p.st, g, fg, ft, p.ev, p.blk, p.t->us_sorted, p.alist, p.blk_beg + sb,
                                   p.n_list, s0, p.row_base, p.inv, w.S, w.SP);
                if (sc) {
                    hipLaunchKernelGGL(k_flux_fields, dim3((g.n_p + 31) / 32 * ((fg.N + 31) / 32) * zr), dim3(64 * kFieldWaves), 0, p.st, g,
                                       fg, ft, p.alist, p.n_list, s0, ns, w.S, w.SP, w.T, w.pb);
                } else if (ns < n_slots) {
                    hipLaunchKernelGGL(k_flux_primary_back, dim3(fg.n_blk, zr), dim3(256), 0, p.st, g, ft, p.alist, p.n_list,
                                       s0, ns, w.SP, w.pb);
                }
                return hipGetLastError();
            });
            if (e != hipSuccess) return e;
        }
        if (!adjoint) continue;
        if (sc) {
            e = stage(1, [&] {
                hipLaunchKernelGGL(k_flux_gather, dim3(fg.n_blk * (fg.N / kSec), nr), dim3(64 * kGatherWaves), 0, p.st, g, fg, ft, ft.beg,
                                   ft.rec_off, ft.rec_n, ft.rec_w, ft.sym, w.T, w.pb);
                return hipGetLastError();
            });
            if (e != hipSuccess) return e;
        }
        // the log-likelihood reads the means and the estimate before its update
        if (p.want_ll && (e = launch_loglik(g, p.rrange + ra, nr, p.mean, f, p.sens, p.ll + ra, p.st)) != hipSuccess)
            return e;
        e = stage(2, [&] {
            const dim3 ug((g.n_p + 63) / 64, nr);
            if (!sc && whole) {
                hipLaunchKernelGGL(p.sens ? k_flux_primary_update<false> : k_flux_primary_update<true>, ug, dim3(256), 0, p.st, g,
                                   ft, p.alist, p.n_list, w.SP, p.sens, f);
                return hipGetLastError();
            }
            auto *kern = p.sens ? k_flux_update<false> : k_flux_update<true>;
            hipLaunchKernelGGL(kern, ug, dim3(64), 0, p.st, g, fg, ft, n_rows, w.pb, p.sens, f, w.fbox);
            return hipGetLastError();
        });
        if (e != hipSuccess) return e;
    }
    return e;
}

}  // namespace lmo
