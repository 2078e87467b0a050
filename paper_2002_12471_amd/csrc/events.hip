// Event ingest: validation, ordering and tile planning.
//
// Events are ordered by (subset, realisation, angle, detector position):
// subsets are visited in order by the OS iteration (Sec. 2.2, subsets by
// detector angle), all realisations of one subset run in the same launches,
// and within one angle neighbouring positions share the path ends their
// position responses reach, so a tile of consecutive events reads one
// contiguous slice of the path table.
#include <hip/hip_runtime.h>
#include <hipcub/device/device_radix_sort.hpp>
#include <math.h>

#include <algorithm>
#include <cstdio>
#include <cstring>

#include "lmosem_int.h"

namespace lmo {

void Arena::begin() {
    used = 0;
    open = true;
    if (asked > size && size < kArenaBytes) {
        release();
        const size_t want = std::min(kArenaBytes, (asked + asked / 4 + (size_t(1) << 20) - 1) >> 20 << 20);
        if (hipMalloc(&base, want) == hipSuccess) size = want;
        else { (void)hipGetLastError(); base = nullptr; }
    }
    asked = 0;
}

void Arena::release() {
    hipFree(base);
    base = nullptr;
    size = 0;
}

hipError_t dev_take(Arena *a, void **p, size_t bytes) {
    const size_t b = (bytes + 255) & ~size_t(255);
    if (a && a->open && b <= kArenaBytes / 2) {
        a->asked += b;
        if (a->used + b <= a->size) {
            *p = a->base + a->used;
            a->used += b;
            return hipSuccess;
        }
    }
    return hipMalloc(p, bytes);
}

void dev_give(Arena *a, void *p) {
    if (!a || !a->owns(p)) hipFree(p);
}

__device__ inline bool valid_event(const Geo &g, int a, float u, float e) {
    return a >= 0 && a < g.n_angles && u >= 0.0f && u < (float)g.n_bins && (double)e >= g.win_lo && (double)e <= g.win_hi;
}

__global__ void k_validate(Geo g, int64_t n, const int32_t *__restrict__ angle,
                           const float *__restrict__ u_bin, const float *__restrict__ energy,
                           int *__restrict__ bad) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int local = 0;
    if (j < n) {
        local = valid_event(g, angle[j], u_bin[j], energy[j]) ? 0 : 1;
    }
    // one atomic per wave
    unsigned long long m = __ballot(local);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(bad, (int)__popcll(m));
}

hipError_t validate_events(const Geo &g, const lmosem_events &ev, int64_t *bad_host, int *bad_dev,
                           hipStream_t st) {
    hipError_t e = hipMemsetAsync(bad_dev, 0, sizeof(int), st);
    if (e != hipSuccess) return e;
    if (ev.n > 0) {
        hipLaunchKernelGGL(k_validate, dim3((unsigned)((ev.n + 255) / 256)), dim3(256), 0, st, g, ev.n,
                           ev.angle, ev.u_bin, ev.energy_kev, bad_dev);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    int h = 0;
    if ((e = hipMemcpyAsync(&h, bad_dev, sizeof(int), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    *bad_host = h;
    return hipSuccess;
}

// key = (group << 32) | position bits; group = (subset * R + realisation) * N_A + angle,
// n_groups for an event outside the ranges
__global__ void k_keys(Geo g, int64_t n, int n_groups, int n_real, const int64_t *__restrict__ offs,
                       const int32_t *__restrict__ angle, const float *__restrict__ u_bin,
                       const float *__restrict__ energy, int force_subset, uint64_t *__restrict__ keys,
                       int *__restrict__ idx) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    idx[j] = (int)j;
    int a = angle[j];
    float u = u_bin[j];
    if (!valid_event(g, a, u, energy[j])) {
        keys[j] = (uint64_t)n_groups << 32;
        return;
    }
    int lo = 0, hi = n_real;           // realisation r with offs[r] <= j < offs[r+1]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (offs[mid] <= j) lo = mid; else hi = mid;
    }
    int sub = force_subset >= 0 ? force_subset : a % g.n_subsets;
    uint64_t grp = ((uint64_t)sub * n_real + lo) * g.n_angles + a;
    uint32_t bits = u > 0.0f ? __float_as_uint(u) : 0u;   // positions are >= 0: bits sort like values
    keys[j] = (grp << 32) | bits;
}

// The events in sorted order, and (the workgroups past them) each group's
// count, by two searches in the sorted keys: counting by atomics took most of
// the ingest where many events share few groups (5000 events of 16 groups: 59 us
// with them, 8 us so; 25 ms of atomics for 12.8M events).
__global__ void k_gather_events(Geo g, int64_t n, int n_groups, const uint64_t *__restrict__ keys,
                                const int *__restrict__ idx, const float *__restrict__ u_bin,
                                const float *__restrict__ energy, const int32_t *__restrict__ angle,
                                int *__restrict__ sa, float *__restrict__ su,
                                float *__restrict__ se, float *__restrict__ efac, int *__restrict__ orig,
                                int *__restrict__ counts) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t padded = (n + blockDim.x - 1) / blockDim.x * blockDim.x;
    if (k >= padded) {
        const int64_t grp = k - padded;
        if (grp >= n_groups) return;
        auto first_of = [&](uint64_t key) {   // first event whose key is at least this
            int64_t lo = 0, hi = n;
            while (lo < hi) { const int64_t m = (lo + hi) >> 1; if (keys[m] >= key) hi = m; else lo = m + 1; }
            return lo;
        };
        counts[grp] = (int)(first_of((uint64_t)(grp + 1) << 32) - first_of((uint64_t)grp << 32));
        return;
    }
    if (k >= n) return;
    int j = idx[k];
    sa[k] = angle[j];
    su[k] = u_bin[j];
    const double x = (double)energy[j] - g.e_c;
    se[k] = (float)x;
    efac[k] = (float)(exp2(-g.c2 * x * x) / g.zk);
    orig[k] = j;
}

// Rank ranges of the tiles, and per tile the number of terms the forward
// kernel evaluates and the number with a non-zero position response: 16 lanes
// per tile, an event each in turn (its two searches are chains of dependent
// loads: 18 -> 5 us for 5000 events, 42 -> 10 us for 7000 on 61 x 53 pixels).
__global__ __launch_bounds__(256) void k_tile_ranks(Geo g, Tile *__restrict__ tiles, int n_tiles,
                                                    const double *__restrict__ us_sorted,
                                                    const float *__restrict__ su, long long *__restrict__ terms,
                                                    long long *__restrict__ useful) {
    const int t = (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4), sub = threadIdx.x & 15;
    if (t >= n_tiles) return;   // (whole groups of lanes)
    Tile tl = tiles[t];
    const double *us = us_sorted + (size_t)tl.angle * g.n_p;
    const double reach = 3.0 * g.sig_u;
    int r0 = g.n_p, r1 = 0;
    long long use = 0;
    for (int e = sub; e < tl.n; e += 16) {
        const double u = ((double)su[tl.e0 + e] - 0.5 * g.n_bins) * g.bin_cm;
        int lo = 0, hi = g.n_p;   // first rank with us > u - reach
        while (lo < hi) { int m = (lo + hi) >> 1; if (us[m] > u - reach) hi = m; else lo = m + 1; }
        const int above = lo;
        lo = 0;
        hi = g.n_p;               // first rank with us >= u + reach
        while (lo < hi) { int m = (lo + hi) >> 1; if (us[m] >= u + reach) hi = m; else lo = m + 1; }
        use += lo - above;
        r0 = min(r0, above);
        r1 = max(r1, lo);
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        r0 = min(r0, __shfl_xor(r0, o, 16));
        r1 = max(r1, __shfl_xor(r1, o, 16));
        use += __shfl_xor(use, o, 16);
    }
    if (sub) return;
    tl.r0 = r0;
    tl.r1 = max(r0, r1);
    tiles[t] = tl;
    terms[t] = (long long)(tl.r1 - tl.r0) * tl.n * g.n_q;
    useful[t] = use * g.n_q;
}

hipError_t launch_event_keys(const Geo &g, int n_groups, int n_real, const int64_t *offs_dev, const lmosem_events &ev,
                             int force_subset, uint64_t *keys, int *idx, hipStream_t st) {
    if (ev.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_keys, dim3((unsigned)((ev.n + 255) / 256)), dim3(256), 0, st, g, ev.n, n_groups, n_real, offs_dev,
                       ev.angle, ev.u_bin, ev.energy_kev, force_subset, keys, idx);
    return hipGetLastError();
}

hipError_t launch_gather_events(const Geo &g, int64_t n, int n_groups, const uint64_t *keys, const int *idx, const lmosem_events &ev,
                                int *sa, float *su, float *se, float *efac, int *orig, int *counts, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_events, dim3((unsigned)((n + 255) / 256 + (n_groups + 255) / 256)), dim3(256), 0, st, g,
                       n, n_groups, keys, idx, ev.u_bin, ev.energy_kev, ev.angle, sa, su, se, efac, orig, counts);
    return hipGetLastError();
}

hipError_t launch_tile_ranks(const Geo &g, Tile *tiles, int n_tiles, const double *us_sorted, const float *su,
                             long long *terms, long long *useful, hipStream_t st) {
    if (n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tile_ranks, dim3((unsigned)((n_tiles + 15) / 16)), dim3(256), 0, st, g, tiles, n_tiles,
                       us_sorted, su, terms, useful);
    return hipGetLastError();
}

int sort_key_bits(int n_groups) {
    int hi_bits = 1;
    while ((1ll << hi_bits) < (long long)n_groups) ++hi_bits;
    return 32 + hi_bits;
}

hipError_t sort_pairs_bytes(int64_t n, int n_groups, size_t &bytes) {
    bytes = 0;
    if (n <= 0) return hipSuccess;
    return hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, (const uint64_t *)nullptr, (uint64_t *)nullptr,
                                              (const int *)nullptr, (int *)nullptr, (int)n, 0,
                                              sort_key_bits(n_groups), (hipStream_t)nullptr);
}

hipError_t sort_pairs(void *tmp, size_t tmp_bytes, const uint64_t *keys, uint64_t *keys2, const int *idx, int *idx2,
                      int64_t n, int n_groups, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    return hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, keys, keys2, idx, idx2, (int)n, 0,
                                              sort_key_bits(n_groups), st);
}

void host_tiles(const Geo &g, const std::vector<int> &counts, int n_angles_used, int ev_tile, std::vector<Tile> &tiles) {
    tiles.clear();
    int64_t pos = 0;
    for (int a = 0; a < n_angles_used; ++a) {
        const int c = counts[a];
        for (int k = 0; k < c; k += ev_tile) tiles.push_back(Tile{(int)(pos + k), std::min(ev_tile, c - k), a, 0, 0, 0});
        pos += c;
    }
}

hipError_t sort_events(const Geo &g, const Tables &tb, const lmosem_events &ev,
                       const std::vector<int64_t> &offs, int force_subset, EvSet &set,
                       hipStream_t st, int64_t &bad, std::string &err) {
    hipError_t e = hipSuccess;
    const int64_t n = ev.n;
    const int n_real = (int)offs.size() - 1;
    const int n_groups = g.n_subsets * n_real * g.n_angles;
    uint64_t *keys = nullptr, *keys2 = nullptr;
    int *idx = nullptr, *idx2 = nullptr, *counts = nullptr;
    int64_t *offs_d = nullptr;
    void *tmp = nullptr;
    bad = 0;
    auto take = [&](auto **p, size_t bytes) { return dev_take(set.arena, p, bytes); };
    auto cleanup = [&]() {
        for (void *p : {(void *)keys, (void *)keys2, (void *)idx, (void *)idx2, (void *)counts, (void *)offs_d, tmp})
            dev_give(set.arena, p);
    };
#define CK(call, what) do { e = (call); if (e != hipSuccess) { err = std::string(what) + ": " + hipGetErrorString(e); cleanup(); return e; } } while (0)
    set.n = n;
    set.n_real = n_real;
    size_t nn = (size_t)std::max<int64_t>(n, 1);
    CK(take(&set.ang, sizeof(int) * nn), "alloc events");
    CK(take(&set.u, sizeof(float) * nn), "alloc events");
    CK(take(&set.e, sizeof(float) * nn), "alloc events");
    CK(take(&set.orig, sizeof(int) * nn), "alloc events");
    CK(take(&set.efac, sizeof(float) * nn), "alloc events");
    set.counts.assign(n_groups + 1, 0);
    if (n > 0) {
        CK(take(&counts, sizeof(int) * (n_groups + 1)), "alloc counts");
        CK(take(&keys, sizeof(uint64_t) * n), "alloc keys");
        CK(take(&keys2, sizeof(uint64_t) * n), "alloc keys");
        CK(take(&idx, sizeof(int) * n), "alloc idx");
        CK(take(&idx2, sizeof(int) * n), "alloc idx");
        if (n_real > 1) {
            CK(take(&offs_d, sizeof(int64_t) * offs.size()), "alloc offsets");
            CK(hipMemcpyAsync(offs_d, offs.data(), sizeof(int64_t) * offs.size(), hipMemcpyHostToDevice, st),
               "upload offsets");
        }
        // events are checked as they are keyed: the invalid ones count as one
        // more group, behind the others
        CK(launch_event_keys(g, n_groups, n_real, offs_d, ev, force_subset, keys, idx, st), "keys");
        size_t tmp_bytes = 0;
        CK(sort_pairs_bytes(n, n_groups + 1, tmp_bytes), "sort size");
        CK(take(&tmp, tmp_bytes), "alloc sort");
        CK(sort_pairs(tmp, tmp_bytes, keys, keys2, idx, idx2, n, n_groups + 1, st), "sort");
        CK(launch_gather_events(g, n, n_groups + 1, keys2, idx2, ev, set.ang, set.u, set.e, set.efac, set.orig, counts, st),
           "gather events");
        CK(hipMemcpyAsync(set.counts.data(), counts, sizeof(int) * (n_groups + 1), hipMemcpyDeviceToHost, st),
           "download counts");
        CK(hipStreamSynchronize(st), "ingest");
    }
    bad = set.counts[n_groups];
    set.counts.resize(std::max(n_groups, 1));
    cleanup();
#undef CK
    return bad ? hipSuccess : plan_tiles(g, tb, set, set.ev_tile, set.chunk_rows, st, err);
}

// Tiles of ev_tile consecutive events per (subset, realisation, angle) group
// and backprojection chunks of chunk_rows rows per (subset, realisation), from
// the group counts of the sorted set; replaces any earlier plan.
hipError_t plan_tiles(const Geo &g, const Tables &tb, EvSet &set, int ev_tile, int chunk_rows,
                      hipStream_t st, std::string &err) {
    hipError_t e = hipSuccess;
    long long *terms_d = nullptr;   // [tiles] terms, then [tiles] useful
    auto cleanup = [&]() { dev_give(set.arena, terms_d); };
#define CK(call, what) do { e = (call); if (e != hipSuccess) { err = std::string(what) + ": " + hipGetErrorString(e); cleanup(); return e; } } while (0)
    dev_give(set.arena, set.plan);
    set.plan = nullptr;
    set.tiles = nullptr; set.chunks = nullptr; set.crange = nullptr; set.rrange = nullptr;
    set.trange = nullptr;
    set.ev_tile = ev_tile;
    set.chunk_rows = chunk_rows;
    const int n_real = set.n_real;
    const std::vector<int> &cnt = set.counts;
    const int EV = ev_tile, CH = chunk_rows;
    std::vector<Tile> tiles;
    std::vector<Chunk> chunks;
    std::vector<int> crange, rrange, trange;
    set.row_off.assign(g.n_subsets + 1, 0);
    set.tile_off.assign(g.n_subsets + 1, 0);
    set.chunk_off.assign(g.n_subsets + 1, 0);
    set.max_rows = 0;
    set.max_chunks = 0;
    int64_t pos = 0;
    for (int i = 0; i < g.n_subsets; ++i) {
        set.row_off[i] = (int)pos;
        set.tile_off[i] = (int)tiles.size();
        set.chunk_off[i] = (int)chunks.size();
        for (int r = 0; r < n_real; ++r) {
            crange.push_back((int)chunks.size() - set.chunk_off[i]);
            rrange.push_back((int)(pos - set.row_off[i]));
            trange.push_back((int)tiles.size() - set.tile_off[i]);
            int64_t real_start = pos;
            for (int a = 0; a < g.n_angles; ++a) {
                int c = cnt[((size_t)i * n_real + r) * g.n_angles + a];
                for (int k = 0; k < c; k += EV)
                    tiles.push_back(Tile{(int)(pos + k), std::min(EV, c - k), a, r, 0, 0});
                pos += c;
            }
            for (int64_t j = real_start; j < pos; j += CH)
                chunks.push_back(Chunk{(int)(j - set.row_off[i]),
                                       (int)(std::min<int64_t>(pos, j + CH) - set.row_off[i]), r, 0});
        }
        crange.push_back((int)chunks.size() - set.chunk_off[i]);
        rrange.push_back((int)(pos - set.row_off[i]));
        trange.push_back((int)tiles.size() - set.tile_off[i]);
        set.max_rows = std::max(set.max_rows, (int)(pos - set.row_off[i]));
        set.max_chunks = std::max(set.max_chunks, (int)chunks.size() - set.chunk_off[i]);
    }
    set.row_off[g.n_subsets] = (int)pos;
    set.tile_off[g.n_subsets] = (int)tiles.size();
    set.chunk_off[g.n_subsets] = (int)chunks.size();
    // [tiles][chunks][crange][rrange][trange] in one block and one copy
    size_t nt = std::max<size_t>(tiles.size(), 1);
    std::vector<char> up;
    auto add = [&](const auto &v) {
        const size_t at = up.size(), bytes = sizeof(v[0]) * v.size();
        up.resize((at + std::max<size_t>(bytes, 1) + 15) & ~size_t(15));
        if (bytes) memcpy(up.data() + at, v.data(), bytes);
        return at;
    };
    const size_t o_tiles = add(tiles), o_chunks = add(chunks), o_crange = add(crange), o_rrange = add(rrange),
                 o_trange = add(trange);
    CK(dev_take(set.arena, &set.plan, up.size()), "alloc tiles");
    char *plan = static_cast<char *>(set.plan);
    set.tiles = reinterpret_cast<Tile *>(plan + o_tiles);
    set.chunks = reinterpret_cast<Chunk *>(plan + o_chunks);
    set.crange = reinterpret_cast<int *>(plan + o_crange);
    set.rrange = reinterpret_cast<int *>(plan + o_rrange);
    set.trange = reinterpret_cast<int *>(plan + o_trange);
    CK(dev_take(set.arena, &terms_d, 2 * sizeof(long long) * nt), "alloc counters");
    CK(hipMemcpyAsync(plan, up.data(), up.size(), hipMemcpyHostToDevice, st), "upload tiles");
    std::vector<long long> terms(2 * nt, 0);
    const long long *useful = terms.data() + nt;
    if (!tiles.empty()) {
        CK(launch_tile_ranks(g, set.tiles, (int)tiles.size(), tb.us_sorted, set.u, terms_d, terms_d + nt, st), "tile ranks");
        CK(hipMemcpyAsync(terms.data(), terms_d, 2 * sizeof(long long) * nt, hipMemcpyDeviceToHost, st),
           "download counters");
    }
    CK(hipStreamSynchronize(st), "tile plan");
    set.terms_sub.assign(g.n_subsets, 0);
    set.useful_sub.assign(g.n_subsets, 0);
    set.max_ranks = 0;
    for (int i = 0; i < g.n_subsets; ++i)
        for (int t = set.tile_off[i]; t < set.tile_off[i + 1]; ++t) {
            set.terms_sub[i] += terms[t];
            set.useful_sub[i] += useful[t];
            set.max_ranks = std::max(set.max_ranks, (int)(terms[t] / ((int64_t)tiles[t].n * g.n_q)));
        }
    cleanup();
#undef CK
    return hipSuccess;
}

}  // namespace lmo
