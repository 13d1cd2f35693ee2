// Density, ghost, force and integrator stages on the leaf cells.
//
// Work unit: one wave (64 lanes) per leaf cell A.  The density sweep of leaves of
// up to 64 particles and the gather force pack the candidates of A's
// neighbour cells into tiles, test them on the matrix units and evaluate the
// pairs in range one per lane (sph_device.h).  The chunked kernels (larger
// leaves, the sorted-axis mode, the pairs-once force): lanes hold up to 64 of
// A's particles (i); when A holds fewer than 64 the wave is split into G
// groups of CI = 64/G lanes and group g walks every G-th neighbour of the
// staged tile, so all lanes stay busy.  A's neighbour-cell list gives the
// cells B; for each, the part of B that can be within range along the pair's
// sort direction (a window of B's sorted projections) is staged in LDS and
// streamed through.  Coordinates are cell-relative: each particle is stored
// relative to its leaf's centre, and the offset between two leaves (with the
// periodic image) is formed in FP64 once per pair of cells.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "sph_ctx.h"
#include "sph_device.h"

// Occupancy target (waves per SIMD, WPE) of the packed density and gather
// force kernels, the measured best at 256^3 clustered: density sweeps of a step
// 5.75 ms at 5 waves, 5.87 at 6 (more spills), 6.22 at 4; the force's LDS holds
// 4 waves (9.45 ms, 9.82 with 3, 21.4 with 5 waves and tiles of 80).
#define SPH_DENS_WAVES 5
#define SPH_FORCEG_WAVES 4
#define SPH_DENS_WAVES64 3
#define SPH_FORCEG_WAVES64 2
// ... and of their forms with several waves per leaf (at 6 the density spills).
#define SPH_WIDE_OCC 4
// List entries staged per batch.
#define SPH_BATCH 32
// Candidates per 16-lane row of a tile: the largest tiles (fewest partly filled
// rounds of pairs) whose LDS leaves the waves above resident.  Density at 32 /
// 28 / 24: 5.87 / 6.10 / 6.00 ms (6 waves); force at 28 / 24: 9.45 / 9.49 ms, 32 at
// 3 waves 9.78.
#define DENS_ROW 32
#define FORCE_ROW 28

// Density: tile, particles and sums of one wave.
template <typename T>
struct PTile {
    typename vec4<T>::type cand[4 * DENS_ROW];  // j in A's frame, w = m
    union {
        float c1[4 * DENS_ROW];                 // row constants of the range tests
        uint16_t list[PAIR_CAP];        // then the pairs
    };
    typename vec4<T>::type si[64];      // i of A: x, y, z (A frame), 1/H
    double sw[64], sd[64];              // sums of the particles
    T s2[64];
    int cnt[64];
    EFlat<T, SPH_BATCH> e;
};
// FP64: the tests' coordinates in FP32
struct PTile64 : PTile<double> {
    float4 fc[4 * DENS_ROW];
};
template <typename T> struct ptile { typedef PTile<T> type; };
template <> struct ptile<double> { typedef PTile64 type; };

// Candidate j of the tile for the range tests (the FP64 tile keeps an FP32
// copy of the coordinates; the FP32 tile is read as it is); returns |p|^2.
template <typename T, typename Tile>
__device__ inline float put_test(Tile& L, int j, T x, T y, T z)
{
    const float fx = (float)x, fy = (float)y, fz = (float)z;
    if constexpr (sizeof(T) == 8) L.fc[j] = make_float4(fx, fy, fz, 1.0f);
    return fx * fx + fy * fy + fz * fz;
}
template <typename T, typename Tile>
__device__ inline float get_test(const Tile& L, int j, int lane)
{
    if constexpr (sizeof(T) == 8) {
        return ((const float*)&L.fc[j])[lane >> 4];
    } else {
        const float v = ((const float*)&L.cand[j])[lane >> 4];
        return lane < 48 ? v : 1.0f;
    }
}

// Density sweep of one leaf (at most 64 particles, box pruning): candidate
// stream, matrix-unit range tests and pair-parallel sums (sph_device.h), then
// the FP64 Newton test.  Bound by VALU issue, which is active in 91% of the
// cycles: about 7.9e3 VALU instructions per leaf at 256^3 clustered, 2.1e4 with
// a ballot loop over the particles per tile and lane = particle sums.  Sweeps
// of a step there 9.9 -> 5.75 ms (FP32C), density stage at 64^3 FP64 2.6 -> 0.95 ms.
// With NW > 1 the waves of the workgroup share the leaf's list; wave 0 adds up
// their sums.
template <typename T, int NW>
__device__ __forceinline__ void density_leaf_packed(const DensArgs& a, int A, typename ptile<T>::type* tiles, int lane, int wave)
{
    typename ptile<T>::type& L = tiles[wave];
    constexpr bool EXTRAP = sizeof(T) == 4;
    typedef typename vec4<T>::type V4;
    const V4* pos4 = (const V4*)a.pos4;
    const int bA = a.l_begin[A], nA = a.l_count[A];
    const double oA[3] = {a.l_origin[3 * A], a.l_origin[3 * A + 1], a.l_origin[3 * A + 2]};
    const DomainInfo& I = a.di[a.l_dom[A]];
    const double hlim = fmin(fmin(I.L[0], I.L[1]), I.L[2]) / 3.0;
    const double s0min = fmin(fmin(I.s0[0], I.s0[1]), I.s0[2]);
    const int ea = a.l_off[A], ne = a.l_off[A + 1] - ea;
    const int e0 = ea + (int)((long long)ne * wave / NW), e1 = ea + (int)((long long)ne * (wave + 1) / NW);
    const double mg = *a.margin;  // list margin (see density_leaf)
    const double hlA = a.l_hlist[A] - mg;
    const bool vi = lane < nA;
    const int i = bA + (vi ? lane : 0);
    const bool act = vi && !a.conv[i];
    const unsigned long long amask = __ballot(act);
    if (amask == 0ull) {
        if (NW == 1 || wave == 0)
            if (lane == 0) a.l_active[A] = 0;
        return;
    }
    const V4 pi = pos4[i];
    const double Hd = a.H[i];
    const double hA = wave_max(act ? Hd : 0.0);
    const T big = T(1e30);
    T bxl = wave_min_t<T>(act ? pi.x : big), bxh = wave_max_t<T>(act ? pi.x : -big);
    T byl = wave_min_t<T>(act ? pi.y : big), byh = wave_max_t<T>(act ? pi.y : -big);
    T bzl = wave_min_t<T>(act ? pi.z : big), bzh = wave_max_t<T>(act ? pi.z : -big);
    // scale: the leaf's box and its largest H are of order 1 below
    const T sc = pow2_scale(fmax((T)hA, fmax(fmax(fmax(-bxl, bxh), fmax(-byl, byh)), fmax(-bzl, bzh))));
    bxl *= sc, bxh *= sc, byl *= sc, byh *= sc, bzl *= sc, bzh *= sc;
    const T hAm = (T)(hA * (1.0 + 1e-5)) * sc;
    const T hA2 = hAm * hAm;
    const int nb = 4 - (__builtin_clzll(amask) >> 4);
    bf16x4 bt[4];
    {
        V4 q = pi;
        q.x *= sc, q.y *= sc, q.z *= sc;
        const float x = (float)q.x, y = (float)q.y, z = (float)q.z, h = (float)((T)Hd * sc);
        const float p2 = x * x + y * y + z * z;
        const bool on = act && p2 < 1e30f;
        test_operand(on ? x : 0.f, on ? y : 0.f, on ? z : 0.f,
                     on ? p2 * (1.0f - PAIR_EPS) - h * h * (1.0f + PAIR_EPS) - 1e-30f : 1e30f, 0.f, (float4*)L.cand, lane, bt);
        q.w = T(1) / ((T)Hd * sc);
        L.si[lane] = q;
        L.sw[lane] = L.sd[lane] = 0.0;
        L.s2[lane] = T(0);
        L.cnt[lane] = 0;
    }
    // the sums of one run of pairs
    auto eval = [&](const uint16_t* list, int n) {
        const int K = (n + 63) >> 6;
        int cur = -1, cnt = 0;
        double sw = 0.0, sd = 0.0;
        T s2 = T(0);
        V4 p;
        auto flush = [&]() {
            lds_add(&L.sw[cur], sw);
            lds_add(&L.sd[cur], sd);
            if (EXTRAP) lds_add(&L.s2[cur], s2);
            lds_add(&L.cnt[cur], cnt);
        };
        for (int e = lane * K; e < min(lane * K + K, n); e++) {
            const int code = list[e], ii = code >> 7;
            if (ii != cur) {
                if (cur >= 0) flush();
                cur = ii;
                p = L.si[ii];
                sw = sd = 0.0;
                s2 = T(0);
                cnt = 0;
            }
            const V4 c = L.cand[code & 127];
            const T dx = c.x - p.x, dy = c.y - p.y, dz = c.z - p.z;
            // (every term is an exact zero at q = 1)
            const T q = fmin(fast_sqrt(dx * dx + dy * dy + dz * dz) * p.w, T(1));
            T w, dw;
            spline_w_dw(q, w, dw);
            sw += (double)(c.w * w);
            sd += (double)(c.w * (T(3) * w + q * dw));
            if (EXTRAP) s2 += c.w * spline_d2(q, dw);
            cnt += q < T(1);
        }
        if (cur >= 0) flush();
    };
    auto run_tile = [&](int len) {
        for (int j = len + lane; j < 4 * DENS_ROW; j += 64) {
            V4 o;
            o.x = o.y = o.z = o.w = T(0);
            L.cand[j] = o;
            put_test<T>(L, j, T(0), T(0), T(0));
            L.c1[test_slot<DENS_ROW>(j)] = 1e30f;
        }
        wave_sync();
        uint32_t M[4] = {0u, 0u, 0u, 0u};
        tile_masks<false, DENS_ROW>(L.c1, nullptr, [&](int j) { return get_test<T>(L, j, lane); }, bt, nb, lane, M);
        for_pairs<DENS_ROW>(M, L.list, lane, []() {}, eval);
        wave_sync();
    };
    const uint32_t last = (uint32_t)(a.n - 1);
    int ncand = 0, eb = e0, p0 = 0, total = 0, start = 0;
    V4 o, pf;
    auto load = [&](int p) {
        o = L.e.o[stream_cell(p, start)];
        pf = pos4[min((uint32_t)(p + lane + unpack_int(o.w)), last)];
    };
    while (true) {
        if (p0 >= total) {  // next batch of cells
            for (total = 0; eb < e1 && total == 0; eb += SPH_BATCH) {
                wave_sync();
                total = load_batch_flat<T>(a.list, eb, min(SPH_BATCH, e1 - eb), lane, a.l_begin, a.l_count, a.l_origin, oA, I, sc,
                                           [&](const ListEntry& E) { return E.dist < hA + mg; }, L.e, start);
            }
            p0 = 0;
            if (total > 0) load(0);
        }
        V4 q;
        unsigned long long mk = 0ull;
        if (total > 0) {
            q.x = fma_t(pf.x, sc, o.x);
            q.y = fma_t(pf.y, sc, o.y);
            q.z = fma_t(pf.z, sc, o.z);
            q.w = pf.w;
            mk = __ballot((p0 + lane < total) & (box_d2<T>(q.x, q.y, q.z, bxl, byl, bzl, bxh, byh, bzh) < hA2));
            p0 += 64;
            if (p0 < total) load(p0);
        }
        const int nk = __popcll(mk);
        if (ncand + nk > 4 * DENS_ROW || total == 0) {
            if (ncand > 0) run_tile(ncand);
            if (total == 0) break;
            ncand = 0;
        }
        if ((mk >> lane) & 1ull) {
            const int slot = ncand + lane_rank(mk);
            L.cand[slot] = q;
            L.c1[test_slot<DENS_ROW>(slot)] = put_test<T>(L, slot, q.x, q.y, q.z) * (1.0f - PAIR_EPS);
        }
        ncand += nk;
    }
    wave_sync();
    double sw = L.sw[lane], sd = L.sd[lane], s2 = (double)L.s2[lane];
    int cnt = L.cnt[lane];
    const double mi = a.m[i];
    if (NW > 1) {
        __syncthreads();
        if (wave != 0) return;
        for (int w = 1; w < NW; w++) {
            sw += tiles[w].sw[lane];
            sd += tiles[w].sd[lane];
            s2 += (double)tiles[w].s2[lane];
            cnt += tiles[w].cnt[lane];
        }
    }
    const bool left = dens_finish<T>(a, i, act, 0, 64, Hd, sw, sd, s2, cnt, hlA, hlim, s0min, mi);
    const unsigned long long lm = __ballot(left);
    if (lane == 0) a.l_active[A] = lm ? 1 : 0;
    wave_sync();
}

template <typename T, bool COMP, int PRUNE>
__device__ void density_leaf(const DensArgs& a, int A, DTile<T>& L, int lane)
{
    // FP32 modes accept a small final Newton update by second-order expansion
    constexpr bool EXTRAP = sizeof(T) == 4;
    typedef typename vec4<T>::type V4;
    const V4* pos4 = (const V4*)a.pos4;
    const int bA = a.l_begin[A], nA = a.l_count[A];
    const double oA[3] = {a.l_origin[3 * A], a.l_origin[3 * A + 1], a.l_origin[3 * A + 2]};
    const DomainInfo& I = a.di[a.l_dom[A]];
    const double hlim = fmin(fmin(I.L[0], I.L[1]), I.L[2]) / 3.0;
    const double s0min = fmin(fmin(I.s0[0], I.s0[1]), I.s0[2]);
    const int e0 = a.l_off[A], e1 = a.l_off[A + 1];
    // particles moved up to mg/2 since the lists were built: list radii shrink
    // by mg and list entries are taken up to mg farther out
    const double mg = *a.margin;
    const double hlA = a.l_hlist[A] - mg;
    bool any_left = false;
    for (int c0 = 0; c0 < nA; c0 += 64) {
        const int nc = min(64, nA - c0);
        const int lg = chunk_log2(nc);
        const int CI = 1 << lg, G = 64 >> lg;
        const int ii = lane & (CI - 1), jg = lane >> lg;
        const bool vi = ii < nc;
        const int i = bA + c0 + (vi ? ii : 0);
        const bool act = vi && !a.conv[i];
        if (__ballot(act) == 0) continue;
        const V4 pi = pos4[i];
        const double Hd = a.H[i];
        const T Hi = (T)Hd, H2 = Hi * Hi, invH = T(1) / Hi;
        Acc<T, COMP> sw, sd;
        T s2 = T(0);
        int cnt = 0;
        const double hA = wave_max(act ? Hd : 0.0);
        // bounding box of the active i (A frame) and the squared pruning radius
        const T big = T(1e30);
        const T bxl = wave_min_t<T>(act ? pi.x : big), bxh = wave_max_t<T>(act ? pi.x : -big);
        const T byl = wave_min_t<T>(act ? pi.y : big), byh = wave_max_t<T>(act ? pi.y : -big);
        const T bzl = wave_min_t<T>(act ? pi.z : big), bzh = wave_max_t<T>(act ? pi.z : -big);
        const T hAm = (T)(hA * (1.0 + 1e-5));
        const T hA2 = hAm * hAm;
        for (int eb = e0; eb < e1; eb += 64) {
            const int nbt = min(64, e1 - eb);
            const int nv = load_batch<T>(a.list, eb, nbt, lane, a.l_begin, a.l_count, a.l_origin, oA, I,
                                         [&](const ListEntry& E) { return E.dist < hA + mg; }, L.e, nullptr, A);
            V4 pf;  // prefetched first cell of the next pair
            if (PRUNE == PRUNE_BOX && nv > 0) {
                const int n0 = L.e.n[0];
                if (lane < n0) pf = pos4[L.e.b[0] + lane];
            }
            // accumulate one in-range pair (i, particle q4 of B)
            auto dens_acc = [&](const V4& q4, T r2) {
                const T q = fast_sqrt(r2) * invH;
                T w, dw;
                spline_w_dw(q, w, dw);
                sw.add(q4.w * w);
                sd.add(q4.w * (T(3) * w + q * dw));
                if (EXTRAP) s2 += q4.w * spline_d2(q, dw);
                cnt++;
            };
            // Pairs of cells in batches of NTD: phase 1 stages each neighbour
            // cell and records the in-range pairs of every lane as bits of a
            // mask; phase 2 evaluates only those pairs.
            for (int k0 = 0; k0 < nv; k0 += NTD) {
                unsigned long long msk[NTD];
                T tox[NTD], toy[NTD], toz[NTD];
#pragma unroll
                for (int u = 0; u < NTD; u++) {
                    msk[u] = 0ull;
                    tox[u] = toy[u] = toz[u] = T(0);
                    const int k = k0 + u;
                    if (k >= nv) continue;
                    const int bB = L.e.b[k], nB = L.e.n[k];
                    const T dox = L.e.ox[k], doy = L.e.oy[k], doz = L.e.oz[k];
                    tox[u] = dox;
                    toy[u] = doy;
                    toz[u] = doz;
                    const T xi = pi.x - dox, yi = pi.y - doy, zi = pi.z - doz;  // i in B's frame
                    V4* tile = L.p[u];
                    if (PRUNE == PRUNE_BOX && nB <= 64) {
                        const V4 pj = pf;
                        if (k + 1 < nv) {
                            const int n1 = L.e.n[k + 1];
                            if (lane < n1) pf = pos4[L.e.b[k + 1] + lane];
                        }
                        const bool in = lane < nB && box_d2<T>(pj.x, pj.y, pj.z, bxl - dox, byl - doy, bzl - doz,
                                                                bxh - dox, byh - doy, bzh - doz) < hA2;
                        const unsigned long long mk = __ballot(in);
                        if (in) tile[mask_rank(mk, lane)] = pj;
                        const int len = __popcll(mk);
                        wave_sync();
                        if (act) {
                            unsigned long long m = 0ull;
                            for (int s = 0, t = jg; t < len; s++, t += G) {
                                const V4 q4 = tile[t];
                                const T dx = q4.x - xi, dy = q4.y - yi, dz = q4.z - zi;
                                if (dx * dx + dy * dy + dz * dz < H2) m |= 1ull << s;
                            }
                            msk[u] = m;
                        }
                    } else {
                        // sorted-axis window (or a cell too large for one tile): one phase
                        int lo = 0, hi = nB;
                        const int dir = L.e.dir[k];
                        const bool srt = PRUNE == PRUNE_SORTED && a.l_sorted[L.e.B[k]] && nB <= 64;
                        if (srt) {
                            double uu[3];
                            sph_dir(dir, uu);
                            const float ki = (float)((double)xi * uu[0] + (double)yi * uu[1] + (double)zi * uu[2]);
                            float kmin = wave_minf(act ? ki - (float)Hd : INFINITY);
                            float kmax = wave_maxf(act ? ki + (float)Hd : -INFINITY);
                            const float eps = 1e-5f * (fabsf(kmin) + fabsf(kmax)) + 1e-6f * (float)hA;
                            sorted_window(a.skey, a.n, dir, bB, nB, lane, kmin - eps, kmax + eps, lo, hi);
                        }
                        for (int p0 = lo; p0 < hi; p0 += 64) {
                            const int len = min(64, hi - p0);
                            if (lane < len) {
                                const int t = p0 + lane;
                                const int jl = srt ? (int)a.sidx[(int64_t)dir * a.n + bB + t] : t;
                                tile[lane] = pos4[bB + jl];
                            }
                            wave_sync();
                            for (int t = jg; t < len; t += G) {
                                const V4 q4 = tile[t];
                                const T dx = q4.x - xi, dy = q4.y - yi, dz = q4.z - zi;
                                const T r2 = dx * dx + dy * dy + dz * dz;
                                if (act && r2 < H2) dens_acc(q4, r2);
                            }
                            wave_sync();
                        }
                        if (PRUNE == PRUNE_BOX && k + 1 < nv) {
                            const int n1 = L.e.n[k + 1];
                            if (lane < n1) pf = pos4[L.e.b[k + 1] + lane];
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < NTD; u++) {
                    unsigned long long m = msk[u];
                    const T xi = pi.x - tox[u], yi = pi.y - toy[u], zi = pi.z - toz[u];
                    const V4* tile = L.p[u];
                    while (m) {
                        const int s = __ffsll((long long)m) - 1;
                        m &= m - 1;
                        const V4 q4 = tile[jg + G * s];
                        const T dx = q4.x - xi, dy = q4.y - yi, dz = q4.z - zi;
                        dens_acc(q4, dx * dx + dy * dy + dz * dz);
                    }
                }
                wave_sync();
            }
            wave_sync();
        }
        const bool left = dens_finish<T>(a, i, act, jg, CI, Hd, sw.total(), sd.total(), (double)s2, cnt, hlA, hlim,
                                         s0min, a.m[i]);
        const unsigned long long lm = __ballot(left);
        if (lm) any_left = true;
    }
    if (lane == 0) a.l_active[A] = any_left ? 1 : 0;
}

template <typename T, bool COMP, int PRUNE>
__global__ __launch_bounds__(256) void k_density(DensArgs a)
{
    __shared__ DTile<T> tiles[WAVES_PER_WG];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (a.gate && uniform(*a.gate) != 0) return;
    const int nL = a.nl_dev ? uniform(*a.nl_dev) : a.n_leaves;
    const int A = uniform(xcd_block(blockIdx.x, gridDim.x) * WAVES_PER_WG + w);
    if (A >= nL) return;
    if (!a.l_active[A]) return;
    if (a.big_only && a.l_count[A] <= 64) return;
    density_leaf<T, COMP, PRUNE>(a, A, tiles[w], lane);
}


// Leaf of workgroup b of a grid over the leaves (-1: none); a grid of single
// waves (NW = 1) leaves those with long lists to the wide workgroups.
template <int NW, typename Args>
__device__ inline int tile_leaf(const Args& a, int b)
{
    const int nL = a.nl_dev ? uniform(*a.nl_dev) : a.n_leaves;
    const int A = uniform(xcd_block(b, gridDim.x));
    if (A >= nL || (NW == 1 && a.l_off[A + 1] - a.l_off[A] > uniform(*a.wide_min))) return -1;
    return A;
}

// The leaves with long lists (a.wide), or every leaf, by workgroups of NW
// waves: work(A, wave).
template <int NW, typename Args, typename Work>
__device__ __forceinline__ void for_wide_leaves(const Args& a, Work work)
{
    const int wave = uniform(threadIdx.x >> 6);
    if (!a.wide) {
        const int A = tile_leaf<NW>(a, blockIdx.x);
        if (A >= 0) work(A, wave);
        return;
    }
    const int n = a.nl_dev ? uniform(*a.n_wide_dev) : a.n_wide;
    // the classes of the list one after another
    const int nL = a.nl_dev ? uniform(*a.nl_dev) : a.n_leaves;
    const int* cl = a.n_wide_dev + (FI_WIDECLASS - FI_NWIDE);
    const int c0 = uniform(cl[0]), c1 = c0 + uniform(cl[1]), c2 = c1 + uniform(cl[2]);
    for (int b = blockIdx.x; b < n; b += gridDim.x) {
        const int k = (b >= c0) + (b >= c1) + (b >= c2);
        const int t = b - (k == 0 ? 0 : k == 1 ? c0 : k == 2 ? c1 : c2);
        work(uniform(a.wide[(size_t)k * nL + t]), wave);
        __syncthreads();  // (the tiles are reused)
    }
}

// Packed density sweep over the leaves of at most 64 particles (box
// pruning), NW waves per leaf.
template <typename T, int WPE, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE, 8))) void k_density_packed(DensArgs a)
{
    __shared__ typename ptile<T>::type tiles[NW];
    if (a.gate && uniform(*a.gate) != 0) return;
    const int lane = threadIdx.x & 63;
    auto leaf = [&](int A, int wave) __attribute__((always_inline)) {
        if (a.l_active[A] && a.l_count[A] <= 64) density_leaf_packed<T, NW>(a, A, tiles, lane, wave);
    };
    if (NW > 1) {
        for_wide_leaves<NW>(a, leaf);
        return;
    }
    const int A = tile_leaf<NW>(a, blockIdx.x);
    if (A >= 0) leaf(A, 0);
}

__global__ __launch_bounds__(256) void k_density_reset(int64_t n, int n_leaves, double* hlo, double* hhi, uint8_t* conv,
                                                       int* l_active, const int* nl_dev)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (nl_dev) n_leaves = *nl_dev;
    if (i < n) {
        hlo[i] = 0.0;
        hhi[i] = INFINITY;
        conv[i] = 0;
    }
    if (i < n_leaves) l_active[i] = 1;
}

// ---------------------------------------------------------------------------
// Ghost: Omega = 1 + H/(3 rho) drho/dH, P = (gamma-1) rho u, A = P/(Omega rho^2)
// ---------------------------------------------------------------------------
enum { GHOST_PAIRS = 0, GHOST_PLIST = 1, GHOST_GATHER = 2 };
template <typename T>
__global__ __launch_bounds__(256) void k_ghost(int64_t n, const double* __restrict__ rho, const double* __restrict__ drho,
                                               const double* __restrict__ H, const double* __restrict__ u,
                                               const double* __restrict__ vx, const double* __restrict__ vy,
                                               const double* __restrict__ vz, double gamma, double* omega, double* P,
                                               typename vec4<T>::type* fv4, T* hf, const int* gate,
                                               const double* __restrict__ ax, const double* __restrict__ ay,
                                               const double* __restrict__ az, const double* __restrict__ dudt,
                                               const double* __restrict__ hdt, int form)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (gate && *gate != 1) return;
    // inside a step the ghost and force use v and u predicted to the end of
    // the step with the forces of its start: x + a dt/2 (hdt = dt/2; 0 outside)
    const double hd = *hdt;
    double ui = u[i], v0 = vx[i], v1 = vy[i], v2 = vz[i];
    if (hd != 0.0) {
        ui += dudt[i] * hd;
        v0 += ax[i] * hd;
        v1 += ay[i] * hd;
        v2 += az[i] * hd;
    }
    const double r = rho[i], h = H[i];
    const double om = 1.0 + h / (3.0 * r) * drho[i];
    const double p = (gamma - 1.0) * r * ui;
    const double A = p / (om * r * r);
    if (omega) omega[i] = om;
    if (P) P[i] = p;
    typename vec4<T>::type f;
    f.x = (T)v0;
    f.y = (T)v1;
    f.z = (T)v2;
    // the pairs-once force takes A and H; the gather forms take the
    // kernel-gradient factor A (8/pi) / H^4, over cells times the -6 of the
    // spline's derivative and with H, over particle lists with 1/H
    const double k = A * INV_PI_8 / (h * h * h * h);
    f.w = form == GHOST_PAIRS ? (T)A : form == GHOST_GATHER ? (T)(-6.0 * k) : (T)k;
    fv4[i] = f;
    hf[i] = form == GHOST_PLIST ? (T)(1.0 / h) : (T)h;
}

// ---------------------------------------------------------------------------
// Force, eqs. (dvdt) and (dudt), symmetric: every unordered pair once.
// Pair cells (A,B): i-side sums in registers, j-side sums in LDS (lanes of a
// group rotate over distinct j), flushed with one atomic add per j and
// quantity.  The cell's own pairs: triangular sweep.  Each unordered pair of
// cells is evaluated by one owner: the lower index if the pair is in both
// cells' lists, else the cell whose list holds it.
// ---------------------------------------------------------------------------
struct ForceArgs {
    int n_leaves;
    int64_t n;
    const int* l_begin;
    const int* l_count;
    const double* l_origin;
    const double* l_hlist;
    const int* l_dom;
    const int* l_off;
    const ListEntry* list;
    const int* l_sorted;
    const void* pos4;
    const void* fv4;
    const void* hf;
    const float* skey;
    const uint16_t* sidx;
    const DomainInfo* di;
    double* ax;
    double* ay;
    double* az;
    double* dudt;
    int32_t* nngb;      // #{j : r_ij < H_i} incl. self at the final H (may be NULL)
    unsigned long long* counters;
    const double* margin;  // list margin: twice the largest displacement since the lists were built
    const int* gate;    // graph mode: run only if *gate == 1 (NULL: always run)
    const int* nl_dev;  // graph mode: leaf count read from the device (NULL: n_leaves)
    const int* wide;        // leaves with lists above *wide_min (NULL: all are taken as such)
    const int* n_wide_dev;  // their number, later their classes' (FI_NWIDE, FI_WIDECLASS)
    const int* wide_min;
    int n_wide;
    int persistent;
};

template <typename T> struct vec2t;
template <> struct vec2t<float> { typedef float2 type; };
template <> struct vec2t<double> { typedef double2 type; };

// One staged neighbour cell of the force stage.
template <typename T>
struct FSlots {
    typename vec4<T>::type p[64];   // x, y, z (B frame), H^2
    typename vec4<T>::type v[64];   // vx, vy, vz, k = A (8/pi) / H^4
    typename vec2t<T>::type mh[64]; // m, 1/H
    T acc[4][64];                   // j-side sums
    int jl[64];                     // local index in B
    int jn[64];                     // j-side neighbour counts (r < H_j)
};

// neighbour cells per two-phase batch (force), and the occupancy target:
// one cell per batch keeps the LDS at 6 KB per wave, and 5 waves per SIMD
// (96 VGPRs, spills outside the pair loops) measured fastest
#ifndef SPH_NTF_F32
#define SPH_NTF_F32 1
#endif
#ifndef SPH_FORCE_WAVES
#define SPH_FORCE_WAVES 5
#endif
#define NTF(T) (sizeof(T) == 4 ? SPH_NTF_F32 : 1)

template <typename T>
struct FTile {
    FSlots<T> s[NTF(T)];
    EBatch<T> e;
};

// Evaluate one pair (i, j) known to be within max(H_i, H_j); d = x_i - x_j.
// Counts the pair for i if r < H_i (and, with JSIDE, for j if r < H_j).
template <typename T, bool COMP, bool JSIDE>
__device__ inline void force_eval(T dx, T dy, T dz, T r2, T mi, T h2i, T ihi, T ki, T vxi, T vyi, T vzi,
                                  const FSlots<T>& sl, int o, FAcc<T, COMP>& ai, FSlots<T>* slw, int& ni)
{
    const typename vec4<T>::type pj = sl.p[o];
    const typename vec4<T>::type fj = sl.v[o];
    const typename vec2t<T>::type mh = sl.mh[o];
    if (r2 < h2i) ni++;
    if (JSIDE && r2 < pj.w) atomicAdd(&slw->jn[o], 1);
    if (!(r2 > T(0))) return;  // coincident particles exert no force
    const T ir = fast_rsqrt(r2);
    const T r = r2 * ir;
    const T Fi = ki * spline_dw(r * ihi);      // A_i dW/dr(r, H_i)
    const T Fj = fj.w * spline_dw(r * mh.y);   // A_j dW/dr(r, H_j)
    const T F = (Fi + Fj) * ir;
    const T dvdr = ((vxi - fj.x) * dx + (vyi - fj.y) * dy + (vzi - fj.z) * dz) * ir;
    const T mjF = mh.x * F;
    ai.ax.add(-mjF * dx);
    ai.ay.add(-mjF * dy);
    ai.az.add(-mjF * dz);
    ai.du.add(mh.x * Fi * dvdr);
    if (JSIDE) {
        const T miF = mi * F;
        atomicAdd(&slw->acc[0][o], miF * dx);
        atomicAdd(&slw->acc[1][o], miF * dy);
        atomicAdd(&slw->acc[2][o], miF * dz);
        atomicAdd(&slw->acc[3][o], mi * Fj * dvdr);
    }
}

template <typename T>
__device__ inline void stage_force_j(FSlots<T>& sl, int slot, const typename vec4<T>::type& p,
                                     const typename vec4<T>::type& f, T h, int jl)
{
    const T ih = fast_rcp(h);
    typename vec4<T>::type q = p, g = f;
    q.w = h * h;
    g.w = f.w * T(INV_PI_8) * ih * ih * ih * ih;
    typename vec2t<T>::type mh;
    mh.x = p.w;
    mh.y = ih;
    sl.p[slot] = q;
    sl.v[slot] = g;
    sl.mh[slot] = mh;
    sl.acc[0][slot] = 0;
    sl.acc[1][slot] = 0;
    sl.acc[2][slot] = 0;
    sl.acc[3][slot] = 0;
    sl.jl[slot] = jl;
    sl.jn[slot] = 0;
}

// Flush the j-side sums of a staged cell (one atomic add per particle and
// quantity; skipped for particles that received nothing).
template <typename T>
__device__ inline unsigned long long flush_j(const ForceArgs& a, const FSlots<T>& sl, int bB, int len, int lane)
{
    int jcnt = 0;
    if (lane < len) {
        const int p = bB + sl.jl[lane];
        const T gx = sl.acc[0][lane], gy = sl.acc[1][lane], gz = sl.acc[2][lane], gu = sl.acc[3][lane];
        if (gx != T(0) || gy != T(0) || gz != T(0) || gu != T(0)) {
            atomicAdd(&a.ax[p], (double)gx);
            atomicAdd(&a.ay[p], (double)gy);
            atomicAdd(&a.az[p], (double)gz);
            atomicAdd(&a.dudt[p], (double)gu);
        }
        jcnt = sl.jn[lane];
        if (jcnt && a.nngb) atomicAdd(&a.nngb[p], jcnt);
    }
    return (unsigned long long)jcnt;
}

template <typename T, bool COMP, int PRUNE>
__device__ void force_leaf(const ForceArgs& a, int A, FTile<T>& tl, int lane)
{
    typedef typename vec4<T>::type V4;
    constexpr int NT = NTF(T);
    const V4* pos4 = (const V4*)a.pos4;
    const V4* fv4 = (const V4*)a.fv4;
    const T* hf = (const T*)a.hf;
    const int bA = a.l_begin[A], nA = a.l_count[A];
    const double oA[3] = {a.l_origin[3 * A], a.l_origin[3 * A + 1], a.l_origin[3 * A + 2]};
    const DomainInfo& I = a.di[a.l_dom[A]];
    const int e0 = a.l_off[A], e1 = a.l_off[A + 1];
    const double mg = *a.margin;  // list margin (see density_leaf)
    unsigned long long npairs = 0, ndens_w = 0;
    for (int c0 = 0; c0 < nA; c0 += 64) {
        const int nc = min(64, nA - c0);
        const int lg = chunk_log2(nc);
        const int CI = 1 << lg, G = 64 >> lg;
        const int ii = lane & (CI - 1), jg = lane >> lg;
        const bool vi = ii < nc;
        const int i = bA + c0 + (vi ? ii : 0);
        const V4 pi = pos4[i];
        const V4 fi = fv4[i];
        const T Hi = hf[i];
        const T h2i = Hi * Hi, ihi = T(1) / Hi;
        const T ki = fi.w * T(INV_PI_8) * ihi * ihi * ihi * ihi;
        FAcc<T, COMP> ai;
        int nni = (jg == 0 && vi) ? 1 : 0;  // neighbour count of i, self included
        const double hA = wave_max(vi ? (double)Hi : 0.0);
        const T big = T(1e30);
        const T bxl = wave_min_t<T>(vi ? pi.x : big), bxh = wave_max_t<T>(vi ? pi.x : -big);
        const T byl = wave_min_t<T>(vi ? pi.y : big), byh = wave_max_t<T>(vi ? pi.y : -big);
        const T bzl = wave_min_t<T>(vi ? pi.z : big), bzh = wave_max_t<T>(vi ? pi.z : -big);
        FSlots<T>& s0l = tl.s[0];

        // the cell's own pairs
        if (nA <= 64) {
            // triangular sweep over the unordered pairs of the cell
            if (lane < nA) stage_force_j<T>(s0l, lane, pos4[bA + lane], fv4[bA + lane], hf[bA + lane], lane);
            wave_sync();
            const int steps = nA / 2;  // pair distances 1..floor(n/2)
            const bool even = (nA & 1) == 0;
            for (int t = jg; t < steps; t += G) {
                int b = ii + 1 + t;
                if (b >= nA) b -= nA;
                const bool ok = vi && !(even && t == steps - 1 && ii >= nA / 2);
                if (ok) {
                    const V4 pj = s0l.p[b];
                    const T dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
                    const T r2 = dx * dx + dy * dy + dz * dz;
                    if (r2 < fmax(h2i, pj.w)) {
                        force_eval<T, COMP, true>(dx, dy, dz, r2, pi.w, h2i, ihi, ki, fi.x, fi.y, fi.z, s0l, b, ai,
                                                  &s0l, nni);
                        npairs++;
                    }
                }
            }
            wave_sync();
            if (jg == 0 && vi) {
                ai.ax.add(s0l.acc[0][ii]);
                ai.ay.add(s0l.acc[1][ii]);
                ai.az.add(s0l.acc[2][ii]);
                ai.du.add(s0l.acc[3][ii]);
                nni += s0l.jn[ii];
            }
            wave_sync();
        } else {
            // large cell: gather over all j != i of the cell (i side only)
            for (int p0 = 0; p0 < nA; p0 += 64) {
                const int len = min(64, nA - p0);
                if (lane < len) {
                    const int p = bA + p0 + lane;
                    stage_force_j<T>(s0l, lane, pos4[p], fv4[p], hf[p], p0 + lane);
                }
                wave_sync();
                for (int t = jg; t < len; t += G) {
                    if (!vi || p0 + t == c0 + ii) continue;
                    const V4 pj = s0l.p[t];
                    const T dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
                    const T r2 = dx * dx + dy * dy + dz * dz;
                    if (r2 < fmax(h2i, pj.w)) {
                        force_eval<T, COMP, false>(dx, dy, dz, r2, pi.w, h2i, ihi, ki, fi.x, fi.y, fi.z, s0l, t,
                                                   ai, nullptr, nni);
                        if (p0 + t > c0 + ii) npairs++;
                    }
                }
                wave_sync();
            }
        }

        // pairs with other cells
        for (int eb = e0; eb < e1; eb += 64) {
            const int nbt = min(64, e1 - eb);
            const double* hl = a.l_hlist;
            const int nv = load_batch<T>(a.list, eb, nbt, lane, a.l_begin, a.l_count, a.l_origin, oA, I,
                                         [&](const ListEntry& E) {
                                             const int B = E.B;
                                             if (B == A) return false;
                                             if (B < A && E.dist < hl[B]) return false;  // owned by B
                                             return E.dist < fmax(hA + mg, hl[B]);
                                         },
                                         tl.e, hl, A);
            V4 pf, ff;
            T hh = T(1);
            if (PRUNE == PRUNE_BOX && nv > 0) {
                const int n0 = tl.e.n[0];
                if (lane < n0) {
                    const int p = tl.e.b[0] + lane;
                    pf = pos4[p];
                    ff = fv4[p];
                    hh = hf[p];
                }
            }
            for (int k0 = 0; k0 < nv; k0 += NT) {
                unsigned long long msk[NT];
                T tox[NT], toy[NT], toz[NT];
                int tlen[NT], tbB[NT];
#pragma unroll
                for (int u = 0; u < NT; u++) {
                    msk[u] = 0ull;
                    tox[u] = toy[u] = toz[u] = T(0);
                    tlen[u] = 0;
                    tbB[u] = 0;
                    const int k = k0 + u;
                    if (k >= nv) continue;
                    FSlots<T>& sl = tl.s[u];
                    const int bB = tl.e.b[k], nB = tl.e.n[k];
                    const T dox = tl.e.ox[k], doy = tl.e.oy[k], doz = tl.e.oz[k];
                    tox[u] = dox;
                    toy[u] = doy;
                    toz[u] = doz;
                    tbB[u] = bB;
                    const T xi = pi.x - dox, yi = pi.y - doy, zi = pi.z - doz;
                    if (PRUNE == PRUNE_BOX && nB <= 64) {
                        const V4 pj = pf, fj = ff;
                        const T hj = hh;
                        if (k + 1 < nv) {
                            const int n1 = tl.e.n[k + 1];
                            if (lane < n1) {
                                const int p = tl.e.b[k + 1] + lane;
                                pf = pos4[p];
                                ff = fv4[p];
                                hh = hf[p];
                            }
                        }
                        const T Rj = fmax((T)hA, hj) * T(1.00001);
                        const bool in = lane < nB && box_d2<T>(pj.x, pj.y, pj.z, bxl - dox, byl - doy, bzl - doz,
                                                                bxh - dox, byh - doy, bzh - doz) < Rj * Rj;
                        const unsigned long long mk = __ballot(in);
                        if (in) stage_force_j<T>(sl, mask_rank(mk, lane), pj, fj, hj, lane);
                        const int len = __popcll(mk);
                        tlen[u] = len;
                        wave_sync();
                        if (vi) {
                            unsigned long long m = 0ull;
                            for (int s = 0, t = jg; t < len; s++, t += G) {
                                const V4 q = sl.p[t];
                                const T dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
                                if (dx * dx + dy * dy + dz * dz < fmax(h2i, q.w)) m |= 1ull << s;
                            }
                            msk[u] = m;
                            npairs += __popcll(m);
                        }
                    } else {
                        // sorted-axis window (or a cell too large for one tile): one phase
                        const T R = fmax((T)hA, tl.e.R[k]);
                        int lo = 0, hi = nB;
                        const int dir = tl.e.dir[k];
                        const bool srt = PRUNE == PRUNE_SORTED && a.l_sorted[tl.e.B[k]] && nB <= 64;
                        if (srt) {
                            double uu[3];
                            sph_dir(dir, uu);
                            const float ki_ = (float)((double)xi * uu[0] + (double)yi * uu[1] + (double)zi * uu[2]);
                            const float Rf = (float)R;
                            float kmin = wave_minf(vi ? ki_ - Rf : INFINITY);
                            float kmax = wave_maxf(vi ? ki_ + Rf : -INFINITY);
                            const float eps = 1e-5f * (fabsf(kmin) + fabsf(kmax)) + 1e-6f * Rf;
                            sorted_window(a.skey, a.n, dir, bB, nB, lane, kmin - eps, kmax + eps, lo, hi);
                        }
                        for (int p0 = lo; p0 < hi; p0 += 64) {
                            const int len = min(64, hi - p0);
                            if (lane < len) {
                                const int t = p0 + lane;
                                const int jl = srt ? (int)a.sidx[(int64_t)dir * a.n + bB + t] : t;
                                const int p = bB + jl;
                                stage_force_j<T>(sl, lane, pos4[p], fv4[p], hf[p], jl);
                            }
                            wave_sync();
                            // group jg owns slots jg, jg+G, ...; lanes of a group rotate over them
                            const int Lg = (jg < len) ? (len - jg + G - 1) / G : 0;
                            const int Lmax = (len + G - 1) / G;
                            const int s0 = (Lg > 0) ? ii % Lg : 0;
                            for (int t = 0; t < Lmax; t++) {
                                if (vi && t < Lg) {
                                    int s = s0 + t;
                                    if (s >= Lg) s -= Lg;
                                    const int o = jg + G * s;
                                    const V4 q = sl.p[o];
                                    const T dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
                                    const T r2 = dx * dx + dy * dy + dz * dz;
                                    if (r2 < fmax(h2i, q.w)) {
                                        force_eval<T, COMP, true>(dx, dy, dz, r2, pi.w, h2i, ihi, ki, fi.x, fi.y,
                                                                  fi.z, sl, o, ai, &sl, nni);
                                        npairs++;
                                    }
                                }
                            }
                            wave_sync();
                            ndens_w += flush_j<T>(a, sl, bB, len, lane);
                            wave_sync();
                        }
                        if (PRUNE == PRUNE_BOX && k + 1 < nv) {
                            const int n1 = tl.e.n[k + 1];
                            if (lane < n1) {
                                const int p = tl.e.b[k + 1] + lane;
                                pf = pos4[p];
                                ff = fv4[p];
                                hh = hf[p];
                            }
                        }
                    }
                }
                // phase 2: in-range pairs only, each lane starting at its own
                // offset so that the lanes of a group touch different j
#pragma unroll
                for (int u = 0; u < NT; u++) {
                    const unsigned long long m = msk[u];
                    if (__ballot(m != 0ull) == 0ull) continue;
                    FSlots<T>& sl = tl.s[u];
                    const T xi = pi.x - tox[u], yi = pi.y - toy[u], zi = pi.z - toz[u];
                    const int len = tlen[u];
                    const int Lg = (jg < len) ? (len - jg + G - 1) / G : 0;
                    const int r0 = (Lg > 0) ? ii % Lg : 0;
                    unsigned long long mh = (r0 > 0) ? (m >> r0) : m;
                    unsigned long long ml = (r0 > 0) ? (m & ((1ull << r0) - 1ull)) : 0ull;
                    while (mh | ml) {
                        int s;
                        if (mh) {
                            s = r0 + __ffsll((long long)mh) - 1;
                            mh &= mh - 1;
                        } else {
                            s = __ffsll((long long)ml) - 1;
                            ml &= ml - 1;
                        }
                        const int o = jg + G * s;
                        const V4 q = sl.p[o];
                        const T dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
                        force_eval<T, COMP, true>(dx, dy, dz, dx * dx + dy * dy + dz * dz, pi.w, h2i, ihi, ki, fi.x,
                                                  fi.y, fi.z, sl, o, ai, &sl, nni);
                    }
                }
                wave_sync();
#pragma unroll
                for (int u = 0; u < NT; u++)
                    if (tlen[u] > 0) ndens_w += flush_j<T>(a, tl.s[u], tbB[u], tlen[u], lane);
                wave_sync();
            }
            wave_sync();
        }
        double sx = ai.ax.total(), sy = ai.ay.total(), sz = ai.az.total(), su = ai.du.total();
        for (int off = CI; off < 64; off <<= 1) {
            sx += __shfl_xor(sx, off);
            sy += __shfl_xor(sy, off);
            sz += __shfl_xor(sz, off);
            su += __shfl_xor(su, off);
        }
        for (int off = CI; off < 64; off <<= 1) nni += __shfl_xor(nni, off);
        if (jg == 0 && vi) {
            atomicAdd(&a.ax[i], sx);
            atomicAdd(&a.ay[i], sy);
            atomicAdd(&a.az[i], sz);
            atomicAdd(&a.dudt[i], su);
            if (a.nngb) atomicAdd(&a.nngb[i], nni);
            ndens_w += nni;
        }
    }
    npairs = wave_sum(npairs);
    ndens_w = wave_sum(ndens_w);
    if (lane == 0 && npairs) count_add(a.counters, PART_NFORCE, npairs);
    if (lane == 0 && ndens_w) count_add(a.counters, PART_NDENS_F, ndens_w);
}

template <typename T, bool COMP, int PRUNE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SPH_FORCE_WAVES, 8))) void k_force(ForceArgs a)
{
    __shared__ FTile<T> tiles[WAVES_PER_WG];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (a.gate && uniform(*a.gate) != 1) return;
    const int nL = a.nl_dev ? uniform(*a.nl_dev) : a.n_leaves;
    if (!a.persistent) {
        const int A = uniform(xcd_block(blockIdx.x, gridDim.x) * WAVES_PER_WG + w);
        if (A >= nL) return;
        force_leaf<T, COMP, PRUNE>(a, A, tiles[w], lane);
        return;
    }
    int k = 0;
    for (int it = 0; it <= nL; it++) {
        const int A = xq_pop(&a.counters[XQ_FORCE], nL, k, lane);
        if (A < 0) break;
        force_leaf<T, COMP, PRUNE>(a, A, tiles[w], lane);
    }
}

// ---------------------------------------------------------------------------
// Gather-form force: each particle of leaf A sums its own pairs r < max(H_i,
// H_j) of eqs. (dvdt) and (dudt) over the cells of A's symmetric list.  Every
// pair is evaluated from both sides (twice the pair arithmetic of the
// pairs-once form) but nothing is accumulated on the j side, so there are no
// global atomics and each output is written once.  Candidate stream,
// matrix-unit range tests (against H_i and H_j) and pair-parallel sums as in
// the density, and bound by VALU issue (active in 84% of the cycles at the 4
// waves per SIMD its LDS holds): 1.1e4 VALU instructions per leaf at 256^3
// clustered (2.6e4 with a ballot loop over the particles per tile), 12.9 -> 9.45
// ms; 64^3 FP64 1.33 -> 0.55 ms.
// ---------------------------------------------------------------------------
template <typename T>
struct GTile {
    typename vec4<T>::type cand[4 * FORCE_ROW];  // j in A's frame: x, y, z, m
    typename vec4<T>::type cv[4 * FORCE_ROW];    // vx, vy, vz, k_j = -6 A_j (8/pi) / H_j^4 (first the particle's index)
    T ch[4 * FORCE_ROW];                         // 1/H_j
    union {
        float c[2][4 * FORCE_ROW];               // row constants of the range tests
        uint16_t list[PAIR_CAP];        // then the pairs
    };
    typename vec4<T>::type si[64];      // i of A: x, y, z (A frame), 1/H_i
    typename vec4<T>::type sv[64];      // vx, vy, vz, k_i
    double sum[4][64];                  // dv/dt, du/dt
    int cnt[64];                        // pairs within H_i
    EFlat<T, SPH_BATCH> e;
};
struct GTile64 : GTile<double> {
    float4 fc[4 * FORCE_ROW];
};
template <typename T> struct gtile { typedef GTile<T> type; };
template <> struct gtile<double> { typedef GTile64 type; };

template <typename T, int NW>
__device__ __forceinline__ void force_leaf_gather(const ForceArgs& a, int A, typename gtile<T>::type* tiles, int lane, int wave)
{
    typename gtile<T>::type& L = tiles[wave];
    typedef typename vec4<T>::type V4;
    const V4* pos4 = (const V4*)a.pos4;
    const V4* fv4 = (const V4*)a.fv4;
    const T* hf = (const T*)a.hf;
    const int bA = a.l_begin[A], nA = a.l_count[A];
    const double oA[3] = {a.l_origin[3 * A], a.l_origin[3 * A + 1], a.l_origin[3 * A + 2]};
    const DomainInfo& I = a.di[a.l_dom[A]];
    const int ea = a.l_off[A], ne = a.l_off[A + 1] - ea;
    const int e0 = ea + (int)((long long)ne * wave / NW), e1 = ea + (int)((long long)ne * (wave + 1) / NW);
    const double mg = *a.margin;  // list margin (see density_leaf)
    const T big = T(1e30);
    unsigned long long npairs = 0, ndens_w = 0, nself = 0;
    for (int c0 = 0; c0 < nA; c0 += 64) {
        const int nc = min(64, nA - c0);
        const bool vi = lane < nc;
        const int i = bA + c0 + (vi ? lane : 0);
        const int nb = (nc + 15) >> 4;
        const V4 pi = pos4[i];
        const T Hi = hf[i];
        const double hA = wave_max(vi ? (double)Hi : 0.0);
        T bxl = wave_min_t<T>(vi ? pi.x : big), bxh = wave_max_t<T>(vi ? pi.x : -big);
        T byl = wave_min_t<T>(vi ? pi.y : big), byh = wave_max_t<T>(vi ? pi.y : -big);
        T bzl = wave_min_t<T>(vi ? pi.z : big), bzh = wave_max_t<T>(vi ? pi.z : -big);
        // scale: the leaf's box and its largest H are of order 1 below
        const T sc = pow2_scale(fmax((T)hA, fmax(fmax(fmax(-bxl, bxh), fmax(-byl, byh)), fmax(-bzl, bzh))));
        bxl *= sc, bxh *= sc, byl *= sc, byh *= sc, bzl *= sc, bzh *= sc;
        const T hAm = (T)(hA * (1.0 + 1e-5)) * sc;
        bf16x4 bt[4];
        int nmax = 0;  // pairs within max(H_i, H_j), self included, of the lane's runs
        {
            V4 q = pi;
            q.x *= sc, q.y *= sc, q.z *= sc;
            const float x = (float)q.x, y = (float)q.y, z = (float)q.z, h = (float)(Hi * sc);
            const float p2 = x * x + y * y + z * z;
            const bool on = vi && p2 < 1e30f;
            nself += __popcll(__ballot(on));
            const float xi = on ? x : 0.f, yi = on ? y : 0.f, zi = on ? z : 0.f;
            const float ci = on ? p2 * (1.0f - PAIR_EPS) - 1e-30f : 1e30f;
            test_operand(xi, yi, zi, ci, on ? -h * h * (1.0f + PAIR_EPS) : 0.f, (float4*)L.cand, lane, bt);
            q.w = T(1) / (Hi * sc);
            L.si[lane] = q;
            L.sv[lane] = fv4[i];
            for (int k = 0; k < 4; k++) L.sum[k][lane] = 0.0;
            L.cnt[lane] = 0;
        }
        // the sums of one run of pairs
        auto eval = [&](const uint16_t* list, int n) {
            const int K = (n + 63) >> 6;
            int cur = -1, cnt = 0;
            double ax = 0.0, ay = 0.0, az = 0.0, du = 0.0;
            V4 p, f;
            auto flush = [&]() {
                lds_add(&L.sum[0][cur], ax);
                lds_add(&L.sum[1][cur], ay);
                lds_add(&L.sum[2][cur], az);
                lds_add(&L.sum[3][cur], du);
                lds_add(&L.cnt[cur], cnt);
            };
            for (int e = lane * K; e < min(lane * K + K, n); e++) {
                const int code = list[e], ii = code >> 7, j = code & 127;
                if (ii != cur) {
                    if (cur >= 0) flush();
                    cur = ii;
                    p = L.si[ii];
                    f = L.sv[ii];
                    ax = ay = az = du = 0.0;
                    cnt = 0;
                }
                const V4 q = L.cand[j], fj = L.cv[j];
                const T ihj = L.ch[j];
                const T dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
                const T r2 = dx * dx + dy * dy + dz * dz;
                // the particle itself and coincident ones exert no force:
                // at r2 = 0 the clamp gives r = 0, dW/dr(0) = 0 and d = 0,
                // so every term below is an exact zero (no branch)
                const T ir = fast_rsqrt(fmax(r2, sizeof(T) == 8 ? T(1e-300) : T(1e-30)));
                const T r = r2 * ir, qi = r * p.w, qj = r * ihj;
                const T Fi = f.w * spline_dw6(qi);   // A_i dW/dr(r, H_i)
                const T Fj = fj.w * spline_dw6(qj);  // A_j dW/dr(r, H_j)
                // (a pair let in by the tests' margin adds nothing, whatever its
                // velocities and factors)
                const bool in = fmin(qi, qj) < T(1);
                const T F = in ? (Fi + Fj) * ir : T(0);
                const T dvdr = ((f.x - fj.x) * dx + (f.y - fj.y) * dy + (f.z - fj.z) * dz) * ir;
                const T mjF = q.w * F;
                ax -= (double)(mjF * dx);
                ay -= (double)(mjF * dy);
                az -= (double)(mjF * dz);
                du += (double)(in ? q.w * Fi * dvdr : T(0));
                cnt += qi < T(1);
                nmax += in;
            }
            if (cur >= 0) flush();
        };
        auto run_tile = [&](int len) {
            for (int j = len + lane; j < 4 * FORCE_ROW; j += 64) {
                V4 o;
                o.x = o.y = o.z = o.w = T(0);
                L.cand[j] = o;
                put_test<T>(L, j, T(0), T(0), T(0));
                L.c[0][test_slot<FORCE_ROW>(j)] = L.c[1][test_slot<FORCE_ROW>(j)] = 1e30f;
            }
            wave_sync();
            // velocities and factors of the candidates: in flight during the tests
            V4 v0, v1;
            if (lane < len) v0 = fv4[((const uint32_t*)&L.cv[lane])[0]];
            if (lane + 64 < len) v1 = fv4[((const uint32_t*)&L.cv[lane + 64])[0]];
            uint32_t M[4] = {0u, 0u, 0u, 0u};
            tile_masks<true, FORCE_ROW>(L.c[0], L.c[1], [&](int j) { return get_test<T>(L, j, lane); }, bt, nb, lane, M);
            for_pairs<FORCE_ROW>(M, L.list, lane, [&]() {
                if (lane < len) L.cv[lane] = v0;
                if (lane + 64 < len) L.cv[lane + 64] = v1;
            }, eval);
            wave_sync();
        };
        const uint32_t last = (uint32_t)(a.n - 1);
        const double* hl = a.l_hlist;
        int ncand = 0, eb = e0, p0 = 0, total = 0, start = 0;
        uint32_t jp = 0;
        V4 o, pf;
        T hp;
        auto load = [&](int p) {
            o = L.e.o[stream_cell(p, start)];
            jp = min((uint32_t)(p + lane + unpack_int(o.w)), last);
            pf = pos4[jp];
            hp = hf[jp];
        };
        while (true) {
            if (p0 >= total) {  // next batch of cells
                for (total = 0; eb < e1 && total == 0; eb += SPH_BATCH) {
                    wave_sync();
                    total = load_batch_flat<T>(a.list, eb, min(SPH_BATCH, e1 - eb), lane, a.l_begin, a.l_count, a.l_origin, oA, I,
                                               sc, [&](const ListEntry& E) { return E.dist < fmax(hA + mg, hl[E.B]); },
                                               L.e, start);
                }
                p0 = 0;
                if (total > 0) load(0);
            }
            V4 q;
            T h;
            uint32_t j;
            unsigned long long mk = 0ull;
            if (total > 0) {
                q.x = fma_t(pf.x, sc, o.x);
                q.y = fma_t(pf.y, sc, o.y);
                q.z = fma_t(pf.z, sc, o.z);
                q.w = pf.w;
                h = hp * sc;
                j = jp;
                const T Rj = fmax(hAm, h * T(1.00001));
                mk = __ballot((p0 + lane < total) &
                              (box_d2<T>(q.x, q.y, q.z, bxl, byl, bzl, bxh, byh, bzh) < Rj * Rj));
                p0 += 64;
                if (p0 < total) load(p0);
            }
            const int nk = __popcll(mk);
            if (ncand + nk > 4 * FORCE_ROW || total == 0) {
                if (ncand > 0) run_tile(ncand);
                if (total == 0) break;
                ncand = 0;
            }
            if ((mk >> lane) & 1ull) {
                const int slot = ncand + lane_rank(mk);
                L.cand[slot] = q;
                ((uint32_t*)&L.cv[slot])[0] = j;  // its velocity and factor are loaded with the tile
                L.ch[slot] = fast_rcp(h);
                const float hs = (float)h;
                const float cj = put_test<T>(L, slot, q.x, q.y, q.z) * (1.0f - PAIR_EPS);
                L.c[0][test_slot<FORCE_ROW>(slot)] = cj;
                L.c[1][test_slot<FORCE_ROW>(slot)] = cj - hs * hs * (1.0f + PAIR_EPS);
            }
            ncand += nk;
        }
        wave_sync();
        npairs += (unsigned long long)nmax;
        if (NW > 1) __syncthreads();
        if (vi && wave == 0) {
            double t[4];
            for (int k = 0; k < 4; k++) t[k] = L.sum[k][lane];
            int cnt = L.cnt[lane];
            for (int w = 1; w < NW; w++) {
                for (int k = 0; k < 4; k++) t[k] += tiles[w].sum[k][lane];
                cnt += tiles[w].cnt[lane];
            }
            a.ax[i] = t[0];
            a.ay[i] = t[1];
            a.az[i] = t[2];
            a.dudt[i] = t[3];
            if (a.nngb) a.nngb[i] = cnt;
            ndens_w += (unsigned long long)cnt;
        }
        if (NW > 1) __syncthreads();
        else wave_sync();
    }
    npairs = wave_sum(npairs);
    ndens_w = wave_sum(ndens_w);
    // ordered pairs, the particles themselves excluded (each is found by the
    // wave that holds the leaf's own entry: the sum modulo 2^64 is right)
    if (wave == 0) npairs -= nself;
    if (lane == 0 && npairs) count_add(a.counters, PART_NFORCE, npairs);
    if (lane == 0 && ndens_w) count_add(a.counters, PART_NDENS_F, ndens_w);
}

template <typename T, int WPE, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE, 8))) void k_force_gather(ForceArgs a)
{
    __shared__ typename gtile<T>::type tiles[NW];
    const int lane = threadIdx.x & 63;
    if (a.gate && uniform(*a.gate) != 1) return;
    if (NW > 1) {
        for_wide_leaves<NW>(a, [&](int A, int wave) __attribute__((always_inline)) { force_leaf_gather<T, NW>(a, A, tiles, lane, wave); });
        return;
    }
    if (!a.persistent) {
        const int A = tile_leaf<NW>(a, blockIdx.x);
        if (A >= 0) force_leaf_gather<T, NW>(a, A, tiles, lane, 0);
        return;
    }
    const int nL = a.nl_dev ? uniform(*a.nl_dev) : a.n_leaves;
    int k = 0;
    for (int it = 0; it <= nL; it++) {
        const int A = xq_pop(&a.counters[XQ_FORCE], nL, k, lane);
        if (A < 0) break;
        if (a.l_off[A + 1] - a.l_off[A] > uniform(*a.wide_min)) continue;
        force_leaf_gather<T, NW>(a, A, tiles, lane, 0);
    }
}

// ---------------------------------------------------------------------------
// Integrator (kick-drift-kick) and FP64 conservation sums.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_kick_drift(int64_t n, double* x, double* y, double* z, double* vx, double* vy,
                                                    double* vz, double* u, const double* __restrict__ ax,
                                                    const double* __restrict__ ay, const double* __restrict__ az,
                                                    const double* __restrict__ dudt, const int32_t* __restrict__ dom,
                                                    const DomainInfo* __restrict__ di, double dt,
                                                    unsigned long long* vmax_bits, double* H, double gm1)
{
    __shared__ double wmax[4];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double sp = 0.0;
    if (i < n) {
        const double h = 0.5 * dt;
        const double v[3] = {vx[i] + ax[i] * h, vy[i] + ay[i] * h, vz[i] + az[i] * h};
        vx[i] = v[0];
        vy[i] = v[1];
        vz[i] = v[2];
        const double du = dudt[i];
        const double ui = u[i] + du * h;
        u[i] = ui;
        if (H && ui > 0.0) {
            // start of the H iteration carried along the flow (see k_h_drift)
            const double e = fmin(fmax(-dt * du / (3.0 * gm1 * ui), -0.6931471805599453), 0.6931471805599453);
            H[i] *= exp(e);
        }
        sp = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
        const DomainInfo& I = di[dom ? dom[i] : 0];
        double* c[3] = {x, y, z};
        for (int a = 0; a < 3; a++) {
            double q = c[a][i] + v[a] * dt;
            q -= I.L[a] * floor(q / I.L[a]);
            if (q >= I.L[a]) q -= I.L[a];
            if (q < 0.0) q = 0.0;
            c[a][i] = q;
        }
    }
    // largest speed of the drift (non-negative doubles order like their bits)
    for (int off = 32; off > 0; off >>= 1) sp = fmax(sp, __shfl_xor(sp, off));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = sp;
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = wmax[0];
        for (int w = 1; w < (int)(blockDim.x >> 6); w++) b = fmax(b, wmax[w]);
        const unsigned long long bits = (unsigned long long)__double_as_longlong(b);
        // most blocks are below the running maximum: skip their atomics
        if (bits > __atomic_load_n(vmax_bits, __ATOMIC_RELAXED)) atomicMax(vmax_bits, bits);
    }
}

// Start of the H iteration carried along the flow: with du/dt = (P/rho^2)
// drho/dt (the energy equation of Sec. 2 against the density sum) and P =
// (gamma-1) rho u, the fractional density change over dt is dt du/dt /
// ((gamma-1) u); rho H^3 stays constant, so H scales by the cube root.
__global__ __launch_bounds__(256) void k_h_drift(int64_t n, double* H, const double* __restrict__ u,
                                                 const double* __restrict__ dudt, double gm1, double dt)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double ui = u[i];
    if (!(ui > 0.0)) return;
    const double e = fmin(fmax(-dt * dudt[i] / (3.0 * gm1 * ui), -0.6931471805599453), 0.6931471805599453);
    H[i] *= exp(e);
}

struct KickArgs {
    const double *ax, *ay, *az, *dudt;
    double h;  // half the step
};

// partial[(d * chunks + chunk) * 5 + k]; chunks per box is chosen so that
// the grid holds about 4096 workgroups (at least 64 per box)
// With kick != nullptr the closing half kick of the step is applied first
// (v += a dt/2, u += du/dt dt/2 with kick = {ax, ay, az, dudt}) and the
// totals are those of the kicked state.
__global__ __launch_bounds__(256) void k_sums_partial(const int* __restrict__ ranges, const double* __restrict__ m,
                                                      double* vx, double* vy, double* vz, double* u,
                                                      double* partial, int chunks, KickArgs kick)
{
    __shared__ double red[5][256];
    const int d = blockIdx.y, ch = blockIdx.x, tid = threadIdx.x;
    const int b = ranges[d], e = ranges[d + 1];
    double s[5] = {0, 0, 0, 0, 0};
    for (int64_t i = b + (int64_t)ch * 256 + tid; i < e; i += (int64_t)chunks * 256) {
        if (kick.ax) {
            vx[i] += kick.ax[i] * kick.h;
            vy[i] += kick.ay[i] * kick.h;
            vz[i] += kick.az[i] * kick.h;
            u[i] += kick.dudt[i] * kick.h;
        }
        const double mm = m[i], v0 = vx[i], v1 = vy[i], v2 = vz[i];
        s[0] += mm;
        s[1] += mm * v0;
        s[2] += mm * v1;
        s[3] += mm * v2;
        s[4] += mm * (0.5 * (v0 * v0 + v1 * v1 + v2 * v2) + u[i]);
    }
    for (int k = 0; k < 5; k++) red[k][tid] = s[k];
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st)
            for (int k = 0; k < 5; k++) red[k][tid] += red[k][tid + st];
        __syncthreads();
    }
    if (tid < 5) partial[((int64_t)d * chunks + ch) * 5 + tid] = red[tid][0];
}

// One workgroup per box: strided partial sums over the chunks, then a tree
// in LDS (fixed order, so the totals are reproducible).
__global__ __launch_bounds__(256) void k_sums_final(const double* __restrict__ partial, double* out, int chunks)
{
    __shared__ double red[5][256];
    const int d = blockIdx.x, tid = threadIdx.x;
    double s[5] = {0, 0, 0, 0, 0};
    for (int ch = tid; ch < chunks; ch += 256)
        for (int k = 0; k < 5; k++) s[k] += partial[((int64_t)d * chunks + ch) * 5 + k];
    for (int k = 0; k < 5; k++) red[k][tid] = s[k];
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st)
            for (int k = 0; k < 5; k++) red[k][tid] += red[k][tid + st];
        __syncthreads();
    }
    if (tid < 5) out[5 * d + tid] = red[tid][0];
}

// Move the partial counts of the last interaction kernel into the counters
// (one workgroup of PART_N threads).
__device__ inline void fold_counts(unsigned long long* cnt)
{
    __shared__ unsigned long long red[PART_USED][PART_N / 64];
    const int tid = threadIdx.x;
    unsigned long long* line = cnt + CNT_PART + tid * PART_STRIDE;
    for (int k = 0; k < PART_USED; k++) {
        const unsigned long long v = line[k];
        if (v) line[k] = 0ull;
        const unsigned long long t = wave_sum(v);
        if ((tid & 63) == 0) red[k][tid >> 6] = t;
    }
    __syncthreads();
    const int to[PART_USED] = {CNT_UNCONV, CNT_NDENS, CNT_DEVAL, CNT_NFORCE, CNT_NDENS_F};
    if (tid == 0)
        for (int k = 0; k < PART_USED; k++)
            for (int w = 0; w < PART_N / 64; w++) cnt[to[k]] += red[k][w];
    __syncthreads();
}

__global__ __launch_bounds__(PART_N) void k_count_fold(unsigned long long* cnt) { fold_counts(cnt); }

// ---------------------------------------------------------------------------
// Host orchestration
// ---------------------------------------------------------------------------
static inline int blocks_for(int64_t n, int t) { return (int)((n + t - 1) / t); }

static int resident_wgs(sph_ctx* c)
{
    if (c->prm.persistent_wgs > 0) return c->prm.persistent_wgs;
    return 256 * 8;  // 256 CUs x 8 workgroups of 4 waves
}

// Leaf capacity of the per-leaf arrays: the grid of a captured launch covers
// it, and the kernels bound the work by the leaf count read on the device.
static int leaf_capacity(sph_ctx* c) { return (int)std::min<size_t>(c->l_begin.cap / sizeof(int), INT32_MAX / 2); }

// The flags and the counters, which lie side by side, in one copy.
struct FlagsCounters {
    int flags[FI_NFLAGS];
    unsigned long long cnt[CNT_N];
};
static sph_status read_flags(sph_ctx* c, FlagsCounters& fc)
{
    SPH_CHECK_HIP(hipMemcpyAsync(&fc, c->flags.p, sizeof(fc), hipMemcpyDeviceToHost, c->stream));
    SPH_CHECK_HIP(hipStreamSynchronize(c->stream));
    return SPH_OK;
}

static void dens_args(sph_ctx* c, const int* gate, bool graph, DensArgs& a, int& nb)
{
    memset(&a, 0, sizeof(a));
    a.n_leaves = c->n_leaves;
    a.n = c->n;
    a.l_begin = (const int*)c->l_begin.p;
    a.l_count = (const int*)c->l_count.p;
    a.l_origin = (const double*)c->l_origin.p;
    a.l_hlist = (const double*)c->l_hlist.p;
    a.l_dom = (const int*)c->l_dom.p;
    a.l_off = (const int*)c->l_off.p;
    a.list = (const ListEntry*)c->list.p;
    a.l_active = (int*)c->l_active.p;
    a.l_sorted = (const int*)c->l_sorted.p;
    a.pos4 = c->pos4.p;
    a.skey = (const float*)c->skey.p;
    a.sidx = (const uint16_t*)c->sidx.p;
    a.di = (const DomainInfo*)c->dom_d.p;
    a.m = c->P.m;
    a.H = c->P.H;
    a.rho = c->P.rho;
    a.drho = c->P.drho_dH;
    a.hlo = (double*)c->hlo.p;
    a.hhi = (double*)c->hhi.p;
    a.conv = (uint8_t*)c->conv.p;
    a.nngb = c->P.nngb;
    a.C_fac = pow(c->prm.kernel_gamma * c->prm.eta, 3.0);
    // FP32 sums resolve rho H^3 to about 1e-7 with compensation and a few
    // 1e-7 without; the residual test is not asked for more than that
    a.h_tol = c->prm.precision == SPH_FP64 ? c->prm.h_tol
              : std::max(c->prm.h_tol, c->prm.precision == SPH_FP32C ? SPH_FP32C_TOL_MIN : SPH_FP32_TOL_MIN);
    a.flags = (int*)c->flags.p;
    a.counters = (unsigned long long*)c->counters.p;
    a.gate = gate;
    a.margin = (const double*)c->dparam.p;
    a.nl_dev = graph ? (const int*)c->flags.p + FI_NLEAVES : nullptr;
    a.wide = (const int*)c->wide.p;
    a.n_wide_dev = (const int*)c->flags.p + FI_NWIDE;
    a.n_wide = graph ? 0 : c->n_wide;
    a.wide_min = (const int*)c->flags.p + FI_WIDEMIN;
    if (graph) a.n_leaves = 0;  // read on the device
    const int nl = graph ? leaf_capacity(c) : c->n_leaves;
    nb = blocks_for(nl, WAVES_PER_WG);
}

// The packed density and gather force kernels of the context's occupancy
// target (FP64: the defaults only).
// Workgroups of the wide launch and its waves per leaf; all: it takes every leaf.
static int wide_grid(sph_ctx* c, bool graph, bool& all, int& waves)
{
    const int nL = graph ? leaf_capacity(c) : c->n_leaves;
    all = c->n_leaves <= SPH_WIDE_ALL;
    waves = all && c->n_leaves > SPH_WIDE_FEW ? 4 : SPH_WIDE_WAVES;
    // (a captured launch covers any number of long lists)
    return all ? nL : graph ? std::min(nL, 1024) : c->n_wide;
}

static void launch_density_packed(sph_ctx* c, bool graph, DensArgs a)
{
    const bool f64 = c->prm.precision == SPH_FP64;
    const int nL = graph ? leaf_capacity(c) : c->n_leaves;
    bool all;
    int waves;
    const int nw = wide_grid(c, graph, all, waves);
    if (all) a.wide = nullptr;
    if (nw > 0 && waves == 4) {
        if (f64) k_density_packed<double, SPH_DENS_WAVES64, 4><<<nw, 256, 0, c->stream>>>(a);
        else k_density_packed<float, SPH_WIDE_OCC, 4><<<nw, 256, 0, c->stream>>>(a);
    } else if (nw > 0) {
        if (f64) k_density_packed<double, SPH_DENS_WAVES64, 8><<<nw, 512, 0, c->stream>>>(a);
        else k_density_packed<float, SPH_WIDE_OCC, 8><<<nw, 512, 0, c->stream>>>(a);
    }
    if (all) return;
    if (f64) {
        k_density_packed<double, SPH_DENS_WAVES64, 1><<<nL, 64, 0, c->stream>>>(a);
        return;
    }
    switch (c->prm.waves_density ? c->prm.waves_density : SPH_DENS_WAVES) {
    case 4: k_density_packed<float, 4, 1><<<nL, 64, 0, c->stream>>>(a); return;
    case 5: k_density_packed<float, 5, 1><<<nL, 64, 0, c->stream>>>(a); return;
    default: k_density_packed<float, 6, 1><<<nL, 64, 0, c->stream>>>(a); return;
    }
}

static void launch_force_gather(sph_ctx* c, bool graph, int nb, ForceArgs a)
{
    const bool f64 = c->prm.precision == SPH_FP64;
    bool all;
    int waves;
    const int nw = wide_grid(c, graph, all, waves);
    if (all) a.wide = nullptr;
    if (nw > 0 && waves == 4) {
        if (f64) k_force_gather<double, SPH_FORCEG_WAVES64, 4><<<nw, 256, 0, c->stream>>>(a);
        else k_force_gather<float, SPH_WIDE_OCC, 4><<<nw, 256, 0, c->stream>>>(a);
    } else if (nw > 0) {
        if (f64) k_force_gather<double, SPH_FORCEG_WAVES64, 8><<<nw, 512, 0, c->stream>>>(a);
        else k_force_gather<float, SPH_WIDE_OCC, 8><<<nw, 512, 0, c->stream>>>(a);
    }
    if (all) return;
    if (f64) k_force_gather<double, SPH_FORCEG_WAVES64, 1><<<nb, 64, 0, c->stream>>>(a);
    else k_force_gather<float, SPH_FORCEG_WAVES, 1><<<nb, 64, 0, c->stream>>>(a);
}

// Density sweeps run as a grid of one wave per leaf in every execution mode:
// the persistent queues were slower here (first sweep 10.2 against 10.0 ms
// at 256^3, and the later sweeps, with most leaves converged, pay a pop per
// leaf where a grid's workgroups of converged leaves exit at once).
static sph_status launch_density(sph_ctx* c, const int* gate, bool graph = false)
{
    DensArgs a;
    int nb = 0;
    dens_args(c, gate, graph, a, nb);
    if (c->prm.lists == SPH_LISTS_PARTICLE) return launch_density_plist(c, a);
    if (nb <= 0) return SPH_OK;
    const bool srt = c->prm.prune == SPH_PRUNE_SORTED;
    if (!srt) {
        launch_density_packed(c, graph, a);
        SPH_CHECK_LAUNCH();
        // leaves above 64 particles (cells that cannot be split further):
        // the chunked two-phase kernel over a plain grid
        if (c->max_leaf <= 64) return SPH_OK;
        a.big_only = 1;
        nb = blocks_for(graph ? leaf_capacity(c) : c->n_leaves, WAVES_PER_WG);
    }
    if (c->prm.precision == SPH_FP64) {
        if (srt) k_density<double, false, PRUNE_SORTED><<<nb, 256, 0, c->stream>>>(a);
        else k_density<double, false, PRUNE_BOX><<<nb, 256, 0, c->stream>>>(a);
    } else if (c->prm.precision == SPH_FP32C) {
        if (srt) k_density<float, true, PRUNE_SORTED><<<nb, 256, 0, c->stream>>>(a);
        else k_density<float, true, PRUNE_BOX><<<nb, 256, 0, c->stream>>>(a);
    } else {
        if (srt) k_density<float, false, PRUNE_SORTED><<<nb, 256, 0, c->stream>>>(a);
        else k_density<float, false, PRUNE_BOX><<<nb, 256, 0, c->stream>>>(a);
    }
    SPH_CHECK_LAUNCH();
    return SPH_OK;
}

static sph_status density_reset(sph_ctx* c)
{
    SPH_TRY(buf_ensure(c->hlo, (size_t)c->n * 8));
    SPH_TRY(buf_ensure(c->hhi, (size_t)c->n * 8));
    SPH_TRY(buf_ensure(c->conv, (size_t)c->n));
    k_density_reset<<<blocks_for(std::max<int64_t>(c->n, c->n_leaves), 256), 256, 0, c->stream>>>(
        c->n, c->n_leaves, (double*)c->hlo.p, (double*)c->hhi.p, (uint8_t*)c->conv.p, (int*)c->l_active.p, nullptr);
    SPH_CHECK_LAUNCH();
    c->st.relists = 0;
    c->st.t_density_kernels_ms = 0.0;
    c->st.n_density_launches = 0;
    c->st.n_dens_evals = 0;
    for (int k = 0; k < 8; k++) c->st.unconv_after[k] = -1;
    return SPH_OK;
}

// Host-driven sweeps: one sweep, read the counters, relist or rebuild if a
// smoothing length outgrew the lists or the grid, repeat until converged.
// `done_sweeps` sweeps were already run on the device (graph mode).
// FP32 modes: cells are split at the build until their extent is at most
// SPH_FP32_EXTENT_RATIO times their smallest H, which bounds the error of
// the cell-relative coordinates against H.  H can shrink far below its value
// at the build during the iteration (a poor initial guess); this flags a
// leaf that could still be split and whose extent (plus the motion since
// the build) now exceeds twice that ratio times its smallest converged H.
__global__ __launch_bounds__(256) void k_extent_check(int n_leaves, const int* __restrict__ l_begin,
                                                      const int* __restrict__ l_count, const double* __restrict__ l_lo,
                                                      const double* __restrict__ l_hi, const int* __restrict__ leaf_node,
                                                      const Node* __restrict__ nodes, int max_level,
                                                      const double* __restrict__ H, double grow, int* flags)
{
    const int A = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6));
    if (A >= n_leaves) return;
    const int lane = threadIdx.x & 63;
    const int b = l_begin[A], n = l_count[A];
    if (n < 2 || nodes[leaf_node[A]].level >= max_level) return;
    double hm = INFINITY;
    for (int p = b + lane; p < b + n; p += 64) hm = fmin(hm, H[p]);
    for (int off = 32; off > 0; off >>= 1) hm = fmin(hm, __shfl_xor(hm, off));
    const double ext = fmax(fmax(l_hi[3 * A] - l_lo[3 * A], l_hi[3 * A + 1] - l_lo[3 * A + 1]),
                            l_hi[3 * A + 2] - l_lo[3 * A + 2]) + grow;
    if (lane == 0 && ext > 2.0 * SPH_FP32_EXTENT_RATIO * hm) atomicOr(flags, FLAG_REBUILD);
}

// FLAG_REBUILD in *flag if a splittable leaf is too wide for its smallest
// converged H (FP32 cell-relative coordinates).
static sph_status extent_check(sph_ctx* c, int* flag)
{
    k_extent_check<<<blocks_for(c->n_leaves, 4), 256, 0, c->stream>>>(
        c->n_leaves, (const int*)c->l_begin.p, (const int*)c->l_count.p, (const double*)c->l_lo.p,
        (const double*)c->l_hi.p, (const int*)c->leaf_node.p, (const Node*)c->nodes.p, c->D, c->P.H, 2.0 * c->delta,
        flag);
    SPH_CHECK_LAUNCH();
    return SPH_OK;
}

static sph_status density_loop(sph_ctx* c, int done_sweeps, unsigned long long unconv0)
{
    int* flags = (int*)c->flags.p;
    unsigned long long* cnt = (unsigned long long*)c->counters.p;
    int sweeps = 0;
    unsigned long long unconv = unconv0;
    int fl = 0;
    unsigned long long nd = 0;  // CNT_NDENS as of the last sweep
    bool prec_rebuilt = false, swept = false;
    sph_status status = SPH_OK;
    for (sweeps = done_sweeps + 1; sweeps <= c->prm.max_h_iter; sweeps++) {
        SPH_CHECK_HIP(hipMemsetAsync(flags, 0, sizeof(int), c->stream));
        SPH_CHECK_HIP(hipMemsetAsync(&cnt[CNT_UNCONV], 0, 8, c->stream));
        SPH_CHECK_HIP(hipEventRecord(c->kev[0], c->stream));
        SPH_TRY(launch_density(c, nullptr));
        SPH_CHECK_HIP(hipEventRecord(c->kev[1], c->stream));
        k_count_fold<<<1, PART_N, 0, c->stream>>>(cnt);
        SPH_CHECK_LAUNCH();
        FlagsCounters fc;
        SPH_TRY(read_flags(c, fc));
        const unsigned long long* hc = fc.cnt;
        fl = fc.flags[FI_FLAGS];
        {
            float ms = 0.f;
            SPH_CHECK_HIP(hipEventElapsedTime(&ms, c->kev[0], c->kev[1]));
            c->st.t_density_kernels_ms += ms;
            c->st.n_density_launches++;
            c->st.n_dens_evals = (int64_t)hc[CNT_DEVAL];
        }
        unconv = hc[CNT_UNCONV];
        nd = hc[CNT_NDENS];
        swept = true;
        if (sweeps <= 8) c->st.unconv_after[sweeps - 1] = (int)std::min<unsigned long long>(unconv, INT32_MAX);
        if (fl & FLAG_BOX_SMALL) status = SPH_ERR_BOX_TOO_SMALL;
        // (inside sph_step the refresh of the next step takes this test
        // over: the lists are rebuilt then if the rule fails)
        if (unconv == 0 && c->prm.precision != SPH_FP64 && !prec_rebuilt && status == SPH_OK &&
            sweeps < c->prm.max_h_iter && !c->in_step) {
            SPH_CHECK_HIP(hipMemsetAsync(flags, 0, sizeof(int), c->stream));
            SPH_TRY(extent_check(c, flags));
            SPH_CHECK_HIP(hipMemcpyAsync(&fl, flags, sizeof(int), hipMemcpyDeviceToHost, c->stream));
            SPH_CHECK_HIP(hipStreamSynchronize(c->stream));
            if (fl & FLAG_REBUILD) {
                // converged on cells too coarse for the final H: rebuild once
                // and evaluate again from the converged H
                prec_rebuilt = true;
                unconv = 1;
                SPH_TRY(build_all(c));
                SPH_TRY(sort_all(c));
                k_density_reset<<<blocks_for(std::max<int64_t>(c->n, c->n_leaves), 256), 256, 0, c->stream>>>(
                    c->n, c->n_leaves, (double*)c->hlo.p, (double*)c->hhi.p, (uint8_t*)c->conv.p,
                    (int*)c->l_active.p, nullptr);
                SPH_CHECK_LAUNCH();
                SPH_CHECK_HIP(hipMemsetAsync(&cnt[CNT_NDENS], 0, 8, c->stream));
                c->st.rebuilds++;
                c->st.precision_rebuilds++;
                continue;
            }
        }
        if (unconv == 0) break;
        if ((fl & FLAG_REBUILD) || ((fl & FLAG_RELIST) && c->delta > 0.0)) {
            // a smoothing length outgrew the top grid, or outgrew its list
            // after particles moved since the build (the walk needs current
            // boxes): rebuild the cells and continue from the current H
            // (brackets restart)
            SPH_TRY(build_all(c));
            SPH_TRY(sort_all(c));
            k_density_reset<<<blocks_for(std::max<int64_t>(c->n, c->n_leaves), 256), 256, 0, c->stream>>>(
                c->n, c->n_leaves, (double*)c->hlo.p, (double*)c->hhi.p, (uint8_t*)c->conv.p, (int*)c->l_active.p, nullptr);
            SPH_CHECK_LAUNCH();
            SPH_CHECK_HIP(hipMemsetAsync(&cnt[CNT_NDENS], 0, 8, c->stream));
            c->st.rebuilds++;
        } else if (fl & FLAG_RELIST) {
            SPH_TRY(relist(c));
            c->st.relists++;
        }
    }
    if (!swept) {
        SPH_CHECK_HIP(hipMemcpyAsync(&nd, &cnt[CNT_NDENS], 8, hipMemcpyDeviceToHost, c->stream));
        SPH_CHECK_HIP(hipStreamSynchronize(c->stream));
    }
    c->st.sweeps = std::min(sweeps, c->prm.max_h_iter);
    c->st.n_unconverged = (int)unconv;
    c->st.n_dens = (int64_t)nd;
    c->dens_done = true;
    c->ghost_done = false;
    c->force_done = false;
    if (status != SPH_OK) return status;
    return unconv ? SPH_ERR_NOT_CONVERGED : SPH_OK;
}

// Density stage: the first sweeps run as a gated sequence on the device (the
// same gate the graph mode uses: after each sweep a one-thread kernel turns
// the gate to "converged" or "the host must take over"), so the common case
// costs one readback for the whole stage; the host loop continues from there
// when more sweeps, a relist or a rebuild are needed.
#define SPH_GATED_SWEEPS 3

__global__ void k_graph_begin(unsigned long long* cnt, int* flags, int* gate);
__global__ void k_sweep_end(unsigned long long* cnt, int* flags, int* gate, int more);

sph_status density_all(sph_ctx* c)
{
    if (!c->sorted) return SPH_ERR_STATE;
    SPH_CHECK_HIP(hipEventRecord(c->ev[0], c->stream));
    SPH_TRY(density_reset(c));
    int* gate = (int*)c->flags.p + FI_GATE;
    unsigned long long* cnt = (unsigned long long*)c->counters.p;
    int* flags = (int*)c->flags.p;
    const int sweeps = std::min(SPH_GATED_SWEEPS, c->prm.max_h_iter);
    k_graph_begin<<<1, 64, 0, c->stream>>>(cnt, flags, gate);
    SPH_CHECK_LAUNCH();
    SPH_CHECK_HIP(hipEventRecord(c->kev[0], c->stream));
    for (int k = 0; k < sweeps; k++) {
        SPH_TRY(launch_density(c, gate));
        k_sweep_end<<<1, PART_N, 0, c->stream>>>(cnt, flags, gate, k + 1 < sweeps);
        SPH_CHECK_LAUNCH();
    }
    SPH_CHECK_HIP(hipEventRecord(c->kev[1], c->stream));
    // the FP32 extent check of a call outside a step, read with the sweeps'
    // outcome (in the host loop, after a sweep of no particle, it cost that sweep
    // and three reads: cold run of 12^3 487 -> 400 us, stages at 127^3 3.75 -> 3.64 ms)
    const bool check = c->prm.precision != SPH_FP64 && !c->in_step;
    if (check) SPH_TRY(extent_check(c, flags + FI_EXTENT));
    FlagsCounters fc;
    SPH_TRY(read_flags(c, fc));
    const int* hfl = fc.flags;
    const unsigned long long* hc = fc.cnt;
    const int g = hfl[FI_GATE], fl = hfl[FI_FLAGS];
    const int done = (int)hc[CNT_GSWEEPS];
    {
        float ms = 0.f;
        SPH_CHECK_HIP(hipEventElapsedTime(&ms, c->kev[0], c->kev[1]));
        c->st.t_density_kernels_ms = ms;
    }
    c->st.n_density_launches = done;
    c->st.n_dens_evals = (int64_t)hc[CNT_DEVAL];
    for (int k = 0; k < 8; k++)
        c->st.unconv_after[k] = k < done && k < CNT_N - CNT_UHIST
                                    ? (int)std::min<unsigned long long>(hc[CNT_UHIST + k], INT32_MAX)
                                    : -1;
    sph_status st = SPH_OK;
    if (g == 1 && (!check || done >= c->prm.max_h_iter || !(hfl[FI_EXTENT] & FLAG_REBUILD))) {
        // converged (cells too coarse for the final H: the host loop rebuilds)
        c->st.sweeps = done;
        c->st.n_unconverged = 0;
        c->st.n_dens = (int64_t)hc[CNT_NDENS];
        c->dens_done = true;
        c->ghost_done = false;
        c->force_done = false;
    } else if (g == 1) {
        st = density_loop(c, done - 1, 1ull);
    } else {
        if (fl & FLAG_BOX_SMALL) {
            c->st.sweeps = done;
            c->st.n_unconverged = (int)std::min<unsigned long long>(hc[CNT_UNCONV], INT32_MAX);
            st = SPH_ERR_BOX_TOO_SMALL;
        } else {
            if ((fl & FLAG_REBUILD) || ((fl & FLAG_RELIST) && c->delta > 0.0)) {
                SPH_TRY(build_all(c));
                SPH_TRY(sort_all(c));
                k_density_reset<<<blocks_for(std::max<int64_t>(c->n, c->n_leaves), 256), 256, 0, c->stream>>>(
                    c->n, c->n_leaves, (double*)c->hlo.p, (double*)c->hhi.p, (uint8_t*)c->conv.p,
                    (int*)c->l_active.p, nullptr);
                SPH_CHECK_LAUNCH();
                SPH_CHECK_HIP(hipMemsetAsync(&cnt[CNT_NDENS], 0, 8, c->stream));
                c->st.rebuilds++;
            } else if (fl & FLAG_RELIST) {
                SPH_TRY(relist(c));
                c->st.relists++;
            }
            st = density_loop(c, done, hc[CNT_UNCONV]);
        }
    }
    SPH_CHECK_HIP(hipEventRecord(c->ev[1], c->stream));
    return st;
}

static sph_status launch_ghost(sph_ctx* c, const double* u, const double* vx, const double* vy, const double* vz,
                               const int* gate)
{
    const double* hdt = (const double*)c->dparam.p + 2;
    const int form = c->prm.lists == SPH_LISTS_PARTICLE          ? GHOST_PLIST
                     : c->prm.force_mode == SPH_FORCE_GATHER ? GHOST_GATHER
                                                             : GHOST_PAIRS;
    if (c->prm.precision == SPH_FP64)
        k_ghost<double><<<blocks_for(c->n, 256), 256, 0, c->stream>>>(
            c->n, c->P.rho, c->P.drho_dH, c->P.H, u, vx, vy, vz, c->prm.gamma, c->P.omega, c->P.P, (double4*)c->fv4.p,
            (double*)c->hf.p, gate, c->P.ax, c->P.ay, c->P.az, c->P.dudt, hdt, form);
    else
        k_ghost<float><<<blocks_for(c->n, 256), 256, 0, c->stream>>>(
            c->n, c->P.rho, c->P.drho_dH, c->P.H, u, vx, vy, vz, c->prm.gamma, c->P.omega, c->P.P, (float4*)c->fv4.p,
            (float*)c->hf.p, gate, c->P.ax, c->P.ay, c->P.az, c->P.dudt, hdt, form);
    SPH_CHECK_LAUNCH();
    return SPH_OK;
}

// Half step of the velocity and energy prediction the ghost applies (a step
// in progress) or 0, uploaded to the device slot the ghost reads.
static sph_status set_prediction(sph_ctx* c)
{
    const double hdt = c->predicted ? c->hdt_h : 0.0;
    if (hdt == c->hdt_up) return SPH_OK;  // (0 since sph_create)
    c->hdt_up = hdt;
    const hipError_t e = hipMemcpyAsync((double*)c->dparam.p + 2, &c->hdt_up, sizeof(double), hipMemcpyHostToDevice,
                                        c->stream);
    if (e != hipSuccess) c->hdt_up = NAN;
    SPH_CHECK_HIP(e);
    return SPH_OK;
}

sph_status ghost_all(sph_ctx* c)
{
    if (!c->dens_done || !c->sorted) return SPH_ERR_STATE;
    const double *u = c->P.u, *vx = c->P.vx, *vy = c->P.vy, *vz = c->P.vz;
    SPH_TRY(set_prediction(c));
    SPH_CHECK_HIP(hipEventRecord(c->ev[2], c->stream));
    SPH_TRY(launch_ghost(c, u, vx, vy, vz, nullptr));
    SPH_CHECK_HIP(hipEventRecord(c->ev[3], c->stream));
    c->ghost_done = true;
    return SPH_OK;
}

static void force_args(sph_ctx* c, const int* gate, bool graph, ForceArgs& a, int& nb)
{
    memset(&a, 0, sizeof(a));
    a.n_leaves = c->n_leaves;
    a.n = c->n;
    a.l_begin = (const int*)c->l_begin.p;
    a.l_count = (const int*)c->l_count.p;
    a.l_origin = (const double*)c->l_origin.p;
    a.l_hlist = (const double*)c->l_hlist.p;
    a.l_dom = (const int*)c->l_dom.p;
    a.l_off = (const int*)c->l_off.p;
    a.list = (const ListEntry*)c->list.p;
    a.l_sorted = (const int*)c->l_sorted.p;
    a.pos4 = c->pos4.p;
    a.fv4 = c->fv4.p;
    a.hf = c->hf.p;
    a.skey = (const float*)c->skey.p;
    a.sidx = (const uint16_t*)c->sidx.p;
    a.di = (const DomainInfo*)c->dom_d.p;
    a.ax = c->P.ax;
    a.ay = c->P.ay;
    a.az = c->P.az;
    a.dudt = c->P.dudt;
    a.nngb = c->P.nngb;
    a.counters = (unsigned long long*)c->counters.p;
    a.persistent = c->prm.exec_mode == SPH_EXEC_PERSISTENT;
    a.gate = gate;
    a.margin = (const double*)c->dparam.p;
    a.nl_dev = graph ? (const int*)c->flags.p + FI_NLEAVES : nullptr;
    a.wide = (const int*)c->wide.p;
    a.n_wide_dev = (const int*)c->flags.p + FI_NWIDE;
    a.n_wide = graph ? 0 : c->n_wide;
    a.wide_min = (const int*)c->flags.p + FI_WIDEMIN;
    if (graph) a.n_leaves = 0;  // read on the device
    const int nl = graph ? leaf_capacity(c) : c->n_leaves;
    // the gather form runs one wave per workgroup
    const int per = c->prm.force_mode == SPH_FORCE_GATHER ? 1 : WAVES_PER_WG;
    nb = blocks_for(nl, per);
    if (a.persistent) nb = std::min(resident_wgs(c) * (WAVES_PER_WG / per), nb);
}

static sph_status launch_force(sph_ctx* c, const int* gate, bool graph = false)
{
    if (c->prm.lists == SPH_LISTS_PARTICLE) return launch_force_plist(c, gate);
    ForceArgs a;
    int nb = 0;
    force_args(c, gate, graph, a, nb);
    if (nb > 0 && c->prm.force_mode == SPH_FORCE_GATHER) {
        launch_force_gather(c, graph, nb, a);
        SPH_CHECK_LAUNCH();
    } else if (nb > 0) {
        const bool srt = c->prm.prune == SPH_PRUNE_SORTED;
        if (c->prm.precision == SPH_FP64) {
            if (srt) k_force<double, false, PRUNE_SORTED><<<nb, 256, 0, c->stream>>>(a);
            else k_force<double, false, PRUNE_BOX><<<nb, 256, 0, c->stream>>>(a);
        } else if (c->prm.precision == SPH_FP32C) {
            if (srt) k_force<float, true, PRUNE_SORTED><<<nb, 256, 0, c->stream>>>(a);
            else k_force<float, true, PRUNE_BOX><<<nb, 256, 0, c->stream>>>(a);
        } else {
            if (srt) k_force<float, false, PRUNE_SORTED><<<nb, 256, 0, c->stream>>>(a);
            else k_force<float, false, PRUNE_BOX><<<nb, 256, 0, c->stream>>>(a);
        }
        SPH_CHECK_LAUNCH();
    }
    return SPH_OK;
}

// Running totals of the interaction counters (device, no host round trip):
// the force stage's N_force (ordered, as counted) and N_dens are added to
// CNT_NFORCE_SUM / CNT_NDENS_SUM after every force launch, which leaves its
// counts in the partial lines.
__global__ __launch_bounds__(PART_N) void k_count_totals(unsigned long long* cnt, const int* gate)
{
    if (gate && *gate != 1) return;
    if (threadIdx.x == 0) cnt[CNT_NFORCE] = cnt[CNT_NDENS_F] = 0ull;
    if (threadIdx.x < XQ_N) cnt[XQ_FORCE + threadIdx.x * XQ_STRIDE] = 0ull;
    __syncthreads();
    fold_counts(cnt);
    if (threadIdx.x == 0) {
        cnt[CNT_NFORCE_SUM] += cnt[CNT_NFORCE];
        cnt[CNT_NDENS_SUM] += cnt[CNT_NDENS_F];
        cnt[CNT_FORCE_CALLS] += 1ull;
    }
}

// Force stage, asynchronous: the counts and the kernel's duration are read by
// sph_get_stats (force_pending).
sph_status force_all(sph_ctx* c)
{
    if (!c->ghost_done || !c->sorted) return SPH_ERR_STATE;
    const size_t nb8 = (size_t)c->n * 8;
    unsigned long long* cnt = (unsigned long long*)c->counters.p;
    SPH_CHECK_HIP(hipEventRecord(c->ev[4], c->stream));
    // (the gather forms write every output; the counts and the task queues are
    // set and cleared by the kernel after the force)
    if (c->prm.force_mode == SPH_FORCE_PAIRS) {
        SPH_CHECK_HIP(hipMemsetAsync(c->P.ax, 0, nb8, c->stream));
        SPH_CHECK_HIP(hipMemsetAsync(c->P.ay, 0, nb8, c->stream));
        SPH_CHECK_HIP(hipMemsetAsync(c->P.az, 0, nb8, c->stream));
        SPH_CHECK_HIP(hipMemsetAsync(c->P.dudt, 0, nb8, c->stream));
        if (c->P.nngb) SPH_CHECK_HIP(hipMemsetAsync(c->P.nngb, 0, (size_t)c->n * 4, c->stream));
    }
    SPH_CHECK_HIP(hipEventRecord(c->kev[2], c->stream));
    SPH_TRY(launch_force(c, nullptr));
    SPH_CHECK_HIP(hipEventRecord(c->kev[3], c->stream));
    k_count_totals<<<1, PART_N, 0, c->stream>>>(cnt, nullptr);
    SPH_CHECK_LAUNCH();
    SPH_CHECK_HIP(hipEventRecord(c->ev[5], c->stream));
    c->force_pending = true;
    c->force_done = true;
    return SPH_OK;
}

// ---------------------------------------------------------------------------
// Graph mode: density sweeps, ghost and force captured in one hipGraph.  The
// sweep count is data dependent, so the graph holds a fixed number of sweeps
// gated by a device flag: 0 = sweeping, 1 = converged (the remaining sweeps
// exit at once, ghost and force run), 2 = the host must take over (lists or
// grid need rebuilding, or H hit the box limit; ghost and force are skipped).
// Counters and outputs are cleared by kernels, not memset nodes.  Grids cover
// the leaf capacity and the kernels read the leaf count from the device, so
// one graph serves every rebuild that keeps the buffers in place; it is
// captured again when any kernel argument changes.
// ---------------------------------------------------------------------------
#define SPH_GRAPH_SWEEPS 4

__global__ void k_graph_begin(unsigned long long* cnt, int* flags, int* gate)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        // the force stage's counters are left to the force stage (they may
        // still be unread by the host)
        cnt[CNT_UNCONV] = 0ull;
        cnt[CNT_NDENS] = 0ull;
        cnt[CNT_DEVAL] = 0ull;
        cnt[CNT_GSWEEPS] = 1ull;  // the first sweep follows
        for (int k = CNT_UHIST; k < CNT_N; k++) cnt[k] = 0ull;
        flags[FI_FLAGS] = 0;
        flags[FI_EXTENT] = 0;
        *gate = 0;
    }
}

// same decision order as the host loop: box limit, converged, rebuild/relist
// more: another sweep is enqueued, and begins here unless the gate is turned
__global__ __launch_bounds__(PART_N) void k_sweep_end(unsigned long long* cnt, int* flags, int* gate, int more)
{
    if (*gate != 0) return;
    fold_counts(cnt);
    if (threadIdx.x == 0) {
        const int f = flags[FI_FLAGS];
        const unsigned long long k = cnt[CNT_GSWEEPS];
        if (k >= 1 && k <= CNT_N - CNT_UHIST) cnt[CNT_UHIST + k - 1] = cnt[CNT_UNCONV];
        if (f & FLAG_BOX_SMALL) *gate = 2;
        else if (cnt[CNT_UNCONV] == 0ull) *gate = 1;
        else if (f & (FLAG_RELIST | FLAG_REBUILD)) *gate = 2;
        else if (more) {
            cnt[CNT_UNCONV] = 0ull;
            flags[FI_FLAGS] = 0;
            cnt[CNT_GSWEEPS] = k + 1;
        }
    }
}

__global__ __launch_bounds__(256) void k_force_zero(int64_t n, double* ax, double* ay, double* az, double* dudt,
                                                    int32_t* nngb, const int* gate)
{
    if (*gate != 1) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        ax[i] = 0.0;
        ay[i] = 0.0;
        az[i] = 0.0;
        dudt[i] = 0.0;
        if (nngb) nngb[i] = 0;
    }
}

template <typename X>
static void key_put(std::vector<uint8_t>& k, const X& x)
{
    const uint8_t* p = (const uint8_t*)&x;
    k.insert(k.end(), p, p + sizeof(X));
}

// Every argument and grid size the graph's launches would take now.
static std::vector<uint8_t> graph_key(sph_ctx* c, const double* u, const double* vx, const double* vy,
                                      const double* vz, int sweeps)
{
    const int* gate = (const int*)c->flags.p + FI_GATE;
    std::vector<uint8_t> k;
    DensArgs da;
    ForceArgs fa;
    int nbd = 0, nbf = 0;
    dens_args(c, gate, true, da, nbd);
    force_args(c, gate, true, fa, nbf);
    key_put(k, da);
    key_put(k, fa);
    key_put(k, nbd);
    key_put(k, nbf);
    key_put(k, sweeps);
    key_put(k, c->n);
    key_put(k, leaf_capacity(c));
    const void* ptrs[] = {u, vx, vy, vz, c->hlo.p, c->hhi.p, c->conv.p, c->l_active.p, c->P.omega, c->P.P, c->fv4.p,
                          c->hf.p, c->P.rho, c->P.drho_dH, c->P.H, c->stream};
    key_put(k, ptrs);
    key_put(k, c->prm.precision);
    key_put(k, c->prm.prune);
    key_put(k, c->prm.exec_mode);
    key_put(k, (int)(c->max_leaf > 64));  // whether the big-leaf density pass is launched
    key_put(k, (int)(c->n_leaves <= SPH_WIDE_ALL) + (int)(c->n_leaves <= SPH_WIDE_FEW));
    const void* pptrs[] = {c->pq.p, c->pR.p, c->plen.p, c->plist.p, c->prem.p, c->ch_p0.p, c->ch_n.p,
                           c->ch_uo.p, c->ch_ro.p, c->ch_U.p, c->P.domain, c->P.nngb};
    key_put(k, pptrs);
    key_put(k, c->n_chunks);
    key_put(k, c->prm.lists);
    key_put(k, c->prm.tile);
    key_put(k, c->prm.waves_density);
    return k;
}

static sph_status capture_dgf(sph_ctx* c, const double* u, const double* vx, const double* vy, const double* vz,
                              int sweeps)
{
    if (c->graph_exec) {
        (void)hipGraphExecDestroy((hipGraphExec_t)c->graph_exec);
        c->graph_exec = nullptr;
    }
    c->graph_key.clear();
    // the caller's stream may be the legacy default stream, which cannot be
    // captured: record on a private stream, launch on the caller's
    if (!c->cap_stream) SPH_CHECK_HIP(hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    const hipStream_t user = c->stream;
    c->stream = c->cap_stream;
    int* gate = (int*)c->flags.p + FI_GATE;
    unsigned long long* cnt = (unsigned long long*)c->counters.p;
    int* flags = (int*)c->flags.p;
    const int* nl_dev = (const int*)c->flags.p + FI_NLEAVES;
    const int nlc = leaf_capacity(c);
    if (hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal) != hipSuccess) {
        c->stream = user;
        return SPH_ERR_HIP;
    }
    sph_status st = SPH_OK;
    k_density_reset<<<blocks_for(std::max<int64_t>(c->n, nlc), 256), 256, 0, c->stream>>>(
        c->n, nlc, (double*)c->hlo.p, (double*)c->hhi.p, (uint8_t*)c->conv.p, (int*)c->l_active.p, nl_dev);
    k_graph_begin<<<1, 64, 0, c->stream>>>(cnt, flags, gate);
    for (int k = 0; k < sweeps && st == SPH_OK; k++) {
        st = launch_density(c, gate, true);
        k_sweep_end<<<1, PART_N, 0, c->stream>>>(cnt, flags, gate, k + 1 < sweeps);
    }
    if (st == SPH_OK) st = launch_ghost(c, u, vx, vy, vz, gate);
    if (c->prm.force_mode == SPH_FORCE_PAIRS)
        k_force_zero<<<blocks_for(c->n, 256), 256, 0, c->stream>>>(c->n, c->P.ax, c->P.ay, c->P.az, c->P.dudt,
                                                                  c->P.nngb, gate);
    if (st == SPH_OK) st = launch_force(c, gate, true);
    k_count_totals<<<1, PART_N, 0, c->stream>>>(cnt, gate);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(c->stream, &g);
    c->stream = user;
    if (st != SPH_OK || e != hipSuccess || !g) {
        if (g) (void)hipGraphDestroy(g);
        (void)hipGetLastError();
        return st != SPH_OK ? st : SPH_ERR_HIP;
    }
    hipGraphExec_t ex = nullptr;
    const hipError_t ie = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (ie != hipSuccess) return SPH_ERR_HIP;
    c->graph_exec = ex;
    c->graph_key = graph_key(c, u, vx, vy, vz, sweeps);
    c->st.graph_captures++;
    return SPH_OK;
}

// Density, ghost and force through the captured graph; the host finishes
// whatever the graph could not (more sweeps, list or grid rebuilds).
sph_status dgf_graph(sph_ctx* c)
{
    if (!c->sorted) return SPH_ERR_STATE;
    const double *u = c->P.u, *vx = c->P.vx, *vy = c->P.vy, *vz = c->P.vz;
    SPH_TRY(set_prediction(c));
    SPH_TRY(buf_ensure(c->hlo, (size_t)c->n * 8));
    SPH_TRY(buf_ensure(c->hhi, (size_t)c->n * 8));
    SPH_TRY(buf_ensure(c->conv, (size_t)c->n));
    const int sweeps = std::min(SPH_GRAPH_SWEEPS, c->prm.max_h_iter);
    if (!c->graph_exec || c->graph_key != graph_key(c, u, vx, vy, vz, sweeps))
        SPH_TRY(capture_dgf(c, u, vx, vy, vz, sweeps));
    c->st.relists = 0;
    c->st.n_density_launches = 0;
    c->st.n_dens_evals = 0;
    for (int k = 0; k < 8; k++) c->st.unconv_after[k] = -1;
    SPH_CHECK_HIP(hipEventRecord(c->ev[0], c->stream));
    SPH_CHECK_HIP(hipGraphLaunch((hipGraphExec_t)c->graph_exec, c->stream));
    SPH_CHECK_HIP(hipEventRecord(c->ev[1], c->stream));
    FlagsCounters fc;
    SPH_TRY(read_flags(c, fc));
    const int* hfl = fc.flags;
    const unsigned long long* hc = fc.cnt;
    const int gate = hfl[FI_GATE], fl = hfl[FI_FLAGS];
    const int gsweeps = (int)hc[CNT_GSWEEPS];
    // the graph's kernels are not timed one by one
    c->st.t_density_kernels_ms = -1.0;
    c->st.t_force_kernel_ms = -1.0;
    c->st.n_density_launches = gsweeps;
    c->st.n_dens_evals = (int64_t)hc[CNT_DEVAL];
    for (int k = 0; k < 8; k++)
        c->st.unconv_after[k] = k < gsweeps && k < CNT_N - CNT_UHIST
                                    ? (int)std::min<unsigned long long>(hc[CNT_UHIST + k], INT32_MAX)
                                    : -1;
    if (gate == 1) {
        c->st.sweeps = gsweeps;
        c->st.n_unconverged = 0;
        c->st.n_force = (int64_t)(c->prm.force_mode == SPH_FORCE_GATHER ? hc[CNT_NFORCE] / 2 : hc[CNT_NFORCE]);
        c->st.n_dens = (int64_t)hc[CNT_NDENS_F];
        c->dens_done = c->ghost_done = c->force_done = true;
        // the whole graph is accounted as the density stage
        for (int k = 2; k < 6; k++) SPH_CHECK_HIP(hipEventRecord(c->ev[k], c->stream));
        return SPH_OK;
    }
    // the host takes over from the state the graph left
    c->st.graph_fallbacks++;
    if (fl & FLAG_BOX_SMALL) return SPH_ERR_BOX_TOO_SMALL;
    if ((fl & FLAG_REBUILD) || ((fl & FLAG_RELIST) && c->delta > 0.0)) {
        SPH_TRY(build_all(c));
        SPH_TRY(sort_all(c));
        k_density_reset<<<blocks_for(std::max<int64_t>(c->n, c->n_leaves), 256), 256, 0, c->stream>>>(
            c->n, c->n_leaves, (double*)c->hlo.p, (double*)c->hhi.p, (uint8_t*)c->conv.p, (int*)c->l_active.p,
            nullptr);
        SPH_CHECK_LAUNCH();
        SPH_CHECK_HIP(hipMemsetAsync(&((unsigned long long*)c->counters.p)[CNT_NDENS], 0, 8, c->stream));
        c->st.rebuilds++;
    } else if (fl & FLAG_RELIST) {
        SPH_TRY(relist(c));
        c->st.relists++;
    }
    sph_status s = density_loop(c, gsweeps, hc[CNT_UNCONV]);
    c->st.t_density_kernels_ms = -1.0;
    SPH_CHECK_HIP(hipEventRecord(c->ev[1], c->stream));
    if (s != SPH_OK) return s;
    SPH_TRY(ghost_all(c));
    return force_all(c);
}

static sph_status sums_impl(sph_ctx* c, double* host_out, KickArgs kick)
{
    const int nd = c->prm.n_domains;
    // one 256-thread workgroup per chunk of a box; at most one chunk per 1024
    // particles (>= 4 per thread) and about 4096 chunks over all boxes
    const int chunks = (int)std::max<int64_t>(
        1, std::min<int64_t>(std::max(64, 4096 / std::max(nd, 1)), (c->n + 1023) / 1024));
    SPH_TRY(buf_ensure(c->dsum_part, (size_t)nd * chunks * 5 * 8 + (size_t)nd * 5 * 8));
    const int* ranges = (const int*)c->dranges.p;
    double* part = (double*)c->dsum_part.p;
    double* out = part + (size_t)nd * chunks * 5;
    dim3 g(chunks, nd);
    k_sums_partial<<<g, 256, 0, c->stream>>>(ranges, c->P.m, c->P.vx, c->P.vy, c->P.vz, c->P.u, part, chunks, kick);
    SPH_CHECK_LAUNCH();
    k_sums_final<<<nd, 256, 0, c->stream>>>(part, out, chunks);
    SPH_CHECK_LAUNCH();
    c->sums_dev = out;
    if (!host_out) {
        c->sums_pending = true;  // read by sph_get_stats
        return SPH_OK;
    }
    SPH_CHECK_HIP(hipMemcpyAsync(host_out, out, (size_t)nd * 5 * 8, hipMemcpyDeviceToHost, c->stream));
    SPH_CHECK_HIP(hipStreamSynchronize(c->stream));
    return SPH_OK;
}

sph_status domain_sums(sph_ctx* c, double* host_out)
{
    KickArgs none{};
    return sums_impl(c, host_out, none);
}

static sph_status step_impl(sph_ctx* c, double dt);

// Particle lists built inside the step (cell rebuilds and relists) size their
// skins and growth allowances for rebuild_steps steps of this length.
sph_status step_all(sph_ctx* c, double dt)
{
    c->list_dt = dt;
    const sph_status s = step_impl(c, dt);
    c->list_dt = 0.0;
    return s;
}

// Displacement bound of the kept lists, on the device: margin += 2 vmax dt.
__global__ void k_margin(double* dparam, double dt)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        double v;
        const unsigned long long b = ((const unsigned long long*)dparam)[1];
        memcpy(&v, &b, 8);
        dparam[0] += 2.0 * v * dt;
    }
}

// One step.  The host reads the device once before the density stage (the
// step's largest speed and whether the kept cells and lists are still valid:
// the cell build is host-driven) and once inside the density stage; the
// force, the closing kick and the FP64 totals are enqueued without waiting
// (the totals are read by sph_get_stats).
static sph_status step_impl(sph_ctx* c, double dt)
{
    if (!c->force_done) return SPH_ERR_STATE;
    const int nb = blocks_for(c->n, 256);
    unsigned long long* vmax_bits = (unsigned long long*)c->dparam.p + 1;
    SPH_CHECK_HIP(hipMemsetAsync(vmax_bits, 0, 8, c->stream));
    // the start of the H iteration is carried along the flow unless the
    // predictor supplies it; fused into the kick-drift unless the predictor
    // records samples (its features read the H before the drift)
    const bool drift = c->prm.h_drift && !(c->h_pred && c->mlp_ready);
    const bool fuse = drift && !c->rec_on;
    k_kick_drift<<<nb, 256, 0, c->stream>>>(c->n, c->P.x, c->P.y, c->P.z, c->P.vx, c->P.vy, c->P.vz, c->P.u, c->P.ax,
                                            c->P.ay, c->P.az, c->P.dudt, c->P.domain, (const DomainInfo*)c->dom_d.p,
                                            dt, vmax_bits, fuse ? c->P.H : nullptr, c->prm.gamma - 1.0);
    SPH_CHECK_LAUNCH();
    c->step_count++;
    SPH_TRY(mlp_pre_build(c, dt));
    if (drift && !fuse) {
        k_h_drift<<<nb, 256, 0, c->stream>>>(c->n, c->P.H, c->P.u, c->P.dudt, c->prm.gamma - 1.0, dt);
        SPH_CHECK_LAUNCH();
    }
    SPH_CHECK_HIP(hipEventRecord(c->ev[6], c->stream));
    const bool keep = c->prm.rebuild_steps > 0 && c->built;
    if (keep) {
        // keep the cells and lists while the displacement margin allows
        k_margin<<<1, 64, 0, c->stream>>>((double*)c->dparam.p, dt);
        SPH_CHECK_LAUNCH();
        if (c->prm.lists == SPH_LISTS_PARTICLE) SPH_TRY(plist_refresh(c, nullptr));
        else SPH_TRY(refresh_leaves(c, nullptr));
    }
    // (the flags follow the parameters)
    struct {
        double dp[8];
        int fl;
    } rb;
    SPH_CHECK_HIP(hipMemcpyAsync(&rb, c->dparam.p, 8 * sizeof(double) + sizeof(int), hipMemcpyDeviceToHost, c->stream));
    if (keep && c->prm.lists == SPH_LISTS_PARTICLE)
        SPH_CHECK_HIP(hipMemcpyAsync(c->stale_h, (unsigned long long*)c->counters.p + CNT_STALE_MOVED, 16,
                                     hipMemcpyDeviceToHost, c->stream));
    SPH_CHECK_HIP(hipStreamSynchronize(c->stream));
    const double* dp = rb.dp;
    const int fl = rb.fl;
    double vmax;
    {
        unsigned long long b;
        memcpy(&b, &dp[1], 8);
        memcpy(&vmax, &b, 8);
    }
    bool fresh = false;
    if (keep) {
        c->margin_h = dp[0];
        c->delta = 0.5 * dp[0];
        fresh = !(fl & FLAG_STALE);
        if (c->prm.lists == SPH_LISTS_PARTICLE) {
            c->st.stale_moved = (int64_t)c->stale_h[0];
            c->st.stale_grown = (int64_t)c->stale_h[1];
        }
    }
    if (fresh) {
        c->steps_since_build++;
    } else {
        // list skin for the coming steps: rebuild_steps times this step's
        // largest displacement
        c->skin_abs = c->prm.rebuild_steps > 0 ? c->prm.rebuild_steps * vmax * dt : 0.0;
        // the density and ghost stages below write rho, drho_dH, omega and P
        // of every particle (all start unconverged) before anything reads them
        c->dens_outputs_dead = true;
        const sph_status sb = build_all(c);
        c->dens_outputs_dead = false;
        SPH_TRY(sb);
    }
    SPH_TRY(sort_all(c));
    SPH_CHECK_HIP(hipEventRecord(c->ev[7], c->stream));
    sph_status s;
    c->hdt_h = 0.5 * dt;
    c->predicted = true;
    c->in_step = true;
    if (c->prm.use_graph) {
        s = dgf_graph(c);
    } else {
        s = density_all(c);
        if (s == SPH_OK) s = ghost_all(c);
        if (s == SPH_OK) s = force_all(c);
    }
    c->predicted = false;
    c->in_step = false;
    if (s != SPH_OK) return s;
    SPH_TRY(mlp_post_step(c));
    // closing half kick, fused with the FP64 totals of the kicked state
    KickArgs kick{c->P.ax, c->P.ay, c->P.az, c->P.dudt, 0.5 * dt};
    SPH_TRY(sums_impl(c, nullptr, kick));
    return SPH_OK;
}
