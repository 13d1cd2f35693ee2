// SPH interpolation of a particle quantity at arbitrary points (paper,
// Sec. 2, eq. (interp)): Q(r) = sum_i m_i Q_i / rho_i W(|r - r_i|, H_i), each
// particle contributing within its own support H_i.
//
// The points are first ordered by box and Morton code of their position and
// cut into blocks of up to 64 that share a box and fit in a top cell.  A wave
// walks the octree of the last build once for a block, 64 cells at a time:
// cells farther from the block's bounding box than their largest H are
// pruned, the leaves left are listed.  The leaves of the blocks of a workgroup
// are then shared out evenly between its waves, whichever block they belong
// to; their particles are tested against the points on the matrix units and
// the pairs in range summed one per lane (sph_device.h).
//
// Distances are minimum-image: every H is below half the box (the top cells
// are at least H wide and there are at least three per axis), so at most one
// image of a particle lies within its support.  Cell boxes are those of the
// build; particles have moved by at most delta since, so a cell is kept while
// its box lies closer than its largest H plus a margin of 2 delta.
#include <math.h>

#include "sph_ctx.h"
#include "sph_device.h"

#define INTERP_INV_PI_8 2.5464790894703255  // 8/pi
#define INTERP_MBITS 10                    // Morton bits per axis of the sort key

namespace {

struct InterpArgs {
    int64_t m_pts;
    const double *px, *py, *pz;
    const int32_t* pdom;
    int n_dom;
    const DomainInfo* di;
    const Node* nodes;
    const double *x, *y, *z, *m, *rho, *H, *Q;
    double margin;
    double* out;
    const uint32_t* perm;  // sorted position -> point index
};

// sqrt(x) for 0 <= x <= 4 to an ulp: the hardware's estimate of 1/sqrt and two
// coupled Newton steps, without the scaling that other arguments need.
__device__ inline double interp_sqrt(double x)
{
    x = fmax(x, 1e-290);
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    return fma(fma(-g, g, x), h, g);
}

// Kernel of q >= 0 without 8 / (pi H^3)
__device__ inline double interp_w(double q)
{
    const double t = 1.0 - q;
    const double in = fma(q * q, fma(6.0, q, -6.0), 1.0), out = 2.0 * t * t * t;
    return q <= 0.5 ? in : out;
}

// Offset d along an axis of length L = 1 / iL as that of the nearest image.
__device__ inline double min_image(double d, double L, double iL) { return fma(-L, rint(d * iL), d); }

// Validated point k wrapped into its box; false for a bad box index or a
// non-finite coordinate.
__device__ inline bool load_point(const InterpArgs& a, int64_t k, double p[3], int& d)
{
    d = a.pdom ? a.pdom[k] : 0;
    p[0] = a.px[k];
    p[1] = a.py[k];
    p[2] = a.pz[k];
    if (d < 0 || d >= a.n_dom || !isfinite(p[0]) || !isfinite(p[1]) || !isfinite(p[2])) return false;
    const DomainInfo& I = a.di[d];
    for (int c = 0; c < 3; c++) {
        p[c] -= I.L[c] * floor(p[c] / I.L[c]);
        if (p[c] >= I.L[c]) p[c] = 0.0;  // a tiny negative input rounds up to L
    }
    return true;
}

// Top cells within reach of the box [lo, hi] (per axis: first cell and
// count, as residues of the periodic grid, each visited once).  Every H is at
// most the smallest top-cell edge once the density stage is done.
__device__ inline void top_range(const DomainInfo& I, const double lo[3], const double hi[3], double margin, int t0[3],
                                 int nt[3])
{
    const double R = fmin(fmin(I.s0[0], I.s0[1]), I.s0[2]) * (1.0 + 1e-9) + margin;
    for (int c = 0; c < 3; c++) {
        const int l = (int)floor((lo[c] - R) / I.s0[c]), h = (int)floor((hi[c] + R) / I.s0[c]);
        nt[c] = min(h - l + 1, I.n_top[c]);
        t0[c] = nt[c] == I.n_top[c] ? 0 : l;
    }
}

__device__ inline int top_index(const DomainInfo& I, const int t0[3], int ix, int iy, int iz)
{
    int c[3] = {t0[0] + ix, t0[1] + iy, t0[2] + iz};
    // (a range that is not the whole axis begins above -n_top and ends below 2 n_top)
    for (int q = 0; q < 3; q++) c[q] += c[q] < 0 ? I.n_top[q] : c[q] >= I.n_top[q] ? -I.n_top[q] : 0;
    return I.top_offset + (c[0] * I.n_top[1] + c[1]) * I.n_top[2] + c[2];
}

// Sort keys: box index in the high bits, Morton code of the position
// (INTERP_MBITS per axis) below; invalid points get the largest key.
__global__ __launch_bounds__(256) void k_interp_keys(InterpArgs a, uint64_t* keys, uint32_t* vals, uint64_t invalid)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.m_pts) return;
    double p[3];
    int d;
    uint64_t key = invalid;
    if (load_point(a, k, p, d)) {
        const DomainInfo& I = a.di[d];
        uint32_t f[3];
        for (int c = 0; c < 3; c++) {
            const double u = p[c] / I.L[c] * (1 << INTERP_MBITS);
            f[c] = (uint32_t)fmin(fmax(u, 0.0), (double)((1 << INTERP_MBITS) - 1));
        }
        uint64_t mort = 0;
        for (int b = INTERP_MBITS - 1; b >= 0; b--)
            mort = (mort << 3) | (((f[0] >> b) & 1u) << 2) | (((f[1] >> b) & 1u) << 1) | ((f[2] >> b) & 1u);
        key = ((uint64_t)d << (3 * INTERP_MBITS)) | mort;
    }
    keys[k] = key;
    vals[k] = (uint32_t)k;
}

// Waves of a workgroup, leaves a wave lists at a time, cells its walk holds.
#define IW 8
#define ILEAF 192
#define ISTACK 512
#define IROW 16  // candidates per 16-lane row of a tile

// Candidates of one wave: up to 4 IROW particles that can reach the block.
struct ITile {
    double4 cand[4 * IROW];       // relative to the block's centre, scaled; w: H, then 1/H^2
    double cf[4 * IROW];          // particle index, then m Q / rho 8 / (pi H^3)
    union {
        float c1[4 * IROW];       // row constants of the range tests
        uint16_t list[PAIR_CAP];  // then the pairs
    };
};
struct ILeaf { int begin, count; };
struct IBlock {
    double p[3][64];    // points relative to the centre, scaled
    double c[3], hw[3]; // bounding box: centre, half-widths
    double sc, isc;     // power of two that makes the box's top cells of order 1, its inverse
    double L[3], iL[3]; // edges of the box, their inverses
    unsigned long long sel;  // lanes with a point of the block
    int dom, n_leaf;
};

// One workgroup per IW groups of G consecutive points of the sorted order, a
// wave per group.  Rounds: each wave takes the next block of its group (or
// goes on with one that filled its list) and lists leaves; then all waves
// share all leaves; then each wave adds up its block's sums.  Sums are made in
// the same order whatever the timing.
//
// Was bound by the few waves with a halo in their block (one wave per 64
// points, cells and leaves one after another: the fullest of 128^3 mesh points
// over 96^3 clustered particles visits 11373 particles, the mean 154) and by
// 65 FP64 instructions per particle visited with 22% of the lanes in range.
// That mesh: 2.87 ms before, 0.73 ms now (VALU active 63% of the time; the rest is
// the walk's latency, with 4 waves a SIMD in 79 KB of LDS and 128 registers).
// 4 waves a workgroup: 2% less time there, but twice the longest share; 16: 9%
// more.
__global__ __launch_bounds__(64 * IW, 4) void k_interp_blocks(InterpArgs a, int G)
{
    __shared__ ITile tile[IW];
    __shared__ IBlock blk[IW];
    __shared__ ILeaf leaf[IW][ILEAF];
    __shared__ int stack[IW][ISTACK];
    __shared__ double S0[IW][64], S1[IW][64];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    ITile& L = tile[wv];
    const int64_t s = ((int64_t)blockIdx.x * IW + wv) * G + lane;
    const bool inr = lane < G && s < a.m_pts;
    const int64_t k = inr ? (int64_t)a.perm[s] : 0;
    double p[3] = {0.0, 0.0, 0.0};
    int d = -1;
    const bool ok = inr && load_point(a, k, p, d);
    if (inr && !ok) a.out[k] = NAN;
    unsigned long long rest = __ballot(ok);  // points in no block yet
    bool open = false;                       // the block's walk is under way
    unsigned long long sel = 0ull;
    int size = 0, tcur = 0, ntop = 0, t0[3] = {0, 0, 0}, nt[3] = {0, 0, 0};
    double sum = 0.0;
    while (__syncthreads_or(open || rest != 0ull)) {
        IBlock& B = blk[wv];
        if (!open) {
            // the largest aligned run of 64, 32, .. 1 lanes from the next point
            // on whose points share a box and fit in a top cell
            sel = 0ull;
            size = tcur = ntop = 0;
            if (rest) {
                const int l0 = __builtin_ctzll(rest);
                const int d0 = __builtin_amdgcn_readlane(d, l0);
                const DomainInfo& I = a.di[d0];
                const double s0min = fmin(fmin(I.s0[0], I.s0[1]), I.s0[2]);
                double lo[3], hi[3];
                for (int g = 64; g > 0; g >>= 1) {
                    sel = rest & ((g == 64 ? ~0ull : (1ull << g) - 1ull) << (l0 & ~(g - 1)));
                    const bool in = (sel >> lane) & 1ull;
                    double ext = 0.0;
                    for (int q = 0; q < 3; q++) {
                        lo[q] = wave_min_t(in ? p[q] : 1e300);
                        hi[q] = wave_max_t(in ? p[q] : -1e300);
                        ext = fmax(ext, hi[q] - lo[q]);
                    }
                    if (__ballot(in && d != d0) == 0ull && ext <= s0min) break;
                }
                top_range(I, lo, hi, a.margin, t0, nt);
                ntop = nt[0] * nt[1] * nt[2];
                const double sc = pow2_scale(s0min);
                const bool in = (sel >> lane) & 1ull;
                for (int q = 0; q < 3; q++) {
                    const double c = 0.5 * (lo[q] + hi[q]);
                    B.p[q][lane] = in ? (p[q] - c) * sc : 0.0;
                    if (lane == 0) {
                        B.c[q] = c;
                        B.hw[q] = 0.5 * (hi[q] - lo[q]);
                        B.L[q] = I.L[q];
                        B.iL[q] = 1.0 / I.L[q];
                    }
                }
                if (lane == 0) {
                    B.sc = sc;
                    B.isc = 1.0 / sc;
                    B.sel = sel;
                    B.dom = d0;
                }
                rest &= ~sel;
                open = true;
                wave_sync();
            }
        }
        // list leaves until the walk ends or the list is full
        int nl = 0;
        if (open) {
            const DomainInfo& I = a.di[B.dom];
            const double bc[3] = {B.c[0], B.c[1], B.c[2]}, bw[3] = {B.hw[0], B.hw[1], B.hw[2]};
            while (nl <= ILEAF - 64) {
                int kk = -1;
                if (size > 0) {
                    // at most 7 cells more for each taken: even one a time from
                    // here down all levels stays within the stack
                    const int t = min(min(64, size), max(1, (ISTACK - 8 * 24 - size) / 7));
                    if (lane < t) kk = stack[wv][size - t + lane];
                    size -= t;
                } else if (tcur < ntop) {
                    const int t = min(min(64, ntop - tcur), (ISTACK - 8 * 24) / 8);
                    if (lane < t) {
                        // (exact: the quotients are far below 2^20)
                        const int id = tcur + lane;
                        const int r = (int)((id + 0.5f) * __builtin_amdgcn_rcpf((float)nt[2]));
                        const int ix = (int)((r + 0.5f) * __builtin_amdgcn_rcpf((float)nt[1]));
                        kk = top_index(I, t0, ix, r - ix * nt[1], id - r * nt[2]);
                    }
                    tcur += t;
                } else {
                    open = false;
                    break;
                }
                wave_sync();
                int fc = -1, nc = 0;
                ILeaf lf = {0, 0};
                bool keep = false;
                if (kk >= 0) {
                    const Node& nd = a.nodes[kk];
                    fc = nd.first_child;
                    nc = nd.n_child;
                    lf.begin = nd.begin;
                    lf.count = nd.count;
                    // squared gap between the cell's box and the block's
                    double d2 = 0.0;
                    for (int q = 0; q < 3; q++) {
                        const double nlo = nd.lo[q], nhi = nd.hi[q];
                        const double g = fmax(fabs(min_image(bc[q] - 0.5 * (nlo + nhi), B.L[q], B.iL[q])) -
                                                  0.5 * (nhi - nlo) - bw[q], 0.0);
                        d2 += g * g;
                    }
                    const double reach = nd.hmax + a.margin;
                    keep = lf.count > 0 && d2 < reach * reach;
                }
                const bool is_leaf = keep && fc < 0;
                const unsigned long long lm = __ballot(is_leaf);
                if (is_leaf) leaf[wv][nl + lane_rank(lm)] = lf;
                nl += __popcll(lm);
                if (!keep || is_leaf) nc = 0;
                for (int q = 0; __ballot(q < nc) != 0ull; q++) {
                    const unsigned long long cm = __ballot(q < nc);
                    if (q < nc) stack[wv][size + lane_rank(cm)] = fc + q;
                    size += __popcll(cm);
                }
                wave_sync();
            }
        }
        if (lane == 0) B.n_leaf = nl;
        S0[wv][lane] = S1[wv][lane] = 0.0;
        __syncthreads();
        // share of wave w: leaves [N w / IW, N (w + 1) / IW) of all blocks'
        int N = 0, own = 0;  // leaves of all blocks, of those before this wave's
#pragma unroll
        for (int w = 0; w < IW; w++) {
            if (w == wv) own = N;
            N += __builtin_amdgcn_readfirstlane(blk[w].n_leaf);
        }
        const int end = N * (wv + 1) / IW;
        for (int b = 0, pb = 0, pe = 0, at = N * wv / IW; at < end; b++, pb = pe) {
            pe = pb + __builtin_amdgcn_readfirstlane(blk[b].n_leaf);
            if (at >= pe) continue;
            const int e = min(end, pe);
            const IBlock& Q = blk[b];
            // sums of the wave that begins a block, and of those that go on
            double* acc = at == pb ? S0[b] : S1[wv];
            const double sc = Q.sc, isc = Q.isc;
            bf16x4 bt[4];
            {
                const float x = (float)Q.p[0][lane], y = (float)Q.p[1][lane], z = (float)Q.p[2][lane];
                const bool on = (Q.sel >> lane) & 1ull;
                test_operand(x, y, z, on ? (x * x + y * y + z * z) * (1.0f - PAIR_EPS) - 1e-30f : 1e30f, 0.f,
                             (float4*)L.cand, lane, bt);
            }
            const int nb = 4 - (__builtin_clzll(Q.sel) >> 4);
            auto eval = [&](const uint16_t* list, int n) __attribute__((always_inline)) {
                const int K = (n + 63) >> 6;
                int cur = -1;
                double v = 0.0, x = 0.0, y = 0.0, z = 0.0;
                for (int i = lane * K; i < min(lane * K + K, n); i++) {
                    const int code = list[i], ii = code >> 7;
                    if (ii != cur) {
                        if (cur >= 0) lds_add(&acc[cur], v);
                        cur = ii;
                        x = Q.p[0][ii];
                        y = Q.p[1][ii];
                        z = Q.p[2][ii];
                        v = 0.0;
                    }
                    const double4 c = L.cand[code & 127];
                    const double dx = c.x - x, dy = c.y - y, dz = c.z - z;
                    const double q2 = fma(dx, dx, fma(dy, dy, dz * dz)) * c.w;
                    const double w = L.cf[code & 127] * interp_w(interp_sqrt(q2));
                    v += q2 < 1.0 ? w : 0.0;
                }
                if (cur >= 0) lds_add(&acc[cur], v);
            };
            auto run_tile = [&](int len) __attribute__((always_inline)) {
                for (int j = len + lane; j < 4 * IROW; j += 64) {
                    L.cand[j] = make_double4(0.0, 0.0, 0.0, 1.0);
                    L.c1[test_slot<IROW>(j)] = 1e30f;
                }
                wave_sync();
                // the weights, while the tests run
                const bool has = lane < len;
                const int j = has ? (int)L.cf[lane] : 0;
                const double hs = L.cand[lane].w, h = hs * isc;
                const double mj = a.m[j], qj = a.Q[j], rj = a.rho[j];
                uint32_t M[4] = {0u, 0u, 0u, 0u};
                tile_masks<false, IROW>(L.c1, nullptr, [&](int t) {
                    const float v = (float)((const double*)&L.cand[t])[lane >> 4];
                    return lane < 48 ? v : 1.0f;
                }, bt, nb, lane, M);
                // (a row of IROW bits, the first candidate's at bit IROW - 1)
                for_pairs<IROW>(M, L.list, lane, [&]() {
                    wave_sync();
                    L.cf[lane] = mj * qj / rj * INTERP_INV_PI_8 / (h * h * h);
                    L.cand[lane].w = 1.0 / (hs * hs);
                }, eval);
                wave_sync();
            };
            int ncand = 0, li = at - pb, p0 = 0;
            const int le = e - pb;
            ILeaf lf = {0, 0};
            double r[3] = {0.0, 0.0, 0.0}, hj = 0.0;
            auto load = [&]() __attribute__((always_inline)) {
                lf = leaf[b][li];
                const int j = lf.begin + min(p0 + lane, lf.count - 1);
                r[0] = a.x[j];
                r[1] = a.y[j];
                r[2] = a.z[j];
                hj = a.H[j];
            };
            load();
            while (true) {
                bool in = false;
                int j = 0;
                double x[3] = {0.0, 0.0, 0.0}, h = 0.0;
                const bool more = li < le;
                if (more) {
                    // the particle's image nearest the block, its gap to the block
                    double g2 = 0.0;
                    for (int q = 0; q < 3; q++) {
                        x[q] = min_image(r[q] - Q.c[q], Q.L[q], Q.iL[q]);
                        const double g = fmax(fabs(x[q]) - Q.hw[q], 0.0);
                        g2 += g * g;
                    }
                    h = hj;
                    j = lf.begin + p0 + lane;
                    in = p0 + lane < lf.count && g2 < h * h;
                    p0 += 64;
                    if (p0 >= lf.count) {
                        li++;
                        p0 = 0;
                    }
                    if (li < le) load();
                }
                const unsigned long long mk = __ballot(in);
                const int nk = __popcll(mk);
                if (ncand + nk > 4 * IROW || !more) {
                    if (ncand > 0) run_tile(ncand);
                    if (!more) break;
                    ncand = 0;
                }
                if (in) {
                    const int slot = ncand + lane_rank(mk);
                    const double4 o = make_double4(x[0] * sc, x[1] * sc, x[2] * sc, h * sc);
                    L.cand[slot] = o;
                    L.cf[slot] = (double)j;
                    const float fx = (float)o.x, fy = (float)o.y, fz = (float)o.z, fh = (float)o.w;
                    L.c1[test_slot<IROW>(slot)] = (fx * fx + fy * fy + fz * fz) * (1.0f - PAIR_EPS) -
                                                  fh * fh * (1.0f + PAIR_EPS);
                }
                ncand += nk;
            }
            at = e;
        }
        __syncthreads();
        // the block's sum: its first wave's, then the later ones' in turn
        double v = S0[wv][lane];
#pragma unroll
        for (int w = 1; w < IW; w++) {
            const int f = N * w / IW;
            if (f < N * (w + 1) / IW && f > own && f < own + nl) v += S1[w][lane];
        }
        if ((sel >> lane) & 1ull) sum += v;
    }
    if (ok) a.out[k] = sum;
}

}  // namespace

extern "C" sph_status sph_interpolate(sph_ctx* c, const double* Q, const double* px, const double* py,
                                      const double* pz, const int32_t* pdom, int64_t m_pts, double* out)
{
    if (!c || m_pts < 0 || ((!Q || !px || !py || !pz || !out) && m_pts > 0)) return SPH_ERR_INVALID;
    if (c->prm.n_domains > 1 && !pdom && m_pts > 0) return SPH_ERR_INVALID;
    PoolScope ps(&c->pool);
    if (!c->dens_done || !c->built) return SPH_ERR_STATE;
    if (m_pts == 0) return SPH_OK;
    if (m_pts > INT32_MAX) return SPH_ERR_INVALID;
    // largest H per cell from the current H (the lists keep their radii)
    SPH_TRY(node_hmax_all(c, false));
    InterpArgs a;
    a.m_pts = m_pts;
    a.px = px;
    a.py = py;
    a.pz = pz;
    a.pdom = pdom;
    a.n_dom = c->prm.n_domains;
    a.di = (const DomainInfo*)c->dom_d.p;
    a.nodes = (const Node*)c->nodes.p;
    a.x = c->P.x;
    a.y = c->P.y;
    a.z = c->P.z;
    a.m = c->P.m;
    a.rho = c->P.rho;
    a.H = c->P.H;
    a.Q = Q;
    a.margin = 2.0 * c->delta;
    a.out = out;
    a.perm = nullptr;
    // sort the points by box and Morton code
    int dom_bits = 1;
    while ((1ll << dom_bits) <= (long long)c->prm.n_domains) dom_bits++;
    const int bits = dom_bits + 3 * INTERP_MBITS;
    for (int q = 0; q < 2; q++) {
        SPH_TRY(buf_ensure(c->ikeys[q], (size_t)m_pts * 8));
        SPH_TRY(buf_ensure(c->ivals[q], (size_t)m_pts * 4));
    }
    const unsigned nb = (unsigned)((m_pts + 255) / 256);
    k_interp_keys<<<nb, 256, 0, c->stream>>>(a, (uint64_t*)c->ikeys[0].p, (uint32_t*)c->ivals[0].p,
                                             (uint64_t)c->prm.n_domains << (3 * INTERP_MBITS));
    SPH_CHECK_LAUNCH();
    int res = 0;
    SPH_TRY(radix_sort(c, (int)m_pts, bits, c->ikeys, c->ivals, &res));
    a.perm = (const uint32_t*)c->ivals[res].p;
    // points per wave: 64, fewer while that leaves less than 4096 waves (half
    // of what the chip holds): few points wait on the longest walk
    int G = 64;
    while (G > 1 && m_pts < (int64_t)G * 4096) G >>= 1;
    k_interp_blocks<<<(unsigned)((m_pts + IW * G - 1) / (IW * G)), 64 * IW, 0, c->stream>>>(a, G);
    SPH_CHECK_LAUNCH();
    return SPH_OK;
}
