// Device-side helpers shared by the interaction kernels of libsph_hip
// (leaf-tile kernels and per-particle list kernels): the cubic-spline kernel
// of Sec. 2, compensated sums, wave reductions, the persistent task queues,
// pair-candidate batches of the neighbour-cell lists, and the density
// sweep's FP64 Newton step on rho H^3 = C.  Not part of the C-ABI.
#pragma once

#include <math.h>

#include "sph_ctx.h"

#define WAVES_PER_WG 4
#define INV_PI_8 2.5464790894703255  // 8/pi: cubic-spline normalisation in 3D

// ---------------------------------------------------------------------------
// Kernel shape, Sec. 2 (cubic spline with compact support H):
//   w(q)  = 1 - 6q^2 + 6q^3 (q <= 1/2),  2(1-q)^3 (1/2 < q < 1)
//   w'(q) = q(18q - 12)     (q <= 1/2), -6(1-q)^2 (1/2 < q < 1)
// ---------------------------------------------------------------------------
template <typename T>
__device__ inline void spline_w_dw(T q, T& w, T& dw)
{
    // both pieces and a select: lanes of a wave fall on both sides of q = 1/2
    const T t = T(1) - q;
    const bool in = q <= T(0.5);
    const T wi = T(1) + q * q * (T(6) * q - T(6)), dwi = q * (T(18) * q - T(12));
    const T wo = T(2) * t * t * t, dwo = T(-6) * t * t;
    w = in ? wi : wo;
    dw = in ? dwi : dwo;
}

// q^2 w''(q) + 2 q w'(q), the q-part of the second H-derivative of H^3 W
template <typename T>
__device__ inline T spline_d2(T q, T dw)
{
    const T di = T(36) * q - T(12), dout = T(12) * (T(1) - q);  // both pieces, then a select
    const T d2 = (q <= T(0.5)) ? di : dout;
    return q * (q * d2 + T(2) * dw);
}

// -w'(q) / 6, zero from q = 1 on (1 - q clamped to [0, 1])
__device__ inline float clamp01(float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, 1.0f); }
__device__ inline double clamp01(double x) { return fmin(fmax(x, 0.0), 1.0); }
template <typename T>
__device__ inline T spline_dw6(T q)
{
    const T t = clamp01(T(1) - q);
    const T vi = q * (T(2) - T(3) * q), vo = t * t;  // both pieces, then a select
    return (q <= T(0.5)) ? vi : vo;
}

template <typename T>
__device__ inline T spline_dw(T q)
{
    const T t = T(1) - q;
    const T vi = q * (T(18) * q - T(12)), vo = T(-6) * t * t;  // both pieces, then a select
    const T v = (q <= T(0.5)) ? vi : vo;
    return (q < T(1)) ? v : T(0);
}

// Square root, reciprocal square root and reciprocal: in FP32 the hardware
// instructions (1 ulp) instead of the longer correctly rounded sequences;
// FP64 keeps the IEEE operations.  Arguments are positive normal numbers.
__device__ inline float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ inline double fast_sqrt(double x) { return sqrt(x); }
__device__ inline float fast_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ inline double fast_rsqrt(double x) { return 1.0 / sqrt(x); }
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double fast_rcp(double x) { return 1.0 / x; }

// Compensated (Kahan) accumulation; COMP = false gives the plain sum.
template <typename T, bool COMP>
struct Acc {
    T s = 0, c = 0;
    __device__ inline void add(T v)
    {
        if (COMP) {
            const T y = v - c;
            const T t = s + y;
            c = (t - s) - y;
            s = t;
        } else {
            s += v;
        }
    }
    __device__ inline double total() const { return COMP ? (double)s - (double)c : (double)s; }
};

// Reductions over the wave, the result in every lane: rotations within the rows
// of 16 lanes (DPP), then swaps of rows and halves.  (Six ds_bpermute steps, at
// the latency of LDS each, took 2 us of the 37 us of a leaf in a small box.)
template <int CTRL>
__device__ inline float lane_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ inline unsigned long long lane_move(unsigned long long v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, true);
    return ((unsigned long long)hi << 32) | lo;
}
template <int CTRL>
__device__ inline double lane_move(double v)
{
    return __builtin_bit_cast(double, lane_move<CTRL>(__builtin_bit_cast(unsigned long long, v)));
}
// v of the lane and of its partner in the next row (HALF: the other half), in
// the same order in both lanes
template <bool HALF>
__device__ inline void lane_pair(uint32_t v, uint32_t& x, uint32_t& y)
{
    if (HALF) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        x = r[0], y = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        x = r[0], y = r[1];
    }
}
template <bool HALF>
__device__ inline void lane_pair(float v, float& x, float& y)
{
    uint32_t a, b;
    lane_pair<HALF>(__builtin_bit_cast(uint32_t, v), a, b);
    x = __builtin_bit_cast(float, a), y = __builtin_bit_cast(float, b);
}
template <bool HALF>
__device__ inline void lane_pair(unsigned long long v, unsigned long long& x, unsigned long long& y)
{
    uint32_t a, b, c, d;
    lane_pair<HALF>((uint32_t)v, a, b);
    lane_pair<HALF>((uint32_t)(v >> 32), c, d);
    x = ((unsigned long long)c << 32) | a, y = ((unsigned long long)d << 32) | b;
}
template <bool HALF>
__device__ inline void lane_pair(double v, double& x, double& y)
{
    unsigned long long a, b;
    lane_pair<HALF>(__builtin_bit_cast(unsigned long long, v), a, b);
    x = __builtin_bit_cast(double, a), y = __builtin_bit_cast(double, b);
}
template <typename V, typename Op>
__device__ inline V wave_reduce(V v, Op op)
{
    v = op(v, lane_move<0x121>(v));
    v = op(v, lane_move<0x122>(v));
    v = op(v, lane_move<0x124>(v));
    v = op(v, lane_move<0x128>(v));
    V x, y;
    lane_pair<false>(v, x, y);
    v = op(x, y);
    lane_pair<true>(v, x, y);
    return op(x, y);
}
template <typename T> __device__ inline T wave_min_t(T v)
{
    return wave_reduce(v, [](T a, T b) { return fmin(a, b); });
}
template <typename T> __device__ inline T wave_max_t(T v)
{
    return wave_reduce(v, [](T a, T b) { return fmax(a, b); });
}
__device__ inline double wave_max(double v) { return wave_max_t<double>(v); }
__device__ inline float wave_minf(float v) { return wave_min_t<float>(v); }
__device__ inline float wave_maxf(float v) { return wave_max_t<float>(v); }
__device__ inline unsigned long long wave_sum(unsigned long long v)
{
    return wave_reduce(v, [](unsigned long long a, unsigned long long b) { return a + b; });
}
// Wave-uniform pop from a device task counter: one atomic by lane 0, its
// result read from the first lane into a scalar register by all lanes, so
// loops that exit on it have a uniform exit condition.  (With every lane in
// the atomic, the compiler sums the lanes' operands in a loop over the wave:
// 64 rounds a pop.)
__device__ inline int wave_pop(unsigned long long* counter, int lane)
{
    int v = 0;
    if (lane == 0) v = (int)atomicAdd(counter, 1ull);
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Task queue of the persistent force kernels.  Task positions [0, nL) are cut into
// XQ_N = 8 contiguous ranges, one per XCD (workgroup b runs on XCD b mod 8),
// each drained through its own counter q[x * XQ_STRIDE].  A wave takes tasks
// from the range of its own XCD first, so the waves running side by side on
// one XCD work on neighbouring leaves and share its L2; once that range is
// empty it helps the other ranges in ring order, which balances ranges of
// unequal cost.  `k` (start at 0) is the number of ranges the wave has found
// empty; returns -1 when all are.  Every successful pop takes a distinct
// position, so a wave's loop over this ends after at most nL + 1 calls.
static_assert(XQ_N == 8, "one task range per XCD");
__device__ inline int xq_pop(unsigned long long* q, int nL, int& k, int lane)
{
    const int home = blockIdx.x & 7;
    while (k < XQ_N) {
        const int x = (home + k) & 7;
        const int lo = (int)(((long long)nL * x) >> 3), hi = (int)(((long long)nL * (x + 1)) >> 3);
        const long long t = (long long)lo + wave_pop(&q[x * XQ_STRIDE], lane);
        if (t < hi) return (int)t;
        k++;
    }
    return -1;
}

__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline void shift_vec(int code, const DomainInfo& I, double* s)
{
    const int sh = code & 255;
    s[0] = (sh / 9 - 1) * I.L[0];
    s[1] = ((sh / 3) % 3 - 1) * I.L[1];
    s[2] = (sh % 3 - 1) * I.L[2];
}

// lanes per i-group for a chunk of nc particles: 8, 16, 32 or 64
__device__ inline int chunk_log2(int nc) { return nc <= 8 ? 3 : (nc <= 16 ? 4 : (nc <= 32 ? 5 : 6)); }

// Window [lo, hi) of B's particles (in the pair's sorted order) whose
// projection lies in [kmin, kmax).  Returns false if B is not sorted.
__device__ inline bool sorted_window(const float* skey, int64_t n, int dir, int bB, int nB, int lane, float kmin,
                                     float kmax, int& lo, int& hi)
{
    const float kb = (lane < nB) ? skey[(int64_t)dir * n + bB + lane] : INFINITY;
    lo = __popcll(__ballot(lane < nB && kb < kmin));
    hi = __popcll(__ballot(lane < nB && kb < kmax));
    return true;
}

// ---------------------------------------------------------------------------
// Pair-candidate selection.  For a neighbour cell B the particles that can
// interact with the wave's i particles are chosen either
//  - PRUNE_BOX: B's particles whose distance to the bounding box of the
//    wave's i particles is below the interaction range (3D test, one load of
//    B's cell per pair of cells, the next cell prefetched into registers), or
//  - PRUNE_SORTED: the window of B's particles sorted along the pair
//    direction whose projections lie within the range of the i projections
//    (the sort stage's per-direction order).
// ---------------------------------------------------------------------------
enum { PRUNE_BOX = 0, PRUNE_SORTED = 1 };

// Squared distance from p to the box [lo, hi].
template <typename T>
__device__ inline T box_d2(T px, T py, T pz, T lx, T ly, T lz, T hx, T hy, T hz)
{
    const T gx = fmax(fmax(lx - px, px - hx), T(0));
    const T gy = fmax(fmax(ly - py, py - hy), T(0));
    const T gz = fmax(fmax(lz - pz, pz - hz), T(0));
    return gx * gx + gy * gy + gz * gz;
}

// lane position among the set lanes of mask below it
__device__ inline int mask_rank(unsigned long long mask, int lane)
{
    const unsigned long long lt = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
    return __popcll(mask & lt);
}

// Add v to a partial count (PART_*) of the workgroup's line.
__device__ inline void count_add(unsigned long long* counters, int what, unsigned long long v)
{
    atomicAdd(&counters[CNT_PART + (blockIdx.x & (PART_N - 1)) * PART_STRIDE + what], v);
}

// Neighbour-entry batch of one wave, in LDS.
template <typename T, int NE = 64>
struct EBatch {
    int b[NE];     // first particle of B
    int n[NE];     // particles of B
    int B[NE];     // leaf index of B
    int dir[NE];   // sort direction of the pair
    T ox[NE], oy[NE], oz[NE];  // origin(B) + periodic shift - origin(A)
    T R[NE];       // interaction range of the pair (force)
};

// ---------------------------------------------------------------------------
// Density sweep + FP64 Newton step (eq. (rho); the smoothing-length
// constraint rho H^3 = C with its derivative 3 H^2 rho Omega).
// ---------------------------------------------------------------------------
struct DensArgs {
    int n_leaves;
    int64_t n;
    const int* l_begin;
    const int* l_count;
    const double* l_origin;
    const double* l_hlist;
    const int* l_dom;
    const int* l_off;
    const ListEntry* list;
    int* l_active;
    const int* l_sorted;
    const void* pos4;
    const float* skey;
    const uint16_t* sidx;
    const DomainInfo* di;
    const double* m;
    double* H;
    double* rho;
    double* drho;
    double* hlo;
    double* hhi;
    uint8_t* conv;
    int32_t* nngb;
    double C_fac;
    double h_tol;
    int* flags;
    unsigned long long* counters;
    const double* margin;  // list margin: twice the largest displacement since the lists were built
    const int* gate;    // graph mode: skip the sweep unless *gate == 0 (NULL: always run)
    const int* nl_dev;  // graph mode: leaf count read from the device (NULL: n_leaves)
    int big_only;       // skip leaves of at most 64 particles (done by the packed kernel)
    const int* wide;        // leaves with lists above *wide_min (NULL: all are taken as such)
    const int* n_wide_dev;  // their number, later their classes' (FI_NWIDE, FI_WIDECLASS)
    const int* wide_min;
    int n_wide;
};

#define NTD 4  // neighbour cells per two-phase batch (density)

template <typename T>
struct DTile {
    typename vec4<T>::type p[NTD][64];  // selected particles of B (B frame), w = m
    EBatch<T> e;
};

// Load the entries [eb, eb + nbt) of A's list, keep those that pass
// keep(E), compact them into the batch; returns their number.
template <typename T, typename Keep, int NE = 64>
__device__ inline int load_batch(const ListEntry* list, int eb, int nbt, int lane, const int* l_begin, const int* l_count,
                                 const double* l_origin, const double* oA, const DomainInfo& I, Keep keep, EBatch<T, NE>& E,
                                 const double* l_hlist, int A)
{
    bool ok = false;
    ListEntry en;
    if (lane < nbt) {
        en = list[eb + lane];
        ok = keep(en);
    }
    const unsigned long long mask = __ballot(ok);
    if (ok) {
        const int s = mask_rank(mask, lane);
        const int B = en.B;
        double sv[3];
        shift_vec(en.code, I, sv);
        E.b[s] = l_begin[B];
        E.n[s] = l_count[B];
        E.B[s] = B;
        E.dir[s] = en.code >> 8;
        E.ox[s] = (T)(l_origin[3 * B] + sv[0] - oA[0]);
        E.oy[s] = (T)(l_origin[3 * B + 1] + sv[1] - oA[1]);
        E.oz[s] = (T)(l_origin[3 * B + 2] + sv[2] - oA[2]);
        E.R[s] = (T)(l_hlist ? l_hlist[B] : 0.0);
    }
    wave_sync();
    return __popcll(mask);
}

// FP64 Newton step of particle i after a sweep at H (Sec. 2: the constraint
// rho H^3 = C, whose H-derivative is 3 H^2 rho Omega): from the sums Sw =
// sum m_j w(q), Sd = sum m_j (3 w + q w') and, in the FP32 modes, S2 = sum
// m_j (q^2 w'' + 2 q w') (the second H-derivative of rho H^3 up to 8/pi /
// H^2), writes rho, d rho/dH and the count, tests |rho H^3 - C| <= tol C,
// and otherwise updates H inside the particle's bracket.  hlA: the largest H
// the particle's neighbour list covers (beyond it the list must be rebuilt);
// hlim: a third of the box edge; s0min: the smallest top-cell edge.
// Returns true if the particle is left unconverged; conv: it is converged.
template <bool EXTRAP>
__device__ inline bool dens_newton(const DensArgs& a, int i, double H, double Sw, double Sd, double S2, int cnt,
                                   double hlA, double hlim, double s0min, double mi, bool& conv)
{
    const double rho = INV_PI_8 / (H * H * H) * Sw;
    const double drho = -INV_PI_8 / (H * H * H * H) * Sd;
    const double C = a.C_fac * mi;
    const double f = INV_PI_8 * Sw - C;              // rho H^3 - C
    const double fp = INV_PI_8 * (3.0 * Sw - Sd) / H; // 3 H^2 rho + H^3 drho/dH
    const double F2 = INV_PI_8 * S2 / (H * H);         // d^2 (rho H^3) / dH^2
    a.rho[i] = rho;
    a.drho[i] = drho;
    if (a.nngb) a.nngb[i] = cnt;
    bool left = false;
    bool done = fabs(f) <= a.h_tol * C;
    if (done && EXTRAP && f != 0.0) {
        // FP32 modes: the residual accepted here still moves rho by
        // f/C |1 - 1/Omega|; one Newton update of H with rho H^3 and its
        // H-derivative from their second-order expansion (as below) leaves
        // only the second-order term
        const double dH = -f / fp;
        const double Hn = H + dH;
        if (fabs(dH) <= 1e-3 * H && Hn <= hlA && Hn <= s0min) {
            const double F1 = INV_PI_8 * Sw + fp * dH + 0.5 * F2 * dH * dH;
            const double F1p = fp + F2 * dH;
            const double H3 = Hn * Hn * Hn;
            a.H[i] = Hn;
            a.rho[i] = F1 / H3;
            a.drho[i] = F1p / H3 - 3.0 * F1 / (H3 * Hn);
        }
    }
    if (!done) {
        double lo = a.hlo[i], hi = a.hhi[i];
        if (f < 0.0) lo = H;
        else hi = H;
        if (f < 0.0 && H >= hlim) {
            atomicOr(a.flags, FLAG_BOX_SMALL);
            done = true;
        } else {
            double Hn = H - f / fp;
            bool newton = true;
            if (!(Hn > lo && Hn < hi) || !isfinite(Hn)) {
                Hn = isinf(hi) ? 2.0 * H : 0.5 * (lo + hi);
                newton = false;
            }
            // at most doubling per sweep: a far-off step would only force
            // needless list and grid rebuilds before the bracket closes
            if (Hn > 2.0 * H) Hn = 2.0 * H;
            if (Hn > hlim) Hn = hlim;
            const double dH = Hn - H;
            if (fabs(dH) <= 4.0 * 2.220446049250313e-16 * H) {
                done = true;  // stalled at round-off: accept H
            } else if (EXTRAP && newton && fabs(dH) <= 1e-3 * H && Hn <= hlA && Hn <= s0min &&
                       fabs(0.5 * F2 * dH * dH) <= 0.5 * a.h_tol * C) {
                // accept the Newton update: rho H^3 and its H-derivative at Hn
                // from their second-order expansion around H
                const double F1 = INV_PI_8 * Sw + fp * dH + 0.5 * F2 * dH * dH;
                const double F1p = fp + F2 * dH;
                const double H3 = Hn * Hn * Hn;
                a.H[i] = Hn;
                a.rho[i] = F1 / H3;
                a.drho[i] = F1p / H3 - 3.0 * F1 / (H3 * Hn);
                done = true;
            } else {
                a.H[i] = Hn;
                a.hlo[i] = lo;
                a.hhi[i] = hi;
                if (Hn > hlA) atomicOr(a.flags, FLAG_RELIST);
                if (Hn > s0min) atomicOr(a.flags, FLAG_REBUILD);
                left = true;
            }
        }
    }
    if (done) a.conv[i] = 1;
    conv = done;
    return left;
}

// Counts of one wave's particles after their Newton step: interactions
// evaluated by the sweep, interactions of the converged particles, particles left.
__device__ inline void dens_count(const DensArgs& a, bool act, bool left, bool conv, int cnt, int lane)
{
    const unsigned long long ev = wave_sum(act ? (unsigned long long)cnt : 0ull);
    const unsigned long long lm = __ballot(left);
    const unsigned long long nd = __ballot(act && !conv) ? wave_sum(conv ? (unsigned long long)cnt : 0ull) : ev;
    if (lane != 0) return;
    if (ev) count_add(a.counters, PART_DEVAL, ev);
    if (nd) count_add(a.counters, PART_NDENS, nd);
    if (lm) count_add(a.counters, PART_UNCONV, (unsigned long long)__popcll(lm));
}

// Sums of one sweep -> rho, d rho/dH, neighbour count, and the FP64 Newton
// step (dens_newton).  The lanes of group 0 (jg == 0) own particle i; partial
// sums of the other groups are folded in first.  Returns true if particle i
// is left unconverged.
template <typename T>
__device__ inline bool dens_finish(const DensArgs& a, int i, bool act, int jg, int CI, double Hd, double Sw0,
                                   double Sd0, double S20, int cnt, double hlA, double hlim, double s0min, double mi)
{
    constexpr bool EXTRAP = sizeof(T) == 4;
    const int lane = threadIdx.x & 63;
    double Sw = Sw0, Sd = Sd0, S2 = S20;
    for (int off = CI; off < 64; off <<= 1) {
        Sw += __shfl_xor(Sw, off);
        Sd += __shfl_xor(Sd, off);
        if (EXTRAP) S2 += __shfl_xor(S2, off);
        cnt += __shfl_xor(cnt, off);
    }
    bool left = false, conv = false;
    if (jg == 0 && act) left = dens_newton<EXTRAP>(a, i, Hd, Sw, Sd, S2, cnt, hlA, hlim, s0min, mi, conv);
    dens_count(a, jg == 0 && act, left, conv, cnt, lane);
    return left;
}

// ---------------------------------------------------------------------------
// Pair selection and pair-parallel evaluation, shared by the density and the
// gather force kernels (one wave per leaf A, lane = particle i of A).
//
// Candidates.  The particles of a batch of neighbour cells form one stream
// (EFlat: prefix sums of the cells' counts), read 64 per step whatever the
// cells hold, so no lane idles on cells of fewer than 64 particles; the
// next step's positions are loaded while this one is tested.  Those within
// reach of the leaf's box are packed into a tile of 4 ROW candidates in LDS (ROW of
// them for each 16-lane row of the masks).
//
// Range tests (tile_masks).  All 4 ROW x 64 tests of a full tile run on the
// matrix units: r^2 - H_i^2 = -2 p_j.p_i + |p_j|^2 + (|p_i|^2 - H_i^2) is a
// product over (x, y, z, 1) plus a row constant, one
// v_mfma_f32_16x16x16_bf16 per 16 x 16 tests, and the sign bits are the mask
// (one v_alignbit per 64 tests instead of the ~11 instructions of a
// per-particle loop with a ballot).  Each factor is a sum of two bfloat16, a
// product x y the three terms xh yh + xh ym + xm yh: half of the float32
// product's matrix time, and work that VALU instructions of other waves
// overlap, which float32 products do not.  What the terms leave out is below 3
// 2^-18 |x y| per coordinate, 2^-16 (|p_i|^2 + |p_j|^2) in all with the
// roundings of the sum, so every constant is shifted by PAIR_EPS = 2^-14 of it
// towards "in range", four times the error.  No pair is lost; the 0.2% that
// are let in wrongly contribute exact zeros below (q >= 1).
// Coordinates and smoothing lengths are scaled by a power of two (exact) to
// order 1, so nothing over- or underflows that did not before; the sums only
// hold r / H and unit vectors, which the scale leaves as they are.
//
// Evaluation.  The set bits become a list of (i, j) pairs ordered by i and
// every lane takes an equal run of it, so all lanes work on pairs in range:
// with lane = particle the same work took as many rounds as the fullest
// particle of each tile has neighbours (18% of the lanes active at 256^3
// clustered).  A lane sums in FP64 (v_add_f64 runs at the FP32 rate, a
// compensated FP32 addition takes four) and adds its sum to the particle's
// LDS accumulator where the run passes from one particle to the next.
// ---------------------------------------------------------------------------
#define PAIR_CAP 512  // pairs listed at a time (a tile usually has ~300)
#define PAIR_EPS 6.1035156e-5f  // 2^-14

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16v2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// a (low half) and b rounded to bfloat16 (nearest even)
__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    const bf16v2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float bf16_high(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }

// Batch of up to NE neighbour cells as one stream of candidates.
template <typename T, int NE>
struct EFlat {
    typename vec4<T>::type o[NE];  // origin(B) + periodic shift - origin(A), scaled; w: first particle minus start
    int st[NE];                    // start of the cell in the stream
};
__device__ inline float pack_int(int v, float) { return __int_as_float(v); }
__device__ inline double pack_int(int v, double) { return (double)v; }
__device__ inline int unpack_int(float v) { return __float_as_int(v); }
__device__ inline int unpack_int(double v) { return (int)v; }

__device__ inline int lane_rank(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Load the entries [eb, eb + nbt) of A's list that pass keep(E) into the
// batch; returns the particles they hold in all.  start: the lane's cell's
// first position in the stream (INT_MAX past the last cell).
template <typename T, typename Keep, int NE>
__device__ inline int load_batch_flat(const ListEntry* list, int eb, int nbt, int lane, const int* l_begin,
                                      const int* l_count, const double* l_origin, const double* oA,
                                      const DomainInfo& I, T sc, Keep keep, EFlat<T, NE>& E, int& start)
{
    // everything of the entry's cell is loaded at once: one latency
    ListEntry en = {0, 0, INFINITY};
    if (lane < nbt) en = list[eb + lane];
    const bool ok = (lane < nbt) && keep(en);
    const int n0 = ok ? l_count[en.B] : 0;
    const unsigned long long mask = __ballot(ok);
    const int n = ok ? n0 : 0;
    static_assert(NE == 32, "the prefix sum below covers two rows");
    int incl = n;
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, true);
    if (lane >= 16) incl += __builtin_amdgcn_readlane(incl, 15);
    if (ok) {
        const int s = lane_rank(mask);
        double sv[3];
        shift_vec(en.code, I, sv);
        typename vec4<T>::type o;
        const double* q = l_origin + 3 * (size_t)en.B;
        const double q0 = q[0], q1 = q[1], q2 = q[2];
        const int b0 = l_begin[en.B];
        o.x = (T)(q0 + sv[0] - oA[0]) * sc;
        o.y = (T)(q1 + sv[1] - oA[1]) * sc;
        o.z = (T)(q2 + sv[2] - oA[2]) * sc;
        o.w = pack_int(b0 - (incl - n), T(0));
        E.o[s] = o;
        E.st[s] = incl - n;
    }
    wave_sync();
    start = lane < __popcll(mask) ? E.st[lane] : 0x7fffffff;
    return __builtin_amdgcn_readlane(incl, NE - 1);
}

// Cell (index in the batch) of the lane's candidate p0 + lane: the cells that
// start by p0, then one more at each lane where a cell starts.
__device__ inline int stream_cell(int p0, int start)
{
    const int d = start - p0;
    const int at = (uint32_t)(d - 1) < 63u ? d << 2 : 0;
    const unsigned long long mask = __ballot(__builtin_amdgcn_ds_permute(at, 1) != 0) >> 1;  // (lane 0 collects the rest)
    return __popcll(__ballot(d <= 0)) - 1 + lane_rank(mask);
}

// Power of two that brings lengths up to x to order 1 (x > 0 finite).
__device__ inline float pow2_scale(float x) { return __builtin_amdgcn_ldexpf(1.0f, -__builtin_amdgcn_frexp_expf(x)); }
__device__ inline double pow2_scale(double x) { return __builtin_amdgcn_ldexp(1.0, -__builtin_amdgcn_frexp_exp(x)); }

// Test operand of the particles i, one value v per lane and block of 16
// particles: lane l holds component l / 16 of (-2x, -2y, -2z, c) of particle
// 16 blk + l % 16, as the four slots (vh, vm, vh, .) that meet a candidate's
// (xh, xh, xm, 1); for c, which meets ones, (ch, cm, 0, cl).  The open slots of
// x, y and z hold the three terms of `own`, a constant that only the first of
// two tests takes in (the second has zeros there).  (x, y, z, c), own: the
// lane's own particle, scaled; tmp: 64 float4 of LDS.
__device__ inline void test_operand(float x, float y, float z, float c, float own, float4* tmp, int lane, bf16x4 b[4])
{
    wave_sync();
    tmp[lane] = make_float4(-2.0f * x, -2.0f * y, -2.0f * z, c);
    wave_sync();
    float v[4];
    for (int k = 0; k < 4; k++) v[k] = ((const float*)&tmp[16 * k + (lane & 15)])[lane >> 4];
    wave_sync();
    const float oh = bf16_high(bf16_pair(own, own)), om = bf16_high(bf16_pair(own, own - oh));
    tmp[lane] = make_float4(oh, om, own - oh - om, 0.0f);
    wave_sync();
    for (int k = 0; k < 4; k++) {
        const float vh = bf16_high(bf16_pair(v[k], v[k])), vm = bf16_high(bf16_pair(v[k], v[k] - vh));
        const float o = ((const float*)&tmp[16 * k + (lane & 15)])[lane >> 4];
        const u32x2 s = {bf16_pair(vh, vm), lane < 48 ? bf16_pair(vh, o) : bf16_pair(0.0f, v[k] - vh - vm)};
        b[k] = __builtin_bit_cast(bf16x4, s);
    }
    wave_sync();
}

// In-range masks of a full tile: bit ROW - 1 - b of M[k] of lane l belongs to
// the particle 16 k + l % 16 and the candidate 4 b + l / 16 (candidates are
// dealt to the four rows in turn: neighbours in the stream are neighbours in
// space, and a particle's pairs come in runs; with a row of ROW consecutive
// candidates each, the fullest lanes had twice the pairs).  coord(j):
// component l / 16 of candidate j (scaled; 1 for l / 16 = 3); c1, c2: row
// constants of the tests against H_i and (TWO) H_j, candidate j's at
// test_slot(j).
template <int ROW>
__device__ inline int test_slot(int j) { return (j & 3) * ROW + (j >> 2); }

template <bool TWO, int ROW, int NB, typename Coord>
__device__ inline void tile_masks_n(const float* c1, const float* c2, Coord coord, const bf16x4 b[4],
                                    int lane, uint32_t M[4])
{
    const int g = lane >> 4;
#pragma unroll
    for (int t = 0; t < ROW / 4; t++) {
        const float v = coord(16 * t + 4 * (lane & 3) + ((lane >> 2) & 3));
        const uint32_t vh = bf16_pair(v, v);
        const uint32_t vm = bf16_pair(v - bf16_high(vh), 1.0f);
        const u32x2 s1 = {vh, vm}, s2 = {vh, lane < 48 ? vm & 0xffffu : vm};
        const bf16x4 a1 = __builtin_bit_cast(bf16x4, s1), a2 = __builtin_bit_cast(bf16x4, s2);
        const f32x4 r1 = *(const f32x4*)(c1 + ROW * g + 4 * t);
        const f32x4 r2 = TWO ? *(const f32x4*)(c2 + ROW * g + 4 * t) : r1;
        f32x4 d1[NB], d2[NB];
#pragma unroll
        for (int k = 0; k < NB; k++) {
            d1[k] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, b[k], r1, 0, 0, 0);
            if (TWO) d2[k] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a2, b[k], r2, 0, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < NB; k++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                uint32_t s = __float_as_uint(d1[k][r]);
                if (TWO) s |= __float_as_uint(d2[k][r]);
                M[k] = __builtin_amdgcn_alignbit(M[k], s, 31);
            }
    }
}
// nb: blocks of 16 particles up to the last that holds any (1..4)
template <bool TWO, int ROW, typename Coord>
__device__ inline void tile_masks(const float* c1, const float* c2, Coord coord, const bf16x4 b[4],
                                  int nb, int lane, uint32_t M[4])
{
    if (nb <= 2) tile_masks_n<TWO, ROW, 2>(c1, c2, coord, b, lane, M);
    else if (nb == 3) tile_masks_n<TWO, ROW, 3>(c1, c2, coord, b, lane, M);
    else tile_masks_n<TWO, ROW, 4>(c1, c2, coord, b, lane, M);
}

// Exclusive prefix sums over (particle, row of 16 lanes) of two 16-bit counts
// packed in v; the totals in `total`.
__device__ inline uint32_t scan_pairs(uint32_t v, int lane, uint32_t& total)
{
    // rows of the same particle
    const auto h = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    uint32_t ex = (lane & 16) ? (uint32_t)h[0] : 0u;
    const uint32_t s = (uint32_t)h[0] + (uint32_t)h[1];
    const auto w = __builtin_amdgcn_permlane32_swap(s, s, false, false);
    if (lane & 32) ex += (uint32_t)w[0];
    const uint32_t own = (uint32_t)w[0] + (uint32_t)w[1];
    // particles of the row
    uint32_t in = own;
    in += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)in, 0x111, 0xf, 0xf, true);
    in += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)in, 0x112, 0xf, 0xf, true);
    in += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)in, 0x114, 0xf, 0xf, true);
    in += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)in, 0x118, 0xf, 0xf, true);
    total = (uint32_t)__builtin_amdgcn_readlane((int)in, 15);
    return in - own + ex;
}

// The pairs of the masks, PAIR_CAP at a time: listed as i << 7 | j in the order
// of i, then eval(list, n) with n of them in the list.  ready() runs before
// the first eval.
template <int ROW, typename Ready, typename Eval>
__device__ inline void for_pairs(const uint32_t M[4], uint16_t* list, int lane, Ready ready, Eval eval)
{
    uint32_t t01, t23;
    const uint32_t e01 = scan_pairs((uint32_t)__popc(M[0]) | ((uint32_t)__popc(M[1]) << 16), lane, t01);
    const uint32_t e23 = scan_pairs((uint32_t)__popc(M[2]) | ((uint32_t)__popc(M[3]) << 16), lane, t23);
    const int n0 = (int)(t01 & 0xffffu), n1 = n0 + (int)(t01 >> 16), n2 = n1 + (int)(t23 & 0xffffu);
    const int np = n2 + (int)(t23 >> 16);
    const int at[4] = {(int)(e01 & 0xffffu), n0 + (int)(e01 >> 16), n1 + (int)(e23 & 0xffffu), n2 + (int)(e23 >> 16)};
    const int code = ((lane & 15) << 7) + (lane >> 4) - 4 * (32 - ROW);
    for (int w = 0; w < np; w += PAIR_CAP) {
        wave_sync();
#pragma unroll
        for (int k = 0; k < 4; k++) {
            uint32_t m = M[k];
            int p = at[k] - w;
            if (np <= PAIR_CAP) {
                while (m) {
                    const int b = __builtin_clz(m);
                    m ^= 0x80000000u >> b;
                    list[p++] = (uint16_t)((k << 11) + code + 4 * b);
                }
            } else {
                while (m) {
                    const int b = __builtin_clz(m);
                    m ^= 0x80000000u >> b;
                    if ((uint32_t)p < (uint32_t)PAIR_CAP) list[p] = (uint16_t)((k << 11) + code + 4 * b);
                    p++;
                }
            }
        }
        if (w == 0) ready();
        wave_sync();
        eval(list, min(PAIR_CAP, np - w));
    }
}

__device__ inline float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

__device__ inline void lds_add(double* p, double v)
{
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ inline void lds_add(float* p, float v)
{
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ inline void lds_add(int* p, int v)
{
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Force sums of one particle (acceleration and du/dt).
template <typename T, bool COMP>
struct FAcc {
    Acc<T, COMP> ax, ay, az, du;
};

