// Bottom solver: the levels from the first one whose data fit the LDS of a
// compute unit down to the coarsest grid, one workgroup per request.
#include "device.h"

// A value kept in a register is rounded as one stored in LDS: products and
// sums are contracted within an expression only.
#pragma clang fp contract(on)

namespace mhs {
namespace {

// ============================================================================
// One workgroup runs a whole V(nu1,nu2) cycle over the small levels of one
// request, from a zero initial guess, in FP64, with exact red-black
// Gauss-Seidel ordering and an exact dense solve on the coarsest grid.  Every
// work array lives in LDS (up to 160 KB on gfx950), so each phase (half-sweep,
// residual, transfer) costs LDS latency, not HBM latency.
//
// A cycle has about forty phases of little work with a barrier after each, so
// what counts is the length of a phase: for the coarse ones the latency
// of a read, seven dependent FP64 operations, a write and a barrier (some 550
// cycles).  A thread owns the same pairs of
// consecutive x nodes (one red, one black) of a level in all its phases: it
// keeps their values, right-hand sides, coefficients and LDS addresses in
// registers and reads one x, two y and two z neighbours per update.  The
// interior nodes of a row (2^L - 1) are 2^(L-1) pairs, so rows map to whole
// groups of lanes.  A row lies in LDS with its odd columns first, so the
// accesses of one colour are to consecutive doubles.  The prolongation corrects the black nodes only, since the
// half-sweep after it replaces the red ones without reading them.  No phase
// branches on a lane's node, so the reads of a thread's pairs go out together:
// a pair that does not exist computes on an existing one and is stored to a
// cell that is never read, a pair's node on the boundary is stored as zero.
// Levels of at most 64 pairs are run by one wave, whose LDS accesses are in
// order, without barriers.
//
// Measured per call in 257^3 solves: 22.3 us for 17^3 nodes (FP32 storage) and
// 19.2 us for 65^2; with a walk over rows in every phase (a division and ten
// LDS reads per node) 32.3 and 35.4 us.
// ============================================================================
static_assert(kBottomMaxPairs == 3 * kBottomThreads, "at most three pairs per thread");

extern __shared__ double smem[];
__device__ __forceinline__ double &at_byte(int off) { return *(double *)((char *)smem + off); }

struct BottomLevel {
    int nx, sxy, lg, cnt, rows, my;
    float rmy; // 1 / my
    int u, f, cf; // byte offsets in LDS
    double cz;
};

__device__ __forceinline__ BottomLevel bottom_level(const BottomItem &b, int l)
{
    BottomLevel v;
    const int nx = b.n[l][0], ny = b.n[l][1], nz = b.n[l][2];
    v.nx = nx;
    v.sxy = nx * ny;
    v.lg = 30 - __builtin_clz((unsigned)(nx - 1)); // 2^lg = (nx - 1) / 2 pairs per row
    v.cnt = 1 << v.lg;
    v.my = ny - 2;
    v.rmy = 1.0f / (float)v.my;
    v.rows = v.my * (b.planar ? 1 : nz - 2);
    v.u = 8 * b.off_u[l];
    v.f = 8 * b.off_f[l];
    v.cf = 8 * b.off_c[l];
    v.cz = b.cz[l];
    return v;
}

// Orders the LDS accesses of the workgroup, or (WAVE) of a wave working alone.
template <bool WAVE>
__device__ __forceinline__ void bottom_sync()
{
    if constexpr (WAVE)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    else
        lds_barrier();
}

// a / d for 0 <= a < 2^20, r = 1.0f / d: (a + 1/2) / d is at least 1/(2d) away
// from an integer, and the product off by less than that.
__device__ __forceinline__ int bottom_div(int a, float r) { return (int)(((float)a + 0.5f) * r); }

// Place of column i in a row of a level with cnt pairs per row: odd columns
// first.
__device__ __forceinline__ int bottom_col(int i, int cnt) { return (i >> 1) + (i & 1 ? 0 : cnt); }

// Full weighting of the residual (ry, rz the byte strides of the finer level)
// at byte offset c: along x and y (xyc; o is the offset of the node before,
// the node after follows that), along z (zc), or both.
__device__ __forceinline__ double bottom_weighted(int c, int o, int ry, int rz, bool xyc, bool zc)
{
    auto row = [&](int d) { return 0.25 * at_byte(o + d) + 0.5 * at_byte(c + d) + 0.25 * at_byte(o + d + 8); };
    auto pl = [&](int d) { return 0.25 * row(d - ry) + 0.5 * row(d) + 0.25 * row(d + ry); };
    if (!zc) return pl(0);
    if (!xyc) return 0.25 * at_byte(c - rz) + 0.5 * at_byte(c) + 0.25 * at_byte(c + rz);
    return 0.25 * pl(-rz) + 0.5 * pl(0) + 0.25 * pl(rz);
}

// Interior node p of level L in x-y-z order.
__device__ __forceinline__ void bottom_node(const BottomLevel &L, int p, bool planar, int &I, int &J, int &K)
{
    const int mx = L.nx - 2;
    const int pr = p / mx, pk = bottom_div(pr, L.rmy);
    I = 1 + p - pr * mx;
    J = 1 + pr - pk * L.my;
    K = planar ? 0 : pk + 1;
}

// Right-hand side of level l from the residual of the level above, in LDS:
// node by node (compact: one value per interior node in x-y-z order).
template <bool PLANAR, bool WAVE>
__device__ __forceinline__ void bottom_restrict(const BottomItem &b, int l, const BottomLevel &L, bool compact)
{
    const BottomLevel F = bottom_level(b, l - 1);
    const bool xyc = L.nx < F.nx, zc = !PLANAR && b.n[l][2] < b.n[l - 1][2];
    const int m = (L.nx - 2) * L.rows, r = 8 * b.off_r;
#pragma unroll 1
    for (int p = (int)threadIdx.x; p < m; p += WAVE ? 64 : kBottomThreads) {
        int I, J, K;
        bottom_node(L, p, PLANAR, I, J, K);
        const int row = r + 8 * (F.nx * (xyc ? 2 * J : J) + F.sxy * (zc ? 2 * K : K));
        const int c = row + 8 * (xyc ? F.cnt + I : bottom_col(I, F.cnt)), o = row + 8 * (I - 1);
        at_byte(L.f + 8 * (compact ? p : bottom_col(I, L.cnt) + L.nx * J + L.sxy * K)) =
            bottom_weighted(c, o, 8 * F.nx, 8 * F.sxy, xyc, zc);
    }
    bottom_sync<WAVE>();
}

// The coarsest grid: u = Minv f over its interior nodes.
template <typename T, bool PLANAR, bool WAVE>
__device__ __forceinline__ void bottom_coarsest(const BottomItem &b)
{
    constexpr int NT = WAVE ? 64 : kBottomThreads;
    const int l = b.nlev - 1, m = b.m;
    const BottomLevel L = bottom_level(b, l);
    const MHS_GLOBAL double *minv = gin<double>(b.minv);
    int I, J, K;
    if (l == 0) {
        for (int p = (int)threadIdx.x; p < m; p += NT) {
            bottom_node(L, p, PLANAR, I, J, K);
            at_byte(L.f + 8 * p) = (double)gin<T>(b.f_top)[I + L.nx * J + L.sxy * K];
        }
        bottom_sync<WAVE>();
    } else {
        bottom_restrict<PLANAR, WAVE>(b, l, L, true);
    }
#pragma unroll 1
    for (int p = (int)threadIdx.x; p < m; p += NT) {
        double acc = 0.0;
        for (int q = 0; q < m; ++q) acc += minv[(size_t)p * m + q] * at_byte(L.f + 8 * q);
        bottom_node(L, p, PLANAR, I, J, K);
        at_byte(L.u + 8 * (bottom_col(I, L.cnt) + L.nx * J + L.sxy * K)) = acc;
    }
    bottom_sync<WAVE>();
}

// The coefficient tables of every level into LDS.
__device__ __forceinline__ void bottom_tables(const BottomItem &b)
{
    const int tid = (int)threadIdx.x;
    constexpr int kAtOnce = 4; // levels whose tables are in flight together
#pragma unroll 1
    for (int l0 = 0; l0 < b.nlev; l0 += kAtOnce) {
        double c[kAtOnce];
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q) {
            const int l = min(l0 + q, b.nlev - 1);
            c[q] = gin<double>(b.coef[l])[min(tid, 4 * b.n[l][2] - 1)];
        }
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q) {
            const int l = l0 + q;
            if (l >= b.nlev) break;
            const int nc = 4 * b.n[l][2];
            if (tid < nc) smem[b.off_c[l] + tid] = c[q];
            for (int e = tid + kBottomThreads; e < nc; e += kBottomThreads)
                smem[b.off_c[l] + e] = gin<double>(b.coef[l])[e];
        }
    }
    lds_barrier();
}

// The pairs of one thread on one level, by colour (0 red, 1 black).
// GEN: the general operator, whose diagonal differs from node to node.
template <bool PLANAR, int NP, bool WAVE, bool GEN>
struct BottomPairs {
    BottomLevel L;
    int r;                      // byte offset of the residual
    int i[NP][2], j[NP], k[NP]; // node coordinates
    int at[NP][2], ext[NP][2];  // byte offsets in u of the node and of its outer x neighbour
    int st[NP][2];              // where the node is stored
    bool on[NP][2], pair[NP];   // an interior node; the pair exists
    bool busy;                  // the wave has pairs
    double u[NP][2], f[NP][2], c0[NP], c1[NP];
    double cd[NP][GEN ? 2 : 1], c3[NP][GEN ? 2 : 1]; // diagonal and its inverse
    double be[NP][GEN ? 2 : 1];                      // b/a

    __device__ __forceinline__ BottomPairs(const BottomItem &b, int l) : L(bottom_level(b, l)), r(8 * b.off_r)
    {
        const int tid = (int)threadIdx.x, cnt = L.cnt, q = tid & (cnt - 1);
        const int per = kBottomThreads >> L.lg;
        bool any = false;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int row = (tid >> L.lg) + p * per;
            pair[p] = row < L.rows;
            any |= pair[p];
            const int rr = pair[p] ? row : 0;
            const int kk = PLANAR ? 0 : bottom_div(rr, L.rmy);
            j[p] = 1 + rr - kk * L.my;
            k[p] = PLANAR ? 0 : kk + 1;
            const int s = (j[p] + k[p] + 1) & 1; // the red node is the pair's first (0) or second
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int sc = c ? 1 - s : s;
                i[p][c] = 1 + 2 * q + sc;
                const int first = L.u + 8 * (L.nx * j[p] + L.sxy * k[p]);
                at[p][c] = first + 8 * (sc ? cnt + q + 1 : q);
                ext[p][c] = first + 8 * (sc ? q + 1 : cnt + q);
                st[p][c] = pair[p] ? at[p][c] : r;
                on[p][c] = !(sc && q == cnt - 1);
                u[p][c] = f[p][c] = 0.0;
            }
        }
        busy = WAVE || __any(any);
        if constexpr (GEN) {
            const MHS_GLOBAL double *bg = gin<double>(b.beta[l]);
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int c = 0; c < 2; ++c) be[p][c] = bg[i[p][c] + L.nx * j[p] + L.sxy * k[p]];
        }
    }
    // coefficients and right-hand side from LDS, and u (on the way up)
    __device__ __forceinline__ void load(bool with_u)
    {
        if (!busy) return;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = L.cf + 32 * k[p];
            c0[p] = at_byte(c);
            c1[p] = at_byte(c + 8);
            if constexpr (GEN) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    cd[p][h] = be[p][h] + at_byte(c + 16);
                    c3[p][h] = 1.0 / cd[p][h];
                }
            } else {
                cd[p][0] = at_byte(c + 16);
                c3[p][0] = at_byte(c + 24);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f[p][h] = at_byte(at[p][h] + (L.f - L.u));
                if (with_u) u[p][h] = on[p][h] ? at_byte(at[p][h]) : 0.0;
            }
        }
    }
    __device__ __forceinline__ double neighbours(int p, int c) const
    {
        const int a = at[p][c], ry = 8 * L.nx, rz = 8 * L.sxy;
        double o = c0[p] * (at_byte(ext[p][c]) + u[p][1 - c]) + c1[p] * (at_byte(a + ry) + at_byte(a - ry));
        if constexpr (!PLANAR) o += L.cz * (at_byte(a + rz) + at_byte(a - rz));
        return o;
    }
    // node c of every pair, in LDS and in the registers
    __device__ __forceinline__ void set(int c, const double (&v)[NP])
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            u[p][c] = on[p][c] ? v[p] : 0.0;
            at_byte(st[p][c]) = u[p][c];
        }
    }
    template <int C>
    __device__ __forceinline__ void colour()
    {
        if (busy) {
            double v[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) v[p] = (f[p][C] - neighbours(p, C)) * c3[p][GEN ? C : 0];
            set(C, v);
        }
        bottom_sync<WAVE>();
    }
    __device__ __forceinline__ void sweeps(int n)
    {
#pragma unroll 1
        for (int s = 0; s < n; ++s) {
            colour<0>();
            colour<1>();
        }
    }
    // n sweeps from u = 0 (the first red half-sweep reads nothing), then the
    // residual, laid out as u
    __device__ __forceinline__ void down(int n)
    {
        if (busy) {
            double v[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) v[p] = f[p][0] * c3[p][0];
            set(0, v);
        }
        bottom_sync<WAVE>();
        colour<1>();
        sweeps(n - 1);
        if (busy) {
            double v[NP][2];
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int a = at[p][c], ry = 8 * L.nx, rz = 8 * L.sxy;
                    double au = c0[p] * (at_byte(ext[p][c]) + u[p][1 - c]) +
                                c1[p] * (at_byte(a + ry) + at_byte(a - ry)) + cd[p][GEN ? c : 0] * u[p][c];
                    if constexpr (!PLANAR) au += L.cz * (at_byte(a + rz) + at_byte(a - rz));
                    v[p][c] = f[p][c] - au;
                }
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int c = 0; c < 2; ++c) at_byte(pair[p] ? at[p][c] + (r - L.u) : r) = v[p][c];
        }
        bottom_sync<WAVE>();
    }
    // the correction of the coarser level C at the black nodes: trilinear
    // (bilinear within planes when the step keeps z), along z when it keeps x
    // and y.  An even index takes its coarse node twice: 0.5 (v + v) is v.
    __device__ __forceinline__ void correct(const BottomLevel &C, bool xyc, bool zc)
    {
        if (busy) {
            double v[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int I = on[p][1] ? i[p][1] : 1, J = j[p], K = k[p];
                const int I0 = xyc ? I >> 1 : I, I1 = xyc ? (I + 1) >> 1 : I;
                const int dx = 8 * (bottom_col(I1, C.cnt) - bottom_col(I0, C.cnt)), dy = xyc && (J & 1) ? 8 * C.nx : 0;
                const int dz = zc && (K & 1) ? 8 * C.sxy : 0;
                const int a = C.u + 8 * (bottom_col(I0, C.cnt) + C.nx * (xyc ? J >> 1 : J) + C.sxy * (zc ? K >> 1 : K));
                auto X = [&](int e) { return 0.5 * (at_byte(e) + at_byte(e + dx)); };
                auto Y = [&](int e) { return 0.5 * (X(e) + X(e + dy)); };
                v[p] = u[p][1] + (PLANAR ? Y(a) : 0.5 * (Y(a) + Y(a + dz)));
            }
            set(1, v);
        }
        bottom_sync<WAVE>();
    }
};

template <bool PLANAR, int NP, bool WAVE, bool GEN>
__device__ __forceinline__ void bottom_down(const BottomItem &b, int l)
{
    BottomPairs<PLANAR, NP, WAVE, GEN> P(b, l);
    bottom_restrict<PLANAR, WAVE>(b, l, P.L, false);
    P.load(false);
    P.down(b.nu1);
}

template <bool PLANAR, int NP, bool WAVE, bool GEN>
__device__ __forceinline__ void bottom_up(const BottomItem &b, int l)
{
    BottomPairs<PLANAR, NP, WAVE, GEN> P(b, l);
    P.load(true);
    const BottomLevel C = bottom_level(b, l + 1);
    P.correct(C, C.nx < P.L.nx, !PLANAR && b.n[l + 1][2] < b.n[l][2]);
    P.sweeps(b.nu2);
}

// The cycle over levels of at most NP pairs per thread; false if the solve
// was done (nothing has been computed then).
template <typename T, bool GEN, bool PLANAR, int NP>
__device__ __forceinline__ bool bottom_cycle(const BottomItem &b)
{
    const int n = b.nlev;
    {
        BottomPairs<PLANAR, NP, false, GEN> P(b, 0);
        const MHS_GLOBAL T *ft = gin<T>(b.f_top);
        const int done = b.state ? gin<SolveState>(b.state)->done : 0;
        T ftop[NP][2];
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int c = 0; c < 2; ++c) ftop[p][c] = ft[P.i[p][c] + P.L.nx * P.j[p] + P.L.sxy * P.k[p]];
        bottom_tables(b);
        if (done) return false;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int c = 0; c < 2; ++c) at_byte((P.pair[p] ? P.at[p][c] : P.L.u) + (P.L.f - P.L.u)) = (double)ftop[p][c];
        P.load(false);
        P.down(b.nu1);
    }
    auto pairs = [&](int l) {
        return ((b.n[l][0] - 1) >> 1) * (b.n[l][1] - 2) * (PLANAR ? 1 : b.n[l][2] - 2);
    };
    int l = 1;
    for (; l < n - 1 && pairs(l) > 64; ++l) {
        if (pairs(l) <= kBottomThreads)
            bottom_down<PLANAR, 1, false, GEN>(b, l);
        else
            bottom_down<PLANAR, 3, false, GEN>(b, l);
    }
    const int w = l; // the first level that one wave runs
    if (w < n - 1) {
        if (threadIdx.x < 64) {
            for (; l < n - 1; ++l) bottom_down<PLANAR, 1, true, GEN>(b, l);
            bottom_coarsest<T, PLANAR, true>(b);
            for (l = n - 2; l >= w; --l) bottom_up<PLANAR, 1, true, GEN>(b, l);
        }
        lds_barrier();
    } else {
        bottom_coarsest<T, PLANAR, false>(b);
    }
    for (l = w - 1; l > 0; --l) {
        if (pairs(l) <= kBottomThreads)
            bottom_up<PLANAR, 1, false, GEN>(b, l);
        else
            bottom_up<PLANAR, 3, false, GEN>(b, l);
    }
    bottom_up<PLANAR, NP, false, GEN>(b, 0);
    return true;
}

template <typename T, bool GEN, bool PLANAR>
__device__ __forceinline__ bool bottom_solve(const BottomItem &b)
{
    const int pairs = ((b.n[0][0] - 1) >> 1) * (b.n[0][1] - 2) * (PLANAR ? 1 : b.n[0][2] - 2);
    if (b.nlev == 1) {
        if (b.state && gin<SolveState>(b.state)->done) return false;
        bottom_coarsest<T, PLANAR, false>(b);
        return true;
    }
    if (pairs <= kBottomThreads) return bottom_cycle<T, GEN, PLANAR, 1>(b);
    if (pairs <= 2 * kBottomThreads) return bottom_cycle<T, GEN, PLANAR, 2>(b);
    return bottom_cycle<T, GEN, PLANAR, 3>(b);
}

template <typename T, bool GEN>
__global__ __launch_bounds__(kBottomThreads) void k_bottom(const BottomItem *__restrict__ items, int nitems, int lds_bytes)
{
    const BottomItem &b = items[blockIdx.x];
    // the item's cache lines, in flight together (its fields are read in
    // several dependent steps), while the LDS is cleared
    {
        const int *w = (const int *)&b;
        int any = 0;
#pragma unroll
        for (int q = 0; q < (int)sizeof(BottomItem) / 64; ++q) any |= w[16 * q];
        asm volatile("" ::"s"(any));
    }
    for (int e = (int)threadIdx.x; e < lds_bytes / 8; e += kBottomThreads) smem[e] = 0.0;
    lds_barrier();
    if (!(b.planar ? bottom_solve<T, GEN, true>(b) : bottom_solve<T, GEN, false>(b))) return;
    const int nx = b.n[0][0], N0 = nx * b.n[0][1] * b.n[0][2];
    const double *u = smem + b.off_u[0];
    MHS_GLOBAL T *ut = gout<T>(b.u_top);
    const float rnx = 1.0f / (float)nx;
    for (int e = (int)threadIdx.x; e < N0; e += kBottomThreads) {
        const int row = bottom_div(e, rnx);
        ut[e] = (T)u[row * nx + bottom_col(e - row * nx, (nx - 1) >> 1)];
    }
}

} // namespace

hipError_t launch_bottom(const BottomItem *items, int nitems, int lds_bytes, bool gen, bool dbl, hipStream_t s)
{
    if (nitems <= 0) return hipSuccess;
    if (lds_bytes <= 0 || lds_bytes > kBottomLdsMax || (gen && !dbl)) return hipErrorInvalidValue;
    static bool attr_set = false;
    if (!attr_set) {
        for (const void *k : {reinterpret_cast<const void *>(&k_bottom<double, false>),
                              reinterpret_cast<const void *>(&k_bottom<float, false>),
                              reinterpret_cast<const void *>(&k_bottom<double, true>)}) {
            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kBottomLdsMax);
            if (e != hipSuccess) return e;
        }
        attr_set = true;
    }
    dim3 grid(nitems), block(kBottomThreads);
    if (gen)
        hipLaunchKernelGGL((k_bottom<double, true>), grid, block, lds_bytes, s, items, nitems, lds_bytes);
    else if (dbl)
        hipLaunchKernelGGL((k_bottom<double, false>), grid, block, lds_bytes, s, items, nitems, lds_bytes);
    else
        hipLaunchKernelGGL((k_bottom<float, false>), grid, block, lds_bytes, s, items, nitems, lds_bytes);
    return hipGetLastError();
}

} // namespace mhs
