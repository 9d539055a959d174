// Two complete red-black Gauss-Seidel sweeps of a 3D level in one pass over
// memory.
#include "device.h"

// Products and sums are contracted within an expression only: a value that an
// update stored and another one reads is rounded in between, as in memory.
#pragma clang fp contract(on)

namespace mhs {
namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// NW words of 32 bits from / to a plane; an offset at or past the plane's end
// reads zeros and drops the store.
template <int NWORD>
__device__ __forceinline__ void bload_words(uint32_t (&w)[NWORD], __amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff)
{
    static_assert(NWORD >= 1 && NWORD <= 4, "at most 16 bytes per load");
    if constexpr (NWORD == 1) {
        w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0);
    } else if constexpr (NWORD == 2) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0);
        w[0] = v.x, w[1] = v.y;
    } else if constexpr (NWORD == 3) {
        const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(r, off, soff, 0);
        w[0] = v.x, w[1] = v.y, w[2] = v.z;
    } else {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0);
        w[0] = v.x, w[1] = v.y, w[2] = v.z, w[3] = v.w;
    }
}
template <int N>
__device__ __forceinline__ void bload_vec(float (&x)[N], __amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff)
{
    uint32_t w[N];
    bload_words<N>(w, r, off, soff);
#pragma unroll
    for (int q = 0; q < N; ++q) x[q] = __builtin_bit_cast(float, w[q]);
}
template <int N>
__device__ __forceinline__ void bload_vec(double (&x)[N], __amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff)
{
    uint32_t w[2 * N];
    bload_words<2 * N>(w, r, off, soff);
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const u32x2 v = {w[2 * q], w[2 * q + 1]};
        x[q] = __builtin_bit_cast(double, v);
    }
}
__device__ __forceinline__ void bstore_vec(const float (&x)[4], __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    const u32x4 v = {__builtin_bit_cast(uint32_t, x[0]), __builtin_bit_cast(uint32_t, x[1]),
                     __builtin_bit_cast(uint32_t, x[2]), __builtin_bit_cast(uint32_t, x[3])};
    __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, 0);
}
__device__ __forceinline__ void bstore_vec(const float (&x)[2], __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    const u32x2 v = {__builtin_bit_cast(uint32_t, x[0]), __builtin_bit_cast(uint32_t, x[1])};
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 0);
}
__device__ __forceinline__ void bstore_vec(const double (&x)[2], __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    const u32x2 a = __builtin_bit_cast(u32x2, x[0]), b = __builtin_bit_cast(u32x2, x[1]);
    const u32x4 v = {a.x, a.y, b.x, b.y};
    __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, 0);
}

// A lane's values of a published row, in one LDS access of 8 bytes (two of 4
// bytes at a stride of 8 would each meet every other bank only).
typedef float f32x2 __attribute__((ext_vector_type(2), may_alias));
template <int N, typename T>
__device__ __forceinline__ void lds_get(T (&x)[N], const T *p)
{
    static_assert(N * sizeof(T) == 8, "one access of 8 bytes");
    if constexpr (N == 2) {
        const f32x2 v = *(const f32x2 *)p;
        x[0] = v.x, x[1] = v.y;
    } else {
        x[0] = p[0];
    }
}
template <int N, typename T>
__device__ __forceinline__ void lds_put(T *p, const T (&x)[N])
{
    static_assert(N * sizeof(T) == 8, "one access of 8 bytes");
    if constexpr (N == 2)
        *(f32x2 *)p = f32x2{x[0], x[1]};
    else
        p[0] = x[0];
}

// The value of the lane below / above, 0 past the ends of a wave or (ROW) of
// its rows of 16 lanes.
template <bool ROW>
__device__ __forceinline__ uint32_t dpp_below(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW ? 0x111 /* row_shr:1 */ : 0x138 /* wave_shr:1 */, 0xf,
                                                 0xf, true);
}
template <bool ROW>
__device__ __forceinline__ uint32_t dpp_above(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW ? 0x101 /* row_shl:1 */ : 0x130 /* wave_shl:1 */, 0xf,
                                                 0xf, true);
}
template <bool ROW>
__device__ __forceinline__ float lane_below(float v)
{
    return __builtin_bit_cast(float, dpp_below<ROW>(__builtin_bit_cast(uint32_t, v)));
}
template <bool ROW>
__device__ __forceinline__ float lane_above(float v)
{
    return __builtin_bit_cast(float, dpp_above<ROW>(__builtin_bit_cast(uint32_t, v)));
}
template <bool ROW>
__device__ __forceinline__ double lane_below(double v)
{
    u32x2 w = __builtin_bit_cast(u32x2, v);
    w.x = dpp_below<ROW>(w.x), w.y = dpp_below<ROW>(w.y);
    return __builtin_bit_cast(double, w);
}
template <bool ROW>
__device__ __forceinline__ double lane_above(double v)
{
    u32x2 w = __builtin_bit_cast(u32x2, v);
    w.x = dpp_above<ROW>(w.x), w.y = dpp_above<ROW>(w.y);
    return __builtin_bit_cast(double, w);
}

// ============================================================================
// Two red-black sweeps, ping-pong (u_in -> u_out), columns in registers.
//
// A thread owns V consecutive x nodes of two consecutive rows and marches up
// in z with the last planes of its columns in registers.  A wave covers
// 64 / LX pairs of rows of LX * V nodes (LX = 2^lgx lanes per row), a
// workgroup a window of NW * 64 / LX row pairs.  At step s it updates the red
// nodes of plane s, the black nodes of plane s-1 (first sweep), the red
// nodes of plane s-2 and the black nodes of plane s-3 (second sweep), then
// writes plane s-3.  The z neighbours of an update are the thread's own
// registers, its x neighbours its own or the next lane's (a lane shift), and
// of its y neighbours one is its own other row: only the outer y neighbour
// comes through LDS.  Every in-plane neighbour an update of step s reads was
// final after step s-1 (the red nodes of plane s-1 for the black ones, and so
// on; the z neighbour updated in the same step is the thread's own), so one
// barrier per step suffices for the four updates, whose LDS reads are all
// issued at its start; the published rows are double-buffered.
//
// A window not at the edge of the array is right only from its fourth node
// inwards (each of the four updates moves one node in), so windows overlap by
// eight nodes and write the part in between; at the edges of the array the
// boundary nodes are fixed and nothing is lost.  A window at the right edge
// ends at the last interior node: the boundary node lies one past it and
// reads as zero (corrections vanish on the boundary), by the zero that a lane
// shift brings in past the wave's end, by the next row's first node, which is
// one too (LX = 2^lgx lanes, a single window of 2^lgx * V + 1 nodes with it),
// or by the zero past a row of 16 lanes (ROW).  ROW takes any number of
// windows in x: nearly square windows have a shorter rim, a plane of 513^2
// in windows of 64 by 64 nodes (FP32, eight waves) computes 1.27 times its
// nodes, in windows of 256 by 24 (twelve waves) 2.25 times.  513 x 513 x 257 in
// FP32 with the correction 191 us, in the longest rows 235; with the restriction
// (64 by 96) 226 against 350; 257^3 with the restriction (64 by 64) 52 against
// 65, without it longer rows are as fast.
// In z a march starts three planes below the planes it writes and ends three
// above.
//
// Old red values are never read (a Gauss-Seidel update does not use its own
// old value), so the prolongation is interpolated at the black nodes only.
//
// Each value is computed by the same expression as in one sweep at a time
// (k_sweep3), so the results are those of two launches of that kernel.
//
// Why: one sweep moves 12-12.5 bytes per node in FP32 and two launches twice
// that; here a pair moves them once, and the registers carry what the LDS
// windows of k_sweep3 carried (per node and sweep 1 LDS read and 1 write
// instead of 7 and 2, one barrier per plane for both sweeps instead of four).
// Measured on the two post-smoothing sweeps of a 257^3 level in FP32: 46
// against 95 us for one request, 581 against 1072 us for twelve merged; twelve
// 257^3 equilibria served together take 26.1 against 46.1 ms with all that is
// described here.  Merged it is bound by memory (1.09 times the compulsory
// bytes at the rate of a copy), alone by its instructions and the planes that
// short chunks read again.
//
// Level 0 of the FP64 path has no right-hand side but Dirichlet data on its
// boundary nodes: those keep their values, and where the side faces carry data
// (ext = 2) the last window of a row or column reaches past the boundary node
// instead of ending before it.  The first pair of a cycle also sums the
// residual of its input.  257^3 in FP64, 9 cycles and the fields: 4.46 ms,
// against 5.22 with single sweeps there (3.73 with the later steps).
//
// kPairRestrict: the launch that ends a level's pre-smoothing also restricts
// its residual (full weighting, as k_restrict3, whose expressions and order of
// sums it keeps: the coarse right-hand sides are the same bits).  At step s the
// residual of plane s-4 is taken from the registers, its outer y neighbours
// from the published rows; a thread has one coarse row, whose lower fine row
// another thread weights in x and publishes.  A coarse node reaches two nodes
// further than a smoothed one, so windows overlap by twelve nodes and a march
// is five steps longer.  It saves reading u and f again (8 of 20.5 bytes per
// node in FP32) and a launch per level: level 0 of 513 x 513 x 257 mixed 198 +
// 149 -> 226 us, of 257^3 46 + 35 -> 57 us, its 65^3 level 6.9 + 6.4 -> 12.7;
// 257^3 mixed in all 3.28 -> 3.06 ms.  With the restriction among the updates
// twelve waves spill, so there it comes after them.
// ============================================================================
template <typename T, int V, int R, int NW, int D, bool ROW, int FLAGS>
__global__ __launch_bounds__(64 * NW) void k_pair3(const LevelItem *__restrict__ items, int nitems)
{
    constexpr bool HAS_F = (FLAGS & kHasF) != 0;
    constexpr bool ZERO_IN = (FLAGS & kZeroIn) != 0;
    constexpr bool PROLONG = (FLAGS & kProlong) != 0;
    constexpr bool KEEPZ = (FLAGS & kPairKeepZ) != 0;
    constexpr bool NORM = (FLAGS & kNorm) != 0;
    // without a right-hand side the boundary nodes carry data (level 0 of the
    // FP64 path) and keep their values; with one they are zero
    constexpr bool DATA = !HAS_F || (FLAGS & kPairEdge) != 0;
    // the general operator: a diagonal of its own at every node
    constexpr bool GEN = (FLAGS & kPairGen) != 0;
    constexpr bool KEEP = DATA || GEN; // nodes that are not updated keep their values
    // the residual of the result, restricted to the coarse right-hand side
    constexpr bool REST = (FLAGS & kPairRestrict) != 0;
    static_assert(!REST || !(KEEP || NORM || PROLONG), "the last pre-smoothing sweeps of a correction");
    constexpr int OV = REST ? kPairOverRest : kPairOver; // nodes that windows overlap by
    static_assert(!DATA || V == 2, "the right edge of a window with data is masked per node of a pair");
    static_assert(!NORM || DATA, "the norm is taken on level 0");
    constexpr int H = V / 2;
    constexpr int RC = R / 2 + 1; // coarse rows under a thread's rows
    constexpr int NS = 5 + D; // register slots: planes s-3 .. s+1+D
    static_assert(NS % 2 == 0, "a round of NS steps keeps the plane's parity");
    constexpr uint32_t es = sizeof(T);
    // published rows: one colour of every row of the window (V/2 values per
    // lane and row), a row of zeros below and above it; four sets (old black
    // of plane s+1, red of s, black of s-1, red of s-2), two buffers
    // (with the norm a fifth: old red of plane s+1)
    // (with the restriction a fifth: black of plane s-3)
    constexpr int kSets = NORM || REST ? 5 : 4;
    constexpr int kSet = (128 * NW + 128) * H;
    // and the residual of the row above each coarse row, for the thread above
    constexpr int kSetC = REST ? (64 * NW + 64) * H : 0;
    static_assert(R == 2, "a thread has one coarse row");
    __shared__ __attribute__((aligned(16))) T S[2 * kSets * kSet + 2 * kSetC];
    __shared__ double red[NW];

    const int tile = launch_tile(items, nitems);
    const LevelItem *it = items + find_item(items, nitems, tile);
    if (it->state && gin<SolveState>(it->state)->done) return;
    const MHS_GLOBAL T *__restrict__ uin = gin<T>(it->u_in);
    MHS_GLOBAL T *__restrict__ uout = gout<T>(it->u_out);
    const MHS_GLOBAL T *__restrict__ fin = gin<T>(it->f);
    const MHS_GLOBAL T *__restrict__ ec = gin<T>(it->ec);
    const MHS_GLOBAL T *__restrict__ bin = gin<T>(it->beta);
    MHS_GLOBAL T *__restrict__ fco = gout<T>(const_cast<void *>(it->ec));
    const MHS_CONST T *__restrict__ coef = gconst<T>(it->coef);
    const T cz = (T)it->cz;
    const int nx = it->nx, ny = it->ny, nz = it->nz;
    const int ncx = it->ncx, ncy = it->ncy, ncz = it->ncz;
    const int kz = it->kz, lgx = ROW ? 4 : it->lgx;
    const int LX = 1 << lgx, WX = LX * V, WY = R * NW * (64 >> lgx);
    int local = tile - it->tile_base;
    const int tx = local % it->ntx;
    local /= it->ntx;
    const int ty = local % it->nty;
    const int tz = local / it->nty;
    const bool lastx = tx == it->ntx - 1, lasty = ty == it->nty - 1;
    const int ext = DATA ? it->ext : 0;
    const int iw = lastx ? max(nx - 1 + ext - WX, 0) : tx * (WX - OV); // window origin (even)
    const int jw = lasty ? max(ny - 1 + ext - WY, 0) : ty * (WY - OV);
    const int xs = tx ? tx * (WX - OV) + 4 : 0, xe = lastx ? nx - 1 : (tx + 1) * (WX - OV) + 4; // nodes written
    const int ys = ty ? ty * (WY - OV) + 4 : 0, ye = lasty ? ny - 1 : (ty + 1) * (WY - OV) + 4;
    const int kb = 1 + tz * kz;
    const int ke = min(kb + kz, nz - 1);
    const size_t sxy = (size_t)nx * ny, csxy = (size_t)ncx * ncy;
    const uint32_t plane_bytes = es * (uint32_t)sxy, cplane_bytes = es * (uint32_t)csxy;
    const int tid = threadIdx.x, lane = tid & 63, lx = lane & (LX - 1);
    const int t = ((tid >> 6) << (6 - lgx)) + (lane >> lgx); // row pair
    const int i0 = iw + V * lx, j0 = jw + R * t;

    // ---- per-thread geometry, the same on every plane ------------------------
    // byte offset of the thread's first row in a plane (a row past the array
    // lies past the plane's end: it reads as zero), rows are row_bytes apart
    const uint32_t row_bytes = es * (uint32_t)nx, crow_bytes = es * (uint32_t)ncx;
    const uint32_t og = es * (uint32_t)(i0 + nx * j0);
    bool upd[R][2]; // [row][0: node 0 of the lane, 1: the others] interior
    bool wr[R];     // row written
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = j0 + r;
        const bool row = j >= 1 && j <= ny - 2;
        upd[r][1] = row && (!DATA || i0 < nx - 2);
        upd[r][0] = row && i0 > 0 && (!DATA || i0 < nx - 1);
        wr[r] = row && i0 >= xs && i0 < xe && j >= ys && j < ye;
    }
    // published rows: the row below the thread's, its first and last, the row
    // above them, at a0 + 0 .. 3 times the row's length
    const int LH = LX * H;
    const int a0 = 2 * t * LH + lx * H;
    const int c0_ = t * LH + lx * H;
    // coarse rows from j0/2, columns i0/2 .. i0/2 + V/2
    const uint32_t cg = es * (uint32_t)((i0 >> 1) + ncx * (j0 >> 1));
    // the rows past the window's ends stay zero
    for (int e = tid; e < 2 * kSets * LX * H; e += 64 * NW) {
        const int set = e / (LX * H), q = e - set * (LX * H);
        S[set * kSet + q] = (T)0;
        S[set * kSet + (2 * NW * (64 >> lgx) + 1) * LX * H + q] = (T)0;
    }

    // coarse nodes written (2 I, 2 J): two nodes further in
    uint32_t rog[H];
    if constexpr (REST) {
        const int cxs = tx ? xs + 2 : 2, cxe = lastx ? nx - 1 : xe + 2;
        const int cys = ty ? ys + 2 : 2, cye = lasty ? ny - 1 : ye + 2;
#pragma unroll
        for (int m = 0; m < H; ++m) {
            const int i = i0 + 2 * m;
            rog[m] = i >= cxs && i < cxe && j0 >= cys && j0 < cye ? es * (uint32_t)((i >> 1) + ncx * (j0 >> 1))
                                                                  : cplane_bytes;
        }
    }

    // cx, cy, 1/d of 64 planes from s0-4
    const int s0 = max(kb - (REST ? 4 : 3), 0) & ~1;
    // (the general operator's are the same on every plane)
    PlaneTab<T> tcx, tcy, tid_, tdd;
    T gcx = (T)0, gcy = (T)0, gdd = (T)0;
    if constexpr (GEN) {
        gcx = coef[0];
        gcy = coef[1];
        gdd = coef[2];
    }
    // planes b .. b + 63
    auto table = [&](int b) {
        if constexpr (!GEN) {
            tcx.load(coef, b, 0, nz);
            tcy.load(coef, b, 1, nz);
            tid_.load(coef, b, 3, nz);
            if constexpr (NORM || REST) tdd.load(coef, b, 2, nz);
        }
    };
    table(s0 - 4);

    T u[NS][R][V], f[NS][R][V], be[GEN ? NS : 1][R][V];
    T dr[R][H]; // red nodes of plane s-4
    // restriction: black nodes of plane s-4, both colours of plane s-5; the
    // residuals of plane s-5 weighted in x (row 0 and 1); the coarse row's sum
    // over the planes below it
    T db[R][H], dbb[R][H], drr[R][H], rx[R][H], sum[H];
    // prolongation: coarse rows interpolated to the thread's two rows, of the
    // coarse plane below and above; the next coarse plane in flight
    T ya[R][H + 1], yb[R][H + 1], raw[RC][H + 1];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int h = 0; h < H; ++h) dr[r][h] = db[r][h] = dbb[r][h] = drr[r][h] = rx[r][h] = sum[h] = (T)0;
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
            for (int v = 0; v < V; ++v) u[q][r][v] = f[q][r][v] = be[GEN ? q : 0][r][v] = (T)0;
#pragma unroll
        for (int h = 0; h <= H; ++h) ya[r][h] = yb[r][h] = raw[r / 2][h] = raw[RC - 1][h] = (T)0;
    }

    auto fetch_u = [&](int p, T(&dst)[R][V]) {
        if constexpr (!ZERO_IN) {
            const auto rs = plane_rsrc(uin + sxy * (size_t)min(max(p, 0), nz - 1), plane_bytes);
#pragma unroll
            for (int r = 0; r < R; ++r) bload_vec<V>(dst[r], rs, og, r * row_bytes);
        }
    };
    auto fetch_f = [&](int p, T(&dst)[R][V]) {
        if constexpr (HAS_F) {
            const auto rs = plane_rsrc(fin + sxy * (size_t)min(max(p, 0), nz - 1), plane_bytes);
#pragma unroll
            for (int r = 0; r < R; ++r) bload_vec<V>(dst[r], rs, og, r * row_bytes);
        }
    };
    auto fetch_b = [&](int p, T(&dst)[R][V]) {
        if constexpr (GEN) {
            const auto rs = plane_rsrc(bin + sxy * (size_t)min(max(p, 0), nz - 1), plane_bytes);
#pragma unroll
            for (int r = 0; r < R; ++r) bload_vec<V>(dst[r], rs, og, r * row_bytes);
        }
    };
    auto fetch_c = [&](int P) {
        if constexpr (PROLONG) {
            const auto rs = plane_rsrc(ec + csxy * (size_t)min(max(P, 0), ncz - 1), cplane_bytes);
#pragma unroll
            for (int r = 0; r < RC; ++r) bload_vec<H + 1>(raw[r], rs, cg, r * crow_bytes);
        }
    };
    // yb becomes the in-flight coarse plane, interpolated in y
    auto take_c = [&]() {
        if constexpr (PROLONG) {
#pragma unroll
            for (int h = 0; h <= H; ++h) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    ya[r][h] = yb[r][h];
                    yb[r][h] = (r & 1) ? (T)0.5 * (raw[r / 2][h] + raw[r / 2 + 1][h]) : raw[r / 2][h];
                }
            }
        }
    };
    // u += I(ec) at the black nodes of a plane of parity par (boundary nodes
    // get the interpolation of the coarse boundary, zero)
    auto correct = [&](int par, T(&up)[R][V]) {
        if constexpr (PROLONG) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int v0 = (r + par + 1) & 1;
                auto z = [&](int h) -> T {
                    if (KEEPZ || !par) return yb[r][h];
                    return (T)0.5 * (ya[r][h] + yb[r][h]);
                };
#pragma unroll
                for (int m = 0; m < H; ++m) {
                    const int v = v0 + 2 * m;
                    const T c = v0 ? (T)0.5 * (z(m) + z(m + 1)) : z(m);
                    up[r][v] += c;
                }
            }
        }
    };
    // a selected, not branched to (the compiler would branch around the update)
    auto keep_or = [](bool c, T a, T old) -> T {
        asm volatile("" : "+v"(a));
        return c ? a : old;
    };
    // 1/d of plane p (GEN: the Laplacian's diagonal, which the node's b/a adds
    // to), 0 on the boundary planes: a node that is not updated is a
    // boundary node, whose value (zero) comes out of the update as zero when
    // its 1/d is zero
    struct Coef {
        T cx, cy, inv;
    };
    auto coef_of = [&](int p) {
        if constexpr (GEN) {
            return Coef{gcx, gcy, gdd};
        } else {
            const T cx = tcx(p), cy = tcy(p), inv = tid_(p);
            return Coef{cx, cy, p >= 1 && p <= nz - 2 ? inv : (T)0};
        }
    };
    Coef q[NS]; // of the planes in the slots
#pragma unroll
    for (int e = 0; e < NS; ++e) q[e] = Coef{(T)0, (T)0, (T)0};
    // the outer y neighbours (row below the thread's first, above its last) of
    // one colour
    struct Rows {
        T below[H], above[H];
    };
    auto outer = [&](const T *below, const T *above) {
        Rows y;
        lds_get<H>(y.below, below);
        lds_get<H>(y.above, above);
        return y;
    };
    // one colour (0 red, 1 black) of plane p: k its coefficients, uc its columns, uu and ud those
    // above and below, S rows at rd; par the plane's parity.  What the second
    // sweep (last) leaves in column 0 is stored with the row: it has to be zero
    // also where a neighbour has overflowed and the product with 1/d = 0 is a
    // NaN, for single sweeps read that column, which they do not write, in a
    // later solve.  (Selects at every node and in both sweeps: 33^3 mixed 1 %
    // slower.  In both sweeps at column 0 in FP64 with the restriction, whose
    // registers then suffice: up to 88 spilled with one.)
    constexpr bool kSelectBoth = sizeof(T) == 8 && REST && !ZERO_IN;
    auto colour = [&](int p, const Coef &k, int par, int col, T(&uc)[R][V], const T(&uu)[R][V], const T(&dn)[R][V], const T(&fp)[R][V],
                      const T(&bp)[R][V], const Rows &y, auto last) {
        const T cx = k.cx, cy = k.cy, invd = k.inv;
        const bool in = p >= 1 && p <= nz - 2;
        constexpr bool SELECT = decltype(last)::value || kSelectBoth;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int v0 = (r + par + col) & 1;
            const bool in1 = upd[r][1] && in, in0 = upd[r][0] && in;
            const T inv1 = KEEP ? invd : upd[r][1] ? invd : (T)0, inv0 = KEEP || SELECT || v0 ? inv1 : upd[r][0] ? invd : (T)0;
#pragma unroll
            for (int m = 0; m < H; ++m) {
                const int v = v0 + 2 * m;
                const T e = v + 1 < V ? uc[r][(v + 1) % V] : lane_above<ROW>(uc[r][0]);
                const T w = v > 0 ? uc[r][(v + V - 1) % V] : lane_below<ROW>(uc[r][V - 1]);
                const T yn = r + 1 < R ? uc[(r + 1) % R][v] : y.above[m];
                const T ys_ = r > 0 ? uc[(r + R - 1) % R][v] : y.below[m];
                const T fv = HAS_F ? fp[r][v] : (T)0;
                const T n = fv - (cx * (e + w) + cy * (yn + ys_) + cz * (uu[r][v] + dn[r][v]));
                const T a = GEN ? n / (bp[r][v] + invd) : n * (v ? inv1 : inv0);
                if constexpr (KEEP)
                    uc[r][v] = keep_or(v ? in1 : in0, a, uc[r][v]);
                else
                    uc[r][v] = SELECT && !v ? keep_or(upd[r][0], a, (T)0) : a;
            }
        }
    };
    // residual of the input iterate at plane p (all values still old; old red
    // of the plane below in ro), its outer neighbours yb (black) and yr (red)
    double acc = 0.0;
    T ro[R][H];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int h = 0; h < H; ++h) ro[r][h] = (T)0;
    auto residual = [&](int p, int par, const T(&uc)[R][V], const T(&uu)[R][V], const T(&dn)[R][V], const T(&fp)[R][V],
                        const T(&bp)[R][V], const Rows &yb_, const Rows &yr) {
        if constexpr (NORM) {
            const T cx = GEN ? gcx : tcx(p), cy = GEN ? gcy : tcy(p), dd = GEN ? gdd : tdd(p);
            const bool in = p >= kb && p < ke;
#pragma unroll
            for (int col = 0; col < 2; ++col) {
                const Rows &y = col ? yr : yb_;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int v0 = (r + par + col) & 1;
#pragma unroll
                    for (int m = 0; m < H; ++m) {
                        const int v = v0 + 2 * m;
                        const T e = v + 1 < V ? uc[r][(v + 1) % V] : lane_above<ROW>(uc[r][0]);
                        const T w = v > 0 ? uc[r][(v + V - 1) % V] : lane_below<ROW>(uc[r][V - 1]);
                        const T yn = r + 1 < R ? uc[(r + 1) % R][v] : y.above[m];
                        const T ys_ = r > 0 ? uc[(r + R - 1) % R][v] : y.below[m];
                        const T d_ = col ? ro[r][m] : dn[r][v];
                        const T dv = GEN ? bp[r][v] + dd : dd;
                        T rv = cx * (e + w) + cy * (yn + ys_) + cz * (uu[r][v] + d_) + dv * uc[r][v];
                        if constexpr (HAS_F) rv = fp[r][v] - rv;
                        const double z = in && wr[r] && upd[r][v ? 1 : 0] ? (double)rv : 0.0;
                        acc += z * z;
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int m = 0; m < H; ++m) ro[r][m] = uc[r][((r + par) & 1) + 2 * m];
        }
    };
    auto publish = [&](int par, int col, const T(&uc)[R][V], T *first, T *last) {
#pragma unroll
        for (int r = 0; r < R; r += R - 1) {
            const int v0 = (r + par + col) & 1;
            T x[H];
#pragma unroll
            for (int m = 0; m < H; ++m) x[m] = uc[r][v0 + 2 * m];
            lds_put<H>(r ? last : first, x);
        }
    };

    Rows y3p{}; // restriction: y3 of the step before
    // the general operator's divisions leave no registers for overlapping the
    // updates
    auto calm = [] {
        if constexpr ((GEN && (PROLONG || NORM)) || (REST && D == 1 && !ZERO_IN)) __builtin_amdgcn_sched_barrier(0);
    };
    // one step at plane s; d: its position in the round of NS steps (s0 is
    // even, so the plane's parity is d's).  Plane s + e lives in slot
    // (d + e + 3) % NS.
    auto step = [&](const int s, auto dc) {
        constexpr int d = decltype(dc)::value;
        constexpr int P = d & 1, Q = P ^ 1;
        constexpr int cm3 = d % NS, cm2 = (d + 1) % NS, cm1 = (d + 2) % NS, c0 = (d + 3) % NS, cp1 = (d + 4) % NS;
        constexpr int cnx = (d + 4 + D) % NS, cnf = (d + 3 + D) % NS;
        // (the offsets of the two buffers stay in scalar registers: folded
        // into the addresses they would take a vector register each)
        int so = Q * kSets * kSet, wo = P * kSets * kSet;
        asm volatile("" : "+s"(so), "+s"(wo));
        const T *rb = S + (a0 + so), *ra = S + (a0 + (so + 3 * LH));
        T *w0 = S + (a0 + (wo + LH)), *w1 = S + (a0 + (wo + 2 * LH));
        T rbelow[H] = {}; // residuals of plane s-5 in the row below, weighted in x
        Rows yr{};        // black nodes of plane s-4
        auto read_rest = [&] {
            if constexpr (REST) {
                int sc = 2 * kSets * kSet + Q * kSetC;
                asm volatile("" : "+s"(sc));
                lds_get<H>(rbelow, S + (c0_ + sc));
                yr = outer(rb + 4 * kSet, ra + 4 * kSet);
            }
        };
        fetch_u(s + 1 + D, u[cnx]);
        fetch_f(s + D, f[cnf]);
        fetch_b(s + D, be[GEN ? cnf : 0]);
        __builtin_amdgcn_sched_barrier(0); // issued before the step's arithmetic
        // plane s+1 gets its correction (coarse plane (s+2)/2 or, on a step
        // that keeps z, s+1)
        if constexpr (PROLONG) {
            if (KEEPZ || Q) {
                take_c();
                fetch_c(KEEPZ ? s + 2 : (s + 4) >> 1);
            }
            correct(Q, u[cp1]);
        }
        Rows y0{};
        if constexpr (!ZERO_IN) y0 = outer(rb, ra);
        // read at the step's start, or (calm) when the update needs them
        // twelve waves: the restriction after the updates, not among them
        constexpr bool CALM = REST && D == 1 && !ZERO_IN;
        constexpr bool LATE = (GEN && (PROLONG || NORM)) || CALM;
        Rows y1, y2, y3;
        if constexpr (!LATE) {
            y1 = outer(rb + kSet, ra + kSet);
            y2 = outer(rb + 2 * kSet, ra + 2 * kSet);
            y3 = outer(rb + 3 * kSet, ra + 3 * kSet);
            read_rest();
        }
        q[c0] = coef_of(s);
        if constexpr (NORM) residual(s, P, u[c0], u[cp1], u[cm1], f[c0], be[GEN ? c0 : 0], y0, outer(rb + 4 * kSet, ra + 4 * kSet));
        calm();
        // first sweep
        if constexpr (ZERO_IN) {
            const T invd = q[c0].inv;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int v0 = (r + P) & 1;
                const bool in = s >= 1 && s <= nz - 2;
                const T inv1 = upd[r][1] ? invd : (T)0, inv0 = v0 ? inv1 : upd[r][0] ? invd : (T)0;
#pragma unroll
                for (int m = 0; m < H; ++m) {
                    const int v = v0 + 2 * m;
                    if constexpr (GEN)
                        u[c0][r][v] = keep_or(upd[r][v ? 1 : 0] && in, f[c0][r][v] / (be[c0][r][v] + invd), (T)0);
                    else
                        u[c0][r][v] = f[c0][r][v] * (v ? inv1 : inv0);
                    // slots are reused: the plane's other nodes start from zero
                    u[c0][r][v ^ 1] = (T)0;
                }
            }
        } else {
            colour(s, q[c0], P, 0, u[c0], u[cp1], u[cm1], f[c0], be[GEN ? c0 : 0], y0, std::false_type{});
        }
        calm();
        if constexpr (LATE) y1 = outer(rb + kSet, ra + kSet);
        colour(s - 1, q[cm1], Q, 1, u[cm1], u[c0], u[cm2], f[cm1], be[GEN ? cm1 : 0], y1, std::false_type{});
        // second sweep
        calm();
        if constexpr (LATE) y2 = outer(rb + 2 * kSet, ra + 2 * kSet);
        colour(s - 2, q[cm2], P, 0, u[cm2], u[cm1], u[cm3], f[cm2], be[GEN ? cm2 : 0], y2, std::true_type{});
        {
            // below plane s-3 only its red nodes are needed, kept in dr
            T dn[R][V];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int m = 0; m < H; ++m) {
                    // red of plane s-4 (parity P) sits above / below the
                    // black nodes of plane s-3 (parity Q): the same columns
                    const int v = ((r + P) & 1) + 2 * m;
                    dn[r][v] = dr[r][m];
                    dn[r][v ^ 1] = (T)0;
                }
            calm();
            if constexpr (LATE) y3 = outer(rb + 3 * kSet, ra + 3 * kSet);
            colour(s - 3, q[cm3], Q, 1, u[cm3], u[cm2], dn, f[cm3], be[GEN ? cm3 : 0], y3, std::true_type{});
            if constexpr (CALM) {
                __builtin_amdgcn_sched_barrier(0);
                read_rest();
            }
            if constexpr (REST) {
                // full weighting: the plane s-5, complete with the row below
                const T q4 = (T)0.25, h2 = (T)0.5;
                T s2[H];
#pragma unroll
                for (int m = 0; m < H; ++m) s2[m] = q4 * rbelow[m] + h2 * rx[0][m] + q4 * rx[1][m];
                const int pc = KEEPZ ? s - 5 : s - 6; // fine plane of the coarse one
                if constexpr (KEEPZ || P == 0) {
                    const auto rs = plane_rsrc(fco + csxy * (size_t)max(KEEPZ ? pc : pc >> 1, 0),
                                               pc >= kb && pc < ke ? cplane_bytes : 0u);
#pragma unroll
                    for (int m = 0; m < H; ++m) bstore(KEEPZ ? s2[m] : sum[m] + q4 * s2[m], rs, rog[m]);
                }
#pragma unroll
                for (int m = 0; m < H; ++m) sum[m] = P == 0 ? q4 * s2[m] : sum[m] + h2 * s2[m];
                // residual of plane s-4
                const T cx = q[cnx].cx, cy = q[cnx].cy, dd = tdd(s - 4);
                auto at = [&](int r, int v) -> T { return (r + P + v) & 1 ? db[r][v >> 1] : dr[r][v >> 1]; };
                T rv[R][V];
#pragma unroll
                for (int r = 0; r < R; ++r) {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        const bool black = (r + P + v) & 1;
                        const T e = v + 1 < V ? at(r, (v + 1) % V) : lane_above<ROW>(at(r, 0));
                        const T w = v > 0 ? at(r, (v + V - 1) % V) : lane_below<ROW>(at(r, V - 1));
                        const Rows &y = black ? y3p : yr;
                        const T yn = r + 1 < R ? at((r + 1) % R, v) : y.above[v >> 1];
                        const T ys_ = r > 0 ? at((r + R - 1) % R, v) : y.below[v >> 1];
                        const T dn = black ? drr[r][v >> 1] : dbb[r][v >> 1];
                        rv[r][v] = f[cnx][r][v] - (cx * (e + w) + cy * (yn + ys_) + cz * (u[cm3][r][v] + dn) +
                                                   dd * at(r, v));
                    }
#pragma unroll
                    for (int m = 0; m < H; ++m) {
                        const T w = m > 0 ? rv[r][(2 * m + V - 1) % V] : lane_below<ROW>(rv[r][V - 1]);
                        rx[r][m] = q4 * w + h2 * rv[r][2 * m] + q4 * rv[r][2 * m + 1];
                    }
                }
                y3p = y3;
                int sc = 2 * kSets * kSet + P * kSetC;
                asm volatile("" : "+s"(sc));
                lds_put<H>(S + (c0_ + (sc + LH)), rx[1]);
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int m = 0; m < H; ++m) {
                        drr[r][m] = dr[r][m];
                        dbb[r][m] = db[r][m];
                        db[r][m] = u[cm3][r][((r + Q + 1) & 1) + 2 * m];
                    }
                publish(Q, 1, u[cm3], w0 + 4 * kSet, w1 + 4 * kSet);
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int m = 0; m < H; ++m) dr[r][m] = u[cm3][r][((r + Q) & 1) + 2 * m];
        }
        if constexpr (!ZERO_IN) publish(Q, 1, u[cp1], w0, w1);
        if constexpr (NORM) publish(Q, 0, u[cp1], w0 + 4 * kSet, w1 + 4 * kSet);
        publish(P, 0, u[c0], w0 + kSet, w1 + kSet);
        publish(Q, 1, u[cm1], w0 + 2 * kSet, w1 + 2 * kSet);
        publish(P, 0, u[cm2], w0 + 3 * kSet, w1 + 3 * kSet);
        const int m = s - 3;
        // (outside the chunk the buffer is empty and drops the stores)
        const auto rs = plane_rsrc(uout + sxy * (size_t)max(m, 0), m >= kb && m < ke ? plane_bytes : 0u);
#pragma unroll
        for (int r = 0; r < R; ++r) bstore_vec(u[cm3][r], rs, wr[r] ? og + r * row_bytes : plane_bytes);
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0); // a step's loads stay in it
    };

    // planes s0-1 .. s0+D into their slots ((p - s0 + 3) % NS)
#pragma unroll
    for (int e = -1; e <= D; ++e) {
        fetch_u(s0 + e, u[(e + 3) % NS]);
        if (e < D) {
            fetch_f(s0 + e, f[(e + 3) % NS]);
            fetch_b(s0 + e, be[GEN ? (e + 3) % NS : 0]);
        }
    }
    if constexpr (PROLONG) {
        // coarse planes for s0-1 and s0; the one of s0+1 in flight
        if constexpr (KEEPZ) {
            fetch_c(s0 - 1);
            take_c();
            correct(1, u[2]);
            fetch_c(s0);
            take_c();
            correct(0, u[3]);
            fetch_c(s0 + 1);
        } else {
            fetch_c((s0 - 1) >> 1);
            take_c();
            fetch_c(s0 >> 1);
            take_c();
            correct(1, u[2]);
            correct(0, u[3]);
            fetch_c((s0 + 2) >> 1);
        }
    }
    // rows that the first step reads before any step has published them must
    // be finite (what it computes from them is not used, but a boundary node
    // is kept by a factor of zero)
#pragma unroll
    for (int e = kSets + 1; e < kSets + 4; ++e)
#pragma unroll
        for (int m = 0; m < H; ++m) S[e * kSet + a0 + LH + m] = S[e * kSet + a0 + 2 * LH + m] = (T)0;
    if constexpr (!ZERO_IN) publish(0, 1, u[3], S + kSets * kSet + a0 + LH, S + kSets * kSet + a0 + 2 * LH);
    if constexpr (NORM) {
        publish(0, 0, u[3], S + (kSets + 4) * kSet + a0 + LH, S + (kSets + 4) * kSet + a0 + 2 * LH);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int m = 0; m < H; ++m) ro[r][m] = u[2][r][((r + 1) & 1) + 2 * m]; // old red of plane s0-1
    }
    lds_barrier();
    // the last step writes plane ke - 1, with the restriction coarse plane
    // ke - 1 or (ke - 1) / 2
    const int send = REST ? ke + (KEEPZ ? 4 : 5) : ke + 2;
    for (int s = s0; s <= send; s += NS) {
        if constexpr (!GEN && pair_max_kz(NW, ROW) > kPairTablePlanes)
            if (s + NS - 1 > tcx.base + 63) table(s - 4); // a long march's next planes
        step(s, std::integral_constant<int, 0>{});
        step(s + 1, std::integral_constant<int, 1>{});
        if (REST && D == 3 && s + 2 > send) break;
        step(s + 2, std::integral_constant<int, 2>{});
        step(s + 3, std::integral_constant<int, 3>{});
        if (REST && D == 3 && s + 4 > send) break;
        step(s + 4, std::integral_constant<int, 4>{});
        step(s + 5, std::integral_constant<int, 5>{});
        if constexpr (NS == 8) {
            if (REST && D == 3 && s + 6 > send) break;
            step(s + 6, std::integral_constant<int, 6>{});
            step(s + 7, std::integral_constant<int, 7>{});
        }
    }
    if constexpr (NORM) {
        const double tot = block_sum<64 * NW>(acc, red);
        if (tid == 0) gout<double>(it->partials)[tile - it->tile_base] = tot;
    }
}

template <typename T, int V, int NW, int D, bool ROW>
hipError_t pair_dispatch(const LevelItem *items, int nitems, int ntiles, int flags, hipStream_t s)
{
    dim3 grid(ntiles), block(64 * NW);
#define MHS_CASE(F)                                                                           \
    case F:                                                                                   \
        hipLaunchKernelGGL((k_pair3<T, V, 2, NW, D, ROW, F>), grid, block, 0, s, items, nitems);   \
        return hipGetLastError();
    switch (flags) {
        MHS_CASE(kHasF) MHS_CASE(kHasF | kZeroIn) MHS_CASE(kHasF | kProlong) MHS_CASE(kHasF | kProlong | kPairKeepZ)
        MHS_CASE(kHasF | kPairRestrict) MHS_CASE(kHasF | kPairRestrict | kPairKeepZ)
        MHS_CASE(kHasF | kZeroIn | kPairRestrict) MHS_CASE(kHasF | kZeroIn | kPairRestrict | kPairKeepZ)
    }
    if constexpr (sizeof(T) == 8) {
        // level 0 of the FP64 path
        switch (flags) {
            MHS_CASE(0) MHS_CASE(kNorm) MHS_CASE(kProlong) MHS_CASE(kProlong | kPairKeepZ)
        }
        // the general operator
        constexpr int G = kHasF | kPairGen, G0 = G | kPairEdge;
        switch (flags) {
            MHS_CASE(G) MHS_CASE(G | kZeroIn) MHS_CASE(G0) MHS_CASE(G0 | kNorm)
        }
        if constexpr (NW <= kPairGenWaves) {
            switch (flags) {
                MHS_CASE(G | kProlong) MHS_CASE(G | kProlong | kPairKeepZ)
                MHS_CASE(G0 | kProlong) MHS_CASE(G0 | kProlong | kPairKeepZ)
            }
        }
    }
#undef MHS_CASE
    return hipErrorInvalidValue;
}

template <typename T, int V>
hipError_t pair_variant(const LevelItem *items, int nitems, int ntiles, int flags, int variant, hipStream_t s)
{
    static_assert(kPairNVariants == 6, "one case per variant");
    switch (variant) {
#define MHS_VAR(N) \
    case N: return pair_dispatch<T, V, kPairVariants[N].waves, kPairVariants[N].depth, kPairVariants[N].row>(items, nitems, ntiles, flags, s);
        MHS_VAR(0) MHS_VAR(1) MHS_VAR(2) MHS_VAR(3) MHS_VAR(4) MHS_VAR(5)
#undef MHS_VAR
    }
    return hipErrorInvalidValue;
}

} // namespace

hipError_t launch_pair3(const LevelItem *items, int nitems, int ntiles, int flags, bool dbl, int variant, hipStream_t s)
{
    if (ntiles <= 0) return hipSuccess;
    return dbl ? pair_variant<double, kPairV64>(items, nitems, ntiles, flags, variant, s)
               : pair_variant<float, kPairV32>(items, nitems, ntiles, flags, variant, s);
}

} // namespace mhs
