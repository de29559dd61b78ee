// Adjoint of the regular force (no counterpart in the paper; it differentiates
// the regular force of section 2 / section 3.2.1 with the neighbour sets held
// fixed).
//
//   L = sum_b  w_a[:,b] . acc_b + w_j[:,b] . jerk_b
//
// For a regular pair (row b with body i, source j), with A = w_a[:,b],
// B = w_j[:,b], r = x_j - x_i, u = v_j - v_i, s = r.u, R3 = |r|^-3,
// R5 = |r|^-5, R7 = |r|^-7:
//   dL/dm_j += (A.r) R3 + (B.u) R3 - 3 s (B.r) R5
//   g_r      = m_j [ A R3 - 3 R5 (s B + (B.r) u) + r (15 s (B.r) R7 - 3 R5 (A.r + B.u)) ]
//   g_u      = m_j [ B R3 - 3 (B.r) R5 r ]
//   dL/dx_j += g_r,  dL/dx_i -= g_r,  dL/dv_j += g_u,  dL/dv_i -= g_u.
//
// One recompute pass, FP64, no per-pair storage and no global atomics on
// values.  Every pair is evaluated once for its row and its body (a row pass
// and a body pass used to recompute the same geometry, about half of the 111
// FP64 instructions that the two spent on a pair): each lane holds R rows in
// registers, bodies pass through LDS in tiles of 64 or 128, and at step s lane l
// meets body l ^ s of a run of 64, so the lanes of a wave work on 64 different bodies.  The
// row's sums stay in registers; the body's seven shares of the lane's R rows
// are added in registers and then to the wave's own LDS sums, without conflict
// and in a fixed order.  Row sums per block of bodies and body sums per block
// of rows go to scratch and are added in block order, so results are bitwise
// deterministic; the "-" terms reach a body in row order.
#include <algorithm>

#include "nb_rows.h"

namespace nb {
namespace {

struct AdjPlan {
    int32_t row_block;       // rows per row block (64 R W)
    int32_t panel_row0;      // first row of this panel
    int32_t panel_rows;      // rows of this panel (its row blocks' rows below n_i)
    int32_t body_blocks;     // blocks of body_len bodies
    int64_t body_len;
    int32_t add;             // body sums of an earlier panel are added to
    double *row_partial;     // [body_blocks][6][panel_rows]
    double *body_partial;    // [row blocks of a panel][7][n]
    int2 *index;             // per body: its first row (n_i: none), 1 if it has others
};

// Exclusion (self pair or neighbour) by the canonical test, run only for
// candidates below the FP64 bound hi: an excluded pair gets the squared
// distance kExclR2, which makes every power of r^-1 from the third up exactly
// zero, so the pair loop holds no select.
__device__ __forceinline__ void exclude(double dx, double dy, double dz, double &r2, double hi,
                                        float rs2f, int32_t jidx, int32_t i)
{
    if (r2 < hi) {
        double ex = dx, ey = dy, ez = dz;
        int32_t jj = jidx;
        opaque(ex, ey, ez);
        opaque(jj);
        if (jj == i || canon_r2f(ex, ey, ez) < rs2f) r2 = kExclR2;
    }
}

// One row in registers with its sums over bodies: with k = -3 R5,
//   sum_j g_r = A C1 + B C2 + H,  sum_j g_u = B C1 + U,
//   C1 = sum m R3,  C2 = sum m k s,  U = sum m k (B.r) r,
//   H = sum m [k (B.r) u + k ((A.r + B.u) - 5 s (B.r) |r|^-2) r].
struct AdjRow {
    double x, y, z, vx, vy, vz, ax, ay, az, bx, by, bz, hi;
    float rs2f;
    int32_t i;
    double C1, C2, Hx, Hy, Hz, Ux, Uy, Uz;
    __device__ __forceinline__ void load(const AdjointArgs &a, int64_t b, int64_t end)
    {
        x = y = z = kFar * 0.5;
        vx = vy = vz = ax = ay = az = bx = by = bz = 0.0;
        hi = -1.0;
        rs2f = -1.0f;
        i = -1;
        C1 = C2 = Hx = Hy = Hz = Ux = Uy = Uz = 0.0;
        if (b >= end) return;
        const int64_t k = a.i_block[b];
        if (k < 0 || k >= a.n) return;
        i = (int32_t)k;
        x = a.xp[k];
        y = a.xp[a.n + k];
        z = a.xp[2 * a.n + k];
        vx = a.vp[k];
        vy = a.vp[a.n + k];
        vz = a.vp[2 * a.n + k];
        ax = a.w_a[b];
        ay = a.w_a[a.n_i + b];
        az = a.w_a[2 * (int64_t)a.n_i + b];
        bx = a.w_j[b];
        by = a.w_j[a.n_i + b];
        bz = a.w_j[2 * (int64_t)a.n_i + b];
        rs2f = (float)a.rs2[b];
        hi = cand_bound_f64(rs2f);
    }
};

// grid = row blocks of the panel x body blocks (row blocks fastest: running
// work-groups share bodies); T bodies staged at a time.  FP64 VALU bound at R
// = 2 (about 75 instructions per pair; the LDS is busy for half of that), LDS
// bound at R = 1.  Held to three waves per SIMD at R = 2 (168 VGPRs, no spill;
// at the compiler's 180 two fit): 65536 rows of 65536 11.15 ms against 11.53.
// The two passes before took 16.2 ms there, 1823 us on 20011 of 20011 (now
// 1150), 545 on 4096 of 4096 (75), 364 on 1024 of 1024 (35).
template <int R, int W, int T>
__global__ __launch_bounds__(kWave * W) __attribute__((amdgpu_waves_per_eu(R == 2 ? 3 : 4))) void adj_pairs_kernel(AdjointArgs a, AdjPlan p)
{
    constexpr int BR = kWave * R * W;
    // planes of 16 bytes: consecutive lanes read consecutive banks
    __shared__ double2 t_xy[T], t_zm[T], t_vxy[T];
    __shared__ double t_vz[T];
    __shared__ double sums[W][7][T];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int32_t row_blocks = (p.panel_rows + BR - 1) / BR;
    const int32_t rb = (int32_t)(blockIdx.x % row_blocks), qb = (int32_t)(blockIdx.x / row_blocks);
    const int64_t j0 = (int64_t)qb * p.body_len;
    const int64_t j1 = j0 + p.body_len < a.n ? j0 + p.body_len : a.n;
    const int64_t row0 = (int64_t)p.panel_row0 + (int64_t)rb * BR;
    const int64_t row_end = (int64_t)p.panel_row0 + p.panel_rows;

    // the bodies' row index starts empty (written by a later launch)
    if (!p.add)
        for (int64_t j = (int64_t)blockIdx.x * (kWave * W) + tid; j < a.n;
             j += (int64_t)gridDim.x * (kWave * W))
            p.index[j] = make_int2(a.n_i, 0);

    AdjRow Q[R];
#pragma unroll
    for (int r = 0; r < R; ++r) Q[r].load(a, row0 + (w * R + r) * kWave + lane, row_end);
    bool mine = false;
#pragma unroll
    for (int r = 0; r < R; ++r) mine = mine || Q[r].i >= 0;
    const bool busy = __ballot(mine) != 0;   // a wave without rows only stages and stores

    for (int64_t c0 = j0; c0 < j1; c0 += T) {
        if (c0 > j0) __syncthreads();   // the last tile's sums are read
        for (int e = tid; e < T; e += kWave * W) {
            const int64_t j = c0 + e;
            const bool live = j < j1;
            t_xy[e] = live ? make_double2(a.xp[j], a.xp[a.n + j]) : make_double2(kFar, kFar);
            t_zm[e] = live ? make_double2(a.xp[2 * a.n + j], a.m[j]) : make_double2(kFar, 0.0);
            t_vxy[e] = live ? make_double2(a.vp[j], a.vp[a.n + j]) : make_double2(0.0, 0.0);
            t_vz[e] = live ? a.vp[2 * a.n + j] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 7; ++k)
            for (int e = lane; e < T; e += kWave) sums[w][k][e] = 0.0;
        __syncthreads();
        const int live = (int)(j1 - c0 < T ? j1 - c0 : T);
        for (int t = 0; busy && t < live; t += kWave) {
#pragma unroll 1
            for (int s = 0; s < kWave; ++s) {
                const int e = t + (lane ^ s);
                const double2 xy = t_xy[e], zm = t_zm[e], vxy = t_vxy[e];
                const double vz = t_vz[e];
                double g[7] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    AdjRow &b = Q[r];
                    const double dx = xy.x - b.x, dy = xy.y - b.y, dz = zm.x - b.z;
                    double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
                    exclude(dx, dy, dz, r2, b.hi, b.rs2f, (int32_t)(c0 + e), b.i);
                    const double ux = vxy.x - b.vx, uy = vxy.y - b.vy, uz = vz - b.vz;
                    const double y = rsqrt_f64(r2);
                    const double y2 = y * y;
                    const double R3 = y * y2, k5 = -3.0 * (R3 * y2);
                    const double sv = __builtin_fma(dz, uz, __builtin_fma(dy, uy, dx * ux));
                    const double Ar = __builtin_fma(b.az, dz, __builtin_fma(b.ay, dy, b.ax * dx));
                    const double Br = __builtin_fma(b.bz, dz, __builtin_fma(b.by, dy, b.bx * dx));
                    const double Bu = __builtin_fma(b.bz, uz, __builtin_fma(b.by, uy, b.bx * ux));
                    const double AB = Ar + Bu, sBr = sv * Br;
                    const double es = k5 * sv, tb = k5 * Br;
                    const double c = k5 * __builtin_fma(-5.0 * sBr, y2, AB);
                    // the body's shares (without its mass)
                    g[0] = __builtin_fma(c, dx, __builtin_fma(tb, ux, __builtin_fma(es, b.bx, __builtin_fma(R3, b.ax, g[0]))));
                    g[1] = __builtin_fma(c, dy, __builtin_fma(tb, uy, __builtin_fma(es, b.by, __builtin_fma(R3, b.ay, g[1]))));
                    g[2] = __builtin_fma(c, dz, __builtin_fma(tb, uz, __builtin_fma(es, b.bz, __builtin_fma(R3, b.az, g[2]))));
                    g[3] = __builtin_fma(tb, dx, __builtin_fma(R3, b.bx, g[3]));
                    g[4] = __builtin_fma(tb, dy, __builtin_fma(R3, b.by, g[4]));
                    g[5] = __builtin_fma(tb, dz, __builtin_fma(R3, b.bz, g[5]));
                    g[6] = __builtin_fma(sBr, k5, __builtin_fma(AB, R3, g[6]));
                    // the row's sums
                    const double m = zm.y, mt = m * tb, mc = m * c;
                    b.C1 = __builtin_fma(m, R3, b.C1);
                    b.C2 = __builtin_fma(m, es, b.C2);
                    b.Hx = __builtin_fma(mt, ux, __builtin_fma(mc, dx, b.Hx));
                    b.Hy = __builtin_fma(mt, uy, __builtin_fma(mc, dy, b.Hy));
                    b.Hz = __builtin_fma(mt, uz, __builtin_fma(mc, dz, b.Hz));
                    b.Ux = __builtin_fma(mt, dx, b.Ux);
                    b.Uy = __builtin_fma(mt, dy, b.Uy);
                    b.Uz = __builtin_fma(mt, dz, b.Uz);
                }
#pragma unroll
                for (int k = 0; k < 7; ++k)
                    __hip_atomic_fetch_add(&sums[w][k][e], g[k], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        __syncthreads();
        double *o = p.body_partial + (int64_t)rb * 7 * a.n + c0;
        for (int e = tid; e < live * 7; e += kWave * W) {
            const int k = e / live, q = e - k * live;
            double v = 0.0;
#pragma unroll
            for (int u = 0; u < W; ++u) v += sums[u][k][q];
            double *d = o + (int64_t)k * a.n + q;
            *d = p.add ? *d + v : v;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const AdjRow &b = Q[r];
        const int64_t k = row0 + (w * R + r) * kWave + lane;
        if (k >= row_end) continue;
        const int64_t st = p.panel_rows;
        double *o = p.row_partial + (int64_t)qb * 6 * st + (k - p.panel_row0);
        o[0] = __builtin_fma(b.ax, b.C1, __builtin_fma(b.bx, b.C2, b.Hx));
        o[st] = __builtin_fma(b.ay, b.C1, __builtin_fma(b.by, b.C2, b.Hy));
        o[2 * st] = __builtin_fma(b.az, b.C1, __builtin_fma(b.bz, b.C2, b.Hz));
        o[3 * st] = __builtin_fma(b.bx, b.C1, b.Ux);
        o[4 * st] = __builtin_fma(b.by, b.C1, b.Uy);
        o[5 * st] = __builtin_fma(b.bz, b.C1, b.Uz);
    }
}

// Sums the row partials of a panel over the body blocks (fixed order) into
// row_part[6][n_i], enters the rows in their bodies' index and flags bad
// indices.  A work-group takes 64 components of rows; its waves share the body
// blocks (a lane that adds them all is a chain of memory round trips, and few
// rows are few lanes: 512 blocks of 1024 rows 123 us with one lane per
// component, 8 so).
constexpr int kReduceWaves = 16;

// Enters a row in its body's index.  A row behind one that is there already only
// sets the flag, if it is not set: where one body has many rows, their atomics and
// stores would queue on one address.
__device__ __forceinline__ void enter_row(int2 *t, int32_t row, int32_t none)
{
    const uint64_t seen = __hip_atomic_load((const uint64_t *)t, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
    if ((int32_t)seen > row && atomicMin(&t->x, row) == none) return;   // the first to come
    if (seen >> 32 == 0)
        __hip_atomic_store(&t->y, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(kWave * kReduceWaves) void adj_rows_reduce(AdjointArgs a, AdjPlan p)
{
    __shared__ double part[kReduceWaves][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t k = (int64_t)blockIdx.x * kWave + lane;
    const int64_t total = 6 * (int64_t)p.panel_rows;
    const int32_t share = (p.body_blocks + kReduceWaves - 1) / kReduceWaves;
    const int32_t q1 = p.body_blocks < (w + 1) * share ? p.body_blocks : (w + 1) * share;
    double s = 0.0;
    if (k < total)
#pragma unroll 8
        for (int32_t q = w * share; q < q1; ++q) s += p.row_partial[(int64_t)q * total + k];
    part[w][lane] = s;
    __syncthreads();
    if (w > 0) return;
    bool bad = false;
    if (k < total) {
        s = 0.0;
#pragma unroll
        for (int u = 0; u < kReduceWaves; ++u) s += part[u][lane];
        const int64_t comp = k / p.panel_rows, row = k - comp * p.panel_rows + p.panel_row0;
        a.row_part[comp * a.n_i + row] = s;
        if (comp == 0) {
            const int64_t i = a.i_block[row];
            bad = i < 0 || i >= a.n;
            if (!bad) enter_row(p.index + i, (int32_t)row, a.n_i);
        }
    }
    const uint64_t bb = __ballot(bad);
    if ((threadIdx.x & (kWave - 1)) == 0 && bb && a.status) atomicOr(a.status, kStBadIndex);
}

// Row sums of rows [b0, b1) added to the bodies [j0, j0 + 64) that they belong to
// (lane l: body j0 + l), in a fixed order, by one wave: per run of 64 rows each
// body finds its rows as a mask (a ballot per bit of the body's place) and takes
// their sums from the lanes that hold them, all bodies at once; a body with many
// of the run's rows gets the wave's sum.
__device__ __forceinline__ void add_rows(const AdjointArgs &a, int64_t j0, int64_t b0, int64_t b1,
                                         double (&D)[6])
{
    constexpr int kAhead = 4;   // runs whose loads go out together
    const int lane = threadIdx.x & (kWave - 1);
    for (; b0 < b1; b0 += kAhead * kWave) {
        int32_t rel[kAhead];
        double v[kAhead][6];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t b = b0 + u * kWave + lane;
            const int64_t d = b < b1 ? a.i_block[b] - j0 : -1;
            rel[u] = d >= 0 && d < kWave && j0 + d < a.n ? (int32_t)d : -1;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int k = 0; k < 6; ++k)
                v[u][k] = rel[u] >= 0
                              ? a.row_part[(int64_t)k * a.n_i + b0 + u * kWave + lane] : 0.0;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            uint64_t mine = __ballot(rel[u] >= 0);   // the rows of body j0 + lane
            if (mine == 0) continue;
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const uint64_t bit = __ballot((rel[u] >> k) & 1);
                mine &= (lane >> k) & 1 ? bit : ~bit;
            }
            uint64_t heavy = __ballot(__popcll(mine) >= 16);
            while (heavy) {   // a body with many of them: the wave's sum
                const int l = __builtin_ctzll(heavy);
                heavy &= heavy - 1;
                double x[6];
#pragma unroll
                for (int k = 0; k < 6; ++k) x[k] = rel[u] == l ? v[u][k] : 0.0;
                group_sums<kWave, 6>(x);
                if (lane == l) {
                    mine = 0;
#pragma unroll
                    for (int k = 0; k < 6; ++k) D[k] += x[k];
                }
            }
            while (__ballot(mine != 0) != 0) {   // a turn per row of the body with most
                const int src = mine ? __builtin_ctzll(mine) : lane;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const double x = __shfl(v[u][k], src, kWave);
                    D[k] += mine ? x : 0.0;
                }
                mine &= mine - 1;
            }
        }
    }
}

// A body's gradient: its partials over the row blocks (fixed order) times its
// mass, less the row sums of the rows whose body it is.  W waves take 64 bodies
// and share the row blocks (W = 1: four waves of a work-group, each on its own).
// A body of one row finds it in the index; where one of the 64 has several
// (duplicate rows), the waves share the call's rows, and their sums are added in
// wave order.  Gradient calls, one wave looking through the rows for one body
// after another / so: 65536 rows of 1024 bodies 12.9 ms / 0.35, 65536 of one body
// 25.3 / 11.8, 20011 rows, a third of them of one body, 2.85 / 1.23, every body of
// 20011 twice 2.75 / 1.16; with the pass over all pairs for the bodies' sums that
// found a body's rows on its way 0.47, 16.0, 1.79 and 1.77.
template <int W>
__global__ __launch_bounds__(W == 1 ? 256 : kWave * W) void adj_bodies_reduce(AdjointArgs a,
                                                                              AdjPlan p,
                                                                              int32_t row_blocks,
                                                                              int64_t first)
{
    __shared__ double part[W][7][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int w = W == 1 ? 0 : wave;
    const int64_t j0 = first + (W == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x) * kWave;
    const int64_t j = j0 + lane;
    const bool live = j < a.n;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    const int32_t share = (row_blocks + W - 1) / W;
    const int32_t q1 = row_blocks < (w + 1) * share ? row_blocks : (w + 1) * share;
    if (live)
#pragma unroll 4
        for (int32_t q = w * share; q < q1; ++q) {
            const double *src = p.body_partial + (int64_t)q * 7 * a.n + j;
#pragma unroll
            for (int k = 0; k < 7; ++k) v[k] += src[(int64_t)k * a.n];
        }
    const int2 t = live ? p.index[j] : make_int2(a.n_i, 0);
    if constexpr (W > 1) {
#pragma unroll
        for (int k = 0; k < 7; ++k) part[w][k][lane] = v[k];
    }
    const bool several = W > 1 ? __syncthreads_or(t.y) != 0 : __ballot(t.y != 0) != 0;
    if (W > 1 && w == 0)
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            v[k] = 0.0;
#pragma unroll
            for (int u = 0; u < W; ++u) v[k] += part[u][k][lane];
        }
    double D[6] = {0, 0, 0, 0, 0, 0};
    if (several) {   // uniform over the work-group
        const int64_t rows = ((a.n_i + kWave - 1) / kWave + W - 1) / W * kWave;
        const int64_t b1 = a.n_i < (w + 1) * rows ? a.n_i : (w + 1) * rows;
        add_rows(a, j0, w * rows, b1, D);
        if constexpr (W > 1) {
            __syncthreads();   // the body sums are read
#pragma unroll
            for (int k = 0; k < 6; ++k) part[w][k][lane] = D[k];
            __syncthreads();
            if (w == 0)
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int u = 1; u < W; ++u) D[k] += part[u][k][lane];
        }
    } else if (w == 0 && t.x < a.n_i) {
#pragma unroll
        for (int k = 0; k < 6; ++k) D[k] = a.row_part[(int64_t)k * a.n_i + t.x];
    }
    if (w > 0) return;
    bool nonfin = false;
    if (live) {
        const double m = a.m[j];
#pragma unroll
        for (int k = 0; k < 6; ++k) v[k] = m * v[k] - D[k];
        a.gx[j] = v[0];
        a.gx[a.n + j] = v[1];
        a.gx[2 * a.n + j] = v[2];
        a.gv[j] = v[3];
        a.gv[a.n + j] = v[4];
        a.gv[2 * a.n + j] = v[5];
        a.gm[j] = v[6];
        nonfin = !finite6(v[0], v[1], v[2], v[3], v[4], v[5]) || !__builtin_isfinite(v[6]);
    }
    const uint64_t f = __ballot(nonfin);
    if (lane == 0 && f && a.status) atomicOr(a.status, kStNonFinite);
}

__global__ __launch_bounds__(256) void adj_clear_kernel(AdjointArgs a)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= a.n) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) a.gx[(int64_t)k * a.n + j] = a.gv[(int64_t)k * a.n + j] = 0.0;
    a.gm[j] = 0.0;
}

size_t round256(size_t b) { return (b + 255) / 256 * 256; }

template <int R, int W, int T>
void launch_pairs(const AdjointArgs &a, const AdjPlan &p, int64_t items, hipStream_t s)
{
    hipLaunchKernelGGL((adj_pairs_kernel<R, W, T>), dim3((unsigned)items), dim3(kWave * W), 0, s, a,
                       p);
}

}  // namespace

// Rows per block, tile, bodies per block and row blocks per panel.  Two
// rows per lane (512 a block) where there are enough rows for it, one (256)
// else: 4096 of 16384 234 us with two, 252 with one.  Tiles of 64 bodies where
// there are few bodies, or fewer than two work-groups per CU with tiles of
// 128, and the serial chain of a tile is much of the call: 1024 rows of 1024
// 35 us with 64, 57 with 128; 256 of 16384 33 and 49; 1024 of 12000 (376
// work-groups) 61 and 72; 1024 of 16384 (512) 75.5 both; 4096 of 16384 222 and
// 217; 2500 of 65536 517 and 497.
// Body blocks are multiples of the tile.  512-row blocks stage tiles of 128 in
// either case: a kernel with tiles of 64 for their body blocks of 64 takes as
// long (2048 of 9000 92.6 us against 93.2, 2049 of 12000 112.7 and 112.8, 2500 of
// 12000 118.6 and 118.7), and blocks of 128 bodies or 256 rows there take longer
// on few work-groups (2048 of 9000 111 and 97 us, 2500 of 9000 113 and 101).
// Body blocks for about 24 items per CU in a launch (48 give the same time and
// twice the row partials).  Entries of at most kAdjointBytes by smaller panels,
// whose launches then take more body blocks (with those of the whole call they
// had 768, 192 and 48 work-groups at 2^18, 2^19 and 2^20 bodies and rows: 195 and
// 1199 ms at the first two, 187 and 749 so, and 3014 at 2^20), then by longer
// body blocks; a call without room for more needs 7 n + 12 n_i values.
AdjointShape adjoint_shape(int64_t n, int32_t n_i, int cus, size_t budget)
{
    AdjointShape sh{};
    sh.row_block = n_i >= 2048 && n > 8192 ? 512 : 256;
    const int64_t blocks = std::max<int64_t>(1, ((int64_t)n_i + sh.row_block - 1) / sh.row_block);
    sh.tile = n > 8192 && blocks * ((n + 127) / 128) >= 2 * (int64_t)cus ? 128 : 64;
    const int64_t tiles = (n + sh.tile - 1) / sh.tile;
    // the row sums are the call's own size and no reason for smaller panels
    const size_t most = std::min(budget, kAdjointBytes + 6 * (size_t)n_i * sizeof(double));
    auto take_panel = [&](int64_t panel_blocks) {
        const int64_t want = ((int64_t)cus * 24 + panel_blocks - 1) / panel_blocks;
        sh.panel_blocks = panel_blocks;
        sh.body_len = (tiles + want - 1) / want * sh.tile;
    };
    take_panel(std::min(blocks, kAdjointPanelRows / sh.row_block));
    while (sh.panel_blocks > 1 && adjoint_scratch_bytes(n, n_i, sh) > most)
        take_panel((sh.panel_blocks + 1) / 2);
    while (sh.body_len < n && adjoint_scratch_bytes(n, n_i, sh) > most) sh.body_len *= 2;
    sh.index_in_gm = adjoint_scratch_bytes(n, n_i, sh) > budget;
    return sh;
}

size_t adjoint_scratch_bytes(int64_t n, int32_t n_i, const AdjointShape &sh)
{
    const int64_t q = (n + sh.body_len - 1) / sh.body_len;
    const int64_t rows = std::min<int64_t>(n_i, sh.panel_blocks * sh.row_block);
    return round256((size_t)q * 6 * rows * sizeof(double)) +
           round256(6 * (size_t)n_i * sizeof(double)) +
           round256((size_t)sh.panel_blocks * 7 * n * sizeof(double)) +
           (sh.index_in_gm ? 0 : round256((size_t)n * sizeof(int2)));
}

hipError_t launch_adjoint(const AdjointArgs &a0, const AdjointShape &sh, void *scratch,
                          hipStream_t s)
{
    AdjointArgs a = a0;
    if (a.n_i == 0) {
        hipLaunchKernelGGL(adj_clear_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s,
                           a);
        return hipGetLastError();
    }
    AdjPlan p{};
    p.row_block = sh.row_block;
    p.body_len = sh.body_len;
    p.body_blocks = (int32_t)((a.n + sh.body_len - 1) / sh.body_len);
    const int64_t panel = (int64_t)sh.panel_blocks * sh.row_block;
    const int64_t rows = std::min<int64_t>(a.n_i, panel);
    char *c = (char *)scratch;
    auto take = [&c](size_t bytes) {
        char *r = c;
        c += round256(bytes);
        return r;
    };
    p.row_partial = (double *)take((size_t)p.body_blocks * 6 * rows * sizeof(double));
    a.row_part = (double *)take(6 * (size_t)a.n_i * sizeof(double));
    p.body_partial = (double *)take((size_t)sh.panel_blocks * 7 * a.n * sizeof(double));
    p.index = sh.index_in_gm ? (int2 *)a.gm : (int2 *)take((size_t)a.n * sizeof(int2));
    int32_t used = 0;   // row-block slots that hold sums
    for (int64_t r0 = 0; r0 < a.n_i; r0 += panel) {
        p.panel_row0 = (int32_t)r0;
        p.panel_rows = (int32_t)std::min<int64_t>(panel, a.n_i - r0);
        p.add = r0 > 0;
        const int32_t blocks = (p.panel_rows + sh.row_block - 1) / sh.row_block;
        used = std::max(used, blocks);
        const int64_t items = (int64_t)blocks * p.body_blocks;
        if (sh.row_block == 512)
            launch_pairs<2, 4, 128>(a, p, items, s);
        else if (sh.tile == 128)
            launch_pairs<1, 4, 128>(a, p, items, s);
        else
            launch_pairs<1, 4, 64>(a, p, items, s);
        const int64_t tot = 6 * (int64_t)p.panel_rows;
        hipLaunchKernelGGL(adj_rows_reduce, dim3((unsigned)((tot + kWave - 1) / kWave)),
                           dim3(kWave * kReduceWaves), 0, s, a, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // waves per 64 bodies of the body sums: few where few rows leave nothing to
    // share (one row of 2^20 bodies, 16 waves against one 555 and 413 us, 2048 rows
    // 6162 and 5790), many where the rows are looked through
    // slices of bodies whose threads fit 32 bits
    constexpr int64_t kSlice = int64_t(1) << 27;
    for (int64_t first = 0; first < a.n; first += kSlice) {
        const int64_t groups = (std::min(kSlice, a.n - first) + kWave - 1) / kWave;
        const dim3 wgs((unsigned)groups), wgs4((unsigned)((groups + 3) / 4));
        if (a.n_i <= 1024)
            hipLaunchKernelGGL(adj_bodies_reduce<1>, wgs4, dim3(256), 0, s, a, p, used, first);
        else if (a.n_i <= 8192)
            hipLaunchKernelGGL(adj_bodies_reduce<4>, wgs, dim3(kWave * 4), 0, s, a, p, used, first);
        else
            hipLaunchKernelGGL(adj_bodies_reduce<16>, wgs, dim3(kWave * 16), 0, s, a, p, used, first);
    }
    return hipGetLastError();
}

}  // namespace nb
