// Device building blocks of the regular-force kernels (gfx950): the
// row-per-lane tile pass and the per-row merge of split partials.  Shared by
// the single-block launch (nb_force.hip) and the batched ensemble
// (nb_batched.hip).
//
// Slot layout of split partials (both launch kinds): a (row, split) pair owns
// one slot, and a row's slots are consecutive (slot = row's first slot +
// split).  part[slot * kSlotComp + k] holds component k of its FP64 sums
// (acc x,y,z, jerk x,y,z, then the mixed plan's two error-scale sums: one
// 64-byte record per slot), seg_cnt[slot] its neighbour count and
// seg_list[slot * kSegCap ...] the first kSegCap neighbours in ascending j.
// The force kernels write whole records; the merge reads a row's records as
// one contiguous run.
#pragma once

#include "nb_internal.h"
#include "nb_pair.h"

namespace nb {

struct alignas(16) JBody {
    static constexpr bool kPacked = false;
    double x, y, z, m;
    double vx, vy, vz;
    float m32;
    int32_t pad;
    __device__ __forceinline__ double mass() const { return m; }
};

// A body of the packed j-set in scalar registers: positions, velocities and
// the mass of the plan's precision.  The mixed plan reads the FP64 mass from
// the record in the rare branch only, which keeps eight scalar registers free.
typedef const __attribute__((address_space(4))) JRec *JRecPtr;
template <bool MIXED>
struct SBody {
    static constexpr bool kPacked = true;
    double x, y, z, vx, vy, vz;
    double m;      // FP64 plan
    float m32;     // mixed plan
    int64_t tail;  // FP64 plan: the record's last two words, see arrive()
    JRecPtr rec;
    __device__ __forceinline__ double mass() const { return MIXED ? rec->m : m; }
    __device__ __forceinline__ void load(JRecPtr p)
    {
        rec = p;
        x = p->x;
        y = p->y;
        z = p->z;
        vx = p->vx;
        vy = p->vy;
        vz = p->vz;
        if constexpr (MIXED)
            m32 = p->m32;
        else {
            m = p->m;
            tail = *(const __attribute__((address_space(4))) int64_t *)&p->m32;
        }
    }
    // A use of every loaded register: the wait for the loads stands here, and
    // loads issued after it are not waited for with them.  Emits no
    // instruction of its own.  The FP64 plan names the unused words of the
    // record too: it is loaded whole, and a register of the load that nothing
    // reads goes to some other value in between, with a wait for the load
    // (a lone wave of the batched kernel: 201 us instead of 146).
    __device__ __forceinline__ void arrive()
    {
        __asm__ volatile("" : "+s"(x), "+s"(y), "+s"(z), "+s"(vx), "+s"(vy), "+s"(vz));
        if constexpr (MIXED)
            __asm__ volatile("" : "+s"(m32));
        else
            __asm__ volatile("" : "+s"(m), "+s"(tail));
    }
};

template <bool MIXED>
struct Row {
    double x, y, z, vx, vy, vz;
    double hi;      // FP64 candidate bound (FP64 plan)
    float rs2f;     // canonical radius
    float candf;    // FP32 candidate bound (mixed plan)
    int32_t i;      // body index, -1 when the lane has no row
    int32_t jend;   // end of the j-range: staged bodies at or past it are padding
    int32_t cnt;    // neighbours found so far (true count)
    int32_t *lst;   // where this row's neighbours go
    int32_t lcap;   // capacity of lst
    // passes that settle rare pairs by runs: the current run of kFold bodies, a
    // bit per body, the pairs that the common path left out, and (mixed, see
    // classify()) those of them inside the radius
    uint32_t hit, nbr;
    Sums<MIXED> S;
    // whether a mixed pair that is left out may be something else than a
    // neighbour or the row's body: with the near bound, or where the radius is
    // below the least candidate bound
    __device__ __forceinline__ bool classify() const { return candf != rs2f; }
};

// Where the rows of one pass write: straight to the caller's outputs, or to
// the slots of one split (slot of row b = slot_base + (b - row_origin) *
// slot_stride, where slot_stride is the split count).
struct Dest {
    bool direct;
    int64_t slot_base;
    int64_t row_origin;
    int64_t slot_stride;
};

__device__ __forceinline__ int64_t dest_slot(const Dest &d, int64_t b)
{
    return d.slot_base + (b - d.row_origin) * d.slot_stride;
}

// The 64-byte partial-sum record of one slot.
__device__ __forceinline__ double2 *slot_rec(const ForceArgs &a, int64_t slot)
{
    return reinterpret_cast<double2 *>(a.part + slot * kSlotComp);
}

template <bool MIXED>
__device__ __forceinline__ void row_init(Row<MIXED> &R, const ForceArgs &a, int64_t b,
                                         int64_t row_end, const Dest &d, float near)
{
    R.S.zero();
    R.cnt = 0;
    R.i = -1;
    R.x = R.y = R.z = kFar * 0.5;   // inert placeholder
    R.vx = R.vy = R.vz = 0.0;
    R.rs2f = -1.0f;
    R.hi = -1.0;
    R.candf = -1.0f;
    R.lst = nullptr;
    R.lcap = 0;
    R.jend = 0;
    R.hit = R.nbr = 0;
    if (b >= row_end) return;
    const int64_t i = a.i_block[b];
    if (i < 0 || i >= a.n) return;   // bad index: handled in the epilogue / merge
    R.i = (int32_t)i;
    R.x = a.xp[i];
    R.y = a.xp[a.n + i];
    R.z = a.xp[2 * a.n + i];
    R.vx = a.vp[i];
    R.vy = a.vp[a.n + i];
    R.vz = a.vp[2 * a.n + i];
    R.rs2f = (float)a.rs2[b];
    R.hi = cand_bound_f64(R.rs2f);
    R.candf = cand_bound_f32(R.rs2f, near);
    if (d.direct) {
        R.lst = a.nb_list + b * (int64_t)a.cap;
        R.lcap = a.cap;
    } else {
        R.lst = a.seg_list + dest_slot(d, b) * kSegCap;
        R.lcap = kSegCap;
    }
}

// Row-per-lane mapping: each lane appends to its own row's list (in j order).
template <bool MIXED>
__device__ __forceinline__ void append(Row<MIXED> &R, int32_t jidx)
{
    if (R.cnt < R.lcap) R.lst[R.cnt] = jidx;
    ++R.cnt;
}

// What the mixed pass does with a near pair (outside the radius, inside the
// near bound), whose term is evaluated in FP64: at once ...
struct NearNow {
    template <class Body>
    __device__ __forceinline__ void take(Row<true> &R, int32_t, const Body &J, double dx, double dy,
                                         double dz)
    {
        add_term_f64(R.S.ax, R.S.ay, R.S.az, R.S.jx, R.S.jy, R.S.jz, dx, dy, dz, J.vx - R.vx,
                     J.vy - R.vy, J.vz - R.vz, J.mass());
    }
};

// ... or later: the lane notes the body in its own LDS queue, and every
// kNearSpan bodies the wave evaluates all that its lanes hold.  At once, the
// 30 FP64 instructions of a term run for one or two lanes of 64, in 28% of the
// steps at n = 2^18 and 7% at 2^20 (512 near pairs per row).  A lane whose
// queue is full takes further pairs at once: a halo row may have most of the
// j-set inside its near bound, and emptying the queue for one lane costs more
// than the term.  Both orders depend on the row alone, so its result does not
// depend on the other lanes.
constexpr int kNearSlots = 16;
constexpr int64_t kNearSpan = 4096;

// The record of one body of the packed j-set, read lane by lane.
__device__ __forceinline__ JBody rec_body(const JRec *r)
{
    const double2 *p = reinterpret_cast<const double2 *>(r);
    const double2 xy = p[0], zvx = p[1], vyz = p[2], m = p[3];
    JBody J;
    J.x = xy.x;
    J.y = xy.y;
    J.z = zvx.x;
    J.vx = zvx.y;
    J.vy = vyz.x;
    J.vz = vyz.y;
    J.m = m.x;
    return J;
}

struct NearLater {
    int32_t (*queue)[kBlock];   // LDS [kNearSlots][kBlock]
    int32_t n;                  // bodies queued
    template <class Body>
    __device__ __forceinline__ void take(Row<true> &R, int32_t jidx, const Body &J, double dx,
                                         double dy, double dz)
    {
        if (n < kNearSlots) {
            queue[n][threadIdx.x] = jidx;
            ++n;
        } else {
            NearNow().take(R, jidx, J, dx, dy, dz);
        }
    }
    // by the whole wave; rec0: the record of body j0
    __device__ __forceinline__ void evaluate(Row<true> &R, const JRec *rec0, int32_t j0)
    {
        for (int q = 0; __ballot(q < n) != 0; ++q)
            if (q < n) {
                const JBody J = rec_body(rec0 + (queue[q][threadIdx.x] - j0));
                add_term_f64(R.S.ax, R.S.ay, R.S.az, R.S.jx, R.S.jy, R.S.jz, J.x - R.x, J.y - R.y,
                             J.z - R.z, J.vx - R.vx, J.vy - R.vy, J.vz - R.vz, J.m);
            }
        n = 0;
    }
};

// Rare branch of a mixed pair (neighbour, self or near pair): appends a
// neighbour or takes a near pair; the pair then gets an excluding squared
// distance.
template <class Body, class Near>
__device__ __forceinline__ void rare_mixed(Row<true> &R, const Body &J, int32_t jidx, float &r2f,
                                           double dx, double dy, double dz, Near &N)
{
    if (r2f < R.candf) {
        double ex = dx, ey = dy, ez = dz;
        int32_t jj = jidx;
        opaque(ex, ey, ez);
        opaque_uniform(jj);
        // padding past the j-range (far away, mass 0) passes the test only for a
        // huge or infinite radius; it is never a neighbour and adds nothing
        if (jj < R.jend && jj != R.i) {
            if (r2f < R.rs2f)
                append(R, jj);
            else
                N.take(R, jj, J, ex, ey, ez);
        }
        r2f = kExclR2F;
    }
}

// Exact canonical test of an FP64 candidate pair; appends a neighbour, and
// excludes it or the self pair (padding has mass 0: its term is exactly zero).
// LATE: the test of the j-range stands after the canonical one (the packed
// pass: 65536 rows of 2^20 71.4 ms against 73.5) or before it (the LDS passes:
// 1024 of 1024 rows 23.7 us against 25.3).
template <bool LATE>
__device__ __forceinline__ void rare_f64(Row<false> &R, int32_t jidx, double &r2, double dx,
                                         double dy, double dz)
{
    if (r2 < R.hi && (LATE || jidx < R.jend)) {
        double ex = dx, ey = dy, ez = dz;
        int32_t jj = jidx;
        opaque(ex, ey, ez);
        opaque_uniform(jj);
        const bool self = jj == R.i;
        const bool nbr =
            (canon_r2f(ex, ey, ez) < R.rs2f) && !self && (!LATE || jj < R.jend);
        if (nbr) append(R, jj);
        if (nbr || self) r2 = kExclR2;
    }
}

// The rare branches of the passes that settle rare pairs by runs: they only
// set the pair's bit in R.hit and give it an excluding squared distance; what
// the pair is, take_hits settles once per run of kFold bodies.  Appending to
// the list in the branch itself takes five nested exec-mask changes and a
// store, and with 69 neighbours among 1024 bodies some lane of a wave has one
// at nearly every body, among 25000 at every sixth.  Passes over
// kRunMaxBodies bodies or more append at once: there the look at the bits of
// every run costs more than it saves.  LDS and packed passes, at once against
// by runs, mixed / FP64: 1024 rows of 1024 23.8 / 17.4 against 21.6 / 16.3 us,
// 4096 of 4096 50.7 / 46.6 against 46.9 / 43.4, 16384 of 16384 275 / 352
// against 268 / 348, 1500 of 65536 127 / 147 both, 300 of 131072 72.0 / 71.0
// against 72.3 / 71.9, 65536 of 2^20 49.7 / 71.5 against 50.2 / 72.3 ms; 160
// clusters of 1000 to 10000 1910 / 2573 against 1802 / 2407 us.
__device__ __forceinline__ void mark_mixed(Row<true> &R, float &r0, float &r1, uint32_t bit,
                                           bool classify)
{
    opaque(R.hit);
    if (classify) R.nbr |= (r0 < R.rs2f ? bit : 0u) | (r1 < R.rs2f ? bit << 1 : 0u);
    const bool c0 = r0 < R.candf, c1 = r1 < R.candf;
    R.hit |= (c0 ? bit : 0u) | (c1 ? bit << 1 : 0u);
    r0 = c0 ? kExclR2F : r0;
    r1 = c1 ? kExclR2F : r1;
}

__device__ __forceinline__ void mark_f64(Row<false> &R, int32_t jidx, double &r2, double dx,
                                         double dy, double dz, uint32_t bit)
{
    if (r2 < R.hi) {
        double ex = dx, ey = dy, ez = dz;
        opaque(ex, ey, ez);
        // the self pair fails the canonical test where the radius is zero
        const bool c = canon_r2f(ex, ey, ez) < R.rs2f || jidx == R.i;
        R.hit |= c ? bit : 0u;
        r2 = c ? kExclR2 : r2;
    }
}

// Settles the pairs that the run of kFold bodies from jb on left out, in j
// order: neighbours go to the list, near pairs (mixed) get their FP64 term; the
// self pair and padding past the j-range (which passes the test for a huge or
// infinite radius only) add nothing.  By the whole wave; at(q): body jb + q.
template <bool MIXED, class At>
__device__ __forceinline__ void take_hits(Row<MIXED> &R, int32_t jb, bool classify, const At &at)
{
    if (__ballot(R.hit != 0) == 0) return;
    uint32_t h = R.hit;
    R.hit = 0;
    if (R.jend - jb < kFold) h &= (1u << (R.jend - jb)) - 1u;
    const uint32_t self = (uint32_t)(R.i - jb);
    if (self < kFold) h &= ~(1u << self);
    if constexpr (MIXED) {
        if (classify) {
            uint32_t f = h & ~R.nbr;
            h &= R.nbr;
            R.nbr = 0;
            while (f) {
                const JBody J = at(__builtin_ctz(f));
                f &= f - 1;
                add_term_f64(R.S.ax, R.S.ay, R.S.az, R.S.jx, R.S.jy, R.S.jz, J.x - R.x, J.y - R.y,
                             J.z - R.z, J.vx - R.vx, J.vy - R.vy, J.vz - R.vz, J.m);
            }
        }
    }
    while (h) {
        append(R, jb + __builtin_ctz(h));
        h &= h - 1;
    }
}

// One row against two consecutive j, with a single branch for the rare cases
// (one exec-mask change per two j).  Mixed: FP64 differences, canonical FP32
// r2f (the neighbour test itself), FP32 terms; pairs with r2f below the
// near bound (neighbours, self, near pairs) take the rare branch.  FP64: FP64
// r2 against the candidate bound, the exact canonical test only for
// candidates.  One minimum and one compare decide for both j whether any lane
// has a rare case (NaN squared distances are never below the bound, alone or
// in the minimum), and a pair handled there gets an excluding squared
// distance, so the common path holds no select.  But the mixed LDS pass that
// handles rare pairs at once does select, and handles them after the FP32 terms
// (which touch other sums, so the bits are the same): there every LDS read of
// the two bodies goes out before the first arithmetic, and the small blocks
// that run it have one or two waves per SIMD, which wait for them.  Force pass
// of 64 rows, rare pairs first against last: 524288 bodies in 512, 1024, 4096
// splits 153.8 / 80.1 / 46.0 against 138.8 / 73.4 / 45.4 us, 262144 86.1 / 47.9
// / 31.0 against 78.7 / 44.1 / 30.5.  Every accumulator receives
// the terms of j and then j+1, as a loop over single j would give them.
// RUN: rare pairs are marked, not handled (bit: the first pair's place in the run).
template <bool MIXED, bool RUN, class Body, class Near>
__device__ __forceinline__ void pair_rows2(Row<MIXED> &R, const Body &J0, const Body &J1,
                                           int32_t jidx0, Near &N, uint32_t bit, bool classify)
{
    if constexpr (MIXED) {
        const double dx0 = J0.x - R.x, dy0 = J0.y - R.y, dz0 = J0.z - R.z;
        const double dx1 = J1.x - R.x, dy1 = J1.y - R.y, dz1 = J1.z - R.z;
        const float fx0 = (float)dx0, fy0 = (float)dy0, fz0 = (float)dz0;
        const float fx1 = (float)dx1, fy1 = (float)dy1, fz1 = (float)dz1;
        float r0 = __builtin_fmaf(fz0, fz0, __builtin_fmaf(fy0, fy0, fx0 * fx0));
        float r1 = __builtin_fmaf(fz1, fz1, __builtin_fmaf(fy1, fy1, fx1 * fx1));
        constexpr bool kTermsFirst = !RUN && !Body::kPacked;
        const bool rare = __builtin_fminf(r0, r1) < R.candf;
        float e0 = r0, e1 = r1;
        if constexpr (kTermsFirst) {
            e0 = r0 < R.candf ? kExclR2F : r0;
            e1 = r1 < R.candf ? kExclR2F : r1;
        } else if (rare) {
            if constexpr (RUN) {
                mark_mixed(R, e0, e1, bit, classify);
            } else {
                rare_mixed(R, J0, jidx0, e0, dx0, dy0, dz0, N);
                rare_mixed(R, J1, jidx0 + 1, e1, dx1, dy1, dz1, N);
            }
        }
        accum_mixed(R.S, fx0, fy0, fz0, e0, J0.vx - R.vx, J0.vy - R.vy, J0.vz - R.vz, J0.m32);
        accum_mixed(R.S, fx1, fy1, fz1, e1, J1.vx - R.vx, J1.vy - R.vy, J1.vz - R.vz, J1.m32);
        if constexpr (kTermsFirst)
            if (rare) {
                rare_mixed(R, J0, jidx0, r0, dx0, dy0, dz0, N);
                rare_mixed(R, J1, jidx0 + 1, r1, dx1, dy1, dz1, N);
            }
    } else {
        const double dx0 = J0.x - R.x, dy0 = J0.y - R.y, dz0 = J0.z - R.z;
        const double dx1 = J1.x - R.x, dy1 = J1.y - R.y, dz1 = J1.z - R.z;
        double r0 = __builtin_fma(dz0, dz0, __builtin_fma(dy0, dy0, dx0 * dx0));
        double r1 = __builtin_fma(dz1, dz1, __builtin_fma(dy1, dy1, dx1 * dx1));
        if (__builtin_fmin(r0, r1) < R.hi) {
            if constexpr (RUN) {
                opaque(R.hit);
                mark_f64(R, jidx0, r0, dx0, dy0, dz0, bit);
                mark_f64(R, jidx0 + 1, r1, dx1, dy1, dz1, bit << 1);
            } else {
                rare_f64<Body::kPacked>(R, jidx0, r0, dx0, dy0, dz0);
                rare_f64<Body::kPacked>(R, jidx0 + 1, r1, dx1, dy1, dz1);
            }
        }
        accum_f64(R.S, dx0, dy0, dz0, r0, J0.vx - R.vx, J0.vy - R.vy, J0.vz - R.vz, J0.m);
        accum_f64(R.S, dx1, dy1, dz1, r1, J1.vx - R.vx, J1.vy - R.vy, J1.vz - R.vz, J1.m);
    }
}

__device__ __forceinline__ void load_body(JBody &J, const ForceArgs &a, int64_t j, int64_t j1)
{
    if (j < j1) {
        J.x = a.xp[j];
        J.y = a.xp[a.n + j];
        J.z = a.xp[2 * a.n + j];
        J.vx = a.vp[j];
        J.vy = a.vp[a.n + j];
        J.vz = a.vp[2 * a.n + j];
        J.m = a.m[j];
    } else {
        J.x = J.y = J.z = kFar;
        J.vx = J.vy = J.vz = 0.0;
        J.m = 0.0;
    }
    J.m32 = (float)J.m;
    J.pad = 0;
}

// Packs bodies [j0, j1) of the SoA planes into records from out on, followed
// by kRecPad padding records.  k, stride: this thread's share.
__device__ __forceinline__ void pack_range(const ForceArgs &a, JRec *out, int64_t j0, int64_t j1,
                                           int64_t k, int64_t stride)
{
    for (int64_t q = k; q < j1 - j0 + kRecPad; q += stride) {
        JBody J;
        load_body(J, a, j0 + q, j1);
        JRec r;
        r.x = J.x;
        r.y = J.y;
        r.z = J.z;
        r.vx = J.vx;
        r.vy = J.vy;
        r.vz = J.vz;
        r.m = J.m;
        r.m32 = J.m32;
        r.pad = 0;
        out[q] = r;
    }
}

// Appends row b (with its j-range) to the FP64 redo list.
__device__ __forceinline__ void redo_push(const ForceArgs &a, int64_t b, int64_t j0, int64_t j1)
{
    const int32_t q = atomicAdd(a.redo_count, 1);
    a.redo_rows[q] = (int32_t)b;
    a.redo_j0[q] = (int32_t)j0;
    a.redo_j1[q] = (int32_t)j1;
}

// One row's final sums and count: to the outputs, or to its split slot.
// [j0, j1) is the row's whole j-range when the destination is direct.
template <bool MIXED>
__device__ __forceinline__ void row_store(const ForceArgs &a, int64_t b, const Dest &d,
                                          bool valid, const Sums<MIXED> &S, int32_t cnt,
                                          bool &ovf, bool &bad, bool &nonfin, int64_t j0,
                                          int64_t j1)
{
    if (d.direct) {
        if (!valid) {
            a.acc[b] = a.acc[a.n_i + b] = a.acc[2 * (int64_t)a.n_i + b] = 0.0;
            a.jerk[b] = a.jerk[a.n_i + b] = a.jerk[2 * (int64_t)a.n_i + b] = 0.0;
            a.nb_count[b] = 0;
            bad = true;
            return;
        }
        a.acc[b] = S.ax;
        a.acc[a.n_i + b] = S.ay;
        a.acc[2 * (int64_t)a.n_i + b] = S.az;
        a.jerk[b] = S.jx;
        a.jerk[a.n_i + b] = S.jy;
        a.jerk[2 * (int64_t)a.n_i + b] = S.jz;
        a.nb_count[b] = cnt;
        ovf = cnt > a.cap;
        nonfin = !finite6(S.ax, S.ay, S.az, S.jx, S.jy, S.jz);
        if (MIXED && a.redo_k > 0.0 &&
            needs_redo(a.redo_k, S.ax, S.ay, S.az, S.jx, S.jy, S.jz, S.va, S.vj))
            redo_push(a, b, j0, j1);
    } else {
        const int64_t slot = dest_slot(d, b);
        double2 *p = slot_rec(a, slot);
        p[0] = make_double2(S.ax, S.ay);
        p[1] = make_double2(S.az, S.jx);
        p[2] = make_double2(S.jy, S.jz);
        p[3] = make_double2(S.va, S.vj);
        a.seg_cnt[slot] = cnt;
    }
}

// ORs bits into a flag word that many waves may want to set: a word that
// already has them is left alone.  Where every row overflows its list (capacity
// 0, say) the atomics of all waves queue on one address: the merge of 20011 rows
// of 20011 bodies took 234 us with them, 59 without most of them.
__device__ __forceinline__ void set_flags(uint32_t *word, uint32_t bits)
{
    const uint32_t have = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((have & bits) != bits) atomicOr(word, bits);
}

__device__ __forceinline__ void flush_flags(const ForceArgs &a, bool ovf, bool bad, bool nonfin)
{
    // called in uniform control flow by every lane of the wave
    const uint64_t o = __ballot(ovf), b = __ballot(bad), f = __ballot(nonfin);
    if ((threadIdx.x & (kWave - 1)) == 0 && (o | b | f)) {
        const uint32_t st =
            (o ? kStOverflow : 0u) | (b ? kStBadIndex : 0u) | (f ? kStNonFinite : 0u);
        if (o) set_flags((uint32_t *)a.overflow, 1u);
        if (a.status) set_flags(a.status, st);
    }
}

// Rows [row0 + r*NB + tid] (r < IR, < row_end) of one work-group of NB
// lanes against bodies [j0, j1), staged through a double-buffered LDS tile
// of T bodies.  With T == NB every lane loads one body of the next tile
// into registers while the current tile is computed (one barrier per tile);
// otherwise each lane loads its T/NB bodies (or one, for T < NB) straight
// into the free buffer when the work-group reaches the tile, so no registers
// are held across the pair loop.  The j order, the FP32 fold points (every
// kFold bodies from j0) and all sums are the same for every T and NB, so
// results do not depend on the tile or work-group shape.  Must be called by
// the whole work-group (it contains barriers).
template <bool MIXED, bool RUN, int IR, int T, int NB>
__device__ __forceinline__ void rows_pass(const ForceArgs &a, JBody (*tile)[T], int64_t row0,
                                          int64_t row_end, int64_t j0, int64_t j1,
                                          const Dest &d, float near)
{
    static_assert(T % kFold == 0 && NB % kWave == 0, "tile and work-group shape");
    constexpr bool kPrefetch = T == NB;
    const int tid = threadIdx.x;
    NearNow N;
    bool classify[IR];
    Row<MIXED> R[IR];
#pragma unroll
    for (int r = 0; r < IR; ++r) {
        row_init(R[r], a, row0 + r * NB + tid, row_end, d, near);
        R[r].jend = (int32_t)j1;
        classify[r] = RUN && MIXED && __ballot(R[r].classify()) != 0;
    }

    // a wave none of whose lanes holds a valid row (the tail of a cluster's
    // last row tile) skips the pair loop; it still stages its share of every
    // tile and meets every barrier
    bool mine = false;
#pragma unroll
    for (int r = 0; r < IR; ++r) mine = mine || R[r].i >= 0;
    const bool wave_busy = __ballot(mine) != 0;

    const int64_t ntiles = j1 > j0 ? (j1 - j0 + T - 1) / T : 0;
    JBody nxt;
    if constexpr (kPrefetch) {
        if (ntiles > 0) {
            load_body(nxt, a, j0 + tid, j1);
            tile[0][tid] = nxt;
        }
        __syncthreads();
    }
    for (int64_t t = 0; t < ntiles; ++t) {
        const int cur = (int)(t & 1);
        const int64_t tbase = j0 + t * T;
        if constexpr (kPrefetch) {
            if (t + 1 < ntiles) load_body(nxt, a, tbase + T + tid, j1);
        } else {
            // buffer cur was last read for tile t-2, and every wave has
            // passed the barrier of tile t-1 since
            for (int k = tid; k < T; k += NB) {
                JBody J;
                load_body(J, a, tbase + k, j1);
                tile[cur][k] = J;
            }
            __syncthreads();
        }
        const JBody *buf = tile[cur];
        // whole runs of kFold up to the last body of the range (a split may
        // be much shorter than a tile)
        const int64_t left = (j1 - tbase + kFold - 1) & ~(int64_t)(kFold - 1);
        const int live = !wave_busy ? 0 : (left < T ? (int)left : T);
        for (int jj = 0; jj < live; jj += kFold) {
            for (int q = 0; q < kFold; q += 2) {
                const int32_t jidx = (int32_t)(tbase + jj + q);
#pragma unroll
                for (int r = 0; r < IR; ++r)
                    pair_rows2<MIXED, RUN>(R[r], buf[jj + q], buf[jj + q + 1], jidx, N, 1u << q,
                                           classify[r]);
            }
            if constexpr (RUN) {
#pragma unroll
                for (int r = 0; r < IR; ++r)
                    take_hits(R[r], (int32_t)tbase + jj, classify[r],
                              [buf, jj](int q) { return buf[jj + q]; });
            }
            if constexpr (MIXED) {
#pragma unroll
                for (int r = 0; r < IR; ++r) R[r].S.fold();
            } else if (((t * T + jj + kFold) & (kFoldF64 - 1)) == 0) {
#pragma unroll
                for (int r = 0; r < IR; ++r) R[r].S.fold();
            }
        }
        if constexpr (kPrefetch) {
            if (t + 1 < ntiles) tile[cur ^ 1][tid] = nxt;
            __syncthreads();
        }
    }
    if constexpr (!kPrefetch) __syncthreads();   // the tile may be reused by the caller

    bool ovf = false, bad = false, nonfin = false;
#pragma unroll
    for (int r = 0; r < IR; ++r) {
        if constexpr (!MIXED) R[r].S.fold();
        const int64_t b = row0 + r * NB + tid;
        if (b < row_end) {
            bool o = false, bd = false, f = false;
            row_store<MIXED>(a, b, d, R[r].i >= 0, R[r].S, R[r].cnt, o, bd, f, j0, j1);
            ovf |= o;
            bad |= bd;
            nonfin |= f;
        }
    }
    flush_flags(a, ovf, bad, nonfin);
}

// LDS of the near-pair queues (the mixed pass of kBlock-lane work-groups that
// handles rare pairs at once).
template <bool MIXED, bool RUN>
__device__ __forceinline__ int32_t (*near_queue())[kBlock]
{
    if constexpr (MIXED && !RUN) {
        __shared__ int32_t q[kNearSlots][kBlock];
        return q;
    } else {
        return nullptr;
    }
}

// One wave's kWave rows [row0, row0 + kWave) against bodies [j0, j1) of the
// packed j-set, whose records start at rec: the bodies are wave-uniform
// operands in scalar registers, loaded two bodies ahead, so the pair loop has
// no LDS traffic, no barrier and no body in vector registers.  The LDS pass
// reads 52 to 56 bytes per lane and pair by broadcast, about 105 (mixed) and
// 112 (FP64) LDS cycles per CU for the 4 x 64 pairs that its SIMDs compute in
// 120 and 165 cycles, which held both back: 65536 rows at n = 2^20 took 56.8
// ms mixed and 79.1 ms FP64 through LDS and take 51.4 and 74.2 ms here (1.34
// and 0.93e12 pairs/s).  What bounds it now is VALU issue: the loop's
// instructions, timed one by one at four waves per SIMD, add up to 53 ns
// (mixed) and 67 ns (FP64) per 64 pairs and SIMD; it takes 47 to 49 and 66 to 71
// (FP32 instructions partly pair up, so the sum is no floor).
// Order and fold points are those of rows_pass, and so are the results but for
// the order of a mixed row's near terms (queue: their queues, mixed pass only).
// Records past j1 up
// to the next multiple of kFold from j0, and two more, must be readable, and
// at the end of the j-set they are padding.
template <bool MIXED, bool RUN>
__device__ __forceinline__ void rows_pass_packed(const ForceArgs &a, const JRec *rec0,
                                                 int64_t row0, int64_t row_end, int64_t j0,
                                                 int64_t j1, const Dest &d, float near,
                                                 int32_t (*queue)[kBlock])
{
    JRecPtr rec = (JRecPtr)rec0;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t b = row0 + lane;
    Row<MIXED> R;
    row_init(R, a, b, row_end, d, near);
    R.jend = (int32_t)j1;
    const bool classify = RUN && MIXED && __ballot(R.classify()) != 0;
    NearLater N{queue, 0};
    if (__ballot(R.i >= 0) != 0) {
        SBody<MIXED> A0, A1, B0, B1;
        A0.load(rec);
        A1.load(rec + 1);
        for (int64_t jb = j0; jb < j1; jb += kFold) {
#pragma unroll 1
            for (int q = 0; q < kFold; q += 4) {
                const int32_t jidx = (int32_t)jb + q;
                A0.arrive();
                A1.arrive();
                B0.load(rec + 2);
                B1.load(rec + 3);
                __builtin_amdgcn_sched_barrier(0);
                pair_rows2<MIXED, RUN>(R, A0, A1, jidx, N, 1u << q, classify);
                B0.arrive();
                B1.arrive();
                rec += 4;
                A0.load(rec);
                A1.load(rec + 1);
                __builtin_amdgcn_sched_barrier(0);
                pair_rows2<MIXED, RUN>(R, B0, B1, jidx + 2, N, 4u << q, classify);
            }
            if constexpr (RUN)
                take_hits(R, (int32_t)jb, classify,
                          [rec0, jb, j0](int q) { return rec_body(rec0 + (jb - j0 + q)); });
            if (MIXED || ((jb - j0 + kFold) & (kFoldF64 - 1)) == 0) R.S.fold();
            if constexpr (MIXED && !RUN)
                if (((jb - j0 + kFold) & (kNearSpan - 1)) == 0 || jb + kFold >= j1)
                    N.evaluate(R, rec0, (int32_t)j0);
        }
    }
    bool ovf = false, bad = false, nonfin = false;
    if constexpr (!MIXED) R.S.fold();
    if (b < row_end)
        row_store<MIXED>(a, b, d, R.i >= 0, R.S, R.cnt, ovf, bad, nonfin, j0, j1);
    flush_flags(a, ovf, bad, nonfin);
}

// Geometry of one row's splits for the merge.
struct MergeGeom {
    int32_t splits;
    int64_t slot0;        // slot of split 0
    int64_t slot_step;    // slot(s) = slot0 + s * slot_step
    int64_t j_begin, j_end, split_len;
};

// The partner's value of a butterfly level inside a row of 16 lanes, moved by
// DPP: quad permutes for offsets 1 and 2, row rotations for 4 and 8.  (Once
// the levels above have run, the sums repeat every 2 * O lanes, so a rotation
// by O reads the same sum as an exchange with lane ^ O.)
template <int O>
__device__ __forceinline__ double row_partner(double v)
{
    constexpr int ctrl = O == 1 ? 0xB1 : O == 2 ? 0x4E : 0x120 + O;
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, ctrl, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(u >> 32), ctrl, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Exchange of 32-lane halves (O = 32) or of neighbouring 16-lane rows (O = 16)
// between two values: x becomes {x low, y low}, y {x high, y high}, where low
// and high are the halves, or the even and the odd rows.
template <int O>
__device__ __forceinline__ void swap_lanes(double &x, double &y)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, x), b = __builtin_bit_cast(uint64_t, y);
    uint32_t r[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t p = (uint32_t)(a >> (32 * h)), q = (uint32_t)(b >> (32 * h));
        const auto t = O == 32 ? __builtin_amdgcn_permlane32_swap(p, q, false, false)
                               : __builtin_amdgcn_permlane16_swap(p, q, false, false);
        r[0][h] = t[0];
        r[1][h] = t[1];
    }
    x = __builtin_bit_cast(double, ((uint64_t)r[0][1] << 32) | r[0][0]);
    y = __builtin_bit_cast(double, ((uint64_t)r[1][1] << 32) | r[1][0]);
}

template <int O, int K>
__device__ __forceinline__ void row_levels(double (&v)[K])
{
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += row_partner<O>(v[k]);
    if constexpr (O > 1) row_levels<O / 2, K>(v);
}

// Sums of K values over the W aligned lanes of a lane group (butterfly,
// largest offset first; every lane of the group gets the results).  Lanes
// exchange through the VALU (swaps of halves and rows, DPP), not through LDS:
// with ds_bpermute_b32 each level of a double cost two trips through the LDS
// pipe and their latency (a 1-row block at N = 2^20 spent 2.2 us of its merge
// in them).  Each value gets the pairs and order of its own butterfly.
template <int W, int K>
__device__ __forceinline__ void group_sums(double (&v)[K])
{
    static_assert(W == 4 || W == 16 || W == kWave, "lane group");
    if constexpr (W == kWave) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double t = v[k];
            swap_lanes<32>(v[k], t);
            v[k] += t;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double t = v[k];
            swap_lanes<16>(v[k], t);
            v[k] += t;
        }
    }
    row_levels<(W == 4 ? 2 : 8), K>(v);
}

// The same sums of G groups of K values over a whole wave, handed out: the
// lanes of part p of the wave (p = lane * G / 64) get the K sums of group p
// in v[0][..].  The first levels halve the values with the lanes (one swap
// serves two values), so four groups of eight cost a quarter of 32 whole
// butterflies.  Same pairs and order per value as group_sums.
template <int G, int K>
__device__ __forceinline__ void group_sums_spread(double (&v)[G][K])
{
    static_assert(G == 1 || G == 2 || G == 4, "groups per wave");
    if constexpr (G == 1) {
        group_sums<kWave, K>(v[0]);
        return;
    } else {
#pragma unroll
        for (int g = 0; g < G / 2; ++g)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                swap_lanes<32>(v[g][k], v[g + G / 2][k]);
                v[g][k] += v[g + G / 2][k];
            }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double t = v[0][k];
            if constexpr (G == 4) t = v[1][k];
            swap_lanes<16>(v[0][k], t);
            v[0][k] += t;
        }
        row_levels<8, K>(v[0]);
    }
}

// A word written by an earlier launch (a counter), read at a uniform address
// through the scalar cache: many work-groups reading one word this way do
// not queue on one memory channel, as uncached vector loads of it do.
__device__ __forceinline__ int32_t load_word_uniform(const int32_t *p)
{
    return *(const __attribute__((address_space(4))) int32_t *)p;
}

// The same for a double that no lane writes during the kernel (an input, or
// data of an earlier kernel): it lands in scalar registers.
__device__ __forceinline__ double load_f64_uniform(const double *p)
{
    return *(const __attribute__((address_space(4))) double *)p;
}

// A record of an earlier launch or upload that no lane writes during the
// kernel, read at a uniform address into scalar registers.
template <class T>
__device__ __forceinline__ T load_uniform(const T *p)
{
    static_assert(sizeof(T) % 4 == 0, "whole words");
    const __attribute__((address_space(4))) uint32_t *q =
        (const __attribute__((address_space(4))) uint32_t *)p;
    uint32_t w[sizeof(T) / 4];
#pragma unroll
    for (size_t k = 0; k < sizeof(T) / 4; ++k) w[k] = q[k];
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// Lanes per row of the single-wave merge for a given split count: the next of
// 4, 16, 64 at or above it.  For S <= W each lane holds at most one partial
// and the lanes past S hold exact zeros, which the butterfly adds before any
// two partials meet, so every W >= S gives the same bits (and the same as one
// whole wave per row).
__host__ __device__ constexpr int merge_width(int64_t splits)
{
    return splits <= 4 ? 4 : (splits <= 16 ? 16 : 64);
}

// Merge of one row by a group of W lanes (W = 64: one whole wave; smaller W:
// 64/W rows per wave): sums the split partials in a fixed order, concatenates
// neighbour segments in split order (ascending j), writes the true count, and
// rebuilds any segment that overflowed its scratch capacity by re-running the
// canonical test over that split's j-range.  has_row = false for a group past
// the last row; every lane of the wave must call this (it ends in a ballot).
template <int W>
__device__ __forceinline__ void merge_row(const ForceArgs &a, int64_t b, bool has_row,
                                          const MergeGeom &g)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int l = lane & (W - 1);       // lane within the row's group
    const int gbase = lane - l;         // first lane of the group
    const uint64_t gmask = W == kWave ? ~0ull : (((1ull << W) - 1) << gbase);
    const int64_t i = has_row ? a.i_block[b] : -1;
    const bool bad = has_row && (i < 0 || i >= a.n);
    const int32_t S = has_row ? g.splits : 0;

    double v[kSlotComp] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int32_t s = l; s < S; s += W) {
        const double2 *p = slot_rec(a, g.slot0 + (int64_t)s * g.slot_step);
#pragma unroll
        for (int k = 0; k < kSlotComp / 2; ++k) {
            const double2 t = p[k];
            v[2 * k] += t.x;
            v[2 * k + 1] += t.y;
        }
    }
    group_sums<W, kSlotComp>(v);

    bool ovf = false, nonfin = false;
    if (bad) {
        if (l == 0) {
            for (int k = 0; k < 3; ++k) {
                a.acc[(int64_t)k * a.n_i + b] = 0.0;
                a.jerk[(int64_t)k * a.n_i + b] = 0.0;
            }
            a.nb_count[b] = 0;
        }
    } else if (has_row) {
        const double xi = a.xp[i], yi = a.xp[a.n + i], zi = a.xp[2 * a.n + i];
        const float rs2f = (float)a.rs2[b];
        int64_t off = 0;   // uniform in the group: neighbours placed so far (true count)
        for (int32_t s0 = 0; s0 < S; s0 += W) {
            const int32_t s = s0 + l;
            const int64_t slot = g.slot0 + (int64_t)s * g.slot_step;
            const int32_t c = s < S ? a.seg_cnt[slot] : 0;
            int64_t inc = c;   // inclusive scan of c over the group
#pragma unroll
            for (int o = 1; o < W; o <<= 1) {
                const int64_t t = __shfl_up(inc, o, W);
                if (l >= o) inc += t;
            }
            const int64_t start = off + inc - c;
            const bool room = c > 0 && start < a.cap;
            const bool rebuild = room && c > kSegCap;
            // segments that fit.  Short ones (at most kLaneCopy entries, the
            // usual case with many splits): each lane copies its own in
            // 16-byte loads (a segment's storage holds kSegCap entries, a
            // multiple of 8, so the loads stay inside it), all segments of the
            // group in flight together.  Longer ones: the whole group copies
            // each in turn (coalesced).
            static_assert(kSegCap % 8 == 0, "segment storage in 8-entry rounds");
            constexpr int64_t kLaneCopy = 16;
            const int64_t take = room ? ((int64_t)c < a.cap - start ? c : a.cap - start) : 0;
            if (room && !rebuild && take <= kLaneCopy) {
                const int4 *src = reinterpret_cast<const int4 *>(a.seg_list + slot * kSegCap);
                int32_t *dst = a.nb_list + b * (int64_t)a.cap + start;
                for (int64_t e = 0; e < take; e += 8) {
                    const int4 u0 = src[e / 4], u1 = src[e / 4 + 1];
                    const int32_t t[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        if (e + k < take) dst[e + k] = t[k];
                }
            }
            uint64_t cp = __ballot(room && !rebuild && take > kLaneCopy) & gmask;
            while (cp) {
                const int q = __builtin_ctzll(cp);
                cp &= cp - 1;
                const int64_t sl = __shfl(slot, q, kWave);
                const int64_t st = __shfl(start, q, kWave);
                const int64_t tk = __shfl(take, q, kWave);
                const int32_t *src = a.seg_list + sl * kSegCap;
                int32_t *dst = a.nb_list + b * (int64_t)a.cap + st;
                for (int64_t e = l; e < tk; e += W) dst[e] = src[e];
            }
            uint64_t rb = __ballot(rebuild) & gmask;
            while (rb) {   // overflowed segments: the group rescans them one by one
                const int q = __builtin_ctzll(rb);
                rb &= rb - 1;
                const int32_t sq = __shfl(s, q, kWave);
                const int64_t st = __shfl(start, q, kWave);
                const int64_t lim = a.cap - st;
                const int64_t jb = g.j_begin + (int64_t)sq * g.split_len;
                const int64_t je = jb + g.split_len < g.j_end ? jb + g.split_len : g.j_end;
                int64_t placed = 0;
                for (int64_t base = jb; base < je && placed < lim; base += W) {
                    const int64_t j = base + l;
                    bool nbr = false;
                    if (j < je && j != i) {
                        const double dx = a.xp[j] - xi, dy = a.xp[a.n + j] - yi,
                                     dz = a.xp[2 * a.n + j] - zi;
                        nbr = canon_r2f(dx, dy, dz) < rs2f;
                    }
                    const uint64_t nm = __ballot(nbr) & gmask;
                    if (nbr) {
                        const int64_t p = placed + lanes_below(nm);
                        if (p < lim) a.nb_list[b * (int64_t)a.cap + st + p] = (int32_t)j;
                    }
                    placed += __popcll(nm);
                }
            }
            off += __shfl(inc, gbase + W - 1, kWave);
        }
        if (l == 0) {
            a.acc[b] = v[0];
            a.acc[a.n_i + b] = v[1];
            a.acc[2 * (int64_t)a.n_i + b] = v[2];
            a.jerk[b] = v[3];
            a.jerk[a.n_i + b] = v[4];
            a.jerk[2 * (int64_t)a.n_i + b] = v[5];
            a.nb_count[b] = (int32_t)off;
            ovf = off > a.cap;
            nonfin = !finite6(v[0], v[1], v[2], v[3], v[4], v[5]);
            if (a.redo_k > 0.0 && needs_redo(a.redo_k, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]))
                redo_push(a, b, g.j_begin, g.j_end);
        }
    }
    flush_flags(a, ovf, bad && l == 0, nonfin);
}

// Chunks of refined row q: its j-range cut into kRedoChunk bodies.
__device__ __forceinline__ int32_t redo_row_chunks(const ForceArgs &a, int32_t q)
{
    const int64_t len = (int64_t)load_word_uniform(a.redo_j1 + q) -
                        (int64_t)load_word_uniform(a.redo_j0 + q);
    return len > 0 ? (int32_t)((len + kRedoChunk - 1) / kRedoChunk) : 0;
}

// The data of refined rows q0 .. q0+nr-1 (nr <= R), uniform over the
// work-group: scalar registers.
template <int R>
struct RedoRows {
    double x[R], y[R], z[R], vx[R], vy[R], vz[R], hi[R];
    float rs2f[R];
    int64_t i[R];
    int64_t j0, j1;   // j-range of row q0
    int nr;
    __device__ __forceinline__ void load(const ForceArgs &a, int32_t q0, int n_rows)
    {
        nr = n_rows;
        j0 = load_word_uniform(a.redo_j0 + q0);
        j1 = load_word_uniform(a.redo_j1 + q0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int32_t q = q0 + (r < nr ? r : 0);
            const int64_t b = load_word_uniform(a.redo_rows + q);
            const int64_t k = load_word_uniform(a.i_block + b);
            i[r] = k;
            x[r] = load_f64_uniform(a.xp + k);
            y[r] = load_f64_uniform(a.xp + a.n + k);
            z[r] = load_f64_uniform(a.xp + 2 * a.n + k);
            vx[r] = load_f64_uniform(a.vp + k);
            vy[r] = load_f64_uniform(a.vp + a.n + k);
            vz[r] = load_f64_uniform(a.vp + 2 * a.n + k);
            rs2f[r] = (float)load_f64_uniform(a.rs2 + b);
            hi[r] = cand_bound_f64(rs2f[r]);
        }
    }
};

// FP64 wave sums over chunk c (c < the chunk count) of rows that share one
// j-range, by a whole work-group: lds[r][k][w] gets component k (acc, jerk) of
// row r over the bodies of wave w.  A lane takes bodies kBlock apart,
// kRedoBatch of them loaded before any is used (a refined row is a chain of
// memory round trips: one body at a time, an 8192-body chunk took 20 us for 2
// us of arithmetic; four at a time or four rows cost a wave of occupancy and
// gave 4.9 and 4.0 ms on 1500 rows of 2^20 bodies against 4.0), and every
// body serves all rows.  Per row the lane order
// and the reductions do not depend on R or nr, so a row gets the same bits in
// any group.  Ends with the work-group synchronised; the caller alternates
// between two lds buffers, so one barrier per chunk is enough.
constexpr int kRedoBatch = 2;
static_assert(kRedoChunk % (kBlock * kRedoBatch) == 0, "whole batches per chunk");

template <int R>
__device__ __forceinline__ void redo_chunk_rows(const ForceArgs &a, const RedoRows<R> &Q,
                                               int32_t c, double (*lds)[6][kBlock / kWave])
{
    const int64_t cj0 = Q.j0 + (int64_t)c * kRedoChunk;
    const int64_t cj1 = cj0 + kRedoChunk < Q.j1 ? cj0 + kRedoChunk : Q.j1;
    Sums<false> S[R];
#pragma unroll
    for (int r = 0; r < R; ++r) S[r].zero();
    for (int64_t jb = cj0 + threadIdx.x; jb - threadIdx.x < cj1; jb += kBlock * kRedoBatch) {
        JBody J[kRedoBatch];
#pragma unroll
        for (int u = 0; u < kRedoBatch; ++u) load_body(J[u], a, jb + u * kBlock, cj1);
#pragma unroll
        for (int u = 0; u < kRedoBatch; ++u) {
            const int64_t j = jb + u * kBlock;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r >= Q.nr) break;
                const double dx = J[u].x - Q.x[r], dy = J[u].y - Q.y[r], dz = J[u].z - Q.z[r];
                double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
                if (r2 < Q.hi[r]) {
                    double ex = dx, ey = dy, ez = dz;
                    opaque(ex, ey, ez);
                    if (j == Q.i[r] || canon_r2f(ex, ey, ez) < Q.rs2f[r]) r2 = kExclR2;
                }
                accum_f64(S[r], dx, dy, dz, r2, J[u].vx - Q.vx[r], J[u].vy - Q.vy[r],
                          J[u].vz - Q.vz[r], J[u].m);
            }
        }
    }
    double v[R][6];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        S[r].fold();
        v[r][0] = S[r].ax;
        v[r][1] = S[r].ay;
        v[r][2] = S[r].az;
        v[r][3] = S[r].jx;
        v[r][4] = S[r].jy;
        v[r][5] = S[r].jz;
    }
    group_sums_spread<R, 6>(v);
    const int lane = threadIdx.x & (kWave - 1);
    if ((lane & (kWave / R - 1)) == 0)
#pragma unroll
        for (int k = 0; k < 6; ++k) lds[lane / (kWave / R)][k][threadIdx.x / kWave] = v[0][k];
    __syncthreads();
}

// A chunk's sum of one component: its wave sums in wave order.
__device__ __forceinline__ double redo_chunk_sum(const double (&w)[kBlock / kWave])
{
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < kBlock / kWave; ++q) t += w[q];
    return t;
}


// Copies entries [from, take) of the neighbour segment of split s (count c)
// to dst: from its slot, or, for an overflowed segment, by rescanning the
// split's j-range in order.
__device__ __forceinline__ void copy_segment(const ForceArgs &a, const MergeGeom &g, int64_t b,
                                             int64_t i, int32_t s, int32_t c, int64_t from,
                                             int64_t take, int32_t *dst)
{
    const int64_t slot = g.slot0 + (int64_t)s * g.slot_step;
    if (c <= kSegCap) {
        const int32_t *src = a.seg_list + slot * kSegCap;
        for (int64_t q = from; q < take; ++q) dst[q] = src[q];
        return;
    }
    const double xi = a.xp[i], yi = a.xp[a.n + i], zi = a.xp[2 * a.n + i];
    const float rs2f = (float)a.rs2[b];
    const int64_t jb = g.j_begin + (int64_t)s * g.split_len;
    const int64_t je = jb + g.split_len < g.j_end ? jb + g.split_len : g.j_end;
    int64_t placed = 0;
    for (int64_t j = jb; j < je && placed < take; ++j) {
        if (j == i) continue;
        const double dx = a.xp[j] - xi, dy = a.xp[a.n + j] - yi, dz = a.xp[2 * a.n + j] - zi;
        if (canon_r2f(dx, dy, dz) < rs2f) {
            if (placed >= from) dst[placed] = (int32_t)j;
            ++placed;
        }
    }
}

// Partial records of splits sb + u * kBlock (u < B) of one row;
// past the last split, split 0's record is loaded (and not added).
template <int B>
__device__ __forceinline__ void merge_load_batch(const ForceArgs &a, const MergeGeom &g,
                                                 int32_t sb, double (&t)[B][kSlotComp])
{
#pragma unroll
    for (int u = 0; u < B; ++u) {
        const int32_t s = sb + u * kBlock;
        const double2 *p = slot_rec(a, g.slot0 + (int64_t)(s < g.splits ? s : 0) * g.slot_step);
#pragma unroll
        for (int k = 0; k < kSlotComp / 2; ++k) {
            const double2 q = p[k];
            t[u][2 * k] = q.x;
            t[u][2 * k + 1] = q.y;
        }
    }
}

template <int B>
__device__ __forceinline__ void merge_add_batch(int32_t S, int32_t sb,
                                                const double (&t)[B][kSlotComp],
                                                double (&v)[kSlotComp])
{
#pragma unroll
    for (int u = 0; u < B; ++u)
        if (sb + u * kBlock < S) {
#pragma unroll
            for (int k = 0; k < kSlotComp; ++k) v[k] += t[u][k];
        }
}

// Merge of one row by a whole work-group, for plans with many splits.  The
// sums stride the splits over the lanes (fixed order: a lane adds its splits
// in increasing order, then the wave butterfly, then the four wave sums in
// wave order).  For the list, lane t owns the contiguous splits [t*K,
// (t+1)*K), and a work-group prefix scan of the lanes' counts places its
// segments, so the list stays in split order.  The work is laid out for few
// memory round trips: a lane's counts are loaded with its partials, and the
// first two entries of all its segments are loaded before any is stored.
// B: strides of split partials, and segment counts, loaded per batch (the least
// of 1, 2, 4, 8 that covers the splits in one; order and bits do not depend on
// it).  Eight for every launch loaded split 0's record up to seven times more
// for each lane and held 163 registers, one holds 100.  Whole calls: one row of
// 2^20 (1024 splits) 18.3 us with eight, 17.3 so; 32 of 131072 (256) 18.2 and
// 16.7, 1024 of 16384 (256) 44.7 and 41.3, 2048 of 131072 (256) 347 and 342.
// Called once per work-group (its LDS arrays are not reused).
template <int B>
__device__ __forceinline__ void merge_row_wg(const ForceArgs &a, int64_t b, const MergeGeom &g,
                                             double (*lds)[kBlock / kWave], int64_t *scan)
{
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), w = tid / kWave;
    const int64_t i = a.i_block[b];
    const bool bad = i < 0 || i >= a.n;
    const int32_t S = g.splits;
    const int32_t K = (S + kBlock - 1) / kBlock;
    const int32_t s0 = tid * K;
    const int32_t nmine = s0 < S ? (S - s0 < K ? S - s0 : K) : 0;

    // sums: the loads of B strides are issued before any is added,
    // so a lane waits on one memory latency per batch, not per split.  The
    // first batch is issued ahead of the lane's first B counts (the
    // memory counter waits in issue order), so both arrive in one round trip.
    double v[kSlotComp] = {0, 0, 0, 0, 0, 0, 0, 0};
    double t[B][kSlotComp];
    merge_load_batch<B>(a, g, tid, t);
    int32_t ck[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
        const int32_t s = s0 + u < S ? s0 + u : S - 1;   // in range; unused past nmine
        const int32_t c = a.seg_cnt[g.slot0 + (int64_t)s * g.slot_step];
        ck[u] = u < nmine ? c : 0;
    }
    merge_add_batch<B>(S, tid, t, v);
    for (int32_t sb = tid + kBlock * B; sb < S; sb += kBlock * B) {
        merge_load_batch<B>(a, g, sb, t);
        merge_add_batch<B>(S, sb, t, v);
    }
    int64_t mine = 0;
#pragma unroll
    for (int u = 0; u < B; ++u) mine += ck[u];
    for (int32_t sb = B; sb < nmine; sb += B) {   // K > B
        int32_t c[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int32_t s = sb + u < nmine ? s0 + sb + u : s0;
            c[u] = a.seg_cnt[g.slot0 + (int64_t)s * g.slot_step];
        }
#pragma unroll
        for (int u = 0; u < B; ++u) mine += sb + u < nmine ? c[u] : 0;
    }

    // one barrier for both reductions: wave butterflies of the sums and a
    // wave scan of the counts, then the four waves' values from LDS
    group_sums<kWave, kSlotComp>(v);
    int64_t inc = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < kSlotComp; ++k) lds[k][w] = v[k];
    if (lane == kWave - 1) scan[w] = inc;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSlotComp; ++k) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kBlock / kWave; ++q) t += lds[k][q];
        v[k] = t;
    }
    int64_t before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < kBlock / kWave; ++q) {
        const int64_t t = scan[q];
        total += t;
        before += q < w ? t : 0;
    }
    const int64_t start = before + inc - mine;

    bool ovf = false, nonfin = false;
    if (!bad) {
        // the lane's segments in batches of B: the first two
        // entries of every segment of a batch are loaded before any is stored
        int32_t *row = a.nb_list + b * (int64_t)a.cap;
        int64_t at = start;
        for (int32_t sb = 0; sb < nmine && at < a.cap; sb += B) {
            if (sb > 0) {
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    const int32_t s = sb + u < nmine ? s0 + sb + u : s0;
                    const int32_t c = a.seg_cnt[g.slot0 + (int64_t)s * g.slot_step];
                    ck[u] = sb + u < nmine ? c : 0;
                }
            }
            int32_t e0[B], e1[B];
            int64_t p = at;
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int32_t *src =
                    a.seg_list + (g.slot0 + (int64_t)(s0 + sb + u) * g.slot_step) * kSegCap;
                const bool ok = ck[u] > 0 && ck[u] <= kSegCap && p < a.cap;
                e0[u] = ok ? src[0] : 0;
                e1[u] = ok && ck[u] > 1 && p + 1 < a.cap ? src[1] : 0;
                p += ck[u];
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int32_t c = ck[u];
                if (c > 0 && at < a.cap) {
                    const int64_t take = (int64_t)c < a.cap - at ? c : a.cap - at;
                    if (c <= kSegCap) {
                        row[at] = e0[u];
                        if (take > 1) row[at + 1] = e1[u];
                        if (take > 2) copy_segment(a, g, b, i, s0 + sb + u, c, 2, take, row + at);
                    } else {
                        copy_segment(a, g, b, i, s0 + sb + u, c, 0, take, row + at);
                    }
                }
                at += c;
            }
        }
        if (tid == 0) {
            a.acc[b] = v[0];
            a.acc[a.n_i + b] = v[1];
            a.acc[2 * (int64_t)a.n_i + b] = v[2];
            a.jerk[b] = v[3];
            a.jerk[a.n_i + b] = v[4];
            a.jerk[2 * (int64_t)a.n_i + b] = v[5];
            a.nb_count[b] = (int32_t)total;
            ovf = total > a.cap;
            nonfin = !finite6(v[0], v[1], v[2], v[3], v[4], v[5]);
            if (a.redo_k > 0.0 &&
                needs_redo(a.redo_k, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]))
                redo_push(a, b, g.j_begin, g.j_end);
        }
    } else if (tid == 0) {
        for (int k = 0; k < 3; ++k) {
            a.acc[(int64_t)k * a.n_i + b] = 0.0;
            a.jerk[(int64_t)k * a.n_i + b] = 0.0;
        }
        a.nb_count[b] = 0;
    }
    flush_flags(a, ovf, bad && tid == 0, nonfin);
}

}  // namespace nb
