// Device-side ray set-up and Siddon walk shared by every projector kernel
// (P, the two P^T strategies, the crossing counter and the trace export), so
// that all of them produce bit-identical segments.  See siddon.hip for the
// design notes.
#pragma once

#include <math.h>

#include "common.h"

namespace tomo {

struct RayState {
    double s[3];   // next crossing on each axis (ray parameter from the entry)
    double ds[3];  // parameter spacing of consecutive planes on each axis
    double send;   // exit parameter
    double dn;     // |d|: converts parameter differences to lengths
    int32_t off;   // flat offset of the current voxel within its frame
    int32_t st[3]; // signed flat stride of a step on each axis
};

// LDS byte address of a pointer into shared memory, and a read at such an
// address: a walk that carries its table entry as an address needs no shift
// or base add per step.
__device__ inline uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)p;
}
__device__ inline uint32_t lds_read_u32(uint32_t a)
{
    return *(__attribute__((address_space(3))) const uint32_t *)(uintptr_t)a;
}

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// n / d from a reciprocal inv ~ 1/d and one residual correction: the
// residual n - q d is exact in FP64 (fma), and q + r inv lands on the exactly
// rounded quotient whenever that quotient is representable, and within an
// ulp otherwise.  So equal quotients from equal data stay equal (ties
// between axes, entries exactly on a plane) at a fraction of a division.
__device__ inline double qdiv(double n, double d, double inv)
{
    const double q = n * inv;
    return fma(fma(-q, d, n), inv, q);
}

// 1 / d from v_rcp_f64 and two Newton steps (five instructions against the
// IEEE division's eleven); measured equal to the correctly rounded
// reciprocal on 2^22 random normal inputs.  qdiv only needs it within an ulp.
// Magnitudes near the ends of the exponent range take the IEEE division.
__device__ inline double recip(double d)
{
    const double a = fabs(d);
    if (a > 0x1p-1000 && a < 0x1p1000) {
        double r = __builtin_amdgcn_rcp(d);
        r = fma(r, fma(-d, r, 1.0), r);
        return fma(r, fma(-d, r, 1.0), r);
    }
    return 1.0 / d;
}

// Line of sight through pixel (col, row): gnomonic pinhole d = w + x u + y v.
// Returns false if the half-line misses the (half-open) box.
// Per-axis entry state, for kernels that need voxel coordinates.
struct RayAxes {
    int idx[3];     // entry voxel index on each axis
    int k0[3];      // index of the first plane crossed on each axis (after the entry)
    double tin;     // ray parameter of the entry point
    double rds[3];  // ~1 / (spacing) before its rounding to the grid (0: axis not crossed)
};

// kObstacle = false leaves out the obstacle's code (only for grids without
// one); true cuts the ray at the obstacle when the grid has one.  V is any
// view record with the pointing fields of ViewDev (o, w, u, v, cd, cp).
template <bool kObstacle = true, class V>
__device__ inline bool ray_setup(const GridDev &g, const V &v, int col, int row,
                                 RayState &r, RayAxes *ax = nullptr)
{
    const double x = ((double)col - v.cp[0]) * v.cd[0];
    const double y = ((double)row - v.cp[1]) * v.cd[1];
    double d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) d[a] = v.w[a] + x * v.u[a] + y * v.v[a];
    r.dn = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);

    // slab clip of t >= 0 against the box (one division per axis, the
    // other quotients from its reciprocal)
    double inv[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) inv[a] = d[a] != 0.0 ? recip(d[a]) : 0.0;
    double tin = 0.0, tout = kFar;
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (d[a] != 0.0) {
            const double t1 = qdiv(g.lo[a] - v.o[a], d[a], inv[a]);
            const double t2 = qdiv(g.hi[a] - v.o[a], d[a], inv[a]);
            tin = fmax(tin, fmin(t1, t2));
            tout = fmin(tout, fmax(t1, t2));
        } else {
            inside = inside && (g.lo[a] <= v.o[a]) && (v.o[a] < g.hi[a]);
        }
    }
    if (!inside || !(tout > tin)) return false;

    int idx[3];
    double sf[3], ds[3], jface[3];
    const int32_t stride[3] = {1, g.n[0], g.n[0] * g.n[1]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int N = g.n[a];
        if (d[a] != 0.0) {
            // voxel entered first: half-open voxels, so a ray starting on a
            // plane belongs to the voxel on the side it moves into
            const double p = qdiv(v.o[a] + tin * d[a] - g.lo[a], g.delta[a], g.inv_delta[a]);
            const bool up = d[a] > 0.0;
            int i = up ? clampi((int)floor(p), 0, N - 1) : clampi((int)ceil(p) - 1, 0, N - 1);
            const double k0 = up ? (double)(i + 1) : (double)i;  // first plane ahead
            sf[a] = qdiv(g.lo[a] + k0 * g.delta[a] - v.o[a], d[a], inv[a]) - tin;
            ds[a] = qdiv(g.delta[a], fabs(d[a]), fabs(inv[a]));
            jface[a] = up ? (double)N - k0 : k0;  // crossings to reach the far face
            int kplane = (int)k0;
            if (sf[a] <= 0.0) {  // rounding put the entry just before plane k0
                i = clampi(i + (up ? 1 : -1), 0, N - 1);
                sf[a] += ds[a];
                jface[a] -= 1.0;
                kplane += up ? 1 : -1;
            }
            idx[a] = i;
            if (ax) {
                ax->k0[a] = kplane;
                ax->rds[a] = fabs(d[a]) * g.inv_delta[a];
            }
            r.st[a] = up ? stride[a] : -stride[a];
        } else {
            // an observer exactly on a plane (k delta from the face) gives k,
            // the voxel above it
            idx[a] = clampi((int)floor(qdiv(v.o[a] - g.lo[a], g.delta[a], g.inv_delta[a])), 0, N - 1);
            if (ax) {
                ax->k0[a] = 0;
                ax->rds[a] = 0.0;
            }
            sf[a] = kFar;
            ds[a] = 0.0;
            jface[a] = 0.0;
            r.st[a] = 0;
        }
    }
    // Only values up to ~3 chords are ever compared: an axis whose first
    // crossing lies beyond 2 chords is never crossed, and a spacing above
    // 2 chords means at most one crossing, so both are capped.  Then every
    // value the walk forms is below span = 4 chords, and a power-of-two grid
    // q with span < 2^51 q makes all the additions exact.
    const double chord = tout - tin, lim = 2.0 * chord;
    int ex = 0;
    (void)frexp(4.0 * chord, &ex);  // 4 chord < 2^ex
    double send = kFar;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (d[a] != 0.0 && sf[a] <= lim) {
            ds[a] = ldexp(rint(ldexp(fmin(ds[a], lim), 51 - ex)), ex - 51);
            sf[a] = ldexp(rint(ldexp(sf[a], 51 - ex)), ex - 51);
            send = fmin(send, sf[a] + jface[a] * ds[a]);
        } else {
            sf[a] = kFar;
            ds[a] = 0.0;
        }
        r.s[a] = sf[a];
        r.ds[a] = ds[a];
    }
    if (kObstacle && g.has_sph) {
        // the obstacle: the line of sight ends where it enters the sphere's
        // interior, found from the closest approach t* of the line to the
        // centre (at distance h): t* - sqrt((R^2 - h^2) / d.d); the end is
        // put on the ray's grid, so that every walk stops at the same value
        double oc[3], dd = 0.0, od = 0.0, oo = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            oc[a] = v.o[a] - g.sph[a];
            dd = fma(d[a], d[a], dd);
            od = fma(oc[a], d[a], od);
            oo = fma(oc[a], oc[a], oo);
        }
        const double r2 = g.sph[3] * g.sph[3];
        if (oo <= r2) return false;  // observer on or inside the sphere
        if (od < 0.0) {
            const double ts = -od / dd;
            double h2 = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double p = fma(ts, d[a], oc[a]);
                h2 = fma(p, p, h2);
            }
            if (h2 < r2) {
                const double tc = ts - sqrt((r2 - h2) / dd) - tin;  // from the entry
                send = fmin(send, ldexp(rint(ldexp(tc, 51 - ex)), ex - 51));
            }
        }
    }
    if (!(send > 0.0) || !(send < kFar)) return false;
    r.send = send;
    r.off = (idx[2] * g.n[1] + idx[1]) * g.n[0] + idx[0];
    if (ax) {
        for (int a = 0; a < 3; ++a) ax->idx[a] = idx[a];
        ax->tin = tin;
    }
    return true;
}

// Stores the set-up of pixel i (ok: ray_setup's result) into a ray table's
// columns d and index words k, n rows each.  Every field is written, also
// for a ray that misses (send = 0), so the table's contents depend on the
// geometry alone.
__device__ inline void ray_table_put(double *__restrict__ d, uint64_t *__restrict__ k, int64_t n, int64_t i,
                                     bool ok, const RayState &r, const RayAxes &ax)
{
    uint64_t w = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        d[a * n + i] = ok ? r.s[a] : 0.0;
        d[(3 + a) * n + i] = ok ? r.ds[a] : 0.0;
        d[(8 + a) * n + i] = ok ? ax.rds[a] : 0.0;
        if (ok) {
            w |= (uint64_t)(uint32_t)ax.idx[a] << (kRayTableSideBits * a);
            if (r.st[a] > 0) w |= 1ull << (60 + a);
        }
    }
    d[6 * n + i] = ok ? r.send : 0.0;
    d[7 * n + i] = ok ? r.dn : 0.0;
    k[i] = w;
}

// Row i of a ray table as loaded, and what a walk from it starts with (r's s,
// ds, st = +-1 or 0, send, dn and ax.idx, ax.rds), bit for bit as ray_setup
// left them.  False: the ray misses the box.  Apart, so that a row can be
// loaded well before it is used.
struct RayRow {
    double d[kRayTableCols];
    uint64_t k;
};
__device__ inline RayRow ray_table_load(const RayTable &t, int64_t i)
{
    RayRow w;
#pragma unroll
    for (int c = 0; c < kRayTableCols; ++c) w.d[c] = t.d[c * t.n + i];
    w.k = t.k[i];
    return w;
}
__device__ inline bool ray_table_take(const RayRow &w, RayState &r, RayAxes &ax)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.s[a] = w.d[a];
        r.ds[a] = w.d[3 + a];
        ax.rds[a] = w.d[8 + a];
        ax.idx[a] = (int)((w.k >> (kRayTableSideBits * a)) & ((1u << kRayTableSideBits) - 1u));
        r.st[a] = r.ds[a] == 0.0 ? 0 : (((w.k >> (60 + a)) & 1u) ? 1 : -1);
    }
    r.send = w.d[6];
    r.dn = w.d[7];
    return r.send > 0.0;
}

// Advances every axis whose next crossing is m: s[a] += ds[a] and o += st[a]
// where s[a] == m (exact on the common grid), the others left alone.  Written
// under the execution mask (v_cmpx), three VALU instructions per axis, against
// five for the same update by selects (a compare, a 0/1 factor and an FMA, a
// select and an add), which the compiler makes of the plain condition; the
// mask is saved and restored by scalar moves, which issue beside other waves'
// VALU instructions.
__device__ inline void advance(double (&s)[3], const double (&ds)[3], double m, uint32_t &o, const uint32_t (&st)[3])
{
    uint64_t sv;
    asm("s_mov_b64 %[sv], exec\n\t"
        "v_cmpx_eq_f64_e32 vcc, %[s0], %[m]\n\t"
        "v_add_f64 %[s0], %[s0], %[d0]\n\t"
        "v_add_u32_e32 %[o], %[o], %[t0]\n\t"
        "s_mov_b64 exec, %[sv]\n\t"
        "v_cmpx_eq_f64_e32 vcc, %[s1], %[m]\n\t"
        "v_add_f64 %[s1], %[s1], %[d1]\n\t"
        "v_add_u32_e32 %[o], %[o], %[t1]\n\t"
        "s_mov_b64 exec, %[sv]\n\t"
        "v_cmpx_eq_f64_e32 vcc, %[s2], %[m]\n\t"
        "v_add_f64 %[s2], %[s2], %[d2]\n\t"
        "v_add_u32_e32 %[o], %[o], %[t2]\n\t"
        "s_mov_b64 exec, %[sv]"
        : [s0] "+&v"(s[0]), [s1] "+&v"(s[1]), [s2] "+&v"(s[2]), [o] "+&v"(o), [sv] "=&s"(sv)
        : [m] "v"(m), [d0] "v"(ds[0]), [d1] "v"(ds[1]), [d2] "v"(ds[2]), [t0] "v"(st[0]), [t1] "v"(st[1]),
          [t2] "v"(st[2])
        : "vcc");
}

// The same with one position per axis: i[a] += st[a] where s[a] == m.
__device__ inline void advance(double (&s)[3], const double (&ds)[3], double m, uint32_t (&i)[3],
                               const uint32_t (&st)[3])
{
    uint64_t sv;
    asm("s_mov_b64 %[sv], exec\n\t"
        "v_cmpx_eq_f64_e32 vcc, %[s0], %[m]\n\t"
        "v_add_f64 %[s0], %[s0], %[d0]\n\t"
        "v_add_u32_e32 %[i0], %[i0], %[t0]\n\t"
        "s_mov_b64 exec, %[sv]\n\t"
        "v_cmpx_eq_f64_e32 vcc, %[s1], %[m]\n\t"
        "v_add_f64 %[s1], %[s1], %[d1]\n\t"
        "v_add_u32_e32 %[i1], %[i1], %[t1]\n\t"
        "s_mov_b64 exec, %[sv]\n\t"
        "v_cmpx_eq_f64_e32 vcc, %[s2], %[m]\n\t"
        "v_add_f64 %[s2], %[s2], %[d2]\n\t"
        "v_add_u32_e32 %[i2], %[i2], %[t2]\n\t"
        "s_mov_b64 exec, %[sv]"
        : [s0] "+&v"(s[0]), [s1] "+&v"(s[1]), [s2] "+&v"(s[2]), [i0] "+&v"(i[0]), [i1] "+&v"(i[1]),
          [i2] "+&v"(i[2]), [sv] "=&s"(sv)
        : [m] "v"(m), [d0] "v"(ds[0]), [d1] "v"(ds[1]), [d2] "v"(ds[2]), [t0] "v"(st[0]), [t1] "v"(st[1]),
          [t2] "v"(st[2])
        : "vcc");
}

// The parameter of the walk's next event.  Without an obstacle the exit is
// itself the crossing of the box's far face, which the exact increments
// reach, so the three crossings bound it.
template <bool kObstacle>
__device__ inline double next_event(const double (&s)[3], double send)
{
    const double m = fmin(s[0], s[1]);
    return kObstacle ? fmin(m, fmin(s[2], send)) : fmin(m, s[2]);
}

// Walk the ray voxel by voxel.  visit(off, dl) receives the flat voxel
// offset and the parameter length of the segment (length = dl * |d|).
// Simultaneous crossings advance every tied axis in one step.  maxit bounds
// the loop whatever the arithmetic does; the loop body holds four steps, so
// the bound is tested once per four (it may run up to three steps past it).
template <class Visit>
__device__ inline void ray_walk(RayState &r, int maxit, Visit &&visit)
{
    double scur = 0.0;
    uint32_t o = (uint32_t)r.off;
    const uint32_t st[3] = {(uint32_t)r.st[0], (uint32_t)r.st[1], (uint32_t)r.st[2]};
    auto step = [&]() {  // true once the ray has ended
        const double m = next_event<true>(r.s, r.send);
        visit((int32_t)o, m - scur);
        advance(r.s, r.ds, m, o, st);
        scur = m;
        return m >= r.send;
    };
    for (int it = 0; it < maxit; it += 4) {
        if (step() || step() || step() || step()) break;
    }
}

// Sum over the ray's segments of length x voxel value, in parameter units:
// load(pos) issues the gather of the voxel at pos (an offset, or one position
// per axis; st its steps) and value(.) turns what it loaded into the voxel's
// value.  Pipelined by one segment: a step issues its voxel's gather before
// it adds the previous segment, so two gathers are in flight per lane and
// each has a whole step to land.  The two pending segments alternate between
// the names a and b, and a lane that ends keeps both as they are, so no
// register is copied (and no gather waited for) at the loop's back edge.
template <bool kObstacle, class Pos, class Step, class Load, class Value>
__device__ inline double ray_integrate(RayState &r, int maxit, Pos &pos, const Step &st, Load &&load, Value &&value)
{
    using T = decltype(load(pos));
    double acc = 0.0, scur = 0.0, da = 0.0, db = 0.0;
    T xa{}, xb{};
    bool a_last = false;
    auto step = [&](T &x, double &d, const T &x_prev, const double &d_prev) {  // true once the ray has ended
        const double m = next_event<kObstacle>(r.s, r.send);
        x = load(pos);
        d = m - scur;
        advance(r.s, r.ds, m, pos, st);
        scur = m;
        acc = fma(d_prev, value(x_prev), acc);
        return m >= r.send;
    };
    for (int it = 0; it < maxit; it += 4) {
        a_last = true;
        if (step(xa, da, xb, db)) break;
        a_last = false;
        if (step(xb, db, xa, da)) break;
        a_last = true;
        if (step(xa, da, xb, db)) break;
        a_last = false;
        if (step(xb, db, xa, da)) break;
    }
    return a_last ? fma(da, value(xa), acc) : fma(db, value(xb), acc);
}

// 1.0 if t else 0.0: only the high word differs, so one select; fma(ds, f,
// s) then equals s + ds or s exactly.
__device__ inline double tie_factor(bool t)
{
    return __builtin_bit_cast(double, (uint64_t)(t ? 0x3FF00000u : 0u) << 32);
}

// Sum over the ray's segments of length x voxel value, in parameter units, for
// launches of a few wavefronts a SIMD (XWalk::few): the axes are updated by
// selects, which do not depend on each other as updates under the mask do, and
// two gathers are in flight per lane.  23 VALU instructions a step.
template <class Load>
__device__ inline double ray_integrate_few(RayState &r, int maxit, uint32_t pos, const uint32_t (&st)[3], Load &&load)
{
    double acc = 0.0, dl_prev = 0.0, scur = 0.0;
    float x_prev = 0.0f;
    auto step = [&]() {  // true once the ray has ended
        const double m = fmin(fmin(r.s[0], r.s[1]), fmin(r.s[2], r.send));
        const uint32_t o = pos;
        const double dl = m - scur;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const bool t = (r.s[a] == m);
            r.s[a] = fma(r.ds[a], tie_factor(t), r.s[a]);  // s + ds or s, exact on the common grid
            pos += t ? st[a] : 0u;
        }
        scur = m;
        const float x = load(o);
        acc = fma(dl_prev, (double)x_prev, acc);
        x_prev = x;
        dl_prev = dl;
        return m >= r.send;
    };
    for (int it = 0; it < maxit; it += 4) {
        if (step() || step() || step() || step()) break;
    }
    return fma(dl_prev, (double)x_prev, acc);
}

// ---- the two hot walks of P as one machine loop each.  What the compiler
// makes of ray_integrate keeps the four exits of a body apart with mask
// arithmetic, register copies and a wait for the newest gather; here a step
// is fifteen VALU instructions and its gather (and, for bricked offsets, an
// add and three LDS reads, each issued as soon as its axis' position is
// known).  A step adds the segment of three steps before, so four gathers are
// in flight per lane.  A lane that ends leaves the execution mask by the
// compare that finds its end; the step's exit block, out of the loop's way,
// adds the segments such lanes still have pending, oldest first.  Every load
// is waited for inside the block.
// Bound by VALU issue where lines of sight are dense (128^3 under 28 x 512^2
// from 4^3 bricks: 0.505 ms, 0.87 of the issue ceiling; 23 to 26.5 VALU per
// step and 0.76 ms from the x-fastest cube before), by L2 where they are as far
// apart as voxels (256^3 under 64 x 256^2: 1.37 ms, 22 GB of lines from L2; 4.64
// ms x-fastest).  One gather in flight less: 5% slower there, even elsewhere.
// The loop starts 16 bytes past a 64-byte line: where a SIMD has one or two
// wavefronts, the instruction fetch shows, and a start at a multiple of 32 bytes
// is slower (x-fastest, offsets 0 / 8 / 16 / 24 / 32 / 48: 160x170x150 under one
// view of 300x200 19.9 / 18.2 / 18.3 / 18.7 / 19.9 / 18.1 us; 92x103x82 under
// 98x58 19.2 / 17.5 / 17.6 / 18.0 / 19.2 / 17.6).
//
// Axis A's update where its crossing is the event M.  TERM reads the axis'
// offset term for the next step.
#define TOMO_AXIS(A, P, M, TERM)                        \
    "v_cmpx_eq_f64_e32 vcc, %[s" A "], %[" M "]\n\t"    \
    "v_add_f64 %[s" A "], %[s" A "], %[d" A "]\n\t"     \
    "v_add_u32_e32 %[" P "], %[" P "], %[t" A "]\n\t"   \
    "s_mov_b64 exec, %[sv]\n\t" TERM(A)
// The same for the axis the lines of sight cross least (z: observers sit near
// the ecliptic): the update is stepped over while no lane of the wave crosses.
#define TOMO_AXIS_RARE(A, P, M, TERM, K)                \
    "v_cmpx_eq_f64_e32 vcc, %[s" A "], %[" M "]\n\t"    \
    "s_cbranch_execz .Ltomo_skip" K "_%=\n\t"           \
    "v_add_f64 %[s" A "], %[s" A "], %[d" A "]\n\t"     \
    "v_add_u32_e32 %[" P "], %[" P "], %[t" A "]\n"     \
    ".Ltomo_skip" K "_%=:\n\t"                          \
    "s_mov_b64 exec, %[sv]\n\t" TERM(A)
// Adds segment Q (length e<Q>, voxel x<Q>) to the sum.
#define TOMO_ADD(Q)                                     \
    "v_cvt_f64_f32_e32 %[cv], %[x" Q "]\n\t"            \
    "v_fma_f64 %[acc], %[e" Q "], %[cv], %[acc]\n\t"
// Step K (0..3): the event's parameter M (the previous one's in MP), segment
// K's gather and length; segment O, the oldest, is added.  MIN: the exit joins
// the minimum (obstacle).
#define TOMO_STEP(K, O, M, MP, MIN, LOAD, TERM, P0, P1, P2)          \
    "v_min_f64 %[" M "], %[s0], %[s1]\n\t"                           \
    "v_min_f64 %[" M "], %[" M "], %[s2]\n\t" MIN(M) LOAD("x" K)     \
    "v_add_f64 %[e" K "], %[" M "], -%[" MP "]\n\t"                  \
    "s_waitcnt vmcnt(3)\n\t" TOMO_ADD(O)                             \
    "v_cmpx_lt_f64_e32 vcc, %[" M "], %[send]\n\t"                   \
    "s_andn2_b64 %[tm], %[sv], exec\n\t"                             \
    "s_cbranch_scc1 .Ltomo_exit" K "_%=\n"                           \
    ".Ltomo_go" K "_%=:\n\t"                                         \
    "s_mov_b64 %[sv], exec\n\t"                                      \
    TOMO_AXIS("0", P0, M, TERM) TOMO_AXIS("1", P1, M, TERM) TOMO_AXIS_RARE("2", P2, M, TERM, K)
// Exit block of step K for the lanes in tm: segments A, B and K.
#define TOMO_EXIT(K, A, B)                              \
    ".Ltomo_exit" K "_%=:\n\t"                          \
    "s_mov_b64 %[sv], exec\n\t"                         \
    "s_mov_b64 exec, %[tm]\n\t"                         \
    "s_waitcnt vmcnt(0)\n\t"                            \
    TOMO_ADD(A) TOMO_ADD(B) TOMO_ADD(K)                 \
    "s_mov_b64 exec, %[sv]\n\t"                         \
    "s_cbranch_execz .Ltomo_end_%=\n\t"                 \
    "s_branch .Ltomo_go" K "_%=\n"
#define TOMO_MIN_NONE(M) ""
#define TOMO_MIN_EXIT(M) "v_min_f64 %[" M "], %[" M "], %[send]\n\t"
#define TOMO_TERM_NONE(A) ""
#define TOMO_TERM_BRICK(A) "ds_read_b32 %[l" A "], %[p" A "]\n\t"
#define TOMO_LOAD_FLAT(X) "buffer_load_dword %[" X "], %[p0], %[rs], 0 offen\n\t"
#define TOMO_LOAD_BRICK(X)                              \
    "s_waitcnt lgkmcnt(0)\n\t"                          \
    "v_add3_u32 %[l0], %[l0], %[l1], %[l2]\n\t"         \
    "buffer_load_dword %[" X "], %[l0], %[rs], 0 offen\n\t"
#define TOMO_WALK(MIN, LOAD, TERM, P0, P1, P2)                    \
    "s_mov_b64 %[en], exec\n\t"                                   \
    "s_mov_b64 %[sv], exec\n\t" TERM("0") TERM("1") TERM("2")     \
    "\n\t.p2align 6\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n" \
    ".Ltomo_walk_%=:\n\t"                                         \
    TOMO_STEP("0", "1", "ma", "mb", MIN, LOAD, TERM, P0, P1, P2)  \
    TOMO_STEP("1", "2", "mb", "ma", MIN, LOAD, TERM, P0, P1, P2)  \
    TOMO_STEP("2", "3", "ma", "mb", MIN, LOAD, TERM, P0, P1, P2)  \
    TOMO_STEP("3", "0", "mb", "ma", MIN, LOAD, TERM, P0, P1, P2)  \
    "s_sub_u32 %[cnt], %[cnt], 1\n\t"                             \
    "s_cmp_lg_u32 %[cnt], 0\n\t"                                  \
    "s_cbranch_scc1 .Ltomo_walk_%=\n\t"                           \
    "s_branch .Ltomo_end_%=\n"                                    \
    TOMO_EXIT("0", "2", "3") TOMO_EXIT("1", "3", "0")             \
    TOMO_EXIT("2", "0", "1") TOMO_EXIT("3", "1", "2")             \
    ".Ltomo_end_%=:\n\t"                                          \
    "s_mov_b64 exec, %[en]\n\t"                                   \
    "s_waitcnt vmcnt(0) lgkmcnt(0)"

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Words of a raw buffer resource over [base, base + bytes), uniform.
__device__ inline u32x4 rsrc_words(const void *base, uint32_t bytes)
{
    const uint64_t b = (uint64_t)(uintptr_t)base;
    u32x4 w;
    w.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    w.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(b >> 32) & 0xffffu));
    w.z = (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes);
    w.w = 0x00020000u;
    return w;
}

// ray_integrate over FP32 gathers at byte offset pos (kBrick false) or at the
// sum of three LDS table entries at the addresses pos[0..2] (kBrick true).
template <bool kObstacle, bool kBrick>
__device__ inline double ray_integrate_buffer(RayState &r, int maxit, uint32_t (&pos)[3], const uint32_t (&st)[3],
                                              u32x4 rs)
{
    double acc = 0.0, ma, mb = 0.0, cv, e0, e1 = 0.0, e2 = 0.0, e3 = 0.0;
    float x0, x1 = 0.0f, x2 = 0.0f, x3 = 0.0f;
    uint32_t l0, l1, l2, cnt = (uint32_t)(maxit + 3) >> 2;
    uint64_t en, sv, tm;
#define TOMO_ASM(MIN, LOAD, TERM, P0, P1, P2)                                                                       \
    asm volatile(TOMO_WALK(MIN, LOAD, TERM, P0, P1, P2)                                                             \
                 : [s0] "+&v"(r.s[0]), [s1] "+&v"(r.s[1]), [s2] "+&v"(r.s[2]), [p0] "+&v"(pos[0]),                  \
                   [p1] "+&v"(pos[1]), [p2] "+&v"(pos[2]), [acc] "+&v"(acc), [e0] "=&v"(e0), [e1] "+&v"(e1),        \
                   [e2] "+&v"(e2), [e3] "+&v"(e3), [x0] "=&v"(x0), [x1] "+&v"(x1), [x2] "+&v"(x2), [x3] "+&v"(x3),  \
                   [ma] "=&v"(ma), [mb] "+&v"(mb), [cv] "=&v"(cv), [l0] "=&v"(l0), [l1] "=&v"(l1), [l2] "=&v"(l2),  \
                   [cnt] "+&s"(cnt), [en] "=&s"(en), [sv] "=&s"(sv), [tm] "=&s"(tm)                                 \
                 : [d0] "v"(r.ds[0]), [d1] "v"(r.ds[1]), [d2] "v"(r.ds[2]), [t0] "v"(st[0]), [t1] "v"(st[1]),       \
                   [t2] "v"(st[2]), [send] "v"(r.send), [rs] "s"(rs)                                                \
                 : "vcc", "scc", "memory")
    if constexpr (kBrick) {
        if constexpr (kObstacle) TOMO_ASM(TOMO_MIN_EXIT, TOMO_LOAD_BRICK, TOMO_TERM_BRICK, "p0", "p1", "p2");
        else TOMO_ASM(TOMO_MIN_NONE, TOMO_LOAD_BRICK, TOMO_TERM_BRICK, "p0", "p1", "p2");
    } else {
        if constexpr (kObstacle) TOMO_ASM(TOMO_MIN_EXIT, TOMO_LOAD_FLAT, TOMO_TERM_NONE, "p0", "p0", "p0");
        else TOMO_ASM(TOMO_MIN_NONE, TOMO_LOAD_FLAT, TOMO_TERM_NONE, "p0", "p0", "p0");
    }
#undef TOMO_ASM
    return acc;
}

// Tile -> (view, pixel of this lane).  Views are sorted by tile_off.
struct LanePixel {
    int view;
    int col, row;
};

// kCurve: the lanes of an 8x8 bundle along a Z-order curve (walks from bricks)
// instead of by rows.
template <bool kCurve = false>
__device__ inline LanePixel lane_pixel(const ViewDev *__restrict__ views, int nviews, int64_t tile,
                                       int log2_bw)
{
    int lo = 0, hi = nviews - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile_off <= tile) lo = mid;
        else hi = mid - 1;
    }
    const int64_t t = tile - views[lo].tile_off;
    const int tpr = views[lo].tiles_x;
    const int tx = (int)(t % tpr), ty = (int)(t / tpr);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    LanePixel lp;
    lp.view = lo;
    if (log2_bw == 0) {  // 8x8 lanes at a 2-pixel pitch, wavefront w offset by (w&1, w>>1)
        lp.col = tx * kTile + (l & 7) * 2 + (w & 1);
        lp.row = ty * kTile + (l >> 3) * 2 + (w >> 1);
        return lp;
    }
    if (kCurve && log2_bw == 3) {
        const int x = (l & 1) | ((l >> 1) & 2) | ((l >> 2) & 4), y = ((l >> 1) & 1) | ((l >> 2) & 2) | ((l >> 3) & 4);
        lp.col = tx * kTile + (w & 1) * 8 + x;
        lp.row = ty * kTile + (w >> 1) * 8 + y;
        return lp;
    }
    const int bw = 1 << log2_bw, bh = 64 >> log2_bw;
    const int wpr = kTile >> log2_bw;  // wave bundles per tile row
    lp.col = tx * kTile + (w % wpr) * bw + (l & (bw - 1));
    lp.row = ty * kTile + (w / wpr) * bh + (l >> log2_bw);
    return lp;
}

template <int64_t kRun = 64>
__device__ inline int64_t block_tile(const Bundle &b)
{
    return xcd_order<kRun>(b.xcd_remap, blockIdx.x, gridDim.x);
}

// P for one 16x16 tile (all threads of the workgroup): each lane's pixel =
// sum over its ray's segments of length x voxel value, written to images.
// kWalk: four and few address a frame below 2^29 voxels by byte offsets; two,
// and the walk that tests the map mask, take every frame.
template <bool kMapMask, bool kDataMask, bool kObstacle, XWalk kWalk>
__device__ inline void project_tile(const GridDev &g, const ViewDev *__restrict__ views, int32_t nviews,
                                    int log2_bw, int64_t tile, int32_t maxit,
                                    const float *__restrict__ cube, const uint8_t *__restrict__ map_mask,
                                    const uint8_t *__restrict__ data_mask, float *__restrict__ images)
{
    const LanePixel lp = lane_pixel(views, nviews, tile, log2_bw);
    const ViewDev &v = views[lp.view];
    if (lp.col >= v.ncol || lp.row >= v.nrow) return;
    const int64_t pix = v.pix_off + (int64_t)lp.row * v.ncol + lp.col;
    float out = 0.0f;
    RayState r;
    if ((!kDataMask || data_mask[pix]) && ray_setup<kObstacle>(g, v, lp.col, lp.row, r)) {
        const float *__restrict__ base = cube + (int64_t)v.frame * g.nvox;
        double acc;
        if constexpr (!kMapMask && kWalk != XWalk::two) {
            const uint32_t st[3] = {(uint32_t)r.st[0] * 4u, (uint32_t)r.st[1] * 4u, (uint32_t)r.st[2] * 4u};
            if constexpr (kWalk == XWalk::few) {
                const auto rc = make_rsrc(base, (uint32_t)(g.nvox * 4));
                acc = ray_integrate_few(r, maxit, (uint32_t)r.off * 4u, st,
                                        [&](uint32_t o) { return buf_load_f32(rc, o); });
            } else {
                uint32_t pos[3] = {(uint32_t)r.off * 4u, 0u, 0u};
                acc = ray_integrate_buffer<kObstacle, false>(r, maxit, pos, st,
                                                             rsrc_words(base, (uint32_t)(g.nvox * 4)));
            }
        } else {
            // a buffer resource spans below 2^32 bytes: a frame of 2^30 voxels
            // takes plain global loads, their offsets clamped into the frame as
            // the buffer's range check would
            const bool wide = g.nvox >= ((int64_t)1 << 30);
            const uint32_t last = (uint32_t)(g.nvox - 1);
            const auto rc = make_rsrc(base, wide ? 0u : (uint32_t)(g.nvox * 4));
            uint32_t pos = (uint32_t)r.off;
            const uint32_t st[3] = {(uint32_t)r.st[0], (uint32_t)r.st[1], (uint32_t)r.st[2]};
            if constexpr (kMapMask) {
                const auto rm = make_rsrc(map_mask, (uint32_t)g.nvox);
                struct Masked {
                    float x;
                    uint32_t keep;
                };
                const auto kept = [](const Masked &t) { return t.keep ? (double)t.x : 0.0; };
                if (wide)
                    acc = ray_integrate<kObstacle>(
                        r, maxit, pos, st, [&](uint32_t o) { return Masked{base[min(o, last)], buf_load_u8(rm, o)}; },
                        kept);
                else
                    acc = ray_integrate<kObstacle>(
                        r, maxit, pos, st,
                        [&](uint32_t o) { return Masked{buf_load_f32(rc, o * 4u), buf_load_u8(rm, o)}; }, kept);
            } else {
                const auto plain = [](float x) { return (double)x; };
                if (wide)
                    acc = ray_integrate<kObstacle>(r, maxit, pos, st, [&](uint32_t o) { return base[min(o, last)]; },
                                                   plain);
                else
                    acc = ray_integrate<kObstacle>(r, maxit, pos, st,
                                                   [&](uint32_t o) { return buf_load_f32(rc, o * 4u); }, plain);
            }
        }
        out = (float)(acc * (r.dn * v.gain));
    }
    images[pix] = out;
}

// Offset of voxel (i0, i1, i2) in its frame of the bricked copy.
__device__ inline uint32_t brick_offset(const BrickDev &bk, int i0, int i1, int i2)
{
    const uint32_t m = (1u << bk.k) - 1u;
    const uint32_t brick = ((uint32_t)(i2 >> bk.k) * (uint32_t)bk.nb[1] + (uint32_t)(i1 >> bk.k)) * (uint32_t)bk.nb[0] +
                           (uint32_t)(i0 >> bk.k);
    return (brick << (3 * bk.k)) | (((uint32_t)i2 & m) << (2 * bk.k)) | (((uint32_t)i1 & m) << bk.k) |
           ((uint32_t)i0 & m);
}

// The bricked offset is a sum of one term per axis: brick_offset(i0, i1,
// i2) = f0(i0) + f1(i1) + f2(i2) with f_a(i) = (i >> k) S_a 2^3k + (i & m)
// 2^(k a), S = (1, nb0, nb0 nb1), since the brick index is linear in the
// per-axis brick coordinates and the in-brick bits do not overlap it.
__device__ inline uint32_t brick_axis_term(const BrickDev &bk, int a, int i)
{
    const uint32_t m = (1u << bk.k) - 1u;
    const uint32_t s = a == 0 ? 1u : (a == 1 ? (uint32_t)bk.nb[0] : (uint32_t)bk.nb[0] * (uint32_t)bk.nb[1]);
    return ((((uint32_t)i >> bk.k) * s) << (3 * bk.k)) + (((uint32_t)i & m) << (bk.k * a));
}

// P for one 16x16 tile from a bricked copy of M x (the map mask applied by
// the copy): the same walk as project_tile, the voxel indices carried per
// axis and the offset formed from them; the same segments summed in the
// same order, so the same bits.  With kLut the offset is the sum of three
// per-axis terms read from LDS (lut: f0 over the n0 x indices, then f1,
// then f2; in bytes unless kWide), one add and three LDS reads per step
// instead of the shifts, masks and multiplies of brick_offset.
template <bool kDataMask, bool kObstacle, bool kLut, bool kWide>
__device__ inline void project_tile_bricked(const GridDev &g, const ViewDev *__restrict__ views, int32_t nviews,
                                            int log2_bw, int64_t tile, int32_t maxit, const float *__restrict__ bricked,
                                            const BrickDev &bk, const uint8_t *__restrict__ data_mask,
                                            float *__restrict__ images, const uint32_t *lut = nullptr)
{
    const LanePixel lp = lane_pixel<true>(views, nviews, tile, log2_bw);
    const ViewDev &v = views[lp.view];
    if (lp.col >= v.ncol || lp.row >= v.nrow) return;
    const int64_t pix = v.pix_off + (int64_t)lp.row * v.ncol + lp.col;
    float out = 0.0f;
    RayState r;
    RayAxes ax;
    if ((!kDataMask || data_mask[pix]) && ray_setup<kObstacle>(g, v, lp.col, lp.row, r, &ax)) {
        const float *__restrict__ base = bricked + (int64_t)v.frame * bk.frame_stride;
        const uint32_t last = (uint32_t)(bk.frame_stride - 1);
        const auto rc = make_rsrc(base, kWide ? 0u : (uint32_t)(bk.frame_stride * 4));
        // positions per axis: the LDS address of the axis' offset term, or
        // the voxel index without a table
        uint32_t i[3], dir[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const uint32_t one = kLut ? 4u : 1u;
            const int tab0 = a == 0 ? 0 : (a == 1 ? g.n[0] : g.n[0] + g.n[1]);
            i[a] = kLut ? lds_address(lut) + 4u * (uint32_t)(tab0 + ax.idx[a]) : (uint32_t)ax.idx[a];
            dir[a] = r.st[a] > 0 ? one : (r.st[a] < 0 ? 0u - one : 0u);
        }
        // the kind of load is fixed per kernel (kWide: frames of 2^30 floats
        // and more, which a buffer resource cannot span)
        double acc;
        if constexpr (kLut && !kWide) {
            acc = ray_integrate_buffer<kObstacle, true>(r, maxit, i, dir,
                                                        rsrc_words(base, (uint32_t)(bk.frame_stride * 4)));
        } else {
            acc = ray_integrate<kObstacle>(
                r, maxit, i, dir,
                [&](const uint32_t (&p)[3]) {
                    const uint32_t off = kLut ? lds_read_u32(p[0]) + lds_read_u32(p[1]) + lds_read_u32(p[2])
                                              : brick_offset(bk, (int)p[0], (int)p[1], (int)p[2]);
                    return kWide ? base[min(off, last)] : buf_load_f32(rc, off * 4u);
                },
                [](float x) { return (double)x; });
        }
        out = (float)(acc * (r.dn * v.gain));
    }
    images[pix] = out;
}

}  // namespace tomo
