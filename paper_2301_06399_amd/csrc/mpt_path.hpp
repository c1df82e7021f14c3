// Device helpers shared by the solver kernels and the kernels around them:
// the bins of the orders, the start points, the guard box.
#pragma once
#include "mpt_internal.hpp"

namespace mpt {

__device__ inline int bin_offset(const int *cnt, int k)  // k = order 1..5
{
    int off = 0;
    for (int j = 1; j < k; j++) off += cnt[j - 1];
    return off;
}

// Uniform double in [0,1) from draw number c of SplitMix64 (Steele, Lea &
// Flood, OOPSLA 2014) started from state `seed`: the state after c+1
// golden-ratio increments, mixed, top 53 bits.
__device__ inline double splitmix_uniform(uint64_t seed, uint64_t c)
{
    uint64_t z = seed + (c + 1u) * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    return (double)(z >> 11) * 0x1.0p-53;
}

// Projection of a point onto an object (FP64 world): the straight-line start
// of each interaction is the projection of the point k/(N+1) of the way from
// TX to RX; the random start (Alg. 1) projects a point uniform in the scene
// box, draw 15 i + 3 k + axis for solve i.
__device__ inline void project(int t, const double *r, const double *P, double *X)
{
    if (t == TP) {
        const double f = r[0] * P[0] + r[1] * P[1] + r[2] * P[2] - r[3];
        for (int i = 0; i < 3; i++) X[i] = P[i] - f * r[i];
    } else if (t == TL) {
        const double s = (P[0] - r[0]) * r[3] + (P[1] - r[1]) * r[4] + (P[2] - r[2]) * r[5];
        for (int i = 0; i < 3; i++) X[i] = r[i] + s * r[3 + i];
    } else if (t == TQ) {
        // one Newton step towards f = 0 along grad f
        const double w[3] = {P[0] - r[0], P[1] - r[1], P[2] - r[2]};
        const double Aw0 = r[3] * w[0] + r[4] * w[1] + r[5] * w[2];
        const double Aw1 = r[4] * w[0] + r[6] * w[1] + r[7] * w[2];
        const double Aw2 = r[5] * w[0] + r[7] * w[1] + r[8] * w[2];
        const double f = w[0] * Aw0 + w[1] * Aw1 + w[2] * Aw2 + r[9] * w[0] + r[10] * w[1] + r[11] * w[2] + r[12];
        const double g[3] = {2.0 * Aw0 + r[9], 2.0 * Aw1 + r[10], 2.0 * Aw2 + r[11]};
        const double gg = g[0] * g[0] + g[1] * g[1] + g[2] * g[2];
        const double s = gg > 0.0 ? f / gg : 0.0;
        for (int i = 0; i < 3; i++) X[i] = P[i] - s * g[i];
    } else {
        const double d[3] = {P[0] - r[0], P[1] - r[1], P[2] - r[2]};
        const double h = d[0] * r[3] + d[1] * r[4] + d[2] * r[5];
        double w[3] = {d[0] - h * r[3], d[1] - h * r[4], d[2] - h * r[5]};
        double lw = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
        if (!(lw > 0.0)) {
            double u2[3];
            across_dir(r + 3, w, u2);
            lw = 1.0;
        }
        for (int i = 0; i < 3; i++) X[i] = r[i] + r[6] * w[i] / lw;
    }
}

__device__ inline bool in_guard(const SceneDev &s, const double *X, int n)
{
    bool ok = true;
    for (int k = 0; k < n; k++)
        for (int i = 0; i < 3; i++) ok = ok && (X[3 * k + i] >= s.glo[i]) && (X[3 * k + i] <= s.ghi[i]);
    return ok;
}

// A packed record in registers: what a straight edge has (its six first
// values), and of the other types the rest.  The kernels before and after the
// solver read the records of random objects, a cache line per lane, and are
// bound by those accesses: each record is read once, in 16-byte loads, instead
// of a few values wherever a branch needs them.
typedef double f64x2 __attribute__((ext_vector_type(2), aligned(16)));
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(8), may_alias));
typedef float f32x2 __attribute__((ext_vector_type(2), aligned(8), may_alias));

template <int J0, int J1>  // r[2 J0 .. 2 J1 - 1]
__device__ __forceinline__ void load_pairs(const double *rec, double *r)
{
#pragma unroll
    for (int j = J0; j < J1; j++) {
        const f64x2 v = reinterpret_cast<const f64x2 *>(rec)[j];
        r[2 * j] = v[0];
        r[2 * j + 1] = v[1];
    }
}

__device__ __forceinline__ void load_record(const double *rec, int id, int ty, double *r)
{
    const double *p = rec + (size_t)id * kRec;
    load_pairs<0, 3>(p, r);
    if (ty != TL) load_pairs<3, kRec / 2>(p, r);
}

__device__ __forceinline__ void load_record(const float *rec, int id, int ty, float *r)
{
    const float *p = rec + (size_t)id * kRec;
    const f32x4 a = *(const f32x4 *)p;
    const f32x2 b = *(const f32x2 *)(p + 4);
    r[0] = a[0], r[1] = a[1], r[2] = a[2], r[3] = a[3], r[4] = b[0], r[5] = b[1];
    if (ty == TL) return;
#pragma unroll
    for (int j = 6; j < kRec; j += 4) {
        const f32x4 v = *(const f32x4 *)(p + j);
#pragma unroll
        for (int q = 0; q < 4; q++) r[j + q] = v[q];
    }
}

// (double)a / (double)b for 1 <= a <= b <= 6 without the division.
__device__ __forceinline__ double small_ratio(int a, int b)
{
    double q = (double)a / 6.0;
    q = b == 5 ? (double)a / 5.0 : q;
    q = b == 4 ? (double)a / 4.0 : q;
    q = b == 3 ? (double)a / 3.0 : q;
    return b == 2 ? (double)a / 2.0 : q;
}

// Fraction along TX -> RX of the straight-line start of interaction k of N:
// k+1 over N+1, or, on a refracting facet (which the ray crosses), the
// point where the segment meets its plane when it does.
__device__ __forceinline__ double line_fraction(int ty, const double *r, const double *tx, const double *rx, int k,
                                                int N)
{
    double a = small_ratio(k + 1, N + 1);
    if (ty == TP && r[16] > 0.0) {
        const double den = r[0] * (rx[0] - tx[0]) + r[1] * (rx[1] - tx[1]) + r[2] * (rx[2] - tx[2]);
        const double c = (den != 0.0) ? (r[3] - (r[0] * tx[0] + r[1] * tx[1] + r[2] * tx[2])) / den : -1.0;
        if (c > 0.0 && c < 1.0) a = c;
    }
    return a;
}

// The solver's scalar type by mode.
template <int MODE> struct ModeT;
template <> struct ModeT<MODE_PLAIN64> { using T = double; };
template <> struct ModeT<MODE_FP32> { using T = float; };
template <> struct ModeT<MODE_FALLBACK64> { using T = double; };

// A plane reflection sends the ray back to the side it came from (the law
// negates the normal component of the direction), so at a root the points
// before and after it lie strictly on the same side of its plane.  When each
// of them is either fixed (TX, RX) or confined to an object that keeps one
// side of the plane everywhere (a plane or straight edge exactly parallel to
// it, off it by more than 1e-9 m), and the two sides differ, no root exists.
// Plain IEEE FP64 without contraction: an exactly parallel pair is found
// parallel whatever the scaling of its normals.
__device__ __forceinline__ double plane_side(const double *n, const double *o, const double *x)
{
#pragma clang fp contract(off)
    return n[0] * (x[0] - o[0]) + n[1] * (x[1] - o[1]) + n[2] * (x[2] - o[2]);
}

// r: the first seven values of the other object's record.
__device__ __forceinline__ bool const_side(const double *r, int ty, const double *n, const double *o, double &side)
{
#pragma clang fp contract(off)
    if (ty == TP) {
        // normals parallel: every point of the other plane is n.(o' - o) off
        if (n[1] * r[2] - n[2] * r[1] != 0.0 || n[2] * r[0] - n[0] * r[2] != 0.0 || n[0] * r[1] - n[1] * r[0] != 0.0)
            return false;
        side = plane_side(n, o, r + 4);
    } else if (ty == TL) {
        if (n[0] * r[3] + n[1] * r[4] + n[2] * r[5] != 0.0) return false;
        side = plane_side(n, o, r);
    } else {
        return false;
    }
    return fabs(side) > 1e-9;
}

// The certificate over the objects of a path, given one after the other.
struct Sides {
    double r[7], a;  // the last object's record and, of a mirror, the side the ray comes from
    int ty;
    bool mirror, known, forbid;
};

__device__ __forceinline__ bool opposite(double a, double b) { return (a < 0.0 && b > 0.0) || (a > 0.0 && b < 0.0); }

__device__ __forceinline__ void sides_next(Sides &c, int k, int n, int ty, const double *r, const double *tx,
                                           const double *rx)
{
    double a = 0.0, b = 0.0;
    if (k == 0) c.forbid = c.mirror = false;
    if (c.mirror && const_side(r, ty, c.r, c.r + 4, b)) c.forbid = c.forbid || (c.known && opposite(c.a, b));
    // a refracting facet passes the ray to its other side
    const bool mirror = ty == TP && !(r[16] > 0.0);
    bool known = true;
    if (mirror) {
        if (k == 0) a = plane_side(r, r + 4, tx);
        else known = const_side(c.r, c.ty, r, r + 4, a);
        if (k == n - 1) c.forbid = c.forbid || (known && opposite(a, plane_side(r, r + 4, rx)));
    }
    c.mirror = mirror;
    c.known = known;
    c.a = a;
    c.ty = ty;
#pragma unroll
    for (int j = 0; j < 7; j++)
        if (j < 6 || ty != TL) c.r[j] = r[j];
}

// True when some point lies outside its object's finite extent by more
// than `margin` metres (rectangle sides, edge ends, paraboloid aperture; a
// circle is its own extent).  FP64 world points and records.
__device__ __forceinline__ bool outside_extent(const double *rec64, int n, const int *id, const int *ty,
                                               const double *X, double margin)
{
    bool out = false;
#pragma unroll
    for (int k = 0; k < kMaxN; k++) {
        if (k >= n) continue;
        const double *r = rec64 + (size_t)id[k] * kRec;
        const double *x = X + 3 * k;
        if (ty[k] == TP) {
            const double e[3] = {x[0] - r[4], x[1] - r[5], x[2] - r[6]};
            const double la = sqrt(r[7] * r[7] + r[8] * r[8] + r[9] * r[9]);
            const double lb = sqrt(r[10] * r[10] + r[11] * r[11] + r[12] * r[12]);
            const double a = (e[0] * r[7] + e[1] * r[8] + e[2] * r[9]) / la;
            const double b = (e[0] * r[10] + e[1] * r[11] + e[2] * r[12]) / lb;
            out = out || a < -margin || a > la + margin || b < -margin || b > lb + margin;
        } else if (ty[k] == TL) {
            const double sp = (x[0] - r[0]) * r[3] + (x[1] - r[1]) * r[4] + (x[2] - r[2]) * r[5];
            out = out || sp < r[6] - margin || sp > r[7] + margin;
        } else if (ty[k] == TQ) {
            const double d[3] = {x[0] - r[0], x[1] - r[1], x[2] - r[2]};
            const double h = d[0] * r[13] + d[1] * r[14] + d[2] * r[15];
            const double w2 = (d[0] - h * r[13]) * (d[0] - h * r[13]) + (d[1] - h * r[14]) * (d[1] - h * r[14]) +
                              (d[2] - h * r[15]) * (d[2] - h * r[15]);
            out = out || w2 > (r[16] + margin) * (r[16] + margin);
        }
    }
    return out;
}

// ------------------------------------------------------------------ start of one path
// The unknowns L (points in the solver's frame, which is shifted by sh, or
// parameters) at the start of a path of n objects and its status: ST_RUNNING,
// or a final one when no iteration is to run (bad input, a start outside the
// guard box, the side certificate).  x0: the row of its start point, or null
// for a start from the straight line or a random point.  One interaction at a
// time, so that few FP64 values are live: its start point, its parameters in
// the parametric form, the guard box test.
template <int MODE, int FORM, typename T>
__device__ __forceinline__ int start_path(const KParams &kp, int64_t sid, int n, const int *id, const int *ty,
                                          const double *rx, const double *sh, const double *x0, T *L)
{
    bool ok = true, inside = true;
    Sides sides;
    const bool rnd = kp.o.init == INIT_RANDOM;
#pragma unroll
    for (int k = 0; k < kMaxN; k++) {
        if (k >= n) continue;
        double r64[kRec];
        load_record(kp.s.rec64, id[k], ty[k], r64);
        if constexpr (MODE != MODE_FALLBACK64) sides_next(sides, k, n, ty[k], r64, kp.s.tx, rx);
        double Xk[3];
        if (x0) {
#pragma unroll
            for (int i = 0; i < 3; i++) {
                Xk[i] = x0[3 * k + i];
                ok = ok && isfinite(Xk[i]);
            }
        } else {
            // the projection onto the object of a point on the TX -> RX
            // segment, or of a random point of the scene box
            const double a = line_fraction(ty[k], r64, kp.s.tx, rx, k, n);
            double P[3];
#pragma unroll
            for (int i = 0; i < 3; i++) {
                if (rnd) {
                    const double u = splitmix_uniform(kp.o.seed, 15u * (uint64_t)sid + 3u * k + i);
                    P[i] = kp.s.lo[i] + u * (kp.s.hi[i] - kp.s.lo[i]);
                } else {
                    P[i] = kp.s.tx[i] + a * (rx[i] - kp.s.tx[i]);
                }
            }
            project(ty[k], r64, P, Xk);
        }
        if constexpr (FORM) {
            // the parameters of the start point; the path starts at X(U),
            // which must lie in the guard box
            double u2[2];
            ok = param_of(ty[k], r64, Xk, u2) && ok;
            if (ty[k] == TQ) {
                // the start point lifted onto the paraboloid
                double e1[3], e2[3];
                across_dir(r64 + 13, e1, e2);
                const double h = r64[17] * (u2[0] * u2[0] + u2[1] * u2[1]);
#pragma unroll
                for (int i = 0; i < 3; i++) Xk[i] = r64[i] + u2[0] * e1[i] + u2[1] * e2[i] + h * r64[13 + i];
            }
            L[2 * k] = (T)u2[0];
            L[2 * k + 1] = (T)u2[1];
        } else {
#pragma unroll
            for (int i = 0; i < 3; i++) L[3 * k + i] = (T)(Xk[i] - sh[i]);
        }
#pragma unroll
        for (int i = 0; i < 3; i++) inside = inside && (Xk[i] >= kp.s.glo[i]) && (Xk[i] <= kp.s.ghi[i]);
    }
    int st = !ok ? ST_BAD : !inside ? ST_DIVERGED : ST_RUNNING;
    if (MODE != MODE_FALLBACK64 && st == ST_RUNNING && sides.forbid) st = ST_LOCALMIN;
    return st;
}

// The points (world) of the unknowns L of n objects, from the records the
// solver uses; zero beyond them.
template <int MAXN, int FORM, typename T>
__device__ __forceinline__ void world_points(const T *rec, int n, const int *id, const int *ty, const T *L,
                                             const double *sh, double *Xw)
{
#pragma unroll
    for (int k = 0; k < MAXN; k++) {
        if (k >= n) {
#pragma unroll
            for (int i = 0; i < 3; i++) Xw[3 * k + i] = 0.0;
            continue;
        }
        if constexpr (FORM) {
            T Xk[3], Tm[3][2], r[kRec];
            load_record(rec, id[k], ty[k], r);
            param_map<T>(ty[k], r, L[2 * k], L[2 * k + 1], Xk, Tm);
#pragma unroll
            for (int i = 0; i < 3; i++) Xw[3 * k + i] = (double)Xk[i] + sh[i];
        } else {
#pragma unroll
            for (int i = 0; i < 3; i++) Xw[3 * k + i] = (double)L[3 * k + i] + sh[i];
        }
    }
}

// A path's whole output row (one cache line): the points, then zeros.
template <int N>
__device__ __forceinline__ void write_row(double *row, const double *X)
{
#pragma unroll
    for (int j = 0; j < kRow; j++) row[j] = (j < 3 * N) ? X[j < 3 * N ? j : 0] : 0.0;
}

// ------------------------------------------------------------------ state rows of the FP32 pass
// The FP32 pass keeps a path's state in a row of 32 words (128 B): written by
// the start kernel, read by a solver lane when it starts the path and written
// when it ends, then turned into the path's results by k_finish, so that a
// lane starts and ends a path with one contiguous access and one round trip
// to memory.  In a large batch the rows lie in bin order in a buffer of their own
// (consecutive lanes, consecutive rows); else they share the path's output row.
//   [0..14] unknowns  [16] cost  [17] |R|_inf  [18] iterations  [19] status
//   [20..22] receiver in the solver's frame  [23] base-4 type code, -1: ended
//   by the start kernel  [24..28] object ids ([24] later: iterations before
//   the straggler launch)  [29] damping [30] plateau reference [31] stall count
//   of a parked path
constexpr int kState = 32;
enum : int { RW_C = 16, RW_IT = 18, RW_ST = 19, RW_RX = 20, RW_CODE = 23, RW_ID = 24, RW_LAM = 29, RW_CREF = 30,
             RW_STAT = 31 };

typedef float f32a __attribute__((may_alias));
typedef int i32a __attribute__((may_alias));

// The state row of bin slot `slot` / solve `sid`.
__device__ __forceinline__ f32a *state_row(const KParams &kp, int64_t slot, int64_t sid)
{
    return kp.rows ? (f32a *)kp.rows + slot * kState : (f32a *)(kp.out.x + sid * kRow);
}

// Rows of 128 bytes (state and point rows) between a wave's lanes, one row
// each, and memory, through LDS.  A lane that stores its own row touches one
// line in each of eight instructions, 64 lines apiece, which the memory pipe
// takes one by one and hands on as eight partial lines; with eight lanes on a
// row an instruction moves eight whole lines.  In LDS a row takes 36 words, so
// that the lanes' 16-byte accesses spread over the banks, and its address
// follows it.  All lanes of the wave call these together.
constexpr int kRowWords = 36;
constexpr int kWaveRows = 64 * kRowWords;  // words of LDS per wave

typedef float f32x4l __attribute__((ext_vector_type(4), aligned(16), may_alias));
typedef uint64_t u64a __attribute__((may_alias));

// Stores the lanes' rows, each at its dst (null: none).
__device__ __forceinline__ void rows_store(float *w, void *dst)
{
    const int lane = __lane_id(), part = (lane & 7) * 4;
    *(u64a *)(w + lane * kRowWords + 32) = (uint64_t)dst;
    wave_sync();
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const float *row = w + (j * 8 + (lane >> 3)) * kRowWords;
        float *p = (float *)*(const u64a *)(row + 32);
        const f32x4l v = *(const f32x4l *)(row + part);
        if (p) *(f32x4 *)(p + part) = v;
    }
    wave_sync();
}

// Loads the lanes' rows from src (a readable row in every lane).
__device__ __forceinline__ void rows_load(float *w, const void *src)
{
    const int lane = __lane_id(), part = (lane & 7) * 4;
    *(u64a *)(w + lane * kRowWords + 32) = (uint64_t)src;
    wave_sync();
    f32x4 v[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const float *p = (const float *)*(const u64a *)(w + (j * 8 + (lane >> 3)) * kRowWords + 32);
        v[j] = *(const f32x4 *)(p + part);
    }
#pragma unroll
    for (int j = 0; j < 8; j++) *(f32x4l *)(w + (j * 8 + (lane >> 3)) * kRowWords + part) = v[j];
    wave_sync();
}

// A path's point row (write_row) in LDS.
template <int N>
__device__ __forceinline__ void stage_row(float *mine, const double *X)
{
    f64x2 *row = (f64x2 *)mine;
#pragma unroll
    for (int j = 0; j < kRow; j += 2)
        row[j / 2] = f64x2{j < 3 * N ? X[j < 3 * N ? j : 0] : 0.0, j + 1 < 3 * N ? X[j + 1 < 3 * N ? j + 1 : 0] : 0.0};
}

// The start of solve `sid` (bin slot `slot`): its unknowns where the solver
// reads them, status ST_RUNNING; or, when no iteration is to run, its
// results: the start points as the solver holds them (zeros for bad input).
// Called by all lanes of a wave, live: the lane has a path; w: kWaveRows words
// of LDS for the wave.
template <int MODE, int FORM>
__device__ __forceinline__ void begin_path(const KParams &kp, bool live, int64_t slot, int64_t sid, int n,
                                           const int *id, const int *ty, const double *rx, const double *x0,
                                           float *w)
{
    using T = typename ModeT<MODE>::T;
    constexpr int D = (FORM ? 2 : 3) * kMaxN;
    double sh[3];
#pragma unroll
    for (int i = 0; i < 3; i++) sh[i] = (MODE == MODE_FP32) ? kp.s.tx[i] : 0.0;
    T L[(D + 3) / 4 * 4];
#pragma unroll
    for (int j = 0; j < (D + 3) / 4 * 4; j++) L[j] = T(0);
    float *mine = w + __lane_id() * kRowWords;
    void *dst = nullptr;
    if (live) {
        const int st = start_path<MODE, FORM>(kp, sid, n, id, ty, rx, sh, x0, L);
        dst = kp.out.x + (size_t)sid * kRow;
        kp.out.status[sid] = (uint8_t)st;
        if (st != ST_RUNNING) {
            if (MODE == MODE_FP32 && kp.rows) state_row(kp, slot, sid)[RW_CODE] = __int_as_float(-1);
            const T *rec = (MODE == MODE_FP32) ? (const T *)kp.s.rec32 : (const T *)kp.s.rec64;
            double Xs[3 * kMaxN];
            world_points<kMaxN, FORM, T>(rec, st == ST_BAD ? 0 : n, id, ty, L, sh, Xs);
            stage_row<kMaxN>(mine, Xs);
            kp.out.cost[sid] = __builtin_huge_val();
            kp.out.iters[sid] = 0;
            if (kp.out.stage) kp.out.stage[sid] = 0;
        } else if constexpr (MODE == MODE_FP32) {
            dst = state_row(kp, slot, sid);
            int code = 0;
#pragma unroll
            for (int k = 0; k < kMaxN; k++) code |= (k < n ? ty[k] : 0) << (2 * k);
            f32x4l *row = (f32x4l *)mine;
#pragma unroll
            for (int j = 0; j < RW_C; j += 4) {
                f32x4l v;
#pragma unroll
                for (int q = 0; q < 4; q++) v[q] = j + q < D ? L[j + q < D ? j + q : 0] : 0.0f;
                row[j / 4] = v;
            }
            row[RW_C / 4] = f32x4l{0.0f, 0.0f, 0.0f, 0.0f};
            row[RW_RX / 4] = f32x4l{(T)(rx[0] - sh[0]), (T)(rx[1] - sh[1]), (T)(rx[2] - sh[2]), __int_as_float(code)};
            row[RW_ID / 4] = f32x4l{__int_as_float(id[0]), __int_as_float(id[1]), __int_as_float(id[2]),
                                    __int_as_float(id[3])};
            row[RW_ID / 4 + 1] = f32x4l{__int_as_float(id[4]), 0.0f, 0.0f, 0.0f};
        } else {
            double Xr[3 * kMaxN];
#pragma unroll
            for (int j = 0; j < 3 * kMaxN; j++) Xr[j] = j < D ? L[j < D ? j : 0] : 0.0;
            stage_row<kMaxN>(mine, Xr);
        }
    }
    rows_store(w, dst);
}

}  // namespace mpt
