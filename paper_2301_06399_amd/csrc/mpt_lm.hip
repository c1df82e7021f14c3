// The Levenberg-Marquardt kernels of the batched solve (gfx950, wave64):
//  k_lm              persistent solver over every order's bin, one lane per
//                    path, lanes refilled from a per-wave chunk of the bin once
//                    enough of them are idle (FP64 plain, FP32 stage or FP64
//                    fallback)
//
// What bounds them: VALU issue (an order-5 FP32 iteration is about 2000 vector
// instructions, four cycles each) and, at one or two waves per SIMD, the
// latency of the chain.  So the loop holds nothing but iterations: starts and
// ends of paths are kernels of their own (k_start, k_finish), a lane reads and
// writes one 128-byte state row, and finished lanes are saved together.  With
// them in the loop an order-5 kernel was 78 KB of code at 256 registers.  The
// stress workload's pass (16.8 M paths of orders 3-5) took 22.0 ms then, in its
// tuned launch; now it takes 9.5, and k_start and k_finish, whose work it held,
// 1.4 and 1.5.  The street canyon's (262,144 paths of orders 1-3) took 466 us, now
// 274, 19 and 56.
//  k_lm_low          the same over orders 1-3
//  k_lm_one          one order's bin
// The file is compiled once per (mode, form, scene in LDS or not), MPT_LM_MODE
// / MPT_LM_FORM / MPT_LM_LDS, so that the instantiations build in parallel
// (one translation unit took eight minutes).
#include "mpt_path.hpp"

namespace mpt {


// ------------------------------------------------------------------ LM lane state
template <typename T>
struct LMOpts {
    int max_iter, max_iter_planar, win, stat_win;
    T frac, tol_step, tol_res, tau_root, lambda0, stat_tol;
};

// What the next pass of a lane does: a step, or only the normal equations of
// a new path's start (a path that was parked has passed its iteration's
// checks already).
enum : int { LANE_STEP = 0, LANE_NEW = 1, LANE_RESUMED = 2 };

// State of one lane's path: the unknowns (3N points, or 2N parameters in the
// parametric form), the normal equations, gradient and cost there, and the
// Levenberg-Marquardt scalars.
template <typename T, int N, int FORM>
struct Lane {
    static constexpr int B = FORM ? 2 : 3, D = B * N, S = Band<N, B>::SIZE;
    T X[D], A[S], g[D];
    T lam, Cref, C, rinf;
    int it, stat, win_it, phase;  // win_it: the iteration of the next plateau test
};

// x / 10, correctly rounded while the quotient is a normal number: the
// remainder of the product with the rounded tenth corrects it (Markstein; the
// product is within one unit in the last place).  Three instructions for the
// ten (FP32) or more of a division.
template <typename T>
__device__ __forceinline__ T tenth(T x)
{
    const T q = x * T(0.1), r = fma(T(-10), q, x);
    return fma(r, T(0.1), q);
}

// One pass of the Levenberg-Marquardt iteration on the cost of Eq. (12) with
// the rescaled rows (FORM 1: of Eq. (15), where the placeholder parameter of
// an edge is held fixed): the step from the lane's normal equations, then
// the normal equations at the trial point, which are the next pass's if the
// step is taken, then the tests that open the next iteration.  The trial's
// cost comes with its normal equations: a pass that evaluated the cost first
// and assembled an accepted point in the next iteration mapped every point and
// formed every direction twice and took 2.62 against 1.76 ms (1,048,576
// paths among curved objects, FP32 parametric), 606 against 410 us (45,769
// planar paths of orders 1-3, FP64 implicit) and 330 against 295 us (262,144
// planar paths, where the longest chains bound it).
// Returns ST_RUNNING or the final status.  REFR: the scene has refracting
// facets (their rows are compiled in).
// FIXED: p.ty is known to the compiler.
template <typename T, int N, int FORM, bool REFR, bool FIXED = false>
__device__ __forceinline__ int lm_pass(const SceneT<T> &sc, const PathIn<T, N> &p, Lane<T, N, FORM> &L,
                                       const LMOpts<T> &o)
{
    using LT = Lane<T, N, FORM>;
    constexpr int B = LT::B, M = LT::D;
    using Bd = Band<N, B>;
    const bool stepping = L.phase == LANE_STEP;
    bool real[M];  // the edges' placeholder parameters are not
#pragma unroll
    for (int i = 0; i < M; i++) real[i] = !(FORM && (i & 1)) || is_surface(p.ty[i / B]);
    T xt[M], dmax = T(0);
#pragma unroll
    for (int i = 0; i < M; i++) xt[i] = L.X[i];
    bool go = true, small = false;  // go: there is a trial point
    if (stepping) {
        T F[LT::S];
#pragma unroll
        for (int i = 0; i < M; i++) dmax = real[i] ? fmax(dmax, L.A[Bd::at(i, i)]) : dmax;
        const T floor_d = T(1e-12) * dmax;
#pragma unroll
        for (int i = 0; i < M; i++)
#pragma unroll
            for (int j = 0; j <= i; j++) {
                if (!Bd::in(i, j)) continue;
                const T a = L.A[Bd::at(i, j)];
                if (i != j) F[Bd::at(i, j)] = a;
                else if (FORM) F[Bd::at(i, i)] = real[i] ? a + L.lam * fmax(a, floor_d) : T(1);
                else F[Bd::at(i, i)] = a + L.lam * fmax(a, floor_d);
            }
        go = chol_band<T, N, B>(F, FIXED ? real : nullptr);
        if (go) {
            T d[M];
#pragma unroll
            for (int i = 0; i < M; i++) d[i] = -L.g[i];
            const T pred = chol_solve_band<T, N, B>(F, d, FIXED ? real : nullptr);  // d <- dx; pred = -g^T dx
            if (o.stat_win > 0 && p.planar) {
                // planes and straight edges: the descent has stalled when the damped
                // model predicts too small a decrease several iterations in a row
                L.stat = (pred < o.stat_tol * L.C) ? L.stat + 1 : 0;
                if (L.stat >= o.stat_win) return (L.rinf <= o.tau_root) ? ST_CONV : ST_LOCALMIN;
            }
            T xinf = T(0), dinf = T(0);
#pragma unroll
            for (int i = 0; i < M; i++) {
                xinf = fmax(xinf, fabs(L.X[i]));
                dinf = fmax(dinf, fabs(d[i]));
                xt[i] = L.X[i] + d[i];
                if constexpr (!FORM) go = go && (xt[i] >= sc.glo[i % 3]) && (xt[i] <= sc.ghi[i % 3]);
            }
            small = dinf <= o.tol_step * (T(1) + xinf);
        }
    }
    bool take = false;
    if (go) {
        T A1[LT::S], g1[M], C1, r1;
        if constexpr (FORM) {
            bool guard;
            take = assemble_param<T, N, REFR, FIXED>(sc, p, xt, A1, g1, C1, r1, guard) &&
                   (!stepping || (guard && C1 < L.C));
        } else {
            take = assemble<T, N, REFR>(sc, p, xt, A1, g1, C1, r1) && (!stepping || C1 < L.C);
        }
        if (take) {
#pragma unroll
            for (int i = 0; i < M; i++)
#pragma unroll
                for (int j = 0; j <= i; j++)
                    if (Bd::in(i, j)) L.A[Bd::at(i, j)] = A1[Bd::at(i, j)];
#pragma unroll
            for (int i = 0; i < M; i++) {
                L.X[i] = xt[i];
                L.g[i] = g1[i];
            }
            L.C = C1;
            L.rinf = r1;
        }
    }
    if (stepping) {
        if (small) return (L.rinf <= o.tau_root) ? ST_CONV : ST_LOCALMIN;
        if (take) {
            L.lam = fmax(tenth(L.lam), T(1e-15) * dmax);
        } else {
            L.lam *= T(10);
            if (L.lam > T(1e12) * dmax) return ST_STALL;
        }
        if (L.it >= (p.planar ? o.max_iter_planar : o.max_iter)) return ST_MAXIT;
    }
    // the next iteration's tests
    if (L.phase != LANE_RESUMED) {
        L.it++;
        if (!stepping) {
            if (!take) return ST_DEGEN;
#pragma unroll
            for (int i = 0; i < M; i++) dmax = real[i] ? fmax(dmax, L.A[Bd::at(i, i)]) : dmax;
            L.lam = o.lambda0 * dmax;
            L.Cref = L.C;
        }
        if (L.rinf <= o.tol_res) return (L.rinf <= o.tau_root) ? ST_CONV : ST_LOCALMIN;
        if (L.it == L.win_it) {
            if (L.C > o.frac * L.Cref) return (L.rinf <= o.tau_root) ? ST_CONV : ST_LOCALMIN;
            L.Cref = L.C;
            L.win_it += o.win;
        }
    }
    L.phase = LANE_STEP;
    return ST_RUNNING;
}

// ------------------------------------------------------------------ persistent LM kernel
// Lane-refill loop for the bin of order N.  Each wave takes a chunk of the bin
// with one atomic, and hands the chunk's paths to its idle lanes once enough
// lanes are idle, so lanes never wait for the slowest path of their wave.
//
// One iteration with the path's primitive types fixed at compile time (digit
// k of CODE, base 4: 0 plane, 1 straight edge), so that no per-type branch
// or select is left in the code.  Bins are type-homogeneous, so most waves
// hold one planar sequence and run one of these variants only.  Used by the
// parametric FP32 kernel: there it shortens an iteration (street canyon LM
// stage 0.550 -> 0.484 ms, room 0.157 -> 0.119 ms, and without the columns of
// the edges' placeholder parameters, which the compiler may not drop by
// itself, 0.295 -> 0.278 and 0.086 -> 0.080 ms); the implicit kernel's larger
// variants made it slower (0.516 -> 0.556 ms).
template <typename T, int N, int FORM, int CODE>
__device__ __forceinline__ int lm_step_fixed(const SceneT<T> &sc, const PathIn<T, N> &p,
                                             Lane<T, N, FORM> &L, const LMOpts<T> &o)
{
    PathIn<T, N> q = p;
#pragma unroll
    for (int k = 0; k < N; k++) q.ty[k] = (CODE >> (2 * k)) & 3;
    q.planar = true;  // planes and straight edges: no refracting facet
    return lm_pass<T, N, FORM, false, true>(sc, q, L, o);
}

// The fixed-type step for the planar sequence `code` of orders 1-3.
template <typename T, int N, int FORM>
__device__ __forceinline__ int lm_step_uniform(int code, const SceneT<T> &sc, const PathIn<T, N> &p,
                                               Lane<T, N, FORM> &L, const LMOpts<T> &o)
{
#define MPT_FIXED(c) \
    case c: return lm_step_fixed<T, N, FORM, c>(sc, p, L, o);
    if constexpr (N == 1) {
        switch (code) { MPT_FIXED(0) MPT_FIXED(1) }
    } else if constexpr (N == 2) {
        switch (code) { MPT_FIXED(0) MPT_FIXED(1) MPT_FIXED(4) MPT_FIXED(5) }
    } else if constexpr (N == 3) {
        switch (code) {
            MPT_FIXED(0) MPT_FIXED(1) MPT_FIXED(4) MPT_FIXED(5) MPT_FIXED(16) MPT_FIXED(17) MPT_FIXED(20) MPT_FIXED(21)
        }
    }
#undef MPT_FIXED
    return -1;
}

// How `size` waves share a bin of `count` paths.  Consecutive slots of a bin
// hold one type sequence, and a wave pays for every type sequence among its
// busy lanes, so a wave takes consecutive slots.  While an equal share is at
// most kStaticChunk paths, that share is all a wave gets (few lanes per wave
// on a small batch: idle lanes cost nothing, a second sequence in the wave
// does); of a longer queue it first takes a quarter of an equal share and then
// draws chunks of a quarter of what is left per wave from the bin's counter.
// No wave's first chunk comes from the counter: 2048 waves drawing at once
// waited 15-30 us for it (one counter is served one atomic at a time).
constexpr int kStaticChunk = 128, kMinChunk = 64, kMaxChunk = 4096;

__device__ __forceinline__ int launch_waves() { return (int)(gridDim.x * (blockDim.x >> 6)); }

// The waves of a launch that take part for `count` paths: all, or, where the host
// asks for it (kp.spread CUs, blocks of one wave), one on each CU while its lanes
// hold the launch's paths and two while two's do (see choose in mpt_api.hip).
__device__ __forceinline__ int used_waves(const KParams &kp, int count)
{
    const int all = launch_waves(), cu = kp.spread;
    if (cu == 0 || count > 2 * 64 * cu) return all;
    return min(all, count > 64 * cu ? 2 * cu : cu);
}

struct BinShare {
    int rank, size;  // this wave among the waves that start with the bin; rank -1: none of them
};

__device__ __forceinline__ int first_chunk(int count, int size)
{
    return min(max(count / size / 4, kMinChunk), kMaxChunk);
}

// Stragglers.  Iteration counts are bimodal (a root converges in a handful of
// iterations, a path without one creeps until the plateau test ends it), so
// once the bin's queue is empty a wave would idle most of its lanes while its
// slowest paths finish.  Instead, when no more than spill_t lanes are still
// busy, the wave parks their state (points, iteration count, damping,
// plateau reference) and leaves; a second launch of the same kernel
// (kp.resume) packs the parked paths densely and finishes them.  The same
// machine code runs every iteration of a path, from the exact state it was
// parked in, so the results are identical bit for bit.

template <int MODE, int N, int FORM = 0, bool TYPED = false, bool REFR = false>
__device__ __forceinline__ void lm_bin(const KParams &kp, const typename ModeT<MODE>::T *__restrict__ srec,
                                       const BinShare share)
{
    using T = typename ModeT<MODE>::T;
    constexpr int D = FORM ? 2 * N : 3 * N;  // unknowns: points, or parameters
    constexpr bool FB = MODE == MODE_FALLBACK64;
    const int lane = __lane_id();
    const bool resume = !FB && kp.resume != 0;
    const int *cnt = resume ? kp.spill_cnt : FB ? kp.fb_cnt : kp.bin_cnt;
    int *head = resume ? kp.spill_head + (N - 1) : kp.head + (FB ? 5 : 0) + (N - 1);
    const int count = cnt[N - 1];
    if (count == 0) return;
    const int off = bin_offset(kp.bin_cnt, N);
    // every path is in some wave's share, or the rest is drawn from `head`
    const bool fixed = share.size > 0 && count <= (int64_t)share.size * kStaticChunk;
    if (fixed && share.rank < 0) return;
    const int c0 = share.size > 0 ? first_chunk(count, share.size) : 0, drawn0 = c0 * share.size;
    const bool may_spill = !resume && !FB && kp.spill_t > 0;

    SceneT<T> sc;
    sc.rec = srec;
    double sh[3];  // origin of the solver's frame
#pragma unroll
    for (int i = 0; i < 3; i++) {
        sh[i] = (MODE == MODE_FP32) ? kp.s.tx[i] : 0.0;
        sc.tx[i] = (MODE == MODE_FP32) ? T(0) : (T)kp.s.tx[i];
        sc.glo[i] = (T)(kp.s.glo[i] - sh[i]);
        sc.ghi[i] = (T)(kp.s.ghi[i] - sh[i]);
    }
    LMOpts<T> o;
    if (MODE == MODE_FP32) {
        o.max_iter = kp.o.max_iter32;
        o.max_iter_planar = kp.o.max_iter32_planar;
        o.tol_step = (T)kp.o.tol_step32;
        o.tol_res = (T)kp.o.tol_res32;
        o.tau_root = (T)kp.o.tau_root32;  // an FP32 point this close is taken for a root
    } else {
        o.max_iter = FB ? kp.o.max_iter_fb : kp.o.max_iter;
        o.max_iter_planar = o.max_iter;
        o.tol_step = (T)kp.o.tol_step;
        o.tol_res = (T)kp.o.tol_res;
        o.tau_root = (T)kp.o.tau_root;
    }
    o.win = kp.o.plateau_win;
    o.frac = (T)kp.o.plateau_frac;
    o.lambda0 = (T)kp.o.lambda0;
    o.stat_win = FB ? 0 : kp.o.stat_win;
    o.stat_tol = (T)kp.o.stat_tol;

    Lane<T, N, FORM> L;
    PathIn<T, N> p;
    int slot = 0, code = 0;
    int ridx = 0;       // the path's state row (FP32) or solve id
    int it0 = 0;        // a resumed path's iteration: opened, its step not yet taken
    int fin = 0;        // final status of a finished path that is not saved yet
    bool active = false, done = false;
    // wave-uniform chunk [cbase, cend) of the bin
    int cbase = 0, cend = 0;
    if (share.rank >= 0) {
        cbase = fixed ? (int)((int64_t)count * share.rank / share.size) : c0 * share.rank;
        cend = fixed ? (int)((int64_t)count * (share.rank + 1) / share.size) : cbase + c0;
    }
    // lanes the wave keeps busy: all, or its share of a small batch
    const int width = (fixed && cend - cbase < 64) ? cend - cbase : 64;
    bool drained = fixed && cbase >= cend;

    while (true) {
        const int busy = (int)__popcll(__ballot(active));
        if (busy == 0 || (!drained && busy + min(kp.refill, width) <= width)) {
            // ---- save the finished paths, together: a store of one or two
            // lanes' results in every iteration costs as much as all lanes'
            if (done) {
                done = false;
                if constexpr (MODE == MODE_FP32) {
                    // the state row: k_finish turns it into the path's results
                    f32a *rf = state_row(kp, ridx, ridx);
#pragma unroll
                    for (int j = 0; j < D; j += 4) {
                        f32x4 v;
#pragma unroll
                        for (int q = 0; q < 4; q++) v[q] = L.X[j + q < D ? j + q : D - 1];
                        *(f32x4 *)(rf + j) = v;
                    }
                    *(f32x4 *)(rf + RW_C) = f32x4{L.C, L.rinf, __int_as_float(L.it), __int_as_float(fin)};
                    // iterations the first launch finished
                    if (kp.spill_t > 0) rf[RW_ID] = __int_as_float(resume ? max(it0 - 1, 0) : L.it);
                } else {
                    int ty[N];
#pragma unroll
                    for (int k = 0; k < N; k++) ty[k] = (code >> (2 * k)) & 3;
                    double Xw[3 * N];
                    world_points<N, FORM, T>(sc.rec, N, p.id, ty, L.X, sh, Xw);
                    write_row<N>(kp.out.x + (size_t)ridx * kRow, Xw);
                    kp.out.cost[ridx] = (double)L.C;
                    kp.out.iters[ridx] = FB ? L.it + kp.out.iters[ridx] : L.it;
                    if (kp.out.stage) {
                        kp.out.stage[(FB ? (size_t)2 * kp.b.n : 0) + ridx] = L.it;
                        if (resume) kp.out.stage[(size_t)3 * kp.b.n + ridx] = L.it - max(it0 - 1, 0);
                    }
                    kp.out.status[ridx] = (uint8_t)(FB ? fin | 0x80 : fin);
                }
            }
            // ---- refill the idle lanes from the wave's chunk (once enough
            // are idle: each refill stalls the wave on the dependent loads of
            // the new paths' inputs)
            if (!drained && cbase >= cend) {
                int b0 = count, ch = 0;
                if (lane == 0) {
                    // an estimate of what is left (other waves draw meanwhile)
                    // sizes the chunk; the add alone hands it out
                    const int left = count - drawn0 -
                                     __hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (left > 0) {
                        ch = min(max(left / (4 * launch_waves()), kMinChunk), kMaxChunk);
                        b0 = drawn0 + atomicAdd(head, ch);
                    }
                }
                cbase = __builtin_amdgcn_readfirstlane(b0);
                cend = min(cbase + __builtin_amdgcn_readfirstlane(ch), count);
                if (cbase >= count) drained = true;
            }
            if (!drained) {
                const uint64_t need = __ballot(!active);
                const int rank = (int)__popcll(need & ((1ull << lane) - 1ull));
                const int take = min((int)__popcll(need), cend - cbase);
                if (!active && rank < take) {
                    slot = off + cbase + rank;
                    if constexpr (!FB)
                        if (resume) slot = kp.spill_list[slot];
                    L.it = 0;
                    L.stat = 0;
                    L.lam = T(0);
                    L.phase = LANE_NEW;
                    L.C = T(__builtin_huge_val());
                    L.rinf = T(__builtin_huge_val());
                    L.Cref = L.C;
                    p.planar = true;
                    if constexpr (MODE == MODE_FP32) {
                        active = true;
                        if (kp.rows) {
                            ridx = slot;
                        } else {
                            ridx = kp.perm[slot];
                            active = kp.out.status[ridx] == ST_RUNNING;
                        }
                        const f32a *rf = state_row(kp, ridx, ridx);
                        const f32x4 rv = *(const f32x4 *)(rf + RW_RX), iv = *(const f32x4 *)(rf + RW_ID);
#pragma unroll
                        for (int j = 0; j < D; j += 4) {
                            const f32x4 v = *(const f32x4 *)(rf + j);
#pragma unroll
                            for (int q = 0; q < 4; q++)
                                if (j + q < D) L.X[j + q < D ? j + q : 0] = v[q];
                        }
#pragma unroll
                        for (int k = 0; k < N && k < 4; k++) p.id[k] = __float_as_int(iv[k]);
                        if constexpr (N > 4) p.id[N - 1] = ((const i32a *)rf)[RW_ID + 4];
#pragma unroll
                        for (int i = 0; i < 3; i++) p.rx[i] = rv[i];
                        code = __float_as_int(rv[3]);
                        active = active && code >= 0;  // else ended by the start kernel
                        if (resume) {
                            // a parked path: its state exactly as it was left
                            L.it = ((const i32a *)rf)[RW_IT];
                            L.lam = rf[RW_LAM];
                            L.Cref = rf[RW_CREF];
                            L.stat = ((const i32a *)rf)[RW_STAT];
                        }
                    } else {
                        // by solve id; the fallback's lists are in no order
                        ridx = FB ? kp.fb_list[slot] : kp.perm[slot];
                        active = FB || kp.out.status[ridx] == ST_RUNNING;
                        code = 0;
#pragma unroll
                        for (int k = 0; k < N; k++) p.id[k] = kp.b.prim[(size_t)k * kp.b.n + ridx];
                        const int ri = kp.b.rx_index[ridx];
#pragma unroll
                        for (int k = 0; k < N; k++)
                            code |= prim_type(p.id[k], kp.s.n_pl, kp.s.n_pl_ln, kp.s.n_pl_ln_q) << (2 * k);
                        double rx[3];
#pragma unroll
                        for (int i = 0; i < 3; i++) {
                            rx[i] = kp.b.rx[3 * (size_t)ri + i];
                            p.rx[i] = (T)rx[i];
                        }
                        if constexpr (FB) {
                            int ty[kMaxN], ids[kMaxN];
#pragma unroll
                            for (int k = 0; k < kMaxN; k++) {
                                ids[k] = p.id[k < N ? k : 0];
                                ty[k] = (code >> (2 * (k < N ? k : 0))) & 3;
                            }
                            // from the FP32 end point (already root-like)
                            const double *row = kp.out.x + (size_t)ridx * kRow;
                            T L0[3 * kMaxN];
                            const int st0 = start_path<MODE, FORM>(kp, ridx, N, ids, ty, rx, sh, row, L0);
#pragma unroll
                            for (int j = 0; j < D; j++) L.X[j] = L0[j];
                            if (st0 != ST_RUNNING) {
                                // finished before the first iteration: the start
                                // points as the solver holds them (zeros for bad
                                // input)
                                double Xs[3 * N];
                                world_points<N, FORM, T>(sc.rec, st0 == ST_BAD ? 0 : N, ids, ty, L.X, sh, Xs);
                                write_row<N>(kp.out.x + (size_t)ridx * kRow, Xs);
                                kp.out.cost[ridx] = __builtin_huge_val();
                                kp.out.status[ridx] = (uint8_t)(st0 | 0x80);
                                active = false;
                            }
                        } else {
                            const double *row = kp.out.x + (size_t)ridx * kRow;
#pragma unroll
                            for (int j = 0; j < D; j++) L.X[j] = row[j];
                            if (resume) {
                                L.it = kp.out.iters[ridx];
                                L.lam = kp.spill_f[ridx];
                                L.Cref = kp.spill_f[(size_t)kp.b.n + ridx];
                                L.stat = (int)kp.spill_f[(size_t)2 * kp.b.n + ridx];
                            }
                        }
                    }
                    it0 = L.it;
                    if (resume && it0 > 0) L.phase = LANE_RESUMED;  // else parked before its first pass
                    // the plateau test opens iterations 1 + win, 1 + 2 win, ...;
                    // the next of them after iteration it0 (1 at the least: the
                    // first iteration only sets the reference)
                    L.win_it = o.win > 0 ? (it0 > 1 ? (it0 - 1) / o.win : 0) * o.win + o.win + 1 : 0;
                    if constexpr (REFR) {
                        if (active) {
#pragma unroll
                            for (int k = 0; k < N; k++) {
                                const int t = (code >> (2 * k)) & 3;
                                p.planar = p.planar &&
                                           (t == TL || (t == TP && sc.rec[(size_t)p.id[k] * kRec + 16] <= T(0)));
                            }
                        }
                    }
                }
                cbase += take;
                if (fixed && cbase >= cend) drained = true;
            }
            if (!__any(active)) {
                if (drained) break;
                continue;
            }
        }
        // the bin is drained and few lanes are busy: park them (wave-uniform)
        if (may_spill && drained && (int)__popcll(__ballot(active)) <= kp.spill_t) {
            if (active) {
                // ---- a parked path: its exact state, for the straggler launch
                if constexpr (MODE == MODE_FP32) {
                    f32a *rf = state_row(kp, ridx, ridx);
#pragma unroll
                    for (int j = 0; j < D; j++) rf[j] = L.X[j];
                    rf[RW_IT] = __int_as_float(L.it);
                    rf[RW_LAM] = L.lam;
                    rf[RW_CREF] = L.Cref;
                    rf[RW_STAT] = __int_as_float(L.stat);
                } else {
                    double *row = kp.out.x + (size_t)ridx * kRow;
#pragma unroll
                    for (int j = 0; j < D; j++) row[j] = L.X[j];
                    kp.out.iters[ridx] = L.it;
                    kp.spill_f[ridx] = (double)L.lam;
                    kp.spill_f[(size_t)kp.b.n + ridx] = (double)L.Cref;
                    kp.spill_f[(size_t)2 * kp.b.n + ridx] = (double)L.stat;
                }
                kp.spill_list[off + atomicAdd(&kp.spill_cnt[N - 1], 1)] = slot;
                active = false;
            }
            continue;
        }
        // ---- one iteration on every busy lane
        // (the bins are sorted by type sequence, so the lanes of a wave mostly
        // share theirs, and the branches on a type skip the others' rows)
        int st = ST_RUNNING;
        bool generic = active;
        if constexpr (TYPED && MODE == MODE_FP32 && FORM == 1 && N <= 3) {
            // every planar path takes its fixed-type step, whatever the other
            // lanes of its wave hold: one sequence after the other.  (The kernel
            // of orders 1-3 beside orders 4 and 5 is not TYPED: its generic step
            // adds the placeholders' columns, which are zeros, and ends in the
            // same result.)
            generic = active && !(REFR ? p.planar : (code & 0x2AA) == 0);
            uint64_t todo = __ballot(active && !generic);
            while (todo) {
                const int c0 = __builtin_amdgcn_readlane(code, (int)__builtin_ctzll(todo));
                const bool mine = active && !generic && code == c0;
                todo &= ~__ballot(mine);
                if (mine) st = lm_step_uniform<T, N, FORM>(c0, sc, p, L, o);
            }
        }
        if (generic) {
#pragma unroll
            for (int k = 0; k < N; k++) p.ty[k] = (code >> (2 * k)) & 3;
            if constexpr (!REFR) p.planar = (code & 0x2AA) == 0;
            st = lm_pass<T, N, FORM, REFR>(sc, p, L, o);
        }
        if (active && st != ST_RUNNING) {
            active = false;
            done = true;
            fin = st;
        }
    }
}

// Waves per SIMD each kernel is compiled for: as many as its registers allow
// without spills (VGPRs per lane of orders 1-5: FP32 parametric 93 / 126 / 168 /
// 198 / 228, implicit 99 / 149 / 220 / 279 / 340; FP64 parametric 136 / 218 / 298 /
// 354 / 411, implicit 163 / 282 / 409 / 512 / 512, the last two with spills).
// Two sets of normal equations are alive while a trial point is assembled; the
// implicit orders 4 and 5 pay for that with one wave instead of two, and
// still gain: 91,571 paths of random starts 0.94 ms at one wave, 1.78 at two
// with 103 spilled registers, 1.24 at two with the trial's cost evaluated alone.
template <int MODE, int N, int FORM = 0> struct Occ { static constexpr int W = 1; };
template <> struct Occ<MODE_FP32, 1, 0> { static constexpr int W = 4; };
template <> struct Occ<MODE_FP32, 2, 0> { static constexpr int W = 3; };
template <> struct Occ<MODE_FP32, 3, 0> { static constexpr int W = 2; };

template <> struct Occ<MODE_PLAIN64, 1, 0> { static constexpr int W = 3; };
template <> struct Occ<MODE_FP32, 1, 1> { static constexpr int W = 4; };
template <> struct Occ<MODE_FP32, 2, 1> { static constexpr int W = 3; };
template <> struct Occ<MODE_FP32, 3, 1> { static constexpr int W = 2; };
template <> struct Occ<MODE_FP32, 4, 1> { static constexpr int W = 2; };
template <> struct Occ<MODE_FP32, 5, 1> { static constexpr int W = 2; };
template <> struct Occ<MODE_PLAIN64, 1, 1> { static constexpr int W = 3; };
template <> struct Occ<MODE_PLAIN64, 2, 1> { static constexpr int W = 2; };

// The mixed-order kernels: order 5's.
template <int MODE, int FORM> struct OccAll { static constexpr int W = (MODE == MODE_FP32 && FORM) ? 2 : 1; };

// Scene records staged in LDS by every block of a persistent launch (the
// whole scene: 651 primitives x 18 floats = 47 KB for the street canyon).
template <int MODE, bool LDS>
__device__ __forceinline__ const typename ModeT<MODE>::T *stage_scene(const KParams &kp)
{
    using T = typename ModeT<MODE>::T;
    const T *g = (MODE == MODE_FP32) ? (const T *)kp.s.rec32 : (const T *)kp.s.rec64;
    if (!LDS) return g;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *l = reinterpret_cast<T *>(smem_raw);
    const int total = kp.s.n_all * kRec;
    for (int i = threadIdx.x; i < total; i += blockDim.x) l[i] = g[i];
    __syncthreads();
    return l;
}

// The waves of a mixed-order launch are dealt to the nonempty orders in
// proportion to their work (paths x order, and a sixteenth of the whole to
// each so that none waits for a wave), long paths first.  lo[k], lo[k - 1]:
// the waves that start with order k.
struct OrderShare {
    int wave, lo[kMaxN + 1];
    __device__ __forceinline__ BinShare of(int k) const
    {
        const int size = lo[k - 1] - lo[k], r = wave - lo[k];
        return {r >= 0 && r < size ? r : -1, size};
    }
};

__device__ __forceinline__ OrderShare order_share(const int *cnt, int max_order, int all)
{
    OrderShare s;
    s.wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    float w[kMaxN + 1], tot = 0.0f, sum = 0.0f;
#pragma unroll
    for (int k = 1; k <= kMaxN; k++) {
        w[k] = (k <= max_order) ? (float)cnt[k - 1] * (float)k : 0.0f;
        tot += w[k];
    }
#pragma unroll
    for (int k = 1; k <= kMaxN; k++) {
        w[k] = (w[k] > 0.0f) ? w[k] + tot * (1.0f / 16.0f) : 0.0f;
        sum += w[k];
    }
    float upto = 0.0f;
    s.lo[kMaxN] = 0;
#pragma unroll
    for (int k = kMaxN; k >= 1; k--) {
        upto += w[k];
        s.lo[k - 1] = min(all, (int)((float)all * (upto / sum) + 0.5f));
    }
    return s;
}

// A bin's turn: its own waves in the first pass, every wave in the second,
// with what its own waves have not taken.
__device__ __forceinline__ bool turn(const BinShare s, int pass) { return pass || s.rank >= 0; }
__device__ __forceinline__ BinShare part(const BinShare s, int pass) { return {pass ? -1 : s.rank, s.size}; }

// One persistent launch over every order (register budget of order 5).
// FORM 0: the implicit form (points as unknowns); 1: the parametric form.
// REFR: the scene has refracting facets; their rows are compiled into this
// kernel only (a branch left in the other kernels slowed the stress
// workload's LM launches by 16% in the parametric and 7% in the implicit
// form, though no lane took it), so such scenes run this schedule.
template <int MODE, bool LDS, int FORM, bool REFR>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OccAll<MODE, FORM>::W, OccAll<MODE, FORM>::W)))
k_lm(KParams kp)
{
    const int *cnt = kp.resume ? kp.spill_cnt : (MODE == MODE_FALLBACK64) ? kp.fb_cnt : kp.bin_cnt;
    const int total = cnt[0] + cnt[1] + cnt[2] + cnt[3] + cnt[4], waves = used_waves(kp, total);
    if (total == 0 || (int)blockIdx.x >= waves) return;  // nothing to solve: skip the staging
    const typename ModeT<MODE>::T *rec = stage_scene<MODE, LDS>(kp);
    // each wave starts with one order (all orders' longest descents begin at
    // once), then helps the others, long paths first so that the short ones
    // fill the tail
    const OrderShare sh = order_share(cnt, 5, waves);
#pragma nounroll
    for (int pass = 0; pass < 2; pass++) {
        if (turn(sh.of(5), pass)) lm_bin<MODE, 5, FORM, true, REFR>(kp, rec, part(sh.of(5), pass));
        if (turn(sh.of(4), pass)) lm_bin<MODE, 4, FORM, true, REFR>(kp, rec, part(sh.of(4), pass));
        if (turn(sh.of(3), pass)) lm_bin<MODE, 3, FORM, true, REFR>(kp, rec, part(sh.of(3), pass));
        if (turn(sh.of(2), pass)) lm_bin<MODE, 2, FORM, true, REFR>(kp, rec, part(sh.of(2), pass));
        if (turn(sh.of(1), pass)) lm_bin<MODE, 1, FORM, true, REFR>(kp, rec, part(sh.of(1), pass));
    }
}

// One persistent launch over orders 3, 2, 1 with the register budget of
// order 3 (twice the waves per SIMD of the all-order kernel in FP32); the
// split schedule runs orders 4 and 5 beside it with their own launches.
template <int MODE, bool LDS, int FORM>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(Occ<MODE, 3, FORM>::W, Occ<MODE, 3, FORM>::W))) k_lm_low(KParams kp)
{
    const int *cnt = kp.resume ? kp.spill_cnt : (MODE == MODE_FALLBACK64) ? kp.fb_cnt : kp.bin_cnt;
    if (cnt[0] + cnt[1] + cnt[2] == 0) return;
    const typename ModeT<MODE>::T *rec = stage_scene<MODE, LDS>(kp);
    const OrderShare sh = order_share(cnt, 3, launch_waves());
#pragma nounroll
    for (int pass = 0; pass < 2; pass++) {
        if (turn(sh.of(3), pass)) lm_bin<MODE, 3, FORM>(kp, rec, part(sh.of(3), pass));
        if (turn(sh.of(2), pass)) lm_bin<MODE, 2, FORM>(kp, rec, part(sh.of(2), pass));
        if (turn(sh.of(1), pass)) lm_bin<MODE, 1, FORM>(kp, rec, part(sh.of(1), pass));
    }
}

// One persistent launch per order, each with its own register budget.
template <int MODE, int N, bool LDS, int FORM>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(Occ<MODE, N, FORM>::W, Occ<MODE, N, FORM>::W))) k_lm_one(KParams kp)
{
    const int total = (kp.resume ? kp.spill_cnt : (MODE == MODE_FALLBACK64) ? kp.fb_cnt : kp.bin_cnt)[N - 1];
    const int waves = N >= 4 ? used_waves(kp, total) : launch_waves();
    if (total == 0 || (int)blockIdx.x >= waves) return;
    const typename ModeT<MODE>::T *rec = stage_scene<MODE, LDS>(kp);
    // fixed-type steps for the planar paths of orders 1-3 here as in the
    // mixed-order kernel (stress LM stage 22.0 -> 21.7 ms, bit-identical)
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    lm_bin<MODE, N, FORM, (N <= 3)>(kp, rec, BinShare{wave, waves});
}

// ------------------------------------------------------------------ kernel table
// order 0: the mixed-order kernel; 1..5: the per-order kernels; 6: the
// kernel of orders 1-3.  refr: the mixed-order kernel with the rows of
// refracting facets (order ignored).  The fallback runs one mixed-order
// launch in the solve's form (from the FP32 end point).
template <int MODE, int FORM, bool LDS>
const void *lm_kernel_of(int order, bool refr)
{
    if (refr) return (const void *)k_lm<MODE, LDS, FORM, true>;
    if constexpr (MODE == MODE_FALLBACK64) {
        return (const void *)k_lm<MODE, LDS, FORM, false>;
    } else {
        switch (order) {
        case 0: return (const void *)k_lm<MODE, LDS, FORM, false>;
        case 1: return (const void *)k_lm_one<MODE, 1, LDS, FORM>;
        case 2: return (const void *)k_lm_one<MODE, 2, LDS, FORM>;
        case 3: return (const void *)k_lm_one<MODE, 3, LDS, FORM>;
        case 4: return (const void *)k_lm_one<MODE, 4, LDS, FORM>;
        case 5: return (const void *)k_lm_one<MODE, 5, LDS, FORM>;
        default: return (const void *)k_lm_low<MODE, LDS, FORM>;
        }
    }
}

template const void *lm_kernel_of<MPT_LM_MODE, MPT_LM_FORM, MPT_LM_LDS != 0>(int order, bool refr);

}  // namespace mpt
