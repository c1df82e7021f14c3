// Kernels around the Levenberg-Marquardt solver of the batched Min-Path-Tracing
// solve (gfx950, wave64); the solver itself is in mpt_lm.hip.
//
//  k_pack            scene records -> packed FP64 world + FP32 TX-local records,
//                    boxes of the facets and patches
//  k_bin_count       histogram of path orders (invalid solves finished here)
//  k_bin_scatter     solve ids grouped by order (one bin per order)
//  k_start           start points and unknowns of the binned paths
//  k_finish          results and routing of the FP32 pass's end points
//  k_polish          FP64 Gauss-Newton polish of the FP32 end points
//  k_accept_*        FP64 acceptance test and ordered compaction
#include "mpt_path.hpp"
#include "mpt_geom.hpp"

namespace mpt {

// ------------------------------------------------------------------ pack
// Ortho-normal pair across a unit vector (Duff et al., "Building an
// orthonormal basis, revisited", JCGT 2017).
__global__ void k_pack(const double *__restrict__ raw, const double *__restrict__ refr, int n_pl, int n_ln, int n_q,
                       int n_c, double tx0, double tx1, double tx2, double *__restrict__ rec64,
                       float *__restrict__ rec32, float *__restrict__ occ)
{
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    const int n_all = n_pl + n_ln + n_q + n_c;
    if (id >= n_all) return;
    const double tx[3] = {tx0, tx1, tx2};
    double o[kRec];
#pragma unroll
    for (int i = 0; i < kRec; i++) o[i] = 0.0;
    // raw arrays are concatenated type-major with their own widths
    const int t = prim_type(id, n_pl, n_pl + n_ln, n_pl + n_ln + n_q);
    size_t off;
    if (t == TP) off = (size_t)id * 13;
    else if (t == TL) off = (size_t)n_pl * 13 + (size_t)(id - n_pl) * 8;
    else if (t == TQ) off = (size_t)n_pl * 13 + (size_t)n_ln * 8 + (size_t)(id - n_pl - n_ln) * 17;
    else off = (size_t)n_pl * 13 + (size_t)n_ln * 8 + (size_t)n_q * 17 + (size_t)(id - n_pl - n_ln - n_q) * 7;
    const double *r = raw + off;
    const int w = (t == TP) ? 13 : (t == TL) ? 8 : (t == TQ) ? 17 : 7;
    for (int i = 0; i < w; i++) o[i] = r[i];
    if (t == TL) across_dir(r + 3, o + 8, o + 11);
    // frames of the parametric form
    if (t == TP) {
        const double l = sqrt(r[7] * r[7] + r[8] * r[8] + r[9] * r[9]);
        for (int i = 0; i < 3; i++) o[13 + i] = l > 0.0 ? r[7 + i] / l : 0.0;
        // refractive indices of a refracting facet (0, 0: a mirror)
        if (refr) {
            o[16] = refr[2 * (size_t)id];
            o[17] = refr[2 * (size_t)id + 1];
        }
    }
    if (t == TC) across_dir(r + 3, o + 7, o + 10);
    if (t == TQ) {
        // a paraboloid of revolution: A = kappa (I - ax ax^T), b = -ax, c = 0
        const double kap = 0.5 * (r[3] + r[6] + r[8]);
        const double *ax = r + 13;
        const double Am[3][3] = {{r[3], r[4], r[5]}, {r[4], r[6], r[7]}, {r[5], r[7], r[8]}};
        double err = fabs(r[12]);
        for (int i = 0; i < 3; i++) {
            err = fmax(err, fabs(r[9 + i] + ax[i]));
            for (int j = 0; j < 3; j++) err = fmax(err, fabs(Am[i][j] - kap * ((i == j ? 1.0 : 0.0) - ax[i] * ax[j])));
        }
        o[17] = (kap > 0.0 && err <= 1e-9 * (1.0 + kap)) ? kap : -1.0;
    }
    for (int i = 0; i < kRec; i++) rec64[(size_t)id * kRec + i] = o[i];
    // TX-local FP32 copy: positions shifted by TX, plane offsets adjusted
    double l[kRec];
    for (int i = 0; i < kRec; i++) l[i] = o[i];
    if (t == TP) {
        l[3] = o[3] - (o[0] * tx[0] + o[1] * tx[1] + o[2] * tx[2]);
        for (int i = 0; i < 3; i++) l[4 + i] = o[4 + i] - tx[i];
    } else {
        for (int i = 0; i < 3; i++) l[i] = o[i] - tx[i];
    }
    for (int i = 0; i < kRec; i++) rec32[(size_t)id * kRec + i] = (float)l[i];
    // the box of a facet or patch
    if (t == TP || t == TQ) occluder_box(t, o, occ + (size_t)(t == TP ? id : id - n_ln) * 8);
}

// ------------------------------------------------------------------ workspace counters
__global__ void k_zero_i32(int *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// ------------------------------------------------------------------ binning
__device__ inline bool finite3(const double *v) { return isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]); }

// Order of a solve, or -1 if the solve is invalid (order, receiver or ids).
__device__ inline int valid_order(const BatchDev &b, int64_t i, int n_all)
{
    const int ord = b.order[i];
    bool bad = ord < 1 || ord > kMaxN;
    const int ri = b.rx_index[i];
    bad = bad || ri < 0 || ri >= b.n_rx;
    if (!bad) {
        bad = !finite3(b.rx + 3 * (size_t)ri);
        for (int k = 0; k < kMaxN; k++)
            if (k < ord) {
                const int id = b.prim[(size_t)k * b.n + i];
                bad = bad || id < 0 || id >= n_all;
            }
    }
    return bad ? -1 : ord;
}

// Binning by (order, sequence of primitive types): solves of one order are
// grouped, and within an order by the base-4 code of their type sequence, so
// the lanes of a wave mostly follow one type path (no divergence between
// reflection and diffraction code).  Key = kKeyBase[order] + code.
constexpr int kBinBlock = 256;
// solves per thread, their loads issued together (stress workload binning:
// 1.34 ms with two solves per thread each loaded as a chain of dependent
// loads; 1.11, 0.73 and 0.69 ms with the loads issued together and two,
// four and eight solves per thread; 0.77-0.80 ms with 16-32 solves per
// thread in chunks of eight, which halves or quarters the blocks' atomics
// on the key counters but loads the ids again after the atomics)
constexpr int kBinItems = 8;
constexpr int kBinPerBlock = kBinBlock * kBinItems;
constexpr int kNumKeys = 4 + 16 + 64 + 256 + 1024;
__device__ __constant__ int kKeyBase[kMaxN + 1] = {0, 0, 4, 20, 84, 340};

// A solve's order, receiver and ids as the binning reads them: every load
// is issued before any is used (the id rows beyond the order are the
// caller's memory as well), so a thread's loads are in flight together
// instead of one dependent round trip after another.  ord = -1 marks an
// invalid solve (the same test as valid_order).
struct SolveIds {
    int ord, ri, id[kMaxN];
};

__device__ inline void load_ids(const BatchDev &b, int64_t i, SolveIds &r)
{
    r.ord = b.order[i];
    r.ri = b.rx_index[i];
#pragma unroll
    for (int k = 0; k < kMaxN; k++) r.id[k] = b.prim[(size_t)k * b.n + i];
}

__device__ inline void check_ids(const BatchDev &b, int n_all, SolveIds &r)
{
    bool bad = r.ord < 1 || r.ord > kMaxN || r.ri < 0 || r.ri >= b.n_rx;
    if (!bad) {
        bad = !finite3(b.rx + 3 * (size_t)r.ri);
#pragma unroll
        for (int k = 0; k < kMaxN; k++)
            if (k < r.ord) bad = bad || r.id[k] < 0 || r.id[k] >= n_all;
    }
    if (bad) r.ord = -1;
}

__device__ inline int bin_key(const SolveIds &r, int a, int bb, int c)
{
    int code = 0, mul = 1;
#pragma unroll
    for (int k = 0; k < kMaxN; k++)
        if (k < r.ord) {
            code += prim_type(r.id[k], a, bb, c) * mul;
            mul *= 4;
        }
    return kKeyBase[r.ord] + code;
}

// The results of an invalid solve.
__device__ __forceinline__ void bad_solve(const BatchDev &b, const OutDev &out, int64_t i)
{
    for (int q = 0; q < kRow; q++) out.x[(size_t)i * kRow + q] = 0.0;
    out.cost[i] = __builtin_huge_val();
    out.iters[i] = 0;
    out.status[i] = ST_BAD;
    if (out.stage)
        for (int q = 0; q < 4; q++) out.stage[(size_t)q * b.n + i] = 0;
}

__global__ void __launch_bounds__(kBinBlock) k_bin_count(BatchDev b, OutDev out, int n_all, int n_pl, int n_pl_ln,
                                                          int n_pl_ln_q, int *__restrict__ key_cnt)
{
    __shared__ int loc[kNumKeys];
    for (int k = threadIdx.x; k < kNumKeys; k += kBinBlock) loc[k] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kBinPerBlock;
    SolveIds r[kBinItems];
#pragma unroll
    for (int j = 0; j < kBinItems; j++) {
        const int64_t i = base + (int64_t)j * kBinBlock + threadIdx.x;
        if (i < b.n) load_ids(b, i, r[j]);
    }
#pragma unroll
    for (int j = 0; j < kBinItems; j++) {
        const int64_t i = base + (int64_t)j * kBinBlock + threadIdx.x;
        if (i < b.n) check_ids(b, n_all, r[j]);
    }
#pragma unroll
    for (int j = 0; j < kBinItems; j++) {
        const int64_t i = base + (int64_t)j * kBinBlock + threadIdx.x;
        if (i >= b.n) break;
        if (r[j].ord < 0) {
            bad_solve(b, out, i);
        } else {
            // the later stages' iteration counts are zero: written here,
            // coalesced, so that the solver kernels store only what a path
            // produces (the solver writes a path's whole point row)
            if (out.stage)
                for (int q = 1; q < 4; q++) out.stage[(size_t)q * b.n + i] = 0;
            atomicAdd(&loc[bin_key(r[j], n_pl, n_pl_ln, n_pl_ln_q)], 1);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kNumKeys; k += kBinBlock)
        if (loc[k]) atomicAdd(&key_cnt[k], loc[k]);
}

// One block: exclusive scan of the key counts -> key offsets; per-order
// totals -> bin counts (the bins of the LM kernels are the orders).
// curved (or null): the start of each order's part of the list of the
// solves with a curved object ([5], then used as cursors by the scatter),
// and curved[25] receives the list's length (the counter slots of the
// solve's workspace are laid out so).
__global__ void __launch_bounds__(1024) k_bin_offsets(const int *__restrict__ key_cnt, int *__restrict__ key_off,
                                                       int *__restrict__ bin_cnt, int *__restrict__ curved)
{
    __shared__ int part[1024];
    __shared__ int offs[kNumKeys + 1];
    const int t = threadIdx.x;
    const int per = (kNumKeys + 1023) / 1024;
    const int lo = t * per, hi = min(lo + per, kNumKeys);
    int c[per], sum = 0;
#pragma unroll
    for (int q = 0; q < per; q++) {
        c[q] = (lo + q < hi) ? key_cnt[lo + q] : 0;
        sum += c[q];
    }
    part[t] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int v = (t >= d) ? part[t - d] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int run = (t == 0) ? 0 : part[t - 1];
#pragma unroll
    for (int q = 0; q < per; q++)
        if (lo + q < hi) {
            key_off[lo + q] = run;
            offs[lo + q] = run;
            run += c[q];
        }
    if (t == 1023) offs[kNumKeys] = part[1023];
    __syncthreads();
    // per-order totals: the keys of one order are contiguous
    __shared__ int ccnt[kMaxN];
    if (t < kMaxN) {
        const int kb = kKeyBase[t + 1], ke = (t + 1 < kMaxN) ? kKeyBase[t + 2] : kNumKeys;
        bin_cnt[t] = offs[ke] - offs[kb];
        ccnt[t] = 0;
    }
    if (!curved) return;
    __syncthreads();
    // the solves with a curved object (a type digit of 2 or 3 in the key),
    // per order: each thread adds its own keys' counts
#pragma unroll
    for (int q = 0; q < per; q++) {
        const int k = lo + q;
        int o = 1;
        while (o < kMaxN && k >= kKeyBase[o + 1]) o++;
        if (k < hi && c[q] && ((k - kKeyBase[o]) & 0x2AA) != 0) atomicAdd(&ccnt[o - 1], c[q]);
    }
    __syncthreads();
    if (t == 0) {
        int run = 0;
        for (int o = 0; o < kMaxN; o++) {
            curved[o] = run;
            run += ccnt[o];
        }
        curved[25] = run;
    }
}

// Each solve's slot in bin order (by_solve: perm[solve] = slot, -1 for an
// invalid solve; else perm[slot] = solve).  With `rows`, the
// solves whose list holds a paraboloid or a circle (a type digit of 2 or 3
// in the key) are also listed there, grouped by order (`curved`: each
// order's cursor, one atomic per block and order), so that the waves of the
// learned start's kernels hold one order each.
__global__ void __launch_bounds__(kBinBlock) k_bin_scatter(BatchDev b, int n_all, int n_pl, int n_pl_ln, int n_pl_ln_q,
                                                            const int *__restrict__ key_off,
                                                            int *__restrict__ key_cursor, int *__restrict__ perm,
                                                            int by_solve, int *__restrict__ rows,
                                                            int *__restrict__ curved)
{
    __shared__ int loc[kNumKeys];
    __shared__ int gbase[kNumKeys];
    __shared__ int ccount[kMaxN], cbase[kMaxN];
    for (int k = threadIdx.x; k < kNumKeys; k += kBinBlock) loc[k] = 0;
    if (threadIdx.x < kMaxN) ccount[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kBinPerBlock;
    int key[kBinItems], rank[kBinItems], crank[kBinItems];
    SolveIds r[kBinItems];
#pragma unroll
    for (int j = 0; j < kBinItems; j++) {
        const int64_t i = base + (int64_t)j * kBinBlock + threadIdx.x;
        r[j].ord = -1;
        if (i < b.n) load_ids(b, i, r[j]);
    }
#pragma unroll
    for (int j = 0; j < kBinItems; j++) {
        const int64_t i = base + (int64_t)j * kBinBlock + threadIdx.x;
        if (i < b.n) check_ids(b, n_all, r[j]);
    }
#pragma unroll
    for (int j = 0; j < kBinItems; j++) {
        const int ord = r[j].ord;
        key[j] = (ord > 0) ? bin_key(r[j], n_pl, n_pl_ln, n_pl_ln_q) : -1;
        rank[j] = (key[j] >= 0) ? atomicAdd(&loc[key[j]], 1) : 0;
        // base-4 type digits: 2 (quadric) and 3 (circle) have bit 1 set
        const bool cur = rows && key[j] >= 0 && ((key[j] - kKeyBase[ord > 0 ? ord : 1]) & 0x2AA) != 0;
        crank[j] = cur ? atomicAdd(&ccount[ord - 1], 1) : -1;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kNumKeys; k += kBinBlock)
        gbase[k] = loc[k] ? key_off[k] + atomicAdd(&key_cursor[k], loc[k]) : 0;
    if (rows && threadIdx.x < kMaxN)
        cbase[threadIdx.x] = ccount[threadIdx.x] ? atomicAdd(&curved[threadIdx.x], ccount[threadIdx.x]) : 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kBinItems; j++) {
        const int64_t i = base + (int64_t)j * kBinBlock + threadIdx.x;
        const int slot = key[j] >= 0 ? gbase[key[j]] + rank[j] : -1;
        if (by_solve) {
            if (i < b.n) perm[i] = slot;
        } else if (slot >= 0) {
            perm[slot] = (int)i;
        }
        if (crank[j] >= 0) rows[cbase[r[j].ord - 1] + crank[j]] = (int)i;
    }
}

// The whole binning of a small batch by one block: clears the workspace's
// counters, counts the keys, scans them and places the solves, with the keys
// and ranks in LDS.  Bound by the latency of its loads.  Four launches (clear,
// count, offsets, scatter) took 26 us and the gaps between them on 16,384
// solves, this one 24.6 us (5.4 us on 64); with more solves the one block's
// loads cost more than the launches.
constexpr int kSmallBin = 16384;
constexpr int kSmallItems = kSmallBin / 1024;

__global__ void __launch_bounds__(1024) k_bin_small(BatchDev b, OutDev out, int n_all, int n_pl, int n_pl_ln,
                                                     int n_pl_ln_q, int *__restrict__ ctr, int n_ctr,
                                                     int *__restrict__ perm, int by_solve)
{
    __shared__ int cnt[2048];        // key counts, then offsets
    __shared__ int wsum[16];
    __shared__ uint16_t skey[kSmallBin], srank[kSmallBin];
    const int t = threadIdx.x, lane = t & 63;
    for (int i = t; i < n_ctr; i += 1024)
        if (i >= kMaxN) ctr[i] = 0;  // the first five receive the orders' totals below
    cnt[t] = cnt[t + 1024] = 0;
    __syncthreads();
    for (int j0 = 0; j0 < kSmallItems; j0 += 4) {
        if ((int64_t)j0 * 1024 >= b.n) break;  // block-uniform
        SolveIds r[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int64_t i = (int64_t)(j0 + j) * 1024 + t;
            if (i < b.n) load_ids(b, i, r[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int64_t i = (int64_t)(j0 + j) * 1024 + t;
            if (i >= b.n) continue;
            check_ids(b, n_all, r[j]);
            skey[i] = 0xffffu;
            if (r[j].ord < 0) {
                bad_solve(b, out, i);
            } else {
                if (out.stage)
                    for (int q = 1; q < 4; q++) out.stage[(size_t)q * b.n + i] = 0;
                const int key = bin_key(r[j], n_pl, n_pl_ln, n_pl_ln_q);
                skey[i] = (uint16_t)key;
                srank[i] = (uint16_t)atomicAdd(&cnt[key], 1);
            }
        }
    }
    __syncthreads();
    // exclusive scan of the counts, two per thread
    const int a0 = cnt[2 * t], a1 = cnt[2 * t + 1];
    int incl = a0 + a1;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int v = __shfl_up(incl, d);
        if (lane >= d) incl += v;
    }
    if (lane == 63) wsum[t >> 6] = incl;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < (t >> 6); w++) before += wsum[w];
    cnt[2 * t] = before + incl - a0 - a1;
    cnt[2 * t + 1] = before + incl - a1;
    __syncthreads();
    if (t < kMaxN) ctr[t] = cnt[t + 1 < kMaxN ? kKeyBase[t + 2] : kNumKeys] - cnt[kKeyBase[t + 1]];
    for (int64_t i = t; i < b.n; i += 1024) {
        const int key = skey[i];
        const int slot = key != 0xffff ? cnt[key] + srank[i] : -1;
        if (by_solve) perm[i] = slot;
        else if (slot >= 0) perm[slot] = (int)i;
    }
}

// ------------------------------------------------------------------ learned start
// The network's points, projected onto their objects, replace the
// straight-line start of a path only when their FP64 cost is lower: the
// solver's own cost judges the prediction.  Writes the chosen start points
// into x0l (rows of the path; one thread per served path).
template <int N, bool REFR>
__device__ void choose_start(const SceneDev &s, const BatchDev &b, int64_t i, double *__restrict__ x0l, double gain)
{
    SceneT<double> s64;
    s64.rec = s.rec64;
    PathIn<double, N> q;
    const int ri = b.rx_index[i];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        s64.tx[c] = s.tx[c];
        s64.glo[c] = s.glo[c];
        s64.ghi[c] = s.ghi[c];
        q.rx[c] = b.rx[3 * (size_t)ri + c];
    }
    q.planar = false;
#pragma unroll
    for (int k = 0; k < N; k++) {
        q.id[k] = b.prim[(size_t)k * b.n + i];
        q.ty[k] = prim_type(q.id[k], s.n_pl, s.n_pl_ln, s.n_pl_ln_q);
    }
    double X0[3 * N], Xn[3 * N];
    bool okn = true;
#pragma unroll
    for (int k = 0; k < N; k++) {
        const double a = line_fraction(q.ty[k], s.rec64 + (size_t)q.id[k] * kRec, s.tx, q.rx, k, N);
        double P[3], Pn[3];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            P[c] = s.tx[c] + a * (q.rx[c] - s.tx[c]);
            Pn[c] = x0l[(size_t)i * kRow + 3 * k + c];
            okn = okn && isfinite(Pn[c]);
        }
        const double *r = s.rec64 + (size_t)q.id[k] * kRec;
        project(q.ty[k], r, P, X0 + 3 * k);
        project(q.ty[k], r, okn ? Pn : P, Xn + 3 * k);
    }
    double c0 = 0.0, r0 = 0.0, c1 = 0.0, r1 = 0.0;
    const bool ok0 = eval_cost<double, N, REFR>(s64, q, X0, nullptr, c0, r0);
    const bool ok1 = okn && eval_cost<double, N, REFR>(s64, q, Xn, nullptr, c1, r1);
    const bool net = ok1 && (!ok0 || c1 < gain * c0);
#pragma unroll
    for (int j = 0; j < 3 * N; j++) x0l[(size_t)i * kRow + j] = net ? Xn[j] : X0[j];
}

template <bool REFR>
__global__ void __launch_bounds__(256) k_learned_choose(SceneDev s, BatchDev b, const int *__restrict__ rows,
                                                        const int *__restrict__ count, int all,
                                                        double *__restrict__ x0l, double gain)
{
    const int64_t m = all ? b.n : (int64_t)*count;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = all ? t : rows[t];
        switch (valid_order(b, i, s.n_all)) {
        case 1: choose_start<1, REFR>(s, b, i, x0l, gain); break;
        case 2: choose_start<2, REFR>(s, b, i, x0l, gain); break;
        case 3: choose_start<3, REFR>(s, b, i, x0l, gain); break;
        case 4: choose_start<4, REFR>(s, b, i, x0l, gain); break;
        case 5: choose_start<5, REFR>(s, b, i, x0l, gain); break;
        default: break;
        }
    }
}

// ------------------------------------------------------------------ start of the paths
// The start of every valid solve, one thread each in solve order (coalesced
// ids): its start point and unknowns to its state row, or, when no iteration
// is to run, its results.  A kernel of its own because the solver's lanes
// start a few paths at a time: there the dependent gathers and the FP64 start
// arithmetic ran on the lanes that happened to be idle, 20 us per refill with
// the wave's other lanes waiting (street canyon, 8 to 12 refills per wave),
// and their registers counted in every iteration.
// The learned starts begin their paths after the network (k_learned_begin).
constexpr int kStartBlock = 256;

// Ids, types and receiver of solve i (valid: checked by the binning).
struct PathRef {
    int n, id[kMaxN], ty[kMaxN];
    double rx[3];
};

__device__ __forceinline__ PathRef path_ref(const SceneDev &s, const BatchDev &b, int64_t i)
{
    PathRef p;
    p.n = b.order[i];
    const int ri = b.rx_index[i];
#pragma unroll
    for (int k = 0; k < kMaxN; k++) p.id[k] = b.prim[(size_t)k * b.n + i];
#pragma unroll
    for (int c = 0; c < 3; c++) p.rx[c] = b.rx[3 * (size_t)ri + c];
#pragma unroll
    for (int k = 0; k < kMaxN; k++) p.ty[k] = prim_type(p.id[k], s.n_pl, s.n_pl_ln, s.n_pl_ln_q);
    return p;
}

// Does the network serve this path (paths with a curved object; planes and
// straight edges keep the straight-line start)?
__device__ __forceinline__ bool served(const KParams &kp, const PathRef &p)
{
    bool net = kp.o.init == INIT_LEARNED_ALL;
    if (kp.o.init == INIT_LEARNED) {
#pragma unroll
        for (int k = 0; k < kMaxN; k++) net = net || (k < p.n && (p.ty[k] == TQ || p.ty[k] == TC));
    }
    return net;
}

// Bound by the memory pipe (78% busy) and the FP64 arithmetic of four types in
// one wave (52%): each record is read once (load_record) and the rows leave
// through LDS (rows_store).  16.8 M paths 2.55 -> 1.43 ms, 4.5 M 0.29 -> 0.19 ms.
template <int MODE, int FORM>
__global__ void __launch_bounds__(kStartBlock) k_start(KParams kp)
{
    __shared__ __align__(16) float rows[kStartBlock / 64 * kWaveRows];
    const int64_t i = (int64_t)blockIdx.x * kStartBlock + threadIdx.x;
    int slot = -1;
    bool live = i < kp.b.n;
    if (live) {
        if (kp.rows) {
            slot = kp.perm[i];
            live = slot >= 0;
        } else {
            live = valid_order(kp.b, i, kp.s.n_all) >= 0;
        }
    }
    PathRef p;
    if (live) {
        p = path_ref(kp.s, kp.b, i);
        live = !served(kp, p);
    }
    if (!__any(live)) return;
    const double *x0 = (kp.o.init == INIT_USER) ? kp.b.x0 + (size_t)i * kRow : nullptr;
    begin_path<MODE, FORM>(kp, live, slot, i, p.n, p.id, p.ty, p.rx, x0, rows + (threadIdx.x >> 6) * kWaveRows);
}

// The learned starts: begin the served paths from the chosen points.
template <int MODE, int FORM>
__global__ void __launch_bounds__(kStartBlock) k_learned_begin(KParams kp, const int *__restrict__ list,
                                                               const int *__restrict__ count)
{
    __shared__ __align__(16) float rows[kStartBlock / 64 * kWaveRows];
    const int64_t m = list ? (int64_t)*count : kp.b.n;
    // all lanes of a wave go round together
    for (int64_t t0 = (int64_t)blockIdx.x * kStartBlock + (threadIdx.x & ~63); t0 < m;
         t0 += (int64_t)gridDim.x * kStartBlock) {
        const int64_t t = t0 + (threadIdx.x & 63);
        bool live = t < m;
        int64_t i = 0;
        int slot = -1;
        PathRef p;
        if (live) {
            i = list ? list[t] : t;
            slot = kp.rows ? kp.perm[i] : -1;
            live = kp.rows ? slot >= 0 : valid_order(kp.b, i, kp.s.n_all) >= 0;
            if (live) p = path_ref(kp.s, kp.b, i);
        }
        begin_path<MODE, FORM>(kp, live, slot, i, p.n, p.id, p.ty, p.rx, kp.x0_learned + (size_t)i * kRow,
                               rows + (threadIdx.x >> 6) * kWaveRows);
    }
}

#define MPT_BY_MODE_FORM(kern, g, ...)                                                                  \
    do {                                                                                                \
        if (mode == MODE_FP32) {                                                                        \
            if (form) hipLaunchKernelGGL((kern<MODE_FP32, 1>), g, dim3(kStartBlock), 0, st, __VA_ARGS__); \
            else hipLaunchKernelGGL((kern<MODE_FP32, 0>), g, dim3(kStartBlock), 0, st, __VA_ARGS__);      \
        } else {                                                                                        \
            if (form) hipLaunchKernelGGL((kern<MODE_PLAIN64, 1>), g, dim3(kStartBlock), 0, st, __VA_ARGS__); \
            else hipLaunchKernelGGL((kern<MODE_PLAIN64, 0>), g, dim3(kStartBlock), 0, st, __VA_ARGS__);   \
        }                                                                                               \
    } while (0)

void launch_start(int mode, int form, const KParams &kp, hipStream_t st)
{
    if (kp.b.n == 0) return;
    MPT_BY_MODE_FORM(k_start, dim3((unsigned)((kp.b.n + kStartBlock - 1) / kStartBlock)), kp);
}

// list, count: the served solves, or null for every solve
void launch_learned_begin(int mode, int form, const KParams &kp, const int *list, const int *count, hipStream_t st)
{
    if (kp.b.n == 0) return;
    const unsigned g = (unsigned)std::min<int64_t>((kp.b.n + kStartBlock - 1) / kStartBlock, 8192);
    MPT_BY_MODE_FORM(k_learned_begin, dim3(g), kp, list, count);
}

// ------------------------------------------------------------------ end of the FP32 pass
// The FP32 pass leaves each path's unknowns, cost, residual, iterations and
// status in its state row; this kernel writes the path's results (world
// points and scalars), routes it, and lists the paths to polish, grouped by
// order.  One thread per solve in solve order, so that every result is
// written coalesced and only the state row is gathered (a whole line).
// The rows go through LDS (rows_load, rows_store): a wave's gather of 64
// rows and store of 64 others cost the memory pipe eight lines an instruction
// instead of 64.  16.8 M paths 1.67 -> 1.51 ms (the pipe 73% busy, most of it
// the records of the extent test), 4.5 M 0.42 -> 0.35 ms.
//
// Routing: FP32 end points whose residual is below the gate look like roots
// and are polished in FP64; the others are final (no path).  FP64 re-solves
// the path from its FP32 end point on numerical trouble in FP32: a degenerate
// iterate, a path of planes and straight edges still far from a root at its
// iteration cap (such descents reach their unique root quickly, so the cap
// alone is no evidence that none exists), or - decided by the polish - a
// converged or stalled FP32 point that does not polish.  A path through a
// refracting facet has a unique root (the optical length is convex), so a
// descent that ends far from a root goes to the FP64 fallback as well.
constexpr int kFinBlock = 256;
// slots per thread at most: a block takes its places in the polish and the
// fallback lists with one device-wide atomic per order, and atomics on one
// counter are served one at a time (8192 blocks' atomics took 0.29 ms on the
// stress workload; an atomic per path to the fallback, 9,200 of them, 0.06 ms of
// the 0.11 ms on 262,144 paths through glass)
constexpr int kFinItems = 16;  // four bits of a thread's word each

enum : int { END_POLISH = 0, END_FALLBACK = 1, END_FINAL = 2 };

// One path's end: its results, and the list it goes to.
template <int FORM, bool REFR>
__device__ __forceinline__ int finish_path(const KParams &kp, int64_t i, int &order, float *mine)
{
    constexpr int D = (FORM ? 2 : 3) * kMaxN;
    const double sh[3] = {kp.s.tx[0], kp.s.tx[1], kp.s.tx[2]};
    const f32x4l *rf = (const f32x4l *)mine;  // the state row
    float L[(D + 3) / 4 * 4];
#pragma unroll
    for (int j = 0; j < D; j += 4) {
        const f32x4l v = rf[j / 4];
#pragma unroll
        for (int q = 0; q < 4; q++) L[j + q] = v[q];
    }
    const f32x4l e = rf[RW_C / 4];
    const float C = e[0], rinf = e[1];
    const int it = __float_as_int(e[2]), st = __float_as_int(e[3]);
    const int late = kp.spill_t > 0 ? it - ((const i32a *)mine)[RW_ID] : 0;
    const PathRef p = path_ref(kp.s, kp.b, i);
    order = p.n;
    bool planar = true, refr_path = false;
#pragma unroll
    for (int k = 0; k < kMaxN; k++)
        if (k < p.n) {
            const bool refr = REFR && p.ty[k] == TP && kp.s.rec64[(size_t)p.id[k] * kRec + 16] > 0.0;
            planar = planar && (p.ty[k] == TL || (p.ty[k] == TP && !refr));
            refr_path = refr_path || refr;
        }
    // the point row replaces the state row
    double *Xw = (double *)mine;
    world_points<kMaxN, FORM, float>(kp.s.rec32, p.n, p.id, p.ty, L, sh, Xw);
    Xw[kRow - 1] = 0.0;
    kp.out.cost[i] = (double)C;
    kp.out.iters[i] = it;
    if (kp.out.stage) {
        kp.out.stage[i] = it;
        if (kp.spill_t > 0) kp.out.stage[(size_t)3 * kp.b.n + i] = late;
    }
    int code = st;
    // on a refracted path the gate is at least 30 times the FP32 rounding
    // level of its residual: a law row carries the rounding of its unit
    // directions (eps32 |X| / shortest segment) times its scale (up to the
    // longest segment), which reaches 1e-2 m on a thin glass pane far from TX
    double gate = kp.o.polish_gate;
    if (refr_path) {
        double rx_w[3], xmax = 0.0, smin = __builtin_huge_val(), smax = 0.0;
#pragma unroll
        for (int c = 0; c < 3; c++) rx_w[c] = (double)(float)(p.rx[c] - sh[c]) + sh[c];
#pragma unroll
        for (int k = 0; k <= kMaxN; k++) {
            if (k > p.n) continue;
            double e2 = 0.0;
#pragma unroll
            for (int c = 0; c < 3; c++) {
                const double a = (k == 0) ? kp.s.tx[c] : Xw[3 * (k > 0 ? k - 1 : 0) + c];
                const double bq = (k == p.n) ? rx_w[c] : Xw[3 * (k < kMaxN ? k : 0) + c];
                e2 += (bq - a) * (bq - a);
                if (k < p.n) xmax = fmax(xmax, fabs(Xw[3 * (k < kMaxN ? k : 0) + c] - kp.s.tx[c]));
            }
            smin = fmin(smin, sqrt(e2));
            smax = fmax(smax, sqrt(e2));
        }
        gate = fmax(gate, 30.0 * 6e-8 * (1.0 + xmax) * smax / fmax(smin, 1e-12));
    }
    const bool small_res = (double)rinf <= gate;
    bool to_polish = small_res && (st == ST_CONV || st == ST_MAXIT || st == ST_LOCALMIN || st == ST_STALL);
    const bool to_fb = (st == ST_DEGEN) || (st == ST_MAXIT && planar && !small_res) || (refr_path && !small_res);
    // a root-like end point far outside a finite extent: the polish and the
    // fallback stay next to it (within a few times its residual), so the path
    // cannot be accepted
    if (to_polish && kp.o.extent_skip > 0.0 &&
        outside_extent(kp.s.rec64, p.n, p.id, p.ty, Xw, kp.o.extent_skip + 100.0 * (double)rinf)) {
        to_polish = false;
        code = ST_OUTSIDE;
    }
    if (to_polish) {
        const bool rootlike = (double)rinf <= kp.o.tau_root32;
        code = (rootlike && (st == ST_CONV || st == ST_STALL)) ? ROUTE_POLISH_FB
               : (st == ST_MAXIT)                             ? ROUTE_POLISH_MAXIT
                                                              : ROUTE_POLISH_LOCALMIN;
    } else if (to_fb && kp.o.fallback) {
        code = ST_RUNNING;
    }
    kp.out.status[i] = (uint8_t)code;
    return to_polish ? END_POLISH : code == ST_RUNNING ? END_FALLBACK : END_FINAL;
}

template <int FORM, bool REFR>
__global__ void __launch_bounds__(kFinBlock, 4) k_finish(KParams kp, int items)
{
    __shared__ __align__(16) float rows[kFinBlock / 64 * kWaveRows];
    __shared__ int lcnt[2 * kMaxN], lbase[2 * kMaxN];  // polish lists, then fallback lists
    float *w = rows + (threadIdx.x >> 6) * kWaveRows;
    if (threadIdx.x < 2 * kMaxN) lcnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * kFinBlock * items + threadIdx.x;
    uint64_t listed = 0;  // four bits per item: 1 + the path's list, or 0
#pragma nounroll
    for (int j = 0; j < items; j++) {
        const int64_t i = b0 + j * kFinBlock;
        const bool live = i < kp.b.n && kp.out.status[i] == ST_RUNNING;
        if (!__any(live)) continue;
        // a lane without a path reads a row that no other wave writes: its own, or
        // the batch's last, which is this wave's as well
        rows_load(w, state_row(kp, live && kp.rows ? kp.perm[i] : 0, min(i, kp.b.n - 1)));
        if (live) {
            int ord;
            const int end = finish_path<FORM, REFR>(kp, i, ord, w + __lane_id() * kRowWords);
            if (end != END_FINAL) {
                const int q = end * kMaxN + ord - 1;
                listed |= (uint64_t)(q + 1) << (4 * j);
                atomicAdd(&lcnt[q], 1);
            }
        }
        rows_store(w, live ? kp.out.x + (size_t)i * kRow : nullptr);
    }
    __syncthreads();
    if (threadIdx.x < 2 * kMaxN) {
        const bool fb = threadIdx.x >= kMaxN;
        const int c = lcnt[threadIdx.x], ord = (int)threadIdx.x - (fb ? kMaxN : 0) + 1;
        int *cnt = fb ? kp.fb_cnt : kp.pol_cnt;
        lbase[threadIdx.x] = bin_offset(kp.bin_cnt, ord) + (c ? atomicAdd(&cnt[ord - 1], c) : 0);
    }
    __syncthreads();
    for (int j = 0; j < items; j++) {
        const int q = (int)(listed >> (4 * j)) & 15;
        if (q) (q > kMaxN ? kp.fb_list : kp.pol_list)[atomicAdd(&lbase[q - 1], 1)] = (int)(b0 + j * kFinBlock);
    }
}

void launch_finish(int form, bool refr, const KParams &kp, int cu, hipStream_t st)
{
    if (kp.b.n == 0) return;
    // one slot per thread while the blocks fit on the device at once
    const int64_t per = (kp.b.n + (int64_t)kFinBlock * cu * 4 - 1) / ((int64_t)kFinBlock * cu * 4);
    const int items = (int)std::min<int64_t>(per, kFinItems);
    const int64_t slots = (int64_t)kFinBlock * items;
    const dim3 g((unsigned)((kp.b.n + slots - 1) / slots)), b(kFinBlock);
    if (form) {
        if (refr) hipLaunchKernelGGL((k_finish<1, true>), g, b, 0, st, kp, items);
        else hipLaunchKernelGGL((k_finish<1, false>), g, b, 0, st, kp, items);
    } else {
        if (refr) hipLaunchKernelGGL((k_finish<0, true>), g, b, 0, st, kp, items);
        else hipLaunchKernelGGL((k_finish<0, false>), g, b, 0, st, kp, items);
    }
}

// ------------------------------------------------------------------ polish
// Undamped FP64 Gauss-Newton from the FP32 end point (world frame).
template <int N, bool REFR>
__device__ void polish_bin(const KParams &kp)
{
    const int count = kp.pol_cnt[N - 1];
    if (count == 0) return;
    const int off = bin_offset(kp.bin_cnt, N);
    SceneT<double> sc;
    sc.rec = kp.s.rec64;
#pragma unroll
    for (int i = 0; i < 3; i++) { sc.tx[i] = kp.s.tx[i]; sc.glo[i] = kp.s.glo[i]; sc.ghi[i] = kp.s.ghi[i]; }
    constexpr int M = 3 * N;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < count; q += gridDim.x * blockDim.x) {
        const int sid = kp.pol_list[off + q];
        PathIn<double, N> p;
        const int ri = kp.b.rx_index[sid];
#pragma unroll
        for (int i = 0; i < 3; i++) p.rx[i] = kp.b.rx[3 * (size_t)ri + i];
#pragma unroll
        for (int k = 0; k < N; k++) {
            p.id[k] = kp.b.prim[(size_t)k * kp.b.n + sid];
            p.ty[k] = prim_type(p.id[k], kp.s.n_pl, kp.s.n_pl_ln, kp.s.n_pl_ln_q);
        }
        double X[M];
#pragma unroll
        for (int j = 0; j < M; j++) X[j] = kp.out.x[(size_t)sid * kRow + j];
        bool ok = true, small = false;
        int steps = 0;
        for (int ps = 0; ps < kp.o.polish_steps && ok && !small; ps++) {
            double A[Band<N>::SIZE], g[M], C, rinf;
            ok = assemble<double, N, REFR>(sc, p, X, A, g, C, rinf);
            if (!ok) break;
            steps++;
            if (rinf <= kp.o.tol_res) { small = true; break; }
            double dmax = 0.0;
#pragma unroll
            for (int i = 0; i < M; i++) dmax = fmax(dmax, A[Band<N>::at(i, i)]);
#pragma unroll
            for (int i = 0; i < M; i++) A[Band<N>::at(i, i)] += 1e-15 * dmax;
            ok = chol_band<double, N>(A);
            if (!ok) break;
#pragma unroll
            for (int i = 0; i < M; i++) g[i] = -g[i];
            chol_solve_band<double, N>(A, g);
            double xinf = 0.0, dinf = 0.0;
#pragma unroll
            for (int i = 0; i < M; i++) {
                xinf = fmax(xinf, fabs(X[i]));
                dinf = fmax(dinf, fabs(g[i]));
                X[i] += g[i];
            }
            small = dinf <= kp.o.tol_step * (1.0 + xinf);
        }
        double C = __builtin_huge_val(), rinf = __builtin_huge_val();
        if (ok) ok = eval_cost<double, N, REFR>(sc, p, X, nullptr, C, rinf) && in_guard(kp.s, X, N);
        const bool root = ok && rinf <= kp.o.tau_root;
        kp.out.iters[sid] += steps;
        if (kp.out.stage) kp.out.stage[(size_t)kp.b.n + sid] = steps;
        if (root) {
#pragma unroll
            for (int j = 0; j < M; j++) kp.out.x[(size_t)sid * kRow + j] = X[j];
            kp.out.cost[sid] = C;
            kp.out.status[sid] = ST_CONV;
        } else {
            const int route = kp.out.status[sid];
            if (route == ROUTE_POLISH_FB && kp.o.fallback) {
                const int qq = atomicAdd(&kp.fb_cnt[N - 1], 1);
                kp.fb_list[off + qq] = sid;
                kp.out.status[sid] = ST_RUNNING;
            } else {
                kp.out.status[sid] = (route == ROUTE_POLISH_MAXIT) ? ST_MAXIT : ST_LOCALMIN;
            }
        }
    }
}

// One kernel for every order: measured faster than one launch per order
// (back to back or concurrent), although order 5 sets its registers.
template <bool REFR>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) k_polish(KParams kp)
{
    polish_bin<5, REFR>(kp);
    polish_bin<4, REFR>(kp);
    polish_bin<3, REFR>(kp);
    polish_bin<2, REFR>(kp);
    polish_bin<1, REFR>(kp);
}

// ------------------------------------------------------------------ acceptance
// The acceptance test of Alg. 1 in FP64: converged, |R|_inf <= tau_res, every
// segment at least min_seg, every point inside its finite extent.
// Smallest |cos| between a reflection's incoming direction and the surface
// normal that acceptance allows.
constexpr double kGraze = 1e-9;

template <int N, bool REFR>
__device__ bool accept_path(const SceneDev &s, const double *rx, const int *id, const int *ty, const double *X,
                            double tau_res, double min_seg)
{
    SceneT<double> sc;
    sc.rec = s.rec64;
#pragma unroll
    for (int i = 0; i < 3; i++) { sc.tx[i] = s.tx[i]; sc.glo[i] = s.glo[i]; sc.ghi[i] = s.ghi[i]; }
    PathIn<double, N> p;
#pragma unroll
    for (int i = 0; i < 3; i++) p.rx[i] = rx[i];
#pragma unroll
    for (int k = 0; k < N; k++) { p.id[k] = id[k]; p.ty[k] = ty[k]; }
    double C, rinf;
    bool ok = eval_cost<double, N, REFR>(sc, p, X, nullptr, C, rinf) && (rinf <= tau_res);
#pragma unroll
    for (int k = 0; k <= N; k++) {
        const double *P = (k == 0) ? s.tx : X + 3 * (k - 1);
        const double *Q = (k == N) ? rx : X + 3 * k;
        const double d[3] = {Q[0] - P[0], Q[1] - P[1], Q[2] - P[2]};
        ok = ok && (sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) >= min_seg);
    }
    double medium = 0.0;  // index of the medium the ray travels in (0: not yet known)
#pragma unroll
    for (int k = 0; k < N; k++) {
        const double *r = s.rec64 + (size_t)id[k] * kRec;
        const double *x = X + 3 * k;
        const double d[3] = {x[0] - r[0], x[1] - r[1], x[2] - r[2]};
        if (ty[k] == TP) {
            const double e[3] = {x[0] - r[4], x[1] - r[5], x[2] - r[6]};
            const double a = e[0] * r[7] + e[1] * r[8] + e[2] * r[9];
            const double b = e[0] * r[10] + e[1] * r[11] + e[2] * r[12];
            const double la = r[7] * r[7] + r[8] * r[8] + r[9] * r[9];
            const double lb = r[10] * r[10] + r[11] * r[11] + r[12] * r[12];
            ok = ok && a >= 0.0 && a <= la && b >= 0.0 && b <= lb;
        } else if (ty[k] == TL) {
            const double sp = d[0] * r[3] + d[1] * r[4] + d[2] * r[5];
            ok = ok && sp >= r[6] && sp <= r[7];
        } else if (ty[k] == TQ) {
            const double h = d[0] * r[13] + d[1] * r[14] + d[2] * r[15];
            const double w[3] = {d[0] - h * r[13], d[1] - h * r[14], d[2] - h * r[15]};
            ok = ok && (w[0] * w[0] + w[1] * w[1] + w[2] * w[2] <= r[16] * r[16]);
        }
        if (ty[k] == TP || ty[k] == TQ) {
            // a grazing reflection is degenerate: the ray passes along the
            // surface unchanged and the point can slide along it
            const double *P = (k == 0) ? s.tx : X + 3 * (k - 1);
            const double v[3] = {x[0] - P[0], x[1] - P[1], x[2] - P[2]};
            double nr[3];
            if (ty[k] == TP) {
                nr[0] = r[0], nr[1] = r[1], nr[2] = r[2];
            } else {
                const double A[3][3] = {{r[3], r[4], r[5]}, {r[4], r[6], r[7]}, {r[5], r[7], r[8]}};
                for (int i = 0; i < 3; i++) nr[i] = 2.0 * (A[i][0] * d[0] + A[i][1] * d[1] + A[i][2] * d[2]) + r[9 + i];
            }
            const double vn = v[0] * nr[0] + v[1] * nr[1] + v[2] * nr[2];
            const double lv = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
            const double ln = sqrt(nr[0] * nr[0] + nr[1] * nr[1] + nr[2] * nr[2]);
            ok = ok && (fabs(vn) >= kGraze * lv * ln);
            if (ty[k] == TP && r[16] > 0.0) {
                // a refracting facet passes the ray to its other side, and the
                // ray arrives in the medium the previous refracting facet of
                // the path sent it into
                const double *Q = (k == N - 1) ? rx : X + 3 * (k + 1);
                const double e[3] = {Q[0] - x[0], Q[1] - x[1], Q[2] - x[2]};
                const double en = e[0] * nr[0] + e[1] * nr[1] + e[2] * nr[2];
                ok = ok && (vn * en > 0.0);
                const double in = (vn < 0.0) ? r[16] : r[17], out = (vn < 0.0) ? r[17] : r[16];
                ok = ok && !(medium > 0.0 && in != medium);
                medium = out;
            }
        }
    }
    return ok;
}

// Pass 1: clear the flags and list the converged solves, the only ones the
// test can accept (a few percent of a batch), so that the FP64 test runs on
// full waves instead of one or two lanes of each.  A block covers
// 256 x kAccItems x kAccChunks solves and takes its part of the list with one
// device-wide atomic (one per wave contended on the counter and cost more
// than the test itself); each chunk's loads are issued together.
constexpr int kAccItems = 16;
constexpr int kAccChunks = 4;
__global__ void __launch_bounds__(256) k_accept_list(BatchDev b, const uint8_t *__restrict__ status,
                                                      uint8_t *__restrict__ acc, int *__restrict__ list,
                                                      int *__restrict__ cnt)
{
    __shared__ int bcount, bbase;
    if (threadIdx.x == 0) bcount = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * 256 * kAccItems * kAccChunks;
    const int lane = __lane_id();
    int r[kAccChunks][kAccItems];
    for (int c = 0; c < kAccChunks; c++) {
        int ord[kAccItems], st[kAccItems];
#pragma unroll
        for (int j = 0; j < kAccItems; j++) {
            const int64_t i = base + (int64_t)(c * kAccItems + j) * 256 + threadIdx.x;
            ord[j] = 0;
            st[j] = 0;
            if (i < b.n) {
                ord[j] = b.order[i];
                st[j] = status[i];
            }
        }
#pragma unroll
        for (int j = 0; j < kAccItems; j++) {
            const int64_t i = base + (int64_t)(c * kAccItems + j) * 256 + threadIdx.x;
            if (i < b.n) acc[i] = 0;
            const bool v = ord[j] >= 1 && ord[j] <= kMaxN && (st[j] & 0x7f) == ST_CONV;
            const uint64_t m = __ballot(v);
            int wb = 0;
            if (lane == 0 && m) wb = atomicAdd(&bcount, (int)__popcll(m));
            wb = __shfl(wb, 0);
            r[c][j] = v ? wb + (int)__popcll(m & ((1ull << lane) - 1ull)) : -1;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) bbase = bcount ? atomicAdd(cnt, bcount) : 0;
    __syncthreads();
    for (int c = 0; c < kAccChunks; c++)
#pragma unroll
        for (int j = 0; j < kAccItems; j++)
            if (r[c][j] >= 0) list[bbase + r[c][j]] = (int)(base + (int64_t)(c * kAccItems + j) * 256 + threadIdx.x);
}

// The test on solve i of order ord.
template <bool REFR>
__device__ __forceinline__ bool accept_solve(const SceneDev &s, const BatchDev &b, const OutDevC &in, int64_t i,
                                             int ord, double tau_res, double min_seg)
{
    const int ri = b.rx_index[i];
    double rx[3], X[3 * kMaxN];
    int id[kMaxN], ty[kMaxN];
    for (int j = 0; j < 3; j++) rx[j] = b.rx[3 * (size_t)ri + j];
    for (int j = 0; j < 3 * kMaxN; j++) X[j] = (j < 3 * ord) ? in.x[(size_t)i * kRow + j] : 0.0;
    bool okid = true;
    for (int k = 0; k < kMaxN; k++) {
        id[k] = (k < ord) ? b.prim[(size_t)k * b.n + i] : 0;
        okid = okid && id[k] >= 0 && id[k] < s.n_all;
        ty[k] = prim_type(id[k], s.n_pl, s.n_pl_ln, s.n_pl_ln_q);
    }
    if (!okid) return false;
    switch (ord) {
    case 1: return accept_path<1, REFR>(s, rx, id, ty, X, tau_res, min_seg);
    case 2: return accept_path<2, REFR>(s, rx, id, ty, X, tau_res, min_seg);
    case 3: return accept_path<3, REFR>(s, rx, id, ty, X, tau_res, min_seg);
    case 4: return accept_path<4, REFR>(s, rx, id, ty, X, tau_res, min_seg);
    default: return accept_path<5, REFR>(s, rx, id, ty, X, tau_res, min_seg);
    }
}

// Pass 2: the test on the listed solves (grid-stride over the list).
template <bool REFR>
__global__ void __launch_bounds__(256) k_accept_eval(SceneDev s, BatchDev b, OutDevC in, double tau_res,
                                                      double min_seg, uint8_t *__restrict__ acc,
                                                      const int *__restrict__ list, const int *__restrict__ cnt)
{
    const int m = *cnt;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < m; t += gridDim.x * blockDim.x) {
        const int64_t i = list[t];
        acc[i] = accept_solve<REFR>(s, b, in, i, b.order[i], tau_res, min_seg) ? 1 : 0;
    }
}

// Accepted solves among a block's 256.
__device__ __forceinline__ int block_count(bool a)
{
    __shared__ int wcnt[4];
    const uint64_t m = __ballot(a);
    if (__lane_id() == 0) wcnt[threadIdx.x >> 6] = (int)__popcll(m);
    __syncthreads();
    return wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
}

// A batch of at most kSmallAccept solves: the test with a thread per solve and
// the blocks' counts in one launch, then k_accept_place.  The six launches below
// are bound by the list's serial passes while a block holds few solves: they took
// 52 us and the gaps between them on 16,384 solves, these two 13 us; on 262,144
// 56 us against 27.  On 1,048,576 it is 95 us against 112: there the few
// converged lanes of a wave cost more than the list of them.
constexpr int64_t kSmallAccept = 1 << 18;

template <bool REFR>
__global__ void __launch_bounds__(256) k_accept_small(SceneDev s, BatchDev b, OutDevC in, double tau_res,
                                                       double min_seg, uint8_t *__restrict__ acc,
                                                       int *__restrict__ block_cnt)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    bool a = false;
    if (i < b.n) {
        const int ord = b.order[i];
        if (ord >= 1 && ord <= kMaxN && (in.status[i] & 0x7f) == ST_CONV)
            a = accept_solve<REFR>(s, b, in, i, ord, tau_res, min_seg);
        acc[i] = a ? 1 : 0;
    }
    const int c = block_count(a);
    if (threadIdx.x == 0) block_cnt[blockIdx.x] = c;
}

// The accepted ids in order: each block adds up the counts before it.
__global__ void __launch_bounds__(256) k_accept_place(const uint8_t *__restrict__ acc, int64_t n,
                                                       const int *__restrict__ block_cnt, int *__restrict__ idx,
                                                       int *__restrict__ count)
{
    __shared__ int before[4], wcnt[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int c = 0;
    for (int q = threadIdx.x; q < (int)blockIdx.x; q += 256) c += block_cnt[q];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool a = i < n && acc[i];
    const uint64_t m = __ballot(a);
    if (lane == 0) before[w] = c, wcnt[w] = (int)__popcll(m);
    __syncthreads();
    int base = before[0] + before[1] + before[2] + before[3];
    for (int j = 0; j < w; j++) base += wcnt[j];
    if (a) idx[base + (int)__popcll(m & ((1ull << lane) - 1ull))] = (int)i;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 255) *count = base + (int)__popcll(m);
}

// Pass 3: accepted solves per block of 256 (for the ordered compaction).
__global__ void __launch_bounds__(256) k_accept_count(const uint8_t *__restrict__ acc, int64_t n,
                                                       int *__restrict__ block_cnt)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int c = block_count((i < n) && acc[i]);
    if (threadIdx.x == 0) block_cnt[blockIdx.x] = c;
}

// Exclusive scan of the per-block counts by one block; total -> *count.
__global__ void __launch_bounds__(1024) k_scan_blocks(int *__restrict__ block_cnt, int nblk, int *__restrict__ count)
{
    // wave w owns a contiguous segment and reads it 64 entries at a time
    // (coalesced, eight loads in flight per lane); the 16 segment totals
    // give each wave its starting offset
    constexpr int kU = 8;
    __shared__ int wtot[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int seg = ((nblk + 15) / 16 + 64 * kU - 1) / (64 * kU) * (64 * kU);
    const int lo = min(w * seg, nblk), hi = min(lo + seg, nblk);
    int s = 0;
    for (int i0 = lo; i0 < hi; i0 += 64 * kU) {
        int v[kU];
#pragma unroll
        for (int u = 0; u < kU; u++) {
            const int i = i0 + 64 * u + lane;
            v[u] = (i < hi) ? block_cnt[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kU; u++) s += v[u];
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    if (lane == 0) wtot[w] = s;
    __syncthreads();
    int run = 0;
    for (int j = 0; j < w; j++) run += wtot[j];
    for (int i0 = lo; i0 < hi; i0 += 64 * kU) {
        int v[kU];
#pragma unroll
        for (int u = 0; u < kU; u++) {
            const int i = i0 + 64 * u + lane;
            v[u] = (i < hi) ? block_cnt[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kU; u++) {
            int incl = v[u];
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int x = __shfl_up(incl, d);
                if (lane >= d) incl += x;
            }
            const int i = i0 + 64 * u + lane;
            if (i < hi) block_cnt[i] = run + incl - v[u];
            run += __shfl(incl, 63);
        }
    }
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int j = 0; j < 16; j++) tot += wtot[j];
        *count = tot;
    }
}

__global__ void __launch_bounds__(256) k_accept_scatter(const uint8_t *__restrict__ acc, int64_t n,
                                                         const int *__restrict__ block_off, int *__restrict__ idx)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool a = (i < n) && acc[i];
    __shared__ int wcnt[4];
    const uint64_t m = __ballot(a);
    const int w = threadIdx.x >> 6;
    if (__lane_id() == 0) wcnt[w] = (int)__popcll(m);
    __syncthreads();
    int base = block_off[blockIdx.x];
    for (int j = 0; j < w; j++) base += wcnt[j];
    if (a) idx[base + (int)__popcll(m & ((1ull << __lane_id()) - 1ull))] = (int)i;
}

// ------------------------------------------------------------------ host launchers
void launch_pack(const double *raw, const double *refr, const SceneDev &s, int n_pl, int n_ln, int n_q, int n_c,
                 hipStream_t st)
{
    const int n = n_pl + n_ln + n_q + n_c;
    if (n == 0) return;
    hipLaunchKernelGGL(k_pack, dim3((n + 127) / 128), dim3(128), 0, st, raw, refr, n_pl, n_ln, n_q, n_c, s.tx[0],
                       s.tx[1], s.tx[2], (double *)s.rec64, (float *)s.rec32, (float *)s.occ);
}

void launch_zero(int *p, int n, hipStream_t st)
{
    hipLaunchKernelGGL(k_zero_i32, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
}

// ctr: the workspace's n_ctr counters, cleared here; the first five receive
// the solves per order, those from 32 on are [3][kNumKeys] (counts, offsets,
// cursors).
void launch_bin(const BatchDev &b, const OutDev &out, const SceneDev &s, int *ctr, int n_ctr, int *perm, bool by_solve,
                int *rows, int *curved, hipStream_t st)
{
    if (b.n > 0 && b.n <= kSmallBin && !rows) {
        hipLaunchKernelGGL(k_bin_small, dim3(1), dim3(1024), 0, st, b, out, s.n_all, s.n_pl, s.n_pl_ln, s.n_pl_ln_q,
                           ctr, n_ctr, perm, by_solve ? 1 : 0);
        return;
    }
    launch_zero(ctr, n_ctr, st);
    if (b.n == 0) return;
    const unsigned g = (unsigned)((b.n + kBinPerBlock - 1) / kBinPerBlock);
    int *kcnt = ctr + 32, *koff = kcnt + kNumKeys, *kcur = kcnt + 2 * kNumKeys;
    hipLaunchKernelGGL(k_bin_count, dim3(g), dim3(kBinBlock), 0, st, b, out, s.n_all, s.n_pl, s.n_pl_ln, s.n_pl_ln_q,
                       kcnt);
    hipLaunchKernelGGL(k_bin_offsets, dim3(1), dim3(1024), 0, st, kcnt, koff, ctr, rows ? curved : nullptr);
    hipLaunchKernelGGL(k_bin_scatter, dim3(g), dim3(kBinBlock), 0, st, b, s.n_all, s.n_pl, s.n_pl_ln, s.n_pl_ln_q,
                       koff, kcur, perm, by_solve ? 1 : 0, rows, curved);
}

// The solver kernel of (mode, form, scene in LDS) for an order or schedule
// (mpt_lm.hip; see lm_kernel_of there for `order` and `refr`).
template <int MODE, int FORM, bool LDS> const void *lm_kernel_of(int order, bool refr);

const void *lm_kernel(int mode, int order, bool lds, int form, bool refr)
{
    switch (mode) {
    case MODE_PLAIN64:
        if (form) return lds ? lm_kernel_of<MODE_PLAIN64, 1, true>(order, refr) : lm_kernel_of<MODE_PLAIN64, 1, false>(order, refr);
        return lds ? lm_kernel_of<MODE_PLAIN64, 0, true>(order, refr) : lm_kernel_of<MODE_PLAIN64, 0, false>(order, refr);
    case MODE_FP32:
        if (form) return lds ? lm_kernel_of<MODE_FP32, 1, true>(order, refr) : lm_kernel_of<MODE_FP32, 1, false>(order, refr);
        return lds ? lm_kernel_of<MODE_FP32, 0, true>(order, refr) : lm_kernel_of<MODE_FP32, 0, false>(order, refr);
    default:
        if (form) return lds ? lm_kernel_of<MODE_FALLBACK64, 1, true>(order, refr) : lm_kernel_of<MODE_FALLBACK64, 1, false>(order, refr);
        return lds ? lm_kernel_of<MODE_FALLBACK64, 0, true>(order, refr) : lm_kernel_of<MODE_FALLBACK64, 0, false>(order, refr);
    }
}

void launch_lm(int mode, int order, bool lds, int form, bool refr, size_t lds_bytes, const KParams &kp, int grid,
               int block, hipStream_t st)
{
    void *args[] = {(void *)&kp};
    hipLaunchKernel(lm_kernel(mode, order, lds, form, refr), dim3(grid), dim3(block), args, lds ? lds_bytes : 0, st);
}

const void *polish_kernel(bool refr) { return refr ? (const void *)k_polish<true> : (const void *)k_polish<false>; }

void launch_learned_choose(const SceneDev &s, const BatchDev &b, const int *rows, const int *count, bool all,
                           double *x0l, double gain, bool refr, hipStream_t st)
{
    if (b.n == 0) return;
    const unsigned g = (unsigned)std::min<int64_t>((b.n + 255) / 256, 2048);
    if (refr) hipLaunchKernelGGL(k_learned_choose<true>, dim3(g), dim3(256), 0, st, s, b, rows, count, all ? 1 : 0, x0l, gain);
    else hipLaunchKernelGGL(k_learned_choose<false>, dim3(g), dim3(256), 0, st, s, b, rows, count, all ? 1 : 0, x0l, gain);
}

void launch_polish(const KParams &kp, bool refr, int grid, int block, hipStream_t st)
{
    if (refr) hipLaunchKernelGGL(k_polish<true>, dim3(grid), dim3(block), 0, st, kp);
    else hipLaunchKernelGGL(k_polish<false>, dim3(grid), dim3(block), 0, st, kp);
}

// ------------------------------------------------------------------ physical validation
// block_cnt: nblk + 1 ints (the last one counts the listed solves); the
// converged solves are listed in idx, which the compaction then overwrites
void launch_accept(const SceneDev &s, const BatchDev &b, const OutDevC &in, double tau_res, double min_seg,
                   uint8_t *acc, int *idx, int *count, int *block_cnt, bool refr, hipStream_t st)
{
    const int nblk = (int)((b.n + 255) / 256);
    if (nblk == 0) {
        hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, st, count, 1);
        return;
    }
    if (b.n <= kSmallAccept) {
        if (refr) hipLaunchKernelGGL(k_accept_small<true>, dim3(nblk), dim3(256), 0, st, s, b, in, tau_res, min_seg, acc, block_cnt);
        else hipLaunchKernelGGL(k_accept_small<false>, dim3(nblk), dim3(256), 0, st, s, b, in, tau_res, min_seg, acc, block_cnt);
        hipLaunchKernelGGL(k_accept_place, dim3(nblk), dim3(256), 0, st, acc, b.n, block_cnt, idx, count);
        return;
    }
    int *lcnt = block_cnt + nblk;
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, st, lcnt, 1);
    const int64_t per_list_block = 256 * kAccItems * kAccChunks;
    hipLaunchKernelGGL(k_accept_list, dim3((unsigned)((b.n + per_list_block - 1) / per_list_block)), dim3(256), 0, st,
                       b, in.status, acc, idx, lcnt);
    const dim3 g(std::min(nblk, 2048));
    if (refr) hipLaunchKernelGGL(k_accept_eval<true>, g, dim3(256), 0, st, s, b, in, tau_res, min_seg, acc, idx, lcnt);
    else hipLaunchKernelGGL(k_accept_eval<false>, g, dim3(256), 0, st, s, b, in, tau_res, min_seg, acc, idx, lcnt);
    hipLaunchKernelGGL(k_accept_count, dim3(nblk), dim3(256), 0, st, acc, b.n, block_cnt);
    hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(1024), 0, st, block_cnt, nblk, count);
    hipLaunchKernelGGL(k_accept_scatter, dim3(nblk), dim3(256), 0, st, acc, b.n, block_cnt, idx);
}

}  // namespace mpt
