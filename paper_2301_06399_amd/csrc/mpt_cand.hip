// Candidate generation of Alg. 1 on the GPU: the visibility matrix of the
// objects, the BS row and the UE columns of the adjacency matrix (Sec. II-C,
// Figs. 3-4), and the enumeration of every simple path BS -> objects -> UE
// of at most max_order objects as interaction lists.
//
//  k_samples        sample points of every object (mpt_geom.hpp)
//  k_vis_pairs      one wave per object and group of objects: lanes test sample
//                   pairs (sides / wedges, then the facets and patches whose
//                   boxes meet the shaft between the objects); the BS row
//  k_vis_rx         one wave per receiver and 64 samples
//  k_cand_last      the ends of the paths through each object
//  k_cand_count     one wave per (receiver, first object): path counts per
//                   order
//  k_scan_*         exclusive scan of the counts (receiver, order, first object)
//  k_cand_fill      one block per (receiver, first object): writes the paths in
//                   increasing object ids at the scanned offsets
#include "mpt_internal.hpp"
#include "mpt_geom.hpp"

namespace mpt {

__global__ void __launch_bounds__(64) k_samples(SceneDev s, int k, double *__restrict__ samp, int *__restrict__ cnt,
                                                float *__restrict__ box, uint32_t *__restrict__ z0, int64_t n0,
                                                uint32_t *__restrict__ z1, int64_t n1)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = g; i < n0 + n1; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < n0) z0[i] = 0u;
        else z1[i - n0] = 0u;
    }
    if (g >= s.n_all) return;
    double lo[3], hi[3];
    cnt[g] = obj_samples(s, g, k, samp + (size_t)g * sample_cap(k) * 3, lo, hi);
    for (int c = 0; c < 3; c++) {
        box[(size_t)g * 8 + c] = (float)lo[c];
        box[(size_t)g * 8 + 4 + c] = (float)hi[c];
    }
}

// Plane and quadric records staged in LDS (or read from HBM without).
struct Occluders {
    const double *prec, *qrec;
};

__device__ __forceinline__ Occluders stage_occluders(const SceneDev &s, double *srec, int lds)
{
    const int npl = s.n_pl, nq = s.n_pl_ln_q - s.n_pl_ln;
    if (lds) {
        for (int j = threadIdx.x; j < npl * kRec; j += blockDim.x) srec[j] = s.rec64[j];
        for (int j = threadIdx.x; j < nq * kRec; j += blockDim.x)
            srec[(size_t)npl * kRec + j] = s.rec64[(size_t)s.n_pl_ln * kRec + j];
        __syncthreads();
        return {srec, srec + (size_t)npl * kRec};
    }
    return {s.rec64, s.rec64 + (size_t)s.n_pl_ln * kRec};
}

// Sample points per object by type (a bound: the lanes a type gets).
__device__ __forceinline__ int type_samples(int t, int k) { return t == TL ? k : t == TC ? 2 * k : k * k; }

// The objects of type t: [lo, hi).
__device__ __forceinline__ void type_range(const SceneDev &s, int t, int &lo, int &hi)
{
    lo = t == TP ? 0 : t == TL ? s.n_pl : t == TQ ? s.n_pl_ln : s.n_pl_ln_q;
    hi = t == TP ? s.n_pl : t == TL ? s.n_pl_ln : t == TQ ? s.n_pl_ln_q : s.n_all;
}

// Occluders whose box meets the shaft, kTile at a time: the wave's lanes test
// one box each and list the survivors in LDS; then every lane tests its own
// segment against the listed ones.  The street canyon's shafts keep 20 to 40 of
// 251 facets; the order of the tests does not change a decision.
constexpr int kTile = 512;

struct CullList {
    uint16_t *list;  // [kTile] of this wave
    int tile, n;     // tile the list holds (-1: none) and its length
};

__device__ __forceinline__ void cull_tile(const SceneDev &s, const Shaft &sh, int tile, CullList &c)
{
    const int nocc = s.n_pl + (s.n_pl_ln_q - s.n_pl_ln), lane = threadIdx.x & 63;
    c.tile = tile;
    c.n = 0;
    wave_sync();  // readers of the last list
    const int hi = min(kTile, nocc - tile * kTile);
    for (int q = 0; q < hi; q += 64) {
        const int o = q + lane;
        bool keep = false;
        if (o < hi) {
            const float4 a = *reinterpret_cast<const float4 *>(s.occ + (size_t)(tile * kTile + o) * 8),
                         b = *reinterpret_cast<const float4 *>(s.occ + (size_t)(tile * kTile + o) * 8 + 4);
            const float box[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            keep = !outside_shaft(sh, box);
        }
        const uint64_t m = __ballot(keep);
        if (keep) c.list[c.n + (int)__popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)o;
        c.n += (int)__popcll(m);
    }
    wave_sync();
}

// The lanes (of `alive`) whose segment no occluder blocks.
__device__ __forceinline__ bool unblocked(const SceneDev &s, const Occluders &oc, const Shaft &sh, CullList &c,
                                          bool alive, const Seg &g, int gi, int gj)
{
    const int nocc = s.n_pl + (s.n_pl_ln_q - s.n_pl_ln);
    for (int tile = 0; tile * kTile < nocc; tile++) {
        if (c.tile != tile) cull_tile(s, sh, tile, c);
        for (int q = 0; q < c.n; q++) {
            if (!__any(alive)) return false;
            const int o = tile * kTile + __builtin_amdgcn_readfirstlane((int)c.list[q]);
            if (alive && blocks(s, oc.prec, oc.qrec, o, g, gi, gj)) alive = false;
        }
    }
    return alive;
}

__device__ __forceinline__ float wave_min(float v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = fminf(v, __shfl_xor(v, d));
    return v;
}

// The samples of every object against one point X (BS or a receiver), 64 of
// the flattened samples (type-major, type_samples per object) per call: bit j
// of `row` is set when a sample of object j sees X.  from_x: the segments run
// from X to the sample (BS), else from the sample to X.  With `los`, the sample
// after the last is BS itself, seen or not in *los.
__device__ __forceinline__ void see_point(const SceneDev &s, const Occluders &oc, CullList c, int k, double min_seg,
                                          const double *__restrict__ samp, const int *__restrict__ cnt, int chunk,
                                          const double *X, bool from_x, uint32_t *row, uint8_t *los)
{
    const int lane = threadIdx.x & 63, sc = sample_cap(k);
    int idx = chunk * 64 + lane, j = -1, sj = 0;
#pragma unroll
    for (int t = 0; t < 4; t++) {
        int lo, hi;
        type_range(s, t, lo, hi);
        const int m = type_samples(t, k), len = (hi - lo) * m;
        if (j < 0 && idx >= 0 && idx < len) {
            j = lo + idx / m;
            sj = idx % m;
        }
        idx -= len;
    }
    const bool is_los = los && idx == 0;  // one past the last sample
    double S[3] = {s.tx[0], s.tx[1], s.tx[2]};
    bool alive = is_los;
    if (j >= 0 && sj < cnt[j]) {
        double d[3];
        for (int i = 0; i < 3; i++) {
            S[i] = samp[((size_t)j * sc + sj) * 3 + i];
            d[i] = X[i] - S[i];
        }
        alive = leaves_obj(s, j, S, d);
    }
    const Seg g = (from_x || is_los) ? segment(is_los ? S : X, is_los ? X : S, min_seg) : segment(S, X, min_seg);
    alive = alive && g.ok;
    if (!__any(alive)) {
        if (is_los) *los = 0;
        return;
    }
    float lo[3], hi[3], x[3];
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const float v = (float)S[i];
        lo[i] = wave_min(alive ? v : __builtin_huge_valf());
        hi[i] = -wave_min(alive ? -v : __builtin_huge_valf());
        x[i] = (float)X[i];
    }
    const Shaft sh = shaft_between(lo, hi, x, x);
    c.tile = -1;
    alive = unblocked(s, oc, sh, c, alive, g, is_los ? -1 : from_x ? -1 : j, is_los ? -1 : from_x ? j : -1);
    if (is_los) *los = alive ? 1 : 0;
    // the first seeing sample of each object sets its bit
    const uint64_t m = __ballot(alive && j >= 0);
    const int first = max(0, lane - sj);
    const uint64_t before = ((1ull << lane) - 1ull) & ~((1ull << first) - 1ull);
    if (alive && j >= 0 && (m & before) == 0) atomicOr(row + (j >> 5), 1u << (j & 31));
}

__device__ __forceinline__ int flat_samples(const SceneDev &s, int k)
{
    int n = 0;
#pragma unroll
    for (int t = 0; t < 4; t++) {
        int lo, hi;
        type_range(s, t, lo, hi);
        n += (hi - lo) * type_samples(t, k);
    }
    return n;
}

// The object pairs i < j, then the BS row.  A wave takes object i and as many
// consecutive objects j of one type as their sample pairs fit its lanes (one
// with several rounds where they do not), culls the occluders once for all of
// them, and sets the bits of the pairs some sample pair of which is free.
// Bound: the chain of box and FP64 tests at three waves per SIMD (waves wait in 35%
// of their cycles, the VALU is busy about half of the time).  One wave per pair with
// every facet tested by every lane took 2.34 ms (and the BS row 0.10 ms) on the street canyon (651 objects,
// 4 samples per side); this takes 0.60 ms for both.
__global__ void __launch_bounds__(256) k_vis_pairs(SceneDev s, int k, double min_seg, const double *__restrict__ samp,
                                                   const int *__restrict__ cnt, const float *__restrict__ obox,
                                                   uint32_t *__restrict__ V, uint32_t *__restrict__ B, int W, int lds)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ uint16_t lists[4][kTile];
    const Occluders oc = stage_occluders(s, reinterpret_cast<double *>(smem_raw), lds);
    const int n = s.n_all, sc = sample_cap(k), lane = threadIdx.x & 63;
    const bool one_tile = s.n_pl + (s.n_pl_ln_q - s.n_pl_ln) <= kTile;
    CullList cull{lists[threadIdx.x >> 6], -1, 0};
    const int wave = __builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
    const int nwave = (int)((gridDim.x * blockDim.x) >> 6);
    const int64_t pairs = (int64_t)n * n;
    const int nbs = (flat_samples(s, k) + 63) / 64;
    for (int64_t p = wave; p < pairs + nbs; p += nwave) {
        if (p >= pairs) {
            see_point(s, oc, cull, k, min_seg, samp, cnt, (int)(p - pairs), s.tx, true, B, nullptr);
            continue;
        }
        const int i = (int)(p / n);
        int slot = (int)(p - (int64_t)i * n);
        const int ti = prim_type(i, s.n_pl, s.n_pl_ln, s.n_pl_ln_q), mi = type_samples(ti, k);
        // slots of one object i: the groups of each type in turn
        int j0 = -1, j1 = 0, mj = 1, grp = 1;
#pragma unroll
        for (int t = 0; t < 4; t++) {
            int lo, hi;
            type_range(s, t, lo, hi);
            const int m = type_samples(t, k), gs = max(1, 64 / (mi * m)), ng = (hi - lo + gs - 1) / gs;
            if (j0 < 0 && slot >= 0 && slot < ng) {
                j0 = lo + slot * gs;
                j1 = min(j0 + gs, hi);
                mj = m;
                grp = gs;
            }
            slot -= ng;
        }
        if (j0 < 0 || j1 - 1 <= i) continue;
        const int tot = mi * mj, ci = cnt[i];
        const float itot = 1.0f / (float)tot, imj = 1.0f / (float)mj;
        Shaft sh;
        bool have = false;
        uint64_t seen = 0;  // lanes with a free sample pair
        cull.tile = -1;
        for (int t0 = 0; t0 < max(tot, 64); t0 += 64) {
            const int idx = t0 + lane;
            const int jj = grp > 1 ? (int)(((float)idx + 0.5f) * itot) : 0, rem = idx - jj * tot;
            const int si = (int)(((float)rem + 0.5f) * imj), sj = rem - si * mj;
            const int j = j0 + jj;
            bool alive = rem < tot && j < j1 && j > i && si < ci && sj < cnt[j < j1 ? j : i];
            Seg g;
            g.ok = false;
            if (alive) {
                const double *P = samp + ((size_t)i * sc + si) * 3, *Q = samp + ((size_t)j * sc + sj) * 3;
                g = segment(P, Q, min_seg);
                const double e[3] = {P[0] - Q[0], P[1] - Q[1], P[2] - Q[2]};
                alive = g.ok && leaves_obj(s, i, P, g.d) && leaves_obj(s, j, Q, e);
            }
            if (!__any(alive)) continue;
            if (!have) {
                float lo[3], hi[3];
                const float *bi = obox + (size_t)i * 8;
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    lo[c] = __builtin_huge_valf();
                    hi[c] = -__builtin_huge_valf();
                }
                for (int q = max(j0, i + 1); q < j1; q++)
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        lo[c] = fminf(lo[c], obox[(size_t)q * 8 + c]);
                        hi[c] = fmaxf(hi[c], obox[(size_t)q * 8 + 4 + c]);
                    }
                sh = shaft_between(bi, bi + 4, lo, hi);
                have = true;
            }
            if (!one_tile) cull.tile = -1;
            seen |= __ballot(unblocked(s, oc, sh, cull, alive, g, i, j));
            if (grp == 1 && seen) break;
        }
        // lane q: group member q
        const uint64_t mask = tot >= 64 ? ~0ull : ((1ull << tot) - 1ull) << (lane < grp ? lane * tot : 0);
        if (lane < grp && (seen & mask)) {
            const int j = j0 + lane;
            atomicOr(V + (size_t)i * W + (j >> 5), 1u << (j & 31));
            atomicOr(V + (size_t)j * W + (i >> 5), 1u << (i & 31));
        }
    }
}

// The UE columns: a wave takes 64 samples of consecutive objects against one
// receiver.  With a wave per object (four of its lanes busy for an edge's four
// samples) and no culling 64 receivers of the street canyon took 0.50 ms, now
// 0.14 ms.
__global__ void __launch_bounds__(256) k_vis_rx(SceneDev s, int k, double min_seg, const double *__restrict__ samp,
                                                const int *__restrict__ cnt, const double *__restrict__ rx, int n_rx,
                                                uint32_t *__restrict__ U, uint8_t *__restrict__ los, int W, int lds)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ uint16_t lists[4][kTile];
    const Occluders oc = stage_occluders(s, reinterpret_cast<double *>(smem_raw), lds);
    const CullList cull{lists[threadIdx.x >> 6], -1, 0};
    const int wave = __builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
    const int nwave = (int)((gridDim.x * blockDim.x) >> 6);
    const int per = (flat_samples(s, k) + 1 + 63) / 64;
    for (int64_t it = wave; it < (int64_t)n_rx * per; it += nwave) {
        const int r = (int)(it / per);
        const double X[3] = {rx[3 * (size_t)r], rx[3 * (size_t)r + 1], rx[3 * (size_t)r + 2]};
        see_point(s, oc, cull, k, min_seg, samp, cnt, (int)(it - (int64_t)r * per), X, false, U + (size_t)r * W,
                  los ? los + r : nullptr);
    }
}

// ------------------------------------------------------------------ enumeration
// The graph: BS -> v iff B[v]; u -> v iff V[u][v] (an edge object u has no
// successor but UE when edges may only come last); v -> UE iff U[r][v].
struct CandGraph {
    const uint32_t *V, *B, *U;
    int n, W, n_pl, n_pl_ln, n_pl_ln_q, edge_last, maxo;
};

__device__ __forceinline__ bool is_edge(const CandGraph &G, int g)
{
    return (g >= G.n_pl && g < G.n_pl_ln) || g >= G.n_pl_ln_q;
}

__device__ __forceinline__ bool bit(const uint32_t *row, int v) { return (row[v >> 5] >> (v & 31)) & 1u; }

// The successors of u (none for an edge object when edges come last).
__device__ __forceinline__ const uint32_t *succ(const CandGraph &G, int u)
{
    return (G.edge_last && is_edge(G, u)) ? nullptr : G.V + (size_t)u * G.W;
}

// Last objects of the paths that extend path[0..d-1] by one: the successors of
// its end that see the receiver (last[end] of them), without those already on
// the path.
__device__ __forceinline__ int count_last(const CandGraph &G, const uint32_t *Ur, const int *last, const int *path,
                                          int d)
{
    const int u = path[d - 1];
    int c = last[u];
    if (c == 0) return 0;  // none, or an edge object with no successor
    const uint32_t *row = G.V + (size_t)u * G.W;
    for (int q = 0; q < d; q++) {
        bool twice = false;
        for (int p = 0; p < q; p++) twice = twice || path[p] == path[q];
        if (!twice && bit(row, path[q]) && bit(Ur, path[q])) c--;
    }
    return c;
}

// Depth-first walk, in increasing object ids and without recursion, of the
// simple paths that extend path[0..d0-1] to o objects, the last one seeing
// the receiver (row Ur).  Counts them (the last objects of a path by `last`,
// without walking them), or writes them from position pos on.
template <bool WRITE>
__device__ int64_t walk_tail(const CandGraph &G, const uint32_t *Ur, const int *last, int *path, int d0, int o, int r,
                             int64_t pos, int64_t cap, int32_t *rx_index, int32_t *order, int32_t *prim)
{
    if (!WRITE && d0 == o - 1) return count_last(G, Ur, last, path, d0);
    const uint32_t *row[kMaxN];
    uint32_t m[kMaxN];
    int w[kMaxN];
    int64_t c = 0;
    int d = d0;
    row[d] = succ(G, path[d - 1]);
    if (!row[d]) return WRITE ? pos : 0;
    w[d] = 0;
    m[d] = row[d][0] & (d == o - 1 ? Ur[0] : ~0u);
    while (d >= d0) {
        while (m[d] == 0u && w[d] + 1 < G.W) {
            w[d]++;
            m[d] = row[d][w[d]] & (d == o - 1 ? Ur[w[d]] : ~0u);
        }
        if (m[d] == 0u) {  // this level is exhausted
            d--;
            continue;
        }
        const int v = (w[d] << 5) + (__ffs(m[d]) - 1);
        m[d] &= m[d] - 1u;
        bool seen = false;
        for (int q = 0; q < d; q++) seen = seen || path[q] == v;
        if (seen) continue;
        path[d] = v;
        if (WRITE && d == o - 1) {
            rx_index[pos] = r;
            order[pos] = o;
            for (int q = 0; q < kMaxN; q++) prim[(size_t)q * cap + pos] = q < o ? path[q] : -1;
            pos++;
            continue;
        }
        if (!WRITE && d == o - 2) {
            c += count_last(G, Ur, last, path, d + 1);
            continue;
        }
        const uint32_t *nr = succ(G, v);
        if (!nr) continue;
        d++;
        row[d] = nr;
        w[d] = 0;
        m[d] = nr[0] & (d == o - 1 ? Ur[0] : ~0u);
    }
    return WRITE ? pos : c;
}

// The objects of a row of bits (null: none) in increasing order into an LDS list
// by the block: the first wave tests 64 objects at a time.
__device__ __forceinline__ int list_bits(const CandGraph &G, const uint32_t *row, uint16_t *list)
{
    __shared__ int nlist;
    __syncthreads();  // readers of the last list
    if (threadIdx.x < 64) {
        int c = 0;
        for (int v0 = 0; row && v0 < G.n; v0 += 64) {
            const int v = v0 + (int)threadIdx.x;
            const bool in = v < G.n && bit(row, v);
            const uint64_t m = __ballot(in);
            if (in) list[c + (int)__popcll(m & ((1ull << threadIdx.x) - 1ull))] = (uint16_t)v;
            c += (int)__popcll(m);
        }
        if (threadIdx.x == 0) nlist = c;
    }
    __syncthreads();
    return nlist;
}

// Inclusive scan over the block (Hillis-Steele in LDS).
__device__ __forceinline__ int64_t block_scan_i64(int64_t v, int64_t *red)
{
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = 1; s < (int)blockDim.x; s <<= 1) {
        const int64_t a = (int)threadIdx.x >= s ? red[threadIdx.x - s] : 0;
        __syncthreads();
        red[threadIdx.x] += a;
        __syncthreads();
    }
    const int64_t t = red[threadIdx.x];
    __syncthreads();
    return t;
}

constexpr int kCandBlock = 256;

// last[r][v]: the successors of v that see receiver r.
__global__ void __launch_bounds__(256) k_cand_last(CandGraph G, int n_rx, int *__restrict__ last)
{
    const int64_t items = (int64_t)n_rx * G.n;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < items; it += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(it / G.n), v = (int)(it % G.n);
        const uint32_t *Ur = G.U + (size_t)r * G.W, *row = succ(G, v);
        int c = 0;
        for (int w = 0; row && w < G.W; w++) c += __popc(row[w] & Ur[w]);
        last[it] = c;
    }
}

// One wave per (receiver, first object); the lanes take its successors.  One
// block each, with the successors listed by one thread and the last objects
// walked one by one, took 0.41 ms for 16 receivers of the street canyon (651
// objects, orders 1-3), now 0.02 ms.
__global__ void __launch_bounds__(256) k_cand_count(CandGraph G, int n_rx, const int *__restrict__ last,
                                                    int64_t *__restrict__ cnt)
{
    const int64_t items = (int64_t)n_rx * G.n;
    const int lane = threadIdx.x & 63;
    const int64_t wave = __builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t it = wave; it < items; it += nwave) {
        const int r = (int)(it / G.n), v1 = (int)(it % G.n);
        const uint32_t *Ur = G.U + (size_t)r * G.W;
        int64_t *out = cnt + (size_t)r * G.maxo * G.n + v1;
        const int *lr = last + (size_t)r * G.n;
        const bool bs = bit(G.B, v1);
        const uint32_t *row = bs ? succ(G, v1) : nullptr;
        for (int o = 1; o <= G.maxo; o++) {
            int64_t c = 0;
            if (o <= 2) {
                c = bs && lane == 0 ? (o == 1 ? (int64_t)bit(Ur, v1) : (int64_t)lr[v1]) : 0;
            } else if (row) {
                for (int v2 = lane; v2 < G.n; v2 += 64) {
                    if (!bit(row, v2)) continue;
                    int path[kMaxN] = {v1, v2};
                    c += walk_tail<false>(G, Ur, lr, path, 2, o, r, 0, 0, nullptr, nullptr, nullptr);
                }
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d);
            }
            if (lane == 0) out[(size_t)(o - 1) * G.n] = c;
        }
    }
}

// Writes the paths of orders up to 3, or (DEEP) of the orders beyond.  The
// blocks that are resident at once list the first objects that see BS and stride
// over (receiver, first object, part): with a block for every object the device
// was mostly busy starting blocks that had nothing to write.  For order 3 a
// first object's successors are split into up to kFillParts consecutive parts
// while that leaves each block about half a part (a part repeats the counts
// before it and its block's scans: 16 receivers' 4.4 M paths took 161 us in 2
// parts, 191 in 4, 279 in 8 and 452 in 16; one thread per path that searched
// its successor and object, in the registers of the deep walk, 528).  Bound by
// the latency of those steps; the stores alone would take 26 us.
constexpr int kFillParts = 8;

template <bool DEEP>
__global__ void __launch_bounds__(kCandBlock) k_cand_fill(CandGraph G, int n_rx, const int *__restrict__ last,
                                                          const int64_t *__restrict__ off, int64_t cap,
                                                          int32_t *__restrict__ rx_index, int32_t *__restrict__ order,
                                                          int32_t *__restrict__ prim)
{
    extern __shared__ uint16_t ids[];  // the first objects, one's successors and, per wave, the ends of one's paths
    uint16_t *first = ids, *list = ids + G.n;
    __shared__ int64_t red[kCandBlock];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint16_t *ends = ids + (size_t)(2 + wave) * G.n;
    const int nf = list_bits(G, G.B, first);
    if (nf == 0) return;
    const int64_t pairs = (int64_t)n_rx * nf;
    const int parts = DEEP || G.maxo < 3 ? 1 : (int)max((int64_t)1, min((int64_t)kFillParts, gridDim.x / (2 * pairs)));
    const int64_t items = pairs * parts;
    for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
        const int part = (int)(it % parts), r = (int)(it / parts / nf), v1 = first[it / parts % nf];
        const uint32_t *Ur = G.U + (size_t)r * G.W;
        const int *lr = last + (size_t)r * G.n;
        const int nl = list_bits(G, succ(G, v1), list);
        for (int o = DEEP ? 4 : 1; o <= (DEEP ? G.maxo : min(G.maxo, 3)); o++) {
            int64_t base = off[((size_t)r * G.maxo + (o - 1)) * G.n + v1];
            if (o == 1) {
                if (part == 0 && threadIdx.x == 0 && bit(Ur, v1)) {
                    rx_index[base] = r;
                    order[base] = 1;
                    for (int q = 0; q < kMaxN; q++) prim[(size_t)q * cap + base] = q < 1 ? v1 : -1;
                }
                continue;
            }
            if (part && o == 2) continue;
            // this block's part of the list, and what the parts before it write
            int e_lo = 0, e_hi = nl;
            if (o == 3) {
                e_lo = (int)((int64_t)nl * part / parts);
                e_hi = (int)((int64_t)nl * (part + 1) / parts);
                int64_t before = 0;
                for (int e = threadIdx.x; e < e_lo; e += blockDim.x) {
                    const int path[2] = {v1, list[e]};
                    before += count_last(G, Ur, lr, path, 2);
                }
                block_scan_i64(before, red);
                base += red[blockDim.x - 1];
                __syncthreads();
            }
            // successors in increasing id, a chunk of blockDim at a time: each
            // thread's subtree count, scanned in list order, gives its offset
            for (int e0 = e_lo; e0 < e_hi; e0 += blockDim.x) {
                const int e = e0 + threadIdx.x;
                int64_t c = 0;
                int v2 = -1;
                if (e < e_hi) {
                    v2 = list[e];
                    int path[kMaxN] = {v1, v2};
                    if constexpr (DEEP) c = walk_tail<false>(G, Ur, lr, path, 2, o, r, 0, 0, nullptr, nullptr, nullptr);
                    else c = o == 2 ? bit(Ur, v2) : count_last(G, Ur, lr, path, 2);
                }
                const int64_t incl = block_scan_i64(c, red);
                const int64_t chunk = red[blockDim.x - 1];
                if (!DEEP && o == 3) {
                    // a wave per successor: each lane lists the objects of one
                    // word of its row, and consecutive lanes write consecutive
                    // paths
                    const int ne = min((int)blockDim.x, e_hi - e0);
                    for (int z = wave; z < ne; z += kCandBlock / 64) {
                        const int64_t at = z ? red[z - 1] : 0;
                        const int m3 = (int)(red[z] - at);
                        if (m3 == 0) continue;
                        const int w2 = list[e0 + z];
                        const uint32_t *row2 = G.V + (size_t)w2 * G.W;
                        int run = 0;
                        for (int w0 = 0; w0 < G.W; w0 += 64) {
                            const int w = w0 + lane;
                            uint32_t m = w < G.W ? row2[w] & Ur[w] : 0u;
                            if ((v1 >> 5) == w) m &= ~(1u << (v1 & 31));
                            if ((w2 >> 5) == w) m &= ~(1u << (w2 & 31));
                            const int pc = __popc(m);
                            int upto = pc;
#pragma unroll
                            for (int d = 1; d < 64; d <<= 1) {
                                const int v = __shfl_up(upto, d);
                                if (lane >= d) upto += v;
                            }
                            for (int q = run + upto - pc; m; m &= m - 1u)
                                ends[q++] = (uint16_t)((w << 5) + (__ffs(m) - 1));
                            run += __shfl(upto, 63);
                        }
                        wave_sync();
                        for (int q = lane; q < m3; q += 64) {
                            const int64_t pos = base + at + q;
                            rx_index[pos] = r;
                            order[pos] = 3;
                            prim[pos] = v1;
                            prim[(size_t)cap + pos] = w2;
                            prim[(size_t)2 * cap + pos] = ends[q];
                            prim[(size_t)3 * cap + pos] = -1;
                            prim[(size_t)4 * cap + pos] = -1;
                        }
                        wave_sync();
                    }
                } else if (c > 0) {
                    int path[kMaxN] = {v1, v2};
                    const int64_t pos = base + incl - c;
                    if constexpr (!DEEP) {
                        rx_index[pos] = r;
                        order[pos] = 2;
                        for (int q = 0; q < kMaxN; q++) prim[(size_t)q * cap + pos] = q < 2 ? path[q] : -1;
                    } else {
                        walk_tail<true>(G, Ur, lr, path, 2, o, r, pos, cap, rx_index, order, prim);
                    }
                }
                __syncthreads();  // red is read above; the next chunk rewrites it
                base += chunk;
            }
        }
    }
}

// Exclusive scan of n int64 values in place: blocks of 1024 (4 per thread),
// their totals, then the offsets added back.
constexpr int kScanPer = 4;

__global__ void __launch_bounds__(256) k_scan_local(int64_t *__restrict__ a, int64_t n, int64_t *__restrict__ sums)
{
    __shared__ int64_t red[256];
    const int64_t b0 = (int64_t)blockIdx.x * 256 * kScanPer + (int64_t)threadIdx.x * kScanPer;
    int64_t v[kScanPer], t = 0;
    for (int q = 0; q < kScanPer; q++) {
        v[q] = (b0 + q < n) ? a[b0 + q] : 0;
        t += v[q];
    }
    const int64_t incl = block_scan_i64(t, red);
    int64_t run = incl - t;
    for (int q = 0; q < kScanPer; q++) {
        if (b0 + q < n) a[b0 + q] = run;
        run += v[q];
    }
    if (threadIdx.x == blockDim.x - 1) sums[blockIdx.x] = incl;
}

// One block: exclusive scan of the block totals (any count), and the grand
// total into sums[nb].
__global__ void __launch_bounds__(256) k_scan_sums(int64_t *__restrict__ sums, int64_t nb)
{
    __shared__ int64_t red[256];
    int64_t carry = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += blockDim.x) {
        const int64_t i = c0 + threadIdx.x;
        const int64_t v = i < nb ? sums[i] : 0;
        const int64_t incl = block_scan_i64(v, red);
        const int64_t chunk = red[blockDim.x - 1];
        __syncthreads();
        if (i < nb) sums[i] = carry + incl - v;
        carry += chunk;
    }
    if (threadIdx.x == 0) sums[nb] = carry;
}

__global__ void __launch_bounds__(256) k_scan_add(int64_t *__restrict__ a, int64_t n, const int64_t *__restrict__ sums)
{
    const int64_t b0 = (int64_t)blockIdx.x * 256 * kScanPer + (int64_t)threadIdx.x * kScanPer;
    const int64_t add = sums[blockIdx.x];
    for (int q = 0; q < kScanPer; q++)
        if (b0 + q < n) a[b0 + q] += add;
}

// ------------------------------------------------------------------ launchers
static size_t occluder_bytes(const SceneDev &s)
{
    return (size_t)(s.n_pl + (s.n_pl_ln_q - s.n_pl_ln)) * kRec * sizeof(double);
}

static int lds_choice(const void *kern, const SceneDev &s, size_t lds_max, size_t &bytes)
{
    bytes = occluder_bytes(s);
    const int lds = bytes <= lds_max && bytes <= 64 * 1024;
    if (lds) hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    else bytes = 0;
    return lds;
}

void launch_samples(const SceneDev &s, int k, double *samp, int *cnt, float *box, uint32_t *z0, int64_t n0,
                    uint32_t *z1, int64_t n1, hipStream_t st)
{
    const int64_t n = std::max<int64_t>(s.n_all, std::min<int64_t>((n0 + n1 + 3) / 4, 64 * 1024));
    if (n == 0) return;
    hipLaunchKernelGGL(k_samples, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, st, s, k, samp, cnt, box, z0, n0, z1,
                       n1);
}

// Blocks of a kernel that stages the occluders: as many as the records let
// reside at once (each stages them once and then walks its items).
static unsigned resident_blocks(int64_t waves, size_t lds_bytes, size_t lds_max, int cu)
{
    const size_t per = lds_bytes + 4 * kTile * sizeof(uint16_t);
    const int64_t fit = std::max<int64_t>(1, std::min<int64_t>(8, (int64_t)(lds_max / per)));
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((waves + 3) / 4, (int64_t)cu * fit));
}

void launch_visibility(const SceneDev &s, int k, double min_seg, const double *samp, const int *cnt, const float *box,
                       uint32_t *V, uint32_t *B, int W, size_t lds_max, int cu, hipStream_t st)
{
    if (s.n_all == 0) return;
    size_t bytes;
    const int lds = lds_choice((const void *)k_vis_pairs, s, lds_max, bytes);
    hipLaunchKernelGGL(k_vis_pairs, dim3(resident_blocks((int64_t)s.n_all * s.n_all, bytes, lds_max, cu)), dim3(256),
                       bytes, st, s, k, min_seg, samp, cnt, box, V, B, W, lds);
}

void launch_visibility_rx(const SceneDev &s, int k, double min_seg, const double *samp, const int *cnt,
                          const double *rx, int n_rx, uint32_t *U, uint8_t *los, int W, size_t lds_max, int cu,
                          hipStream_t st)
{
    if (n_rx == 0) return;
    size_t bytes;
    const int lds = lds_choice((const void *)k_vis_rx, s, lds_max, bytes);
    const int64_t waves = (int64_t)n_rx * ((int64_t)s.n_all * std::max(k * k, 2 * k) / 64 + 1);
    hipLaunchKernelGGL(k_vis_rx, dim3(resident_blocks(waves, bytes, lds_max, cu)), dim3(256), bytes, st, s, k, min_seg,
                       samp, cnt, rx, n_rx, U, los, W, lds);
}

static CandGraph graph_of(const SceneDev &s, const uint32_t *V, const uint32_t *B, const uint32_t *U, int W,
                          int maxo, int edge_last)
{
    CandGraph G;
    G.V = V;
    G.B = B;
    G.U = U;
    G.n = s.n_all;
    G.W = W;
    G.n_pl = s.n_pl;
    G.n_pl_ln = s.n_pl_ln;
    G.n_pl_ln_q = s.n_pl_ln_q;
    G.edge_last = edge_last;
    G.maxo = maxo;
    return G;
}

void launch_cand_count(const SceneDev &s, const uint32_t *V, const uint32_t *B, const uint32_t *U, int W, int n_rx,
                       int maxo, int edge_last, int64_t *cnt, int64_t *sums, int *last, int cu, hipStream_t st)
{
    const CandGraph G = graph_of(s, V, B, U, W, maxo, edge_last);
    const int64_t items = (int64_t)n_rx * s.n_all;
    hipLaunchKernelGGL(k_cand_last, dim3((unsigned)std::min<int64_t>((items + 255) / 256, (int64_t)cu * 8)), dim3(256),
                       0, st, G, n_rx, last);
    hipLaunchKernelGGL(k_cand_count, dim3((unsigned)std::min<int64_t>((items + 3) / 4, (int64_t)cu * 8)), dim3(256), 0,
                       st, G, n_rx, last, cnt);
    // exclusive scan over (receiver, order, first object)
    const int64_t n = items * maxo;
    const int64_t nb = (n + 256 * kScanPer - 1) / (256 * kScanPer);
    hipLaunchKernelGGL(k_scan_local, dim3((unsigned)nb), dim3(256), 0, st, cnt, n, sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(256), 0, st, sums, nb);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(256), 0, st, cnt, n, sums);
}

void launch_cand_fill(const SceneDev &s, const uint32_t *V, const uint32_t *B, const uint32_t *U, int W, int n_rx,
                      int maxo, int edge_last, const int64_t *off, const int *last, int64_t cap, int32_t *rx_index,
                      int32_t *order, int32_t *prim, int cu, hipStream_t st)
{
    const CandGraph G = graph_of(s, V, B, U, W, maxo, edge_last);
    const int64_t items = (int64_t)n_rx * s.n_all;
    if (items == 0) return;
    const size_t bytes = (size_t)(2 + kCandBlock / 64) * s.n_all * sizeof(uint16_t);
    hipLaunchKernelGGL(k_cand_fill<false>, dim3((unsigned)std::min<int64_t>(items * kFillParts, (int64_t)cu * 8)),
                       dim3(kCandBlock), bytes, st, G, n_rx, last, off, cap, rx_index, order, prim);
    if (maxo > 3)
        hipLaunchKernelGGL(k_cand_fill<true>, dim3((unsigned)std::min<int64_t>(items, (int64_t)cu * 3)),
                           dim3(kCandBlock), bytes, st, G, n_rx, last, off, cap, rx_index, order, prim);
}

}  // namespace mpt
