// Physical validation of accepted paths on the GPU (mpt_visible): between
// interactions a ray travels in free space (Sec. II), so a kept path's
// segments may not cross another facet or paraboloid patch, and a segment at
// a wedged straight edge must leave it into free space.
//
//  k_vis_list   compacts the accepted solves into a list, clears visible[]
//  k_visible    a group of lanes per accepted solve: every segment against every
//               facet and patch (a lane each) and the edges' wedges
#include "mpt_internal.hpp"
#include "mpt_geom.hpp"

namespace mpt {

__global__ void k_vis_zero(int *p) { if (threadIdx.x == 0) p[0] = 0; }

// The accepted solves, compacted (in no particular order) into list[1..],
// their count in list[0]; visible[] cleared for every solve.  A block takes
// its places with one device-wide atomic (one per wave was served one at a
// time: 2.27 ms on 16.8 M solves, 0.28 ms on 4.4 M).
constexpr int kListItems = 16;  // solves per thread at most

__global__ void __launch_bounds__(256) k_vis_list(const uint8_t *__restrict__ acc, int64_t n, int *__restrict__ list,
                                                  uint8_t *__restrict__ vis, int items)
{
    __shared__ uint16_t loc[256 * kListItems];
    __shared__ int total, base;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * 256 * items;
    for (int j = 0; j < items; j++) {
        const int q = j * 256 + (int)threadIdx.x;
        const int64_t i = b0 + q;
        const bool a = i < n && acc[i] != 0;
        if (i < n) vis[i] = 0;
        const uint64_t m = __ballot(a);
        if (!m) continue;
        int w = 0;
        if (__lane_id() == 0) w = atomicAdd(&total, (int)__popcll(m));
        w = __shfl(w, 0);
        if (a) loc[w + (int)__popcll(m & ((1ull << __lane_id()) - 1ull))] = (uint16_t)q;
    }
    __syncthreads();
    if (threadIdx.x == 0) base = total ? atomicAdd(list, total) : 0;
    __syncthreads();
    for (int q = threadIdx.x; q < total; q += 256) list[1 + base + q] = (int)(b0 + loc[q]);
}

// G lanes per accepted solve of the list: visible[i] = 1 when no segment is
// blocked.  A lane tests one facet or patch at a time, its box against the
// segment first, and the path ends at its first blocked segment.  In a city scene
// most kept paths have one, and a thread per path walked every facet for the
// slowest path of its wave: 0.76 ms against 0.40 ms with a wave per path on the
// accepted paths of 16 receivers' candidates in the street canyon (251 facets),
// 0.29 against 0.04 ms on the 32,000 of its 262,144 random lists.  With few
// occluders and many paths a wave per path leaves most lanes idle and the paths'
// loads one after the other, and a path gets four lanes: the call on 655,360 kept
// paths of the room (6 facets) takes 168 us that way, 855 with a wave each (a
// thread each: 389), on 107,304 among 40 patches 147 and 212; but on 415 among 61
// facets 77 and 56.  Plane and quadric records are staged in LDS when `lds` is set.
template <int G>
__global__ void __launch_bounds__(256) k_visible(SceneDev s, BatchDev b, OutDevC in, const int *__restrict__ list,
                                                 double min_seg, uint8_t *__restrict__ vis, int *__restrict__ count,
                                                 int lds, int wide)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ int kept;
    double *srec = reinterpret_cast<double *>(smem_raw);
    const int npl = s.n_pl, nq = s.n_pl_ln_q - s.n_pl_ln, nocc = npl + nq;
    const int na = list[0];
    if (G == 64 ? na > wide : na <= wide) return;  // the other kernel's list
    constexpr int kPaths = 64 / G;                 // of a wave
    if ((int)(blockIdx.x * (blockDim.x >> 6)) * kPaths >= na) return;  // block-uniform
    if (threadIdx.x == 0) kept = 0;
    if (lds) {
        for (int j = threadIdx.x; j < npl * kRec; j += blockDim.x) srec[j] = s.rec64[j];
        for (int j = threadIdx.x; j < nq * kRec; j += blockDim.x)
            srec[(size_t)npl * kRec + j] = s.rec64[(size_t)s.n_pl_ln * kRec + j];
    }
    __syncthreads();
    const double *prec = lds ? srec : s.rec64;
    const double *qrec = lds ? srec + (size_t)npl * kRec : s.rec64 + (size_t)s.n_pl_ln * kRec;
    const int lane = threadIdx.x & (G - 1), nwave = (int)((gridDim.x * blockDim.x) >> 6);
    const int wave = __builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
    // this path's lanes in a ballot (the lanes of one path stay together)
    const uint64_t group = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1ull) << ((threadIdx.x & 63) & ~(G - 1));
    int mine = 0;
    for (int t = G == 64 ? wave : wave * kPaths + (int)((threadIdx.x & 63) / G); t < na; t += nwave * kPaths) {
        const int64_t i = list[1 + t];
        const int n = b.order[i], ri = b.rx_index[i];
        bool ok = true;
        double P[3] = {s.tx[0], s.tx[1], s.tx[2]};
        int ip = -1;
        for (int k = 0; ok && k <= n; k++) {
            double Q[3];
            for (int c = 0; c < 3; c++) Q[c] = (k == n) ? b.rx[3 * (size_t)ri + c] : in.x[(size_t)i * kRow + 3 * k + c];
            const int iq = (k == n) ? -1 : b.prim[(size_t)k * b.n + i];
            const Seg g = segment(P, Q, min_seg);
            ok = g.ok;
            // the segment's ends on straight edges: both leave into free space
            if (ok && s.wedge && ip >= npl && ip < s.n_pl_ln && vis_wedge(s.wedge + 7 * (size_t)(ip - npl), P, Q))
                ok = false;
            if (ok && s.wedge && iq >= npl && iq < s.n_pl_ln && vis_wedge(s.wedge + 7 * (size_t)(iq - npl), Q, P))
                ok = false;
            if (ok) {
                const float p[3] = {(float)P[0], (float)P[1], (float)P[2]}, q[3] = {(float)Q[0], (float)Q[1], (float)Q[2]};
                const Shaft sh = shaft_between(p, p, q, q);
                for (int o0 = 0; ok && o0 < nocc; o0 += G) {
                    const int o = o0 + lane;
                    bool hit = false;
                    if (o < nocc) {
                        const float4 lo = *reinterpret_cast<const float4 *>(s.occ + (size_t)o * 8),
                                     hi = *reinterpret_cast<const float4 *>(s.occ + (size_t)o * 8 + 4);
                        const float box[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                        if (!outside_shaft(sh, box)) hit = blocks(s, prec, qrec, o, g, ip, iq);
                    }
                    ok = (__ballot(hit) & group) == 0;
                }
            }
            for (int c = 0; c < 3; c++) P[c] = Q[c];
            ip = iq;
        }
        if (ok && lane == 0) {
            vis[i] = 1;
            mine++;
        }
    }
    if (mine) atomicAdd(&kept, mine);
    __syncthreads();
    if (threadIdx.x == 0 && kept) atomicAdd(count, kept);
}

template <int G>
static void launch_lanes(const SceneDev &s, const BatchDev &b, const OutDevC &in, const int *list, double min_seg,
                         uint8_t *vis, int *count, size_t lds_max, int cu, int wide, hipStream_t st)
{
    const size_t bytes = (size_t)(s.n_pl + (s.n_pl_ln_q - s.n_pl_ln)) * kRec * sizeof(double);
    const int lds = bytes <= lds_max && bytes <= 64 * 1024;
    if (lds) hipFuncSetAttribute((const void *)k_visible<G>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    // the accepted count is on the device: the blocks that fit at once, each
    // looping over the list
    const int64_t fit = lds ? std::max<int64_t>(1, std::min<int64_t>(8, (int64_t)(lds_max / (bytes + 64)))) : 8;
    const int64_t per = 4 * (64 / G);
    const unsigned g = (unsigned)std::min<int64_t>((b.n + per - 1) / per, (int64_t)cu * fit);
    hipLaunchKernelGGL(k_visible<G>, dim3(g), dim3(256), lds ? bytes : 0, st, s, b, in, list, min_seg, vis, count, lds,
                       wide);
}

void launch_visible(const SceneDev &s, const BatchDev &b, const OutDevC &in, const uint8_t *acc, double min_seg,
                    uint8_t *vis, int *count, int *list, size_t lds_max, int cu, hipStream_t st)
{
    hipLaunchKernelGGL(k_vis_zero, dim3(1), dim3(64), 0, st, count);
    if (b.n == 0) return;
    hipLaunchKernelGGL(k_vis_zero, dim3(1), dim3(64), 0, st, list);
    // one solve per thread while the blocks fit on the device at once
    const int items = (int)std::min<int64_t>(kListItems, (b.n + 256 * (int64_t)cu * 4 - 1) / (256 * (int64_t)cu * 4));
    hipLaunchKernelGGL(k_vis_list, dim3((unsigned)((b.n + 256 * items - 1) / (256 * items))), dim3(256), 0, st, acc,
                       b.n, list, vis, items);
    // Up to `wide` paths a wave each, more four lanes each: those take nocc / 4 tests
    // one after the other, a wave one, but 16 paths go through a wave at once.  The
    // lines were about 2,500 paths at 6 occluders, 16,000 at 41, 25,000 at 61, 36,000
    // at 91, that is nocc / 20 paths to each of 8192 resident waves; above 96
    // occluders every list gets waves (200, 100,000 paths: 267 us against 296).  The
    // list's length is on the device: both kernels are launched where it decides, and
    // one of them ends at once.
    const int nocc = s.n_pl + (s.n_pl_ln_q - s.n_pl_ln);
    const int64_t line = nocc <= 96 ? (int64_t)nocc * cu * 8 * 4 / 20 : INT32_MAX;
    const int wide = (int)std::min<int64_t>(line, INT32_MAX);
    launch_lanes<64>(s, b, in, list, min_seg, vis, count, lds_max, cu, wide, st);
    if (b.n > wide) launch_lanes<4>(s, b, in, list, min_seg, vis, count, lds_max, cu, wide, st);
}

}  // namespace mpt
