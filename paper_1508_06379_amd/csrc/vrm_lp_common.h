// Pieces shared by the LP kernels of libvrm: the stencil outputs, the tie-break of
// the canonical cost, queue appends and counters.
#pragma once
#include <hip/hip_runtime.h>

#include "vrm_device.h"
#include "vrm_internal.h"
#include "vrm_simplex.h"

namespace vrm {

__device__ __forceinline__ int cell_of_pos(const GridState& g, float x, float y, int& cx, int& cy)
{
    float fx = (x - g.x0) * g.inv_cs;
    float fy = (y - g.y0) * g.inv_cs;
    fx = fminf(fmaxf(fx, 0.0f), (float)(g.nx - 1));
    fy = fminf(fmaxf(fy, 0.0f), (float)(g.ny - 1));
    cx = (int)fx;
    cy = (int)fy;
    return cy * g.nx + cx;
}

// wave-aggregated append of `want` (0/1) items; returns the slot or -1
__device__ __forceinline__ int wave_append(int* counter, bool want)
{
    uint64_t m = __ballot(want);
    int lane = lane_id();
    int before = __popcll(m & ((1ull << lane) - 1ull));
    int total = __popcll(m);
    int leader = total ? __ffsll((unsigned long long)m) - 1 : 0;
    int base = 0;
    if (total && lane == leader) base = atomicAdd(counter, total);
    base = __shfl(base, leader, VRM_WAVE);
    return want ? base + before : -1;
}

struct StencilOut {
    int32_t* small_idx;
    float* small_f;
    float* fii;
    uint8_t* status;
    int32_t* full_k;
    int32_t* full_idx;
    float* full_f;
    uint16_t* feat;      // feature rows of solved LPs (collection), or NULL
    float* lab;          // label rows (basis indicators, fractions) of solved LPs, or NULL
    int max_rows;
    const float* pred;   // warm start: small LPs 8 logits, complete ones kMlpOut outputs per queue item; or NULL
    int32_t* prev;       // basis (column ids) of each particle's last stencil, [id][kPrevIds]: recorded if non-NULL
    int prev_cap;        // rows of prev: particles with larger ids keep no basis (they start cold)
    int use_prev;        // warm start from prev instead of pred
    uint64_t* pmask;         // crash basis as a column mask per complete-neighbourhood queue item (size-binned path)
    uint8_t* pivhist;        // by particle id (< prev_cap): pivots of its last cold complete LP
    const int32_t* cloud_id;   // ids by cloud index
    int32_t* sten_idx;   // [i][kStenRow] the stencils of the run are kept here (or NULL), see kStenRow
    uint8_t* seg_mask;   // [i] segments that carry a five-row LP's fractions, kept for the next stage, or NULL
    ptrdiff_t sten_f;    // distance from a column's entry to its fraction
};

// entry e of particle i's kept stencil; the row's end: count of entries (-1: no stencil) and fhat_ii
__device__ __forceinline__ void keep_entry(const StencilOut& out, int i, int e, int pj, float v)
{
    int32_t* p = out.sten_idx + (size_t)i * kStenRow + e;
    p[0] = pj;
    p[out.sten_f] = __float_as_int(v);
}
__device__ __forceinline__ void keep_end(const StencilOut& out, int i, int count, float fii)
{
    keep_entry(out, i, kStenRow - 1, count, fii);
}

constexpr int kPrevIds = 9;

// the previous basis of particle `own` as a mask over columns with ids cid(j), j < k
template <class ColId>
__device__ __forceinline__ uint64_t prev_mask(const int32_t* prev, int own, int k, ColId cid)
{
    int pv[kPrevIds];
#pragma unroll
    for (int r = 0; r < kPrevIds; ++r) pv[r] = prev[(size_t)own * kPrevIds + r];
    uint64_t m = 0;
    for (int j = 0; j < k; ++j) {
        const int id = cid(j);
        if (id < 0) continue;
        bool in = false;
#pragma unroll
        for (int r = 0; r < kPrevIds; ++r) in = in || pv[r] == id;
        if (in) m |= 1ull << j;
    }
    return m;
}

// record the basic columns' ids as the particle's basis
template <class ColId>
__device__ __forceinline__ void record_basis(int32_t* prev, int own, uint64_t basis, ColId cid)
{
    int c = 0;
    while (basis && c < kPrevIds) {
        const int j = __ffsll((unsigned long long)basis) - 1;
        basis &= basis - 1;
        prev[(size_t)own * kPrevIds + c++] = cid(j);
    }
    for (; c < kPrevIds; ++c) prev[(size_t)own * kPrevIds + c] = -1;
}

__device__ __forceinline__ void count_add(int* p, bool v)
{
    uint64_t m = __ballot(v);
    if (m && lane_id() == __ffsll((unsigned long long)m) - 1) atomicAdd(p, __popcll(m));
}
__device__ __forceinline__ void count_add(int64_t* p, bool v)
{
    uint64_t m = __ballot(v);
    if (m && lane_id() == __ffsll((unsigned long long)m) - 1)
        atomicAdd(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__popcll(m));
}

// Tie-break of the canonical cost: 2^-10 rank(id); for the removal LP (q = 1)
// 2^-16 rank^2, convex in the rank because on a lattice the id ranks of
// opposite neighbours are symmetric and would tie under a linear weight.
// Exact in FP32 for ranks < 64.
__device__ __forceinline__ float tie_weight(unsigned rank, int q)
{
    return q == 1 ? 0x1p-16f * (float)(rank * rank) : 0.0009765625f * (float)rank;
}

// add the tie-break to a double-float cost (exact at these magnitudes)
__device__ __forceinline__ df add_rank(df C, int rank, int q)
{
    df w = two_sum(C.hi, tie_weight((unsigned)rank, q));
    w.lo += C.lo;
    return fast_two_sum(w.hi, w.lo);
}

__device__ __forceinline__ uint64_t member_key(float d2, int id)
{
    return ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)id;
}

// Positions of a group's list (sixteen lanes, one DPP row; a lane's members e = sub + 16 q
// with keys mk[q], their counts of smaller keys in pos[q]) where keys are equal: equal
// distance and equal id, which a cloud with distinct ids does not have.  Such members would
// share a position and leave the next one unwritten; the one later in the list goes first.
template <int Q>
__device__ __forceinline__ void separate_equal_keys(const uint64_t* keys, int nm, int sub, const uint64_t (&mk)[Q],
                                                    int (&pos)[Q])
{
    int sum = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) sum += sub + 16 * q < nm ? pos[q] : 0;
    sum += __builtin_amdgcn_mov_dpp(sum, 0xB1, 0xF, 0xF, true);
    sum += __builtin_amdgcn_mov_dpp(sum, 0x4E, 0xF, 0xF, true);
    sum += __builtin_amdgcn_mov_dpp(sum, 0x141, 0xF, 0xF, true);
    sum += __builtin_amdgcn_mov_dpp(sum, 0x140, 0xF, 0xF, true);
    if (!__any(sum != nm * (nm - 1) / 2)) return;   // 0, 1, ..., nm - 1: all different
    for (int o = 0; o < 16 * Q; ++o) {
        const uint64_t k = keys[o];
#pragma unroll
        for (int q = 0; q < Q; ++q) pos[q] += o < nm && k == mk[q] && o > sub + 16 * q ? 1 : 0;
    }
}

constexpr int kSiftW = 24;

// The closest member of each 45-degree segment around slot t (Sec. 4.3, ties by the
// smaller id) into s_bd, s_best [segment][256 threads]; adds to kfull the members
// within R_full h.
__device__ __forceinline__ void scan_segments(int t, float xi, float yi, const GridState& g,
                                              const int32_t* __restrict__ cell_start, const float* __restrict__ xs,
                                              const float* __restrict__ ys, const int32_t* __restrict__ ids,
                                              const LaunchParams& P, float* s_bd, int* s_best, int tid, int& kfull)
{
    int cx, cy;
    cell_of_pos(g, xi, yi, cx, cy);
    // the rows of three cells are contiguous in slot order: one list of the three
    int base[3], end[3], total = 0;
#pragma unroll
    for (int o = 0; o < 3; ++o) {
        const int yy = cy + o - 1;
        const bool in = yy >= 0 && yy < g.ny;
        const int yc = in ? yy : cy;
        const int u0 = cell_start[yc * g.nx + max(cx - 1, 0)];
        const int u1 = cell_start[yc * g.nx + min(cx + 1, g.nx - 1) + 1];
        base[o] = u0 - total;
        total += in ? u1 - u0 : 0;
        end[o] = total;
    }
    // positions read eight at a time: one memory latency per eight candidates
    for (int k0 = 0; k0 < total; k0 += 8) {
        float bx[8], by[8];
        int bu[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = min(k0 + e, total - 1);   // past the end: a repeat, not visited
            bu[e] = k + (k < end[0] ? base[0] : k < end[1] ? base[1] : base[2]);
            bx[e] = load32(xs, bu[e]);
            by[e] = load32(ys, bu[e]);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int u = bu[e];
            if (k0 + e >= total || u == t) continue;
            float dx = bx[e] - xi;
            float dy = by[e] - yi;
            float d2 = d2_f32(dx, dy);
            if (d2 < P.lo2) continue;
            if (d2 <= P.hi2f) ++kfull;
            if (d2 > P.hi2) continue;
            const int at = segment_f32(dx, dy) * 256 + tid;
            const float cur = s_bd[at];
            if (d2 <= cur) {
                bool take = d2 < cur;
                if (!take) {
                    // equal distance: the smaller id wins
                    const int cb = s_best[at];
                    take = cb >= 0 && ids[u] < ids[cb];
                }
                if (take) {
                    s_bd[at] = d2;
                    s_best[at] = u;
                }
            }
        }
    }
}

// the column record of a queued small LP (see SmallRec): its members in best (slots, -1: none)
__device__ __forceinline__ void write_small_record(const SmallRec& rec, int p1, int i, float xi, float yi,
                                                   const int (&best)[VRM_NSEG], const int32_t* __restrict__ perm,
                                                   const float* __restrict__ xs, const float* __restrict__ ys,
                                                   const int32_t* __restrict__ ids, const LaunchParams& P)
{
    rec.i[p1] = i;
    const size_t cap = (size_t)rec.cap;
    int idb[VRM_NSEG];
#pragma unroll
    for (int s = 0; s < VRM_NSEG; ++s) idb[s] = best[s] >= 0 ? ids[best[s]] : 0x7fffffff;
    int packed = 0;
#pragma unroll
    for (int s = 0; s < VRM_NSEG; ++s) {
        int rank = 0;
#pragma unroll
        for (int o = 0; o < VRM_NSEG; ++o) rank += idb[o] < idb[s] ? 1 : 0;
        packed |= rank << (3 * s);
        const int u = best[s];
        df X{0.0f, 0.0f}, Y{0.0f, 0.0f};
        int pj = -1;
        if (u >= 0) {
            exact_offset(xi, yi, xs[u], ys[u], P.scale2e, X, Y);
            pj = perm[u];
        }
        rec.pj[s * cap + p1] = pj;
        rec.off[(4 * s + 0) * cap + p1] = X.hi;
        rec.off[(4 * s + 1) * cap + p1] = X.lo;
        rec.off[(4 * s + 2) * cap + p1] = Y.hi;
        rec.off[(4 * s + 3) * cap + p1] = Y.lo;
    }
    rec.rank[p1] = packed;
}

}  // namespace vrm

// launcher (vrm_lp_group.hip): complete LPs with sixteen lanes each, as the last LP
// launch of a stencil run: those of the queue q_full, or, where it holds more than
// `limit` (the launches before have then solved them), those left in q_retry
int vrm_lp_group_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp,
                     const vrm::StencilOut& out, int apply, bool stored, int limit, int max_blocks);
// launchers (vrm_verify.hip): the nine-row LPs of the diffused particles from the bases
// in the kept rows; what they do not settle is queued in q_full.  keep_f: also keep the
// fractions.  count_hits: the settled ones are warm-start hits.
int vrm_verify_bases_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp, bool keep_f,
                         bool count_hits);
// the small neighbourhoods and five-row LPs of the diffused particles from the segment
// masks of the stage before, or (from_prev) from the bases recorded by particle id in
// prev; what they do not settle is queued as by the neighbourhood kernel.  prev: also
// record the settled bases there, and count them as warm-start hits.
int vrm_verify_small_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp, int32_t* prev,
                         bool from_prev);
// the kept rows from the bases recorded by particle id (c->prev)
int vrm_bases_from_prev_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n);
// launcher (vrm_lp_group.hip): the removal's identity LPs of the slots in `taken`
int vrm_rm_lp_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp, const int32_t* taken,
                  uint8_t* removed, bool stored);
