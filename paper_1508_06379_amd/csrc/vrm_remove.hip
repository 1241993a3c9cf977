// Particle removal (Sec. 6, outlook): a particle closer than r h to another
// gives its circulation to its complete neighbourhood (r h .. R_full h) by
// the first-order identity LP -- sum g = 1, sum g r = 0, g >= 0, minimising
// sum g (|r/h|^2 + 2^-16 rank^2) -- and is dropped.  Candidates are taken
// greedily in id order, skipping one within R_full h of a taken candidate (so
// no removed particle receives circulation); one whose LP is infeasible stays.
//
// The whole call is enqueued at once: the kernels read the queues' lengths on the
// device, and the host waits once, for the record that the compaction publishes.
// (A copy of the queues to the host after every step of it, six in all, and library
// selections and scans took 350 of a call's 1037 us for 2.7M particles.)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "vrm_lp_common.h"

using namespace vrm;

namespace {

constexpr uint8_t kRmNone = 0, kRmUndecided = 1, kRmIn = 2, kRmOut = 3;

// What a call starts from: empty queues and marks.  A non-finite circulation sets
// kBadGamma, and then nothing is changed.  (By particle: from the slots' kernel, through
// perm, the marks and the circulations cost it more than this launch.)
__global__ __launch_bounds__(256) void k_rm_begin(int n, const float* __restrict__ gamma, GridState* gs,
                                                  uint8_t* __restrict__ removed, Queues* q)
{
    bool bad = false;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        bad = bad || !(fabsf(gamma[i]) <= 3.4028235e38f);
        removed[i] = 0;
    }
    if (__any(bad) && lane_id() == 0 && !(gs->bad & kBadPos)) atomicOr(&gs->bad, kBadGamma);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        q->n_cand = 0;
        q->n_accepted = 0;
        q->n_rm_uncertified = 0;
        for (int k = 0; k < kRmRounds; ++k) q->rm_open[k] = 0;
    }
}

// Candidates: a particle closer than r h to another (per slot), to the queue and to the
// slots' states.
// Bound by the loads of the neighbours: only the cells that the square of side 2 r h
// around the particle touches are read, a quarter of the block of nine (r h is less than
// half a cell).  A workgroup takes a run of slots and appends its candidates once, so that
// few atomics meet on the queue's length.  2.7M particles: 120 us with all nine cells, now
// 73.
constexpr int kCandBlock = 512, kCandBlocks = 1024, kCandBuf = 2048;
__global__ __launch_bounds__(kCandBlock) void k_rm_candidates(int n, const float* __restrict__ xs,
                                                              const float* __restrict__ ys,
                                                              const int32_t* __restrict__ cell_start,
                                                              const GridState* gs, LaunchParams P,
                                                              uint8_t* __restrict__ state, Queues* qs,
                                                              int32_t* __restrict__ cand)
{
    __shared__ int32_t s_buf[kCandBuf];
    __shared__ int s_n, s_at;
    if (threadIdx.x == 0) s_n = 0;
    const GridState g = *gs;
    // an upper bound of |x_j - x_i| over the pairs whose FP32 squared distance is below
    // lo2f; a cell index is monotone in the position, rounding included
    const float rad = sqrtf(P.lo2f) * (1.0f + 9.5367431640625e-7f);
    const int chunk = (n + gridDim.x - 1) / gridDim.x;
    const int lo = min((long)n, (long)blockIdx.x * chunk), hi = min(n, lo + chunk);
    __syncthreads();
    auto flush = [&] {
        __syncthreads();
        const int m = s_n;
        if (threadIdx.x == 0 && m) s_at = atomicAdd(&qs->n_cand, m);
        __syncthreads();
        for (int k = threadIdx.x; k < m; k += kCandBlock) cand[s_at + k] = s_buf[k];
        __syncthreads();
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
    };
    for (int t0 = lo; t0 < hi; t0 += kCandBlock) {
        const int t = t0 + threadIdx.x;
        bool close = false;
        // (slots exist only for finite positions)
        if (t < hi && !g.bad) {
            const float xi = xs[t], yi = ys[t];
            const float xa = xi - rad, xb = xi + rad, ya = yi - rad, yb = yi + rad;
            int cx0, cy0, cx1, cy1;
            cell_of_pos(g, xa - fabsf(xa) * 2.384185791015625e-7f, ya - fabsf(ya) * 2.384185791015625e-7f, cx0, cy0);
            cell_of_pos(g, xb + fabsf(xb) * 2.384185791015625e-7f, yb + fabsf(yb) * 2.384185791015625e-7f, cx1, cy1);
            // two rows of cells at a time (seldom more) as one list, eight particles at a
            // time; past its end the last one again
            for (int yy = cy0; yy <= cy1 && !close; yy += 2) {
                const int u0 = cell_start[yy * g.nx + cx0], len0 = cell_start[yy * g.nx + cx1 + 1] - u0;
                int v0 = 0, total = len0;
                if (yy < cy1) {
                    v0 = cell_start[(yy + 1) * g.nx + cx0] - len0;
                    total = cell_start[(yy + 1) * g.nx + cx1 + 1] - v0;
                }
                for (int k0 = 0; k0 < total && !close; k0 += 8) {
                    float bx[8], by[8];
                    int v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int k = min(k0 + e, total - 1);
                        v[e] = k + (k < len0 ? u0 : v0);
                        bx[e] = load32(xs, v[e]);
                        by[e] = load32(ys, v[e]);
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        close = close || (v[e] != t && d2_f32(bx[e] - xi, by[e] - yi) < P.lo2f);
                }
            }
        }
        if (t < hi) state[t] = close ? kRmUndecided : kRmNone;
        const uint64_t m = __ballot(close);
        int at = 0;
        if (m && lane_id() == 0) at = atomicAdd(&s_n, __popcll(m));
        at = __shfl(at, 0, VRM_WAVE) + __popcll(m & ((1ull << lane_id()) - 1ull));
        if (close) s_buf[at] = t;
        __syncthreads();
        if (s_n > kCandBuf - kCandBlock) flush();   // (the same for every thread)
        __syncthreads();
    }
    flush();
}

// One round of the greedy selection in id order: an undecided candidate with a
// taken candidate within R_full h is out; one with no smaller-id candidate
// still undecided there is taken.  States only go from undecided to taken or
// out, so reading a neighbour's state while it changes is safe: both values
// lead to a decision the sequential greedy pass also makes (nor does it matter whether a
// cache holds an older one).  Bound by latency: eight neighbours are read at once.  A round that leaves a candidate undecided sets
// rm_open[round]; the rounds after one that left none do nothing.
constexpr int kMisBlock = 1024, kMisBlocks = 512;
__global__ __launch_bounds__(kMisBlock) void k_rm_mis_round(int round, const int32_t* __restrict__ cand,
                                                            const float* __restrict__ xs, const float* __restrict__ ys,
                                                            const int32_t* __restrict__ ids,
                                                            const int32_t* __restrict__ cell_start,
                                                            const GridState* gs, LaunchParams P, uint8_t* state,
                                                            Queues* qs, int32_t* __restrict__ taken)
{
    __shared__ int s_n, s_at, s_open;
    const GridState g = *gs;
    if (g.bad || (round > 0 && !qs->rm_open[round - 1])) return;
    if (threadIdx.x == 0) s_open = 0;
    const int nc = qs->n_cand;
    // other threads change the states during the round
    auto state_of = [&](int u) { return __hip_atomic_load(&state[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); };
    auto decide = [&](int u, uint8_t v) {
        __hip_atomic_store(&state[u], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    };
    for (int k0 = blockIdx.x * kMisBlock; k0 < nc; k0 += gridDim.x * kMisBlock) {
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
        const int k = k0 + threadIdx.x;
        bool take = false;
        int t = 0;
        if (k < nc && state_of(t = cand[k]) == kRmUndecided) {
            const float xi = xs[t], yi = ys[t];
            const int id = ids[t];
            int cx, cy;
            cell_of_pos(g, xi, yi, cx, cy);
            bool in_near = false, smaller_open = false;
            for (int oy = -1; oy <= 1; ++oy) {
                const int yy = cy + oy;
                if (yy < 0 || yy >= g.ny) continue;
                const int u0 = cell_start[yy * g.nx + max(cx - 1, 0)];
                const int u1 = cell_start[yy * g.nx + min(cx + 1, g.nx - 1) + 1];
                for (int u = u0; u < u1; u += 8) {
                    uint8_t su[8];
                    float bx[8], by[8];
                    int bi[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int v = min(u + e, u1 - 1);
                        su[e] = state_of(v);
                        bx[e] = xs[v];
                        by[e] = ys[v];
                        bi[e] = ids[v];
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const bool near = u + e < u1 && u + e != t && !(d2_f32(bx[e] - xi, by[e] - yi) > P.hi2f);
                        in_near = in_near || (near && su[e] == kRmIn);
                        smaller_open = smaller_open || (near && su[e] == kRmUndecided && bi[e] < id);
                    }
                }
            }
            if (in_near) {
                decide(t, kRmOut);
            } else if (!smaller_open) {
                decide(t, kRmIn);
                take = true;
            } else {
                s_open = 1;
            }
        }
        const uint64_t m = __ballot(take);
        int at = 0;
        if (m && lane_id() == 0) at = atomicAdd(&s_n, __popcll(m));
        at = __shfl(at, 0, VRM_WAVE) + __popcll(m & ((1ull << lane_id()) - 1ull));
        __syncthreads();
        if (threadIdx.x == 0 && s_n) s_at = atomicAdd(&qs->n_accepted, s_n);
        __syncthreads();
        if (take) taken[s_at + at] = t;
        __syncthreads();
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_open) qs->rm_open[round] = 1;
}

// Received circulation, and the particles that stay, in their order, moved to the front
// in place, in one pass.  A tile's particles are in registers before the tile publishes
// its count, and a particle is only moved to a place whose tile has published: no place
// is written before it has been read.  Tiles are taken by ticket and look back only at
// lower tickets, which run already and publish their counts before they wait, so every
// wait ends.  A circulation that changed is also written back where it stood (past the
// new count that is where it stays), write-through and waited for before the count is
// published, so that what a later tile puts there comes after it, whichever L2 holds it.
// Bound by HBM: 20 bytes read and up to 16 written per particle.
// 2.7M particles: 60 us as four kernels (apply, scan, gather, copy), now 36.
constexpr int kPackBlock = 512, kPackPer = 8, kPackTile = kPackBlock * kPackPer;
static_assert(kPackTiles * (long)kPackTile >= (1l << 26), "a tile word for every tile of the largest cloud");
constexpr uint64_t kTileSum = 1ull << 32, kTileAll = 2ull << 32;   // under the call's number

__global__ __launch_bounds__(kPackBlock) void k_rm_pack(int n, float* x, float* y, float* gamma, int32_t* id,
                                                        float* acc, const uint8_t* __restrict__ removed,
                                                        const GridState* gs, Queues* qs, CellScratch* sc,
                                                        int32_t* n_dev, HostQueues* host, int32_t seq)
{
    constexpr int W = kPackBlock / 64;
    __shared__ int s_tile, s_before;
    __shared__ int s_cnt[kPackPer * W], s_off[kPackPer * W];
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    // nothing to move (or the choice has not been completed): the record only
    if (gs->bad || qs->rm_open[kRmRounds - 1] || qs->n_accepted == 0) {
        if (blockIdx.x == 0 && tid == 0) publish(qs, gs, n, host, seq);
        return;
    }
    if (tid == 0) s_tile = atomicAdd(&sc->pack_ticket, 1);
    __syncthreads();
    const int tile = s_tile, base = tile * kPackTile;
    float bx[kPackPer], by[kPackPer], bg[kPackPer], ba[kPackPer];
    int32_t bi[kPackPer];
    uint8_t gone[kPackPer];
    uint32_t keep = 0;   // bit e: element e stays
    int at[kPackPer];
#pragma unroll
    for (int e = 0; e < kPackPer; ++e) {
        const int k = min(base + e * kPackBlock + tid, n - 1);
        gone[e] = removed[k];
        bg[e] = gamma[k];
        ba[e] = acc[k];
        bx[e] = x[k];
        by[e] = y[k];
        bi[e] = id[k];
    }
#pragma unroll
    for (int e = 0; e < kPackPer; ++e) {
        const int i = base + e * kPackBlock + tid;
        const bool stays = i < n && !gone[e];
        if (i < n) {
            const float s = bg[e] + ba[e];
            if (__float_as_uint(s) != __float_as_uint(bg[e]))
                __hip_atomic_store(&gamma[i], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (ba[e] != 0.0f) acc[i] = 0.0f;
            bg[e] = s;
        }
        const uint64_t m = __ballot(stays);
        at[e] = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) s_cnt[e * W + w] = __popcll(m);
        keep |= stays ? 1u << e : 0u;
    }
    // this thread's loads have arrived and its stores are done, then everyone's
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid < 64) {
        // element rows in order, the waves of a row in order
        static_assert(kPackPer * W == 64, "one count per lane");
        const int c = s_cnt[lane];
        int incl = c;
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, VRM_WAVE);
            if (lane >= o) incl += v;
        }
        s_off[lane] = incl - c;
        const int total = __shfl(incl, 63, VRM_WAVE);
        const uint64_t call = (uint64_t)(uint32_t)seq << 34;
        if (lane == 0)
            __hip_atomic_store(&sc->pack[tile], call | (tile == 0 ? kTileAll : kTileSum) | (uint32_t)total,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int before = 0;
        // look back, 64 tiles at a time: a lane's tile, or an empty sum past the first
        for (int end = tile; end > 0; end -= 64) {
            const int j = end - 1 - lane;
            uint64_t v = call | kTileAll;
            if (j >= 0)
                while ((v = __hip_atomic_load(&sc->pack[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 34 !=
                       call >> 34)
                    __builtin_amdgcn_s_sleep(1);
            const uint64_t all = __ballot((v & kTileAll) != 0);
            // up to the nearest tile whose word holds the sum of everything before it
            const int stop = all ? __ffsll((unsigned long long)all) - 1 : 63;
            int part = lane <= stop ? (int)(uint32_t)v : 0;
            for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, VRM_WAVE);
            before += part;
            if (all) break;
        }
        if (lane == 0) {
            if (tile > 0)
                __hip_atomic_store(&sc->pack[tile], call | kTileAll | (uint32_t)(before + total), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            s_before = before;
            if (tile == (int)gridDim.x - 1) {
                // every ticket has been taken
                __hip_atomic_store(&sc->pack_ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *n_dev = before + total;
                publish(qs, gs, before + total, host, seq);
            }
        }
    }
    __syncthreads();
    const int before = s_before;
#pragma unroll
    for (int e = 0; e < kPackPer; ++e) {
        const int i = base + e * kPackBlock + tid;
        const int j = before + s_off[e * W + w] + at[e];
        if ((keep >> e & 1u) && j != i) {
            x[j] = bx[e];
            y[j] = by[e];
            gamma[j] = bg[e];
            id[j] = bi[e];
        }
    }
}

__global__ void k_rm_reset_rounds(Queues* q)
{
    for (int k = 0; k < kRmRounds; ++k) q->rm_open[k] = 0;
}

}  // namespace

// Particle removal over the current cell list (slot order).  Waits for the counts (the last
// tile of the compaction publishes them): the arrays are complete in stream order.  Returns
// the new particle count or a negative error.
int vrm_remove_run(vrm_ctx* c, vrm_cloud* cl, int32_t n, const LaunchParams& lp, bool stored, int32_t* n_candidates)
{
    hipStream_t s = c->stream;
    if (n_candidates) *n_candidates = 0;
    if (n == 0) return n;
    int32_t* cand = c->cperm;
    int32_t* taken = c->aidx;
    uint8_t* removed = c->tmp_u8;
    hipLaunchKernelGGL(k_rm_begin, dim3(std::min((n + 1023) / 1024, 1024)), dim3(256), 0, s, n, cl->gamma_dev, c->grid,
                       removed, c->queues);
    hipLaunchKernelGGL(k_rm_candidates, dim3(std::min((n + kCandBlock - 1) / kCandBlock, kCandBlocks)),
                       dim3(kCandBlock), 0, s, n, c->xs, c->ys, c->cell_start, c->grid, lp, c->cstate, c->queues, cand);
    for (int rounds = kRmRounds;; rounds += kRmRounds) {
        const int nbm = std::min((n + kMisBlock - 1) / kMisBlock, kMisBlocks);
        for (int k = 0; k < kRmRounds; ++k)
            hipLaunchKernelGGL(k_rm_mis_round, dim3(nbm), dim3(kMisBlock), 0, s, k, cand, c->xs, c->ys, c->ids,
                               c->cell_start, c->grid, lp, c->cstate, c->queues, taken);
        VRM_HIP(hipGetLastError());
        if (int r = vrm_rm_lp_run(c, cl, n, lp, taken, removed, stored)) return r;
        const int32_t seq = ++c->q_seq;
        hipLaunchKernelGGL(k_rm_pack, dim3((n + kPackTile - 1) / kPackTile), dim3(kPackBlock), 0, s, n, cl->x_dev,
                           cl->y_dev, cl->gamma_dev, cl->id_dev, c->acc, removed, c->grid, c->queues, c->cell_scratch,
                           cl->n_dev, c->q_host, seq);
        VRM_HIP(hipGetLastError());
        Queues q;
        if (int r = vrm_wait_queues(c, seq, q)) return r;
        if (q.nonfinite) return vrm_nonfinite(c, q.nonfinite);   // nothing changed
        if (n_candidates) *n_candidates = q.n_cand;
        if (!q.rm_open[kRmRounds - 1]) return q.n_now;
        if (rounds > 4 * (long)q.n_cand + 64) return vrm_fail(VRM_E_STATE, "removal: selection did not converge");
        hipLaunchKernelGGL(k_rm_reset_rounds, dim3(1), dim3(1), 0, s, c->queues);
    }
}
