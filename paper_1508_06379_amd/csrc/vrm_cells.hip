// Cell lists, reduced-operator selection and particle insertion of libvrm.
//
// Cell list: a counting sort of the particles into square cells of edge
// max(R, R_full) h (so a 3 x 3 block of cells covers every neighbourhood),
// over the bounding box found on the device.  Selection: Sec. 3.5, eq.
// reduced_bound, by a radix select on the bits of |Gamma| with FP64 bucket
// sums.  Insertion: Sec. 4.2, with conflicts between candidates resolved to
// the greedy result in (id, segment) order by rounds of the lexicographically
// first independent set.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <rocprim/device/device_radix_sort.hpp>

#include "vrm_device.h"
#include "vrm_internal.h"

using namespace vrm;

namespace {

// The grid of a cloud: its bounding box, and by the last workgroup the cells.  Bound by
// latency for small clouds and by HBM for large ones: eight particles of a thread are in
// flight at once, and every workgroup leaves its box in a slot of its own (four atomics
// of every workgroup on one address each were 18 of 35 us at 2.7M particles).
constexpr int kBoxPer = 8;
// cells of a side: a position past the last is given that one's index as a float, which
// holds whole numbers up to 2^24 (a longer side's last index may round to one past it)
constexpr long long kMaxSide = 1ll << 24;
__global__ __launch_bounds__(256) void k_grid(const float* __restrict__ x, const float* __restrict__ y, int n,
                                              const int32_t* __restrict__ n_dev, GridState* g, CellScratch* sc, float cs,
                                              int ncell_cap, vrm_counters* cnt)
{
    if (n_dev) n = *n_dev;
    uint32_t mnx = 0xffffffffu, mny = 0xffffffffu, mxx = 0u, mxy = 0u;
    bool bad = false;
    const int stride = gridDim.x * 256;
    auto take = [&](float xv, float yv) {
        if (!(fabsf(xv) <= 3.4028235e38f) || !(fabsf(yv) <= 3.4028235e38f)) {
            bad = true;   // NaN or infinite: reported, never given a cell
            return;
        }
        const uint32_t kx = ordered_key(xv), ky = ordered_key(yv);
        mnx = min(mnx, kx);
        mny = min(mny, ky);
        mxx = max(mxx, kx);
        mxy = max(mxy, ky);
    };
    for (long i = blockIdx.x * 256 + threadIdx.x; i < n; i += (long)kBoxPer * stride) {
        float xv[kBoxPer], yv[kBoxPer];
#pragma unroll
        for (int e = 0; e < kBoxPer; ++e) {
            const long k = min(i + (long)e * stride, (long)n - 1);   // past the end: a repeat
            xv[e] = x[k];
            yv[e] = y[k];
        }
#pragma unroll
        for (int e = 0; e < kBoxPer; ++e) take(xv[e], yv[e]);
    }
    __shared__ uint32_t red[4][4];
    // over the wave, then over the four waves
    auto reduce = [&] {
        for (int o = 32; o > 0; o >>= 1) {
            mnx = min(mnx, (uint32_t)__shfl_xor((int)mnx, o, VRM_WAVE));
            mny = min(mny, (uint32_t)__shfl_xor((int)mny, o, VRM_WAVE));
            mxx = max(mxx, (uint32_t)__shfl_xor((int)mxx, o, VRM_WAVE));
            mxy = max(mxy, (uint32_t)__shfl_xor((int)mxy, o, VRM_WAVE));
        }
        const int w = threadIdx.x >> 6;
        __syncthreads();
        if (lane_id() == 0) {
            red[0][w] = mnx;
            red[1][w] = mny;
            red[2][w] = mxx;
            red[3][w] = mxy;
        }
        __syncthreads();
        for (int k = 0; k < 4; ++k) {
            mnx = min(mnx, red[0][k]);
            mny = min(mny, red[1][k]);
            mxx = max(mxx, red[2][k]);
            mxy = max(mxy, red[3][k]);
        }
    };
    reduce();
    uint32_t old = 0u;
    if (threadIdx.x < 4)
        old = atomicExch(&sc->box[threadIdx.x][blockIdx.x],
                         threadIdx.x == 0 ? mnx : threadIdx.x == 1 ? mny : threadIdx.x == 2 ? mxx : mxy);
    if (__any(bad) && lane_id() == 0) old |= (uint32_t)atomicOr(&sc->bad_seen, kBadPos);
    asm volatile("" ::"v"(old));   // waits for the atomics' results
    if (!last_here(sc->done)) return;
    for (int k = threadIdx.x; k < (int)gridDim.x; k += 256) {
        mnx = min(mnx, __hip_atomic_load(&sc->box[0][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        mny = min(mny, __hip_atomic_load(&sc->box[1][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        mxx = max(mxx, __hip_atomic_load(&sc->box[2][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        mxy = max(mxy, __hip_atomic_load(&sc->box[3][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    reduce();
    if (threadIdx.x != 0) return;
    const int32_t bad_seen = __hip_atomic_load(&sc->bad_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sc->bad_seen = 0;
    g->bad = (g->bad & ~kBadPos) | bad_seen;
    float xmin = 0.0f, ymin = 0.0f, xmax = 0.0f, ymax = 0.0f;
    if (mnx != 0xffffffffu) {
        xmin = ordered_key_inv(mnx);
        ymin = ordered_key_inv(mny);
        xmax = ordered_key_inv(mxx);
        ymax = ordered_key_inv(mxy);
    }
    g->cs = cs;
    const float inv_cs = 1.0f / cs, x0 = xmin - cs, y0 = ymin - cs;
    g->inv_cs = inv_cs;
    g->x0 = x0;
    g->y0 = y0;
    double fx = ((double)xmax - (double)x0) * (double)inv_cs;
    double fy = ((double)ymax - (double)y0) * (double)inv_cs;
    long long nx = (long long)fmin(fx, 1.0e9) + 2;
    long long ny = (long long)fmin(fy, 1.0e9) + 2;
    int clamped = 0;
    if (nx * ny > ncell_cap || max(nx, ny) > kMaxSide) {
        // keep the aspect ratio; far particles share the edge cells (still exact, slower)
        const double f = fmin(sqrt((double)ncell_cap / (double)(nx * ny)), 1.0);
        // (a side alone may exceed the capacity: a few particles in a long, thin box)
        nx = min(max((long long)(nx * f), 1ll), min((long long)ncell_cap, kMaxSide));
        ny = min(min(ny, ncell_cap / nx), kMaxSide);
        clamped = 1;
    }
    g->nx = (int)nx;
    g->ny = (int)ny;
    g->ncells = (int)(nx * ny);
    g->clamped = clamped;
    if (clamped) atomicAdd(&cnt->n_grid_clamped, 1);
}

__device__ __forceinline__ void cell_xy(const GridState& g, float x, float y, int& cx, int& cy)
{
    float fx = (x - g.x0) * g.inv_cs;
    float fy = (y - g.y0) * g.inv_cs;
    fx = fminf(fmaxf(fx, 0.0f), (float)(g.nx - 1));
    fy = fminf(fmaxf(fy, 0.0f), (float)(g.ny - 1));
    cx = (int)fx;
    cy = (int)fy;
}
__device__ __forceinline__ int cell_index(const GridState& g, float x, float y)
{
    int cx, cy;
    cell_xy(g, x, y, cx, cy);
    return cy * g.nx + cx;
}

// count: particles per cell, zero before and after a build (k_cell_starts clears it)
__global__ __launch_bounds__(256) void k_count(const float* __restrict__ x, const float* __restrict__ y, int n,
                                               const int32_t* __restrict__ n_dev, const GridState* gs, int32_t* count,
                                               int32_t* rank)
{
    if (n_dev) n = min(n, *n_dev);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = i < n;
    const GridState g = *gs;
    if (g.bad & kBadPos) return;   // a non-finite position: no cell indices (the same for every thread)
    const int c = live ? cell_index(g, x[i], y[i]) : -1;
    // The rank only has to be unique within the cell.  The cloud is kept in cell order,
    // so the lanes of a wave form runs of one cell: the first lane of a run adds for all,
    // one atomic in flight per lane.  (Grouping the lanes of equal cells wherever they
    // are, in rounds, each round's atomic waiting for the one before, took 73 us for 2.7M
    // particles, with the atomics issued together 55, now 15.)
    const int lane = lane_id();
    const int left = __shfl_up(c, 1, VRM_WAVE);
    const uint64_t heads = __ballot(lane == 0 || c != left);
    const int head = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
    const uint64_t after = lane == 63 ? 0ull : heads & (~0ull << (lane + 1));
    const int at = lane - head, size = (after ? __ffsll((unsigned long long)after) - 1 : 64) - lane;   // of a head
    int base = 0;
    if (live && head == lane) base = atomicAdd(&count[c], size);
    base = __shfl(base, head, VRM_WAVE);
    if (live) rank[i] = base + at;
}

// exclusive scan over the workgroup
__device__ __forceinline__ int block_exclusive_scan(int v, int& total)
{
    __shared__ int wsum[16];
    const int lane = lane_id(), w = threadIdx.x >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, VRM_WAVE);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    const int nw = blockDim.x >> 6;
    int off = 0, tot = 0;
    for (int k = 0; k < nw; ++k) {
        const int s = wsum[k];
        if (k < w) off += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return off + incl - v;
}

// First slots of the cells: the exclusive scan of the counts, which are cleared, in one
// launch.  A workgroup takes its chunk by a ticket, publishes the chunk's sum with the
// launch's number in one 64-bit word, and adds the sums of the chunks before it: it waits
// only for workgroups with lower tickets, which run already and publish before they
// wait, so every wait ends whatever else runs on the GPU.  (Three launches before; each
// is 4.6 us of a small cloud's stage.)  The launch's number is the ticket's upper part:
// kCellParts divides 2^32, so it stays in step when the counter wraps.
__global__ __launch_bounds__(1024) void k_cell_starts(int32_t* __restrict__ count, int32_t* __restrict__ start,
                                                      const GridState* g, CellScratch* sc)
{
    __shared__ uint32_t s_ticket;
    const int t = threadIdx.x;
    if (t == 0) s_ticket = atomicAdd(&sc->ticket, 1u);
    const int nc = g->ncells;
    __syncthreads();
    const int b = (int)(s_ticket % kCellParts);
    const uint32_t launch = s_ticket / kCellParts + 1u;
    // whole groups of four cells (the counts past the last cell are zero)
    const int chunk = ((nc + kCellParts - 1) / kCellParts + 3) & ~3;
    const int lo = min(nc, b * chunk), hi = min(nc, lo + chunk);
    int sum = 0;
    for (int c = lo + 4 * t; c < hi; c += 4 * 1024) {
        const int4 v = *reinterpret_cast<const int4*>(&count[c]);
        sum += v.x + v.y + v.z + v.w;
    }
    int total;
    (void)block_exclusive_scan(sum, total);
    if (t == 0)
        __hip_atomic_store(&sc->part[b], ((uint64_t)launch << 32) | (uint32_t)total, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    int before = 0;
    if (t < b) {
        uint64_t v;
        while ((uint32_t)((v = __hip_atomic_load(&sc->part[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 32) !=
               launch)
            __builtin_amdgcn_s_sleep(1);
        before = (int)(uint32_t)v;
    }
    int carry;
    (void)block_exclusive_scan(before, carry);
    for (int c0 = lo; c0 < hi; c0 += 4 * 1024) {
        const int c = c0 + 4 * t;
        int4 v = {0, 0, 0, 0};
        if (c < hi) {
            v = *reinterpret_cast<const int4*>(&count[c]);
            *reinterpret_cast<int4*>(&count[c]) = int4{0, 0, 0, 0};
        }
        int tot;
        const int ex = carry + block_exclusive_scan(v.x + v.y + v.z + v.w, tot);
        carry += tot;
        const int o[4] = {ex, ex + v.x, ex + v.x + v.y, ex + v.x + v.y + v.z};
        if (c + 3 < hi) {
            *reinterpret_cast<int4*>(&start[c]) = int4{o[0], o[1], o[2], o[3]};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c + e < hi) start[c + e] = o[e];
        }
    }
    if (b == kCellParts - 1 && t == 0) start[nc] = carry;
}

__global__ __launch_bounds__(256) void k_scatter(const float* __restrict__ x, const float* __restrict__ y,
                                                 const int32_t* __restrict__ id, int n,
                                                 const int32_t* __restrict__ n_dev,
                                                 const int32_t* __restrict__ start, const int32_t* __restrict__ rank,
                                                 int32_t* perm, float* xs, float* ys, int32_t* ids, const GridState* gs)
{
    if (n_dev) n = min(n, *n_dev);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const GridState g = *gs;
    if (i >= n || (g.bad & kBadPos)) return;
    const float xi = x[i], yi = y[i];
    const int t = start[cell_index(g, xi, yi)] + rank[i];
    perm[t] = i;
    xs[t] = xi;
    ys[t] = yi;
    ids[t] = id[i];
}

// ------------------------------------------------------ reduced operator
// Ranking key (Sec. 3.5): the bits of |Gamma| in FP32, monotone in the value
// for non-negative floats; particles with equal keys form one group, left out
// together.  Radix passes resolve the whole key: 11, 11 and 10 bits with a context's bins,
// four of 8 bits with those of the selection without a context.
__device__ __forceinline__ uint32_t selection_key(float a) { return __float_as_uint(a); }

// The state before a selection: nothing picked, every bin zero.  The last pass leaves
// it so (the context's selections need no launch for it); a fresh state, and one that
// overlapping calls may have spoiled, is set by this kernel.
__global__ __launch_bounds__(256) void k_sel_init(SelectState* s, double* bins, int nbins, GridState* gs)
{
    const int t = threadIdx.x;
    for (int b = t; b < nbins; b += blockDim.x) bins[b] = 0.0;
    if (t < 17) s->done_blocks[t] = 0;
    if (t == 0) {
        s->max_seen = 0u;
        s->bad_seen = 0;
        s->max_id = -1;
        s->done = 2u;   // of no particle at all: none is diffused
        s->threshold = 0u;
        if (gs) gs->bad &= ~kBadGamma;
    }
}

__global__ void k_publish_queues(const Queues* q, const GridState* g, const int32_t* n_dev, HostQueues* h, int32_t seq)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) publish(q, g, n_dev ? *n_dev : 0, h, seq);
}

constexpr int kSelBlock = 1024;
constexpr int kSelLds = 8192;   // FP64 bins in LDS, all copies

// inclusive FP64 scan over the workgroup in thread order (the same association in every run)
__device__ __forceinline__ double block_scan_f64(double v, double* wtot)
{
    const int lane = lane_id(), w = threadIdx.x >> 6;
    double incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const double u = __shfl_up(incl, o, VRM_WAVE);
        if (lane >= o) incl += u;
    }
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    double off = 0.0;
    for (int k = 0; k < w; ++k) off += wtot[k];
    return off + incl;
}

// One radix pass over BITS bits of the key from `shift` up, and the choice of the bin
// where the cumulative sum first exceeds the bound by the last workgroup to finish.
// A bin holds FP32 values that share at least the top seven bits of their exponent,
// i.e. values in [2^E, 2^(E+2)) that are multiples of 2^(E-23); up to 2^26 of them sum
// to below 2^(E+28), a multiple of 2^(E-23) with at most 51 significant bits, so every
// FP64 bin sum is exact and does not depend on the order of the atomics.  The first
// pass also finds non-finite circulations (kBadGamma) and the largest id.
// Neighbouring particles have circulations of one magnitude, so a wave's first-pass
// atomics fall on one or two bins: the bins have copies for the lanes (32 of 256 bins,
// 8 of 1024), next to each other.  With one copy the pass took 99 us for 1.4M particles
// (10 us for 40k).  The workgroups' sums meet by atomics whose results are waited for,
// so the last workgroup reads complete bins without a fence (which would write back the
// caches of every XCD once per workgroup).
// With n_dev the count is the device's (nothing is done with one outside 0..n), and the
// first pass hands it to the host: while the passes run, the host reads it and enqueues
// the launches that need it.
template <int BITS, bool FIRST>
__global__ __launch_bounds__(kSelBlock) void k_sel_pass(const float* __restrict__ g, const int32_t* __restrict__ ids,
                                                        int n, const int32_t* __restrict__ n_dev, SelectState* s,
                                                        double* bins, int shift, double factor, GridState* gs,
                                                        vrm_counters* cnt, Queues* qs, HostQueues* host, int32_t seq)
{
    if (n_dev) {
        const int n_now = *n_dev;
        if (FIRST && blockIdx.x == 0 && threadIdx.x == 0) publish(nullptr, nullptr, n_now, host, seq);
        if (n_now < 0 || n_now > n) return;
        n = n_now;
    }
    constexpr int NB = 1 << BITS;
    constexpr int USED = FIRST ? NB / 2 : NB;   // the sign bit is zero
    constexpr int COPIES = kSelLds / USED < 32 ? kSelLds / USED : 32;
    __shared__ double h[USED * COPIES];
    __shared__ double wtot[kSelBlock / 64];
    __shared__ uint32_t s_mid[FIRST ? kSelBlock / 64 : 1];
    __shared__ int s_first;
    const int t = threadIdx.x;
    const bool done = !FIRST && s->done != 0u;
    const uint32_t pre = FIRST ? 0u : s->key_prefix;
    if (!done) {
        for (int b = t; b < USED * COPIES; b += kSelBlock) h[b] = 0.0;
        __syncthreads();
        const int copy = lane_id() & (COPIES - 1);
        bool bad = false;
        uint32_t mid = 0u;
        for (int i = blockIdx.x * kSelBlock + t; i < n; i += gridDim.x * kSelBlock) {
            const float a = fabsf(g[i]);
            const uint32_t key = selection_key(a);
            if (FIRST) {
                bad = bad || key >= 0x7f800000u;
                if (ids) mid = max(mid, ids[i] >= 0 ? (uint32_t)ids[i] + 1u : 0u);
            } else if ((key ^ pre) >> (shift + BITS)) {
                continue;
            }
            atomicAdd(&h[((key >> shift) & (NB - 1)) * COPIES + copy], (double)a);
        }
        if (FIRST) {
            for (int o = 32; o > 0; o >>= 1) mid = max(mid, (uint32_t)__shfl_xor((int)mid, o, VRM_WAVE));
            // one atomic of a workgroup (one of every wave, on the one address, took 45 us
            // for 640k particles)
            if (lane_id() == 0) s_mid[t >> 6] = mid;
            const int any = __syncthreads_or(bad);
            if (t == 0) {
                for (int k = 0; k < kSelBlock / 64; ++k) mid = max(mid, s_mid[k]);
                uint32_t old = atomicMax(&s->max_seen, mid);
                if (any) old |= (uint32_t)atomicOr(&s->bad_seen, 1);
                asm volatile("" ::"v"(old));   // waits for the atomics' results
            }
        }
        __syncthreads();
        for (int b = t; b < USED; b += kSelBlock) {
            double v = 0.0;
            for (int c = 0; c < COPIES; ++c) v += h[b * COPIES + c];   // exact: any order
            if (v != 0.0) {
                const double old = atomicAdd(&bins[b], v);
                asm volatile("" ::"v"(old));
            }
        }
    }
    if (t == 0) s_first = NB;
    if (!last_here(s->done_blocks)) return;
    if (FIRST) {
        // what the step's later kernels start from
        if (cnt && t < kCounterStripes)
            reinterpret_cast<vrm_counters*>(reinterpret_cast<char*>(cnt) + t * kCounterStride)->n_diffused = 0;
        if (t == 0) {
            const uint32_t m = __hip_atomic_load(&s->max_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int32_t bad = __hip_atomic_load(&s->bad_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s->max_id = (int32_t)m - 1;
            s->max_seen = 0u;
            s->bad_seen = 0;
            gs->bad = (gs->bad & ~kBadGamma) | (bad ? kBadGamma : 0);
            if (qs) {
                qs->n_cand = 0;
                qs->n_accepted = 0;
                qs->small_state = 0;
            }
        }
    }
    if (done) return;
    // PB consecutive bins per thread
    constexpr int PB = NB > kSelBlock ? NB / kSelBlock : 1;
    double v[PB], sum = 0.0;
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        const int b = PB * t + p;
        v[p] = b < USED ? __hip_atomic_load(&bins[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
        if (b < USED) bins[b] = 0.0;
        sum += v[p];
    }
    const double incl = block_scan_f64(sum, wtot);
    double total = 0.0;
    for (int k = 0; k < kSelBlock / 64; ++k) total += wtot[k];
    const double bound = FIRST ? factor * total : s->bound, prefix = FIRST ? 0.0 : s->prefix;
    double before[PB], at = incl - sum;
    int mine = NB;
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        before[p] = at;
        at = p == PB - 1 ? incl : at + v[p];
        if (mine == NB && prefix + at > bound) mine = PB * t + p;
    }
    if (mine < NB && mine < USED) atomicMin(&s_first, mine);
    __syncthreads();
    const int first = s_first;
    if (t == 0) {
        if (FIRST) {
            s->norm1 = total;
            s->bound = bound;
        }
        if (first == NB) {
            // every particle in the current key range is left out
            const uint64_t top = (uint64_t)pre + ((uint64_t)NB << shift);
            s->threshold = top > 0xffffffffull ? 0xffffffffu : (uint32_t)top;
            s->done = top > 0xffffffffull ? 2u : 1u;
        } else {
            const uint32_t p = pre | ((uint32_t)first << shift);
            s->key_prefix = p;
            s->threshold = p;
            s->done = shift == 0 ? 1u : 0u;
        }
        if (first == NB) s->prefix = 0.0;
    }
    // cumulative sum below the chosen bin, for the next pass
#pragma unroll
    for (int p = 0; p < PB; ++p)
        if (PB * t + p == first) s->prefix = prefix + before[p];
}

// Diffused: |Gamma| >= fl32(T (1 - 2^-16)), T the first key that does not fit:
// the particle that reaches the bound and every particle within a relative
// 2^-16 below it are diffused (circulations equal in exact arithmetic differ by
// round-off once computed: 2^-16 covers the stated 1e-5 per-value bound and the
// random-walk round-off of FP32 circulations over 10^2 SSP-RK3 steps).
constexpr float kTieBand = 0.9999847412109375f;   // 1 - 2^-16

__device__ __forceinline__ bool is_diffused(const SelectState* s, float g)
{
    return s->done != 2u && fabsf(g) >= __uint_as_float(s->threshold) * kTieBand;
}

__global__ __launch_bounds__(256) void k_sel_mask(const float* __restrict__ g, int n, const SelectState* s,
                                                  uint8_t* diffused, uint8_t* mask_out, vrm_counters* cnt)
{
    if (cnt) cnt = counter_stripe(cnt);
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    bool d = false;
    if (i < n) {
        d = is_diffused(s, g[i]);
        diffused[i] = d ? 1 : 0;
        if (mask_out) mask_out[i] = d ? 1 : 0;
    }
    uint64_t m = __ballot(d);
    if (cnt && lane_id() == 0 && m) atomicAdd(&cnt->n_diffused, __popcll(m));
}

// ------------------------------------------------------------ insertion
// Candidates: every empty segment of a diffused particle (slot order); the kernel also
// writes the diffused set that the selection's threshold defines.
// L lanes per particle (aligned groups; L = 4 for clouds up to kCandCoopMaxN
// particles, where one lane per particle leaves the chip mostly idle and the
// chain of loads of one scan sets the time): the lanes scan interleaved
// candidates and OR their occupied segments; the group's lead lane appends.
constexpr int kCandCoopMaxN = 1 << 18;

template <int L>
__global__ __launch_bounds__(256) void k_candidates(int n, const int32_t* __restrict__ perm,
                                                    const float* __restrict__ xs, const float* __restrict__ ys,
                                                    const int32_t* __restrict__ ids,
                                                    const int32_t* __restrict__ cell_start,
                                                    const float* __restrict__ gamma, const SelectState* sel,
                                                    uint8_t* diffused, vrm_counters* cnt, const GridState* gs,
                                                    LaunchParams P, Queues* qs, int cand_cap, float* cx, float* cy,
                                                    uint64_t* ckey, uint8_t* cstate)
{
    const int sub = threadIdx.x & (L - 1);
    const int t = blockIdx.x * (256 / L) + threadIdx.x / L;
    int occupied = 0xff;
    float xi = 0.0f, yi = 0.0f;
    bool dif = false;
    if (t < n && !gs->bad) {
        const int i = perm[t];
        dif = is_diffused(sel, gamma[i]);
        if (sub == 0) diffused[i] = dif ? 1 : 0;
    }
    const uint64_t members = __ballot(dif && sub == 0);
    if (lane_id() == 0 && members) atomicAdd(&counter_stripe(cnt)->n_diffused, __popcll(members));
    if (dif) {
        occupied = 0;
        const GridState g = *gs;
        xi = xs[t];
        yi = ys[t];
        // the cells that the square around the particle touches (an upper bound of the
        // offsets whose FP32 squared length is within hi2; cell indices are monotone)
        const float rad = sqrtf(P.hi2) * (1.0f + 9.5367431640625e-7f);
        const float xa = xi - rad, xb = xi + rad, ya = yi - rad, yb = yi + rad;
        int cx0, cy0, cx1, cy1;
        cell_xy(g, xa - fabsf(xa) * 2.384185791015625e-7f, ya - fabsf(ya) * 2.384185791015625e-7f, cx0, cy0);
        cell_xy(g, xb + fabsf(xb) * 2.384185791015625e-7f, yb + fabsf(yb) * 2.384185791015625e-7f, cx1, cy1);
        // until every segment is occupied (inside a cloud: after about half of them)
        for (int yy = cy0; yy <= cy1 && occupied != 0xff; ++yy) {
            // the cells of a row are contiguous in slot order
            const int u0 = cell_start[yy * g.nx + cx0], u1 = cell_start[yy * g.nx + cx1 + 1];
            // positions read eight at a time: one memory latency per eight candidates
            for (int ub = u0 + sub; ub < u1 && occupied != 0xff; ub += 8 * L) {
                float bx[8], by[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int v = min(ub + L * e, u1 - 1);   // past the end: a repeat, not visited
                    bx[e] = load32(xs, v);
                    by[e] = load32(ys, v);
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int u = ub + L * e;
                    if (u >= u1 || u == t) continue;
                    float dx = bx[e] - xi;
                    float dy = by[e] - yi;
                    float d2 = d2_f32(dx, dy);
                    if (d2 < P.lo2 || d2 > P.hi2) continue;
                    occupied |= 1 << segment_f32(dx, dy);
                }
            }
        }
    }
#pragma unroll
    for (int o = 1; o < L; o <<= 1) occupied |= __shfl_xor(occupied, o, VRM_WAVE);
    __shared__ int s_app[17];
    int empty = (~occupied) & 0xff;
    int want = sub == 0 ? __popc(empty) : 0;
    int base = block_append_n(&qs->n_cand, want, s_app);
    if (want) {
        int id = ids[t];
        int k = 0;
        for (int s = 0; s < VRM_NSEG; ++s) {
            if (!(empty & (1 << s))) continue;
            int p = base + k++;
            if (p >= cand_cap) continue;
            float xc, yc;
            candidate_f32(xi, yi, P.rad, s, xc, yc);
            cx[p] = xc;
            cy[p] = yc;
            ckey[p] = ((uint64_t)(uint32_t)id << 3) | (uint64_t)s;
            cstate[p] = 0;
        }
    }
}

// The candidates in cell order, as the rounds read them: position and key by slot.
struct CandSlots {
    float* x;
    float* y;
    uint64_t* key;
    uint8_t* state;     // 0 undecided, 1 accepted, 2 rejected
    int32_t* taken;     // accepted slots, in no order
    uint32_t* mask;     // by particle id, a byte each: segments with an accepted candidate
};

// Cleared marks of the ids in the cloud (up to the capacity) and of the rounds.
__global__ __launch_bounds__(256) void k_ins_begin(int capacity, const SelectState* sel, CandSlots C, Queues* qs)
{
    const int words = ((int)min((long)sel->max_id + 1, (long)capacity) + 3) / 4;
    for (int k = blockIdx.x * 256 + threadIdx.x; k < words; k += gridDim.x * 256) C.mask[k] = 0u;
    if (blockIdx.x == 0 && threadIdx.x < kRmRounds) qs->rm_open[threadIdx.x] = 0;
}

__global__ __launch_bounds__(256) void k_ins_scatter(const float* __restrict__ cx, const float* __restrict__ cy,
                                                     const uint64_t* __restrict__ ckey, int nc,
                                                     const int32_t* __restrict__ start,
                                                     const int32_t* __restrict__ rank, CandSlots C, const GridState* gs)
{
    const int a = blockIdx.x * 256 + threadIdx.x;
    if (a >= nc) return;
    const float x = cx[a], y = cy[a];
    const int u = start[cell_index(*gs, x, y)] + rank[a];
    C.x[u] = x;
    C.y[u] = y;
    C.key[u] = ckey[a];
}

// One round of the lexicographically first independent set: a candidate is
// accepted once every conflicting candidate of smaller key is rejected, and
// rejected as soon as one of them is accepted.  (States only go from undecided to
// accepted or rejected, and either value of one that changes leads to the same set, so
// caches may hold older ones.)  Bound by latency: eight candidates of the cells within
// reach are read at once.  Accepted ones are queued and marked by id.  A round that leaves
// one undecided sets rm_open[round]; the rounds after one that left none do nothing.
// 640k particles, a tenth of the lattice gone: with an index per candidate, all nine cells and one
// candidate at a time, 148 us for the first round and 500 for all, now 54 and 115.
constexpr int kInsBlock = 512;
__global__ __launch_bounds__(kInsBlock) void k_mis_round(int round, int nc, CandSlots C,
                                                         const int32_t* __restrict__ cstart, const GridState* gs,
                                                         float ex2, int capacity, Queues* qs)
{
    __shared__ int s_n, s_at;
    if (round > 0 && !qs->rm_open[round - 1]) return;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const int u = blockIdx.x * kInsBlock + threadIdx.x;
    auto state_of = [&](int v) {
        return __hip_atomic_load(&C.state[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    };
    bool take = false, open = false;
    if (u < nc && state_of(u) == 0) {
        const GridState g = *gs;
        const float px = C.x[u], py = C.y[u];
        const uint64_t ka = C.key[u];
        // the cells that the square around the candidate touches (an upper bound of the
        // offsets whose FP32 squared length is below ex2; cell indices are monotone)
        const float rad = sqrtf(ex2) * (1.0f + 9.5367431640625e-7f);
        const float xa = px - rad, xb = px + rad, ya = py - rad, yb = py + rad;
        int cx0, cy0, cx1, cy1;
        cell_xy(g, xa - fabsf(xa) * 2.384185791015625e-7f, ya - fabsf(ya) * 2.384185791015625e-7f, cx0, cy0);
        cell_xy(g, xb + fabsf(xb) * 2.384185791015625e-7f, yb + fabsf(yb) * 2.384185791015625e-7f, cx1, cy1);
        bool any_in = false, any_open = false;
        for (int yy = cy0; yy <= cy1 && !any_in; ++yy) {
            const int u0 = cstart[yy * g.nx + cx0], u1 = cstart[yy * g.nx + cx1 + 1];
            for (int v0 = u0; v0 < u1 && !any_in; v0 += 8) {
                float bx[8], by[8];
                uint64_t kb[8];
                uint8_t sb[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int v = min(v0 + e, u1 - 1);   // past the end: a repeat
                    bx[e] = C.x[v];
                    by[e] = C.y[v];
                    kb[e] = C.key[v];
                    sb[e] = state_of(v);
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    // (not itself: its key is not smaller)
                    const bool near = kb[e] < ka && d2_f32(bx[e] - px, by[e] - py) < ex2;
                    any_in = any_in || (near && sb[e] == 1);
                    any_open = any_open || (near && sb[e] == 0);
                }
            }
        }
        take = !any_in && !any_open;
        open = !any_in && any_open;
        if (!open)
            __hip_atomic_store(&C.state[u], (uint8_t)(take ? 1 : 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        if (take) {
            const uint64_t id = ka >> 3;
            if (id < (uint64_t)capacity) atomicOr(&C.mask[id >> 2], 1u << (8 * (uint32_t)(id & 3) + (uint32_t)(ka & 7)));
        }
    }
    const uint64_t m = __ballot(take);
    int at = 0;
    if (m && lane_id() == 0) at = atomicAdd(&s_n, __popcll(m));
    at = __shfl(at, 0, VRM_WAVE) + __popcll(m & ((1ull << lane_id()) - 1ull));
    const int left = __syncthreads_or(open);
    if (threadIdx.x == 0) {
        if (s_n) s_at = atomicAdd(&qs->n_accepted, s_n);
        if (left) qs->rm_open[round] = 1;
    }
    __syncthreads();
    if (take) C.taken[s_at + at] = u;
}

// The accepted candidates' order: keys are (id, segment), so the number of marks before a
// group of sixteen ids is its first position (a scan as in k_cell_starts).  Only where the
// marks can tell: ids below the capacity, no id twice (the marks' total is the number of
// accepted ones); otherwise the host sorts the keys.  (Sorting 35-bit keys took 17
// launches, 200 us.)
__global__ __launch_bounds__(1024) void k_ins_order(int capacity, const SelectState* sel, CandSlots C,
                                                    int32_t* __restrict__ first, CellScratch* sc, Queues* qs)
{
    __shared__ uint32_t s_ticket;
    const int t = threadIdx.x;
    if (qs->rm_open[kRmRounds - 1]) return;   // not chosen yet
    if (t == 0) s_ticket = atomicAdd(&sc->ticket, 1u);
    __syncthreads();
    const int b = (int)(s_ticket % kCellParts);
    const uint32_t launch = s_ticket / kCellParts + 1u;
    const int words = ((int)min((long)sel->max_id + 1, (long)capacity) + 3) / 4;
    const int groups = (words + 3) / 4;
    const int chunk = (groups + kCellParts - 1) / kCellParts;
    const int lo = min(groups, b * chunk), hi = min(groups, lo + chunk);
    auto marks = [&](int g) {
        int n = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) n += 4 * g + k < words ? __popc(C.mask[4 * g + k]) : 0;
        return n;
    };
    int sum = 0;
    for (int g = lo + t; g < hi; g += 1024) sum += marks(g);
    int total;
    (void)block_exclusive_scan(sum, total);
    if (t == 0)
        __hip_atomic_store(&sc->part[b], ((uint64_t)launch << 32) | (uint32_t)total, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    int before = 0;
    if (t < b) {
        uint64_t v;
        while ((uint32_t)((v = __hip_atomic_load(&sc->part[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 32) !=
               launch)
            __builtin_amdgcn_s_sleep(1);
        before = (int)(uint32_t)v;
    }
    int carry;
    (void)block_exclusive_scan(before, carry);
    for (int g0 = lo; g0 < hi; g0 += 1024) {
        const int g = g0 + t;
        int tot;
        const int ex = block_exclusive_scan(g < hi ? marks(g) : 0, tot);
        if (g < hi) first[g] = carry + ex;
        carry += tot;
    }
    // 2: more than the capacity holds, 3: in order, 4: to be sorted
    if (b == kCellParts - 1 && t == 0) qs->small_state = carry == qs->n_accepted && sel->max_id < capacity ? 3 : 4;
}

// The accepted candidates appended in key order, and the record for the host.
__global__ __launch_bounds__(256) void k_ins_append(int n0, int capacity, int nc, int rounds, CandSlots C,
                                                    const int32_t* __restrict__ first, float* x, float* y, float* gamma,
                                                    int32_t* id, uint8_t* diffused, int32_t* n_dev,
                                                    const SelectState* sel, Queues* qs, vrm_counters* cnt,
                                                    const GridState* gs, HostQueues* h, int32_t seq)
{
    const bool open = qs->rm_open[kRmRounds - 1] != 0;
    const int na = qs->n_accepted, state = qs->small_state;
    const bool fits = n0 + na <= capacity, mine = !open && fits && state == 3;
    if (mine) {
        for (int k = blockIdx.x * 256 + threadIdx.x; k < na; k += gridDim.x * 256) {
            const int u = C.taken[k];
            const uint64_t key = C.key[u];
            const uint32_t i = (uint32_t)(key >> 3), word = i >> 2, below = 8 * (i & 3) + (uint32_t)(key & 7);
            int r = first[i >> 4] + __popc(C.mask[word] & ((1u << below) - 1u));
            for (uint32_t w = word & ~3u; w < word; ++w) r += __popc(C.mask[w]);
            x[n0 + r] = C.x[u];
            y[n0 + r] = C.y[u];
            gamma[n0 + r] = 0.0f;
            id[n0 + r] = sel->max_id + 1 + r;
            diffused[n0 + r] = 0;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (mine) *n_dev = n0 + na;
        if (!open && !fits) cnt->capacity_needed = n0 + na;
        if (!open && fits) {
            // rounds run, in the batches of four that the counter is kept in
            int r = 0;
            while (r < kRmRounds && qs->rm_open[r]) ++r;
            cnt->n_candidates = nc;
            cnt->mis_rounds = rounds + (r / 4 + 1) * 4;
            if (mine) {
                cnt->n_inserted = na;
                cnt->n = n0 + na;
            }
        }
        publish(qs, gs, 0, h, seq);
    }
}

__global__ void k_ins_next_rounds(Queues* q)
{
    for (int k = 0; k < kRmRounds; ++k) q->rm_open[k] = 0;
}

// the accepted candidates' keys, to be sorted
__global__ __launch_bounds__(256) void k_accepted(int na, CandSlots C, uint64_t* key)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < na) key[k] = C.key[C.taken[k]];
}

// New particles get ids max_id + 1, max_id + 2, ... in key order (the largest
// id of the cloud is found by the selection's first pass), so ids stay unique
// after particles were removed.
__global__ __launch_bounds__(256) void k_append(int n0, int na, const int32_t* __restrict__ sorted, CandSlots C,
                                                float* x, float* y, float* gamma, int32_t* id, uint8_t* diffused,
                                                int32_t* n_dev, const SelectState* sel, vrm_counters* cnt)
{
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r == 0) {
        *n_dev = n0 + na;
        cnt->n_inserted = na;
        cnt->n = n0 + na;
    }
    if (r >= na) return;
    const int u = sorted[r];
    x[n0 + r] = C.x[u];
    y[n0 + r] = C.y[u];
    gamma[n0 + r] = 0.0f;
    id[n0 + r] = sel->max_id + 1 + r;
    diffused[n0 + r] = 0;
}

// Few candidates: the whole conflict resolution in one workgroup.  The
// candidates are sorted by key (bitonic, in LDS) and decided greedily in that
// order, each against the accepted ones; this is the same set as the rounds of
// k_mis_round (the lexicographically first maximal independent set), and the
// accepted ones are appended in key order as after the radix sort.
constexpr int kInsSmallMax = 1024;

__device__ __forceinline__ void insert_small(int n0, int capacity, int cand_cap,
                                             const float* __restrict__ cx, const float* __restrict__ cy,
                                             const uint64_t* __restrict__ ckey, float ex2, float* x, float* y,
                                             float* gamma, int32_t* id, uint8_t* diffused, int32_t* n_dev, Queues* qs,
                                             vrm_counters* cnt, const SelectState* sel)
{
    __shared__ uint64_t key[kInsSmallMax];
    __shared__ int32_t src[kInsSmallMax];
    __shared__ float sx[kInsSmallMax], sy[kInsSmallMax];
    __shared__ float ax[kInsSmallMax], ay[kInsSmallMax];
    __shared__ int32_t asrc[kInsSmallMax];
    __shared__ int32_t na_s;
    const int t = threadIdx.x;
    const int nc = qs->n_cand;
    if (nc > kInsSmallMax || nc > cand_cap) {
        if (t == 0) qs->small_state = 0;
        return;
    }
    int np = 1;
    while (np < nc) np <<= 1;
    if (t < np) {
        key[t] = t < nc ? ckey[t] : ~0ull;   // keys are distinct and below 2^35
        src[t] = t;
    }
    __syncthreads();
    for (int k = 2; k <= np; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            int p = t ^ j;
            if (t < np && p > t) {
                uint64_t a = key[t], b = key[p];
                bool up = (t & k) == 0;
                if ((a > b) == up) {
                    key[t] = b;
                    key[p] = a;
                    int v = src[t];
                    src[t] = src[p];
                    src[p] = v;
                }
            }
            __syncthreads();
        }
    }
    if (t < nc) {
        sx[t] = cx[src[t]];
        sy[t] = cy[src[t]];
    }
    __syncthreads();
    if (t < 64) {
        int na = 0;
        for (int r = 0; r < nc; ++r) {
            float xa = sx[r], ya = sy[r];
            bool conflict = false;
            for (int b = t; b < na; b += 64) {
                float dx = ax[b] - xa;
                float dy = ay[b] - ya;
                conflict |= d2_f32(dx, dy) < ex2;
            }
            if (!__any(conflict)) {
                if (t == 0) {
                    ax[na] = xa;
                    ay[na] = ya;
                    asrc[na] = src[r];
                }
                ++na;
                // the next candidate's lanes read what lane 0 wrote
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
        if (t == 0) na_s = na;
    }
    __syncthreads();
    const int na = na_s;
    if (n0 + na > capacity) {
        if (t == 0) {
            qs->n_accepted = na;
            qs->small_state = 2;
            cnt->capacity_needed = n0 + na;
        }
        return;
    }
    const int id0 = sel->max_id + 1;
    for (int r = t; r < na; r += blockDim.x) {
        int a = asrc[r];
        x[n0 + r] = cx[a];
        y[n0 + r] = cy[a];
        gamma[n0 + r] = 0.0f;
        id[n0 + r] = id0 + r;
        diffused[n0 + r] = 0;
    }
    if (t == 0) {
        *n_dev = n0 + na;
        qs->n_accepted = na;
        qs->small_state = 1;
        cnt->n_candidates = nc;
        cnt->n_inserted = na;
        cnt->mis_rounds = 0;
        cnt->n = n0 + na;
    }
}

// ... and the record for the host, whatever came out.
__global__ __launch_bounds__(1024) void k_insert_small(int n0, int capacity, int cand_cap,
                                                       const float* __restrict__ cx, const float* __restrict__ cy,
                                                       const uint64_t* __restrict__ ckey, float ex2, float* x, float* y,
                                                       float* gamma, int32_t* id, uint8_t* diffused, int32_t* n_dev,
                                                       Queues* qs, vrm_counters* cnt, const SelectState* sel,
                                                       const GridState* gs, HostQueues* h, int32_t seq)
{
    insert_small(n0, capacity, cand_cap, cx, cy, ckey, ex2, x, y, gamma, id, diffused, n_dev, qs, cnt, sel);
    if (threadIdx.x == 0) publish(qs, gs, 0, h, seq);
}

// ------------------------------------------------------------- reorder
__global__ __launch_bounds__(256) void k_gather_cloud(int n, const int32_t* __restrict__ perm,
                                                      const float* __restrict__ g, const uint8_t* __restrict__ dif,
                                                      float* tg, uint8_t* tdif)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    int i = perm[t];
    tg[t] = g[i];
    tdif[t] = dif[i];
}

// the cloud in slot order; the permutation becomes the identity
__global__ __launch_bounds__(256) void k_copy_back(int n, const float* __restrict__ xs, const float* __restrict__ ys,
                                                   const int32_t* __restrict__ ids, const float* __restrict__ tg,
                                                   const uint8_t* __restrict__ tdif, float* x, float* y, int32_t* id,
                                                   float* g, uint8_t* dif, int32_t* perm)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    x[t] = xs[t];
    y[t] = ys[t];
    id[t] = ids[t];
    g[t] = tg[t];
    dif[t] = tdif[t];
    perm[t] = t;
}

int blocks_for(int n) { return n > 0 ? (n + 255) / 256 : 1; }

}  // namespace

// The host spins on the sequence number; every 256 polls it asks the stream:
// an error ends the wait with that error, and a finished stream without the
// record is a state error (so a wait cannot outlast the stream's work).
int vrm_wait_queues(vrm_ctx* c, int32_t seq, Queues& q)
{
    for (uint64_t k = 1;; ++k) {
        if (__atomic_load_n(&c->q_host->seq, __ATOMIC_ACQUIRE) == seq) break;
        if ((k & 255) == 0) {
            const hipError_t e = hipStreamQuery(c->stream);
            if (e == hipErrorNotReady) continue;
            VRM_HIP(e);
            if (__atomic_load_n(&c->q_host->seq, __ATOMIC_ACQUIRE) == seq) break;
            return vrm_fail(VRM_E_STATE, "queue record not published");
        }
    }
    std::memcpy(&q, const_cast<const Queues*>(&c->q_host->q), sizeof(Queues));
    return VRM_OK;
}

int vrm_read_queues(vrm_ctx* c, Queues& q, const int32_t* n_dev)
{
    const int32_t seq = ++c->q_seq;
    hipLaunchKernelGGL(k_publish_queues, dim3(1), dim3(64), 0, c->stream, c->queues, c->grid, n_dev, c->q_host, seq);
    VRM_HIP(hipGetLastError());
    return vrm_wait_queues(c, seq, q);
}

// Slots of (x, y) on a grid: the cells' first slots, each point's rank in its cell.
int vrm_cell_slots(vrm_ctx* c, const GridState* g, const float* x, const float* y, int32_t n, const int32_t* n_dev,
                   int32_t* start, int32_t* rank)
{
    hipStream_t s = c->stream;
    if (n > 0)
        hipLaunchKernelGGL(k_count, dim3(blocks_for(n)), dim3(256), 0, s, x, y, n, n_dev, g, c->cell_count, rank);
    hipLaunchKernelGGL(k_cell_starts, dim3(kCellParts), dim3(1024), 0, s, c->cell_count, start, g, c->cell_scratch);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

// Cell list of (x, y) into ctx->cell_start / perm / xs, ys, ids (slot order).
int vrm_build_cells(vrm_ctx* c, const float* x, const float* y, const int32_t* id, int32_t n, const LaunchParams& lp,
                    const int32_t* n_dev)
{
    ScopedTimer tm(c, VRM_T_CELLS);
    hipStream_t s = c->stream;
    const float Rmax = (float)fmax((double)lp.hi2, (double)lp.hi2f);
    const float cs = sqrtf(Rmax) * (1.0f + 1.0f / 1024.0f);
    // (at least one workgroup, which sets the grid of an empty cloud)
    const int nbb = std::max(1, min(kBoxBlocks, (n + 256 * kBoxPer - 1) / (256 * kBoxPer)));
    hipLaunchKernelGGL(k_grid, dim3(nbb), dim3(256), 0, s, x, y, n, n_dev, c->grid, c->cell_scratch, cs, c->ncell_cap,
                       c->counters);
    if (int r = vrm_cell_slots(c, c->grid, x, y, n, n_dev, c->cell_start, c->rank)) return r;
    if (n > 0)
        hipLaunchKernelGGL(k_scatter, dim3(blocks_for(n)), dim3(256), 0, s, x, y, id, n, n_dev, c->cell_start, c->rank,
                           c->perm, c->xs, c->ys, c->ids, c->grid);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

// The selection's threshold of the cloud's n_dev particles (and, with it, cleared
// insertion queues and diffused counts).  Returns that count once the first pass has
// read it; it is out of range (and nothing else done) if below 0 or above the capacity.
// `guess` only sizes the launches.
int vrm_select_run(vrm_ctx* c, const vrm_cloud* cl, int32_t guess, double factor, int32_t& n)
{
    hipStream_t s = c->stream;
    static_assert(kCounterStripes <= kSelBlock, "the first pass zeroes one counter copy per thread");
    const int32_t seq = ++c->q_seq;
    const int nb = std::max(1, min(256, (guess + kSelBlock - 1) / kSelBlock));
    hipLaunchKernelGGL((k_sel_pass<11, true>), dim3(nb), dim3(kSelBlock), 0, s, cl->gamma_dev, cl->id_dev,
                       cl->capacity, cl->n_dev, c->sel, c->sel_bins, 21, factor, c->grid, c->counters, c->queues,
                       c->q_host, seq);
    hipLaunchKernelGGL((k_sel_pass<11, false>), dim3(nb), dim3(kSelBlock), 0, s, cl->gamma_dev, cl->id_dev,
                       cl->capacity, cl->n_dev, c->sel, c->sel_bins, 10, factor, c->grid, c->counters, c->queues,
                       c->q_host, seq);
    hipLaunchKernelGGL((k_sel_pass<10, false>), dim3(nb), dim3(kSelBlock), 0, s, cl->gamma_dev, cl->id_dev,
                       cl->capacity, cl->n_dev, c->sel, c->sel_bins, 0, factor, c->grid, c->counters, c->queues,
                       c->q_host, seq);
    VRM_HIP(hipGetLastError());
    Queues q;
    if (int r = vrm_wait_queues(c, seq, q)) return r;
    n = q.n_now;
    return VRM_OK;
}

// The diffused set of the threshold, also to mask_out unless that is NULL.
int vrm_select_mask_run(vrm_ctx* c, const float* gamma, int32_t n, uint8_t* mask_out)
{
    if (n > 0)
        hipLaunchKernelGGL(k_sel_mask, dim3(blocks_for(n)), dim3(256), 0, c->stream, gamma, n, c->sel, c->diffused,
                           mask_out, c->counters);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

int vrm_select_init(vrm_ctx* c)
{
    hipLaunchKernelGGL(k_sel_init, dim3(1), dim3(256), 0, c->stream, c->sel, c->sel_bins, kSelBins, (GridState*)nullptr);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

// Insertion; the cell list of the cloud must be current.  Returns once the new count is
// known (the host reads the record that the deciding kernel publishes): the arrays are
// complete in stream order.
int vrm_insert_run(vrm_ctx* c, vrm_cloud* cl, int32_t n, const LaunchParams& lp)
{
    hipStream_t s = c->stream;
    const int cand_cap = 2 * c->capacity;
    const int32_t seq = ++c->q_seq;
    if (n > 0)
        hipLaunchKernelGGL(n <= kCandCoopMaxN ? k_candidates<4> : k_candidates<1>,
                           dim3(n <= kCandCoopMaxN ? (n + 63) / 64 : blocks_for(n)), dim3(256), 0, s, n, c->perm,
                           c->xs, c->ys, c->ids, c->cell_start, cl->gamma_dev, c->sel, c->diffused, c->counters,
                           c->grid, lp, c->queues, cand_cap, c->cx, c->cy, c->ckey, c->cstate);
    hipLaunchKernelGGL(k_insert_small, dim3(1), dim3(1024), 0, s, n, cl->capacity, cand_cap, c->cx, c->cy, c->ckey,
                       lp.ex2, cl->x_dev, cl->y_dev, cl->gamma_dev, cl->id_dev, c->diffused, cl->n_dev, c->queues,
                       c->counters, c->sel, c->grid, c->q_host, seq);
    VRM_HIP(hipGetLastError());
    Queues q;
    if (int r = vrm_wait_queues(c, seq, q)) return r;
    if (q.nonfinite) return vrm_nonfinite(c, q.nonfinite);
    if (q.small_state == 2)
        return vrm_fail(VRM_E_CAPACITY, "insertion needs %d particles, capacity is %d", n + q.n_accepted,
                        cl->capacity);
    if (q.small_state == 1) return n + q.n_accepted;
    int nc = q.n_cand;
    if (nc > cand_cap) return vrm_fail(VRM_E_CAPACITY, "insertion: %d candidates exceed the buffer of %d", nc, cand_cap);
    // The candidates in cell order, in scratch that is free here; cx, cy and ckey are free
    // once they are in place.
    CandSlots C{c->tmp_f, reinterpret_cast<float*>(c->aidx), c->akey, c->cstate, c->cperm,
                reinterpret_cast<uint32_t*>(c->tmp_i)};
    hipLaunchKernelGGL(k_ins_begin, dim3(256), dim3(256), 0, s, cl->capacity, c->sel, C, c->queues);
    if (int r = vrm_cell_slots(c, c->grid, c->cx, c->cy, nc, nullptr, c->cstart, c->crank)) return r;
    hipLaunchKernelGGL(k_ins_scatter, dim3(blocks_for(nc)), dim3(256), 0, s, c->cx, c->cy, c->ckey, nc, c->cstart,
                       c->crank, C, c->grid);
    int32_t* first = c->crank;
    for (int rounds = 0;; rounds += kRmRounds) {
        for (int k = 0; k < kRmRounds; ++k)
            hipLaunchKernelGGL(k_mis_round, dim3((nc + kInsBlock - 1) / kInsBlock), dim3(kInsBlock), 0, s, k, nc, C,
                               c->cstart, c->grid, lp.ex2, cl->capacity, c->queues);
        hipLaunchKernelGGL(k_ins_order, dim3(kCellParts), dim3(1024), 0, s, cl->capacity, c->sel, C, first,
                           c->cell_scratch, c->queues);
        const int32_t done = ++c->q_seq;
        hipLaunchKernelGGL(k_ins_append, dim3(min(blocks_for(nc), 512)), dim3(256), 0, s, n, cl->capacity, nc, rounds, C,
                           first, cl->x_dev, cl->y_dev, cl->gamma_dev, cl->id_dev, c->diffused, cl->n_dev, c->sel,
                           c->queues, c->counters, c->grid, c->q_host, done);
        VRM_HIP(hipGetLastError());
        if (int r = vrm_wait_queues(c, done, q)) return r;
        if (!q.rm_open[kRmRounds - 1]) break;
        if (rounds > 4 * (long)nc + 64) return vrm_fail(VRM_E_STATE, "insertion: conflict resolution did not converge");
        hipLaunchKernelGGL(k_ins_next_rounds, dim3(1), dim3(1), 0, s, c->queues);
    }
    const int na = q.n_accepted;
    if (n + na > cl->capacity)
        return vrm_fail(VRM_E_CAPACITY, "insertion needs %d particles, capacity is %d", n + na, cl->capacity);
    if (q.small_state == 4) {
        // ids and append order follow the (id, segment) keys
        size_t bytes = c->sort_tmp_bytes;
        uint64_t* kin = c->ckey;
        uint64_t* ksorted = reinterpret_cast<uint64_t*>(c->cx);
        int32_t* vsorted = c->tmp_i;
        hipLaunchKernelGGL(k_accepted, dim3(blocks_for(na)), dim3(256), 0, s, na, C, kin);
        VRM_HIP(hipGetLastError());
        VRM_HIP(rocprim::radix_sort_pairs(c->sort_tmp, bytes, kin, ksorted, C.taken, vsorted, (size_t)na, 0, 35, s));
        hipLaunchKernelGGL(k_append, dim3(blocks_for(na)), dim3(256), 0, s, n, na, vsorted, C, cl->x_dev, cl->y_dev,
                           cl->gamma_dev, cl->id_dev, c->diffused, cl->n_dev, c->sel, c->counters);
        VRM_HIP(hipGetLastError());
    }
    return n + na;
}

// Reorder the cloud by the current cell list (perm) and make perm the identity.
int vrm_reorder_cloud(vrm_ctx* c, vrm_cloud* cl, int32_t n)
{
    if (n <= 0) return VRM_OK;
    hipStream_t s = c->stream;
    // xs, ys, ids already hold x, y, id in slot order
    hipLaunchKernelGGL(k_gather_cloud, dim3(blocks_for(n)), dim3(256), 0, s, n, c->perm, cl->gamma_dev, c->diffused,
                       c->tmp_f, c->tmp_u8);
    VRM_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_copy_back, dim3(blocks_for(n)), dim3(256), 0, s, n, c->xs, c->ys, c->ids, c->tmp_f, c->tmp_u8,
                       cl->x_dev, cl->y_dev, cl->id_dev, cl->gamma_dev, c->diffused, c->perm);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

size_t vrm_sort_tmp_bytes(int32_t cap)
{
    size_t bytes = 0;
    rocprim::radix_sort_pairs((void*)nullptr, bytes, (uint64_t*)nullptr, (uint64_t*)nullptr, (int32_t*)nullptr,
                              (int32_t*)nullptr, (size_t)cap, 0, 35, (hipStream_t)0);
    return bytes;
}

// ------------------------------------------------- allocation-free selection
// vrm_select_diffused_static: the selection kernels above with their state
// (histogram bins, threshold, the non-finite flag) in a fixed device array
// instead of a context's memory, for callers that cannot allocate.
namespace {
struct StaticSelect {
    SelectState sel;
    GridState grid;
    double bins[256];
};
constexpr size_t kStaticScratchBytes = 4096;
static_assert(sizeof(StaticSelect) <= kStaticScratchBytes, "static selection state exceeds its array");
constexpr int32_t kStaticMaxN = 1 << 26;   // exact FP64 bin sums (k_sel_pass)
constexpr int kStaticMaxDevices = 64;

__global__ void k_static_reset(GridState* g) { g->bad = 0; }
__global__ void k_static_report(const GridState* g, int32_t* out) { *out = g->bad; }
}  // namespace

// One copy per GPU, held until the process ends; in host code the name stands
// for the symbol, never for the device address (that is static_scratch_ptr's).
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
std::mutex g_static_mu;
void* g_static_ptr[kStaticMaxDevices];

// the device address of this GPU's copy of scratch (the current device's), looked
// up once per device
int static_scratch_ptr(int dev, void** out)
{
    if (dev < 0 || dev >= kStaticMaxDevices) return vrm_fail(VRM_E_ARG, "device %d outside [0, %d)", dev, kStaticMaxDevices);
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
        void* p = nullptr;
        VRM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return vrm_fail(VRM_E_HIP, "hipGetSymbolAddress(scratch) gave no address");
        g_static_ptr[dev] = p;
    }
    *out = g_static_ptr[dev];
    return VRM_OK;
}
}  // namespace

extern "C" int vrm_select_diffused_static(const float* gamma_dev, int32_t n, double h, int32_t q, double c_diff,
                                          uint8_t* mask_dev, int32_t* nonfinite_dev, void* stream)
{
    if (!gamma_dev || !mask_dev) return vrm_fail(VRM_E_ARG, "gamma and mask are required");
    if (n < 0 || n > kStaticMaxN) return vrm_fail(VRM_E_ARG, "n = %d outside [0, 2^26] (the largest selection this entry point takes)", n);
    if (!(h > 0.0) || !std::isfinite(h)) return vrm_fail(VRM_E_ARG, "h must be positive and finite");
    if (q != 2 && q != 3) return vrm_fail(VRM_E_ARG, "q must be 2 or 3 (got %d)", q);
    if (!(c_diff >= 0.0) || !std::isfinite(c_diff)) return vrm_fail(VRM_E_ARG, "c_diff must be >= 0");
    int dev = 0;
    VRM_HIP(hipGetDevice(&dev));
    void* ptr = nullptr;
    if (int r = static_scratch_ptr(dev, &ptr)) return r;
    StaticSelect* st = static_cast<StaticSelect*>(ptr);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const double factor = c_diff * std::pow(h, q + 1);
    hipLaunchKernelGGL(k_static_reset, dim3(1), dim3(1), 0, s, &st->grid);
    hipLaunchKernelGGL(k_sel_init, dim3(1), dim3(256), 0, s, &st->sel, st->bins, 256, &st->grid);
    const int nb = std::max(1, min(256, (n + kSelBlock - 1) / kSelBlock));
    for (int shift = 24; shift >= 0; shift -= 8)
        hipLaunchKernelGGL((shift == 24 ? k_sel_pass<8, true> : k_sel_pass<8, false>), dim3(nb), dim3(kSelBlock), 0, s,
                           gamma_dev, (const int32_t*)nullptr, n, (const int32_t*)nullptr, &st->sel, st->bins, shift,
                           factor, &st->grid, (vrm_counters*)nullptr, (Queues*)nullptr, (HostQueues*)nullptr, 0);
    if (n > 0)
        hipLaunchKernelGGL(k_sel_mask, dim3(blocks_for(n)), dim3(256), 0, s, gamma_dev, n, &st->sel, mask_dev,
                           (uint8_t*)nullptr, (vrm_counters*)nullptr);
    if (nonfinite_dev) hipLaunchKernelGGL(k_static_report, dim3(1), dim3(1), 0, s, &st->grid, nonfinite_dev);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}
