// Velocity that the particles induce on themselves: direct sum, and by boxes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "vrm_device.h"
#include "vrm_lp_common.h"

using namespace vrm;

namespace {

// One pair: t (1 - e) with the offset and |D|^2 scaled (below).
__device__ __forceinline__ void pair(float dx, float dy, float g, float& u, float& v)
{
    const float r2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, 1e-30f));
    const float ex = __builtin_amdgcn_exp2f(-r2);
    const float t = __builtin_amdgcn_rcpf(r2) * g;
    const float f = __builtin_fmaf(-t, ex, t);
    u = __builtin_fmaf(-dy, f, u);
    v = __builtin_fmaf(dx, f, v);
}

// Particles that a box may hold.  A fuller one leaves the cloud to the direct sum: it has no
// expansion (one wave forms a box's, and would be the launch's time).
constexpr int kBoxMost = 4096;

// Whether the boxes do the sum: every box has its expansion, and their instruction slots (16
// per pair, about 48 per target and far box) are clearly below those of all pairs.  A cloud of
// a few boxes (eps of its size), or with most particles in a few boxes (an outlier stretches
// the grid), is summed directly.
__device__ __forceinline__ bool by_boxes(const BoxState& st)
{
    return (st.fullest >> 32) <= (unsigned long long)kBoxMost && (double)st.work < 0.7 * (double)st.all_pairs;
}

// ------------------------------------------------------------ Biot-Savart (direct sum)
// u(x_i) = sum_j Gamma_j K_eps(x_i - x_j) with K_eps(d) = (-d_y, d_x) (1 - exp(-|d|^2 / eps^2))
// / (2 pi |d|^2) and K_eps(0) = 0 (Sec. 3.4 eq. nsode, the regularised kernel of Sec. 5).
// Each thread accumulates kBsT targets; a workgroup streams one chunk of the
// sources (blockIdx.y) through LDS in tiles of kBsTile, and the chunks' partial
// sums meet in u, v by atomics (distinct addresses: no contention).
// Positions are scaled by s = sqrt(log2 e) / eps, so that with D = s d the
// exponential is exp2(-|D|^2) and the pair term is s Gamma_j (-D_y, D_x)
// (1 - 2^-|D|^2) / (2 pi |D|^2): per pair two differences, two FMAs for |D|^2,
// exp2, a reciprocal, one product, one FMA for t - t e and two accumulating
// FMAs; s multiplies the sums once.  The 1e-30 added to |D|^2 makes the self
// term 0 * finite instead of a branch.
constexpr int kBsBlock = 256;
constexpr int kBsT = 2;
constexpr int kBsTile = 512;

__global__ __launch_bounds__(kBsBlock) void k_biot_savart(const int32_t* __restrict__ n_dev,
                                                          const float* __restrict__ x, const float* __restrict__ y,
                                                          const float* __restrict__ g, float sc, int chunk,
                                                          float* u, float* v, const BoxState* st,
                                                          const int32_t* __restrict__ start,
                                                          const float4* __restrict__ src)
{
    __shared__ float4 s_src[kBsTile];
    // offsets from the origin, or from a particle where most are (their rounding is then
    // that of the cloud's size, wherever it is)
    float xo = 0.0f, yo = 0.0f;
    if (st) {
        if (by_boxes(*st)) return;
        const float4 q = src[start[(uint32_t)st->fullest]];
        if (fabsf(q.x) <= 1e30f && fabsf(q.y) <= 1e30f) {
            xo = q.x;
            yo = q.y;
        }
    }
    const int n = *n_dev;
    const int tid = threadIdx.x;
    float xt[kBsT], yt[kBsT], su[kBsT], sv[kBsT];
#pragma unroll
    for (int k = 0; k < kBsT; ++k) {
        const int a = blockIdx.x * (kBsBlock * kBsT) + k * kBsBlock + tid;
        xt[k] = a < n ? (x[a] - xo) * sc : 0.0f;
        yt[k] = a < n ? (y[a] - yo) * sc : 0.0f;
        su[k] = 0.0f;
        sv[k] = 0.0f;
    }
    const float inv2pi = 0.15915494309189535f;
    const int j0 = blockIdx.y * chunk, j1 = min(j0 + chunk, n);
    for (int base = j0; base < j1; base += kBsTile) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kBsTile / kBsBlock; ++q) {
            const int e = q * kBsBlock + tid, j = base + e;
            s_src[e] = j < j1 ? make_float4((x[j] - xo) * sc, (y[j] - yo) * sc, g[j] * inv2pi, 0.0f)
                              : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        __syncthreads();
#pragma unroll 4
        for (int e = 0; e < kBsTile; ++e) {
            const float4 s = s_src[e];
#pragma unroll
            for (int k = 0; k < kBsT; ++k) {
                const float dx = xt[k] - s.x, dy = yt[k] - s.y;
                pair(dx, dy, s.z, su[k], sv[k]);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kBsT; ++k) {
        const int a = blockIdx.x * (kBsBlock * kBsT) + k * kBsBlock + tid;
        if (a < n) {
            atomicAdd(&u[a], su[k] * sc);
            atomicAdd(&v[a], sv[k] * sc);
        }
    }
}

__global__ void k_zero_uv(const int32_t* __restrict__ n_dev, float* u, float* v)
{
    const int n = *n_dev;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        u[i] = 0.0f;
        v[i] = 0.0f;
    }
}

// ------------------------------------------------------------ Biot-Savart (boxes)
// The same sum with the particles binned into square boxes.  A target adds the sources of
// the 5 x 5 boxes around its own pair by pair, as above, and every other box by its
// multipole expansion: with z = x + i y, c the box's centre, s its side and
// w = s / (z - c), the sources' u - i v is (-i / (2 pi s)) sum_k a_k w^(k + 1), where
// a_k = sum_j Gamma_j ((z_j - c) / s)^k (the expansion of 1 / (z - z_j)).
// For a box d boxes away |z_j - c| <= s / sqrt(2) and |z - c| >= (d - 1/2) s, so term k falls
// as (0.707 / (d - 1/2))^k: 14 terms leave 2e-8 of a box's part at d = 3, 10 leave 9e-9 from
// d = 5 and 8 leave 6e-9 from d = 8.  The regularisation is left out for these boxes:
// s >= 2.1 eps puts them 4.2 eps away, where exp(-d^2 / eps^2) is below 2^-25.  (Both are
// below the rounding of the FP32 sums.)  Offsets of near sources are taken from a particle
// of the work item before they are scaled, so they are as exact as the positions allow.
// Instruction slots per target: 16 N directly; here 16 * 25 N / M + 48 M with M boxes (the
// two meet near M = sqrt(8 N)).  Bound by VALU issue; a work item is half the sources of
// 128 targets so that the CUs' loads are even (one item for all sources: 110 us, a
// third of the CUs with twice the others' work).  A cloud with a non-finite or huge value
// gets one box, and with it the direct sum.
// 40k particles: 549 us directly, now 123; error against 64 bits 2.8e-7, now 8e-8.
// 120k: 4360 us, now 382.
constexpr int kTerms = 14;
constexpr int kNear = 2;            // boxes on each side that are summed pair by pair
constexpr int kBoxT = 128;          // targets of a work item, two per lane
constexpr int kBoxFill = 109;       // mean particles of a box, or a multiple: a work item nearly full
constexpr int kBoxWaves = 4;
constexpr int kBoxParts = 2;        // work items that share the sources of the same targets
// below: the direct sum (12000 particles: 70 us directly; 14000: 90 directly, 67 by boxes; 20000: 151, 73)
constexpr int kBoxMinN = 14000;

// A box's part at the offset (dx, dy) from its centre, in units of its side: with
// w = 1 / (dx + i dy), S = sum_k a_k w^(k + 1), and u - i v = -i S, so u = Im S, v = Re S.
template <int TERMS>
__device__ __forceinline__ void far_box(float dx, float dy, const float* __restrict__ a, float& u, float& v)
{
    const float r = __builtin_amdgcn_rcpf(__builtin_fmaf(dx, dx, dy * dy));
    const float wr = dx * r, wi = -dy * r;
    float sr = a[2 * TERMS - 2], si = a[2 * TERMS - 1];
#pragma unroll
    for (int k = TERMS - 2; k >= 0; --k) {
        const float t = __builtin_fmaf(-si, wi, __builtin_fmaf(sr, wr, a[2 * k]));
        si = __builtin_fmaf(si, wr, __builtin_fmaf(sr, wi, a[2 * k + 1]));
        sr = t;
    }
    v += __builtin_fmaf(-si, wi, sr * wr);
    u += __builtin_fmaf(si, wr, sr * wi);
}

// The boxes' grid, by the last workgroup.
__global__ __launch_bounds__(256) void k_bs_grid(const float* __restrict__ x, const float* __restrict__ y,
                                                 const float* __restrict__ gamma, int n,
                                                 const int32_t* __restrict__ n_dev, BoxState* st, float eps, int max_boxes)
{
    n = min(n, *n_dev);
    uint32_t mnx = 0xffffffffu, mny = 0xffffffffu, mxx = 0u, mxy = 0u;
    bool bad = false;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const float xv = x[i], yv = y[i];
        bad = bad || !(fabsf(xv) <= 1e30f) || !(fabsf(yv) <= 1e30f) || !(fabsf(gamma[i]) <= 1e30f);
        const uint32_t kx = ordered_key(xv), ky = ordered_key(yv);
        mnx = min(mnx, kx);
        mny = min(mny, ky);
        mxx = max(mxx, kx);
        mxy = max(mxy, ky);
    }
    __shared__ uint32_t red[4][4];
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
        old = atomicExch(&st->box[threadIdx.x][blockIdx.x],
                         threadIdx.x == 0 ? mnx : threadIdx.x == 1 ? mny : threadIdx.x == 2 ? mxx : mxy);
    if (__any(bad) && lane_id() == 0) old |= (uint32_t)atomicOr(&st->bad_seen, 1);
    asm volatile("" ::"v"(old));   // waits for the atomics' results
    if (!last_here(st->done)) return;
    for (int k = threadIdx.x; k < (int)gridDim.x; k += 256) {
        mnx = min(mnx, __hip_atomic_load(&st->box[0][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        mny = min(mny, __hip_atomic_load(&st->box[1][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        mxx = max(mxx, __hip_atomic_load(&st->box[2][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        mxy = max(mxy, __hip_atomic_load(&st->box[3][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    reduce();
    if (threadIdx.x != 0) return;
    const int32_t bad_seen = __hip_atomic_load(&st->bad_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    st->bad_seen = 0;
    st->items = 0;
    st->work = 0;
    st->fullest = 0;
    st->all_pairs = (unsigned long long)max(n, 0) * (unsigned long long)max(n, 0);
    GridState g{};
    g.x0 = g.y0 = 0.0f;
    g.cs = g.inv_cs = 1.0f;
    g.nx = g.ny = 1;
    if (!bad_seen && n > 0) {
        const float xmin = ordered_key_inv(mnx), ymin = ordered_key_inv(mny);
        const double lx = (double)ordered_key_inv(mxx) - xmin, ly = (double)ordered_key_inv(mxy) - ymin;
        // boxes wanted: particles over the fill, a multiple of it where N is large
        const double fill = kBoxFill * fmax(1.0, floor(sqrt(n / 8.0) / kBoxFill + 0.5));
        double s = fmax(sqrt(lx * ly * fill / n), fmax(lx, ly) * fill / n);
        s = fmax(s, 2.1 * (double)eps);
        // a box holds its sources only if no index is clamped: a larger side, not fewer boxes
        long nx = 0, ny = 0;
        bool found = false;
        for (int k = 0; k < 400 && s > 0.0 && !found; ++k) {
            nx = (long)fmin(lx / s, 1e9) + 1;
            ny = (long)fmin(ly / s, 1e9) + 1;
            found = nx * ny <= max_boxes;
            if (!found) s *= 1.25;
        }
        if (found && s <= 1e30 && s >= 1e-30) {
            g.x0 = xmin;
            g.y0 = ymin;
            g.cs = (float)s;
            g.inv_cs = 1.0f / g.cs;
            g.nx = (int)nx;
            g.ny = (int)ny;
        }
    }
    g.ncells = g.nx * g.ny;
    st->g = g;
}

// The sources in box order: position, Gamma / 2 pi, and the particle's index; and the
// sums cleared.
__global__ __launch_bounds__(256) void k_bs_scatter(const float* __restrict__ x, const float* __restrict__ y,
                                                    const float* __restrict__ gamma, int n,
                                                    const int32_t* __restrict__ n_dev,
                                                    const int32_t* __restrict__ start, const int32_t* __restrict__ rank,
                                                    float4* __restrict__ src, const BoxState* st, float* u, float* v)
{
    n = min(n, *n_dev);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    u[i] = 0.0f;
    v[i] = 0.0f;
    const float xi = x[i], yi = y[i];
    int bx, by;
    cell_of_pos(st->g, xi, yi, bx, by);
    src[start[by * st->g.nx + bx] + rank[i]] =
        make_float4(xi, yi, gamma[i] * 0.15915494309189535f, __int_as_float(i));
}

__device__ __forceinline__ float2 box_centre(const GridState& g, int bx, int by)
{
    return make_float2(__builtin_fmaf((float)bx + 0.5f, g.cs, g.x0), __builtin_fmaf((float)by + 0.5f, g.cs, g.y0));
}

// A wave per box: its expansion (unless it holds more than kBoxMost particles: then the
// direct sum does the cloud), its work items to the list, and its share of the work.  The
// shares sum to at most N (N + 3 boxes), below 2^53 for the largest cloud.
constexpr int kMpWaves = 8;
__global__ __launch_bounds__(64 * kMpWaves) void k_bs_multipoles(const int32_t* __restrict__ start,
                                                                 const float4* __restrict__ src,
                                                                 float* __restrict__ coef, int2* __restrict__ items,
                                                                 BoxState* st)
{
    __shared__ int s_want[kMpWaves], s_at;
    __shared__ unsigned long long s_work[kMpWaves], s_full[kMpWaves];
    const GridState g = st->g;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = lane_id();
    const int box = blockIdx.x * kMpWaves + w, bx = box % g.nx, by = box / g.nx;
    int j0 = 0, j1 = 0, near = 0, boxes = 0;
    if (box < g.ncells) {
        j0 = start[box];
        j1 = start[box + 1];
        const int xa = max(bx - kNear, 0), xb = min(bx + kNear, g.nx - 1);
#pragma unroll
        for (int o = -kNear; o <= kNear; ++o) {
            const int yy = min(max(by + o, 0), g.ny - 1);
            const int len = start[yy * g.nx + xb + 1] - start[yy * g.nx + xa];
            near += yy == by + o ? len : 0;
            boxes += yy == by + o ? xb - xa + 1 : 0;
        }
    }
    const bool most = j1 - j0 > kBoxMost;
    const int want = kBoxParts * ((j1 - j0 + kBoxT - 1) / kBoxT);
    if (lane == 0) {
        s_want[w] = want;
        s_full[w] = ((unsigned long long)(j1 - j0) << 32) | (unsigned)box;
        // pairs, a far box being worth three
        s_work[w] = (unsigned long long)(j1 - j0) * (unsigned long long)(near + 3 * (g.ncells - boxes));
    }
    __syncthreads();
    int before = 0, total = 0;
    for (int k = 0; k < kMpWaves; ++k) {
        before += k < w ? s_want[k] : 0;
        total += s_want[k];
    }
    if (threadIdx.x == 0 && total) {
        s_at = atomicAdd(&st->items, total);
        unsigned long long work = 0;
        for (int k = 0; k < kMpWaves; ++k) {
            work += s_work[k];
            s_full[0] = max(s_full[0], s_full[k]);
        }
        atomicAdd(&st->work, work);
        atomicMax(&st->fullest, s_full[0]);
    }
    __syncthreads();
    for (int k = lane; k < want; k += 64) items[s_at + before + k] = make_int2(box, k);
    if (most) return;
    if (box >= g.ncells) return;
    const float2 c = box_centre(g, bx, by);
    // real parts in the first sixteen places, imaginary in the others (two of each unused)
    float a[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) a[k] = 0.0f;
    for (int j = j0 + lane; j < j1; j += 64) {
        const float4 q = src[j];
        const float zx = (q.x - c.x) * g.inv_cs, zy = (q.y - c.y) * g.inv_cs;
        float pr = q.z, pi = 0.0f;
#pragma unroll
        for (int k = 0; k < kTerms; ++k) {
            a[k] += pr;
            a[16 + k] += pi;
            const float t = pr * zx - pi * zy;
            pi = pr * zy + pi * zx;
            pr = t;
        }
    }
    // sums over the wave: at every step a lane gives half of its places away, so lane l
    // ends with place l / 2 (31 exchanges and one instead of six of each place)
    auto halve = [&](auto h) {
        constexpr int half = decltype(h)::value, o = 2 * half;
        const bool upper = (lane & o) != 0;
#pragma unroll
        for (int k = 0; k < half; ++k) {
            const float keep = upper ? a[k + half] : a[k], give = upper ? a[k] : a[k + half];
            a[k] = keep + __shfl_xor(give, o, VRM_WAVE);
        }
    };
    halve(std::integral_constant<int, 16>{});
    halve(std::integral_constant<int, 8>{});
    halve(std::integral_constant<int, 4>{});
    halve(std::integral_constant<int, 2>{});
    halve(std::integral_constant<int, 1>{});
    a[0] += __shfl_xor(a[0], 1, VRM_WAVE);
    const int place = lane >> 1, k = place & 15;
    if ((lane & 1) == 0 && k < kTerms) coef[(size_t)box * (2 * kTerms) + 2 * k + (place >> 4)] = a[0];
}

// A work item is up to 128 targets of one box, two per lane, by a workgroup whose waves
// share the sources and the far boxes and meet in LDS.
__global__ __launch_bounds__(64 * kBoxWaves) void k_bs_boxes(const int32_t* __restrict__ start,
                                                             const float4* __restrict__ src,
                                                             const float* __restrict__ coef,
                                                             const int2* __restrict__ items,
                                                             const BoxState* __restrict__ st, float sc, float* u, float* v)
{
    __shared__ float4 s_src[kBoxWaves][64];
    __shared__ float s_sum[kBoxWaves][4][64];
    if (!by_boxes(*st)) return;
    const GridState g = st->g;
    const int nitems = st->items;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const int2 item = items[it];
        const int box = __builtin_amdgcn_readfirstlane(item.x), bx = box % g.nx, by = box / g.nx;
        const float2 c = box_centre(g, bx, by);
        const int tile = __builtin_amdgcn_readfirstlane(item.y) / kBoxParts;
        const int part = __builtin_amdgcn_readfirstlane(item.y) % kBoxParts;
        const int t0 = start[box] + tile * kBoxT, t1 = start[box + 1];
        const float4 ref = src[t0];
        float xt[2], yt[2], xn[2], yn[2], su[2] = {0.0f, 0.0f}, sv[2] = {0.0f, 0.0f};
        int index[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int t = t0 + 64 * k + lane;
            const float4 q = src[min(t, t1 - 1)];
            // offsets from the box's centre (for the boxes), from the first target (for pairs)
            xt[k] = q.x - c.x;
            yt[k] = q.y - c.y;
            xn[k] = (q.x - ref.x) * sc;
            yn[k] = (q.y - ref.y) * sc;
            index[k] = t < t1 ? __float_as_int(q.w) : -1;
        }
        // the boxes around, pair by pair: their sources are one run per row of boxes
        int base[2 * kNear + 1], end[2 * kNear + 1], total = 0;
#pragma unroll
        for (int o = 0; o <= 2 * kNear; ++o) {
            const int yy = by + o - kNear;
            int u0 = 0, len = 0;
            if (yy >= 0 && yy < g.ny) {
                u0 = start[yy * g.nx + max(bx - kNear, 0)];
                len = start[yy * g.nx + min(bx + kNear, g.nx - 1) + 1] - u0;
            }
            base[o] = u0 - total;
            total += len;
            end[o] = total;
        }
        constexpr int kStep = 64 * kBoxWaves * kBoxParts;
        for (int e0 = 64 * (part * kBoxWaves + w); e0 < total; e0 += kStep) {
            const int e = min(e0 + lane, total - 1);
            int j = base[2 * kNear];
#pragma unroll
            for (int o = 2 * kNear - 1; o >= 0; --o) j = e < end[o] ? base[o] : j;
            float4 q = src[j + e];
            if (e0 + lane >= total) q.z = 0.0f;   // past the end: nothing
            q.x = (q.x - ref.x) * sc;
            q.y = (q.y - ref.y) * sc;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            s_src[w][lane] = q;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll 4
            for (int k = 0; k < 64; ++k) {
                const float4 s = s_src[w][k];
                pair(xn[0] - s.x, yn[0] - s.y, s.z, su[0], sv[0]);
                pair(xn[1] - s.x, yn[1] - s.y, s.z, su[1], sv[1]);
            }
        }
        // the pair terms carry the scale of the offsets
        su[0] *= sc;
        su[1] *= sc;
        sv[0] *= sc;
        sv[1] *= sc;
        // every other box by its expansion, in units of its side
        float fu[2] = {0.0f, 0.0f}, fv[2] = {0.0f, 0.0f};
        const float xb0 = xt[0] * g.inv_cs, yb0 = yt[0] * g.inv_cs, xb1 = xt[1] * g.inv_cs, yb1 = yt[1] * g.inv_cs;
        auto far = [&](auto terms, int m, int dx, int dy) {
            const float* __restrict__ a = coef + (size_t)m * (2 * kTerms);
            far_box<decltype(terms)::value>(xb0 + (float)dx, yb0 + (float)dy, a, fu[0], fv[0]);
            far_box<decltype(terms)::value>(xb1 + (float)dx, yb1 + (float)dy, a, fu[1], fv[1]);
        };
        int mx = part * kBoxWaves + w, my = 0;
        for (int m = mx; m < g.ncells; m += kBoxWaves * kBoxParts, mx += kBoxWaves * kBoxParts) {
            while (mx >= g.nx) {
                mx -= g.nx;
                ++my;
            }
            const int dx = bx - mx, dy = by - my, d = max(abs(dx), abs(dy));
            if (d <= kNear) continue;
            if (d >= 8)
                far(std::integral_constant<int, 8>{}, m, dx, dy);
            else if (d >= 5)
                far(std::integral_constant<int, 10>{}, m, dx, dy);
            else
                far(std::integral_constant<int, kTerms>{}, m, dx, dy);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            s_sum[w][2 * k][lane] = __builtin_fmaf(fu[k], g.inv_cs, su[k]);
            s_sum[w][2 * k + 1][lane] = __builtin_fmaf(fv[k], g.inv_cs, sv[k]);
        }
        __syncthreads();
        if (w < 2) {
            float a = 0.0f, b = 0.0f;
#pragma unroll
            for (int k = 0; k < kBoxWaves; ++k) {
                a += s_sum[k][2 * w][lane];
                b += s_sum[k][2 * w + 1][lane];
            }
            const int i = w == 0 ? index[0] : index[1];
            if (i >= 0) {
                // (onto zero, by two items: the same sum in either order)
                static_assert(kBoxParts == 2, "sums that do not depend on their order");
                atomicAdd(&u[i], a);
                atomicAdd(&v[i], b);
            }
        }
        __syncthreads();
    }
}

int blocks_for(int n) { return n > 0 ? (n + 255) / 256 : 1; }

}  // namespace

int vrm_biot_savart_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, double eps, float* u, float* v)
{
    if (n <= 0) return VRM_OK;
    hipStream_t s = c->stream;
    const float sc = (float)(sqrt(1.4426950408889634) / eps);
    const bool boxes = n >= kBoxMinN;
    BoxState* st = c->bs_state;
    if (boxes) {
        // in scratch that only insertions and removals use
        float4* src = reinterpret_cast<float4*>(c->akey);
        int2* items = reinterpret_cast<int2*>(c->ckey);
        float* coef = c->tmp_f;
        // twice the boxes wanted (an oblong cloud's edges), and expansions that fit
        const int most = std::min(3 * (n / (2 * kTerms)), 2 * (n / kBoxFill) + 64);
        const int nb = std::max(1, std::min(kBoxBlocks, (n + 1023) / 1024));
        hipLaunchKernelGGL(k_bs_grid, dim3(nb), dim3(256), 0, s, cl->x_dev, cl->y_dev, cl->gamma_dev, n, cl->n_dev, st,
                           (float)eps, most);
        if (int r = vrm_cell_slots(c, &st->g, cl->x_dev, cl->y_dev, n, cl->n_dev, c->cstart, c->crank)) return r;
        hipLaunchKernelGGL(k_bs_scatter, dim3(blocks_for(n)), dim3(256), 0, s, cl->x_dev, cl->y_dev, cl->gamma_dev, n,
                           cl->n_dev, c->cstart, c->crank, src, st, u, v);
        hipLaunchKernelGGL(k_bs_multipoles, dim3((most + kMpWaves - 1) / kMpWaves), dim3(64 * kMpWaves), 0, s, c->cstart,
                           src, coef, items, st);
        hipLaunchKernelGGL(k_bs_boxes, dim3(std::min(n / 32 + 1, 4096)), dim3(64 * kBoxWaves), 0, s, c->cstart, src, coef,
                           items, st, sc, u, v);
    } else {
        hipLaunchKernelGGL(k_zero_uv, dim3(min(blocks_for(n), 1024)), dim3(256), 0, s, cl->n_dev, u, v);
    }
    const int tx = (n + kBsBlock * kBsT - 1) / (kBsBlock * kBsT);
    // source chunks: enough workgroups to fill the chip (>= 2048), whole tiles each
    const int tiles = (n + kBsTile - 1) / kBsTile;
    const int sy = max(1, min(tiles, (2048 + tx - 1) / tx));
    const int chunk = ((tiles + sy - 1) / sy) * kBsTile;
    const int ny = (n + chunk - 1) / chunk;
    hipLaunchKernelGGL(k_biot_savart, dim3(tx, ny), dim3(kBsBlock), 0, s, cl->n_dev, cl->x_dev, cl->y_dev,
                       cl->gamma_dev, sc, chunk, u, v, boxes ? st : nullptr, c->cstart, reinterpret_cast<const float4*>(c->akey));
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}
