// Complete-neighbourhood LPs from a known basis: within a step the particles move by
// a small fraction of h between the stages, and the basis of a particle's stencil
// one stage earlier is almost always the basis of the next one.  Checking a basis
// needs no simplex, no sorted column list and no explicit inverse: factor the M x M
// matrix of the basic columns, refine the basic solution, and price every column of
// the neighbourhood once.  What the check does not settle goes to the LP kernels.
//
// The check is the fast certificate of ThreadSimplex::certify: the basic values from
// one refinement step with an extended-precision residual, accepted when the first
// correction is at most 1e-5 of the values (which leaves them accurate to 1e-10), all
// values >= -kCertX, and every other column's reduced cost clear of zero by kFastMargin
// times the measured error -- here the first correction plus the largest relative
// reduced cost of a basic column, which is zero in exact arithmetic.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "vrm_lp_common.h"

using namespace vrm;

namespace {

// Householder factorisation of the M x M matrix a (columns: the basic columns), in
// place: R above the diagonal, its reciprocal diagonal in rd, the reflectors' vectors
// on and below it, H_k = I + bi_k v_k v_k^T.  No pivoting, so no dynamic indices.
template <int M>
struct Qr {
    float a[M][M], rd[M], bi[M];

    __device__ __forceinline__ void factor()
    {
#pragma unroll
        for (int k = 0; k < M; ++k) {
            float s2 = 0.0f;
#pragma unroll
            for (int i = k; i < M; ++i) s2 = __builtin_fmaf(a[i][k], a[i][k], s2);
            if (k == M - 1) {
                rd[k] = __builtin_amdgcn_rcpf(a[k][k]);
                bi[k] = 0.0f;
                break;
            }
            const float nrm = __builtin_amdgcn_sqrtf(s2);
            const float alpha = a[k][k] > 0.0f ? -nrm : nrm;
            a[k][k] -= alpha;
            rd[k] = __builtin_amdgcn_rcpf(alpha);
            bi[k] = __builtin_amdgcn_rcpf(alpha * a[k][k]);
#pragma unroll
            for (int j = k + 1; j < M; ++j) {
                float s = 0.0f;
#pragma unroll
                for (int i = k; i < M; ++i) s = __builtin_fmaf(a[i][k], a[i][j], s);
                s *= bi[k];
#pragma unroll
                for (int i = k; i < M; ++i) a[i][j] = __builtin_fmaf(s, a[i][k], a[i][j]);
            }
        }
    }
    __device__ __forceinline__ void reflect(int k, float (&w)[M]) const
    {
        float s = 0.0f;
#pragma unroll
        for (int i = k; i < M; ++i) s = __builtin_fmaf(a[i][k], w[i], s);
        s *= bi[k];
#pragma unroll
        for (int i = k; i < M; ++i) w[i] = __builtin_fmaf(s, a[i][k], w[i]);
    }
    // w <- V^-1 w
    __device__ __forceinline__ void solve(float (&w)[M]) const
    {
#pragma unroll
        for (int k = 0; k < M - 1; ++k) reflect(k, w);
#pragma unroll
        for (int k = M - 1; k >= 0; --k) {
            float s = w[k];
#pragma unroll
            for (int j = k + 1; j < M; ++j) s = __builtin_fmaf(-a[k][j], w[j], s);
            w[k] = s * rd[k];
        }
    }
    // w <- V^-T w
    __device__ __forceinline__ void solve_t(float (&w)[M]) const
    {
#pragma unroll
        for (int k = 0; k < M; ++k) {
            float s = w[k];
#pragma unroll
            for (int j = 0; j < k; ++j) s = __builtin_fmaf(-a[j][k], w[j], s);
            w[k] = s * rd[k];
        }
#pragma unroll
        for (int k = M - 2; k >= 0; --k) reflect(k, w);
    }
};

// x0 = V^-1 b and one refinement step from the residual b - V x0, summed with its
// rounding errors over the exact offsets; returns |correction| / |x|
template <int M>
__device__ __forceinline__ float refined_solution(const Qr<M>& qr, const float (&bx)[M], const float (&by)[M],
                                                  float xi, float yi, const LaunchParams& P, float (&x)[M])
{
    float x0[M];
#pragma unroll
    for (int a = 0; a < M; ++a) x0[a] = rhs_row<M>(a) ? P.bt_hi : 0.0f;
    qr.solve(x0);
    float hi[M], lo[M];
#pragma unroll
    for (int a = 0; a < M; ++a) {
        hi[a] = rhs_row<M>(a) ? P.bt_hi : 0.0f;
        lo[a] = rhs_row<M>(a) ? P.bt_lo : 0.0f;
    }
#pragma unroll
    for (int c = 0; c < M; ++c) {
        df X, Y, v[M];
        exact_offset(xi, yi, bx[c], by[c], P.scale2e, X, Y);
        mono_df<M>(X, Y, v);
        const float nx = -x0[c];
#pragma unroll
        for (int a = 0; a < M; ++a) {
            const float p = v[a].hi * nx;
            float pe = __builtin_fmaf(v[a].hi, nx, -p);
            pe = __builtin_fmaf(v[a].lo, nx, pe);
            const df s = two_sum(hi[a], p);
            hi[a] = s.hi;
            lo[a] += s.lo + pe;
        }
        __builtin_amdgcn_sched_barrier(0);   // one column at a time: its monomials' registers are reused
    }
    float res[M];
#pragma unroll
    for (int a = 0; a < M; ++a) res[a] = hi[a] + lo[a];
    qr.solve(res);
    float dmax = 0.0f, xmax = 0.0f;
#pragma unroll
    for (int r = 0; r < M; ++r) {
        dmax = fmaxf(dmax, fabsf(res[r]));
        x[r] = x0[r] + res[r];
        xmax = fmaxf(xmax, fabsf(x[r]));
    }
    return dmax / fmaxf(xmax, 1e-30f);
}

// a value the compiler may not tie to earlier expressions of it: the monomials are
// cheaper formed again than kept in 81 registers
__device__ __forceinline__ void fresh(float& v) { asm volatile("" : "+v"(v)); }

constexpr int kVBlock = 64;
constexpr int kVBins = 10;   // buckets of members between the nine basic ids: six bits each in one word

// Bound by VALU issue (about 8600 instructions per wave of 64 LPs: the scan of ~120
// candidates a quarter, the factorisation and solves a third, pricing a quarter) at two
// waves per SIMD (188 VGPRs; at three, 24 spilled).  22.5M LPs: 8.7 ms, against 43 ms for
// their column lists and cold LPs; 0.4 % are left for the sixteen-lane kernel (0.45 ms).
// Consecutive blocks on consecutive XCDs: a block of the cloud per XCD took 9.8 ms.
// One thread per particle, slot order (the lanes of a wave share cells).  Members of
// the neighbourhood go to a list in LDS (slot, and the number of basic ids below the
// member's id).  The tie-break of the cost needs id ranks: a basic column's is exact
// (the members below it, from the bucket counts), another column's at least the number
// of members in lower buckets; only where that bound does not settle the sign of a
// reduced cost is the exact rank counted.
template <int M>
__global__ __launch_bounds__(kVBlock) __attribute__((amdgpu_waves_per_eu(2))) void k_verify(
    int nb, const int32_t* __restrict__ n_dev, const int32_t* __restrict__ perm, const float* __restrict__ xs,
    const float* __restrict__ ys, const int32_t* __restrict__ ids, const int32_t* __restrict__ cell_start,
    const GridState* gs, const uint8_t* __restrict__ diffused, const float* __restrict__ px,
    const float* __restrict__ py, const int32_t* __restrict__ pid, const float* __restrict__ gamma, float* acc,
    LaunchParams P, const int32_t* __restrict__ sten_idx, float* sten_f, int32_t* q_full, Queues* qs,
    vrm_counters* cnt, int count_hits)
{
    static_assert(M == 9, "nine-row LPs");
    __shared__ uint32_t s_list[VRM_KMAX * kVBlock];
    cnt = counter_stripe(cnt);
    const int lane = threadIdx.x;
    const int n = min(*n_dev, nb);
    const int t = blockIdx.x * kVBlock + lane;
    int i = 0;
    bool live = t < n && !gs->bad;
    if (live) {
        i = perm[t];
        live = diffused[i];
    }
    bool ok = false;
    int k = 0;
    if (live) {
        const GridState g = *gs;
        const float xi = xs[t], yi = ys[t];
        int idx[kStenRow];
        {
            const int4* row = reinterpret_cast<const int4*>(sten_idx + (size_t)i * kStenRow);
#pragma unroll
            for (int q = 0; q < kStenRow / 4; ++q) {
                const int4 a = row[q];
                idx[4 * q] = a.x, idx[4 * q + 1] = a.y, idx[4 * q + 2] = a.z, idx[4 * q + 3] = a.w;
            }
        }
        ok = idx[kStenRow - 1] == M;
#pragma unroll
        for (int r = 0; r < M; ++r) {
            ok = ok && (unsigned)idx[r] < (unsigned)n;
            idx[r] = ok ? idx[r] : i;
        }
        // the basic columns' positions and ids
        float bpx[M], bpy[M];
        int bid[M];
#pragma unroll
        for (int r = 0; r < M; ++r) {
            bpx[r] = px[idx[r]];
            bpy[r] = py[idx[r]];
            bid[r] = pid[idx[r]];
            const float d2 = d2_f32(bpx[r] - xi, bpy[r] - yi);
            ok = ok && !(d2 < P.lo2f) && !(d2 > P.hi2f);   // still in the neighbourhood (and not the particle itself)
        }
        // the members (the particle itself is nearer than r h)
        int cx, cy;
        cell_of_pos(g, xi, yi, cx, cy);
        for (int oy = -1; oy <= 1 && ok; ++oy) {
            const int yy = cy + oy;
            if (yy < 0 || yy >= g.ny) continue;
            const int u0 = cell_start[yy * g.nx + max(cx - 1, 0)];
            const int u1 = cell_start[yy * g.nx + min(cx + 1, g.nx - 1) + 1];
            for (int ub = u0; ub < u1; ub += 8) {
                float bx[8], by[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int v = min(ub + e, u1 - 1);
                    bx[e] = xs[v];
                    by[e] = ys[v];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d2 = d2_f32(bx[e] - xi, by[e] - yi);
                    const bool mem = ub + e < u1 && !(d2 < P.lo2f) && !(d2 > P.hi2f);
                    s_list[min(k, VRM_KMAX - 1) * kVBlock + lane] = (uint32_t)(ub + e) << 4;
                    k += mem ? 1 : 0;
                }
            }
        }
        // a longer list is cut to its nearest members: left to the LP kernels.  The
        // write after the last member of a full list went to its last entry.
        ok = ok && k < VRM_KMAX && k >= M;
        k = min(k, VRM_KMAX - 1);
        if (ok) {
            // buckets: the number of basic ids below each member's id
            uint64_t hist = 0;
            for (int j0 = 0; j0 < k; j0 += 4) {
                uint32_t u[4];
                int id[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    u[e] = s_list[min(j0 + e, k - 1) * kVBlock + lane];
                    id[e] = ids[u[e] >> 4];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    int m = 0;
#pragma unroll
                    for (int r = 0; r < M; ++r) m += bid[r] < id[e] ? 1 : 0;
                    if (j0 + e < k) {
                        hist += 1ull << (6 * m);
                        s_list[(j0 + e) * kVBlock + lane] = u[e] | (uint32_t)m;
                    }
                }
            }
            // members in lower buckets, per bucket (at most 48: no carry between the fields)
            uint64_t below = 0;
            {
                uint32_t at = 0;
#pragma unroll
                for (int m = 0; m < kVBins; ++m) {
                    below |= (uint64_t)at << (6 * m);
                    at += (uint32_t)(hist >> (6 * m)) & 63u;
                }
            }
            Qr<M> qr;
            float c[M], y[M], x[M];
#pragma unroll
            for (int r = 0; r < M; ++r) {
                const float X = (bpx[r] - xi) * P.scale2e, Y = (bpy[r] - yi) * P.scale2e;
                float v[M];
                mono<M>(X, Y, v);
#pragma unroll
                for (int a = 0; a < M; ++a) qr.a[a][r] = v[a];
                int pos = 0;
#pragma unroll
                for (int q = 0; q < M; ++q) pos += bid[q] < bid[r] ? 1 : 0;
                // the members up to its own id, less itself
                const uint32_t rank = ((uint32_t)(below >> (6 * pos)) & 63u) + ((uint32_t)(hist >> (6 * pos)) & 63u) - 1u;
                const float d2 = X * X + Y * Y;
                c[r] = __builtin_fmaf(d2 * d2, P.cs_hi, tie_weight(rank, 3));
                __builtin_amdgcn_sched_barrier(0);
            }
            qr.factor();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < M; ++r) fresh(bpx[r]), fresh(bpy[r]);
            const float first = refined_solution<M>(qr, bpx, bpy, xi, yi, P, x);
            // prices, with one refinement step
#pragma unroll
            for (int r = 0; r < M; ++r) fresh(bpx[r]), fresh(bpy[r]);
#pragma unroll
            for (int r = 0; r < M; ++r) y[r] = c[r];
            qr.solve_t(y);
            {
                float w[M];
#pragma unroll
                for (int r = 0; r < M; ++r) {
                    float v[M];
                    mono<M>((bpx[r] - xi) * P.scale2e, (bpy[r] - yi) * P.scale2e, v);
                    float s = c[r];
#pragma unroll
                    for (int a = 0; a < M; ++a) s = __builtin_fmaf(-y[a], v[a], s);
                    w[r] = s;
                    __builtin_amdgcn_sched_barrier(0);
                }
                qr.solve_t(w);
#pragma unroll
                for (int a = 0; a < M; ++a) y[a] += w[a];
            }
            float ya[M];
#pragma unroll
            for (int a = 0; a < M; ++a) ya[a] = fabsf(y[a]);
#pragma unroll
            for (int r = 0; r < M; ++r) fresh(bpx[r]), fresh(bpy[r]);
            float eta = 0.0f;
#pragma unroll
            for (int r = 0; r < M; ++r) {
                float d, sc;
                reduced_horner((bpx[r] - xi) * P.scale2e, (bpy[r] - yi) * P.scale2e, c[r], y, ya, 1.0f, d, sc);
                eta = fmaxf(eta, fabsf(d) * __builtin_amdgcn_rcpf(sc));
                ok = ok && x[r] >= -kCertX;
                __builtin_amdgcn_sched_barrier(0);
            }
            const float margin = kFastMargin * (first + eta + 1.1920929e-07f);
            ok = ok && first <= 1e-5f && eta <= 1e-5f;
            // columns whose reduced cost does not clear the margin: the basic ones, and
            // any other must be looked at again
            uint64_t low = 0;
            for (int j0 = 0; j0 < k; j0 += 4) {
                uint32_t u[4];
                float bx[4], by[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    u[e] = s_list[min(j0 + e, k - 1) * kVBlock + lane];
                    bx[e] = xs[u[e] >> 4];
                    by[e] = ys[u[e] >> 4];
                }
                uint32_t l4 = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float X = (bx[e] - xi) * P.scale2e, Y = (by[e] - yi) * P.scale2e;
                    const float d2 = X * X + Y * Y;
                    const uint32_t rank = (uint32_t)(below >> (6 * (u[e] & 15u))) & 63u;
                    const float cc = __builtin_fmaf(d2 * d2, P.cs_hi, tie_weight(rank, 3));
                    float d, sc;
                    reduced_horner(X, Y, cc, y, ya, 1.0f, d, sc);
                    if (j0 + e < k && !(d >= margin * sc)) l4 |= 1u << e;
                }
                low |= (uint64_t)l4 << j0;
            }
            if (ok && __popcll(low) != M) {
                int lid[M];
#pragma unroll
                for (int r = 0; r < M; ++r) lid[r] = pid[sten_idx[(size_t)i * kStenRow + r]];
                while (low && ok) {
                    const int j = __ffsll((unsigned long long)low) - 1;
                    low &= low - 1;
                    const uint32_t u = s_list[j * kVBlock + lane] >> 4;
                    const int id = ids[u];
                    bool basic = false;
#pragma unroll
                    for (int r = 0; r < M; ++r) basic = basic || lid[r] == id;
                    if (basic) continue;
                    uint32_t rank = 0;
                    for (int o = 0; o < k; ++o) rank += ids[s_list[o * kVBlock + lane] >> 4] < id ? 1u : 0u;
                    const float X = (xs[u] - xi) * P.scale2e, Y = (ys[u] - yi) * P.scale2e;
                    const float d2 = X * X + Y * Y;
                    const float cc = __builtin_fmaf(d2 * d2, P.cs_hi, tie_weight(rank, 3));
                    float d, sc;
                    reduced_horner(X, Y, cc, y, ya, 1.0f, d, sc);
                    ok = d >= margin * sc;
                }
            }
            if (ok) {
                // the stencil, as finish_lp forms it
                float sum = 0.0f;
#pragma unroll
                for (int r = 0; r < M; ++r) {
                    x[r] = x[r] > 0.0f ? x[r] : 0.0f;
                    sum += x[r];
                }
                const float tiny = 9.313225746154785e-10f * sum;
                sum = 0.0f;
                const float g_i = gamma[i];
                const double dsc = P.det ? det_scale(g.gmax_bits) : 0.0;
#pragma unroll
                for (int r = 0; r < M; ++r) {
                    x[r] = x[r] < tiny ? 0.0f : x[r];
                    sum += x[r];
                    if (x[r] != 0.0f) acc_add(acc, sten_idx[(size_t)i * kStenRow + r], x[r], g_i, dsc);
                    if (sten_f) sten_f[(size_t)i * kStenRow + r] = x[r];
                }
                acc_add(acc, i, -sum, g_i, dsc);
                if (sten_f) sten_f[(size_t)i * kStenRow + kStenRow - 1] = -sum;
            }
        }
    }
    const int p = wave_append(&qs->n_full, live && !ok);
    if (live && !ok) q_full[p] = t;
    const uint64_t hits = __ballot(live && ok);
    int cols = live && ok ? k : 0;
    for (int o = 32; o > 0; o >>= 1) cols += __shfl_xor(cols, o, VRM_WAVE);
    if (lane == 0 && hits) {
        const unsigned long long h = (unsigned long long)__popcll(hits);
        atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->n_full), h);
        atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->redistributions), h);
        atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->cert_rounds), h);
        atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->full_cols), (unsigned long long)cols);
        if (count_hits) atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->warm_hit), h);
    }
}

// Small neighbourhoods and their five-row LPs, the basis known by its segments: the
// scan of k_small_nbhd, then the check on the eight columns it found (one per segment,
// so another particle in a segment does not void the hint).  Nothing is written for an
// LP that the check settles: no record, no queue entry.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_verify_small(
    int nb, const int32_t* __restrict__ n_dev, const int32_t* __restrict__ perm, const float* __restrict__ xs,
    const float* __restrict__ ys, const int32_t* __restrict__ ids, const int32_t* __restrict__ cell_start,
    const GridState* gs, const uint8_t* __restrict__ diffused, const float* __restrict__ gamma, float* acc,
    LaunchParams P, uint8_t* seg_mask, int32_t* prev, int prev_cap, int from_prev, SmallRec rec,
    int32_t* q_small, int32_t* q_full, Queues* qs, vrm_counters* cnt)
{
    constexpr int M = 5;
    __shared__ float s_bd[VRM_NSEG * 256];
    __shared__ int s_best[VRM_NSEG * 256];
    __shared__ int s_app[17];
    cnt = counter_stripe(cnt);
    const int n = min(*n_dev, nb);
    const int tid = threadIdx.x;
    const int t = blockIdx.x * 256 + tid;
    bool dif = t < n && !gs->bad;   // no cell list while a value is not finite
    int i = 0;
    if (dif) {
        i = perm[t];
        dif = diffused[i];
    }
#pragma unroll
    for (int s = 0; s < VRM_NSEG; ++s) {
        s_bd[s * 256 + tid] = INFINITY;
        s_best[s * 256 + tid] = -1;
    }
    int best[VRM_NSEG];
    int ksmall = 0;
    bool ok = false;
    if (dif) {
        const float xi = xs[t], yi = ys[t];
        int kfull = 0;
        scan_segments(t, xi, yi, *gs, cell_start, xs, ys, ids, P, s_bd, s_best, tid, kfull);
        int id[VRM_NSEG];
        uint32_t present = 0;
#pragma unroll
        for (int s = 0; s < VRM_NSEG; ++s) {
            best[s] = s_best[s * 256 + tid];
            present |= best[s] >= 0 ? 1u << s : 0u;
            id[s] = best[s] >= 0 ? ids[best[s]] : 0x7fffffff;
            // the columns' positions by segment (an absent one: the particle's own)
            s_bd[s * 256 + tid] = best[s] >= 0 ? xs[best[s]] : xi;
            s_best[s * 256 + tid] = __float_as_int(best[s] >= 0 ? ys[best[s]] : yi);
        }
        ksmall = __popc(present);
        const int own = prev ? ids[t] : 0;
        uint32_t mask = 0;
        if (from_prev) {
            // segments whose member was in the particle's previous basis
            int pv[M];
#pragma unroll
            for (int r = 0; r < M; ++r)
                pv[r] = (unsigned)own < (unsigned)prev_cap ? prev[(size_t)own * kPrevIds + r] : -1;
#pragma unroll
            for (int s = 0; s < VRM_NSEG; ++s)
#pragma unroll
                for (int r = 0; r < M; ++r) mask |= pv[r] == id[s] ? 1u << s : 0u;
            seg_mask[i] = (uint8_t)mask;   // for the next stage
        } else {
            mask = seg_mask[i];
        }
        ok = __popc(mask) == M && (mask & ~present) == 0;
        if (ok) {
            uint32_t ranks = 0;   // id rank of segment s's column at bit 3 s
#pragma unroll
            for (int s = 0; s < VRM_NSEG; ++s) {
                uint32_t rank = 0;
#pragma unroll
                for (int o = 0; o < VRM_NSEG; ++o) rank += id[o] < id[s] ? 1u : 0u;
                ranks |= (rank & 7u) << (3 * s);
            }
            // offset and FP32 cost of segment s's column, from LDS
            auto column = [&](int s, float& X, float& Y) -> float {
                X = (s_bd[s * 256 + tid] - xi) * P.scale2e;
                Y = (__int_as_float(s_best[s * 256 + tid]) - yi) * P.scale2e;
                const float d2 = X * X + Y * Y;
                return __builtin_fmaf(d2 * __builtin_sqrtf(d2), P.cs_hi, tie_weight((ranks >> (3 * s)) & 7u, 2));
            };
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // read them back: registers are short
            float bpx[M], bpy[M], c[M], y[M], x[M];
            uint32_t left = mask;
            Qr<M> qr;
#pragma unroll
            for (int r = 0; r < M; ++r) {
                const int s = __ffs((int)left) - 1;
                left &= left - 1;
                bpx[r] = s_bd[s * 256 + tid];
                bpy[r] = __int_as_float(s_best[s * 256 + tid]);
                float v[M], X, Y;
                c[r] = column(s, X, Y);
                y[r] = c[r];
                mono<M>(X, Y, v);
#pragma unroll
                for (int a = 0; a < M; ++a) qr.a[a][r] = v[a];
            }
            qr.factor();
            const float first = refined_solution<M>(qr, bpx, bpy, xi, yi, P, x);
            qr.solve_t(y);
            {
                float w[M];
#pragma unroll
                for (int r = 0; r < M; ++r) {
                    float v[M];
                    mono<M>((bpx[r] - xi) * P.scale2e, (bpy[r] - yi) * P.scale2e, v);
                    float s = c[r];
#pragma unroll
                    for (int a = 0; a < M; ++a) s = __builtin_fmaf(-y[a], v[a], s);
                    w[r] = s;
                }
                qr.solve_t(w);
#pragma unroll
                for (int a = 0; a < M; ++a) y[a] += w[a];
            }
            // every column priced: the basic ones measure the error, the others must clear it
            float eta = 0.0f, low = __builtin_inff();
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int s = 0; s < VRM_NSEG; ++s) {
                float v[M], X, Y;
                const float cs = column(s, X, Y);
                mono<M>(X, Y, v);
                float d, sc;
                reduced(v, cs, y, true, d, sc);
                const float key = d * __builtin_amdgcn_rcpf(sc);
                const bool basic = (mask >> s) & 1u, other = ((present & ~mask) >> s) & 1u;
                eta = basic ? fmaxf(eta, fabsf(key)) : eta;
                low = other ? fminf(low, key) : low;
            }
            const float margin = kFastMargin * (first + eta + 1.1920929e-07f);
            ok = first <= 1e-5f && eta <= 1e-5f && low >= margin * 1.00000095367431640625f;
#pragma unroll
            for (int r = 0; r < M; ++r) ok = ok && x[r] >= -kCertX;
            if (ok) {
                // the stencil, as finish_lp forms it
                float sum = 0.0f;
#pragma unroll
                for (int r = 0; r < M; ++r) {
                    x[r] = x[r] > 0.0f ? x[r] : 0.0f;
                    sum += x[r];
                }
                const float tiny = 9.313225746154785e-10f * sum;
                sum = 0.0f;
                const float g_i = gamma[i];
                const double dsc = P.det ? det_scale(gs->gmax_bits) : 0.0;
                left = mask;
#pragma unroll
                for (int r = 0; r < M; ++r) {
                    const int s = __ffs((int)left) - 1;
                    left &= left - 1;
                    x[r] = x[r] < tiny ? 0.0f : x[r];
                    sum += x[r];
                    int u = 0;
#pragma unroll
                    for (int q = 0; q < VRM_NSEG; ++q) u = q == s ? best[q] : u;
                    if (x[r] != 0.0f) acc_add(acc, perm[u], x[r], g_i, dsc);
                    if (prev && (unsigned)own < (unsigned)prev_cap) prev[(size_t)own * kPrevIds + r] = ids[u];
                }
                acc_add(acc, i, -sum, g_i, dsc);
                if (prev && (unsigned)own < (unsigned)prev_cap)
#pragma unroll
                    for (int r = M; r < kPrevIds; ++r) prev[(size_t)own * kPrevIds + r] = -1;
            }
        }
    }
    const bool small_ok = dif && !ok && ksmall >= M;
    const int p1 = block_append_n(&qs->n_small, small_ok ? 1 : 0, s_app);
    if (small_ok) {
        q_small[p1] = t;
        write_small_record(rec, p1, i, xs[t], ys[t], best, perm, xs, ys, ids, P);
    }
    const bool full = dif && !ok && !small_ok;
    const int p2 = block_append_n(&qs->n_full, full ? 1 : 0, s_app);
    if (full) q_full[p2] = t;
    const uint64_t hits = __ballot(ok);
    if (lane_id() == 0 && hits) {
        const unsigned long long h = (unsigned long long)__popcll(hits);
        atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->n_small), h);
        atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->redistributions), h);
        if (prev) atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->warm_hit), h);
    }
}

// The previous-basis warm start keeps bases by id (they outlive the reordering of the
// cloud); rows of column indices for k_verify from them.  inv[id]: the particle of an
// id; an id that left the cloud may find any particle, whose own id then differs.
__global__ __launch_bounds__(256) void k_index_of_id(int nb, const int32_t* __restrict__ n_dev,
                                                     const int32_t* __restrict__ id, int cap, int32_t* inv)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= min(*n_dev, nb)) return;
    const int d = id[i];
    if ((unsigned)d < (unsigned)cap) inv[d] = i;
}

__global__ __launch_bounds__(256) void k_bases_from_prev(int nb, const int32_t* __restrict__ n_dev,
                                                         const int32_t* __restrict__ id, int cap,
                                                         const int32_t* __restrict__ inv,
                                                         const int32_t* __restrict__ prev, int32_t* sten_idx)
{
    const int n = min(*n_dev, nb);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int own = id[i];
    int row[kStenRow];
    bool ok = (unsigned)own < (unsigned)cap;
#pragma unroll
    for (int r = 0; r < kPrevIds; ++r) {
        const int d = ok ? prev[(size_t)own * kPrevIds + r] : -1;
        const int j = (unsigned)d < (unsigned)cap ? inv[d] : -1;
        ok = ok && (unsigned)j < (unsigned)n && id[j] == d;
        row[r] = ok ? j : -1;
    }
    row[9] = row[10] = -1;
    row[kStenRow - 1] = ok ? kPrevIds : -1;
    int4* out = reinterpret_cast<int4*>(sten_idx + (size_t)i * kStenRow);
#pragma unroll
    for (int q = 0; q < kStenRow / 4; ++q) out[q] = int4{row[4 * q], row[4 * q + 1], row[4 * q + 2], row[4 * q + 3]};
}

}  // namespace

int vrm_bases_from_prev_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n)
{
    // the ranks of the cell build are not needed any more: their array holds the map
    int32_t* inv = c->rank;
    const int grid = (n + 255) / 256;
    hipLaunchKernelGGL(k_index_of_id, dim3(grid), dim3(256), 0, c->stream, n, cl->n_dev, cl->id_dev, c->capacity, inv);
    hipLaunchKernelGGL(k_bases_from_prev, dim3(grid), dim3(256), 0, c->stream, n, cl->n_dev, cl->id_dev, c->capacity,
                       inv, c->prev, sten_rows(c, 9).idx);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

int vrm_verify_small_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const LaunchParams& lp, int32_t* prev,
                         bool from_prev)
{
    hipLaunchKernelGGL(k_verify_small, dim3((n + 255) / 256), dim3(256), 0, c->stream, n, cl->n_dev, c->perm, c->xs,
                       c->ys, c->ids, c->cell_start, c->grid, c->diffused, cl->gamma_dev, c->acc, lp, c->tmp_u8, prev,
                       c->capacity, from_prev ? 1 : 0, c->srec, c->q_small, c->q_full, c->queues, c->counters);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

int vrm_verify_bases_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const LaunchParams& lp, bool keep_f,
                         bool count_hits)
{
    const StenRows rows = sten_rows(c, 9);
    const int grid = (n + kVBlock - 1) / kVBlock;
    hipLaunchKernelGGL(k_verify<9>, dim3(grid), dim3(kVBlock), 0, c->stream, n, cl->n_dev, c->perm, c->xs, c->ys, c->ids,
                       c->cell_start, c->grid, c->diffused, cl->x_dev, cl->y_dev, cl->id_dev, cl->gamma_dev, c->acc, lp,
                       rows.idx, keep_f ? rows.f : nullptr, c->q_full, c->queues, c->counters, count_hits ? 1 : 0);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}
