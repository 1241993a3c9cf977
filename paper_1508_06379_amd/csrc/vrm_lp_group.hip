// Complete-neighbourhood LPs with sixteen lanes each, for launches too small to
// fill the chip with one thread per LP.
//
// The one-thread kernels (vrm_lp.hip) are one wave's chain of dependent
// instructions per 64 LPs; with fewer waves than SIMDs that chain is the launch's
// time.  Here a DPP row of sixteen lanes solves one LP, collection included: the
// lanes scan the cells together, each holds three columns (column s + 16 c), and
// lane r < M holds row r of B^-1, the basic value, cost and column of row r, and
// column r of B^-1 (the prices need the columns, the pivot elements the rows).
// Broadcasts within the row are DPP operands, the leaving row travels through LDS.
// Every value is formed by the same operations in the same order as in
// ThreadSimplex, so both take the same pivots and end on the same basis in the same
// row order: stencils, statuses, their order and the pivot counts are identical.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "vrm_lp_common.h"

using namespace vrm;

namespace {

constexpr int kGL = 16;                      // lanes per LP (a DPP row)
constexpr int kGBlock = 256;
constexpr int kGGroups = kGBlock / kGL;      // LPs per workgroup
constexpr int kGSets = VRM_KMAX / kGL;       // columns per lane
constexpr int kGList = 64;                   // members a group's list holds
constexpr int kGListStride = kGList + 4;
static_assert(kGSets * kGL == VRM_KMAX, "three whole sets of sixteen columns");

// A group's LDS.  The member list is dead once the columns are placed, so the
// basis' monomials and the leaving row share its space.
struct GroupLds {
    union {
        struct {
            uint64_t key[kGListStride];   // bits of d2 over the id: one comparison orders (d2, id)
            int u[kGListStride];
            int pos[kGListStride];
        } list;
        struct {
            float row[12];                // row l of B^-1, then its pivot element, value and column
            float2 mono[9][9];            // [basis row][moment]: exact monomials of the basic columns
        } lp;
    };
    float4 col[VRM_KMAX];                 // scaled offset, FP32 cost, (slot << 6) | id rank
    float pad[4];                         // the four groups of a wave start in different banks
};

// the value of lane K of this lane's row
template <int K>
__device__ __forceinline__ int bc(int v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x150 + K, 0xF, 0xF, true);
}
template <int K>
__device__ __forceinline__ float bc(float v)
{
    return __int_as_float(bc<K>(__float_as_int(v)));
}
template <class F, int... I>
__device__ __forceinline__ void sfor_impl(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
// f(0), f(1), ..., f(N - 1) with compile-time indices
template <int N, class F>
__device__ __forceinline__ void sfor(F&& f)
{
    sfor_impl(f, std::make_integer_sequence<int, N>{});
}

template <int CTRL>
__device__ __forceinline__ float dppf(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dppu(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
// reductions over a row: lanes xor 1, xor 2, the mirror of eight, the mirror of sixteen
__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, dppf<0xB1>(v));
    v = fmaxf(v, dppf<0x4E>(v));
    v = fmaxf(v, dppf<0x141>(v));
    return fmaxf(v, dppf<0x140>(v));
}
__device__ __forceinline__ float row_min(float v)
{
    v = fminf(v, dppf<0xB1>(v));
    v = fminf(v, dppf<0x4E>(v));
    v = fminf(v, dppf<0x141>(v));
    return fminf(v, dppf<0x140>(v));
}
__device__ __forceinline__ uint32_t row_umin(uint32_t v)
{
    v = min(v, dppu<0xB1>(v));
    v = min(v, dppu<0x4E>(v));
    v = min(v, dppu<0x141>(v));
    return min(v, dppu<0x140>(v));
}
__device__ __forceinline__ float quad_min(float v)
{
    v = fminf(v, dppf<0xB1>(v));
    return fminf(v, dppf<0x4E>(v));
}
// order the LDS accesses of a wave's lanes on both sides
__device__ __forceinline__ void lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The simplex of one LP on a row of lanes (see ThreadSimplex for what each step
// does and why).  Lanes s >= M hold zeros and never qualify in a reduction.
template <int M>
struct GroupSimplex {
    static constexpr int ART = 64;
    static constexpr int kQ = M == 3 ? 1 : M == 5 ? 2 : 3;
    int s, gb;                 // lane in the row, the row's first lane in the wave
    GroupLds* L;
    const LaunchParams* P;
    const float* xs;
    const float* ys;
    float xi, yi;
    int k, kw;                 // columns, and the prefix priced (the working set, then all)
    float cx[kGSets], cy[kGSets], cc[kGSets];   // this lane's columns
    float BR[M], BC[M];        // row s and column s of B^-1
    float xb, cb;              // basic value and cost of row s
    int bs;                    // basic column of row s; 64 + s: artificial
    uint32_t basic, blocked;   // bit c: this lane's column of set c is basic; blocked until the next pivot
    bool any_blocked;
    float cert_key;
    int cert_rounds, cert_exact;

    __device__ __forceinline__ uint32_t votes(bool p) const { return (uint32_t)(__ballot(p) >> gb) & 0xFFFFu; }
    __device__ __forceinline__ bool row_lane() const { return s < M; }
    __device__ __forceinline__ static bool rhs_lane(int r) { return M == 3 ? r == 0 : (r == 2 || r == 4); }

    __device__ void init()
    {
#pragma unroll
        for (int a = 0; a < M; ++a) {
            BR[a] = s == a ? 1.0f : 0.0f;
            BC[a] = s == a ? 1.0f : 0.0f;
        }
        xb = (rhs_lane(s) ? P->bt_hi : 0.0f) + kPerturb * P->bt_hi * (1.0f + 0.618f * (float)s);
        if (!row_lane()) xb = 0.0f;
        cb = 0.0f;
        bs = row_lane() ? ART + s : 0x7fffffff;
        basic = 0;
        blocked = 0;
        any_blocked = false;
        cert_key = -__builtin_inff();
        cert_rounds = 0;
        cert_exact = 0;
    }

    // prices of the basis in every lane
    __device__ __forceinline__ void prices(bool p2, float (&y)[M]) const
    {
        const float w = p2 ? cb : (bs >= ART ? 1.0f : 0.0f);
        float own = 0.0f;
        sfor<M>([&](auto r) { own = __builtin_fmaf(bc<r>(w), BC[r], own); });
        sfor<M>([&](auto a) { y[a] = bc<a>(own); });
    }

    __device__ __forceinline__ void reduced_cost(float x, float Y, float c, const float (&y)[M], bool p2, float& d,
                                                 float& sc) const
    {
        if constexpr (M == 9) {
            float ya[M];
#pragma unroll
            for (int a = 0; a < M; ++a) ya[a] = fabsf(y[a]);
            reduced_horner(x, Y, c, y, ya, p2 ? 1.0f : 0.0f, d, sc);
        } else {
            float v[M];
            mono<M>(x, Y, v);
            reduced(v, c, y, p2, d, sc);
        }
    }

    // Entering column: sets of sixteen (one column per lane) in list order, the
    // choice within the first group of four that holds an improving column.
    __device__ int price(const float (&y)[M], bool p2, bool bland)
    {
        const uint32_t out = basic | blocked;
        int e = -1;
        float mk = __builtin_inff();
#pragma unroll
        for (int c = 0; c < kGSets; ++c) {
            if (e >= 0 || kGL * c >= kw) continue;
            float d, sc;
            reduced_cost(cx[c], cy[c], cc[c], y, p2, d, sc);
            const float key = d * __builtin_amdgcn_rcpf(sc);
            const bool in = kGL * c + s < kw && !(out & (1u << c));
            mk = fminf(mk, in ? key : __builtin_inff());
            const bool ok = in && d < -kTolD * sc && (bland || key < 0.0f);
            const uint32_t m = votes(ok);
            if (m) {
                const int f = __ffs((int)m) - 1;
                if (bland) {
                    e = kGL * c + f;
                } else {
                    const float kk = ok ? key : __builtin_inff();
                    const float best = quad_min(kk);
                    const uint32_t w = votes(ok && kk == best && (s >> 2) == (f >> 2));
                    e = kGL * c + __ffs((int)w) - 1;
                }
            }
        }
        if (e < 0) cert_key = (!any_blocked && kw == k) ? row_min(mk) : -__builtin_inff();
        else cert_key = -__builtin_inff();
        return e;
    }

    // this row's entry of B^-1 v for the column at (rx, ry)
    __device__ __forceinline__ float alpha_of(float rx, float ry) const
    {
        float v[M];
        mono<M>(rx, ry, v);
        float t = 0.0f;
#pragma unroll
        for (int a = 0; a < M; ++a) t = __builtin_fmaf(BR[a], v[a], t);
        return t;   // 0 in lanes s >= M
    }

    // leaving row (lowest ratio, then lowest basic column), -1 if none
    __device__ __forceinline__ int ratio_test(float alpha, float x, bool phase2) const
    {
        const float eps = kTolPiv * row_max(fabsf(alpha));
        const bool special = phase2 && bs >= ART && fabsf(alpha) > eps;
        const bool ok = row_lane() && (special || alpha > eps);
        // + 0 makes a negative zero positive: the bits then order as the values
        const float ratio = special ? 0.0f : fmaxf(x, 0.0f) * __builtin_amdgcn_rcpf(alpha) + 0.0f;
        const uint32_t u = ok ? __float_as_uint(ratio) : 0xffffffffu;
        const uint32_t um = row_umin(u);
        if (um == 0xffffffffu) return -1;
        const uint32_t b = ok && u == um ? (uint32_t)bs : 0xffffffffu;
        const uint32_t bm = row_umin(b);
        return __ffs((int)votes(b == bm)) - 1;
    }

    __device__ void pivot(int l, int e, float alpha, float ce)
    {
        lds_fence();   // the previous row has been read
        if (s == l) {
#pragma unroll
            for (int a = 0; a < M; ++a) L->lp.row[a] = BR[a];
            L->lp.row[9] = alpha;
            L->lp.row[10] = xb;
            L->lp.row[11] = __int_as_float(bs);
        }
        lds_fence();
        const float inv = 1.0f / L->lp.row[9];
        float row[M];
#pragma unroll
        for (int a = 0; a < M; ++a) row[a] = L->lp.row[a] * inv;
        const float own = row_lane() ? L->lp.row[s] * inv : 0.0f;   // column s of the scaled row
        const float xl = L->lp.row[10] * inv;
        const int old = __float_as_int(L->lp.row[11]);
        const bool me = s == l;
        const float na = -alpha;   // 0 in lanes s >= M
#pragma unroll
        for (int a = 0; a < M; ++a) BR[a] = me ? row[a] : __builtin_fmaf(na, row[a], BR[a]);
        // the same update by columns: row l becomes 1 * own + 0 * (its old value)
        const float mul = me ? 1.0f : na, keep = me ? 0.0f : 1.0f;
        sfor<M>([&](auto r) { BC[r] = __builtin_fmaf(bc<r>(mul), own, bc<r>(keep) * BC[r]); });
        xb = me ? xl : __builtin_fmaf(na, xl, xb);
        bs = me ? e : bs;
        cb = me ? ce : cb;
        if (old < ART && s == (old & (kGL - 1))) basic &= ~(1u << (old / kGL));
        if (s == (e & (kGL - 1))) basic |= 1u << (e / kGL);
        blocked = 0;
        any_blocked = false;
    }

    // both phases from the artificial basis: 0 optimal, 1 infeasible, 2 iteration limit
    __device__ int run(int& piv)
    {
        const int bland_after = 3 * (k + M);
        const int limit = 10 * (k + M) + 20;
        bool p2 = false;
        for (int it = 0;; ++it) {
            if (it >= limit) return 2;
            float y[M];
            prices(p2, y);
            const int e = price(y, p2, it >= bland_after);
            if (e < 0) {
                if (p2) {
                    if (kw < k) {
                        kw = k;
                        continue;
                    }
                    return 0;
                }
                float art = 0.0f;
                const float mine = bs >= ART && row_lane() ? fabsf(xb) : 0.0f;
                sfor<M>([&](auto r) { art += bc<r>(mine); });
                if (art > kTolFeas * P->bt_hi) {
                    if (kw < k) {
                        kw = k;
                        continue;
                    }
                    return 1;
                }
                cb = bs < ART ? L->col[bs].z : 0.0f;
                blocked = 0;
                any_blocked = false;
                p2 = true;
                it = -1;
                continue;
            }
            const float4 q = L->col[e];
            const float alpha = alpha_of(q.x, q.y);
            const int l = ratio_test(alpha, xb, p2);
            if (l < 0) {
                if (s == (e & (kGL - 1))) blocked |= 1u << (e / kGL);
                any_blocked = true;
                continue;
            }
            pivot(l, e, alpha, p2 ? q.z : 0.0f);
            ++piv;
        }
    }

    __device__ __forceinline__ void exact_col(int j, df& X, df& Y, int& rank) const
    {
        const int m = __float_as_int(L->col[j].w);
        const int u = (int)((unsigned)m >> 6);
        exact_offset(xi, yi, xs[u], ys[u], P->scale2e, X, Y);
        rank = m & 63;
    }

    // exact monomials of row s's basic column (the unit vector of an artificial one)
    // for every lane of the row to read
    __device__ __forceinline__ void place_monomials(df& C)
    {
        lds_fence();
        C = {0.0f, 0.0f};
        if (row_lane()) {
            df v[M];
            if (bs < ART) {
                df X, Y;
                int rank;
                exact_col(bs, X, Y, rank);
                mono_df<M>(X, Y, v);
                C = add_rank(cost_df(X, Y, *P), rank, P->q);
            } else {
#pragma unroll
                for (int a = 0; a < M; ++a) v[a] = {bs - ART == a ? 1.0f : 0.0f, 0.0f};
            }
#pragma unroll
            for (int a = 0; a < M; ++a) L->lp.mono[s][a] = {v[a].hi, v[a].lo};
        }
        lds_fence();
    }

    // The basic solution for the exact right-hand side (row s's value in x, zero in
    // lanes s >= M); returns |first correction| / |x|.  place_monomials first.
    __device__ float refine_primal(df& x) const
    {
        float v = 0.0f;
#pragma unroll
        for (int a = 0; a < M; ++a) v += rhs_row<M>(a) ? BR[a] : 0.0f;
        x = {v * P->bt_hi, 0.0f};
        float first_corr = 1.0f;
        const int a = s < M ? s : 0;
        const df b = rhs_lane(a) ? df{P->bt_hi, P->bt_lo} : df{0.0f, 0.0f};
        for (int it = 0; it < kMaxRefine; ++it) {
            df acc{0.0f, 0.0f};
            sfor<M>([&](auto r) {
                const float2 w = L->lp.mono[r][a];
                acc = df_add(acc, df_mul(df{w.x, w.y}, df{bc<r>(x.hi), bc<r>(x.lo)}));
            });
            const df rr = df_add(b, df_neg(acc));
            const float res = rr.hi + rr.lo;
            float d = 0.0f;
            sfor<M>([&](auto q) { d = __builtin_fmaf(BR[q], bc<q>(res), d); });
            if (!row_lane()) d = 0.0f;
            x = df_add(x, df{d, 0.0f});
            const float dmax = row_max(fabsf(d));
            const float xmax = row_max(fabsf(x.hi));
            if (it == 0) first_corr = dmax / fmaxf(xmax, 1e-30f);
            if (dmax <= 9.313225746154785e-10f * xmax || (it == 0 && first_corr <= 9.5367431640625e-07f)) break;
        }
        return first_corr;
    }

    // 0 optimal, 1 infeasible, 3 not certified
    __device__ int certify(df& x, int& piv)
    {
        for (int round = 0; round < P->max_cert; ++round) {
            ++cert_rounds;
            df C;
            place_monomials(C);
            const float first_corr = refine_primal(x);
            if (votes(row_lane() && bs >= ART && fabsf(x.hi + x.lo) > kCertX)) return 1;
            if (first_corr <= 1e-5f) {
                const float margin = kFastMargin * (first_corr + 1.1920929e-07f);
                if (!votes(row_lane() && bs < ART && x.hi + x.lo < -kCertX)) {
                    bool dual_ok;
                    if (round == 0 && cert_key >= margin * 1.00000095367431640625f) {
                        dual_ok = true;
                    } else {
                        float yf[M];
                        prices(true, yf);
                        bool ok = true;
#pragma unroll
                        for (int c = 0; c < kGSets; ++c) {
                            float v[M];
                            mono<M>(cx[c], cy[c], v);
                            float d, sc;
                            reduced(v, cc[c], yf, true, d, sc);
                            const int j = kGL * c + s;
                            ok = ok && (j >= k || (basic & (1u << c)) || !(d < margin * sc));
                        }
                        dual_ok = votes(!ok) == 0;
                    }
                    if (dual_ok) return 0;
                }
            }
            cert_exact = 1;
            // prices refined to double-float; lane a holds price a
            const float w = cb;
            float own = 0.0f;
            sfor<M>([&](auto r) { own = __builtin_fmaf(bc<r>(w), BC[r], own); });
            df y{own, 0.0f};
            const int me = s < M ? s : 0;
            for (int it = 0; it < kMaxRefine; ++it) {
                // c_B - B^T y in row s
                df t = bs < ART ? C : df{0.0f, 0.0f};
                sfor<M>([&](auto a) {
                    const float2 m = L->lp.mono[me][a];
                    t = df_add(t, df_neg(df_mul(df{m.x, m.y}, df{bc<a>(y.hi), bc<a>(y.lo)})));
                });
                const float res = row_lane() ? t.hi + t.lo : 0.0f;
                float d = 0.0f;
                sfor<M>([&](auto r) { d = __builtin_fmaf(BC[r], bc<r>(res), d); });
                if (!row_lane()) d = 0.0f;
                y = df_add(y, df{d, 0.0f});
                const float dmax = row_max(fabsf(d));
                const float ymax = row_max(row_lane() ? fabsf(y.hi) : 0.0f);
                if (dmax <= 9.313225746154785e-10f * ymax) break;
            }
            df yv[M];
            sfor<M>([&](auto a) { yv[a] = {bc<a>(y.hi), bc<a>(y.lo)}; });
            // the most negative exact basic value below -kCertX leaves (lowest row among equals)
            const float xv = x.hi + x.lo;
            const bool neg = row_lane() && bs < ART && xv < -kCertX;
            if (votes(neg)) {
                const float key = neg ? -xv : 0.0f;
                const float worst = row_max(key);
                const int lrow = __ffs((int)votes(neg && key == worst)) - 1;
                lds_fence();
                if (s == lrow)
#pragma unroll
                    for (int a = 0; a < M; ++a) L->lp.row[a] = BR[a];
                lds_fence();
                float wrow[M];
#pragma unroll
                for (int a = 0; a < M; ++a) wrow[a] = L->lp.row[a];
                // dual ratio of this lane's columns; the lowest, then the first column
                uint32_t bu = 0xffffffffu;
                int bj = 0x7fffffff;
                for (int c = 0; c < kGSets; ++c) {
                    const int j = kGL * c + s;
                    if (j >= k || (basic & (1u << c))) continue;
                    df X, Y;
                    int rank;
                    exact_col(j, X, Y, rank);
                    df v[M];
                    mono_df<M>(X, Y, v);
                    float ww = 0.0f;
                    df t = add_rank(cost_df(X, Y, *P), rank, P->q);
#pragma unroll
                    for (int a = 0; a < M; ++a) {
                        ww = __builtin_fmaf(wrow[a], v[a].hi, ww);
                        t = df_add(t, df_neg(df_mul(v[a], yv[a])));
                    }
                    if (!(ww < -kTolPiv)) continue;
                    const uint32_t u = __float_as_uint(fmaxf(t.hi + t.lo, 0.0f) / (-ww) + 0.0f);
                    if (u < bu) {
                        bu = u;
                        bj = j;
                    }
                }
                const uint32_t um = row_umin(bu);
                if (um == 0xffffffffu) return 1;
                const int e = (int)row_umin(bu == um ? (uint32_t)bj : 0x7fffffffu);
                const float4 q = L->col[e];
                const float alpha = alpha_of(q.x, q.y);
                pivot(lrow, e, alpha, q.z);
                ++piv;
                continue;
            }
            // exact reduced costs; Bland's entering column
            int e = -1;
            for (int c = 0; c < kGSets && e < 0; ++c) {
                const int j = kGL * c + s;
                bool below = false;
                if (j < k && !(basic & (1u << c))) {
                    df X, Y;
                    int rank;
                    exact_col(j, X, Y, rank);
                    df v[M];
                    mono_df<M>(X, Y, v);
                    df t = add_rank(cost_df(X, Y, *P), rank, P->q);
                    float sc = fabsf(t.hi);
#pragma unroll
                    for (int a = 0; a < M; ++a) {
                        const df p = df_mul(v[a], yv[a]);
                        t = df_add(t, df_neg(p));
                        sc += fabsf(p.hi);
                    }
                    below = t.hi + t.lo < -kCertD * sc;
                }
                const uint32_t m = votes(below);
                if (m) e = kGL * c + __ffs((int)m) - 1;
            }
            if (e < 0) return 0;
            const float4 q = L->col[e];
            const float alpha = alpha_of(q.x, q.y);
            const int l = ratio_test(alpha, xv, true);
            if (l < 0) return 3;
            pivot(l, e, alpha, q.z);
            ++piv;
        }
        df C;
        place_monomials(C);
        refine_primal(x);
        return 3;
    }
};

// Members of the complete neighbourhood of slot t with a key up to thr, scanned by
// the lanes of a row; STORE: appended to the group's list (the first kGList).
template <bool STORE>
__device__ int scan_members(int t, float xi, float yi, const GridState& g, const int32_t* __restrict__ cell_start,
                            const float* __restrict__ xs, const float* __restrict__ ys, const int32_t* __restrict__ ids,
                            const LaunchParams& P, uint64_t thr, GroupLds& L, int s, int gb)
{
    int cx, cy;
    cell_of_pos(g, xi, yi, cx, cy);
    // the rows of three cells are contiguous in slot order: candidate e of the block
    // is slot base[row] + e, and the lanes load four candidates each at a time (one
    // memory latency per 64 candidates)
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
    int count = 0;
    for (int e0 = 0; e0 < total; e0 += 4 * kGL) {
        int u[4], id[4];
        float x[4], y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = min(e0 + kGL * q + s, total - 1);   // past the end: a repeat, not a member
            u[q] = e + (e < end[0] ? base[0] : e < end[1] ? base[1] : base[2]);
            x[q] = xs[u[q]];
            y[q] = ys[u[q]];
            id[q] = ids[u[q]];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float d2 = d2_f32(x[q] - xi, y[q] - yi);
            const uint64_t key = member_key(d2, id[q]);
            const bool mem = e0 + kGL * q + s < total && u[q] != t && !(d2 < P.lo2f) && !(d2 > P.hi2f) && key <= thr;
            const uint32_t m = (uint32_t)(__ballot(mem) >> gb) & 0xFFFFu;
            if constexpr (STORE) {
                const int at = count + __popc(m & ((1u << s) - 1u));
                if (mem && at < kGList) {
                    L.list.key[at] = key;
                    L.list.u[at] = u[q];
                }
            }
            count += __popc(m);
        }
    }
    return count;
}

// Bound by VALU issue once the chip is full (4.3 ns per 9-row LP; about 2300 VALU
// instructions per LP, four LPs of a wave waiting for the one with most pivots) and
// below that by one LP's chain: 18 iterations of about 2800 cycles, and the scan.
// Three waves per SIMD (168 VGPRs): two (180) and four (128, spilled) took 370 and
// 325 against 287 us for 57k LPs.  57k LPs take 270 us (510 us as column lists and
// one-thread LPs).
// Costs of the columns j < exact_n from the exact offsets, of the others from the
// FP32 ones; the simplex starts on the nearest `work` columns (the choices of the
// one-thread kernels, so that the pivots are theirs)
template <int M>
__global__ __launch_bounds__(kGBlock) __attribute__((amdgpu_waves_per_eu(M == 3 ? 5 : 3))) void k_lp_group(const int32_t* __restrict__ perm, const float* __restrict__ xs,
                                                      const float* __restrict__ ys, const int32_t* __restrict__ ids,
                                                      const int32_t* __restrict__ cell_start, const GridState* gs,
                                                      const int32_t* __restrict__ q_full, Queues* qs,
                                                      const float* __restrict__ gamma, float* acc, LaunchParams P,
                                                      StencilOut out, int apply, vrm_counters* cnt, int exact_n,
                                                      int work, const int32_t* __restrict__ q_retry, int limit)
{
    enum { kPiv, kCols, kFull, kInf, kUnc, kTrunc, kRounds, kExact, kCounts };
    __shared__ GroupLds lds[kGGroups];
    __shared__ int s_cnt[kCounts];
    const int tid = threadIdx.x, s = tid & (kGL - 1), gb = lane_id() & ~(kGL - 1);
    GroupLds& L = lds[tid / kGL];
    if (tid < kCounts) s_cnt[tid] = 0;
    __syncthreads();
    // more than `limit` in q_full: the launches before solved them, but for the retry queue
    const bool left = M != 3 && qs->n_full > limit;
    const GridState g = *gs;
    // (M = 3, the removal: nothing if a circulation is not finite or the choice of the
    // particles is not complete)
    const int nitems = M == 3 ? (g.bad || qs->rm_open[kRmRounds - 1] ? 0 : qs->n_accepted)
                       : left ? qs->n_retry : qs->n_full;
    const int32_t* __restrict__ queue = left ? q_retry : q_full;
    const double dsc = M != 3 && P.det && apply ? det_scale(g.gmax_bits) : 0.0;
    for (int item = blockIdx.x * kGGroups + tid / kGL; item < nitems; item += gridDim.x * kGGroups) {
        const int t = queue[item];
        const int i = perm[t];
        const float xi = xs[t], yi = ys[t];
        lds_fence();   // the previous LP's reads are done
        int nm = scan_members<true>(t, xi, yi, g, cell_start, xs, ys, ids, P, ~0ull, L, s, gb);
        const bool truncated = nm > VRM_KMAX;
        if (nm > kGList) {
            // the VRM_KMAX-th smallest key, by bisection, and the members up to it
            uint64_t lo = 0, hi = ~0ull;
            while (lo < hi) {
                const uint64_t mid = lo + ((hi - lo) >> 1);
                if (scan_members<false>(t, xi, yi, g, cell_start, xs, ys, ids, P, mid, L, s, gb) >= VRM_KMAX)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            lds_fence();
            nm = min(scan_members<true>(t, xi, yi, g, cell_start, xs, ys, ids, P, lo, L, s, gb), kGList);
        }
        // up to three sentinels, so the ranking reads whole groups of four
        const int nm4 = (nm + 3) & ~3;
        if (nm + s < nm4) L.list.key[nm + s] = member_key(__builtin_inff(), 0x7fffffff);
        lds_fence();
        uint64_t mk[kGList / kGL];
        int pos[kGList / kGL], rk[kGList / kGL];
#pragma unroll
        for (int q = 0; q < kGList / kGL; ++q) {
            const int e = s + kGL * q;
            mk[q] = e < nm ? L.list.key[e] : 0ull;
            pos[q] = 0;
            rk[q] = 0;
        }
        for (int o = 0; o < nm4; o += 4) {
            const ulonglong2 ka = *reinterpret_cast<const ulonglong2*>(&L.list.key[o]);
            const ulonglong2 kb = *reinterpret_cast<const ulonglong2*>(&L.list.key[o + 2]);
            const uint64_t kk[4] = {ka.x, ka.y, kb.x, kb.y};
#pragma unroll
            for (int q = 0; q < kGList / kGL; ++q) {
                if (kGL * q < nm) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        pos[q] += kk[w] < mk[q] ? 1 : 0;
                        rk[q] += (uint32_t)kk[w] < (uint32_t)mk[q] ? 1 : 0;
                    }
                }
            }
        }
        separate_equal_keys(L.list.key, nm, s, mk, pos);
        const int k = min(nm, VRM_KMAX);
        if (nm > VRM_KMAX) {
            // id ranks among the VRM_KMAX nearest only
#pragma unroll
            for (int q = 0; q < kGList / kGL; ++q)
                if (s + kGL * q < nm) L.list.pos[s + kGL * q] = pos[q];
            lds_fence();
#pragma unroll
            for (int q = 0; q < kGList / kGL; ++q) rk[q] = 0;
            for (int o = 0; o < nm; ++o) {
                const uint32_t id = (uint32_t)L.list.key[o];
                const bool kept = L.list.pos[o] < VRM_KMAX;
#pragma unroll
                for (int q = 0; q < kGList / kGL; ++q) rk[q] += (kept && id < (uint32_t)mk[q]) ? 1 : 0;
            }
        }
#pragma unroll
        for (int q = 0; q < kGList / kGL; ++q) {
            const int e = s + kGL * q;
            if (e < nm && pos[q] < VRM_KMAX)
                L.col[pos[q]].w = __int_as_float((int)(((unsigned)L.list.u[e] << 6) | (unsigned)rk[q]));
        }
        lds_fence();
        GroupSimplex<M> lp;
        lp.s = s;
        lp.gb = gb;
        lp.L = &L;
        lp.P = &P;
        lp.xs = xs;
        lp.ys = ys;
        lp.xi = xi;
        lp.yi = yi;
        lp.k = k;
        lp.kw = min(k, work);
#pragma unroll
        for (int c = 0; c < kGSets; ++c) {
            const int j = kGL * c + s;
            lp.cx[c] = 0.0f;
            lp.cy[c] = 0.0f;
            lp.cc[c] = 0.0f;
            if (j < k) {
                const int m = __float_as_int(L.col[j].w);
                const int u = (int)((unsigned)m >> 6);
                df X, Y;
                exact_offset(xi, yi, xs[u], ys[u], P.scale2e, X, Y);
                float cost;
                if (j < exact_n) {
                    cost = add_rank(cost_df(X, Y, P), m & 63, P.q).hi;
                } else {
                    const float d2 = X.hi * X.hi + Y.hi * Y.hi;
                    const float w = P.q == 1 ? d2 : P.q == 2 ? d2 * __builtin_sqrtf(d2) : d2 * d2;
                    cost = __builtin_fmaf(w, P.cs_hi, tie_weight((unsigned)m & 63u, P.q));
                }
                lp.cx[c] = X.hi;
                lp.cy[c] = Y.hi;
                lp.cc[c] = cost;
                L.col[j].x = X.hi;
                L.col[j].y = Y.hi;
                L.col[j].z = cost;
            }
        }
        lds_fence();
        lp.init();
        int piv = 0, st = 1, certified = 1;
        df x{0.0f, 0.0f};
        if (k > 0) st = lp.run(piv);
        if (st != 1) {
            const int c = lp.certify(x, piv);
            st = c == 1 ? 1 : 0;
            if (c == 3) {
                // kept only if the exact values meet the conditions
                const float v = x.hi + x.lo;
                const bool bad = lp.bs < lp.ART ? v < -kCertX : fabsf(v) > kCertX;
                if (lp.votes(lp.row_lane() && bad)) st = 1;
                certified = 0;
            }
        }
        float fii = 0.0f;
        int nz = 0;
        if (st == 0) {
            const float tv = x.hi + x.lo;
            float v = (lp.row_lane() && lp.bs < lp.ART && tv > 0.0f) ? tv : 0.0f;
            float sum = 0.0f;
            sfor<M>([&](auto r) { sum += bc<r>(v); });
            const float tiny = 9.313225746154785e-10f * sum;
            v = v < tiny ? 0.0f : v;
            sum = 0.0f;
            sfor<M>([&](auto r) { sum += bc<r>(v); });
            fii = -sum;
            const uint32_t m = lp.votes(v != 0.0f);
            nz = __popc(m);
            const float g_i = gamma[i];
            if (v != 0.0f) {
                const int at = __popc(m & ((1u << s) - 1u));
                const int pj = perm[(unsigned)__float_as_int(L.col[lp.bs].w) >> 6];
                if (apply) acc_add(acc, pj, v, g_i, dsc);
                if (out.sten_idx) keep_entry(out, i, at, pj, v);
                if (out.full_idx) {
                    out.full_idx[(size_t)i * VRM_KMAX + at] = pj;
                    out.full_f[(size_t)i * VRM_KMAX + at] = v;
                }
            }
            if (M == 3) {
                if (s == 0) out.status[i] = 1;   // removed
            } else if (s == 0) {
                if (apply) acc_add(acc, i, fii, g_i, dsc);
                if (out.full_k) {
                    out.full_k[i] = nz;
                    out.fii[i] = fii;
                    out.status[i] = VRM_ST_FULL;
                }
            }
            if (out.prev) {
                // the basic columns' ids, by column, as the particle's basis
                const int own = ids[t];
                if ((unsigned)own < (unsigned)out.prev_cap) {
                    const int b = lp.row_lane() && lp.bs < lp.ART ? lp.bs : 0x7fffffff;
                    int before = 0;
                    sfor<M>([&](auto r) { before += bc<r>(b) < b ? 1 : 0; });
                    const int have = __popc(lp.votes(b != 0x7fffffff));
                    if (b != 0x7fffffff)
                        out.prev[(size_t)own * kPrevIds + before] = ids[(unsigned)__float_as_int(L.col[b].w) >> 6];
                    if (s >= have && s < kPrevIds) out.prev[(size_t)own * kPrevIds + s] = -1;
                }
            }
        } else if (M != 3 && s == 0 && out.status) {
            out.status[i] = VRM_ST_INFEASIBLE;
        }
        if (s == 0) {
            if (out.sten_idx) keep_end(out, i, st == 0 ? nz : -1, fii);
            // no basis of the small neighbourhood: a mask of an earlier step must not
            // decide how the next stage solves this LP (its last bits depend on that)
            if (M == 5 && out.seg_mask) out.seg_mask[i] = 0;
            if (piv) atomicAdd(&s_cnt[kPiv], piv);
            if (st == 0) {
                atomicAdd(&s_cnt[kCols], k);
                atomicAdd(&s_cnt[kFull], 1);
                if (!certified) atomicAdd(&s_cnt[kUnc], 1);
            } else {
                atomicAdd(&s_cnt[kInf], 1);
            }
            if (truncated) atomicAdd(&s_cnt[kTrunc], 1);
            if constexpr (M == 9) {
                atomicAdd(&s_cnt[kRounds], lp.cert_rounds);
                if (lp.cert_exact) atomicAdd(&s_cnt[kExact], 1);
            }
        }
    }
    __syncthreads();
    if constexpr (M == 3) {
        if (tid == 0 && s_cnt[kUnc]) atomicAdd(&qs->n_rm_uncertified, s_cnt[kUnc]);
        return;
    }
    if (tid < kCounts && s_cnt[tid]) {
        vrm_counters* c = counter_stripe(cnt);
        int64_t* to[kCounts] = {&c->pivots, &c->full_cols, &c->n_full, &c->n_infeasible, &c->n_uncertified,
                                &c->n_truncated, &c->cert_rounds, &c->cert_exact};
        int64_t* p = to[0];
#pragma unroll
        for (int q = 1; q < kCounts; ++q) p = tid == q ? to[q] : p;
        atomicAdd(reinterpret_cast<unsigned long long*>(p), (unsigned long long)s_cnt[tid]);
        if (tid == kFull && apply)
            atomicAdd(reinterpret_cast<unsigned long long*>(&c->redistributions), (unsigned long long)s_cnt[kFull]);
    }
    // The last LP launch of a stencil run: its last workgroup empties the queues.  Every
    // workgroup has used the count by then, and nothing else of the launch touches them.
    if (tid == 0 && last_block(qs)) {
        qs->last_small = qs->n_small;
        qs->last_full = qs->n_full;
        qs->n_small = 0;
        qs->n_full = 0;
        qs->n_retry = 0;
        qs->n_defer = 0;
    }
}

}  // namespace

// The removal's identity LPs: of the slots in `taken` (n_accepted of the queues), with
// removed[particle] set where the circulation was given away.  One thread per LP with
// its columns in LDS (three waves per CU) took 154 us for a removal from 2.7M particles
// (one particle in twenty close to another), now 95; three waves per SIMD 115.
int vrm_rm_lp_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const LaunchParams& lp, const int32_t* taken,
                  uint8_t* removed, bool stored)
{
    StencilOut out{};
    out.status = removed;
    const int grid = std::max(1, std::min((n + kGGroups - 1) / kGGroups, 5 * 256));
    hipLaunchKernelGGL(k_lp_group<3>, dim3(grid), dim3(kGBlock), 0, c->stream, c->perm, c->xs, c->ys, c->ids,
                       c->cell_start, c->grid, taken, c->queues, cl->gamma_dev, c->acc, lp, out, 1, c->counters,
                       stored ? VRM_KMAX : 0, VRM_KMAX, (const int32_t*)nullptr, 0);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

// Canonical stencils, cold.  stored: the one-thread kernel of the same cloud keeps its costs.
int vrm_lp_group_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const LaunchParams& lp, const StencilOut& out,
                     int apply, bool stored, int limit, int max_blocks)
{
    const int grid = std::max(1, std::min((n + kGGroups - 1) / kGGroups, max_blocks));
    const int exact_n = lp.m == 9 ? kSiftW : (stored ? VRM_KMAX : 0);
    const int work = lp.m == 9 ? kSiftW : VRM_KMAX;
    hipLaunchKernelGGL((lp.m == 9 ? k_lp_group<9> : k_lp_group<5>), dim3(grid), dim3(kGBlock), 0, c->stream, c->perm,
                       c->xs, c->ys, c->ids, c->cell_start, c->grid, c->q_full, c->queues, cl->gamma_dev, c->acc, lp,
                       out, apply, c->counters, exact_n, work, c->q_retry, limit);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}
