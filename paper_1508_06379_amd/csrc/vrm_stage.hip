// Runge-Kutta stage combination, FP64 verification and the prescribed
// velocity harness of libvrm.
//
// Stage update: Sec. 3.3 (Euler steps; SSP Runge-Kutta schemes are convex
// combinations of them) with the Shu-Osher SSP-RK3 weights, applied to
// Gamma with dGamma_i/dt = nu sum_j f_ji Gamma_j (Sec. 3.4, eq. nsode) and to
// the positions with the caller's velocity.
#include <hip/hip_runtime.h>

#include "vrm_device.h"
#include "vrm_internal.h"

using namespace vrm;

namespace {

// n_dev (optional): the particle count read on the device (graph replays), else n.
// det: the accumulator holds 64-bit fixed-point sums (scale det_scale).  While a
// non-finite value is flagged the accumulator is cleared and the cloud is left
// as it is.
__global__ __launch_bounds__(256) void k_combine(int n, const int32_t* __restrict__ n_dev, float a, float b, float dt,
                                                 float lam, const float* __restrict__ x0, const float* __restrict__ y0,
                                                 const float* __restrict__ g0, float* x, float* y, float* g,
                                                 const float* __restrict__ u, const float* __restrict__ v, float* acc,
                                                 const GridState* gs, int det)
{
    if (n_dev) n = *n_dev;
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float sum;
    if (det) {
        unsigned long long* acc64 = reinterpret_cast<unsigned long long*>(acc);
        const long long w = (long long)acc64[i];
        acc64[i] = 0ull;
        sum = (float)((double)w * (1.0 / det_scale(gs->gmax_bits)));
    } else {
        sum = acc[i];
        acc[i] = 0.0f;
    }
    if (gs->bad) return;
    g[i] = combined_gamma(a, b, dt, lam * sum, g[i], a != 0.0f ? g0[i] : 0.0f);
    if (u) {
        float xn = __builtin_fmaf(dt, u[i], x[i]);
        float yn = __builtin_fmaf(dt, v[i], y[i]);
        float xs = b * xn, ys = b * yn;
        if (a != 0.0f) {
            xs = __builtin_fmaf(a, x0[i], xs);
            ys = __builtin_fmaf(a, y0[i], ys);
        }
        x[i] = xs;
        y[i] = ys;
    } else if (a != 0.0f) {
        // zero velocity: positions stay exactly y^n (the convex combination is the identity)
        x[i] = x0[i];
        y[i] = y0[i];
    }
}

// FP64 moment residual of each stencil (rows 1 <= |alpha| <= q, relative to
// b = 2), circulation and l1 norm, and the largest sum_j fhat_ij.
__global__ __launch_bounds__(256) void k_verify(int n, const float* __restrict__ x, const float* __restrict__ y,
                                                const float* __restrict__ g, double h, int q,
                                                const int32_t* __restrict__ sidx, const float* __restrict__ sf,
                                                const uint8_t* __restrict__ status, const int32_t* __restrict__ fk,
                                                const int32_t* __restrict__ fidx, const float* __restrict__ ff,
                                                unsigned long long* out)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    double res = 0.0, i0 = 0.0, l1 = 0.0, fsum = 0.0;
    if (i < n) {
        double gi = (double)g[i];
        i0 = gi;
        l1 = fabs(gi);
        int st = status ? status[i] : 3;
        if (st == VRM_ST_WARM) st = (fk && fk[i] > 0) ? 1 : 0;   // warm-started: small or complete
        if (st <= 1) {
            double m[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            double xi = (double)x[i], yi = (double)y[i];
            int k = st == 0 ? VRM_NSEG : fk[i];
            for (int t = 0; t < k; ++t) {
                int j;
                double f;
                if (st == 0) {
                    j = sidx[(size_t)i * VRM_NSEG + t];
                    f = (double)sf[(size_t)i * VRM_NSEG + t];
                } else {
                    j = fidx[(size_t)i * VRM_KMAX + t];
                    f = (double)ff[(size_t)i * VRM_KMAX + t];
                }
                if (j < 0) continue;
                double rx = ((double)x[j] - xi) / h, ry = ((double)y[j] - yi) / h;
                m[0] += f * rx;
                m[1] += f * ry;
                m[2] += f * rx * rx;
                m[3] += f * rx * ry;
                m[4] += f * ry * ry;
                m[5] += f * rx * rx * rx;
                m[6] += f * rx * rx * ry;
                m[7] += f * rx * ry * ry;
                m[8] += f * ry * ry * ry;
                fsum += f;
            }
            m[2] -= 2.0;
            m[4] -= 2.0;
            int rows = q == 2 ? 5 : 9;
            for (int a = 0; a < rows; ++a) res = fmax(res, fabs(m[a]) / 2.0);
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        res = fmax(res, __shfl_xor(res, o, VRM_WAVE));
        fsum = fmax(fsum, __shfl_xor(fsum, o, VRM_WAVE));
        i0 += __shfl_xor(i0, o, VRM_WAVE);
        l1 += __shfl_xor(l1, o, VRM_WAVE);
    }
    if (lane_id() == 0) {
        atomicMax(&out[0], (unsigned long long)__double_as_longlong(res));
        atomicAdd((double*)&out[1], i0);
        atomicAdd((double*)&out[2], l1);
        atomicMax(&out[3], (unsigned long long)__double_as_longlong(fsum));
    }
}

// y^n of the step; also flags a non-finite circulation (kBadGamma) and, for the
// fixed-point accumulation (det), finds max |Gamma^n| (k_gmax_reset first)
__global__ __launch_bounds__(256) void k_save_base(int n, const int32_t* __restrict__ n_dev,
                                                   const float* __restrict__ x, const float* __restrict__ y,
                                                   const float* __restrict__ g, float* x0, float* y0, float* g0,
                                                   GridState* gs, int det)
{
    if (n_dev) n = *n_dev;
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t bits = 0u;
    if (i < n) {
        const float gi = g[i];
        x0[i] = x[i];
        y0[i] = y[i];
        g0[i] = gi;
        bits = __float_as_uint(fabsf(gi));
    }
    if (__any(bits >= 0x7f800000u) && lane_id() == 0) atomicOr(&gs->bad, kBadGamma);
    if (det) {
        // an atomic only where it raises the value just read: one of every wave on the one
        // address took 291 us for 1M particles, now 35
        if (bits >= 0x7f800000u) bits = 0u;
        for (int o = 32; o > 0; o >>= 1) bits = max(bits, (uint32_t)__shfl_xor((int)bits, o, VRM_WAVE));
        __shared__ uint32_t wave_max[4];
        if (lane_id() == 0) wave_max[threadIdx.x >> 6] = bits;
        __syncthreads();
        if (threadIdx.x == 0) {
            bits = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
            if (bits > __hip_atomic_load(&gs->gmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&gs->gmax_bits, bits);
        }
    }
}

__global__ void k_gmax_reset(GridState* gs) { gs->gmax_bits = 0u; }

__global__ void k_verify_init(unsigned long long* out)
{
    out[0] = 0ull;
    out[1] = 0ull;
    out[2] = 0ull;
    out[3] = 0ull;
}

// Prescribed velocity of Lamb-Oseen vortices (centre, core sigma, circulation G):
// u(x) = sum_k G_k (-d_y, d_x) (1 - exp(-|d|^2 / (sigma_k^2 + 4 nu t))) / (2 pi |d|^2),
// d = x - centre_k, and 0 at a centre.  Time = t, or *t_dev + t when t_dev is
// given (graph replays).  Each thread holds kVelT targets, so the per-vortex
// constants a = G / (2 pi) and b = log2(e) / (sigma^2 + 4 nu t) (one hardware
// reciprocal) are paid once per kVelT pairs; a pair costs two differences, two
// FMAs for |d|^2, exp2(-b |d|^2), a reciprocal of |d|^2, one product, one FMA
// for t - t e, a select and two accumulating FMAs, with no IEEE division.
// A pair with |d|^2 <= 1e-30 (a target on a centre) contributes 0.
constexpr int kVelT = 4;

__global__ __launch_bounds__(256) void k_velocity(int n, const int32_t* __restrict__ n_dev,
                                                  const float* __restrict__ x, const float* __restrict__ y,
                                                  const float* __restrict__ vort, int nv, double nu, double t,
                                                  const double* __restrict__ t_dev, float* u, float* v)
{
    if (n_dev) n = *n_dev;
    const int base = blockIdx.x * (256 * kVelT) + threadIdx.x;
    if (base >= n) return;
    const double tt = t_dev ? *t_dev + t : t;
    const float four_nu_t = (float)(4.0 * nu * tt);
    const float inv2pi = 0.15915494309189535f, log2e = 1.4426950408889634f;
    float xi[kVelT], yi[kVelT], su[kVelT], sv[kVelT];
#pragma unroll
    for (int j = 0; j < kVelT; ++j) {
        const int i = min(base + 256 * j, n - 1);
        xi[j] = x[i];
        yi[j] = y[i];
        su[j] = 0.0f;
        sv[j] = 0.0f;
    }
    for (int k = 0; k < nv; ++k) {
        const float cx = vort[4 * k], cy = vort[4 * k + 1], s = vort[4 * k + 2];
        const float a = vort[4 * k + 3] * inv2pi;
        const float b = -log2e * __builtin_amdgcn_rcpf(__builtin_fmaf(s, s, four_nu_t));
#pragma unroll
        for (int j = 0; j < kVelT; ++j) {
            const float dx = xi[j] - cx, dy = yi[j] - cy;
            const float r2 = __builtin_fmaf(dx, dx, dy * dy);
            const float ex = __builtin_amdgcn_exp2f(b * r2);
            const float tr = __builtin_amdgcn_rcpf(r2) * a;
            const float f = r2 > 1e-30f ? __builtin_fmaf(-tr, ex, tr) : 0.0f;
            su[j] = __builtin_fmaf(-f, dy, su[j]);
            sv[j] = __builtin_fmaf(f, dx, sv[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < kVelT; ++j) {
        const int i = base + 256 * j;
        if (i < n) {
            u[i] = su[j];
            v[i] = sv[j];
        }
    }
}

int blocks_for(int n) { return n > 0 ? (n + 255) / 256 : 1; }

}  // namespace

int vrm_combine_run(vrm_ctx* c, vrm_cloud* cl, int32_t n, const float* u, const float* v, double dt, float lam,
                    int stage, int det)
{
    if (n <= 0) return VRM_OK;
    hipLaunchKernelGGL(k_combine, dim3(blocks_for(n)), dim3(256), 0, c->stream, n, cl->n_dev, kStageA[stage], kStageB[stage],
                       (float)dt, lam, c->x0, c->y0, c->g0, cl->x_dev, cl->y_dev, cl->gamma_dev, u, v, c->acc, c->grid,
                       det);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

int vrm_save_base_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, int det)
{
    if (n <= 0) return VRM_OK;
    if (det) hipLaunchKernelGGL(k_gmax_reset, dim3(1), dim3(1), 0, c->stream, c->grid);
    hipLaunchKernelGGL(k_save_base, dim3(blocks_for(n)), dim3(256), 0, c->stream, n, cl->n_dev, cl->x_dev, cl->y_dev,
                       cl->gamma_dev, c->x0, c->y0, c->g0, c->grid, det);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

int vrm_verify_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const LaunchParams& lp, double h,
                   const vrm_stencils* st, double* report)
{
    unsigned long long* out = reinterpret_cast<unsigned long long*>(report);
    hipLaunchKernelGGL(k_verify_init, dim3(1), dim3(1), 0, c->stream, out);
    if (n > 0) {
        hipLaunchKernelGGL(k_verify, dim3(blocks_for(n)), dim3(256), 0, c->stream, n, cl->x_dev, cl->y_dev,
                           cl->gamma_dev, h, lp.q, st ? st->small_idx_dev : nullptr,
                           st ? st->small_f_dev : nullptr, st ? st->status_dev : nullptr,
                           st ? st->full_k_dev : nullptr, st ? st->full_idx_dev : nullptr,
                           st ? st->full_f_dev : nullptr, out);
    }
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

int vrm_velocity_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const float* vort, int32_t nv, double nu, double t,
                     float* u, float* v, const double* t_dev)
{
    if (n <= 0) return VRM_OK;
    hipLaunchKernelGGL(k_velocity, dim3((n + 256 * kVelT - 1) / (256 * kVelT)), dim3(256), 0, c->stream, n, cl->n_dev, cl->x_dev, cl->y_dev,
                       vort, nv, nu, t, t_dev, u, v);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}
