// Parameter-vector kernels of the PCG solve (Alg. 2), the preconditioner (Sec. III-G) and
// the line search (Alg. 3).  One thread handles one unit (float4 = the 4 parameters of a
// voxel or texel) in a grid-stride loop over a fixed grid of kVecGrid workgroups, so every
// dot product is reduced the same way on every call: FP64 per-thread sums, FP64 wave and
// workgroup reduction, one partial per workgroup.  The kernel that needs the sum adds the partials
// itself, every workgroup in the same order: at most 16 KB from L2 each, where a launch of its own
// takes 4.6 us.  A PCG iteration is then J^T J v and three vector kernels (k_dot, k_pcg_update,
// k_pcg_direction); with the sums and the clearing of A p in launches of their own it was six, 29 us
// at 32^3 where J^T J v takes 165.  All PCG scalars stay on the device, one row of `hist` per
// iteration, so that no workgroup overwrites what another still reads; the stop rules of Alg. 2
// are evaluated there and raise a flag that every later kernel of the solve checks, so the
// host can enqueue a whole solve without reading anything back.
#include "perf_internal.h"

#include <math.h>

namespace perf {
namespace {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Workgroup sum of two doubles; thread 0 stores them.
__device__ __forceinline__ void block_sum2(double a, double b, double* oa, double* ob) {
    __shared__ double red[2][kVecBlock / 64];
    a = wave_sum(a);
    b = wave_sum(b);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        red[0][wave] = a;
        red[1][wave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int i = 0; i < kVecBlock / 64; ++i) {
            sa += red[0][i];
            sb += red[1][i];
        }
        if (oa) *oa = sa;
        if (ob) *ob = sb;
    }
}

// Sum of n partials by one workgroup of BLOCK threads in a fixed order (deterministic).
template <int BLOCK>
__device__ __forceinline__ double fixed_order_sum(const double* p, int64_t n) {
    __shared__ double red[BLOCK / 64];
    double s[4] = {0.0, 0.0, 0.0, 0.0};  // four loads in flight
    for (int64_t i = threadIdx.x; i < n; i += 4 * BLOCK) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k * BLOCK < n) s[k] += p[i + k * BLOCK];
    }
    const double w = wave_sum((s[0] + s[1]) + (s[2] + s[3]));
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) red[wave] = w;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < BLOCK / 64; ++i) t += red[i];
    return t;
}

__device__ __forceinline__ double dot4(float4 a, float4 b) {
    return (double)a.x * b.x + (double)a.y * b.y + (double)a.z * b.z + (double)a.w * b.w;
}

// z = M^-1 r for one unit, from the preconditioner in scaled form.  Every stored value stays in
// FP32 range whatever the scale of the block (t = D^-1/2 is at most the inverse square root of
// the smallest subnormal), and the unscaled inverse is never formed.
//   Jacobi   t per parameter: z = t (t r).
//   Block    (t_d, t_f, e~, 1/s): D^-1/2 = diag(t_d, t_d, t_d, t_f), the normalised block
//            [[I, e~], [e~^T, 1]] and its Schur complement s = 1 - |e~|^2; with y = D^-1/2 r the
//            block is solved by elimination, z_sigma = (y_sigma - e~ . y_c) / s,
//            z_c = y_c - e~ z_sigma, then z = D^-1/2 z.  Elimination keeps the FP32 rounding
//            error along the block's own near-null direction; multiplying by the explicit
//            inverse, whose entries reach 1/s, would spread it over every direction.
//   Learned  (t_d, t_f, L row by row): z = D^-1/2 L (L^T (D^-1/2 r)); a unit on the exact-block
//            fallback holds the block form (-t_d, t_f, e~, 1/s) instead, told apart by t_d < 0.
template <int KIND>
__device__ __forceinline__ float4 precond_apply(const float* __restrict__ minv, int64_t u, float4 r) {
    if constexpr (KIND == PERF_PRECOND_NONE) {
        return r;
    } else if constexpr (KIND == PERF_PRECOND_JACOBI) {
        const float4 t = reinterpret_cast<const float4*>(minv)[u];
        return make_float4(t.x * (t.x * r.x), t.y * (t.y * r.y), t.z * (t.z * r.z), t.w * (t.w * r.w));
    } else if constexpr (KIND == PERF_PRECOND_BLOCK4) {
        const float4* q = reinterpret_cast<const float4*>(minv) + 2 * u;
        const float4 q0 = q[0], q1 = q[1];
        const float td = q0.x, tf = q0.y, e0 = q0.z, e1 = q0.w, e2 = q1.x, is = q1.y;
        const float y0 = td * r.x, y1 = td * r.y, y2 = td * r.z, y3 = tf * r.w;
        const float zs = (y3 - (e0 * y0 + e1 * y1 + e2 * y2)) * is;
        return make_float4(td * (y0 - e0 * zs), td * (y1 - e1 * zs), td * (y2 - e2 * zs), tf * zs);
    } else {
        const float4* q = reinterpret_cast<const float4*>(minv) + 3 * u;
        const float4 q0 = q[0], q1 = q[1];
        if (q0.x < 0.0f) {
            // a unit on the exact-block fallback: the block form, with t_d stored negated
            const float td = -q0.x, tf = q0.y, e0 = q0.z, e1 = q0.w, e2 = q1.x, is = q1.y;
            const float y0 = td * r.x, y1 = td * r.y, y2 = td * r.z, y3 = tf * r.w;
            const float zs = (y3 - (e0 * y0 + e1 * y1 + e2 * y2)) * is;
            return make_float4(td * (y0 - e0 * zs), td * (y1 - e1 * zs), td * (y2 - e2 * zs), tf * zs);
        }
        const float4 q2 = q[2];
        const float td = q0.x, tf = q0.y;
        const float l00 = q0.z, l10 = q0.w, l11 = q1.x, l20 = q1.y, l21 = q1.z, l22 = q1.w, l30 = q2.x, l31 = q2.y,
                    l32 = q2.z, l33 = q2.w;
        const float y0 = td * r.x, y1 = td * r.y, y2 = td * r.z, y3 = tf * r.w;
        // w = L^T y, then v = L w
        const float w0 = l00 * y0 + l10 * y1 + l20 * y2 + l30 * y3;
        const float w1 = l11 * y1 + l21 * y2 + l31 * y3;
        const float w2 = l22 * y2 + l32 * y3;
        const float w3 = l33 * y3;
        return make_float4(td * (l00 * w0), td * (l10 * w0 + l11 * w1), td * (l20 * w0 + l21 * w1 + l22 * w2),
                           tf * (l30 * w0 + l31 * w1 + l32 * w2 + l33 * w3));
    }
}

__global__ void k_zero(float* __restrict__ p, int64_t n, float* __restrict__ q, int64_t m) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0.0f;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += stride) q[i] = 0.0f;
}

__global__ void k_zero_u64(unsigned long long* p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

// One partial per ray workgroup: 125 000 for 16 M rays took a workgroup of 256 threads 150 us.
constexpr int kSumBlock = 1024;
__global__ __launch_bounds__(kSumBlock) void k_sum_partials(const double* p, int64_t n, double scale, double* out) {
    const double s = fixed_order_sum<kSumBlock>(p, n);
    if (threadIdx.x == 0) *out = scale * s;
}

// The objective of line-search trial j of a batch into mu[j]; raises *done when it exceeds the trial
// before (prev for the first of the batch), which ends the search (Alg. 3).
__global__ __launch_bounds__(kSumBlock) void k_sum_trial(const double* p, int64_t n, int j, double prev, double* mu,
                                                         int* done) {
    if (j > 0 && *done) return;
    const double s = 0.5 * fixed_order_sum<kSumBlock>(p, n);
    if (threadIdx.x == 0) {
        mu[j] = s;
        if (s > (j > 0 ? mu[j - 1] : prev)) *done = 1;
    }
}

// Scaled form of the preconditioner (Sec. III-G) from the blocks [[d I, e], [e^T, f]], FP64 inside.
// Jacobi: (t_d, t_d, t_d, t_f) with t = 1/sqrt(diagonal), 0 for a zero diagonal, so that
// M^-1 = t^2 = 1/diag(J^T J).  Block: after a ridge rho = 1e-6 max(d, f), t_d = (d + rho)^-1/2,
// t_f = (f + rho)^-1/2, the normalised coupling e~ = t_d t_f e and 1/s with s = 1 - |e~|^2, the
// Schur complement of the normalised block [[I, e~], [e~^T, 1]]: (t_d, t_f, e~, 1/s, 0, 0).
__device__ __forceinline__ void invert_unit(int kind, const float b[5], int64_t u, float* __restrict__ out) {
    const double d = b[0], e0 = b[1], e1 = b[2], e2 = b[3], f = b[4];
    if (kind == PERF_PRECOND_JACOBI) {
        const float td = d > 0.0 ? (float)(1.0 / sqrt(d)) : 0.0f;
        const float tf = f > 0.0 ? (float)(1.0 / sqrt(f)) : 0.0f;
        reinterpret_cast<float4*>(out)[u] = make_float4(td, td, td, tf);
    } else {
        float4* o = reinterpret_cast<float4*>(out) + 2 * u;
        const double m = fmax(d, f);
        if (!(m > 0.0) || !isfinite(d + e0 + e1 + e2 + f)) {  // no ray, or a non-finite block
            o[0] = o[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            return;
        }
        const double rho = 1e-6 * m;
        const double td = 1.0 / sqrt(d + rho), tf = 1.0 / sqrt(f + rho);
        const double a0 = e0 * td * tf, a1 = e1 * td * tf, a2 = e2 * td * tf;
        const double is = 1.0 / (1.0 - (a0 * a0 + a1 * a1 + a2 * a2));
        o[0] = make_float4((float)td, (float)tf, (float)a0, (float)a1);
        o[1] = make_float4((float)a2, (float)is, 0.0f, 0.0f);
    }
}

__global__ void k_invert(int kind, const float* __restrict__ blocks, int64_t units, float* __restrict__ out) {
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < units; u += (int64_t)gridDim.x * blockDim.x) {
        float b[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) b[i] = blocks[5 * u + i];
        invert_unit(kind, b, u, out);
    }
}

__global__ void k_finish_grad(int kind, const double* __restrict__ grad64, const double* __restrict__ blocks64,
                              int64_t units, float* __restrict__ grad, float* __restrict__ blocks,
                              float* __restrict__ out) {
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < units; u += (int64_t)gridDim.x * blockDim.x) {
        if (grad) {
            const double* g = grad64 + 4 * u;
            float* o = grad + 4 * u;  // (no alignment beyond a float's is asked of the caller)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (float)g[i];
        }
        if (blocks) {
            float b[5];
#pragma unroll
            for (int i = 0; i < 5; ++i) blocks[5 * u + i] = b[i] = (float)blocks64[5 * u + i];
            if (out && kind != PERF_PRECOND_NONE) invert_unit(kind, b, u, out);
        }
    }
}

// r = b, z = M^-1 r, p = z, delta = 0, Ap = 0; partials of r.r and r.z
template <int KIND>
__global__ void k_pcg_init(const float4* __restrict__ b, const float* __restrict__ minv, float4* __restrict__ r,
                           float4* __restrict__ z, float4* __restrict__ p, float4* __restrict__ delta,
                           float4* __restrict__ Ap, int64_t units, double* partials) {
    double rr = 0.0, rz = 0.0;
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < units; u += (int64_t)gridDim.x * blockDim.x) {
        const float4 ru = b[u];
        const float4 zu = precond_apply<KIND>(minv, u, ru);
        r[u] = ru;
        z[u] = zu;
        p[u] = zu;
        delta[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        Ap[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        rr += dot4(ru, ru);
        rz += dot4(ru, zu);
    }
    block_sum2(rr, rz, partials + blockIdx.x, partials + gridDim.x + blockIdx.x);
}

__global__ void k_pcg_init_fin(const double* partials, int64_t nb, double* sc, double* hist, int* fl) {
    const double rr = fixed_order_sum<kVecBlock>(partials, nb);
    const double rz = fixed_order_sum<kVecBlock>(partials + nb, nb);
    for (int i = threadIdx.x; i < kHistDoubles; i += kVecBlock)
        if (i != H_RZ) hist[i] = 0.0;
    if (threadIdx.x == 0) {
        sc[S_R0] = rr;
        hist[H_RZ] = rz;
        fl[I_ITERS] = 0;
        fl[I_DONE] = rr == 0.0 ? 1 : 0;
        fl[I_FLAGS] = rr == 0.0 ? PERF_FLAG_CONVERGED : 0;
    }
}

__global__ void k_dot(const float4* __restrict__ a, const float4* __restrict__ b, int64_t units, double* partials,
                      const int* done) {
    if (*done) return;
    double s = 0.0;
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < units; u += (int64_t)gridDim.x * blockDim.x)
        s += dot4(a[u], b[u]);
    block_sum2(s, 0.0, partials + blockIdx.x, nullptr);
}

// Whether the solve had ended, the same for the whole workgroup: workgroup 0 may raise the flag meanwhile.
__device__ __forceinline__ bool solve_done(const int* fl) {
    __shared__ int done;
    if (threadIdx.x == 0) done = fl[I_DONE];
    __syncthreads();
    return done != 0;
}

// With one readback, and the product's events taken from its dispatch, a step of 3 iterations on 32^3
// voxels went from 1143 to 1058 us, on 64^3 from 5133 (5 iterations) to 4873.
// alpha from the partials of p.Ap; delta += alpha p; r -= alpha Ap; z = M^-1 r; Ap = 0 for the next
// product; partials of r.r and r.z
template <int KIND>
__global__ void k_pcg_update(const float* __restrict__ minv, float4* __restrict__ delta, float4* __restrict__ r,
                             float4* __restrict__ z, const float4* __restrict__ p, float4* __restrict__ Ap,
                             int64_t units, const double* dots, double* partials, double* hist, int* fl) {
    if (solve_done(fl)) return;
    const double pAp = fixed_order_sum<kVecBlock>(dots, gridDim.x);
    const bool broken = !(pAp > 0.0) || !isfinite(pAp);
    const double alpha = broken ? 0.0 : hist[H_RZ] / pAp;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        hist[H_PAP] = pAp;
        hist[H_ALPHA] = alpha;
        if (broken) {
            fl[I_FLAGS] |= PERF_FLAG_BREAKDOWN;
            fl[I_DONE] = 1;  // (a workgroup that sees it early would have stopped here too)
        }
    }
    if (broken) return;
    const float a = (float)alpha;
    double rr = 0.0, rz = 0.0;
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < units; u += (int64_t)gridDim.x * blockDim.x) {
        const float4 pu = p[u], Apu = Ap[u];
        float4 d = delta[u], ru = r[u];
        d.x += a * pu.x; d.y += a * pu.y; d.z += a * pu.z; d.w += a * pu.w;
        ru.x -= a * Apu.x; ru.y -= a * Apu.y; ru.z -= a * Apu.z; ru.w -= a * Apu.w;
        const float4 zu = precond_apply<KIND>(minv, u, ru);
        delta[u] = d;
        r[u] = ru;
        z[u] = zu;
        Ap[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        rr += dot4(ru, ru);
        rz += dot4(ru, zu);
    }
    block_sum2(rr, rz, partials + blockIdx.x, partials + gridDim.x + blockIdx.x);
}

// R and beta of iteration `it` from the partials, the stop rules (Alg. 2), then p = z + beta p
__global__ void k_pcg_direction(const float4* __restrict__ z, float4* __restrict__ p, int64_t units,
                                const double* partials, int it, PcgStop stop, const double* sc, double* hist, int* fl) {
    if (solve_done(fl)) return;
    const double R = fixed_order_sum<kVecBlock>(partials, gridDim.x);
    const double rz_new = fixed_order_sum<kVecBlock>(partials + gridDim.x, gridDim.x);
    const double R_prev = it > 0 ? hist[H_R - H_COUNT] : sc[S_R0];
    const double beta = rz_new / hist[H_RZ];
    int done = 0, flag = 0;
    if (stop.abs_eps > 0.0 && R < stop.abs_eps) {
        done = 1;
        flag = PERF_FLAG_CONVERGED;
    } else if (stop.rel_tol > 0.0 && sqrt(R / sc[S_R0]) <= stop.rel_tol) {
        done = 1;
        flag = PERF_FLAG_CONVERGED;
    } else if (stop.stall > 0.0 && R / R_prev > stop.stall) {
        done = 1;
        flag = PERF_FLAG_STALL;
    } else if (it + 1 >= stop.max_iters) {
        done = 1;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        hist[H_R] = R;
        fl[I_ITERS] = it + 1;
        if (done) {
            fl[I_FLAGS] |= flag;
            fl[I_DONE] = 1;  // (a workgroup that sees it early would have stopped here too)
        } else {
            hist[H_BETA] = beta;
            hist[H_COUNT + H_RZ] = rz_new;
        }
    }
    if (done) return;
    const float b = (float)beta;
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < units; u += (int64_t)gridDim.x * blockDim.x) {
        const float4 zu = z[u];
        float4 pu = p[u];
        pu.x = zu.x + b * pu.x;
        pu.y = zu.y + b * pu.y;
        pu.z = zu.z + b * pu.z;
        pu.w = zu.w + b * pu.w;
        p[u] = pu;
    }
}

__device__ __forceinline__ unsigned short f32_to_bf16_rne(float f) {
    const unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);  // quiet NaN
    const unsigned r = u + 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(r >> 16);
}

// xt = proj(x + gamma delta): sigma >= 0 on voxels, alpha in [0,1] on texels
// done: a line search that has ended skips the trial; with `first` the search (batch) starts here.
__global__ void k_trial(const float4* __restrict__ x, const float4* __restrict__ delta, float gamma, int64_t units,
                        int nvox, float4* __restrict__ xt, ushort4* __restrict__ xb, int* done, bool first) {
    if (done && first && blockIdx.x == 0 && threadIdx.x == 0) *done = 0;
    if (done && !first && *done) return;
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < units; u += (int64_t)gridDim.x * blockDim.x) {
        float4 v = x[u];
        if (delta) {
            const float4 d = delta[u];
            v.x += gamma * d.x;
            v.y += gamma * d.y;
            v.z += gamma * d.z;
            v.w += gamma * d.w;
            v.w = (u < nvox) ? fmaxf(v.w, 0.0f) : fminf(fmaxf(v.w, 0.0f), 1.0f);
        }
        if (xt) xt[u] = v;
        if (xb) {
            ushort4 q;
            q.x = f32_to_bf16_rne(v.x);
            q.y = f32_to_bf16_rne(v.y);
            q.z = f32_to_bf16_rne(v.z);
            q.w = f32_to_bf16_rne(v.w);
            xb[u] = q;
        }
    }
}

__global__ void k_pack_bf16(const float* __restrict__ in, unsigned short* __restrict__ out, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = f32_to_bf16_rne(in[i]);
}

__global__ void k_check_finite(const float* __restrict__ p, int64_t n, int* flag) {
    int bad = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        bad |= !isfinite(p[i]);
    if (bad) atomicOr(flag, 1);
}

// features [units][PERF_MLP_NFEAT] from the parameters and the blocks of the gradient pass:
// sigma/alpha, colour (3), log d, log f
__device__ __forceinline__ float bf16f(unsigned short b) { return __uint_as_float(((unsigned)b) << 16); }

__global__ void k_features(const void* __restrict__ xp, int x_bf16, const float* __restrict__ blocks, int64_t units,
                           float* __restrict__ feat) {
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < units; u += (int64_t)gridDim.x * blockDim.x) {
        float4 xv;
        if (x_bf16) {
            const ushort4 q = reinterpret_cast<const ushort4*>(xp)[u];
            xv = make_float4(bf16f(q.x), bf16f(q.y), bf16f(q.z), bf16f(q.w));
        } else {
            xv = reinterpret_cast<const float4*>(xp)[u];
        }
        const float* b = blocks + 5 * u;
        float* f = feat + PERF_MLP_NFEAT * u;
        f[0] = xv.w;
        f[1] = xv.x;
        f[2] = xv.y;
        f[3] = xv.z;
        f[4] = logf(fmaxf(b[0], 0.0f) + 1e-12f);
        f[5] = logf(fmaxf(b[4], 0.0f) + 1e-12f);
    }
}

// Training rows of the learned preconditioner: every unit some ray touches (max(d, f) > 0) is
// kept with probability keep, decided by a counter-based hash of (seed, unit), and the kept
// rows are packed in unit order.  Workgroup g of a fixed grid owns one contiguous chunk of
// units: it counts its kept rows, one workgroup turns the counts into offsets, and each
// workgroup then writes its rows at its offset in order (deterministic output).
__device__ __forceinline__ unsigned mix32(unsigned h) {
    h ^= h >> 16;
    h *= 0x85ebca6bu;
    h ^= h >> 13;
    h *= 0xc2b2ae35u;
    h ^= h >> 16;
    return h;
}
// A row is eligible when some ray touches the unit and its block and features are finite (a unit
// whose parameters ran off during a poorly conditioned step can carry infinite sums).
__device__ __forceinline__ bool keep_row(const float* __restrict__ feat, const float* __restrict__ blocks, int64_t u,
                                         unsigned seed, unsigned thresh) {
    const float* b = blocks + 5 * u;
    bool ok = fmaxf(b[0], b[4]) > 0.0f;
#pragma unroll
    for (int i = 0; i < 5; ++i) ok &= isfinite(b[i]);
#pragma unroll
    for (int i = 0; i < PERF_MLP_NFEAT; ++i) ok &= isfinite(feat[PERF_MLP_NFEAT * u + i]);
    return ok && mix32(seed ^ mix32((unsigned)u ^ (unsigned)(u >> 32) * 0x9e3779b9u)) < thresh;
}

// kept rows of the workgroup's chunk before each thread's unit in this pass of the chunk
__device__ __forceinline__ int block_exclusive_count(bool flag, int* total) {
    __shared__ int wsum[kVecBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long bal = __ballot(flag);
    const int before_in_wave = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int before = before_in_wave, all = 0;
#pragma unroll
    for (int i = 0; i < kVecBlock / 64; ++i) {
        before += (i < wave) ? wsum[i] : 0;
        all += wsum[i];
    }
    __syncthreads();
    *total = all;
    return before;
}

__global__ __launch_bounds__(kVecBlock) void k_rows_count(const float* __restrict__ feat,
                                                          const float* __restrict__ blocks, int64_t units,
                                                          int64_t chunk, unsigned seed, unsigned thresh,
                                                          long long* counts) {
    const int64_t lo = blockIdx.x * chunk, hi = min(lo + chunk, units);
    long long c = 0;
    for (int64_t base = lo; base < hi; base += kVecBlock) {
        const int64_t u = base + threadIdx.x;
        int total;
        (void)block_exclusive_count(u < hi && keep_row(feat, blocks, u, seed, thresh), &total);
        c += total;
    }
    if (threadIdx.x == 0) counts[blockIdx.x] = c;
}

__global__ void k_rows_offsets(long long* counts, int nb) {
    if (threadIdx.x == 0) {
        long long run = 0;
        for (int i = 0; i < nb; ++i) {
            const long long c = counts[i];
            counts[i] = run;
            run += c;
        }
        counts[nb] = run;
    }
}

__global__ __launch_bounds__(kVecBlock) void k_rows_write(const float* __restrict__ feat, const float* __restrict__ blocks,
                                                          int64_t units, int64_t chunk, unsigned seed, unsigned thresh,
                                                          const long long* offsets, int64_t cap,
                                                          float* __restrict__ feat_out, float* __restrict__ blocks_out) {
    const int64_t lo = blockIdx.x * chunk, hi = min(lo + chunk, units);
    long long at = offsets[blockIdx.x];
    for (int64_t base = lo; base < hi; base += kVecBlock) {
        const int64_t u = base + threadIdx.x;
        const bool k = u < hi && keep_row(feat, blocks, u, seed, thresh);
        int total;
        const int before = block_exclusive_count(k, &total);
        const long long dst = at + before;
        if (k && dst < cap) {
#pragma unroll
            for (int i = 0; i < PERF_MLP_NFEAT; ++i) feat_out[PERF_MLP_NFEAT * dst + i] = feat[PERF_MLP_NFEAT * u + i];
#pragma unroll
            for (int i = 0; i < 5; ++i) blocks_out[5 * dst + i] = blocks[5 * u + i];
        }
        at += total;
    }
}

unsigned grid_for(int64_t n) {
    int64_t g = (n + kVecBlock - 1) / kVecBlock;
    if (g > kVecGrid) g = kVecGrid;
    if (g < 1) g = 1;
    return (unsigned)g;
}

}  // namespace

hipError_t launch_zero(float* p, int64_t n, hipStream_t st, float* q, int64_t m) {
    if (n <= 0 && m <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero, dim3(grid_for(n > m ? n : m)), dim3(kVecBlock), 0, st, p, n, q, m);
    return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long* p, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_u64, dim3(grid_for(n)), dim3(kVecBlock), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_sum_partials(const double* partials, int64_t n, double scale, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kSumBlock), 0, st, partials, n, scale, out);
    return hipGetLastError();
}

hipError_t launch_sum_trial(const double* partials, int64_t n, int j, double prev, double* mu, int* done, hipStream_t st) {
    hipLaunchKernelGGL(k_sum_trial, dim3(1), dim3(kSumBlock), 0, st, partials, n, j, prev, mu, done);
    return hipGetLastError();
}

hipError_t launch_finish_grad(int kind, const double* grad64, const double* blocks64, int64_t units, float* grad,
                              float* blocks, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_finish_grad, dim3(grid_for(units)), dim3(kVecBlock), 0, st, kind, grad64, blocks64, units, grad,
                       blocks, out);
    return hipGetLastError();
}

hipError_t launch_precond_invert(int kind, const float* blocks, int64_t units, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_invert, dim3(grid_for(units)), dim3(kVecBlock), 0, st, kind, blocks, units, out);
    return hipGetLastError();
}

namespace {

template <int KIND>
void pcg_init_kind(const PcgVectors& v, int64_t units, double* partials, unsigned g, hipStream_t st) {
    hipLaunchKernelGGL(k_pcg_init<KIND>, dim3(g), dim3(kVecBlock), 0, st, (const float4*)v.r, v.minv, (float4*)v.r,
                       (float4*)v.z, (float4*)v.p, (float4*)v.delta, (float4*)v.Ap, units, partials);
}

template <int KIND>
void pcg_update_kind(const PcgVectors& v, int64_t units, double* partials, double* hist, int* iflags, unsigned g,
                     hipStream_t st) {
    hipLaunchKernelGGL(k_pcg_update<KIND>, dim3(g), dim3(kVecBlock), 0, st, v.minv, (float4*)v.delta, (float4*)v.r,
                       (float4*)v.z, (const float4*)v.p, (float4*)v.Ap, units, partials + 2 * kVecGrid, partials, hist,
                       iflags);
}

}  // namespace

hipError_t launch_pcg_init(int kind, const PcgVectors& v, int64_t units, double* partials, double* scalars, double* hist,
                           int* iflags, hipStream_t st) {
    const unsigned g = grid_for(units);
    switch (kind) {
        case PERF_PRECOND_NONE: pcg_init_kind<PERF_PRECOND_NONE>(v, units, partials, g, st); break;
        case PERF_PRECOND_JACOBI: pcg_init_kind<PERF_PRECOND_JACOBI>(v, units, partials, g, st); break;
        case PERF_PRECOND_BLOCK4: pcg_init_kind<PERF_PRECOND_BLOCK4>(v, units, partials, g, st); break;
        default: pcg_init_kind<PERF_PRECOND_LEARNED>(v, units, partials, g, st); break;
    }
    hipLaunchKernelGGL(k_pcg_init_fin, dim3(1), dim3(kVecBlock), 0, st, partials, (int64_t)g, scalars, hist, iflags);
    return hipGetLastError();
}

// The vector part of iteration `it`, after Ap = A p: partials[0 .. 2g) hold r.r and r.z, those of p.Ap
// start at 2 kVecGrid.
hipError_t launch_pcg_iteration(int kind, const PcgVectors& v, int64_t units, int it, const PcgStop& stop,
                                double* partials, const double* scalars, double* hist, int* iflags, hipStream_t st) {
    const unsigned g = grid_for(units);
    double* row = hist + H_COUNT * it;
    hipLaunchKernelGGL(k_dot, dim3(g), dim3(kVecBlock), 0, st, (const float4*)v.p, (const float4*)v.Ap, units,
                       partials + 2 * kVecGrid, iflags + I_DONE);
    switch (kind) {
        case PERF_PRECOND_NONE: pcg_update_kind<PERF_PRECOND_NONE>(v, units, partials, row, iflags, g, st); break;
        case PERF_PRECOND_JACOBI: pcg_update_kind<PERF_PRECOND_JACOBI>(v, units, partials, row, iflags, g, st); break;
        case PERF_PRECOND_BLOCK4: pcg_update_kind<PERF_PRECOND_BLOCK4>(v, units, partials, row, iflags, g, st); break;
        default: pcg_update_kind<PERF_PRECOND_LEARNED>(v, units, partials, row, iflags, g, st); break;
    }
    hipLaunchKernelGGL(k_pcg_direction, dim3(g), dim3(kVecBlock), 0, st, (const float4*)v.z, (float4*)v.p, units,
                       (const double*)partials, it, stop, scalars, row, iflags);
    return hipGetLastError();
}

hipError_t launch_trial(const float* x, const float* delta, float gamma, int64_t units, int nvox, float* xt,
                        uint16_t* xb16, hipStream_t st, int* done, bool first) {
    hipLaunchKernelGGL(k_trial, dim3(grid_for(units)), dim3(kVecBlock), 0, st, reinterpret_cast<const float4*>(x),
                       reinterpret_cast<const float4*>(delta), gamma, units, nvox, reinterpret_cast<float4*>(xt),
                       reinterpret_cast<ushort4*>(xb16), done, first);
    return hipGetLastError();
}

hipError_t launch_pack_bf16(const float* in, uint16_t* out, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_bf16, dim3(grid_for(n)), dim3(kVecBlock), 0, st, in, out, n);
    return hipGetLastError();
}

hipError_t launch_check_finite(const float* p, int64_t n, int* flag, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_finite, dim3(grid_for(n)), dim3(kVecBlock), 0, st, p, n, flag);
    return hipGetLastError();
}

hipError_t launch_training_rows(const float* feat, const float* blocks, int64_t units, unsigned seed, float keep,
                                float* feat_out, float* blocks_out, int64_t cap, long long* counts, hipStream_t st) {
    const int nb = kVecGrid;
    const int64_t chunk = (units + nb - 1) / nb;
    const double t = fmin(fmax((double)keep, 0.0), 1.0) * 4294967296.0;
    const unsigned thresh = t >= 4294967295.0 ? 0xffffffffu : (unsigned)t;
    hipLaunchKernelGGL(k_rows_count, dim3(nb), dim3(kVecBlock), 0, st, feat, blocks, units, chunk, seed, thresh,
                       counts);
    hipLaunchKernelGGL(k_rows_offsets, dim3(1), dim3(64), 0, st, counts, nb);
    hipLaunchKernelGGL(k_rows_write, dim3(nb), dim3(kVecBlock), 0, st, feat, blocks, units, chunk, seed, thresh, counts,
                       cap, feat_out, blocks_out);
    return hipGetLastError();
}

hipError_t launch_unit_features(const void* x, int x_dtype, const float* blocks, int64_t units, float* feat,
                                hipStream_t st) {
    hipLaunchKernelGGL(k_features, dim3(grid_for(units)), dim3(kVecBlock), 0, st, x, x_dtype == PERF_BF16 ? 1 : 0,
                       blocks, units, feat);
    return hipGetLastError();
}

}  // namespace perf
