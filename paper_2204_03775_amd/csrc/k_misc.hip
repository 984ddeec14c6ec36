// Kernels outside the time step: the k range check at set-up, batch
// counter clearing, and the adjoint run's receiver injection, misfit
// reduction and gradient output.

#include "wave_dev.h"
#include "wave_kernels.h"

namespace wavek {

// Adds k * trace_grad[row][r] at the receiver cells: one thread per distinct
// cell, summing its receivers in a fixed order (deterministic, no atomics).
// Only phi^nt needs it; the adjoint steps add their own level's.
__global__ void inject_receivers(float *phi, const float *__restrict__ k, const long long *__restrict__ cell_off,
                                 const int *__restrict__ cell_start, const int *__restrict__ cell_rec,
                                 int ncells, const float *__restrict__ tg_row)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncells)
        return;
    float s = 0.f;
    for (int i = cell_start[c]; i < cell_start[c + 1]; ++i)
        s += tg_row[cell_rec[i]];
    const long long o = cell_off[c];
    phi[o] = fmaf(k[o], s, phi[o]);
}

// The source value of the forward step that made this level is k at the
// source cell times a fixed wavelet value, so its derivative with respect to
// that k adds lambda s / k = phi s / k^2 there (lambda = phi / k); one
// thread, summed apart from the imaging terms.
__global__ void source_term(const float *phi, const float *k, long long off, const float *s, double *sum)
{
    const double kk = k[off];
    *sum += (double)phi[off] * (double)*s / (kk * kk);
}

// Imaging terms of one or two adjoint levels as a pass of their own: sum (+)=
// (G phi_b / k) lap_b, then + (G phi_a / k) lap_a (the older level b first;
// phi_b may be NULL).  One thread per group of four cells, 16-byte accesses
// throughout: the groups of every array start on 16 bytes, and a ragged last
// group's cells past nx hold padding nobody reads.
__global__ __launch_bounds__(256) void imaging_terms(const float *__restrict__ phi_a, const float *__restrict__ lap_a,
                                                     const float *__restrict__ phi_b, const float *__restrict__ lap_b,
                                                     const float *__restrict__ k, const float *__restrict__ gx,
                                                     const float *__restrict__ gy, const float *__restrict__ gz,
                                                     int nx, int ny, int nz, int px, int x0, long long plane,
                                                     int lpx, long long lplane, int first, double *sum)
{
    typedef double dv2 __attribute__((ext_vector_type(2)));
    const int nxq = (nx + 3) / 4;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= ny * nxq)
        return;
    const int y = q / nxq, x = 4 * (q - y * nxq);
    float gxy[4];
    for (int e = 0; e < 4; ++e)
        gxy[e] = x + e < nx ? gx[x + e] * gy[y] : 0.f;
    auto load = [](const float *p) { return *reinterpret_cast<const f4 *>(p); };
    for (int z = blockIdx.z; z < nz; z += gridDim.z) {
        const long long f = (long long)(z + kGhost) * plane + (long long)(y + kGhost) * px + x0 + x;
        const long long l = z * lplane + (long long)y * lpx + x;
        const f4 kk = load(k + f), pa = load(phi_a + f), la = load(lap_a + l);
        f4 pb{}, lb{};
        if (phi_b) {
            pb = load(phi_b + f);
            lb = load(lap_b + l);
        }
        dv2 *s = reinterpret_cast<dv2 *>(sum + l);
        double t[4] = {0.0, 0.0, 0.0, 0.0};
        if (!first) {
            const dv2 s0 = s[0], s1 = s[1];
            t[0] = s0.x, t[1] = s0.y, t[2] = s1.x, t[3] = s1.y;
        }
        for (int e = 0; e < 4; ++e) {
            const float g = gxy[e] * gz[z];
            if (phi_b)
                t[e] += (double)((g * pb.v[e]) / kk.v[e] * lb.v[e]);
            t[e] += (double)((g * pa.v[e]) / kk.v[e] * la.v[e]);
        }
        s[0] = dv2{t[0], t[1]};
        s[1] = dv2{t[2], t[3]};
    }
}

// k = (v dt)^2 per cell, formed in FP64 and rounded once to FP32 (dense
// [n] arrays).
__global__ __launch_bounds__(256) void velocity_to_k(const float *__restrict__ v, long long n, double dt,
                                                    float *k)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const double vd = (double)v[i] * dt;
        k[i] = (float)(vd * vd);
    }
}

// misfit = 0.5 sum (traces - d_obs)^2 in FP64 (one work-group, fixed
// summation order, differences taken exactly); residual = traces - d_obs
// rounded to FP32 when requested.  One work-group's loop is a chain of memory
// latencies, so every thread has eight values of each array in flight.
__global__ __launch_bounds__(1024) void misfit_kernel(const float *__restrict__ tr,
                                                      const float *__restrict__ obs, long long n,
                                                      float *residual, double *out)
{
    constexpr int U = 8;
    __shared__ double part[1024];
    double acc = 0.0;
    long long i = threadIdx.x;
    for (; i + (U - 1) * 1024ll < n; i += U * 1024ll) {
        float a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u] = tr[i + u * 1024ll];
            b[u] = obs[i + u * 1024ll];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double r = (double)a[u] - (double)b[u];  // exact
            if (residual)
                residual[i + u * 1024ll] = (float)r;  // == the FP32 difference
            acc += r * r;
        }
    }
    for (; i < n; i += 1024) {
        const double r = (double)tr[i] - (double)obs[i];
        if (residual)
            residual[i] = (float)r;
        acc += r * r;
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        *out = 0.5 * part[0];
}

// dense[z][y][x] (+)= sum; the source cell (src, or -1) also gets *src_sum.
// With v set, the chain rule to velocity: dJ/dv = dJ/dk * 2 dt^2 v
// (k = (v dt)^2).  Blocks along rows: no division by the grid's sizes.
__global__ __launch_bounds__(256) void grad_to_dense(const double *__restrict__ sum, double *dense, int nx,
                                                    int ny, int nz, int lpx, long long lplane, int accumulate,
                                                    const float *__restrict__ v, double two_dt2, long long src,
                                                    const double *__restrict__ src_sum)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= nx)
        return;
    for (int z = blockIdx.z; z < nz; z += gridDim.z)
        for (int y = blockIdx.y; y < ny; y += gridDim.y) {
            const long long i = ((long long)z * ny + y) * nx + x;
            double g = sum[z * lplane + (long long)y * lpx + x];
            if (i == src)
                g += *src_sum;
            if (v)
                g *= two_dt2 * (double)v[i];
            dense[i] = accumulate ? dense[i] + g : g;
        }
}

// Clears both ticket sets at the start of a batched run (a kernel rather
// than a memset, so that it can sit in a captured graph).
__global__ void clear_counters(int *c)
{
    if (threadIdx.x < 16)
        c[kTicketStride * threadIdx.x] = 0;
}

// Zero n ints (a kernel, not a memset, so that it can sit in a captured graph).
__global__ __launch_bounds__(256) void zero_ints(int *p, long long n)
{
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
        p[i] = 0;
}

// Max and a non-finite (or negative) flag of an FP32 k over the interior, as
// float bit patterns (valid for non-negative values; negatives raise the
// flag).  One atomic per block at most, and none where it would change
// nothing: atomics on one address are served one after another (the former
// three per block of 1024 blocks took 39 us on the smallest grid).
__global__ __launch_bounds__(256) void k_range(const float *__restrict__ k, int nx, int ny, int nz,
                                               int px, int x0, long long plane, unsigned *out)
{
    __shared__ unsigned smax[256], sbad[256];
    unsigned mx = 0u, bad = 0u;
    for_interior_groups(nx, ny, nz, [&](int z, int y, int x, int n) {
        const float *p = k + (long long)(z + kGhost) * plane + (long long)(y + kGhost) * px + x0 + x;
        const f4 v = *reinterpret_cast<const f4 *>(p);
        for (int e = 0; e < 4; ++e) {
            if (e >= n)
                continue;  // right-ghost cells: ignored
            if (!(v.v[e] >= 0.f) || !(v.v[e] < INFINITY))
                bad = 1u;
            else  // -0.0 passes the test above, and as bits it exceeds every positive value
                mx = max(mx, __float_as_uint(fabsf(v.v[e])));
        }
    });
    const int t = threadIdx.y * blockDim.x + threadIdx.x;
    smax[t] = mx;
    sbad[t] = bad;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s) {
            smax[t] = max(smax[t], smax[t + s]);
            sbad[t] |= sbad[t + s];
        }
        __syncthreads();
    }
    if (t == 0) {
        if (smax[0] > out[0])
            atomicMax(&out[0], smax[0]);
        if (sbad[0])
            atomicOr(&out[1], sbad[0]);
    }
}

// Counts non-finite values: the interior of a field (FP32 or 16-bit bits,
// by storage type) into out[0], n trace values into out[1].
__global__ __launch_bounds__(256) void count_nonfinite(const void *__restrict__ field, int kind, int nx,
                                                      int ny, int nz, int px, int x0, long long plane,
                                                      const float *__restrict__ traces, long long n,
                                                      int *out)
{
    int bad_f = 0, bad_t = 0;
    for_interior_groups(nx, ny, nz, [&](int z, int y, int x, int cells) {
        const long long p = (long long)(z + kGhost) * plane + (long long)(y + kGhost) * px + x0 + x;
        if (kind == WAVE_F32) {
            const f4 v = *reinterpret_cast<const f4 *>(static_cast<const float *>(field) + p);
            for (int e = 0; e < 4; ++e)
                bad_f += e < cells && !isfinite(v.v[e]);
        } else {
            const ushort4 v = *reinterpret_cast<const ushort4 *>(static_cast<const unsigned short *>(field) + p);
            const unsigned b[4] = {v.x, v.y, v.z, v.w};
            const unsigned m = (kind == WAVE_F16 || kind == WAVE_F16_UV) ? 0x7c00u : 0x7f80u;
            for (int e = 0; e < 4; ++e)
                bad_f += e < cells && (b[e] & m) == m;  // all-ones exponent: infinity or NaN
        }
    });
    const long long block = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    for (long long i = block * 256 + threadIdx.y * blockDim.x + threadIdx.x; i < n; i += 256ll * gridDim.x * gridDim.y)
        bad_t += !isfinite(traces[i]);
    if (bad_f)
        atomicAdd(&out[0], bad_f);
    if (bad_t)
        atomicAdd(&out[1], bad_t);
}

}  // namespace wavek
