// Kernel declarations for the host code of libwave.so (wave.hip); the
// kernels are defined in wave_step.h (instantiated by the k_*.hip units)
// and k_misc.hip.
#pragma once

#include "wave_dev.h"

namespace wavek {

// Calls f(z, y, x, n) for the interior's groups of up to four cells of a row
// (n = 4, fewer in a ragged last group), x a multiple of 4: groups start on
// 16 (FP32) or 8 (16-bit) bytes.  Blocks take blockDim.y rows at a time, so a
// row's place costs one 32-bit division however long it is (a 64-bit division
// of a cell number per cell costs more than moving the cell); gridDim.y blocks
// share a row (see RowBlocks).
template <class F>
__device__ __forceinline__ void for_interior_groups(int nx, int ny, int nz, F &&f)
{
    const unsigned rows = (unsigned)ny * (unsigned)nz;
    for (unsigned row = blockIdx.x * blockDim.y + threadIdx.y; row < rows; row += gridDim.x * blockDim.y) {
        const int z = (int)(row / (unsigned)ny), y = (int)(row - (unsigned)z * (unsigned)ny);
        for (int x = 4 * (blockIdx.y * blockDim.x + threadIdx.x); x < nx; x += 4 * blockDim.x * gridDim.y)
            f(z, y, x, min(4, nx - x));
    }
}

// kernels (defined in the k_*.hip translation units)
template <int KIND, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_tiled(StepArgs a);
template <int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_tiled_cached(StepArgs a);
template <bool CACHED, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_tiled_lap(StepArgs a);
template <int MODE, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void adjoint_tiled(StepArgs a);
// Waves per SIMD the registers of step_batch must allow: four for FP32 tiles of
// one row whose halo is one group a thread.  They come to 131 registers, three
// over the 128 four waves have, and 128 cost nothing (no spills): two
// work-groups of 512 threads a CU instead of one (schedule 0, six shots of
// 120..300 cells a side in 128 x 16 tiles and eight chunks each, 40 steps:
// 10.2 -> 8.6 ms).
constexpr int batch_waves(int kind, int txv, int ty, int ry)
{
    return kind == WAVE_F32 && ry == 1 && 8 * txv + 2 * ty <= txv * ty ? 4 : 1;
}
template <int KIND, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY, batch_waves(KIND, TXV, TY, RY)) void step_batch(
    const ShotDesc *__restrict__ shots, BatchItems it, int j);
template <int KIND, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_batch_run(const ShotDesc *__restrict__ shots, BatchItems it,
                                                           RunSync rs);
template <int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_flow(const ShotDesc *__restrict__ shots, FlowPlan p);
template <int KIND>
__global__ __launch_bounds__(256) void step_naive(StepArgs a);
template <int KIND>
__global__ void sample_naive(const void *__restrict__ f, const long long *__restrict__ off, int nrec,
                             float *row, const int *exps, int slot);
template <int SRC, int DST>
__global__ __launch_bounds__(256) void convert_interior(const void *__restrict__ src, void *dst, int nx,
                                                        int ny, int nz, int spx, int sx0, long long sp,
                                                        int dpx, int dx0, long long dp, float scale,
                                                        const int *exps, int slot);
__global__ void clear_counters(int *c);
__global__ __launch_bounds__(256) void zero_ints(int *p, long long n);
__global__ __launch_bounds__(256) void k_range(const float *__restrict__ k, int nx, int ny, int nz,
                                               int px, int x0, long long plane, unsigned *out);
__global__ void inject_receivers(float *phi, const float *__restrict__ k,
                                 const long long *__restrict__ cell_off,
                                 const int *__restrict__ cell_start, const int *__restrict__ cell_rec,
                                 int ncells, const float *__restrict__ tg_row);
__global__ void source_term(const float *phi, const float *k, long long off, const float *s, double *sum);
__global__ __launch_bounds__(256) void imaging_terms(const float *__restrict__ phi_a, const float *__restrict__ lap_a,
                                                     const float *__restrict__ phi_b, const float *__restrict__ lap_b,
                                                     const float *__restrict__ k, const float *__restrict__ gx,
                                                     const float *__restrict__ gy, const float *__restrict__ gz,
                                                     int nx, int ny, int nz, int px, int x0, long long plane,
                                                     int lpx, long long lplane, int first, double *sum);
__global__ __launch_bounds__(256) void velocity_to_k(const float *__restrict__ v, long long n, double dt,
                                                    float *k);
__global__ __launch_bounds__(1024) void misfit_kernel(const float *__restrict__ tr,
                                                      const float *__restrict__ obs, long long n,
                                                      float *residual, double *out);
__global__ __launch_bounds__(256) void count_nonfinite(const void *__restrict__ field, int kind, int nx,
                                                      int ny, int nz, int px, int x0, long long plane,
                                                      const float *__restrict__ traces, long long n,
                                                      int *out);
__global__ __launch_bounds__(256) void grad_to_dense(const double *__restrict__ sum, double *dense, int nx,
                                                    int ny, int nz, int lpx, long long lplane, int accumulate,
                                                    const float *__restrict__ v, double two_dt2, long long src,
                                                    const double *__restrict__ src_sum);

}  // namespace wavek
