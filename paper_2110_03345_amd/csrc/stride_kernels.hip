// HIP kernels for gfx950 (CDNA4): leapfrog step of the acoustic wave
// equation with a 2r-order Laplacian and a sponge layer, fused with point
// injection, point sampling and (adjoint variant) the imaging condition.
//
// Forward (paper Sec. 2.4, constant density, no attenuation; second order in
// time):   C = a (2 A + k (L A + S)) - b B,          a = b = 1 outside the sponge
// Adjoint (exact transpose, Sec. 2.2 adjoint PDE):  the same update with
//          A = w^{m+1}, B = w^{m+2}, S = R^T g^m,  plus the imaging term
//          G += w^{m+1} (L u^m + S^m)   (gradient w.r.t. k; Sec. 2.2 reduced
//          gradient <grad_m L* w, dm>).
//
// The step kernels and what bounds them: step_kernels.h, step3d_body.h (3D) and
// step2d_resident.h (2D sweeps kept on the chip).
//
// This file holds the small kernels and the launchers; the step kernels
// live in step_kernels.h and compile in their own translation units.
#include "step_kernels.h"

#include <algorithm>
#include <cstdlib>

namespace stride {

// Tile shape of the 2D kernels (the host sizes launch shapes with it): the
// constants of common.h.  A build with STRIDE_TILE_SWEEP compiles every shape
// the sweeps try and reads the choice from the environment
// (STRIDE_RY2D[_ADJ], STRIDE_WAVES2D[_ADJ]); the library as shipped ignores
// the environment.
void tile_shape_2d(bool adjoint, int* ry, int* waves)
{
#ifdef STRIDE_TILE_SWEEP
    const char* er = getenv(adjoint ? "STRIDE_RY2D_ADJ" : "STRIDE_RY2D");
    const char* ew = getenv(adjoint ? "STRIDE_WAVES2D_ADJ" : "STRIDE_WAVES2D");
    int r = er && *er ? atoi(er) : kRy2d;
    int w = ew && *ew ? atoi(ew) : kWaves2d;
    if (w == 8) {
        r = 4;
    } else {
        w = 4;
        if (r != 2 && r != 8)
            r = 4;
    }
    *ry = r;
    *waves = w;
#else
    (void)adjoint;
    *ry = kRy2d;
    *waves = kWaves2d;
#endif
}

// Point values are read once per step.  Loaded with the non-temporal policy
// they do not evict the stencil field's halo, which pays beyond the Infinity
// Cache (forward step at 316^3: 92.7 us against 103.9); while the fields a step
// touches stay in that cache from step to step the ordinary policy finds them
// there (252^3: 47.4 against 55.9 us, storing v 57.8 against 68.3, 188^3: 22.8
// against 26.7).  The fields counted are those that live from step to step:
// wavefields, k, G and the second stencil or point field.
bool stream_3d(const Dims& d, bool adjoint, int mode)
{
    const bool one = mode == kImageV || mode == kAdjPlain;
    const int fields = (adjoint && !one) || mode == kMedium || mode == kMediumY0 ? 5
                       : mode == kCorrect || mode == kImageV                    ? 4
                                                                                : 3;
    return fields * d.total * 4 > kCacheBytes;
}

namespace {

// ------------------------------------------------------------ small kernels

__global__ void sample_kernel(SampleSet smp, const float* field, int step)
{
    sample_block(smp, field, step, blockIdx.x);
}

__global__ void fill_kernel(float* p, long long n, float v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride)
        p[i] = v;
}

__global__ void copy_kernel(float* dst, const float* src, long long n)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride)
        dst[i] = src[i];
}

// k = dt^2 vp_pad^2 with vp edge-replicated into the sponge; computed in
// double and rounded once.
__global__ void prep_k_kernel(Dims d, const float* vp, double dt, float* k)
{
    long long npts = (long long)d.n[0] * d.n[1] * d.n[2];
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < npts; i += stride) {
        int c[3];
        long long r = i;
        for (int a = 2; a >= 0; --a) {
            c[a] = (int)(r % d.n[a]);
            r /= d.n[a];
        }
        long long src = 0, dst = 0;
        for (int a = 0; a < 3; ++a) {
            int pa = min(max(c[a] - d.nb, 0), d.phys[a] - 1);
            if (d.n[a] == 1)
                pa = 0;
            src = src * d.phys[a] + pa;
            dst += (long long)c[a] * (a < d.nd ? d.st[a] : 0);
        }
        double v = (double)vp[src];
        k[dst] = (float)(dt * dt * v * v);
    }
}

// Medium fields on the padded grid (see launch_prep_medium).  The physical
// index of any padded (or beyond-padded) coordinate is its clamp into the
// physical grid, which is both the edge replication into the sponge and the
// constant continuation of ln rho beyond the array.
__device__ __forceinline__ long long phys_index(const Dims& d, const int c[3])
{
    long long src = 0;
    for (int a = 0; a < 3; ++a) {
        int pa = a < d.nd ? min(max(c[a] - d.nb, 0), d.phys[a] - 1) : 0;
        src = src * d.phys[a] + pa;
    }
    return src;
}

// ln rho over the physical grid, in FP64.
__global__ void ln_kernel(const float* rho, long long n, double* out)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = log((double)rho[i]);
}

// One logarithm per point, kept (lr; NULL: constant density), instead of one per
// tap: 0.4 ms at 252^3, order 10, against 1.6.
__global__ void prep_medium_kernel(Dims d, Fd1 fd, const float* vp, const double* lr,
                                   const float* alpha0, int att_power, double dt, float* g0,
                                   float* g1, float* g2, float* att)
{
    const long long npts = (long long)d.n[0] * d.n[1] * d.n[2];
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    float* gam[3] = {g0, g1, g2};
    for (; i < npts; i += stride) {
        int c[3];
        long long r = i;
        for (int a = 2; a >= 0; --a) {
            c[a] = (int)(r % d.n[a]);
            r /= d.n[a];
        }
        long long dst = 0;
        for (int a = 0; a < d.nd; ++a)
            dst += (long long)c[a] * d.st[a];
        const long long src = phys_index(d, c);
        for (int a = 0; a < d.nd; ++a) {
            double sum = 0.0;
            if (lr) {
                for (int j = 1; j <= fd.r; ++j) {
                    int cp[3] = {c[0], c[1], c[2]}, cm[3] = {c[0], c[1], c[2]};
                    cp[a] += j;
                    cm[a] -= j;
                    sum += fd.d[j] * (lr[phys_index(d, cp)] - lr[phys_index(d, cm)]);
                }
            }
            gam[a][dst] = (float)(-sum * fd.inv_dx[a]);
        }
        double at = 0.0;
        if (alpha0) {
            at = 2.0 * (double)alpha0[src] * (double)vp[src];
            if (att_power == 2)
                at /= dt;
        }
        att[dst] = (float)at;
    }
}

// Value checks of rho and alpha0, and max vp^2 (1 + 2 beta) for the stability
// limit of the y = 2 term (see launch_medium_check).
__global__ void medium_check_kernel(const float* vp, const float* rho, const float* alpha0,
                                    long long n, int att_power, double dt, unsigned* flags)
{
    __shared__ unsigned smax, sbad;
    if (threadIdx.x == 0) {
        smax = 0u;
        sbad = 0u;
    }
    __syncthreads();
    unsigned m = 0u, bad = 0u;
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        if (rho && !(rho[i] > 0.f && isfinite(rho[i])))
            bad = 1u;
        double beta = 0.0;
        if (alpha0) {
            const float al = alpha0[i];
            if (!(al >= 0.f && isfinite(al)))
                bad = 1u;
            else if (att_power == 2)
                beta = 2.0 * (double)al * (double)vp[i] / dt;
        }
        const double v = (double)vp[i];
        const float e = (float)(v * v * (1.0 + 2.0 * beta));
        if (e >= 0.f && isfinite(e))
            m = max(m, __float_as_uint(e));
        else
            bad = 1u;
    }
    atomicMax(&smax, m);
    atomicOr(&sbad, bad);
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicMax(&flags[3], smax);
        atomicOr(&flags[2], sbad);
    }
}

// Transposed source filter of the fourth-order scheme, one row per block,
// in place (the row is staged in LDS first).
__global__ __launch_bounds__(256) void time_filter3_kernel(float* rows, int nt)
{
    extern __shared__ float row[];
    float* r = rows + (long long)blockIdx.x * nt;
    for (int j = threadIdx.x; j < nt; j += 256)
        row[j] = r[j];
    __syncthreads();
    for (int j = threadIdx.x; j < nt; j += 256) {
        const float lo = j >= 1 ? row[j - 1] : 0.f;
        const float hi = j + 1 < nt ? row[j + 1] : 0.f;
        r[j] = fmaf(10.f, row[j], lo + hi) / 12.f;
    }
}

// Zero-phase low-pass of one [nt] row per block (band-limiting for the
// frequency blocks of an inversion): the Hann-windowed sinc taps
// h_k = 2 fc dt sinc(2 fc k dt) (0.5 + 0.5 cos(pi k / (K + 1))), |k| <= K,
// normalised to unit sum, are built in LDS (FP64, rounded once), the row is
// staged in LDS (so out may alias in), and each thread convolves its samples
// with zeros beyond the record.
__global__ __launch_bounds__(256) void lowpass_kernel(const float* in, float* out, int nt,
                                                      double fdt, int K)
{
    extern __shared__ float lds[];
    float* h = lds;                  // 2K + 1 taps
    float* row = lds + 2 * K + 1;    // nt samples
    __shared__ double part[256];
    const double pi = 3.14159265358979323846;
    double sum = 0.0;
    for (int k = -K + (int)threadIdx.x; k <= K; k += 256) {
        const double x = 2.0 * fdt * k;
        const double sc = k == 0 ? 1.0 : sin(pi * x) / (pi * x);
        const double v = 2.0 * fdt * sc * (0.5 + 0.5 * cos(pi * k / (K + 1.0)));
        sum += v;
    }
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    const double total = part[0];
    for (int k = -K + (int)threadIdx.x; k <= K; k += 256) {
        const double x = 2.0 * fdt * k;
        const double sc = k == 0 ? 1.0 : sin(pi * x) / (pi * x);
        h[k + K] = (float)(2.0 * fdt * sc * (0.5 + 0.5 * cos(pi * k / (K + 1.0))) / total);
    }
    const float* src = in + (long long)blockIdx.x * nt;
    for (int n = threadIdx.x; n < nt; n += 256)
        row[n] = src[n];
    __syncthreads();
    float* dst = out + (long long)blockIdx.x * nt;
    for (int n = threadIdx.x; n < nt; n += 256) {
        const int klo = max(-K, n - nt + 1), khi = min(K, n);
        float acc = 0.f;
        for (int k = klo; k <= khi; ++k)
            acc = fmaf(h[k + K], row[n - k], acc);
        dst[n] = acc;
    }
}

// Gradient-descent step of the inversion loop: gmax = max |m g| (as float
// bits; order-independent, so reproducible), then vp = clamp(vp - step m g /
// gmax, vmin, vmax) with the mask m (1 where absent).
__global__ __launch_bounds__(256) void grad_absmax_kernel(const float* g, const float* mask,
                                                          long long n, unsigned* gmax)
{
    __shared__ unsigned smax;
    if (threadIdx.x == 0)
        smax = 0u;
    __syncthreads();
    unsigned m = 0u;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const float v = fabsf(mask ? mask[i] * g[i] : g[i]);
        m = max(m, __float_as_uint(v));
    }
    atomicMax(&smax, m);
    __syncthreads();
    if (threadIdx.x == 0)
        atomicMax(gmax, smax);
}

__global__ void descent_kernel(float* vp, const float* g, const float* mask, long long n,
                               float step, float vmin, float vmax, const unsigned* gmax)
{
    const float gm = __uint_as_float(*gmax);
    const float scale = gm > 0.f ? step / gm : 0.f;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const float d = mask ? mask[i] * g[i] : g[i];
        vp[i] = fminf(fmaxf(fmaf(-scale, d, vp[i]), vmin), vmax);
    }
}

// Residual r = traces - observed and J = 1/2 sum r^2 in FP64.  Block b reduces
// a fixed contiguous range in a fixed tree order and misfit_final_kernel adds
// the partial sums in block order, so the result is bitwise reproducible.
__global__ __launch_bounds__(256) void residual_partial_kernel(const float* traces,
                                                               const float* observed,
                                                               float* residual, long long n,
                                                               double* partial)
{
    __shared__ double part[256];
    const long long per = (n + gridDim.x - 1) / gridDim.x;
    const long long lo = per * blockIdx.x;
    const long long hi = min(n, lo + per);
    double acc = 0.0;
    for (long long i = lo + threadIdx.x; i < hi; i += 256) {
        float r = traces[i] - observed[i];
        residual[i] = r;
        acc += (double)r * (double)r;
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        partial[blockIdx.x] = part[0];
}

__global__ __launch_bounds__(256) void misfit_final_kernel(const double* partial, int nparts,
                                                           double* misfit)
{
    __shared__ double part[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 256)
        acc += partial[i];
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        *misfit = 0.5 * part[0];
}

// Transpose of edge-replicating padding along one axis.  The input is viewed
// as [m0][nin][m2] with strides (s_outer, s_axis, 1), the output is dense
// [m0][nout][m2] with nin = nout + 2 nb: output cell j collects input cell
// j + nb, and the two edge cells also collect the nb cells replicated from
// them.  With vp given, the output is 2 * sum / vp (the last pass of dvp).
// With div given (laid out like the input), each input cell is divided by it.
__global__ void pad_transpose_axis_kernel(const float* in, const float* div, long long s_outer,
                                          long long s_axis, float* out, long long m0, int nout,
                                          long long m2, int nb, const float* vp)
{
    const long long total = m0 * nout * m2;
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < total; i += stride) {
        const long long i2 = i % m2;
        const long long r = i / m2;
        const int j = (int)(r % nout);
        const long long i0 = r / nout;
        const int lo = j == 0 ? 0 : j + nb;
        const int hi = j == nout - 1 ? j + 2 * nb : j + nb;
        const long long base = i0 * s_outer + i2;
        const float* src = in + base;
        float acc = 0.f;
        if (div)
            for (int k = lo; k <= hi; ++k)
                acc += src[(long long)k * s_axis] / div[base + (long long)k * s_axis];
        else
            for (int k = lo; k <= hi; ++k)
                acc += src[(long long)k * s_axis];
        out[i] = vp ? 2.f * acc / vp[i] : acc;
    }
}

// max(vp) (as the bit pattern of a positive float, which orders like the
// float) and a flag for non-positive or non-finite values.
__global__ void vp_check_kernel(const float* vp, long long n, unsigned* flags)
{
    __shared__ unsigned smax, sbad;
    if (threadIdx.x == 0) {
        smax = 0u;
        sbad = 0u;
    }
    __syncthreads();
    unsigned m = 0u, bad = 0u;
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        float v = vp[i];
        if (!(v > 0.f) || !isfinite(v))
            bad = 1u;
        else
            m = max(m, __float_as_uint(v));
    }
    atomicMax(&smax, m);
    atomicOr(&sbad, bad);
    __syncthreads();
    // atomics on one word queue up (30 us at 1024^2 with two per block, 14 now): only
    // where they change it
    if (threadIdx.x == 0) {
        if (smax > __hip_atomic_load(&flags[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(&flags[0], smax);
        if (sbad)
            atomicOr(&flags[1], sbad);
    }
}

int grid_for(long long n, int threads)
{
    long long b = (n + threads - 1) / threads;
    if (b > 65536)
        b = 65536;
    if (b < 1)
        b = 1;
    return (int)b;
}

}  // namespace


// Step launches go to the translation unit of their family.
void launch_family_2d(bool adjoint, int R, int mode, const Dims& d, const StencilCoef& cf,
                      const SpongeCoef& sp, const LaunchShape& ls, const StepParams& p, hipStream_t s);
void launch_family_3d_fwd(int R, int mode, const Dims& d, const StencilCoef& cf, const SpongeCoef& sp,
                          const LaunchShape& ls, const StepParams& p, hipStream_t s);
void launch_family_3d_adj(int R, int mode, const Dims& d, const StencilCoef& cf, const SpongeCoef& sp,
                          const LaunchShape& ls, const StepParams& p, hipStream_t s);
void launch_batched_2d(bool adjoint, int R, int mode, const Dims& d, const StencilCoef& cf,
                       const LaunchShape& ls, const SlotStep* table, int nslots, int max_samples,
                       hipStream_t s);
void launch_batched_3d_fwd(int R, int mode, const Dims& d, const StencilCoef& cf,
                           const LaunchShape& ls, const SlotStep* table, int nslots, int max_samples,
                           hipStream_t s);
void launch_batched_3d_adj(int R, int mode, const Dims& d, const StencilCoef& cf,
                           const LaunchShape& ls, const SlotStep* table, int nslots, int max_samples,
                           hipStream_t s);

void launch_step_mode(const Dims& d, int R, bool adjoint, int mode, const StencilCoef& cf,
                      const SpongeCoef& sp, const LaunchShape& ls, const StepParams& p, hipStream_t s)
{
    if (d.nd == 2)
        launch_family_2d(adjoint, R, mode, d, cf, sp, ls, p, s);
    else if (adjoint)
        launch_family_3d_adj(R, mode, d, cf, sp, ls, p, s);
    else
        launch_family_3d_fwd(R, mode, d, cf, sp, ls, p, s);
}

void launch_step(const Dims& d, int R, bool adjoint, const StencilCoef& cf, const SpongeCoef& sp,
                 const LaunchShape& ls, const StepParams& p, hipStream_t s)
{
    launch_step_mode(d, R, adjoint, kStep, cf, sp, ls, p, s);
}

void launch_step_batched(const Dims& d, int R, bool adjoint, int mode, const StencilCoef& cf,
                         const LaunchShape& ls, const SlotStep* table, int nslots, int max_samples,
                         hipStream_t s)
{
    if (d.nd == 2)
        launch_batched_2d(adjoint, R, mode, d, cf, ls, table, nslots, max_samples, s);
    else if (adjoint)
        launch_batched_3d_adj(R, mode, d, cf, ls, table, nslots, max_samples, s);
    else
        launch_batched_3d_fwd(R, mode, d, cf, ls, table, nslots, max_samples, s);
}

__global__ void accumulate_kernel(float* dst, const float* src, long long n)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride)
        dst[i] += src[i];
}

void launch_accumulate(float* dst, const float* src, long long n, hipStream_t s)
{
    hipLaunchKernelGGL(accumulate_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, dst, src, n);
}

void launch_sample(const SampleSet& smp, const float* field, int step, hipStream_t s)
{
    if (smp.count <= 0)
        return;
    int blocks = (smp.count * sample_lanes(smp.ntap) + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(sample_kernel, dim3(blocks), dim3(kThreads), 0, s, smp, field, step);
}

void launch_fill(float* p, long long n, float v, hipStream_t s)
{
    hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, v);
}

void launch_copy(float* dst, const float* src, long long n, hipStream_t s)
{
    hipLaunchKernelGGL(copy_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, dst, src, n);
}

__global__ void poison_kernel(const unsigned* err, Outputs out, unsigned* report)
{
    if (!*err)
        return;
    if (report && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(report, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    for (int a = 0; a < 3; ++a)
        for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; out.p[a] && i < out.n[a];
             i += (long long)gridDim.x * blockDim.x)
            out.p[a][i] = __uint_as_float(0x7fffffffu);   // (two of them: a double NaN)
}

void launch_poison(const unsigned* err, const Outputs& out, hipStream_t s, unsigned* report)
{
    const long long n = std::max({out.n[0], out.n[1], out.n[2]});
    if (n > 0)
        hipLaunchKernelGGL(poison_kernel, dim3(std::min(grid_for(n, 256), 256)), dim3(256), 0, s, err, out,
                           report);
}

// flag |= bit when any of the n values is NaN or infinite.
template <class T>
__global__ void finite_scan_kernel(const T* p, long long n, unsigned* flag, unsigned bit)
{
    bool bad = false;
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride)
        bad |= !isfinite(p[i]);
    if (bad)
        atomicOr(flag, bit);
}

void launch_finite_scan(const float* p, long long n, unsigned* flag, unsigned bit, hipStream_t s)
{
    hipLaunchKernelGGL(finite_scan_kernel<float>, dim3(std::min(grid_for(n, 256), 2048)), dim3(256),
                       0, s, p, n, flag, bit);
}

void launch_finite_scan(const double* p, long long n, unsigned* flag, unsigned bit, hipStream_t s)
{
    hipLaunchKernelGGL(finite_scan_kernel<double>, dim3(std::min(grid_for(n, 256), 2048)), dim3(256),
                       0, s, p, n, flag, bit);
}

// Perfectly matched layer.  Per axis a whose layer holds a point (zeta_a > 0):
//   chi_a = E chi_a + (1 - E) (D2_a u - D_a psi_a),  psi_a' = E psi_a + (1 - E) D_a u,
// and u^{n+1} += k sum_a (-D_a psi_a - chi_a), the axes taken in order 0, 1, 2.
// Neighbours beyond the padded array read 0.  A thread corrects four points of a
// row, in one launch over three ranges of blocks: the planes of axis 0 in its
// layer (3D), then within the physical planes the rows of axis 1 in its layer,
// then within the physical rows the quads that touch axis 2's layer.  The waves
// of a block are consecutive planes (first range) or rows (second) of the same
// columns, which keeps most neighbours in L1.  At 220^3 with a layer of 30: 88 us
// a step (110 with a thread per point and a launch per range); L1 then waits on
// lines still on their way to it for 40% of the time, the vector units are busy
// for 30%, and two to sixteen waves to a block or fewer loads in flight make no
// difference.
struct PmlGeom {
    int nn[3];        // 3D-ised padded extents (axis 0 of a 2D grid has extent 1)
    int st[3];        // strides in floats (pitched rows)
    int pl[3];        // physical extents
    int b;            // layer width of axes 1 and 2 (and of axis 0 in 3D)
    int b0;           // layer width of axis 0 (0 in 2D)
    int three;
};

using PmlVec = StepVec<4>;

// A quad of a layer: its plane (uniform over the wave), row, first column and
// byte offset in the plane.
struct PmlAt {
    long long plane;     // element offset of the plane
    int plane_bytes;
    int i0, i1, i2;
    int off;
};

__device__ __forceinline__ int pml_depth(const PmlGeom& g, int ax, int i)
{
    const int b = ax == 0 ? g.b0 : g.b, hi = b + g.pl[ax] - 1;
    return i < b ? b - i : (i > hi ? i - hi : 0);
}

__device__ __forceinline__ float pml_decay(const PmlGeom& g, const PmlParams& pp, int ax, int depth)
{
    const float frac = (float)depth / (float)(ax == 0 ? g.b0 : g.b);
    const float zeta = pp.zmax[g.three ? ax : ax - 1] * frac * frac;
    return __expf(-zeta * pp.dt);   // hardware exp2: a few ulp, far inside the tolerance
}

// Term of axis AX at four points, of which those with on[k] are in its layer (the
// others keep their memory variables and get no term); corr: the sum so far.
// Neighbours are read with buffer loads, whose range check gives the zeros
// beyond the array: one select per load instead of one per value.
template <int R, bool NT, int AX>
__device__ __forceinline__ void pml_axis_term(const StencilCoef& cf, const PmlParams& pp,
                                              const PmlGeom& g, const PmlAt& at, const bool* on,
                                              PmlVec& corr)
{
    const int a = g.three ? AX : AX - 1;        // axis of the solver's Dims / coefficients
    const auto ru = plane_rsrc(pp.u + at.plane, at.plane_bytes);
    const auto rp = plane_rsrc(pp.psi[a] + at.plane, at.plane_bytes);
    const auto rc = plane_rsrc(pp.chi[a] + at.plane, at.plane_bytes);
    const PmlVec u0 = bloadv<4, 0>(ru, at.off), p0 = bloadv<4, 0>(rp, at.off);
    PmlVec chi = bloadv<4, 0>(rc, at.off);
    PmlVec d2, d1u = PmlVec(0.f), d1p = PmlVec(0.f);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        d2[k] = pp.c0[a] * u0[k];
    if constexpr (AX == 2) {
        constexpr int H = (R + 3) / 4 * 4;
        float ur[4 + 2 * H], pr[4 + 2 * H];
#pragma unroll
        for (int q = 0; q < 4 + 2 * H; q += 4) {
            const int x = at.i2 + q - H;
            const int off = x >= 0 && x < g.nn[2] ? at.off + (q - H) * 4 : kNoByte;
            const PmlVec uv = q == H ? u0 : bloadv<4, 0>(ru, off);
            const PmlVec pv = q == H ? p0 : bloadv<4, 0>(rp, off);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                ur[q + k] = uv[k];
                pr[q + k] = pv[k];
            }
        }
        if (g.nn[2] % 4 != 0)       // rows ending inside a quad
#pragma unroll
            for (int q = 0; q < 4 + 2 * H; ++q) {
                const bool in = at.i2 + q - H < g.nn[2];
                ur[q] = in ? ur[q] : 0.f;
                pr[q] = in ? pr[q] : 0.f;
            }
#pragma unroll
        for (int j = 1; j <= R; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                d2[k] = fmaf(cf.c[a][j], ur[H + k + j] + ur[H + k - j], d2[k]);
                d1u[k] = fmaf(cf.d[a][j], ur[H + k + j] - ur[H + k - j], d1u[k]);
                d1p[k] = fmaf(cf.d[a][j], pr[H + k + j] - pr[H + k - j], d1p[k]);
            }
    } else {
#pragma unroll
        for (int j = 1; j <= R; ++j) {
            PmlVec up, um, qp, qm;
            if constexpr (AX == 0) {
                const long long s = (long long)j * g.st[0];
                const int bp = at.i0 + j < g.nn[0] ? at.plane_bytes : 0;
                const int bm = at.i0 - j >= 0 ? at.plane_bytes : 0;
                const long long lp = at.plane + (bp ? s : 0), lm = at.plane - (bm ? s : 0);
                up = bloadv<4, 0>(plane_rsrc(pp.u + lp, bp), at.off);
                um = bloadv<4, 0>(plane_rsrc(pp.u + lm, bm), at.off);
                qp = bloadv<4, 0>(plane_rsrc(pp.psi[a] + lp, bp), at.off);
                qm = bloadv<4, 0>(plane_rsrc(pp.psi[a] + lm, bm), at.off);
            } else {
                const int s = j * g.st[1] * 4;
                const int op = at.i1 + j < g.nn[1] ? at.off + s : kNoByte;
                const int om = at.i1 - j >= 0 ? at.off - s : kNoByte;
                up = bloadv<4, 0>(ru, op);
                um = bloadv<4, 0>(ru, om);
                qp = bloadv<4, 0>(rp, op);
                qm = bloadv<4, 0>(rp, om);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                d2[k] = fmaf(cf.c[a][j], up[k] + um[k], d2[k]);
                d1u[k] = fmaf(cf.d[a][j], up[k] - um[k], d1u[k]);
                d1p[k] = fmaf(cf.d[a][j], qp[k] - qm[k], d1p[k]);
            }
        }
    }
    PmlVec next;
    float E = 0.f;
    if constexpr (AX < 2)
        E = pml_decay(g, pp, AX, pml_depth(g, AX, AX == 0 ? at.i0 : at.i1));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if constexpr (AX == 2)
            E = pml_decay(g, pp, AX, pml_depth(g, AX, at.i2 + k));
        const float c = fmaf(E, chi[k], (1.f - E) * (d2[k] - d1p[k]));
        const float n = fmaf(E, p0[k], (1.f - E) * d1u[k]);
        chi[k] = on[k] ? c : chi[k];
        next[k] = on[k] ? n : p0[k];
        corr[k] = on[k] ? corr[k] - (d1p[k] + c) : corr[k];
    }
    bstorev<4, NT ? 2 : 0>(rc, at.off, chi);
    bstorev<4, NT ? 2 : 0>(plane_rsrc(pp.psin[a] + at.plane, at.plane_bytes), at.off, next);
}

// The correction of points (i0, i1, 4 q ..), i0 uniform over the wave.  Rows are
// pitched to whole quads; points past the end of a row keep what they hold.
template <int R, bool NT>
__device__ __forceinline__ void pml_quad(const StencilCoef& cf, const PmlParams& pp, const PmlGeom& g,
                                         int i0, int i1, int q)
{
    PmlAt at;
    at.i0 = i0;
    at.i1 = i1;
    at.i2 = 4 * q;
    at.plane = (long long)i0 * g.st[0];
    at.plane_bytes = g.st[1] * g.nn[1] * 4;
    at.off = (i1 * g.st[1] + at.i2) * 4;
    PmlVec corr = PmlVec(0.f);
    bool live[4], x[4], any = false, on[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        live[k] = at.i2 + k < g.nn[2];
        x[k] = live[k] && pml_depth(g, 2, at.i2 + k) != 0;
        any = any || x[k];
    }
    const bool z = g.three && pml_depth(g, 0, i0) != 0, y = pml_depth(g, 1, i1) != 0;
    const auto rn = plane_rsrc(pp.un + at.plane, at.plane_bytes);
    PmlVec un = bloadv<4, 0>(rn, at.off);
    const PmlVec kv = bloadv<4, 0>(plane_rsrc(pp.k + at.plane, at.plane_bytes), at.off);
    if (z)
        pml_axis_term<R, NT, 0>(cf, pp, g, at, live, corr);
    if (y)
        pml_axis_term<R, NT, 1>(cf, pp, g, at, live, corr);
    if (any)
        pml_axis_term<R, NT, 2>(cf, pp, g, at, x, corr);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        on[k] = x[k] || (live[k] && (z || y));
        un[k] = on[k] ? fmaf(kv[k], corr[k], un[k]) : un[k];
    }
    bstorev<4, NT ? 2 : 0>(rn, at.off, un);
}

// Ranges of a correction launch: blocks of kPmlWaves waves (one per plane or row
// of a group), 64 quads of a plane's or row's list each.
struct PmlRanges {
    int nq;                  // quads of a row
    int ql, qr;              // axis 2's layer: quads [0, ql) and [qr, nq)
    int cols0, cols1, cols2; // blocks per group of planes / rows
    int end0, end1, end2;    // last block of each range, exclusive
};

constexpr int kPmlWaves = 4;

// NT: non-temporal stores.
template <int R, bool NT>
__global__ __launch_bounds__(64 * kPmlWaves) void pml_layer_kernel(StencilCoef cf, PmlParams pp, PmlGeom g,
                                                        PmlRanges r)
{
    const int b = xcd_logical(blockIdx.x, gridDim.x);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63;
    if (b < r.end0) {
        // column block fastest but for the plane group: neighbouring groups of
        // planes run next to each other
        const int groups = (g.b0 + kPmlWaves - 1) / kPmlWaves;
        const int col = b / (2 * groups), gr = b - col * 2 * groups;
        const int side = gr >= groups;
        const int zl = (gr - side * groups) * kPmlWaves + wave, t = col * 64 + lane;
        if (zl >= g.b0 || t >= g.nn[1] * r.nq)
            return;
        const int i1 = t / r.nq;
        pml_quad<R, NT>(cf, pp, g, side ? g.b0 + g.pl[0] + zl : zl, i1, t - i1 * r.nq);
    } else if (b < r.end1) {
        const int groups = (2 * g.b + kPmlWaves - 1) / kPmlWaves;
        const int e = b - r.end0, plane = e / (groups * r.cols1), f = e - plane * groups * r.cols1;
        const int col = f / groups;
        const int rl = (f - col * groups) * kPmlWaves + wave, q = col * 64 + lane;
        if (rl >= 2 * g.b || q >= r.nq)
            return;
        pml_quad<R, NT>(cf, pp, g, g.b0 + plane, rl < g.b ? rl : g.pl[1] + rl, q);
    } else if (b < r.end2) {
        const int nl = r.ql + r.nq - r.qr;
        const int e = b - r.end1, plane = e / r.cols2;
        const int t = (e - plane * r.cols2) * (64 * kPmlWaves) + (int)threadIdx.x, i1 = t / nl, ql = t - i1 * nl;
        if (i1 >= g.pl[1])
            return;
        pml_quad<R, NT>(cf, pp, g, g.b0 + plane, g.b + i1, ql < r.ql ? ql : r.qr + ql - r.ql);
    }
}

void launch_pml_correction(const Dims& d, int R, const StencilCoef& cf, const PmlParams& pp,
                           hipStream_t s)
{
    const bool three = d.nd == 3;
    PmlGeom g{};
    g.three = three ? 1 : 0;
    g.nn[0] = three ? d.n[0] : 1;
    g.nn[1] = three ? d.n[1] : d.n[0];
    g.nn[2] = three ? d.n[2] : d.n[1];
    g.st[0] = three ? (int)d.st[0] : 0;
    g.st[1] = three ? (int)d.st[1] : (int)d.st[0];
    g.st[2] = 1;
    g.pl[0] = three ? d.phys[0] : 1;
    g.pl[1] = three ? d.phys[1] : d.phys[0];
    g.pl[2] = three ? d.phys[2] : d.phys[1];
    g.b = d.nb;
    g.b0 = three ? d.nb : 0;
    if (g.b <= 0)
        return;
    PmlRanges r{};
    r.nq = (g.nn[2] + 3) / 4;
    r.ql = std::min((g.b + 3) / 4, r.nq);
    r.qr = std::max((g.b + g.pl[2]) / 4, r.ql);
    r.cols0 = (g.nn[1] * r.nq + 63) / 64;
    r.cols1 = (r.nq + 63) / 64;
    r.cols2 = (g.pl[1] * (r.ql + r.nq - r.qr) + 64 * kPmlWaves - 1) / (64 * kPmlWaves);
    r.end0 = 2 * ((g.b0 + kPmlWaves - 1) / kPmlWaves) * r.cols0;
    r.end1 = r.end0 + (2 * g.b + kPmlWaves - 1) / kPmlWaves * r.cols1 * g.pl[0];
    r.end2 = r.end1 + r.cols2 * g.pl[0];
    const dim3 grid((unsigned)((r.end2 + kXcds - 1) / kXcds * kXcds));
    // What it writes is read in the next step: kept in the Infinity Cache while what a
    // step touches (u, u', k, and psi, psi', chi of the layer of each axis) fits 0.85 of
    // it.  Beyond that non-temporal stores leave the room to what is read in this
    // launch; us a step with the leapfrog, order 10, layer 30, ordinary / non-temporal:
    // 160^3 51 / 64, 200^3 85 / 109, 210^3 (210 MiB) 112 / 119, 220^3 (226 MiB) 131 / 127,
    // 316^3 312 / 308.
    double fields = 3.0;
    for (int ax = three ? 0 : 1; ax < 3; ++ax)
        fields += 3.0 * 2.0 * (ax == 0 ? g.b0 : g.b) / g.nn[ax];
    const bool nt = fields * 4.0 * (double)d.total > 0.85 * (double)kCacheBytes;
    const auto kernel = R == 4 ? (nt ? pml_layer_kernel<4, true> : pml_layer_kernel<4, false>)
                               : (nt ? pml_layer_kernel<5, true> : pml_layer_kernel<5, false>);
    hipLaunchKernelGGL(kernel, grid, dim3(64 * kPmlWaves), 0, s, cf, pp, g, r);
}

// Padded coordinates of linear index t over the padded grid (no pitch) and the
// sponge rate there.
__device__ __forceinline__ void padded_coords(const Dims& d, long long t, int c[3])
{
    c[2] = 0;
    if (d.nd == 3) {
        const long long plane = (long long)d.n[1] * d.n[2];
        c[0] = (int)(t / plane);
        const long long r = t - (long long)c[0] * plane;
        c[1] = (int)(r / d.n[2]);
        c[2] = (int)(r - (long long)c[1] * d.n[2]);
    } else {
        c[0] = (int)(t / d.n[1]);
        c[1] = (int)(t - (long long)c[0] * d.n[1]);
    }
}

__device__ __forceinline__ float sponge_eta(const Dims& d, const SpongeCoef& sp, const int c[3])
{
    float eta = 0.f;
    for (int a = 0; a < d.nd; ++a) {
        const int dep = layer_depth(c[a], d.n[a], d.nb);
        eta = fmaf(sp.e[a], (float)(dep * dep), eta);
    }
    return eta;
}

// 2D: one thread per padded point of a 64 x 8 tile, two rows per thread.  The
// block first stages in LDS the stencil operand y over the tile and its R-wide
// halo, and the density products gamma_0 w^{m+1} (tile and row halo) and gamma_1
// w^{m+1} (tile and column halo).  Neighbours beyond the padded array read 0.
// The sums run in the same order as the point-wise definition: centre, then per
// axis the taps j = 1..R.
constexpr int kMadjRows = 8;

template <int R, bool Y2>
__global__ __launch_bounds__(256) void medium_adjoint_kernel(Dims d, StencilCoef cf, SpongeCoef sp,
                                                             MediumAdjParams mp)
{
    constexpr int TW = kTileX + 2 * R, TH = kMadjRows + 2 * R;
    __shared__ float Yt[TH][TW];
    __shared__ float Zy[TH][kTileX];
    __shared__ float Zx[kMadjRows][TW];
    const int tid = (int)threadIdx.x;
    const int x0 = (int)blockIdx.x * kTileX, y0 = (int)blockIdx.y * kMadjRows;
    const int ny = d.n[0], nx = d.n[1];
    const long long sty = d.st[0];
    auto yv = [&](long long q) {
        if constexpr (Y2)
            return fmaf(mp.att[q], mp.w1[q] - mp.w2[q], mp.w1[q]);
        else
            return mp.w1[q];
    };
    for (int e = tid; e < TH * TW; e += 256) {
        const int ly = e / TW, lx = e - ly * TW;
        const int gy = y0 + ly - R, gx = x0 + lx - R;
        float v = 0.f;
        if (gy >= 0 && gy < ny && gx >= 0 && gx < nx)
            v = yv(gy * sty + gx);
        Yt[ly][lx] = v;
    }
    for (int e = tid; e < TH * kTileX; e += 256) {
        const int ly = e / kTileX, lx = e - ly * kTileX;
        const int gy = y0 + ly - R, gx = x0 + lx;
        float v = 0.f;
        if (gy >= 0 && gy < ny && gx < nx) {
            const long long q = gy * sty + gx;
            v = mp.gam[0][q] * mp.w1[q];
        }
        Zy[ly][lx] = v;
    }
    for (int e = tid; e < kMadjRows * TW; e += 256) {
        const int ly = e / TW, lx = e - ly * TW;
        const int gy = y0 + ly, gx = x0 + lx - R;
        float v = 0.f;
        if (gy < ny && gx >= 0 && gx < nx) {
            const long long q = gy * sty + gx;
            v = mp.gam[1][q] * mp.w1[q];
        }
        Zx[ly][lx] = v;
    }
    __syncthreads();
    const int lx = tid & 63;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int ly = (tid >> 6) * 2 + r;
        const int gy = y0 + ly, gx = x0 + lx;
        if (gy >= ny || gx >= nx)
            continue;
        const int c[3] = {gy, gx, 0};
        const long long p = gy * sty + gx;
        const float w1 = mp.w1[p];
        float lap_y = cf.c0 * Yt[ly + R][lx + R];
        float dens = 0.f;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            float sy = 0.f, sz = 0.f;
#pragma unroll
            for (int jj = 1; jj <= R; ++jj) {
                float yp, ym, zp, zm;
                if (a == 0) {
                    yp = Yt[ly + R + jj][lx + R];
                    ym = Yt[ly + R - jj][lx + R];
                    zp = Zy[ly + R + jj][lx];
                    zm = Zy[ly + R - jj][lx];
                } else {
                    yp = Yt[ly + R][lx + R + jj];
                    ym = Yt[ly + R][lx + R - jj];
                    zp = Zx[ly][lx + R + jj];
                    zm = Zx[ly][lx + R - jj];
                }
                sy = fmaf(cf.c[a][jj], yp + ym, sy);
                sz = fmaf(cf.d[a][jj], zp - zm, sz);
            }
            lap_y += sy;
            dens += sz;
        }
        float eta = sponge_eta(d, sp, c);
        if (mp.att && mp.att_power == 0)
            eta += mp.att[p];
        mp.w0[p] = leapfrog(w1, mp.w2[p], mp.k[p], lap_y - dens, eta, sp.half_dt);
        if (mp.H)
            mp.G[p] = fmaf(w1, mp.H[p], mp.G[p]);
    }
}

// 3D form: the march of the 3D steps.  A block takes a 64 x 8 tile and zc planes,
// a thread two points of a row; the taps along axis 0 of y and of z = gam_0 w^{m+1}
// come from register queues, those in the plane from LDS (y over the tile and
// its whole frame, gam_1 w^{m+1} over the rows of the frame, gam_2 w^{m+1} over its
// columns; two buffers, one barrier per plane).  Bound by memory: eleven fields
// pass once per step.  At 252^3, order 10: 172 us a step (4.1 TB/s of needed
// bytes); 337 with a thread per point and every tap along axis 0 loaded again.
template <int R, bool Y2>
__global__ __launch_bounds__(256) void medium_adjoint3d_kernel(Dims d, StencilCoef cf, SpongeCoef sp,
                                                               LaunchShape ls, MediumAdjParams mp)
{
    constexpr int VX = kVx3dTwo, NT = 64 * kWaves3d;
    using V = StepVec<VX>;
    constexpr int LPR = kTileX / VX, TY = kWaves3d * VX;
    constexpr int HQ = (R + VX - 1) / VX * VX;
    constexpr int LW = kTileX + 2 * HQ, LH = TY + 2 * R;
    constexpr int Q = 2 * R + 1;
    constexpr int NYH = 2 * R * LPR, XPR = 2 * HQ / VX, NH = NYH + XPR * TY;
    constexpr int HL = (NH + NT - 1) / NT;
    __shared__ __align__(16) float sY[2][LH * LW], sZ1[2][LH * kTileX], sZ2[2][TY * LW];

    const int lb = xcd_logical(blockIdx.x, ls.tile_blocks_pad);
    if (lb >= ls.tile_blocks)
        return;
    const int zci = lb / ls.tiles_xy, tile = lb - zci * ls.tiles_xy;
    const int y0 = tile / ls.tiles_x * TY, x0 = tile % ls.tiles_x * kTileX;
    const int n0 = d.n[0], n1 = d.n[1], n2 = d.n[2];
    const int z0 = zci * ls.zc, z1 = min(z0 + ls.zc, n0);
    const long long s0 = d.st[0];
    const int s1 = (int)d.st[1], plane_bytes = (int)(s0 * 4);
    const int tid = (int)threadIdx.x, row = tid / LPR, col = tid % LPR * VX;
    const int gx = x0 + col, gy = y0 + row;
    const int bo = gx < n2 && gy < n1 ? (gy * s1 + gx) * 4 : kNoByte;
    const int lo = (row + R) * LW + col + HQ;
    const bool ragged = n2 % VX != 0 && x0 + kTileX + HQ > n2;
    const int dyd = layer_depth(gy, n1, d.nb);
    const float dy2 = (float)(dyd * dyd);
    float dx2[VX];
#pragma unroll
    for (int k = 0; k < VX; ++k) {
        const int dxd = layer_depth(gx + k, n2, d.nb);
        dx2[k] = (float)(dxd * dxd);
    }
    // frame vectors of this thread: places in y and in z_1 or z_2, byte offset
    int hl[HL], hz[HL], ho[HL], hx[HL];
    bool rows[HL];
#pragma unroll
    for (int h = 0; h < HL; ++h) {
        const int i = tid + h * NT;
        hl[h] = -1;
        hz[h] = hx[h] = 0;
        ho[h] = kNoByte;
        rows[h] = i < NYH;
        if (i < NH) {
            int ly, lx;
            if (i < NYH) {
                const int hr = i / LPR;
                ly = hr < R ? hr - R : TY + hr - R;
                lx = i % LPR * VX;
                hz[h] = (ly + R) * kTileX + lx;
            } else {
                const int c = (i - NYH) % XPR;
                ly = (i - NYH) / XPR;
                lx = c < XPR / 2 ? c * VX - HQ : kTileX + (c - XPR / 2) * VX;
                hz[h] = ly * LW + lx + HQ;
            }
            const int g = x0 + lx, y = y0 + ly;
            hl[h] = (ly + R) * LW + lx + HQ;
            hx[h] = g;
            if (y >= 0 && y < n1 && g >= 0 && g < n2)
                ho[h] = (y * s1 + g) * 4;
        }
    }
    auto rsrc_in = [&](const float* f, int z) { return plane_rsrc(f + z * s0, plane_bytes); };
    auto rsrc = [&](const float* f, int z) {
        const bool in = z >= 0 && z < n0;
        return plane_rsrc(f + (in ? z : 0) * s0, in ? plane_bytes : 0);
    };
    auto operand = [&](const V& w1, const V& w2, const V& at) {
        if constexpr (!Y2)
            return w1;
        V y;
#pragma unroll
        for (int k = 0; k < VX; ++k)
            y[k] = fmaf(at[k], w1[k] - w2[k], w1[k]);
        return y;
    };
    auto product = [&](const V& g, const V& w) {
        V z;
#pragma unroll
        for (int k = 0; k < VX; ++k)
            z[k] = g[k] * w[k];
        return z;
    };
    // raw values of vectors on their way: lead plane, frame, point values
    V lw1, lw2, lat, lg0, fw1[HL], fw2[HL], fat[HL], fg[HL];
    V pw1, pw2, pk, pat, pH, pG, pg1, pg2;
    auto prefetch_lead = [&](int z) {
        lw1 = bloadv<VX, 0>(rsrc(mp.w1, z), bo);
        lg0 = bloadv<VX, 0>(rsrc(mp.gam[0], z), bo);
        if constexpr (Y2) {
            lw2 = bloadv<VX, 0>(rsrc(mp.w2, z), bo);
            lat = bloadv<VX, 0>(rsrc(mp.att, z), bo);
        }
    };
    auto prefetch_frame = [&](int z) {
#pragma unroll
        for (int h = 0; h < HL; ++h) {
            fw1[h] = bloadv<VX, 0>(rsrc_in(mp.w1, z), ho[h]);
            // (the rows of the frame: whole waves)
            fg[h] = rows[h] ? bloadv<VX, 0>(rsrc_in(mp.gam[1], z), ho[h])
                            : bloadv<VX, 0>(rsrc_in(mp.gam[2], z), ho[h]);
            if constexpr (Y2) {
                fw2[h] = bloadv<VX, 0>(rsrc_in(mp.w2, z), ho[h]);
                fat[h] = bloadv<VX, 0>(rsrc_in(mp.att, z), ho[h]);
            }
        }
        pg1 = bloadv<VX, 0>(rsrc_in(mp.gam[1], z), bo);
        pg2 = bloadv<VX, 0>(rsrc_in(mp.gam[2], z), bo);
        if constexpr (Y2)
            pw1 = bloadv<VX, 0>(rsrc_in(mp.w1, z), bo);
    };
    auto prefetch_points = [&](int z) {
        pw2 = bloadv<VX, 0>(rsrc_in(mp.w2, z), bo);
        pk = bloadv<VX, 0>(rsrc_in(mp.k, z), bo);
        if constexpr (!Y2)      // (no attenuation: an empty descriptor, loads of 0)
            pat = bloadv<VX, 0>(mp.att ? rsrc_in(mp.att, z) : plane_rsrc(mp.k, 0), bo);
        pH = bloadv<VX, STRIDE_STREAM_AUX>(mp.H ? rsrc_in(mp.H, z) : plane_rsrc(mp.k, 0), bo);
        pG = bloadv<VX, 0>(rsrc_in(mp.G, z), bo);
    };

    // queue slot (i + t) % Q holds plane z0 + i + t - R at march iteration i
    V qy[Q], qz[Q];
#pragma unroll
    for (int t = 0; t < 2 * R; ++t) {
        prefetch_lead(z0 - R + t);
        qy[t] = operand(lw1, lw2, lat);
        qz[t] = product(lg0, lw1);
    }
    prefetch_lead(z0 + R);
    prefetch_frame(z0);
    prefetch_points(z0);

    int buf = 0;
    for (int zb = z0; zb < z1; zb += Q)
        unrolled_while<Q>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            constexpr int slot_lead = (u + 2 * R) % Q, slot_c = (u + R) % Q;
            const int z = zb + u;
            if (z >= z1)
                return false;
            qy[slot_lead] = operand(lw1, lw2, lat);
            qz[slot_lead] = product(lg0, lw1);
            const V w1 = Y2 ? pw1 : qy[slot_c];
            float *Y = sY[buf], *Z1 = sZ1[buf], *Z2 = sZ2[buf];
            *(V*)&Y[lo] = qy[slot_c];
            *(V*)&Z1[(row + R) * kTileX + col] = product(pg1, w1);
            *(V*)&Z2[row * LW + col + HQ] = product(pg2, w1);
#pragma unroll
            for (int h = 0; h < HL; ++h)
                if (hl[h] >= 0) {
                    *(V*)&Y[hl[h]] = operand(fw1[h], fw2[h], fat[h]);
                    *(V*)&(rows[h] ? Z1 : Z2)[hz[h]] = product(fg[h], fw1[h]);
                }
            if (ragged) {
#pragma unroll
                for (int k = 1; k < VX; ++k) {
                    if (gx + k >= n2)
                        Y[lo + k] = Z2[row * LW + col + HQ + k] = 0.f;
#pragma unroll
                    for (int h = 0; h < HL; ++h)
                        if (hl[h] >= 0 && hx[h] + k >= n2) {
                            Y[hl[h] + k] = 0.f;
                            if (!rows[h])
                                Z2[hz[h] + k] = 0.f;
                        }
                }
            }
            if (z + 1 < z1) {
                prefetch_lead(z + 1 + R);
                prefetch_frame(z + 1);
            }
            __syncthreads();

            // centre, then per axis the taps j = 1 .. R
            V lap, dens = V(0.f), sy = V(0.f), sz = V(0.f);
#pragma unroll
            for (int k = 0; k < VX; ++k)
                lap[k] = cf.c0 * qy[slot_c][k];
            auto add = [&]() {
#pragma unroll
                for (int k = 0; k < VX; ++k) {
                    lap[k] += sy[k];
                    dens[k] += sz[k];
                }
                sy = sz = V(0.f);
            };
            auto tap = [&](int a, int j, const V& yp, const V& ym, const V& zp, const V& zm) {
#pragma unroll
                for (int k = 0; k < VX; ++k) {
                    sy[k] = fmaf(cf.c[a][j], yp[k] + ym[k], sy[k]);
                    sz[k] = fmaf(cf.d[a][j], zp[k] - zm[k], sz[k]);
                }
            };
#pragma unroll
            for (int j = 1; j <= R; ++j)
                tap(0, j, qy[(u + R + j) % Q], qy[(u + R - j + Q) % Q], qz[(u + R + j) % Q],
                    qz[(u + R - j + Q) % Q]);
            add();
            const float* Zc = Z1 + (row + R) * kTileX + col;
#pragma unroll
            for (int j = 1; j <= R; ++j)
                tap(1, j, *(const V*)(Y + lo + j * LW), *(const V*)(Y + lo - j * LW),
                    *(const V*)(Zc + j * kTileX), *(const V*)(Zc - j * kTileX));
            add();
            __builtin_amdgcn_sched_barrier(0);      // bounds the LDS vectors in flight
            {
                float xs[VX + 2 * HQ], zs[VX + 2 * HQ];
#pragma unroll
                for (int i = 0; i < VX + 2 * HQ; i += VX) {
                    const V a = *(const V*)(Y + lo - HQ + i);
                    const V c = *(const V*)(Z2 + row * LW + col + i);
#pragma unroll
                    for (int k = 0; k < VX; ++k) {
                        xs[i + k] = a[k];
                        zs[i + k] = c[k];
                    }
                }
#pragma unroll
                for (int j = 1; j <= R; ++j)
#pragma unroll
                    for (int k = 0; k < VX; ++k) {
                        sy[k] = fmaf(cf.c[2][j], xs[HQ + k + j] + xs[HQ + k - j], sy[k]);
                        sz[k] = fmaf(cf.d[2][j], zs[HQ + k + j] - zs[HQ + k - j], sz[k]);
                    }
            }
            add();
            const int dzd = layer_depth(z, n0, d.nb);
            const float e0 = fmaf(sp.e[0], (float)(dzd * dzd), 0.f);
            V out, G;
#pragma unroll
            for (int k = 0; k < VX; ++k) {
                float eta = fmaf(sp.e[2], dx2[k], fmaf(sp.e[1], dy2, e0));
                if constexpr (!Y2)
                    eta = mp.att ? eta + pat[k] : eta;
                out[k] = leapfrog(w1[k], pw2[k], pk[k], lap[k] - dens[k], eta, sp.half_dt);
                G[k] = fmaf(w1[k], pH[k], pG[k]);
            }
            bstorev<VX>(rsrc_in(mp.w0, z), bo, out);
            if (mp.H)
                bstorev<VX>(rsrc_in(mp.G, z), bo, G);
            if (z + 1 < z1)
                prefetch_points(z + 1);
            buf ^= 1;
            return true;
        });
}

template <int R>
void launch_medium_adjoint_r(const Dims& d, const StencilCoef& cf, const SpongeCoef& sp,
                             const LaunchShape& ls, const MediumAdjParams& mp, hipStream_t s)
{
    const bool y2 = mp.att && mp.att_power == 2;
    if (d.nd == 3) {
        const dim3 g((unsigned)ls.tile_blocks_pad), b(64 * kWaves3d);
        if (y2)
            hipLaunchKernelGGL((medium_adjoint3d_kernel<R, true>), g, b, 0, s, d, cf, sp, ls, mp);
        else
            hipLaunchKernelGGL((medium_adjoint3d_kernel<R, false>), g, b, 0, s, d, cf, sp, ls, mp);
        return;
    }
    const dim3 g((unsigned)((d.n[1] + kTileX - 1) / kTileX),
                 (unsigned)((d.n[0] + kMadjRows - 1) / kMadjRows));
    if (y2)
        hipLaunchKernelGGL((medium_adjoint_kernel<R, true>), g, dim3(256), 0, s, d, cf, sp, mp);
    else
        hipLaunchKernelGGL((medium_adjoint_kernel<R, false>), g, dim3(256), 0, s, d, cf, sp, mp);
}

void launch_medium_adjoint(const Dims& d, int R, const StencilCoef& cf, const SpongeCoef& sp,
                           const LaunchShape& ls, const MediumAdjParams& mp, hipStream_t s)
{
    R == 4 ? launch_medium_adjoint_r<4>(d, cf, sp, ls, mp, s)
           : launch_medium_adjoint_r<5>(d, cf, sp, ls, mp, s);
}

// One block per step-kernel block of the table's launch shape; each thread
// takes the table's entries tid, tid + 256, ...; the first entry of a point
// sums the point's run in entry order (so every point is written by one
// thread, and always in the same order).
__global__ __launch_bounds__(256) void inject_table_kernel(Dims d, LaunchShape ls, InjTable T,
                                                           const float* sig, int stride, int step,
                                                           const float* k, const float* att,
                                                           int att_power, SpongeCoef sp, float* out)
{
    const int b = blockIdx.x;
    const int e0 = T.ptr[b], e1 = T.ptr[b + 1];
    const int zci = b / ls.tiles_xy;
    const int tile = b - zci * ls.tiles_xy;
    const int y0 = (tile / ls.tiles_x) * ls.ty;
    const int x0 = (tile % ls.tiles_x) * kTileX;
    const int plane = ls.ty * kTileX;
    for (int e = e0 + (int)threadIdx.x; e < e1; e += blockDim.x) {
        const TileEntry head = T.ent[e];
        if (head.run <= 0)
            continue;
        const float v = tile_point_signal(T.ent + e, head, sig, stride, step);
        const int pz = head.local / plane;
        const int rem = head.local - pz * plane;
        int c[3];
        if (d.nd == 3) {
            c[0] = zci * ls.zc + pz;
            c[1] = y0 + rem / kTileX;
            c[2] = x0 + rem % kTileX;
        } else {
            c[0] = y0 + rem / kTileX;
            c[1] = x0 + rem % kTileX;
            c[2] = 0;
        }
        const long long p = d.nd == 3 ? c[0] * d.st[0] + c[1] * d.st[1] + c[2] : c[0] * d.st[0] + c[1];
        float eta = sponge_eta(d, sp, c);
        if (att && att_power == 0)
            eta += att[p];
        const float a = eta == 0.f ? 1.f : __builtin_amdgcn_rcpf(fmaf(eta, sp.half_dt, 1.f));
        out[p] = fmaf(a * k[p], v, out[p]);
    }
}

void launch_inject_table(const Dims& d, const LaunchShape& ls, const InjTable& T, const float* sig,
                         int stride, int step, const float* k, const float* att, int att_power,
                         const SpongeCoef& sp, float* out, hipStream_t s)
{
    if (ls.tile_blocks <= 0)
        return;
    hipLaunchKernelGGL(inject_table_kernel, dim3(ls.tile_blocks), dim3(256), 0, s, d, ls, T, sig,
                       stride, step, k, att, att_power, sp, out);
}

void launch_vp_check(const float* vp, long long n, unsigned* flags, hipStream_t s)
{
    launch_fill(reinterpret_cast<float*>(flags), 2, 0.f, s);
    hipLaunchKernelGGL(vp_check_kernel, dim3(grid_for(n, 256) < 1024 ? grid_for(n, 256) : 1024),
                       dim3(256), 0, s, vp, n, flags);
}

void launch_prep_medium(const Dims& d, const Fd1& fd, const float* vp, const float* rho,
                        const float* alpha0, int att_power, double dt, float* const gam[3],
                        float* att, double* lr, hipStream_t s)
{
    long long n = (long long)d.n[0] * d.n[1] * d.n[2];
    const long long np = (long long)d.phys[0] * d.phys[1] * d.phys[2];
    if (rho)
        hipLaunchKernelGGL(ln_kernel, dim3(grid_for(np, 256)), dim3(256), 0, s, rho, np, lr);
    hipLaunchKernelGGL(prep_medium_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, d, fd, vp,
                       rho ? lr : nullptr, alpha0, att_power, dt, gam[0], gam[1], d.nd == 3 ? gam[2] : gam[1], att);
}

void launch_medium_check(const float* vp, const float* rho, const float* alpha0, long long n,
                         int att_power, double dt, unsigned* flags, hipStream_t s)
{
    launch_fill(reinterpret_cast<float*>(flags + 2), 2, 0.f, s);
    hipLaunchKernelGGL(medium_check_kernel, dim3(grid_for(n, 256) < 1024 ? grid_for(n, 256) : 1024),
                       dim3(256), 0, s, vp, rho, alpha0, n, att_power, dt, flags);
}

void launch_time_filter3(float* rows, int count, int nt, hipStream_t s)
{
    if (count <= 0 || nt <= 0)
        return;
    hipLaunchKernelGGL(time_filter3_kernel, dim3(count), dim3(256), sizeof(float) * (size_t)nt, s, rows,
                       nt);
}

int lowpass_taps(double dt, double f_max)
{
    return (int)std::ceil(2.0 / (f_max * dt));
}

void launch_lowpass(const float* in, float* out, int count, int nt, double dt, double f_max,
                    hipStream_t s)
{
    const int K = lowpass_taps(dt, f_max);
    const size_t lds = sizeof(float) * (size_t)(2 * K + 1 + nt);
    hipLaunchKernelGGL(lowpass_kernel, dim3(count), dim3(256), lds, s, in, out, nt, f_max * dt, K);
}

void launch_descent(float* vp, const float* g, const float* mask, long long n, float step,
                    float vmin, float vmax, unsigned* work, hipStream_t s)
{
    launch_fill(reinterpret_cast<float*>(work), 1, 0.f, s);
    const int blocks = grid_for(n, 256) < 1024 ? grid_for(n, 256) : 1024;
    hipLaunchKernelGGL(grad_absmax_kernel, dim3(blocks), dim3(256), 0, s, g, mask, n, work);
    hipLaunchKernelGGL(descent_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, vp, g, mask, n, step,
                       vmin, vmax, work);
}

void launch_prep_k(const Dims& d, const float* vp, double dt, float* k, hipStream_t s)
{
    long long n = (long long)d.n[0] * d.n[1] * d.n[2];
    hipLaunchKernelGGL(prep_k_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, d, vp, dt, k);
}

void launch_residual_misfit(const float* traces, const float* observed, float* residual,
                            long long n, double* misfit, double* partial, hipStream_t s)
{
    hipLaunchKernelGGL(residual_partial_kernel, dim3(kMisfitParts), dim3(256), 0, s, traces,
                       observed, residual, n, partial);
    hipLaunchKernelGGL(misfit_final_kernel, dim3(1), dim3(256), 0, s, partial, kMisfitParts, misfit);
}

void launch_finalize_dvp(const Dims& d, const float* G, const float* kdiv, const float* vp,
                         float* dvp, float* tmp0, float* tmp1, hipStream_t s)
{
    // P^T one axis at a time, innermost first; the first pass reads the
    // pitched field, later passes dense intermediates, the last writes dvp.
    const int nd = d.nd;
    long long ext[3] = {d.n[0], d.n[1], d.n[2]};
    const float* in = G;
    float* tmp[2] = {tmp0, tmp1};
    for (int a = nd - 1; a >= 0; --a) {
        long long m0 = 1, m2 = 1;
        for (int q = 0; q < a; ++q)
            m0 *= ext[q];
        for (int q = a + 1; q < nd; ++q)
            m2 *= ext[q];
        const long long s_outer = a == nd - 1 ? d.st[nd - 2] : ext[a] * m2;
        const long long s_axis = a == nd - 1 ? 1 : m2;
        float* out = a == 0 ? dvp : tmp[a & 1];
        const long long cnt = m0 * d.phys[a] * m2;
        hipLaunchKernelGGL(pad_transpose_axis_kernel, dim3(grid_for(cnt, 256)), dim3(256), 0, s, in,
                           a == nd - 1 ? kdiv : nullptr, s_outer, s_axis, out, m0, d.phys[a], m2,
                           d.nb, a == 0 ? vp : nullptr);
        ext[a] = d.phys[a];
        in = out;
    }
}

}  // namespace stride
