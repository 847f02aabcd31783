// disk.hip -- the thin-disk line test (Sec. 4.2.1) on the GPU: one lane per pixel integrates
// its ray with the chosen integrator until the first crossing of the equatorial plane, locates
// the crossing by Newton iterations on theta(lambda) (each an integrated partial step from the
// state before the crossing), and, if the crossing lies on the Keplerian disk between the ISCO
// and the outer radius, records the ratio g = E_obs/E_em and the observed intensity g^3 r^-2
// (emission proportional to r^-2, no absorption; higher-order images are not counted).  Two
// further kernels bin the pixel fluxes by g into the line profile, in a fixed order.
#include "device_types.hpp"
#include "ks_geodesic.hpp"
#include "plasma.hpp"
#include "launch.hpp"

#include <algorithm>

namespace {

constexpr double HALF_PI = 1.5707963267948966;

// One step, and sin and cos of theta with it (those of y[2] on entry and on return).
template <int INTEG>
__device__ inline void disk_step(const rk::Spin<double>& sp, double* y, double* acc, bool& have_acc, double dl,
                                 bool corrector, bool chained, double* s, double* c)
{
    if (INTEG == INTEG_RK4) {
        rk::rk4_step_angles(sp, y, dl, chained, s, c);
        return;
    }
    const double th0 = y[2], s0 = *s, c0 = *c;
    if (INTEG == INTEG_RK2) {
        rk::rk2_step(sp, y, dl, s0, c0);
    } else {
        if (!have_acc) rk::ks_accel<true>(sp, y, s0, c0, acc);
        rk::verlet_step(sp, y, acc, dl, corrector, s0, c0);
        have_acc = true;
    }
    rk::sincos_shift(th0, s0, c0, y[2], s, c);
}

// One lane per pixel, a wave per 8 x 8 pixels (whose rays end after about as many steps; 64 pixels of
// a row took a tenth more iterations).  Bound by vector-instruction issue for many tiles (424
// instructions an iteration, 67% of the issue rate at 1024^2) and by the longest ray below a round of
// them (650 steps of 1.2 us).  A ray that has crossed the plane keeps the step before the crossing and
// waits for the rays of its wave: the lanes cross at many different steps, and refined where each one
// crosses, the three further steps of a crossing ran for the whole wave every time.  Work-groups of
// one wave take tiles from a counter.  Three waves per SIMD hold the registers without scratch (the
// test of eps has to stay in the loop: hoisted, it is compiled into two loops, with scratch).
// Measured before and after (ms, a = 0.9375, i = 60 deg, RK4): 64^2 1.02 0.66; 256^2 1.23 0.79; 512^2
// 1.49 1.18; 724^2 2.84 1.81.
template <int INTEG, int WPE = 3>
__global__ void __attribute__((amdgpu_flat_work_group_size(DISK_THREADS, DISK_THREADS), amdgpu_waves_per_eu(WPE, 8)))
disk_kernel(DiskParams p)
{
    const int tiles_x = (int)((p.nx + 7u) / 8u), tiles_y = (int)((p.ny + 7u) / 8u), tiles = tiles_x * tiles_y;
    const rk::Spin<double> sp = rk::make_spin(p.a, p.M);
    const bool corrector = p.integrator == INTEG_VERLET_CORR;
    unsigned long long c_steps = 0, c_disk = 0;
    // the state before the step, in LDS: 24 registers that the step needs at three waves per SIMD
    __shared__ double keep[INTEG == INTEG_VERLET ? 14 : 10][DISK_THREADS];
    const int lane = threadIdx.x;
    for (int tile = blockIdx.x; tile < tiles;) {
        // rows from the middle outwards: those around the hole hold the longest rays
        const int k = tile / tiles_x, row = tiles_y / 2 + ((k & 1) ? -(k + 1) / 2 : k / 2);
        const int px = tile % tiles_x * 8 + (lane & 7), py = row * 8 + (lane >> 3);
        const bool inside = (unsigned)px < (unsigned)p.nx && (unsigned)py < (unsigned)p.ny;
        const long long pix = (long long)py * p.nx + px;
        const double alpha = -p.fov + (px + 0.5) * p.dalpha;
        const double beta = -p.fov + (py + 0.5) * p.dbeta;
        double y[8], acc[4] = {0.0, 0.0, 0.0, 0.0};
        bool have_acc = false, had_acc = false;
        rk::camera_ray(p.cam, alpha, beta, y);
        double s, c, lam = 0.0;
        rt::sincos_small(y[2], &s, &c);
        int steps = 0, status = inside ? RAY_RUNNING : RAY_IDLE;
        double g = 0.0, I = 0.0;
        while (status == RAY_RUNNING) {
            const double dl = -rk::step_size(p.eps, y);
            const double h0 = y[2] - HALF_PI;
#pragma unroll
            for (int i = 0; i < 8; ++i) keep[i][lane] = y[i];
            keep[8][lane] = s;
            keep[9][lane] = c;
            if (INTEG == INTEG_VERLET) {
#pragma unroll
                for (int i = 0; i < 4; ++i) keep[10 + i][lane] = acc[i];
                had_acc = have_acc;
            }
            disk_step<INTEG>(sp, y, acc, have_acc, dl, corrector, p.eps <= rk::EPS_CHAINED, &s, &c);
            ++steps;
            const double h1 = y[2] - HALF_PI;
            // a sum is finite only if its terms are (one that overflows is looked at again)
            if (!::isfinite(((y[0] + y[1]) + (y[2] + y[3])) + ((y[4] + y[5]) + (y[6] + y[7])))) {
                bool fin = true;
#pragma unroll
                for (int i = 0; i < 8; ++i) fin = fin && ::isfinite(y[i]);
                if (!fin) status = RAY_NUMERIC;
            }
            if (status != RAY_RUNNING) {
            } else if (h0 * h1 < 0.0) {
                lam = dl * h0 / (h0 - h1);   // linear estimate of the crossing's affine parameter
                status = RAY_PLANE;
            } else {
                if (rk::reflect_pole(y)) {
                    have_acc = false;
                    rt::sincos_small(y[2], &s, &c);
                }
                if (y[1] < p.r_stop)
                    status = RAY_HORIZON;
                else if (y[1] > p.cam.r)
                    status = RAY_ESCAPED;
                else if (steps >= p.max_steps)
                    status = RAY_MAXSTEP;
            }
        }
        if (status == RAY_PLANE) {
#pragma unroll 1
            for (int it = 0; it < 3; ++it) {   // two Newton iterations
#pragma unroll
                for (int i = 0; i < 8; ++i) y[i] = keep[i][lane];
                s = keep[8][lane];
                c = keep[9][lane];
                if (INTEG == INTEG_VERLET) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i] = keep[10 + i][lane];
                    have_acc = had_acc;
                }
                disk_step<INTEG>(sp, y, acc, have_acc, lam, corrector, p.eps <= rk::EPS_CHAINED, &s, &c);
                if (it < 2) lam += (HALF_PI - y[2]) / y[6];
            }
            const double rc = y[1];
            if (rc >= p.r_in && rc <= p.r_out) {
                const double omega = 1.0 / (rc * ::sqrt(rc) + p.a);
                double nr, cb;
                rt::sincos_small(y[2], &s, &c);
                pl::fluid_frame(p.a, p.a * p.a, p.M, y, s, c, omega, &nr, &cb);
                g = 1.0 / nr;
                I = g * g * g / (rc * rc);
                status = RAY_DISK;
            }
        }
        if (inside) {
            if (p.intensity) p.intensity[pix] = I;
            if (p.redshift) p.redshift[pix] = g;
            if (p.status) p.status[pix] = status;
            if (p.steps) p.steps[pix] = steps;
        }
        c_steps += steps;
        c_disk += status == RAY_DISK;
        // the next tile of the launch (the counter starts behind the waves' first ones)
        unsigned next = 0;
        if (lane == 0) next = (unsigned)atomicAdd(p.counter, 1ull);
        tile = (int)__builtin_amdgcn_readfirstlane(next);
    }
    // one atomic per wave and counter
    for (int off = 32; off > 0; off >>= 1) {
        c_steps += __shfl_down(c_steps, off, 64);
        c_disk += __shfl_down(c_disk, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(p.stats + 0, c_steps);
        atomicAdd(p.stats + 1, c_disk);
    }
}

// profile[b] = sum of intensity * dA over the pixels whose g falls in bin b, in a fixed order.
// Pass 1: one work-group per chunk of pixels and PROFILE_BINS bins, a sum per bin in each lane and a
// fixed tree over the lanes.  Pass 2: one lane per bin adds its chunks in order.  (One work-group per
// bin over all pixels read every image 256 times, one load at a time in flight: 405 us for 512^2
// pixels and 256 bins.)
constexpr int PROFILE_BINS = 16;

__global__ void __launch_bounds__(256) disk_profile_kernel(const double* intensity, const double* redshift,
                                                           long long n, long long chunk, int n_bins, double g_lo,
                                                           double g_hi, double dA, double* part)
{
    const int b0 = blockIdx.x * PROFILE_BINS;
    const long long first = (long long)blockIdx.y * chunk;
    const long long last = first + chunk < n ? first + chunk : n;
    double s[PROFILE_BINS];
#pragma unroll
    for (int k = 0; k < PROFILE_BINS; ++k) s[k] = 0.0;
    for (long long i = first + threadIdx.x; i < last; i += 256) {
        const double I = intensity[i];
        const double q = (redshift[i] - g_lo) / (g_hi - g_lo) * n_bins;
        const int bin = I > 0.0 && q >= 0.0 && q < (double)n_bins ? (int)q - b0 : -1;
#pragma unroll
        for (int k = 0; k < PROFILE_BINS; ++k) s[k] += bin == k ? I * dA : 0.0;
    }
    __shared__ double red[4][PROFILE_BINS];
#pragma unroll
    for (int k = 0; k < PROFILE_BINS; ++k) {
        for (int off = 32; off > 0; off >>= 1) s[k] += __shfl_down(s[k], off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][k] = s[k];
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < PROFILE_BINS && b0 + k < n_bins)
        part[(long long)blockIdx.y * n_bins + b0 + k] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
}

__global__ void __launch_bounds__(64) disk_profile_sum_kernel(const double* part, int chunks, int n_bins,
                                                              double* profile)
{
    const int b = blockIdx.x * 64 + threadIdx.x;
    if (b >= n_bins) return;
    double s = 0.0;
#pragma unroll 8
    for (int k = 0; k < chunks; ++k) s += part[(long long)k * n_bins + b];
    profile[b] = s;
}

}  // namespace

hipError_t launch_disk(const DiskParams& p, int blocks, hipStream_t st)
{
    if (p.integrator == INTEG_RK2)
        hipLaunchKernelGGL(disk_kernel<INTEG_RK2>, dim3(blocks), dim3(DISK_THREADS), 0, st, p);
    else if (p.integrator == INTEG_VERLET || p.integrator == INTEG_VERLET_CORR)
        hipLaunchKernelGGL(disk_kernel<INTEG_VERLET>, dim3(blocks), dim3(DISK_THREADS), 0, st, p);
    else
        hipLaunchKernelGGL(disk_kernel<INTEG_RK4>, dim3(blocks), dim3(DISK_THREADS), 0, st, p);
    return hipGetLastError();
}

// Chunks of at least 4096 pixels, no more than 256 of them and no more than 8 MB of partial sums.
int disk_profile_chunks(long long n, int n_bins)
{
    const long long most = std::max(1, std::min(256, (1 << 20) / n_bins));
    return (int)std::min((n + 4095) / 4096, most);
}

hipError_t launch_disk_profile(const double* intensity, const double* redshift, long long n, int n_bins, double g_lo,
                               double g_hi, double dA, double* part, double* profile, hipStream_t st)
{
    const int chunks = disk_profile_chunks(n, n_bins);
    hipLaunchKernelGGL(disk_profile_kernel, dim3((n_bins + PROFILE_BINS - 1) / PROFILE_BINS, chunks), dim3(256), 0,
                       st, intensity, redshift, n, (n + chunks - 1) / chunks, n_bins, g_lo, g_hi, dA, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(disk_profile_sum_kernel, dim3((n_bins + 63) / 64), dim3(64), 0, st, part, chunks, n_bins,
                       profile);
    return hipGetLastError();
}
