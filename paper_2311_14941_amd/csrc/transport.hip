// Transport step of the operator-split driver: explicit first-order upwind
// advection along x plus diffusion on a uniform 2-D grid, every cell with
// its own (local) time step.  This is the cheap mixing operator that sits
// between chemistry substeps (paper Sec. 2.5: chemistry per cell, local time
// stepping); it is not part of the chemistry integration.
//
// With u >= 0, Co = u dt/dx, Fo = D dt/dx^2 and Co + 4 Fo <= 1 the update
//   q' = q - Co (q - q_W) + Fo (q_E + q_W + q_N + q_S - 4 q)
// is a convex combination of neighbouring values, so mass fractions stay in
// [0, 1] and keep summing to one.  Boundaries: x = 0 takes the inflow
// profile (Dirichlet), the other three are zero-gradient.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace scdev {

// One thread per cell and group of KC components (species-major rows of ld
// values, cells row-major c = iy*nx + ix).  Bound by memory: a row is read
// once from HBM (its north, south, east and west reads hit the caches) and
// written once.  The cell's place and its two coefficients, an integer and
// two double divisions, are taken once per KC values; with one thread per
// value, divided out of a 64-bit index, the arithmetic was the bound.
// Consecutive workgroups go to the eight dies in turn, each with its own L2: a
// die takes a contiguous part of the work instead, so that the rows to the
// north and south are in the L2 that read them, and the stores go past the
// caches that hold those rows.  601 x 512 cells and 54 rows, 271 MB: 112 us with
// a thread per value, 87 with six, 86 with the dies' parts, 82 with the stores;
// 88, 86 and 85 with two, three and nine components a thread.
constexpr int KC = 6;
constexpr uint32_t DIES = 8;
__global__ void __launch_bounds__(256) k_transport2d(int nx, int ny, int ncomp, const double *in, int64_t ld,
                                                     const double *u, const double *dt, double dx, double D,
                                                     const double *inflow, double *out, int64_t c0)
{
    const int64_t n = (int64_t)nx * ny;
    uint32_t bx = blockIdx.x, by = blockIdx.y;
    if ((uint64_t)gridDim.x * gridDim.y <= INT32_MAX) {
        const uint32_t b = by * gridDim.x + bx, all = gridDim.x * gridDim.y, die = b % DIES;
        const uint32_t t = die * (all / DIES) + min(die, all % DIES) + b / DIES;
        by = t / gridDim.x;
        bx = t - by * gridDim.x;
    }
    const int64_t c = c0 + (int64_t)bx * blockDim.x + threadIdx.x;
    if (c >= n) return;
    int iy, ix;
    if (n <= INT32_MAX) {
        iy = (int)((uint32_t)c / (uint32_t)nx);
        ix = (int)((uint32_t)c - (uint32_t)iy * (uint32_t)nx);
    } else {
        iy = (int)(c / nx);
        ix = (int)(c - (int64_t)iy * nx);
    }
    const double co = u[c] * dt[c] / dx;
    const double fo = D * dt[c] / (dx * dx);
    const int64_t e = ix < nx - 1 ? 1 : 0, s = iy > 0 ? -nx : 0, nth = iy < ny - 1 ? nx : 0;
    for (int64_t k0 = (int64_t)by * KC; k0 < ncomp; k0 += (int64_t)gridDim.y * KC) {
        double v[KC][5];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int64_t kk = min(k0 + k, (int64_t)ncomp - 1);
            const double *q = in + kk * ld + c;
            const double *w = ix > 0 ? q - 1 : inflow + kk * ny + iy;
            v[k][0] = q[0];
            v[k][1] = *w;
            v[k][2] = q[e];
            v[k][3] = q[nth];
            v[k][4] = q[s];
        }
#pragma unroll
        for (int k = 0; k < KC; ++k)
            if (k0 + k < ncomp)
                __builtin_nontemporal_store(v[k][0] - co * (v[k][0] - v[k][1]) +
                                                fo * (v[k][2] + v[k][1] + v[k][3] + v[k][4] - 4.0 * v[k][0]), out + (k0 + k) * ld + c);
    }
}

hipError_t launch_transport2d(int nx, int ny, int ncomp, const double *in, int64_t ld, const double *u,
                              const double *dt, double dx, double D, const double *inflow, double *out,
                              hipStream_t s)
{
    const int64_t n = (int64_t)nx * ny, part = (int64_t)1 << 31;  // cells of one launch, below its 2^32 threads
    const unsigned gy = (unsigned)std::min<int64_t>((ncomp + (int64_t)KC - 1) / KC, 65535);
    for (int64_t c0 = 0; c0 < n; c0 += part) {
        const unsigned gx = (unsigned)((std::min(part, n - c0) + 255) / 256);
        hipLaunchKernelGGL(k_transport2d, dim3(gx, gy), dim3(256), 0, s, nx, ny, ncomp, in, ld, u, dt, dx, D, inflow,
                           out, c0);
    }
    return hipGetLastError();
}

}  // namespace scdev
