// Analog random-walk cell transmission for gfx950 (paper: section "Monte Carlo Method",
// eq. 4 flight lengths, implicit capture of eqs. 5-6): the walk kernel over the engine of
// gmc_walk.hpp, the first-flight split and the standalone exit decoder.
#include "gmc_device.hpp"
#include "gmc_internal.hpp"
#include "gmc_walk.hpp"

namespace gmc {

namespace {

constexpr int kWalkThreads = 256;

// The conditions p.* of walks 0 .. n-1 to their exit records (see run_walks).  Bound by vector
// issue, then by the longest walk; six blocks per CU (80 registers a lane).
// The XY kernels spill 18 and 25 registers, all but one outside the loops over flights (stored where the regime
// changes, read where a walk ends): 2^20 walks of mixed cells 150 us against 109 in flatland, at
// tau = 100 951 against 609, with 1.27 times the flights (E[path] = 1 against pi / 4).
template <bool ANALOG, bool XY>
__global__ __launch_bounds__(kWalkThreads, kWalkBlocksPerCu) void walk_kernel(WalkParams p)
{
    __shared__ WalkGroups groups[kWalkThreads / 64];
    __shared__ uint32_t pool;
    run_walks<ANALOG, XY, false>(
        p.n, p.seed, groups, &pool,
        [&](int64_t i) {
            WalkStart w;
            const float s = p.sin_th[i];
            const float la = p.log_aspect ? p.log_aspect[i] : 0.0f;
            w.wa = la == 0.0f ? 1.0f : expf(la);
            w.x = p.x_in ? p.x_in[i] : 0.0f;       // birth inside the cell, or entry on the left face
            w.y = p.y_in[i];
            w.u = p.x_in ? p.cos_phi[i] : (XY ? p.omega_x[i] : sqrtf(fmaxf(__builtin_fmaf(-s, s, 1.0f), 0.0f)));
            w.v = s;
            w.tau = expf(p.log_tau[i]);
            w.c = p.c[i];
            w.stream = p.id_base + (uint64_t)i;
            w.key = p.seed;
            return w;
        },
        [&](int64_t i, int face, float pos, float u, float v, float len, uint32_t ncoll) {
            p.face[i] = face;
            p.pos[i] = pos;
            p.dcos[i] = u;
            p.dsin[i] = v;
            p.path[i] = len;
            if (p.ncoll) p.ncoll[i] = ncoll;
        });
}

template <bool ANALOG>
void launch_walk_mode(const WalkParams &p, int grid, hipStream_t s)
{
    const dim3 g(grid), b(kWalkThreads);
    if (p.omega_x && !p.x_in) hipLaunchKernelGGL((walk_kernel<ANALOG, true>), g, b, 0, s, p);
    else hipLaunchKernelGGL((walk_kernel<ANALOG, false>), g, b, 0, s, p);
}

__global__ __launch_bounds__(256) void decode_kernel(const float *__restrict__ raw, int64_t n,
                                                     int32_t *face, float *pos, float *dcos,
                                                     float *dsin, float *path, int32_t *flags)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Exit e;
    const int f = decode_exit(raw[i], raw[n + i], raw[2 * n + i], raw[3 * n + i], raw[4 * n + i], e);
    face[i] = e.face;
    pos[i] = e.pos;
    dcos[i] = e.u;
    dsin[i] = e.v;
    path[i] = e.path;
    if (flags) flags[i] = f;
}

}  // namespace

hipError_t launch_walk(const WalkParams &p, int grid, hipStream_t s)
{
    if (p.mode == 1) launch_walk_mode<true>(p, grid, s);
    else launch_walk_mode<false>(p, grid, s);
    return hipGetLastError();
}

// First-flight split of n canonical transmissions (uncollided_exit): flag[i] = 1 and the exit
// record written for an uncollided crossing, flag[i] = 0 and the record left untouched otherwise.
__global__ __launch_bounds__(256) void split_kernel(WalkParams p, int32_t *flag)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.n) return;
    const float s = p.sin_th[i];
    const float la = p.log_aspect ? p.log_aspect[i] : 0.0f;
    const float wa = la == 0.0f ? 1.0f : expf(la);
    const float u = p.omega_x ? p.omega_x[i] : sqrtf(fmaxf(1.0f - s * s, 0.0f));
    Exit e;
    const bool unc = uncollided_exit(expf(p.log_tau[i]), p.c[i], p.y_in[i], u, s, wa,
                                     split_draw(p.seed, p.id_base + (uint64_t)i), e);
    flag[i] = unc ? 1 : 0;
    if (unc) {
        p.face[i] = e.face;
        p.pos[i] = e.pos;
        p.dcos[i] = e.u;
        p.dsin[i] = e.v;
        p.path[i] = e.path;
    }
}

hipError_t launch_split(const WalkParams &p, int32_t *flag, hipStream_t s)
{
    const int64_t blocks = (p.n + 255) / 256;
    hipLaunchKernelGGL(split_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, flag);
    return hipGetLastError();
}

hipError_t launch_decode(const float *raw, int64_t n, int32_t *face, float *pos, float *dcos,
                         float *dsin, float *path, int32_t *flags, hipStream_t s)
{
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(decode_kernel, dim3((unsigned)blocks), dim3(256), 0, s, raw, n, face, pos,
                       dcos, dsin, path, flags);
    return hipGetLastError();
}

}  // namespace gmc
