// The three drifts of a step, D_x D_y D_z of Eq. (5), on small spatial meshes
// in one launch (FP32 storage): the bits of vlasov_advect_z, _y, _x in
// sequence.
//
// A drift does not mix velocity cells, so a work-group can hold the whole mesh
// of eight consecutive u_z values in LDS (8^3 cells: 18 KiB), sweep z, y and x
// on it in place, and touch memory once.  Such grids live in the caches, and
// three launches of the line walks are bound by their latency: rows of a few
// waves per SIMD, prologues and tails.  The pieces of a cell are 32 bytes, so
// the four work-groups of a 128-byte line are placed on one XCD, whose L2 then
// reads the line once.
//
// Drifts of a step, three launches -> this one (us): 8^3 cells of 8^3
// 17 -> 10, of 16^3 39 -> 19; 8 x 8 x 16 cells of 16^3 46 -> 35; 16 x 16 x 8
// cells of 16^3 64 -> 44.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.hpp"
#include "rows.hpp"
#include "sl_mpp5.hpp"

namespace vlasov {

namespace {

constexpr int W = 8;                      // u_z values per work-group
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct SmallMesh {
    DriftAxis ax[3];
    long Nu;
    int xcd;                              // tiles fill groups of 32: place lines on one XCD
};

// One periodic line of M cells in LDS (frame position 0 at x, `step` floats
// between cells) advanced by N + mu cells, in place.
template <int M>
__device__ __forceinline__ void drift_line(float* x, int step, const LineShift& sh)
{
    float v[M];
#pragma unroll
    for (int k = 0; k < M; ++k) v[k] = x[k * step];
    line_update_regs<M, true>(v, sh, [&](int j, float y) { x[((j + sh.N) & (M - 1)) * step] = y; });
}

__device__ __forceinline__ void drift_any(int M, float* x, int step, const LineShift& sh)
{
    if (M == 8) drift_line<8>(x, step, sh);
    else drift_line<16>(x, step, sh);
}

__global__ void __launch_bounds__(1024) k_drift_small(const float* __restrict__ fin,
                                                      float* __restrict__ fout, SmallMesh a)
{
    extern __shared__ __align__(16) float lds[];
    __shared__ LineShift tab[W + 2];      // of the W u_z values, of u_y and of u_x
    const int nx = a.ax[0].n, ny = a.ax[1].n, nz = a.ax[2].n;
    const int nuy = a.ax[1].nu, nuz = a.ax[2].nu;
    int tile = blockIdx.x;
    if (a.xcd) {
        const int s = tile >> 3;          // work-groups go to the eight XCDs in turn
        tile = 4 * ((s >> 2) * 8 + (tile & 7)) + (s & 3);
    }
    const long u0 = (long)tile * W;       // first velocity element
    const int row = nz * W + W;           // floats per (x, y) row in LDS: a pad of W keeps
                                          // the z-lines of a wave on different banks
    const int t = threadIdx.x, nt = blockDim.x;
    const int pieces = nx * ny * nz * (W / 4);

    {
        const double sz = cell_shift(a.ax[2], (int)(u0 % nuz) + t);
        const double sy = cell_shift(a.ax[1], (int)(u0 / nuz) % nuy);
        const double sx = cell_shift(a.ax[0], (int)(u0 / nuz / nuy));
        const LineShift sh = split_shift(t < W ? sz : (t == W ? sy : sx),
                                         t < W ? nz : (t == W ? ny : nx), true);
        if (t < W + 2) tab[t] = sh;
    }
    constexpr int U = 8;
    for (int i0 = t; i0 < pieces; i0 += U * nt) {
        floatx4 q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u * nt, pieces - 1);
            q[u] = *reinterpret_cast<const floatx4*>(fin + (long)(i >> 1) * a.Nu + u0 + 4 * (i & 1));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * nt;
            if (i < pieces) {
                const int c = i >> 1, r = c / nz;
                *reinterpret_cast<floatx4*>(lds + r * row + (c - r * nz) * W + 4 * (i & 1)) = q[u];
            }
        }
    }
    __syncthreads();
    const int w = t & (W - 1);
    {
        // z: lines (x, y), every lane its own shift
        const LineShift sh = tab[w];
        const int step = sh.neg ? -W : W, first = sh.neg ? (nz - 1) * W : 0;
        for (int l = t / W; l < nx * ny; l += nt / W) drift_any(nz, lds + l * row + first + w, step, sh);
    }
    __syncthreads();
    {
        const LineShift sh = uniform_shift(tab[W]);
        const int step = sh.neg ? -row : row, first = sh.neg ? (ny - 1) * row : 0;
        for (int l = t / W; l < nx * nz; l += nt / W) {
            const int ix = l / nz;
            drift_any(ny, lds + ix * ny * row + (l - ix * nz) * W + first + w, step, sh);
        }
    }
    __syncthreads();
    {
        const LineShift sh = uniform_shift(tab[W + 1]);
        const int S = ny * row;
        const int step = sh.neg ? -S : S, first = sh.neg ? (nx - 1) * S : 0;
        for (int l = t / W; l < ny * nz; l += nt / W) {
            const int iy = l / nz;
            drift_any(nx, lds + iy * row + (l - iy * nz) * W + first + w, step, sh);
        }
    }
    __syncthreads();
    for (int i = t; i < pieces; i += nt) {
        const int c = i >> 1, r = c / nz;
        *reinterpret_cast<floatx4*>(fout + (long)c * a.Nu + u0 + 4 * (i & 1)) =
            *reinterpret_cast<const floatx4*>(lds + r * row + (c - r * nz) * W + 4 * (i & 1));
    }
}

size_t small_lds(const DriftAxis (&ax)[3])
{
    return (size_t)ax[0].n * ax[1].n * (ax[2].n * W + W) * sizeof(float);
}

}  // namespace

// Meshes of which at least two work-groups share a CU (2048 cells, 72 KiB), and
// no more work-groups than are resident at once: 2^23 values.  Beyond that the
// phases of a work-group (load, three sweeps, store, a barrier between) leave
// the memory idle while the line walks stream: 8^3 cells of 32^3 88 us either
// way, 8 x 8 x 16 cells of 32^3 144 us by z and y, x against 222 here, 16^3
// cells of 8^3 (one work-group per CU) 32 against 36.
bool drift_small_supported(const DriftAxis (&ax)[3], long Nu, size_t lds_limit)
{
    for (int k = 0; k < 3; ++k)
        if (ax[k].n != 8 && ax[k].n != 16) return false;
    const long cells = (long)ax[0].n * ax[1].n * ax[2].n;
    if (cells > 2048 || Nu > (1L << 23) / cells || ax[2].nu % W != 0) return false;
    return small_lds(ax) + 2048 <= lds_limit;
}

hipError_t launch_drift_small(const float* fin, float* fout, const DriftAxis (&ax)[3], long Nu,
                              hipStream_t st)
{
    SmallMesh a;
    for (int k = 0; k < 3; ++k) a.ax[k] = ax[k];
    a.Nu = Nu;
    const long tiles = Nu / W;
    a.xcd = tiles % 32 == 0;
    const size_t lds = small_lds(ax);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_drift_small),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // a thread per line of the axis with the most lines, at most 1024
    const int cells = ax[0].n * ax[1].n * ax[2].n;
    int least = ax[0].n < ax[1].n ? ax[0].n : ax[1].n;
    if (ax[2].n < least) least = ax[2].n;
    const int lines = cells / least * W;
    hipLaunchKernelGGL(k_drift_small, dim3((unsigned)tiles), dim3((unsigned)(lines < 1024 ? lines : 1024)),
                       lds, st, fin, fout, a);
    return hipGetLastError();
}

}  // namespace vlasov
