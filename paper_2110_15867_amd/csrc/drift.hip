// The y and x drifts of one step (Eq. 3) in one pass over f (FP32 storage):
// D_x D_y of Eq. (5), the bits of vlasov_advect_y followed by
// vlasov_advect_x.
//
// Each drift alone is bound by HBM (one read and one write of f, about 31
// vector instructions per cell, half of the vector issue rate), so the pair
// gains from touching f once.  A wave owns one u_x, u_y, a segment of S
// cells along y, and 64 lanes of (z, u_z): both shifts are then the same in
// all its lanes.  It streams along x: for each plane a thread loads the S + 5
// rows its segment's y-sweep reads (the five shared ones come from the
// caches: the segments of a line are the waves of one work-group), advances
// the S cells along y in registers, and feeds them to S x-walks whose
// five-plane windows live in registers.  No LDS exchange and no barrier; LDS
// holds the first five y-swept planes of each thread, which close the
// periodic x-lines at the end.
//
// S = 8 where it divides well: the extra interface and rows of a segment cost
// (S + 1) / S, and the x-windows take 6 S registers of the 128 that four waves
// per SIMD leave (carrying the planes' differences too would save three
// instructions per cell but spills at S = 8: twice the time).
// Measured on 64 x 64 x 32 cells of 32^3: 8.8 ms against 13.8 for the two
// drifts, 3.9 TB/s and 0.85 of the vector issue rate; 32^3 of 32^3 with shifts
// of 2.5 cells 2.19 ms against 3.28.  (The curvature minmods evaluated only
// where a wave fails the Suresh-Huynh test: 8.9 and 2.27 ms.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.hpp"
#include "rows.hpp"
#include "sl_mpp5.hpp"

namespace vlasov {

namespace {

template <int S>
__global__ void __launch_bounds__(1024) k_drift_yx(const float* __restrict__ fin,
                                                   float* __restrict__ fout, DriftArgs a)
{
    extern __shared__ float heads[];
    const int lane = threadIdx.x & 63;
    const int seg = uniform_sgpr((int)(threadIdx.x >> 6));
    // work-group -> (z group, u_z chunk, u_x, u_y), u_y fastest
    int b = blockIdx.x;
    if (a.pair) {
        // work-groups go to the eight XCDs in turn: b and b + 8 take the pair
        const int s = b >> 3;
        b = 2 * ((s >> 1) * 8 + (b & 7)) + (s & 1);
    }
    const int jy = b % a.y.nu;
    b /= a.y.nu;
    const int jx = b % a.x.nu;
    b /= a.x.nu;
    const int chunk = b % a.jchunks;
    const int iz0 = (b / a.jchunks) * a.zi;
    const int zl = lane / a.W, jz = chunk * 64 + lane % a.W;
    if (zl >= a.zi || iz0 + zl >= a.nz || jz >= a.nuz) return;    // (no barrier follows)

    const LineShift sx = uniform_shift(split_shift(cell_shift(a.x, jx), a.x.n, true));
    const LineShift sy = uniform_shift(split_shift(cell_shift(a.y, jy), a.y.n, true));
    const int nx = a.x.n, ny = a.y.n;

    // byte offsets: of this lane inside a row, and of the rows inside a plane
    const unsigned voff = (unsigned)(((long)(iz0 + zl) * a.Nu + ((long)jx * a.y.nu + jy) * a.nuz + jz) * 4);
    const unsigned row_bytes = (unsigned)((long)a.nz * a.Nu * 4);
    const long plane = (long)ny * a.nz * a.Nu;
    const unsigned plane_bytes = (unsigned)(plane * 4);
    int i0 = seg * S;
    if (i0 > ny - S) i0 = ny - S;             // the last segment overlaps (same values)
    unsigned rin[S + 5], rout[S];
#pragma unroll
    for (int k = 0; k < S + 5; ++k) {
        const int r = i0 - sy.N - 3 + k;
        int p = (sy.neg ? ny - 1 - r : r) % ny;
        if (p < 0) p += ny;
        rin[k] = (unsigned)p * row_bytes;
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
        rout[s] = (unsigned)(sy.neg ? ny - 1 - (i0 + s) : i0 + s) * row_bytes;

    // planes in the x frame of the walk: rows -N-3, -N-2, ...
    int px = (sx.neg ? nx - 1 + sx.N + 3 : -sx.N - 3) % nx;
    if (px < 0) px += nx;
    const int dx = sx.neg ? -1 : 1;
    auto load_plane = [&](float (&v)[S + 5]) {
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(fin + px * plane, plane_bytes);
#pragma unroll
        for (int k = 0; k < S + 5; ++k)
            v[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff, (int)rin[k], 0));
        px += dx;
        px = px == nx ? 0 : (px < 0 ? nx - 1 : px);
    };

    float* head = heads + threadIdx.x;        // [5][S] values, blockDim.x apart
    float nxt[S + 5];
    load_plane(nxt);
    float w[5][S], phi_old[S];
    float kx[S];              // curvature minmod below the next interface
#pragma unroll
    for (int s = 0; s < S; ++s) {
        phi_old[s] = 0.0f;
        kx[s] = 0.0f;
#pragma unroll
        for (int q = 0; q < 5; ++q) w[q][s] = 0.0f;
    }
    const int T = nx + 5;                     // planes the x-walks read
#pragma unroll 1
    for (int t0 = 0; t0 < T; t0 += 5) {
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const int t = t0 + q;
            if (t >= T) break;
            if (t < nx) {
                // y-sweep of the segment in this plane
                float v[S + 5];
#pragma unroll
                for (int k = 0; k < S + 5; ++k) v[k] = nxt[k];
                if (t + 1 < nx) load_plane(nxt);
                float dm2 = v[1] - v[0], dm1 = v[2] - v[1], d0 = v[3] - v[2], dp1 = v[4] - v[3];
                float cy = dp1 - d0, ky = curv_minmod(d0 - dm1, cy);
                float phi = flux_mag_mm(Stencil{v[0], v[1], v[2], v[3], v[4], dm2, dm1, d0, dp1}, sy,
                                        curv_minmod(dm1 - dm2, d0 - dm1), ky);
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    dm2 = dm1; dm1 = d0; d0 = dp1;
                    dp1 = v[s + 5] - v[s + 4];
                    const float cn = dp1 - d0, kn = curv_minmod(cy, cn);
                    const float ph = flux_mag_mm(
                        Stencil{v[s + 1], v[s + 2], v[s + 3], v[s + 4], v[s + 5], dm2, dm1, d0, dp1},
                        sy, ky, kn);
                    cy = cn;
                    ky = kn;
                    w[q][s] = v[s + 3] - (ph - phi);
                    phi = ph;
                }
                if (t0 == 0) {
#pragma unroll
                    for (int s = 0; s < S; ++s) head[(q * S + s) * blockDim.x] = w[q][s];
                }
            } else {
#pragma unroll
                for (int s = 0; s < S; ++s) w[q][s] = head[((t - nx) * S + s) * blockDim.x];
            }
            if (t < 4) continue;
            // x interfaces: the window t-4 .. t, centre t-2
            int po = t - 5;
            po = sx.neg ? nx - 1 - po : po;
            const __amdgpu_buffer_rsrc_t ro = row_rsrc(fout + (t >= 5 ? po : 0) * plane, plane_bytes);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const float xa = w[(q + 1) % 5][s], xb = w[(q + 2) % 5][s], xc = w[(q + 3) % 5][s];
                const float xd = w[(q + 4) % 5][s], xe = w[q][s];
                const float e0 = xb - xa, e1 = xc - xb, e2 = xd - xc, e3 = xe - xd;
                const float c0 = e2 - e1, kn = curv_minmod(c0, e3 - e2);
                const float kb = t == 4 ? curv_minmod(e1 - e0, c0) : kx[s];
                const float ph = flux_mag_mm(Stencil{xa, xb, xc, xd, xe, e0, e1, e2, e3}, sx, kb, kn);
                kx[s] = kn;
                if (t >= 5)
                    __builtin_amdgcn_raw_buffer_store_b32(
                        __builtin_bit_cast(unsigned, xc - (ph - phi_old[s])), ro, (int)voff, (int)rout[s], 0);
                phi_old[s] = ph;
            }
        }
    }
}

// Cells along y per segment: the fewest interfaces, (S + 1) per segment.
int segment_cells(int ny)
{
    int best = 8, cost = 1 << 30;
    for (int S = 8; S >= 5; --S) {
        const int c = ((ny + S - 1) / S) * (S + 1);
        if (c < cost) {
            cost = c;
            best = S;
        }
    }
    return best;
}

}  // namespace

// Work-groups, cells per segment and threads of the fused pass.
struct DriftShape {
    double groups;
    int S, threads;
    size_t lds() const { return (size_t)5 * S * threads * sizeof(float); }
};

static DriftShape drift_shape(const DriftArgs& a)
{
    DriftShape r;
    const int zi = a.nuz < 64 ? 64 / a.nuz : 1;
    r.groups = (double)((a.nz + zi - 1) / zi) * ((a.nuz + 63) / 64) * a.x.nu * a.y.nu;
    r.S = segment_cells(a.y.n);
    // below four waves per SIMD the walk waits on its loads: more, shorter
    // segments are worth their interfaces (16^3 cells of 16^3, 2048 waves at
    // S = 8, 4096 at 5: 63 -> 54 us)
    if (r.groups * ((a.y.n + r.S - 1) / r.S) < 4096.0 && a.y.n <= 80) r.S = 5;
    r.threads = 64 * ((a.y.n + r.S - 1) / r.S);
    return r;
}

// Where the fused pass is taken, besides what its indexing needs (one
// work-group of at most sixteen segments per y-line, 32-bit offsets inside a
// plane, lines of at least a segment and its wrap, LDS for the closing planes
// of its threads: 160 KiB for 16 segments of 8):
//  * u_z lines that fill waves and cache lines (16, 32 or a multiple of 64
//    values): with 8 the pieces of a row are 32 bytes (48^3 cells of 8^3: step
//    895 us fused, 801 apart), with 20 four lanes idle and lines straddle
//    (48^3 of 10 x 12 x 20: 3.67 ms, 3.25 apart);
//  * two waves for each of the chip's 1024 SIMDs: a wave streams a whole
//    x-line, so fewer leave it waiting on its own loads (8^3 of 16^3, 512
//    waves: 77 us, 72 apart; 16^3 of 16^3, 2048 waves: equal; 20^3 of 16^3:
//    359 us, 392 apart).
bool drift_yx_supported(const DriftArgs& a, size_t lds_limit)
{
    if (a.x.n < 8 || a.y.n < 8) return false;
    if (a.nuz != 16 && a.nuz != 32 && a.nuz % 64 != 0) return false;
    const int S = segment_cells(a.y.n), segs = (a.y.n + S - 1) / S;
    if (segs > 16) return false;
    if ((double)a.y.n * a.nz * a.Nu * 4.0 >= 4294967296.0) return false;
    const DriftShape r = drift_shape(a);
    return r.groups * segs >= 2048.0 && r.groups < 2147483647.0 && r.lds() <= lds_limit;
}

hipError_t launch_drift_yx(const float* fin, float* fout, DriftArgs a, hipStream_t st)
{
    a.W = a.nuz < 64 ? a.nuz : 64;
    a.zi = a.W < 64 ? 64 / a.W : 1;
    a.jchunks = (a.nuz + 63) / 64;
    const DriftShape r = drift_shape(a);
    const unsigned grid = (unsigned)r.groups, nt = (unsigned)r.threads;
    // uz-lines of 16 values are half a cache line; its other half is the next
    // u_y's, fetched again if that runs under another L2
    a.pair = a.nuz == 16 && a.y.nu % 2 == 0 && grid % 16 == 0;
    const size_t lds = r.lds();
#define VL_DRIFT(SV)                                                                            \
    {                                                                                           \
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_drift_yx<SV>),  \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,     \
                                                 (int)lds);                                      \
        if (e != hipSuccess) return e;                                                          \
        hipLaunchKernelGGL(k_drift_yx<SV>, dim3(grid), dim3(nt), lds, st, fin, fout, a);         \
    }
    switch (r.S) {
        case 5: VL_DRIFT(5) break;
        case 6: VL_DRIFT(6) break;
        case 7: VL_DRIFT(7) break;
        default: VL_DRIFT(8) break;
    }
#undef VL_DRIFT
    return hipGetLastError();
}

}  // namespace vlasov
