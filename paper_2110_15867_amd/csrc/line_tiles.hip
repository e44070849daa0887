// z and y sweeps of lines whose integer shifts differ from lane to lane,
// through LDS tiles of whole lines.
//
// A z shift follows the contiguous u_z index (a y shift the u_y one, of which a
// wave holds several), so the lanes of a wave move in both directions and,
// beyond a Courant number of one, by different whole cells.  Walking straight
// from HBM (k_position) every lane then needs its own row addresses (64-bit
// arithmetic per row and lane, for the scales too) and a six-cell window with
// both stencils to pick from: 66 (FP32) to 90 (BF16) vector instructions per
// cell, which bound it.  Here a wave loads the tile of its 64
// lanes (M rows of 64 values, 16-byte accesses, each row and scale read once),
// and every lane walks its own line out of LDS in its own upwind frame: a row
// costs one LDS read and two integer instructions, whatever the shift, and the
// mirrored walk needs no stencil selects.  The results return to the tile and
// leave row by row, so an FP16/BF16 scale is a maximum over the row's few
// lanes of four values each.  A tile belongs to one wave: no barrier.
//
// Same operations per interface as the other walks: the bits of k_position's
// sweep.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "launch.hpp"
#include "rows.hpp"
#include "sl_mpp5.hpp"

namespace vlasov {

namespace {

// Per-lane constants of a line: the limiter acts on fh = f_j + r (fhat - f_j)
// with upper-limit factor ab on the stencil or its mirror image, and the flux
// is f lim, plus f_j on a comp line (flux_mag_mm's two forms, picked by
// select; a product with one and a sum with zero change no bit).
struct LaneLine {
    float v0, v1, v2, v3, mu, alpha, r, ab, f;
    bool comp;
};

__device__ __forceinline__ LaneLine lane_line(const LineShift& sh)
{
    LaneLine l;
    l.v0 = sh.v0; l.v1 = sh.v1; l.v2 = sh.v2; l.v3 = sh.v3;
    l.mu = sh.mu;
    l.alpha = sh.alpha;
    l.comp = sh.comp;
    l.r = sh.comp ? -sh.q : 1.0f;
    l.ab = sh.comp ? sh.alpha_c : sh.alpha;
    l.f = sh.comp ? -sh.muc : sh.mu;
    return l;
}

__device__ __forceinline__ float flux_lane(const Stencil& s, const LaneLine& l, float Mm, float Mp)
{
    float y = l.v0 * s.dm2;                            // fhat - f_j
    y = fmaf(l.v1, s.dm1, y);
    y = fmaf(l.v2, s.d0, y);
    y = fmaf(l.v3, s.dp1, y);
    const float m = med3(s.d0, l.alpha * s.dm1, 0.0f); // f_MP - f_j
    float pre = l.mu * (s.c + y);
    if (__builtin_expect(med3(y, 0.0f, m) != y, 0)) {
        Stencil t = s;
        t.d = l.comp ? s.b : s.d;
        t.d0 = l.comp ? -s.dm1 : s.d0;
        t.dm1 = l.comp ? -s.d0 : s.dm1;
        const float lim = mp_bounded_m(fmaf(l.r, y, s.c), t, l.ab, l.comp ? Mp : Mm,
                                       l.comp ? Mm : Mp);
        pre = fmaf(l.f, lim, l.comp ? s.c : 0.0f);
    }
    return med3(pre, 0.0f, s.c);
}

template <int P, int M, int NUZ>
__global__ void __launch_bounds__(256) k_line_tiles(const typename Codec<P>::T* __restrict__ fin,
                                                 const float* __restrict__ sin,
                                                 typename Codec<P>::T* __restrict__ fout,
                                                 float* __restrict__ sout, PosArgs a)
{
    using T = typename Codec<P>::T;
    constexpr unsigned ROW = 64 * sizeof(float);          // bytes of a tile row
    constexpr unsigned TILE = M * ROW;                    // a power of two
    constexpr int G = NUZ / 4;                            // lanes per uz-line in row order
    __shared__ __align__(16) float lds[4 * M * 64];
    const long wave = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const long wpr = a.I / 64;                            // waves per row
    if (wave >= a.O * wpr) return;                        // whole waves; no barrier follows
    const int lane = threadIdx.x & 63;
    char* tile = reinterpret_cast<char*>(lds) + (threadIdx.x >> 6) * TILE;
    const long o = wave / wpr;
    const long k0 = (wave - o * wpr) * 64;
    const long e0 = uniform_long(o * (long)M * a.I + k0);             // row 0, lane 0
    const long s0 = uniform_long(o * (long)M * (a.I / NUZ) + k0 / NUZ);

    // row order: lane (rr, c) holds values 4 c .. 4 c + 3 of row 4 g + rr
    const int rr = lane >> 4, c = lane & 15;
    const long sI = a.I / NUZ;
    const long eoff = rr * a.I + 4 * c, soff = rr * sI + c / G;
    {
        Pack<T, 4> q[M / 4];
        float sc[M / 4];
#pragma unroll
        for (int g = 0; g < M / 4; ++g) {
            q[g] = *reinterpret_cast<const Pack<T, 4>*>(fin + e0 + 4 * g * a.I + eoff);
            sc[g] = Codec<P>::scaled ? sin[s0 + 4 * g * sI + soff] : 1.0f;
        }
#pragma unroll
        for (int g = 0; g < M / 4; ++g) {
            float4 v;
            v.x = decode<P>(q[g].v[0], sc[g]);
            v.y = decode<P>(q[g].v[1], sc[g]);
            v.z = decode<P>(q[g].v[2], sc[g]);
            v.w = decode<P>(q[g].v[3], sc[g]);
            *reinterpret_cast<float4*>(tile + (4 * g + rr) * ROW + 16 * c) = v;
        }
    }
    // z: the shift follows the u_z index (k0 is a multiple of 64); y: the uz-line's u_y
    const int j = a.pst == 1 ? lane % NUZ
                             : (int)(((unsigned)(k0 / NUZ % a.nshift) + lane / NUZ) % (unsigned)a.nshift);
    const LineShift sh = split_shift(a.shift[j], M, true);
    const LaneLine l = lane_line(sh);
    wave_fence();

    // the lane's rows in its own frame, wrapped within the tile's power of two
    const unsigned col = 4u * lane;
    const int step = sh.neg ? -(int)ROW : (int)ROW;
    const unsigned first = sh.neg ? (M - 1) * ROW : 0;               // frame row 0
    unsigned at = (first + (unsigned)((-sh.N - 3) * step)) & (TILE - 1);
    auto next = [&]() {
        const float x = *reinterpret_cast<const float*>(tile + (at | col));
        at = (at + (unsigned)step) & (TILE - 1);
        return x;
    };
    float y[M];
    {
        float xm2 = next(), xm1 = next(), x0 = next(), xp1 = next(), xp2 = next();
        const float head[5] = {xm2, xm1, x0, xp1, xp2};
        float dm2 = xm1 - xm2, dm1 = x0 - xm1, d0 = xp1 - x0, dp1 = xp2 - xp1;
        float cj = dp1 - d0, kj = curv_minmod(d0 - dm1, cj);
        float phi_old = flux_lane(Stencil{xm2, xm1, x0, xp1, xp2, dm2, dm1, d0, dp1}, l,
                                  curv_minmod(dm1 - dm2, d0 - dm1), kj);
#pragma unroll
        for (int i = 0; i < M; ++i) {
            xm2 = xm1; xm1 = x0; x0 = xp1; xp1 = xp2;
            dm2 = dm1; dm1 = d0; d0 = dp1;
            xp2 = i < M - 5 ? next() : head[i - (M - 5)];
            dp1 = xp2 - xp1;
            const float cp = dp1 - d0;
            const float Mp = curv_minmod(cj, cp);
            const float phi =
                flux_lane(Stencil{xm2, xm1, x0, xp1, xp2, dm2, dm1, d0, dp1}, l, kj, Mp);
            cj = cp;
            kj = Mp;
            y[i] = x0 - (phi - phi_old);
            phi_old = phi;
        }
    }
    wave_fence();
    {
        unsigned w = first | col;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            *reinterpret_cast<float*>(tile + w) = y[i];
            w += (unsigned)step;
        }
    }
    wave_fence();
#pragma unroll
    for (int g = 0; g < M / 4; ++g) {
        const float4 v = *reinterpret_cast<const float4*>(tile + (4 * g + rr) * ROW + 16 * c);
        const float x[4] = {v.x, v.y, v.z, v.w};
        float inv = 1.0f;
        if (Codec<P>::scaled) {
            // from 0, as the other writers: a NaN never becomes the scale of its line
            float m = 0.0f;
#pragma unroll
            for (int u = 0; u < 4; ++u) m = fmaxf(m, fabsf(x[u]));
            m = group_max_nonneg<G>(m);
            inv = inv_scale(m);
            if (c % G == 0) sout[s0 + 4 * g * sI + soff] = m;
        }
        Pack<T, 4> q;
#pragma unroll
        for (int u = 0; u < 4; ++u) q.v[u] = quantize<P>(x[u], inv);
        *reinterpret_cast<Pack<T, 4>*>(fout + e0 + 4 * g * a.I + eoff) = q;
    }
}

template <int P, int M>
hipError_t launch_m(const void* fin, const float* sin, void* fout, float* sout, const PosArgs& a,
                    hipStream_t st)
{
    using T = typename Codec<P>::T;
    const unsigned blocks = (unsigned)((a.O * (a.I / 64) + 3) / 4);
    auto kern = a.nuz == 16 ? k_line_tiles<P, M, 16>
                            : (a.nuz == 32 ? k_line_tiles<P, M, 32> : k_line_tiles<P, M, 64>);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, st, (const T*)fin, sin, (T*)fout, sout, a);
    return hipGetLastError();
}

template <int P>
hipError_t launch_p(const void* fin, const float* sin, void* fout, float* sout, const PosArgs& a,
                    hipStream_t st)
{
    switch (a.M) {
        case 16: return launch_m<P, 16>(fin, sin, fout, sout, a, st);
        case 32: return launch_m<P, 32>(fin, sin, fout, sout, a, st);
        default: return launch_m<P, 64>(fin, sin, fout, sout, a, st);
    }
}

}  // namespace

// z sweeps (the shift follows u_z) and y sweeps (u_y) of compiled line lengths
// whose rows hold whole waves of whole uz-lines.  z, lines of 16 and 32 cells:
// always (32^3 cells of 32^3 with shifts up to 2.5 cells: FP32 1.89 -> 1.43 ms,
// BF16 2.58 -> 1.36; 64 x 64 x 32 cells with shifts below one: FP32 6.04 ->
// 5.89 ms, FP16, the paired walk, 6.58 -> 5.16).  Lines of 64 cells, whose
// tiles leave two waves per SIMD: where some line moves by a cell or more
// (16 x 16 x 64 cells of 32^3 with 2.5: FP32 1.07 -> 0.89 ms, FP16 1.13 -> 0.88;
// with 0.3: FP32 0.77 from HBM, 0.90 from tiles, FP16 0.79 and 0.85).
//
// y, uz-lines of 16 values: always.  A wave of k_position that shares one u_y
// reads pieces of 64 bytes or less, and one of consecutive elements holds 16
// values of u_y (32^3 cells of 16^3: FP32 333 -> 223 us, FP16 with shifts up to
// 2.5 cells 630 -> 176, 0.3 271 -> 161; 64^3 cells FP32 2.84 -> 1.83 ms).
// uz-lines of 32 values: FP16/BF16 lines of 16 and 32 cells where some line
// moves by a cell or more, so that the lanes of a wave read different rows
// (32^3 cells of 32^3, FP16: 2.5 cells 1.80 -> 1.36 ms, 0.3 cells 1.27 from HBM
// and 1.36 from tiles; lines of 64 cells 4.9 and 6.3 ms; FP32 1.68 and 1.91).
bool line_tiles_supported(int prec, const PosArgs& a)
{
    const bool z = a.pst == 1 && a.nshift == a.nuz && a.V == 1;
    if (!z && a.pst != a.nuz) return false;
    if (a.nuz != 16 && a.nuz != 32 && a.nuz != 64) return false;
    if (a.M != 16 && a.M != 32 && a.M != 64) return false;
    if (a.I % 64 != 0 || a.O * (a.I / 64) > 4 * 0x7fffffffL) return false;
    if (z ? a.M != 64 : a.nuz == 16) return true;
    if (!z && (a.nuz != 32 || a.M == 64 || prec == PREC_F32)) return false;
    for (int j = 0; j < a.nshift; ++j)
        if (fabs(a.shift[j]) >= 1.0) return true;
    return false;
}

hipError_t launch_line_tiles(int prec, const void* fin, const float* sin, void* fout, float* sout,
                          const PosArgs& a, hipStream_t st)
{
    if (a.O * a.I == 0) return hipSuccess;
    switch (prec) {
        case PREC_F16: return launch_p<PREC_F16>(fin, sin, fout, sout, a, st);
        case PREC_BF16: return launch_p<PREC_BF16>(fin, sin, fout, sout, a, st);
        default: return launch_p<PREC_F32>(fin, sin, fout, sout, a, st);
    }
}

}  // namespace vlasov
