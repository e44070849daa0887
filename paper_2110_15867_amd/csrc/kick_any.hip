// Fused velocity kick for velocity blocks of any shape that fits LDS and has
// no kernel of its own (the cubic 16^3 and 32^3 blocks): ux, uy and uz of one
// half step (Eq. 5) on one cell's block per work-group, one HBM read and one
// write of f instead of three.
//
// The three single sweeps of such shapes are bound by latency and access:
// runtime line lengths, so rows requested one at a time, and u_z lines walked
// by one thread each straight from HBM (uncoalesced).  Here the block is
// loaded and stored with consecutive threads on consecutive values, and a
// thread walks one line at a time out of LDS, in place, in groups of four
// cells (four LDS reads in flight, window slots renamed instead of moved).
// Several work-groups share a CU, so one's loads and stores overlap another's
// arithmetic without a prefetch of its own.
// Measured on 20 x 18 x 15 cells of 24 x 20 x 18 (FP32): 0.19 ms per kick, 2.0
// TB/s and about 0.6 of the vector issue rate, against 0.94 ms for the three
// sweeps (0.71 of it in u_z).
//
// Results are the bits of the three single sweeps in every storage form: the
// walk performs walk_uniform's operations, and with FP16/BF16 storage the
// values between the sweeps are rounded to codes in LDS as the sweeps store
// them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.hpp"
#include "rows.hpp"
#include "sl_mpp5.hpp"

namespace vlasov {

namespace {

// One line of M cells in LDS advanced in place by its fractional shift: frame
// position p at x[p * step] (step negative for a mirrored walk).  Ghosts are
// zero or wrap (PER).  Same operations as line_update_regs.  Returns the flux
// through the upper face of the last cell.
template <bool PER>
__device__ __forceinline__ float sweep_line(float* x, int step, int M, const LineShift& sh)
{
    auto at = [&](int p) -> float& { return x[p * step]; };
    // X(k) before anything is written
    auto early = [&](int k) -> float {
        if (PER) {
            k %= M;
            if (k < 0) k += M;
            return at(k);
        }
        return k >= 0 && k < M ? at(k) : 0.0f;
    };
    const float xm3 = early(-3);
    float xm2 = early(-2), xm1 = early(-1), x0 = early(0), xp1 = early(1);
    const float wrap0 = PER ? early(M) : 0.0f, wrap1 = PER ? early(M + 1) : 0.0f;
    const float e0 = xm2 - xm3;
    float dm2 = xm1 - xm2, dm1 = x0 - xm1, d0 = xp1 - x0;
    // curvature minmods carried from interface to interface (flux_mag_mm)
    const float Dm1 = dm1 - dm2;
    float D0 = d0 - dm1;
    float Mm = curv_minmod(dm2 - e0, Dm1);
    float phi_prev;
    {
        const float Mp = curv_minmod(Dm1, D0);
        phi_prev = flux_mag_mm(Stencil{xm3, xm2, xm1, x0, xp1, e0, dm2, dm1, d0}, sh, Mm, Mp);
        Mm = Mp;
    }
    auto cell = [&](int j, float xp2) {
        const float dp1 = xp2 - xp1;
        const float Dp = dp1 - d0;
        const float Mp = curv_minmod(D0, Dp);
        const float phi =
            flux_mag_mm(Stencil{xm2, xm1, x0, xp1, xp2, dm2, dm1, d0, dp1}, sh, Mm, Mp);
        at(j) = x0 - (phi - phi_prev);
        phi_prev = phi;
        xm2 = xm1; xm1 = x0; x0 = xp1; xp1 = xp2;
        dm2 = dm1; dm1 = d0; d0 = dp1;
        D0 = Dp; Mm = Mp;
    };
#pragma unroll 1
    for (int j0 = 0; j0 < M; j0 += 4) {
        float n[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = j0 + 2 + q;                 // (uniform)
            n[q] = k < M ? at(k) : (k == M ? wrap0 : wrap1);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (j0 + q < M) cell(j0 + q, n[q]);
    }
    return phi_prev;
}

// The integer part N > 0 of the shift, out_{j+N} = y_j (translate_line with a
// runtime length): periodic lines rotate in place by three reversals.
template <bool PER>
__device__ __forceinline__ void shift_line(float* x, int step, int M, int N)
{
    auto at = [&](int p) -> float& { return x[p * step]; };
    if (PER) {
        auto rev = [&](int lo, int hi) {
            for (int i = lo, k = hi - 1; i < k; ++i, --k) {
                const float u = at(i);
                at(i) = at(k);
                at(k) = u;
            }
        };
        rev(0, M);
        rev(0, N);
        rev(N, M);
        return;
    }
    for (int p = M - 1; p >= N; --p) at(p) = at(p - N);
    const int nz = N < M ? N : M;
    for (int p = 0; p < nz; ++p) at(p) = 0.0f;
}

// acc + a of lane 0, 1, .. G-1 of each aligned group of G lanes, in that order.
template <int G>
__device__ __forceinline__ float add_group(float acc, float a)
{
    if constexpr (G == 1) {
        return acc + a;
    } else if constexpr (G == 2) {
        acc += dpp_mov<0xA0>(a);                       // quad_perm [0,0,2,2]
        return acc + dpp_mov<0xF5>(a);                 // quad_perm [1,1,3,3]
    } else {
        acc += dpp_mov<0x00>(a);                       // quad_perm [0,0,0,0], ...
        acc += dpp_mov<0x55>(a);
        acc += dpp_mov<0xAA>(a);
        return acc + dpp_mov<0xFF>(a);
    }
}

// The flux through the upper face of cell j (-9 <= j < M) of a vacuum line
// before it is swept: sweep_line's operations on that interface.
__device__ __forceinline__ float face_flux(const float* x, int step, int M, const LineShift& sh, int j)
{
    auto at = [&](int k) { return k >= 0 && k < M ? x[k * step] : 0.0f; };
    const float a = at(j - 2), b = at(j - 1), c = at(j), d = at(j + 1), e = at(j + 2);
    const float dm2 = b - a, dm1 = c - b, d0 = d - c, dp1 = e - d;
    const float D0 = d0 - dm1;
    return flux_mag_mm(Stencil{a, b, c, d, e, dm2, dm1, d0, dp1}, sh, curv_minmod(dm1 - dm2, D0),
                       curv_minmod(D0, dp1 - d0));
}

// What a group of G lines (consecutive lanes; with `one`, its own) lets out
// when whole rows leave (N > 0), before the sweep in place overwrites them: a
// single sweep of ux or uy walks G lines per thread with one FP32 sum over
// them, row by row -- the first two rows past the upper face, the flux through
// it, then the rows further out -- and this adds the same values in the same
// order.  Rare (a kick moves less than a cell unless the field is strong), and a
// call: inlined, a kick of 8^3 cells of 8^3 took 9.7 us instead of 9.4 for
// the code it fetches.
template <int G>
__device__ __attribute__((noinline)) float rows_out(const float* x, int step, int M, LineShift sh, bool one)
{
    auto add = [&](float s, float v) { return one ? s + v : add_group<G>(s, v); };
    float acc = 0.0f;
    const int first = M - sh.N, near = first + 2 < M ? first + 2 : M;
    for (int p = max(first, 0); p < near; ++p) acc = add(acc, x[p * step]);
    acc = add(acc, face_flux(x, step, M, sh, first - 1));
    for (int p = max(near, 0); p < M; ++p) acc = add(acc, x[p * step]);
    return acc;
}

// One vacuum line swept and translated; returns the content its group of G
// lines lets out (rows_out's sum; for N = 0 the flux through the upper face),
// in every lane.
template <int G>
__device__ __forceinline__ float vacuum_line(float* x, int step, int M, const LineShift& sh, bool one)
{
    auto add = [&](float s, float v) { return one ? s + v : add_group<G>(s, v); };
    const int N = sh.N;
    float acc = 0.0f;
    if (__builtin_expect(N > 0, 0)) acc = rows_out<G>(x, step, M, sh, one);
    const float phi = sweep_line<false>(x, step, M, sh);
    if (__builtin_expect(N == 0, 1)) return add(acc, phi);
    shift_line<false>(x, step, M, N);
    return acc;
}

// e / d for e, d below 2^16: the product with ceil(2^32 / d) (exact while
// e * d < 2^32)
struct SmallDiv {
    unsigned d, m;
    __host__ __device__ explicit SmallDiv(int dd)
        : d((unsigned)dd), m(dd == 1 ? 0u : (unsigned)((0x100000000ull + (unsigned)dd - 1) / (unsigned)dd))
    {
    }
    __device__ int div(int e) const { return m == 0u ? e : (int)__umulhi((unsigned)e, m); }
};

struct AnyArgs {
    int nu[3];
    int lz;              // padded uz-line in LDS, odd
    SmallDiv dz;
    AnyArgs(const int n[3]) : nu{n[0], n[1], n[2]}, lz(n[2] | 1), dz(n[2]) {}
};

template <int P, int V, bool PER>
__global__ void __launch_bounds__(1024) k_kick_any(const typename Codec<P>::T* __restrict__ fin,
                                                   const float* __restrict__ sin,
                                                   typename Codec<P>::T* __restrict__ fout,
                                                   float* __restrict__ sout, KickArgs a, AnyArgs b)
{
    using T = typename Codec<P>::T;
    extern __shared__ float lds[];
    __shared__ LineShift shifts[3];
    __shared__ double red[3][16];
    const long cell = blockIdx.x;
    const int nz = b.nu[2], lz = b.lz;
    const int nlz = b.nu[0] * b.nu[1];              // uz-lines
    const int nv = nlz * nz;
    float* lmax = lds + nlz * lz;                   // scale per uz-line (scaled storage)
    const T* src = fin + cell * nv;
    const float* ssrc = sin + cell * nlz;
    // the cell's outflow total so far, needed only at the end
    double prev = 0.0;
    if (a.outflow != nullptr && !PER && threadIdx.x == 0) prev = a.outflow[cell];

    // the block into LDS; the three shift splits are made by one lane each
    // while the loads are in flight
    constexpr int U = 4;
    for (int e0 = threadIdx.x * V; e0 < nv; e0 += U * blockDim.x * V) {
        Pack<T, V> q[U];
        float sc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * blockDim.x * V;
            if (e < nv) {
                q[u] = *reinterpret_cast<const Pack<T, V>*>(src + e);
                sc[u] = Codec<P>::scaled ? ssrc[b.dz.div(e)] : 1.0f;
            }
        }
        if (e0 < 3 * V && e0 / V < 3) {
            const int k = e0 / V;
            shifts[k] = split_shift((double)a.g[(long)k * a.cells + cell] * a.factor[k], b.nu[k], PER);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * blockDim.x * V;
            if (e < nv) {
                const int l = b.dz.div(e);
                float* dst = lds + l * lz + (e - l * nz);
#pragma unroll
                for (int v = 0; v < V; ++v) dst[v] = decode<P>(q[u].v[v], sc[u]);
            }
        }
    }
    // (blocks of fewer than three vectors)
    if ((int)threadIdx.x < 3 && (int)threadIdx.x * V >= nv)
        shifts[threadIdx.x] = split_shift((double)a.g[(long)threadIdx.x * a.cells + cell] *
                                              a.factor[threadIdx.x], b.nu[threadIdx.x], PER);
    __syncthreads();

    double out[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int ax = 0; ax < 3; ++ax) {
        const LineShift sh = uniform_shift(shifts[ax]);
        const int M = uniform_sgpr(b.nu[ax]);
        // lines (o, k): k over jz (ux: also jy, as o) at stride S
        const int S = ax == 0 ? b.nu[1] * lz : (ax == 1 ? lz : 1);
        const int os = ax == 0 ? lz : (ax == 1 ? b.nu[1] * lz : lz);
        const int nl = ax == 0 ? b.nu[1] * nz : (ax == 1 ? b.nu[0] * nz : nlz);
        const int step = sh.neg ? -S : S;
        double mine = 0.0;
        for (int l = threadIdx.x; l < nl; l += blockDim.x) {
            const int o = ax == 2 ? l : b.dz.div(l);
            const int base = o * os + (ax == 2 ? 0 : l - o * nz);
            float* x = lds + base + (sh.neg ? (M - 1) * S : 0);
            if (PER) {
                sweep_line<true>(x, step, M, sh);
                if (sh.N > 0) shift_line<true>(x, step, M, sh.N);
            } else {
                const float ofl = vacuum_line<V>(x, step, M, sh, ax == 2);
                if (ax == 2 || threadIdx.x % V == 0) mine += (double)ofl;
            }
            if (Codec<P>::scaled && ax == 2) {
                float* z = lds + l * lz;
                float m = 0.0f;
                for (int i = 0; i < nz; ++i) m = fmaxf(m, fabsf(z[i]));
                lmax[l] = m;
                sout[cell * nlz + l] = m;
            }
        }
        out[0] = ax == 0 ? mine : out[0];
        out[1] = ax == 1 ? mine : out[1];
        out[2] = ax == 2 ? mine : out[2];
        __syncthreads();
        if (Codec<P>::scaled && ax < 2) {
            // what a sweep stores and the next one loads: codes and back
            for (int l = threadIdx.x; l < nlz; l += blockDim.x) {
                float* z = lds + l * lz;
                float m = 0.0f;
                for (int i = 0; i < nz; ++i) m = fmaxf(m, fabsf(z[i]));
                const float inv = inv_scale(m);
                for (int i = 0; i < nz; ++i) z[i] = decode<P>(quantize<P>(z[i], inv), m);
            }
            __syncthreads();
        }
    }

    T* dst = fout + cell * nv;
    for (int e = threadIdx.x * V; e < nv; e += blockDim.x * V) {
        const int l = b.dz.div(e);
        const float* z = lds + l * lz + (e - l * nz);
        const float inv = Codec<P>::scaled ? inv_scale(lmax[l]) : 1.0f;
        Pack<T, V> q;
#pragma unroll
        for (int v = 0; v < V; ++v) q.v[v] = quantize<P>(z[v], inv);
        *reinterpret_cast<Pack<T, V>*>(dst + e) = q;
    }
    if (a.outflow != nullptr && !PER) {
        // the three axes' FP64 sums, over each wave and then in wave order
        const int wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const double w = wave_sum_f64(out[ax]);
            if ((threadIdx.x & 63) == 0) red[ax][wave] = w;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                double tot = 0.0;
                for (int q = 0; q < nw; ++q) tot += red[ax][q];
                prev += tot * a.du3;
            }
            a.outflow[cell] = prev;
        }
    }
}

size_t any_lds_bytes(int prec, const int nu[3])
{
    const size_t lines = (size_t)nu[0] * nu[1];
    return (lines * (size_t)(nu[2] | 1) + (prec == PREC_F32 ? 0 : lines)) * sizeof(float);
}

template <int P, int V>
hipError_t launch_any_v(const void* fin, const float* sin, void* fout, float* sout,
                        const KickArgs& a, hipStream_t st)
{
    using T = typename Codec<P>::T;
    const AnyArgs b(a.nu);
    const size_t lds = any_lds_bytes(P, a.nu);
    auto kern = a.periodic ? k_kick_any<P, V, true> : k_kick_any<P, V, false>;
    if (lds > ((size_t)48 << 10)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // about 16 waves per CU over the work-groups whose blocks share its LDS,
    // and no more threads than the sweep with the most lines has lines
    const int share = (int)(((size_t)160 << 10) / (lds + 2048));
    int nt = 1024 / (share < 1 ? 1 : share);
    const long most = max(max((long)a.nu[1] * a.nu[2], (long)a.nu[0] * a.nu[2]),
                          (long)a.nu[0] * a.nu[1]);
    if (nt > most) nt = (int)most;
    nt = (nt + 63) / 64 * 64;
    hipLaunchKernelGGL(kern, dim3((unsigned)a.cells), dim3((unsigned)nt), lds, st, (const T*)fin,
                       sin, (T*)fout, sout, a, b);
    return hipGetLastError();
}

template <int P>
hipError_t launch_any_p(const void* fin, const float* sin, void* fout, float* sout,
                        const KickArgs& a, hipStream_t st)
{
    // vectors that lie within a uz-line
    if (a.nu[2] % 4 == 0) return launch_any_v<P, 4>(fin, sin, fout, sout, a, st);
    if (a.nu[2] % 2 == 0) return launch_any_v<P, 2>(fin, sin, fout, sout, a, st);
    return launch_any_v<P, 1>(fin, sin, fout, sout, a, st);
}

}  // namespace

bool kick_any_supported(int prec, const int nu[3], size_t lds_limit)
{
    // (2 KiB for the static part; indices inside a block stay below 2^16)
    if ((double)nu[0] * nu[1] * (nu[2] + 2.0) >= 60000.0) return false;
    const size_t lds = any_lds_bytes(prec, nu) + 2048;
    if (lds > lds_limit) return false;
    // FP16/BF16 blocks that leave room for one work-group per CU round their
    // intermediate values in LDS with nothing to overlap it: taken only where
    // no strided sweep has a compiled line length (16 x 16 x 12 cells, FP16:
    // 40 x 16 x 32 0.35 ms, 0.31 as three sweeps; 33 x 36 x 32 0.63 and 0.72)
    auto compiled = [](int m) { return m == 16 || m == 32 || m == 64; };
    return prec == PREC_F32 || 2 * lds <= lds_limit || !(compiled(nu[0]) || compiled(nu[1]));
}

hipError_t launch_kick_any(int prec, const void* fin, const float* sin, void* fout, float* sout,
                           const KickArgs& a, hipStream_t st)
{
    if (a.cells == 0) return hipSuccess;
    switch (prec) {
        case PREC_F16: return launch_any_p<PREC_F16>(fin, sin, fout, sout, a, st);
        case PREC_BF16: return launch_any_p<PREC_BF16>(fin, sin, fout, sout, a, st);
        default: return launch_any_p<PREC_F32>(fin, sin, fout, sout, a, st);
    }
}

}  // namespace vlasov
