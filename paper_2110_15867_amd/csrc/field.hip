// Acceleration field of a density on the periodic spatial mesh: the Poisson
// equation (Eq. 2), nabla^2 phi = c (rho - mean rho) with c = 4 pi G a^2,
// solved by the discrete Fourier transform as the convolution method the
// paper uses for its mesh part (section 3), and g = -grad phi, the speed of
// the velocity sweeps (Eq. 4).  In Fourier space, with k_a = 2 pi m_a / L_a
// and m_a the signed index:
//   phi_k = -c rho_k / |k|^2 (phi_0 = 0: the mean drops out),
//   g_a,k = -i k_a phi_k, with k_a = 0 on the Nyquist plane of an even
//   axis (the derivative of a real Nyquist mode has no real representation).
//
// FP64 throughout, five launches over the half spectrum (the density is real,
// so k_z runs over 0 .. n_z/2):
//   z forward (two real lines as one complex line), y forward,
//   x forward, the Green's function, and x inverse of phi and -i k_x phi,
//   y inverse of the three components, z inverse of the three components
//   (again two real lines per complex one) with the FP32 store.
// A component needs only its own x- and y-derivative factor: k_y is constant
// along an x-line and k_z along an x- or y-line, so the x pass makes two
// arrays (phi and -i k_x phi) and the y pass three.  Every pass transforms
// bundles of lines in LDS by mixed-radix Stockham steps (the transform of a
// line of n costs n (sum of the factors) instead of n^2, and each value is
// read from HBM once per pass instead of n times).
//
// The mesh is small next to phase space (64^3: 2 MB of density) and each pass
// is a few microseconds, so the time is launches and latency: many small
// work-groups (8 complex lines each: 264 to 792 of them on 64^3), loads of a
// whole bundle in flight at once.  Measured on 64^3: 38 us per solve (passes
// of 6 to 13 us); 401 us as 19 launches of one-output-per-thread direct sums
// (12 passes of 33 us, each reading every value 64 times through the caches).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.hpp"

namespace vlasov {

namespace {

// unit: 2 pi / L of the axis (from the host: an FP64 division per value and
// axis took longer than the transforms)
__device__ __forceinline__ double wavenumber(int i, int n, double unit)
{
    const int m = 2 * i < n ? i : i - n;                 // signed index (Nyquist: -n/2)
    return unit * (double)m;
}

// the factor of the derivative along an axis: k, or 0 on its Nyquist plane
__device__ __forceinline__ double derivative_k(int i, int n, double unit)
{
    return (n % 2 == 0 && 2 * i == n) ? 0.0 : wavenumber(i, n, unit);
}

struct Mesh {
    int n[3];
    double unit[3];                       // 2 pi / L
    double coupling;
    long cells;
};

// ---------------------------------------------------------------------------
// Transforms of bundles of lines in LDS
// ---------------------------------------------------------------------------
constexpr int kMaxFactors = 16;
constexpr int kLines = 8;                 // complex lines per work-group
constexpr int kMaxLine = 256;             // longest line of the LDS transforms: two or three
                                          // buffers of 8 lines and the twiddles, 100 KiB

struct FftPlan {
    int n;
    int nf;
    int f[kMaxFactors];                   // radices, product n
};

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 w)
{
    return make_double2(fma(a.x, w.x, -(a.y * w.y)), fma(a.x, w.y, a.y * w.x));
}
// exp(-+ i pi/2) a, forward or inverse
template <bool INV>
__device__ __forceinline__ double2 crot(double2 a)
{
    return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

template <bool INV>
__device__ __forceinline__ void dft4(double2& a, double2& b, double2& c, double2& d)
{
    const double2 s = cadd(a, c), t = csub(a, c), u = cadd(b, d), v = crot<INV>(csub(b, d));
    a = cadd(s, u);
    b = cadd(t, v);
    c = csub(s, u);
    d = csub(t, v);
}

// DFT of R values in registers; w = exp(-2 pi i / R) powers from the line's
// twiddle table (tw[q * n / R]) for the odd radices
template <int R, bool INV>
__device__ __forceinline__ void dft_small(double2 (&v)[R], const double2* tw, int n)
{
    if constexpr (R == 2) {
        const double2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else if constexpr (R == 8) {
        const double h = 0.70710678118654752440;
        dft4<INV>(v[0], v[2], v[4], v[6]);
        dft4<INV>(v[1], v[3], v[5], v[7]);
        // odd part times exp(-+ i pi k / 4), k = 0..3
        const double2 o1 = v[3], o2 = v[5], o3 = v[7];
        const double2 r1 = INV ? make_double2(h * (o1.x - o1.y), h * (o1.x + o1.y))
                               : make_double2(h * (o1.x + o1.y), h * (o1.y - o1.x));
        const double2 r2 = crot<INV>(o2);
        const double2 r3 = INV ? make_double2(-h * (o3.x + o3.y), h * (o3.x - o3.y))
                               : make_double2(h * (o3.y - o3.x), -h * (o3.x + o3.y));
        const double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
        v[0] = cadd(e0, o0); v[4] = csub(e0, o0);
        v[1] = cadd(e1, r1); v[5] = csub(e1, r1);
        v[2] = cadd(e2, r2); v[6] = csub(e2, r2);
        v[3] = cadd(e3, r3); v[7] = csub(e3, r3);
    } else {
        double2 out[R];
        const int step = n / R;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            double2 s = v[0];
#pragma unroll
            for (int q = 1; q < R; ++q) {
                double2 w = tw[((k * q) % R) * step];
                if (INV) w.y = -w.y;
                s.x = fma(v[q].x, w.x, fma(-v[q].y, w.y, s.x));
                s.y = fma(v[q].x, w.y, fma(v[q].y, w.x, s.y));
            }
            out[k] = s;
        }
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = out[k];
    }
}

// One Stockham step of radix R: values j + q n/R (q = 0..R-1) of a line times
// w^(q (j mod ns) n / (ns R)), their R-point DFT, to (j / ns) ns R + j mod ns
// + q ns.  ns: product of the radices done before.
template <int R, bool INV>
__device__ __forceinline__ void stockham_step(const double2* in, double2* out, const double2* tw,
                                              int n, int ns)
{
    const int m = n / R;
    const int ts = n / (ns * R);
    for (int i = threadIdx.x; i < m * kLines; i += blockDim.x) {
        const int line = i % kLines, j = i / kLines;
        const int k = j % ns;
        double2 v[R];
#pragma unroll
        for (int q = 0; q < R; ++q) v[q] = in[(j + q * m) * kLines + line];
#pragma unroll
        for (int q = 1; q < R; ++q) {
            double2 w = tw[q * k * ts];
            if (INV) w.y = -w.y;
            v[q] = cmul(v[q], w);
        }
        dft_small<R, INV>(v, tw, n);
        const int d = (j / ns) * ns * R + k;
#pragma unroll
        for (int q = 0; q < R; ++q) out[(d + q * ns) * kLines + line] = v[q];
    }
}

// The same for any radix (a prime factor above 7): one output per thread.
template <bool INV>
__device__ __forceinline__ void stockham_any(const double2* in, double2* out, const double2* tw,
                                             int n, int ns, int R)
{
    const int m = n / R;
    for (int i = threadIdx.x; i < n * kLines; i += blockDim.x) {
        const int line = i % kLines, e = i / kLines;
        const int j = e % m, p = e / m;          // butterfly and output index
        const int k = j % ns;
        const int ts = n / (ns * R);
        // twiddle of term q: w^(q k ts + q p n / R)
        const int inc = (int)(((long)k * ts + (long)p * m) % n);
        int t = 0;
        double2 s = make_double2(0.0, 0.0);
        for (int q = 0; q < R; ++q) {
            double2 w = tw[t];
            if (INV) w.y = -w.y;
            const double2 x = in[(j + q * m) * kLines + line];
            s.x = fma(x.x, w.x, fma(-x.y, w.y, s.x));
            s.y = fma(x.x, w.y, fma(x.y, w.x, s.y));
            t += inc;
            if (t >= n) t -= n;
        }
        out[((j / ns) * ns * R + k + p * ns) * kLines + line] = s;
    }
}

// Transform of the bundle in A (B: scratch of the same size); returns the
// buffer that holds the result.  Begins and ends with a barrier.
template <bool INV>
__device__ double2* transform(double2* A, double2* B, const double2* tw, const FftPlan& p)
{
    int ns = 1;
    __syncthreads();
    for (int s = 0; s < p.nf; ++s) {
        const int R = p.f[s];
        switch (R) {
            case 2: stockham_step<2, INV>(A, B, tw, p.n, ns); break;
            case 3: stockham_step<3, INV>(A, B, tw, p.n, ns); break;
            case 4: stockham_step<4, INV>(A, B, tw, p.n, ns); break;
            case 5: stockham_step<5, INV>(A, B, tw, p.n, ns); break;
            case 7: stockham_step<7, INV>(A, B, tw, p.n, ns); break;
            case 8: stockham_step<8, INV>(A, B, tw, p.n, ns); break;
            default: stockham_any<INV>(A, B, tw, p.n, ns, R); break;
        }
        ns *= R;
        double2* t = A;
        A = B;
        B = t;
        __syncthreads();
    }
    return A;
}

// put(i, get(i)) for i < total over the work-group, eight loads in flight per
// thread before the first is used (one at a time the loads of a bundle were
// a chain of memory latencies: 12 us per pass instead of 8)
template <class T, class Get, class Put>
__device__ __forceinline__ void batched(int total, Get&& get, Put&& put)
{
    constexpr int U = 8;
    for (int i0 = threadIdx.x; i0 < total; i0 += U * blockDim.x) {
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * blockDim.x;
            if (i < total) v[u] = get(i);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * blockDim.x;
            if (i < total) put(i, v[u]);
        }
    }
}

// tw[m] = exp(-2 pi i m / n), m < n, in LDS (each work-group its own: n
// sincospi are cheaper than a launch)
__device__ __forceinline__ void twiddles(double2* tw, int n)
{
    for (int m = threadIdx.x; m < n; m += blockDim.x) {
        double s, c;
        sincospi(2.0 * (double)m / (double)n, &s, &c);
        tw[m] = make_double2(c, -s);
    }
}

// z forward: the real lines 2 b, 2 b + 1 (b = the complex line of the bundle)
// as one complex line a + i b, then a_k = (Z_k + conj Z_{n-k}) / 2 and
// b_k = (Z_k - conj Z_{n-k}) / 2i for k <= n/2.
__global__ void __launch_bounds__(256) k_fft_z_fwd(const double* __restrict__ rho,
                                                   double2* __restrict__ S, int rows, FftPlan p)
{
    extern __shared__ double2 sm[];
    const int n = p.n, nh = n / 2 + 1;
    double2* A = sm;
    double2* B = sm + n * kLines;
    double2* tw = B + n * kLines;
    const int r0 = blockIdx.x * 2 * kLines;
    double* Ad = reinterpret_cast<double*>(A);
    const int have = (rows - r0 < 2 * kLines ? rows - r0 : 2 * kLines) * n;
    batched<double>(2 * kLines * n,
        [&](int i) { return i < have ? rho[(long)r0 * n + i] : 0.0; },
        [&](int i, double x) {
            const int r = i / n, l = i - r * n;
            Ad[(l * kLines + r / 2) * 2 + (r & 1)] = x;
        });
    twiddles(tw, n);
    const double2* Z = transform<false>(A, B, tw, p);
    for (int i = threadIdx.x; i < 2 * kLines * nh; i += blockDim.x) {
        const int r = i / nh, k = i - r * nh;
        if (r0 + r >= rows) continue;
        const double2 u = Z[k * kLines + r / 2];
        const double2 v = Z[(k == 0 ? 0 : n - k) * kLines + r / 2];
        S[(long)r0 * nh + i] = (r & 1) ? make_double2(0.5 * (u.y + v.y), 0.5 * (v.x - u.x))
                                       : make_double2(0.5 * (u.x + v.x), 0.5 * (u.y - v.y));
    }
}

// One bundle of strided complex lines: nl of them from element `base`, rows
// `stride` apart.
__device__ __forceinline__ void load_lines(double2* A, const double2* src, long base, long stride,
                                           int n, int nl)
{
    batched<double2>(n * kLines,
        [&](int i) {
            const int line = i % kLines, l = i / kLines;
            return line < nl ? src[base + (long)l * stride + line] : make_double2(0.0, 0.0);
        },
        [&](int i, double2 x) { A[i] = x; });
}

// y forward, in place: lines along i1 of S[n0][n1][nh], bundles of k_z.
__global__ void __launch_bounds__(256) k_fft_y_fwd(double2* __restrict__ S, int nh, int tiles,
                                                   FftPlan p)
{
    extern __shared__ double2 sm[];
    const int n = p.n;
    double2* A = sm;
    double2* B = sm + n * kLines;
    double2* tw = B + n * kLines;
    const int i0 = blockIdx.x / tiles, c0 = (blockIdx.x % tiles) * kLines;
    const int nl = nh - c0 < kLines ? nh - c0 : kLines;
    const long base = (long)i0 * n * nh + c0;
    load_lines(A, S, base, nh, n, nl);
    twiddles(tw, n);
    const double2* Z = transform<false>(A, B, tw, p);
    for (int i = threadIdx.x; i < n * kLines; i += blockDim.x) {
        const int line = i % kLines, l = i / kLines;
        if (line < nl) S[base + (long)l * nh + line] = Z[i];
    }
}

// x forward, phi_k, x inverse of phi (to P, which may be S itself) and of
// -i k_x phi (to Q).
__global__ void __launch_bounds__(256) k_fft_x(const double2* S, double2* P, double2* __restrict__ Q,
                                               int nh, int tiles, FftPlan p, Mesh a)
{
    extern __shared__ double2 sm[];
    const int n = p.n;
    double2* A = sm;
    double2* B = sm + n * kLines;
    double2* tw = B + n * kLines;
    double2* K = tw + n;                      // phi_k, kept for the second inverse
    const int i1 = blockIdx.x / tiles, c0 = (blockIdx.x % tiles) * kLines;
    const int nl = nh - c0 < kLines ? nh - c0 : kLines;
    const long base = (long)i1 * nh + c0, stride = (long)a.n[1] * nh;
    load_lines(A, S, base, stride, n, nl);
    twiddles(tw, n);
    const double2* Z = transform<false>(A, B, tw, p);
    const double ky = wavenumber(i1, a.n[1], a.unit[1]);
    for (int i = threadIdx.x; i < n * kLines; i += blockDim.x) {
        const int line = i % kLines, l = i / kLines;
        const double kx = wavenumber(l, n, a.unit[0]);
        const double kz = wavenumber(c0 + line, a.n[2], a.unit[2]);
        const double k2 = fma(kz, kz, fma(ky, ky, kx * kx));
        const bool zero = l == 0 && i1 == 0 && c0 + line == 0;
        const double s = zero || line >= nl ? 0.0 : -a.coupling / k2;
        K[i] = make_double2(s * Z[i].x, s * Z[i].y);
    }
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
        for (int i = threadIdx.x; i < n * kLines; i += blockDim.x) {
            if (pass == 0) {
                A[i] = K[i];
            } else {
                // -i k (x + i y) = k y - i k x
                const double kx = derivative_k(i / kLines, n, a.unit[0]);
                A[i] = make_double2(kx * K[i].y, -kx * K[i].x);
            }
        }
        const double2* R = transform<true>(A, B, tw, p);
        double2* dst = pass == 0 ? P : Q;
        for (int i = threadIdx.x; i < n * kLines; i += blockDim.x) {
            const int line = i % kLines, l = i / kLines;
            if (line < nl) dst[base + (long)l * stride + line] = R[i];
        }
        __syncthreads();
    }
}

// y inverse of component blockIdx.y: of -i k_x phi (0), -i k_y phi (1) and
// phi, times -i k_z (2), to G[component][n0][n1][nh].
__global__ void __launch_bounds__(256) k_fft_y_inv(const double2* __restrict__ P,
                                                   const double2* __restrict__ Q,
                                                   double2* __restrict__ G, int nh, int tiles,
                                                   FftPlan p, Mesh a)
{
    extern __shared__ double2 sm[];
    const int n = p.n, comp = blockIdx.y;
    double2* A = sm;
    double2* B = sm + n * kLines;
    double2* tw = B + n * kLines;
    const int i0 = blockIdx.x / tiles, c0 = (blockIdx.x % tiles) * kLines;
    const int nl = nh - c0 < kLines ? nh - c0 : kLines;
    const long base = (long)i0 * n * nh + c0;
    load_lines(A, comp == 0 ? Q : P, base, nh, n, nl);
    if (comp == 1) {
        for (int i = threadIdx.x; i < n * kLines; i += blockDim.x) {
            const double ky = derivative_k(i / kLines, n, a.unit[1]);   // (the thread's own values)
            A[i] = make_double2(ky * A[i].y, -ky * A[i].x);
        }
    }
    twiddles(tw, n);
    const double2* R = transform<true>(A, B, tw, p);
    double2* dst = G + (long)comp * a.n[0] * n * nh;
    for (int i = threadIdx.x; i < n * kLines; i += blockDim.x) {
        const int line = i % kLines, l = i / kLines;
        if (line >= nl) continue;
        double2 x = R[i];
        if (comp == 2) {
            const double kz = derivative_k(c0 + line, a.n[2], a.unit[2]);
            x = make_double2(kz * x.y, -kz * x.x);
        }
        dst[base + (long)l * nh + line] = x;
    }
}

// z inverse: the half spectra of two real lines a, b as Z_k = a_k + i b_k
// with their Hermitian extension; the transform's real part is a, its
// imaginary part b.  `rows` lines of all three components.
__global__ void __launch_bounds__(256) k_fft_z_inv(const double2* __restrict__ G,
                                                   float* __restrict__ g, long rows, double inv_n,
                                                   FftPlan p)
{
    extern __shared__ double2 sm[];
    const int n = p.n, nh = n / 2 + 1;
    double2* A = sm;
    double2* B = sm + n * kLines;
    double2* tw = B + n * kLines;
    double2* H = tw + n;                      // half spectra of the 2 kLines real lines
    const long r0 = (long)blockIdx.x * 2 * kLines;
    const int have = (int)(rows - r0 < 2 * kLines ? rows - r0 : 2 * kLines) * nh;
    batched<double2>(2 * kLines * nh,
        [&](int i) { return i < have ? G[r0 * nh + i] : make_double2(0.0, 0.0); },
        [&](int i, double2 x) { H[i] = x; });
    __syncthreads();
    for (int i = threadIdx.x; i < n * kLines; i += blockDim.x) {
        const int line = i % kLines, k = i / kLines;
        const bool up = 2 * k > n;                      // conjugate half
        const int kk = up ? n - k : k;
        double2 u = H[2 * line * nh + kk], v = H[(2 * line + 1) * nh + kk];
        // a real line's k = 0 and Nyquist values are real
        if (kk == 0 || 2 * kk == n) u.y = v.y = 0.0;
        if (up) {
            u.y = -u.y;
            v.y = -v.y;
        }
        A[i] = make_double2(u.x - v.y, u.y + v.x);
    }
    twiddles(tw, n);
    const double2* R = transform<true>(A, B, tw, p);
    const double* Rd = reinterpret_cast<const double*>(R);
    for (int i = threadIdx.x; i < 2 * kLines * n; i += blockDim.x) {
        const int r = i / n, l = i - r * n;
        if (r0 + r < rows) g[r0 * n + i] = (float)(Rd[(l * kLines + r / 2) * 2 + (r & 1)] * inv_n);
    }
}

// Radices of n: 8s first (their butterflies keep the most in registers), then
// 4, 2 and the odd primes.
bool make_plan(int n, FftPlan& p)
{
    p.n = n;
    p.nf = 0;
    int m = n;
    const int pref[6] = {8, 4, 2, 7, 5, 3};
    for (int r : pref)
        while (m % r == 0) {
            p.f[p.nf++] = r;
            m /= r;
        }
    for (int r = 11; m > 1; r += 2)
        while (m % r == 0) {
            p.f[p.nf++] = r;
            m /= r;
        }
    return p.nf <= kMaxFactors;               // n <= 256: at most 3 + 8 radices
}

size_t lds_bytes(int n, int extra) { return ((size_t)2 * n * kLines + n + extra) * sizeof(double2); }
// of the passes that hold most: x with phi_k beside its lines, z inverse with
// the half spectra
size_t lds_x(int n) { return lds_bytes(n, n * kLines); }
size_t lds_z_inv(int n) { return lds_bytes(n, 2 * kLines * (n / 2 + 1)); }

// two values of a bundle per thread (64 threads at least, 256 at most): the
// loads, stores and spectral factors of a bundle are short chains, the
// radix-8 butterflies of the first wave the only serial part
unsigned threads_for(int n) { return n <= 16 ? 64 : (n <= 32 ? 128 : 256); }

// more than 64 KiB of dynamic LDS (lines beyond 160 cells) has to be asked for
template <class K>
hipError_t allow_lds(K kern, size_t bytes)
{
    if (bytes <= (size_t)64 << 10) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_field_fft(const double* rho, float* g, const Mesh& a, void* work,
                            hipStream_t st)
{
    const int n0 = a.n[0], n1 = a.n[1], n2 = a.n[2], nh = n2 / 2 + 1;
    FftPlan p[3];
    for (int d = 0; d < 3; ++d)
        if (!make_plan(a.n[d], p[d])) return hipErrorInvalidValue;
    // half spectra S (then phi after the x inverse), Q and the three
    // components, within the workspace's five complex [cells] arrays (nh <= n2)
    const size_t half = field_align((size_t)n0 * n1 * nh * sizeof(double2));
    double2* S = (double2*)work;
    double2* Q = (double2*)((char*)work + half);
    double2* G = (double2*)((char*)work + 2 * half);
    const int tiles = (nh + kLines - 1) / kLines;
    const int rows = n0 * n1;
    const long rows3 = 3L * rows;
    const size_t lx = lds_x(n0), ly = lds_bytes(n1, 0);
    const size_t lf = lds_bytes(n2, 0), li = lds_z_inv(n2);
    hipError_t e;
    if ((e = allow_lds(k_fft_z_fwd, lf)) != hipSuccess) return e;
    if ((e = allow_lds(k_fft_y_fwd, ly)) != hipSuccess) return e;
    if ((e = allow_lds(k_fft_x, lx)) != hipSuccess) return e;
    if ((e = allow_lds(k_fft_y_inv, ly)) != hipSuccess) return e;
    if ((e = allow_lds(k_fft_z_inv, li)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_fft_z_fwd, dim3((rows + 2 * kLines - 1) / (2 * kLines)),
                       dim3(threads_for(n2)), lf, st, rho, S, rows, p[2]);
    hipLaunchKernelGGL(k_fft_y_fwd, dim3((unsigned)n0 * tiles), dim3(threads_for(n1)), ly, st, S,
                       nh, tiles, p[1]);
    hipLaunchKernelGGL(k_fft_x, dim3((unsigned)n1 * tiles), dim3(threads_for(n0)), lx, st, S, S, Q,
                       nh, tiles, p[0], a);
    hipLaunchKernelGGL(k_fft_y_inv, dim3((unsigned)n0 * tiles, 3), dim3(threads_for(n1)), ly, st,
                       S, Q, G, nh, tiles, p[1], a);
    hipLaunchKernelGGL(k_fft_z_inv, dim3((unsigned)((rows3 + 2 * kLines - 1) / (2 * kLines))),
                       dim3(threads_for(n2)), li, st, G, g, rows3, 1.0 / (double)a.cells, p[2]);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Meshes with an axis beyond kMaxLine cells, or whose lines LDS does not hold: plain separable DFTs, one output
// element per thread and one axis per pass, with exact twiddle indices
// (k l mod n).
// ---------------------------------------------------------------------------
// tw[m] = exp(-2 pi i m / n)
__global__ void __launch_bounds__(256) k_twiddles(double2* __restrict__ tw, int n)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    double s, c;
    sincospi(2.0 * (double)m / (double)n, &s, &c);
    tw[m] = make_double2(c, -s);
}

// One DFT pass along `axis` of a complex [n0][n1][n2] array (real input when
// `rin` is given).  Forward: sum_l x_l exp(-2 pi i k l / n); inverse: the
// conjugate twiddles (no 1/n).
__global__ void __launch_bounds__(256) k_dft_axis(const double2* __restrict__ in,
                                                  const double* __restrict__ rin,
                                                  double2* __restrict__ out,
                                                  const double2* __restrict__ tw, int n0, int n1,
                                                  int n2, int axis, int inverse)
{
    const long cells = (long)n0 * n1 * n2;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= cells) return;
    const int i2 = (int)(t % n2);
    const int i1 = (int)((t / n2) % n1);
    const int i0 = (int)(t / ((long)n1 * n2));
    const int n = axis == 0 ? n0 : (axis == 1 ? n1 : n2);
    const long stride = axis == 0 ? (long)n1 * n2 : (axis == 1 ? n2 : 1);
    const int k = axis == 0 ? i0 : (axis == 1 ? i1 : i2);
    const long base = t - (long)k * stride;              // element l = 0 of this line
    double re = 0.0, im = 0.0;
    int m = 0;                                           // k * l mod n
    for (int l = 0; l < n; ++l) {
        const double2 w = tw[m];
        const double wi = inverse ? -w.y : w.y;
        if (rin != nullptr) {
            const double x = rin[base + (long)l * stride];
            re = fma(x, w.x, re);
            im = fma(x, wi, im);
        } else {
            const double2 x = in[base + (long)l * stride];
            re = fma(x.x, w.x, fma(-x.y, wi, re));
            im = fma(x.x, wi, fma(x.y, w.x, im));
        }
        m += k;
        if (m >= n) m -= n;
    }
    out[t] = make_double2(re, im);
}

// phi_k and the three components g_a,k = -i k_a phi_k
__global__ void __launch_bounds__(256) k_poisson(const double2* __restrict__ R,
                                                 double2* __restrict__ G, Mesh a)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= a.cells) return;
    const int i2 = (int)(t % a.n[2]);
    const int i1 = (int)((t / a.n[2]) % a.n[1]);
    const int i0 = (int)(t / ((long)a.n[1] * a.n[2]));
    const int idx[3] = {i0, i1, i2};
    double k2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double k = wavenumber(idx[d], a.n[d], a.unit[d]);
        k2 = fma(k, k, k2);
    }
    double2 phi = make_double2(0.0, 0.0);
    if (t != 0) {
        const double s = -a.coupling / k2;
        phi = make_double2(s * R[t].x, s * R[t].y);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double kd = derivative_k(idx[d], a.n[d], a.unit[d]);
        // -i kd (phi.x + i phi.y) = kd phi.y - i kd phi.x
        G[(long)d * a.cells + t] = make_double2(kd * phi.y, -kd * phi.x);
    }
}

__global__ void __launch_bounds__(256) k_field_store(const double2* __restrict__ X,
                                                     float* __restrict__ g, long cells,
                                                     double inv_n)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= cells) return;
    g[t] = (float)(X[t].x * inv_n);
}

hipError_t launch_field_direct(const double* rho, float* g, const Mesh& a, void* work,
                               hipStream_t st)
{
    const long cells = a.cells;
    const int n0 = a.n[0], n1 = a.n[1], n2 = a.n[2];
    double2* tw[3];
    char* p = (char*)work;
    for (int d = 0; d < 3; ++d) {
        tw[d] = (double2*)p;
        p += field_align((size_t)a.n[d] * sizeof(double2));
    }
    double2* A = (double2*)p;
    p += field_align((size_t)cells * sizeof(double2));
    double2* B = (double2*)p;
    p += field_align((size_t)cells * sizeof(double2));
    double2* G = (double2*)p;
    const unsigned blocks = (unsigned)((cells + 255) / 256);
    for (int d = 0; d < 3; ++d)
        hipLaunchKernelGGL(k_twiddles, dim3((a.n[d] + 255) / 256), dim3(256), 0, st, tw[d], a.n[d]);
    // forward: z (from the real density), y, x
    hipLaunchKernelGGL(k_dft_axis, dim3(blocks), dim3(256), 0, st, (const double2*)nullptr, rho, A,
                       tw[2], n0, n1, n2, 2, 0);
    hipLaunchKernelGGL(k_dft_axis, dim3(blocks), dim3(256), 0, st, A, (const double*)nullptr, B,
                       tw[1], n0, n1, n2, 1, 0);
    hipLaunchKernelGGL(k_dft_axis, dim3(blocks), dim3(256), 0, st, B, (const double*)nullptr, A,
                       tw[0], n0, n1, n2, 0, 0);
    hipLaunchKernelGGL(k_poisson, dim3(blocks), dim3(256), 0, st, A, G, a);
    const double inv_n = 1.0 / (double)cells;
    for (int d = 0; d < 3; ++d) {
        const double2* Gd = G + (long)d * cells;
        hipLaunchKernelGGL(k_dft_axis, dim3(blocks), dim3(256), 0, st, Gd, (const double*)nullptr,
                           B, tw[0], n0, n1, n2, 0, 1);
        hipLaunchKernelGGL(k_dft_axis, dim3(blocks), dim3(256), 0, st, B, (const double*)nullptr,
                           A, tw[1], n0, n1, n2, 1, 1);
        hipLaunchKernelGGL(k_dft_axis, dim3(blocks), dim3(256), 0, st, A, (const double*)nullptr,
                           B, tw[2], n0, n1, n2, 2, 1);
        hipLaunchKernelGGL(k_field_store, dim3(blocks), dim3(256), 0, st, B, g + (long)d * cells,
                           cells, inv_n);
    }
    return hipGetLastError();
}

}  // namespace

bool field_fft_supported(const int n[3], size_t lds_limit)
{
    if (n[0] > kMaxLine || n[1] > kMaxLine || n[2] > kMaxLine) return false;
    return lds_x(n[0]) <= lds_limit && lds_bytes(n[1], 0) <= lds_limit && lds_z_inv(n[2]) <= lds_limit;
}

hipError_t launch_field(const double* rho, float* g, const FieldArgs& a, void* work,
                        hipStream_t st)
{
    if (a.cells == 0) return hipSuccess;
    Mesh m;
    for (int d = 0; d < 3; ++d) {
        m.n[d] = a.n[d];
        m.unit[d] = 2.0 * 3.141592653589793 / a.L[d];
    }
    m.coupling = a.coupling;
    m.cells = a.cells;
    if (field_fft_supported(a.n, lds_limit()))
        return launch_field_fft(rho, g, m, work, st);
    return launch_field_direct(rho, g, m, work, st);
}

}  // namespace vlasov
