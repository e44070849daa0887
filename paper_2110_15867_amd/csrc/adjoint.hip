// Tangent-linear and adjoint sweeps (FP32 storage only).
//
// With the limiter's selections frozen at the forward input, one sweep of a
// line is a linear map of the cell values, f' = J f, and a smooth function of
// the fractional shift nu (through the semi-Lagrangian weights and the
// factor mu of the flux).  Each interface flux is linearised as
//   Phi = sum_k W_k f_{j+k} (upwind frame, k = -2..2),  dPhi/dmu,
// by re-running the forward arithmetic of flux_mag on the forward input with
// the same FP32 operations, so every selection (early-out, curvature
// minmods, bounds, median, positivity clamp) is the forward's own, and then
// reading off which candidate each selection returned.  Ties between equal
// candidates are resolved as in the FP64 oracle: min and max keep their first
// argument, the median is max(min(x,y), min(max(x,y),z)).
//
//  tangent: out_dot_i = v_{i-N} - (Phi_dot_{j+1/2} - Phi_dot_{j-1/2}), j = i-N,
//           Phi_dot = W . v + dPhi/dmu * mu_dot
//  adjoint: lam_in_r = lam_{r+N} + sum_{k} psi_{r-k} W_{r-k}[k],
//           psi_j = lam_{j+N+1} - lam_{j+N}, lam_mu = sum_j psi_j dPhi_j/dmu
// (all in the walk frame of the line; lines with a negative shift are walked
// mirrored, where mu = -nu).  Each input cell is written once, when the last
// of the five interfaces that read it has added its term.
//
// One thread per line.  Lines along x, y, z, ux and uy are read with direct
// strided loads (neighbouring lanes take neighbouring elements of a row, so
// every access is coalesced); the contiguous uz-lines go through LDS tiles of
// whole lines, loaded and stored with 16-byte accesses, as in the forward uz
// sweep.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.hpp"
#include "rows.hpp"
#include "sl_mpp5.hpp"

namespace vlasov {

namespace {

// Derivatives of the interface-value weights with respect to mu.
struct WeightSlopes {
    float d0, d1, d2, d3, d4;
};

__device__ __forceinline__ WeightSlopes sl5_weight_slopes(float mu)
{
    const float m2 = mu * mu, m3 = m2 * mu;
    const float k = 1.0f / 120.0f;
    WeightSlopes s;
    s.d0 = (4.0f * m3 - 10.0f * mu) * k;
    s.d1 = -(16.0f * m3 - 15.0f * m2 - 60.0f * mu + 5.0f) * k;
    s.d2 = (24.0f * m3 - 45.0f * m2 - 80.0f * mu + 75.0f) * k;
    s.d3 = -(16.0f * m3 - 45.0f * m2 - 20.0f * mu + 75.0f) * k;
    s.d4 = (4.0f * m3 - 15.0f * m2 + 10.0f * mu + 5.0f) * k;
    return s;
}

// Linear form over the stencil (a, b, c, d, e), with the derivative with
// respect to mu in slot 5 (the stencil values do not depend on mu).
struct Lin {
    float w[6];
};

__device__ __forceinline__ Lin lin_zero()
{
    Lin r;
#pragma unroll
    for (int q = 0; q < 6; ++q) r.w[q] = 0.0f;
    return r;
}

__device__ __forceinline__ Lin lin_unit(int k)
{
    Lin r = lin_zero();
    r.w[k] = 1.0f;
    return r;
}

__device__ __forceinline__ Lin lin_comb(float p, const Lin& x, float q, const Lin& y)
{
    Lin r;
#pragma unroll
    for (int i = 0; i < 6; ++i) r.w[i] = p * x.w[i] + q * y.w[i];
    return r;
}

__device__ __forceinline__ Lin lin_scale(float p, const Lin& x)
{
    Lin r;
#pragma unroll
    for (int i = 0; i < 6; ++i) r.w[i] = p * x.w[i];
    return r;
}

// A value with its linear form.
struct VL {
    float v;
    Lin l;
};
struct FluxLin {
    float W[5];     // d phi / d (a..e)
    float dmu;      // d phi / d mu
};

// Selections on (value, candidate index) pairs with the FP64 oracle's tie
// rules (min and max keep their first argument on a tie; the median is
// max(min(x,y), min(max(x,y),z))): every selection is decided on the
// values, and the linear form is built for the winning candidate only.
struct Pick {
    float v;
    int id;
};
__device__ __forceinline__ Pick pmin2(const Pick& x, const Pick& y) { return x.v <= y.v ? x : y; }
__device__ __forceinline__ Pick pmax2(const Pick& x, const Pick& y) { return x.v >= y.v ? x : y; }
__device__ __forceinline__ Pick pmed3(const Pick& x, const Pick& y, const Pick& z)
{
    return pmax2(pmin2(x, y), pmin2(pmax2(x, y), z));
}
// minmod of four; id 4 stands for the zero it returns when signs differ
__device__ __forceinline__ Pick pminmod4(const Pick& w, const Pick& x, const Pick& y, const Pick& z)
{
    if (w.v > 0.0f && x.v > 0.0f && y.v > 0.0f && z.v > 0.0f)
        return pmin2(pmin2(w, x), pmin2(y, z));
    if (w.v < 0.0f && x.v < 0.0f && y.v < 0.0f && z.v < 0.0f)
        return pmax2(pmax2(w, x), pmax2(y, z));
    return Pick{0.0f, 4};
}

// curv_minmod on (value, candidate): the value with curv_minmod's FP32
// operations (so the bounds that use it are the forward's), the candidate
// the oracle's minmod of four picks where its value is the same, else the
// one the value came from (m = minmod(Da, Db), or 4m - o with o the other).
__device__ __forceinline__ Pick pcurv_minmod(float Da, float Db)
{
    const float v = curv_minmod(Da, Db);
    const Pick w = pminmod4(Pick{fmaf(4.0f, Da, -Db), 0}, Pick{fmaf(4.0f, Db, -Da), 1},
                            Pick{Da, 2}, Pick{Db, 3});
    if (w.v == v) return Pick{v, w.id};
    if (v == 0.0f) return Pick{v, 4};
    const bool a_least = med3(Da, Db, 0.0f) == Da;
    if (v == (a_least ? Da : Db)) return Pick{v, a_least ? 2 : 3};
    return Pick{v, a_least ? 0 : 1};
}

// Form of the curvature minmod that won: candidates 4 Da - Db (0),
// 4 Db - Da (1), Da (2), Db (3), zero (4).
__device__ __forceinline__ Lin minmod_form(int id, const Lin& Da, const Lin& Db)
{
    switch (id) {
        case 0: return lin_comb(4.0f, Da, -1.0f, Db);
        case 1: return lin_comb(4.0f, Db, -1.0f, Da);
        case 2: return Da;
        case 3: return Db;
        default: return lin_zero();
    }
}

__device__ __forceinline__ Lin curvature_form(const Lin& l, const Lin& m, const Lin& r)
{
    return lin_comb(1.0f, lin_comb(1.0f, l, -2.0f, m), 1.0f, r);
}

// mp_bounded on (value, form) pairs: the values with mp_bounded's FP32
// operations, so every selection is the forward's.  u[] are the forms of the
// stencil's a..e (the upwind frame's cells, or mirrored for a comp line);
// the upper-limit factor alpha carries its mu-derivative alpha_mu.  The
// candidates of the bounds are c (0), d (1), fMD (2), fUL (3), fLC (4) and
// the unlimited value fhat (5).
__device__ VL mp_bounded_lin(const VL& fhat, const Stencil& s, const Lin (&u)[5], float alpha,
                             float alpha_mu)
{
    const float Dmv = s.dm1 - s.dm2, D0v = s.d0 - s.dm1, Dpv = s.dp1 - s.d0;
    // curv_minmod(Da, Db) = minmod(4Da-Db, 4Db-Da, Da, Db)
    const Pick Mp = pcurv_minmod(D0v, Dpv);
    const Pick Mm = pcurv_minmod(Dmv, D0v);
    const Pick c{s.c, 0};
    const Pick d{s.d, 1};
    const Pick fMD{fmaf(-0.5f, Mp.v, fmaf(0.5f, s.d0, s.c)), 2};
    const Pick fUL{fmaf(alpha, s.dm1, s.c), 3};
    const Pick fLC{fmaf(4.0f / 3.0f, Mm.v, fmaf(0.5f, s.dm1, s.c)), 4};
    const Pick lo = pmax2(pmin2(pmin2(c, d), fMD), pmin2(pmin2(c, fUL), fLC));
    const Pick hi = pmin2(pmax2(pmax2(c, d), fMD), pmax2(pmax2(c, fUL), fLC));
    const Pick r = pmed3(Pick{fhat.v, 5}, lo, hi);
    VL out;
    out.v = r.v;
    switch (r.id) {
        case 5: out.l = fhat.l; break;
        case 0: out.l = u[2]; break;
        case 1: out.l = u[3]; break;
        case 3: {
            const Lin cb = lin_comb(1.0f, u[2], -1.0f, u[1]);                 // c - b
            out.l = lin_comb(alpha, cb, 1.0f, u[2]);
            out.l.w[5] += alpha_mu * s.dm1;
            break;
        }
        case 2: {
            const Lin D0 = curvature_form(u[1], u[2], u[3]);
            const Lin Dp = curvature_form(u[2], u[3], u[4]);
            out.l = lin_comb(0.5f, lin_comb(1.0f, u[2], 1.0f, u[3]), -0.5f,
                             minmod_form(Mp.id, D0, Dp));
            break;
        }
        default: {
            const Lin cb = lin_comb(1.0f, u[2], -1.0f, u[1]);
            const Lin Dm = curvature_form(u[0], u[1], u[2]);
            const Lin D0 = curvature_form(u[1], u[2], u[3]);
            out.l = lin_comb(4.0f / 3.0f, minmod_form(Mm.id, Dm, D0), 1.0f,
                             lin_comb(0.5f, cb, 1.0f, u[2]));
            break;
        }
    }
    return out;
}

// The forward flux with its frozen linearisation.  The values follow
// flux_mag / mp_flux / mp_bounded operation by operation, so every selection
// is the forward's (the clamp of a comp line is read on the complement, see
// below).
__device__ FluxLin flux_lin(const Stencil& s, const LineShift& sh, const WeightSlopes& ds)
{
    float y = sh.v0 * s.dm2;
    y = fmaf(sh.v1, s.dm1, y);
    y = fmaf(sh.v2, s.d0, y);
    y = fmaf(sh.v3, s.dp1, y);
    const float m = med3(s.d0, sh.alpha * s.dm1, 0.0f);
    // y = fhat - c as a form: the weights, and d fhat / d mu
    VL Y;
    Y.v = y;
    Y.l.w[0] = sh.w0; Y.l.w[1] = sh.w1; Y.l.w[2] = sh.w2 - 1.0f; Y.l.w[3] = sh.w3;
    Y.l.w[4] = sh.w4;
    float ydmu = ds.d0 * s.a;
    ydmu = fmaf(ds.d1, s.b, ydmu);
    ydmu = fmaf(ds.d2, s.c, ydmu);
    ydmu = fmaf(ds.d3, s.d, ydmu);
    ydmu = fmaf(ds.d4, s.e, ydmu);
    Y.l.w[5] = ydmu;
    const Lin uc = lin_unit(2);
    const bool early = med3(y, 0.0f, m) == y;
    FluxLin out;
    VL r;
    if (!sh.comp) {
        VL F{s.c + y, lin_comb(1.0f, uc, 1.0f, Y.l)};
        if (!early) {
            // d alpha / d mu = -1/mu^2 (0 where alpha is held at its cap)
            const float a_mu = sh.mu * (kAlphaCap + 1.0f) <= 1.0f ? 0.0f : -1.0f / (sh.mu * sh.mu);
            const Lin u[5] = {lin_unit(0), lin_unit(1), lin_unit(2), lin_unit(3), lin_unit(4)};
            F = mp_bounded_lin(F, s, u, sh.alpha, a_mu);
        }
        // positivity clamp med3(mu L, 0, c), oracle tie rules
        VL pre{sh.mu * F.v, lin_scale(sh.mu, F.l)};
        pre.l.w[5] = fmaf(sh.mu, F.l.w[5], F.v);
        const Pick k = pmed3(Pick{pre.v, 0}, Pick{0.0f, 1}, Pick{s.c, 2});
        r.v = k.v;
        r.l = k.id == 0 ? pre.l : (k.id == 1 ? lin_zero() : uc);
    } else {
        // complement: ghat = c - q y on the mirrored stencil with alpha_c; what
        // leaves through the complement side is Psi = med3(mu' ghat_lim, 0, c)
        // and Phi = c - Psi.  The selections of that clamp are taken on Psi,
        // as the split at the nearest integer takes them (its tie rules differ
        // from those of the same clamp written on Phi where c = 0).
        // dq/dmu = 1/mu'^2, d alpha_c/dmu = 1/mu'^2 (0 where held at its cap),
        // dmu'/dmu = -1.
        const float q_mu = 1.0f / (sh.muc * sh.muc);
        VL G{fmaf(-sh.q, y, s.c), lin_comb(1.0f, uc, -sh.q, Y.l)};
        G.l.w[5] = -sh.q * Y.l.w[5] - q_mu * y;
        if (!early) {
            const float ac_mu = sh.muc * (kAlphaCap + 1.0f) <= 1.0f ? 0.0f : q_mu;
            const Stencil mst{s.e, s.d, s.c, s.b, s.a, -s.dp1, -s.d0, -s.dm1, -s.dm2};
            const Lin u[5] = {lin_unit(4), lin_unit(3), lin_unit(2), lin_unit(1), lin_unit(0)};
            G = mp_bounded_lin(G, mst, u, sh.alpha_c, ac_mu);
        }
        VL P{sh.muc * G.v, lin_scale(sh.muc, G.l)};
        P.l.w[5] = sh.muc * G.l.w[5] - G.v;
        const Pick k = pmed3(Pick{P.v, 0}, Pick{0.0f, 1}, Pick{s.c, 2});
        const Lin psi = k.id == 0 ? P.l : (k.id == 1 ? lin_zero() : uc);
        r.v = s.c - k.v;
        r.l = lin_comb(1.0f, uc, -1.0f, psi);
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) out.W[q] = r.l.w[q];
    out.dmu = r.l.w[5];
    return out;
}

// Stencil of interface j+1/2 in the walk frame from a 5-value window.
__device__ __forceinline__ Stencil make_stencil(const float* w)
{
    return Stencil{w[0], w[1], w[2], w[3], w[4], w[1] - w[0], w[2] - w[1], w[3] - w[2],
                   w[4] - w[3]};
}

using Reader32 = GlobalReader<PREC_F32, 1, false>;

// Tangent of one line: x = forward input, v = input tangent, mu_dot = d mu.
__device__ void line_tangent(Reader32& rx, Reader32& rv, float* out, long stride, int M, int dir,
                             const LineShift& sh, bool periodic, float mu_dot)
{
    const WeightSlopes ds = sl5_weight_slopes(sh.mu);
    const int N = sh.N;
    float wx[5], wv[5];
    rx.seek(-N - 3);
    rv.seek(-N - 3);
    for (int q = 0; q < 5; ++q) {
        rx.next(&wx[q]);
        rv.next(&wv[q]);
    }
    auto dphi = [&](const float* xs, const float* vs) {
        const FluxLin fl = flux_lin(make_stencil(xs), sh, ds);
        float t = fl.dmu * mu_dot;
#pragma unroll
        for (int q = 0; q < 5; ++q) t = fmaf(fl.W[q], vs[q], t);
        return t;
    };
    float old = dphi(wx, wv);                     // interface j0 - 1/2
    for (int i = 0; i < M; ++i) {
        for (int q = 0; q < 4; ++q) {
            wx[q] = wx[q + 1];
            wv[q] = wv[q + 1];
        }
        rx.next(&wx[4]);
        rv.next(&wv[4]);
        const float nw = dphi(wx, wv);            // interface j + 1/2, j = i - N
        const int p = dir > 0 ? i : M - 1 - i;
        out[(long)p * stride] = wv[2] - (nw - old);
        old = nw;
    }
}

// ---------------------------------------------------------------------------
// Adjoint of one line, scatter form.  Interface j adds psi_j W_j[k] to the
// five rows j-2+k it reads (psi_j = lam_{j+N+1} - lam_{j+N}); the rows under
// construction are five registers, each started with its identity term
// lam_{r+N} at interface r-2 and finished by interface r+2, so a row's terms
// are added in interface order, and an interface's weights live only while it
// is handled.
//
// Most interfaces pass the Suresh-Huynh test and are not clamped: their
// weights are the line's constants E, and a wave whose 64 lanes all agree does
// the test, five FMAs and the shift derivative, about 30 vector instructions.
// Otherwise the bounds' selections are evaluated for all lanes by selects (no
// divergent branches), about 90 more: the winner is read off by equality from
// three-way minima and maxima, and its weights are assembled from the
// curvature minmod's two integers.  The values are those of mp_bounded_lin,
// operation by operation, so the weights have its bits.
// Bound by vector instructions.  Measured on 32^3 x 16^3 in mid-run, where
// nearly every wave has a limited lane (ms per launch): u_x, u_y 1.03 -> 0.53,
// u_z 1.12 -> 0.62, x, y, z 0.90 -> 0.51 on average, against the gather form
// (a 5 x 5 window of weights per lane, pairwise selections, linear forms
// behind a divergent switch; 248 -> 143 vector instructions per cell in u_x,
// u_y).
// ---------------------------------------------------------------------------
// A line's limiter side: whether the bounds act on the complement (see
// LineShift), the same for a whole wave (kPlain, kComp) or picked per lane.
enum Side { kPlain = 0, kComp = 1, kPerLane = 2 };

struct AdjLine {
    float E[5];      // weights of an interface that is neither bounded nor clamped
    float a_mu;      // d alpha / d mu of the bounds' upper limit
    float q_mu;      // d q / d mu (comp lines)
    WeightSlopes ds;
};

__device__ __forceinline__ AdjLine adj_line(const LineShift& sh)
{
    AdjLine L;
    L.ds = sl5_weight_slopes(sh.mu);
    const float y[5] = {sh.w0, sh.w1, sh.w2 - 1.0f, sh.w3, sh.w4};
    const float cap = kAlphaCap + 1.0f;
    if (!sh.comp) {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            L.E[k] = sh.mu * (k == 2 ? 1.0f + y[k] : y[k]);
        }
        L.a_mu = sh.mu * cap <= 1.0f ? 0.0f : -1.0f / (sh.mu * sh.mu);
        L.q_mu = 0.0f;
    } else {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const float qy = -sh.q * y[k];
            const float p = sh.muc * (k == 2 ? 1.0f + qy : qy);
            L.E[k] = k == 2 ? 1.0f - p : -p;
        }
        L.q_mu = 1.0f / (sh.muc * sh.muc);
        L.a_mu = sh.muc * cap <= 1.0f ? 0.0f : L.q_mu;
    }
    return L;
}

__device__ __forceinline__ AdjLine uniform_adj(const AdjLine& a)
{
    AdjLine u;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        u.E[k] = uniform_f32(a.E[k]);
    }
    u.a_mu = uniform_f32(a.a_mu);
    u.q_mu = uniform_f32(a.q_mu);
    u.ds.d0 = uniform_f32(a.ds.d0);
    u.ds.d1 = uniform_f32(a.ds.d1);
    u.ds.d2 = uniform_f32(a.ds.d2);
    u.ds.d3 = uniform_f32(a.ds.d3);
    u.ds.d4 = uniform_f32(a.ds.d4);
    return u;
}

// The curvature minmod's winning form p Da + q Db as the integers (p, q), for
// v = curv_minmod(Da, Db): the candidate pcurv_minmod picks.  With m the
// argument of least magnitude (Da of equal ones) and o the other, a nonzero v
// is m or 4 m - o (4 o - m never has the least magnitude), and 4 m - o is the
// earlier candidate of the two where they tie.
__device__ __forceinline__ void minmod_weights(float Da, float Db, float v, float& p, float& q)
{
    const bool first = fabsf(Da) <= fabsf(Db);
    const float m = first ? Da : Db, o = first ? Db : Da;
    const bool single = v == m && fmaf(4.0f, m, -o) != m;
    const float own = v == 0.0f ? 0.0f : (single ? 1.0f : 4.0f);
    const float other = v == 0.0f || single ? 0.0f : -1.0f;
    p = first ? own : other;
    q = first ? other : own;
}

// Weights W of one interface in a wave some lane of which the limiter bounds
// or clamps, and with MU the derivative dmu (in: that of the unlimited flux).
// fv: the unlimited value (ghat for a comp line); kl, kh: the curvature
// minmods at j-1/2 and j+1/2 of the stencil as it lies.
//
// The median's value X needs three-way minima and maxima only; the candidate
// it came from is read off by equality, which reproduces the tie rules of
// mp_bounded_lin's pairwise selections: X = fhat means the unlimited value
// (first argument of every minimum and maximum it enters), then f_j (first on
// both sides of the bounds), and otherwise the side (f_j, f_{j+1}, f_MD)
// before the side (f_j, f_UL, f_LC), the lower bound before the upper one,
// and within a side the earlier candidate.
//
// The winner's form is, in the frame of its side's four cells (j-1 .. j+2 for
// f_MD's, j-2 .. j+1 for f_LC's), K (p, q-2p, p-2q, q) + (0, b1, b2, 0) with
// p = q = 0 unless a curvature minmod won.
template <int SIDE, bool MU>
__device__ __forceinline__ void bounded_weights(const Stencil& s, const LineShift& sh,
                                                const AdjLine& L, float kl, float kh, bool early,
                                                float fv, float (&W)[5], float& dmu)
{
    const bool comp = SIDE == kPerLane ? sh.comp : SIDE == kComp;
    // stencil of the bounds: mirrored for a comp line
    const float td = comp ? s.b : s.d;
    const float tm1 = comp ? -s.d0 : s.dm1, t0 = comp ? -s.dm1 : s.d0;
    const float al = comp ? sh.alpha_c : sh.alpha;
    const float Mp = comp ? kl : kh, Mm = comp ? kh : kl;
    const float fMD = fmaf(-0.5f, Mp, fmaf(0.5f, t0, s.c));
    const float fUL = fmaf(al, tm1, s.c);
    const float fLC = fmaf(4.0f / 3.0f, Mm, fmaf(0.5f, tm1, s.c));
    const float loA = fminf(fminf(s.c, td), fMD), hiA = fmaxf(fmaxf(s.c, td), fMD);
    const float lo = fmaxf(loA, fminf(fminf(s.c, fUL), fLC));
    const float hi = fminf(hiA, fmaxf(fmaxf(s.c, fUL), fLC));
    const float X = early ? fv : med3(fv, lo, hi);
    const bool un = X == fv;
    const bool isc = X == s.c;
    const bool sideA = (X == lo ? loA : hiA) == X && !isc;
    const bool isd = X == td, isul = X == fUL;
    const bool curved = !isc && !(sideA ? isd : isul);     // f_MD or f_LC
    // the minmod's curvatures: at j and j+1 (f_MD) or j-1 and j (f_LC); a comp
    // line's are the same ones in reverse order (a rounded difference changes
    // sign exactly)
    const float cm = s.dm1 - s.dm2, D0 = s.d0 - s.dm1, cp = s.dp1 - s.d0;
    const float Dm = comp ? cp : cm, Dp = comp ? cm : cp;
    float p, q;
    minmod_weights(sideA ? D0 : Dm, sideA ? Dp : D0, curved ? (sideA ? Mp : Mm) : 0.0f, p, q);
    const float K = sideA ? -0.5f : 4.0f / 3.0f;
    const float b1 = sideA ? (isd ? 0.0f : 0.5f) : (isc ? 0.0f : (isul ? -al : -0.5f));
    const float b2 = sideA ? (isd ? 1.0f : 0.5f) : (isc ? 1.0f : (isul ? al + 1.0f : 1.5f));
    const float g0 = K * p, g1 = K * fmaf(-2.0f, p, q) + b1;
    const float g2 = K * fmaf(-2.0f, q, p) + b2, g3 = K * q;
    const float v[5] = {sideA ? 0.0f : g0, sideA ? g0 : g1, sideA ? g1 : g2, sideA ? g2 : g3,
                        sideA ? g3 : 0.0f};
    const float fac = comp ? sh.muc : sh.mu;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const float o = SIDE == kPerLane ? (comp ? v[4 - i] : v[i]) : v[SIDE == kComp ? 4 - i : i];
        const float w = fac * o;
        // comp: Phi = c - Psi
        W[i] = un ? L.E[i] : (comp ? (i == 2 ? 1.0f - w : -w) : w);
    }
    if (MU) {
        const float r5 = sideA || isc || !isul ? 0.0f : L.a_mu * tm1;
        const float d = comp ? -(sh.muc * r5 - X) : fmaf(sh.mu, r5, X);
        dmu = un ? dmu : d;
    }
    // positivity clamp med3(factor X, 0, c) with the oracle's tie rules
    // (max(min(x, 0), min(max(x, 0), c)), first argument on a tie)
    const float pre = fac * X;
    if (__ballot(!(pre >= 0.0f && pre <= s.c)) != 0) {
        const Pick k = pmed3(Pick{pre, 0}, Pick{0.0f, 1}, Pick{s.c, 2});
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const float u = i == 2 ? 1.0f : 0.0f;
            const float zero = comp ? u : 0.0f, whole = comp ? 0.0f : u;
            W[i] = k.id == 0 ? W[i] : (k.id == 1 ? zero : whole);
        }
        if (MU) dmu = k.id == 0 ? dmu : 0.0f;
    }
}

// One interface: adds psi W[k] to the five rows in acc and, with MU, psi
// dPhi/dmu to lam_mu where `count` says so.  ghost: the upwind cell lies in
// the vacuum outside the line (c = 0).  Its flux is clamped to 0 whatever the
// limiter does, and neither its weights nor its shift derivative reach the
// line unless the value ties with the clamp: an unlimited value of 0, or a
// flux factor so small that the product may be 0.
template <int SIDE, bool MU>
__device__ __forceinline__ void flux_scatter(const Stencil& s, const LineShift& sh,
                                             const AdjLine& L, float kl, float kh, float ps,
                                             float (&acc)[5], bool ghost, bool count, float& lam_mu)
{
    const bool comp = SIDE == kPerLane ? sh.comp : SIDE == kComp;
    float y = sh.v0 * s.dm2;
    y = fmaf(sh.v1, s.dm1, y);
    y = fmaf(sh.v2, s.d0, y);
    y = fmaf(sh.v3, s.dp1, y);
    const float fv = comp ? fmaf(-sh.q, y, s.c) : s.c + y;
    const float fac = comp ? sh.muc : sh.mu;
    if (ghost && __ballot(!(fabsf(fv) > 0.0f && fac > 1e-6f)) == 0) return;
    const float m = med3(s.d0, sh.alpha * s.dm1, 0.0f);
    const bool early = med3(y, 0.0f, m) == y;
    const float pre = fac * fv;
    float dmu = 0.0f;
    if (MU) {
        // d fhat / d mu, or d ghat / d mu of a comp line
        float t = L.ds.d0 * s.a;
        t = fmaf(L.ds.d1, s.b, t);
        t = fmaf(L.ds.d2, s.c, t);
        t = fmaf(L.ds.d3, s.d, t);
        t = fmaf(L.ds.d4, s.e, t);
        const float f5 = comp ? -sh.q * t - L.q_mu * y : t;
        dmu = comp ? -(sh.muc * f5 - fv) : fmaf(sh.mu, f5, fv);
    }
    const bool plain = early && pre >= 0.0f && pre <= s.c;
    if (__ballot(!plain) == 0) {
#pragma unroll
        for (int k = 0; k < 5; ++k) acc[k] = fmaf(ps, L.E[k], acc[k]);
    } else {
        float W[5];
        bounded_weights<SIDE, MU>(s, sh, L, kl, kh, early, fv, W, dmu);
#pragma unroll
        for (int k = 0; k < 5; ++k) acc[k] = fmaf(ps, W[k], acc[k]);
    }
    if (MU && count) lam_mu = fmaf(ps, dmu, lam_mu);
}

// Rows of a line in frame order, `step` bytes apart (negative for a mirrored
// walk): frame row r lies at `p + lane`, with the row pointer uniform over the
// wave where the lanes share the walk, so that a row costs a few scalar
// instructions and one load.  Rows outside [0, M) read zero (vacuum) or wrap
// (PER).
template <bool PER>
struct RowStream {
    const char* p;       // row r of lane offset 0
    unsigned lane;       // byte offset of this lane
    long step;
    int r, M;

    __device__ RowStream(const char* first, unsigned off, long st, int m)
        : p(first), lane(off), step(st), r(0), M(m) {}
    // from row 0 to row q
    __device__ void seek(int q)
    {
        if (PER) {
            q %= M;
            if (q < 0) q += M;
        }
        p += (long)(q - r) * step;
        r = q;
    }
    __device__ float next()
    {
        float x = 0.0f;
        if (PER || (unsigned)r < (unsigned)M) x = *reinterpret_cast<const float*>(p + lane);
        ++r;
        p += step;
        if (PER && r == M) {
            r = 0;
            p -= (long)M * step;
        }
        return x;
    }
};

// The same for a line in LDS.
template <bool PER>
struct LdsStream {
    const float* p;
    int step, r, M;

    __device__ LdsStream(const float* first, int st, int m) : p(first), step(st), r(0), M(m) {}
    __device__ void seek(int q)
    {
        if (PER) {
            q %= M;
            if (q < 0) q += M;
        }
        p += (q - r) * step;
        r = q;
    }
    __device__ float next()
    {
        float x = 0.0f;
        if (PER || (unsigned)r < (unsigned)M) x = *p;
        ++r;
        p += step;
        if (PER && r == M) {
            r = 0;
            p -= M * step;
        }
        return x;
    }
};

// x = forward input, lam = output adjoint, both read in frame order (rx from
// row -4, rl from row N - 2); writes lam_in and returns lam_mu (MU).  The
// walk is rolled in groups of CH interfaces whose rows were requested one
// group earlier, so 2 CH loads are in flight while a group is worked on, at
// any line length.
template <int SIDE, bool MU, bool PER, class R, class Put>
__device__ __forceinline__ float line_adjoint_side(R rx, R rl, Put&& put, int M,
                                                   const LineShift& sh, const AdjLine& L)
{
    constexpr int CH = 4;
    const int N = sh.N;
    float w[5];                          // x_{j-2..j+2}, of j = -2 after the first read
    rx.seek(-4);
#pragma unroll
    for (int q = 1; q < 5; ++q) w[q] = rx.next();
    rl.seek(N - 2);
    float la = rl.next(), lb = rl.next();   // lam_{j+N}, lam_{j+N+1}
    float xn[CH], ln[CH];                // x_{j+2} and lam_{j+N+2} of the group's interfaces
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        xn[q] = rx.next();
        ln[q] = rl.next();
    }
    float acc[5];                        // rows j-2 .. j+2
#pragma unroll
    for (int q = 0; q < 5; ++q) acc[q] = 0.0f;
    float dm2 = 0.0f, dm1 = w[2] - w[1], d0 = w[3] - w[2], dp1 = w[4] - w[3];
    // the newest curvature and its minmod with the one before it, carried from
    // interface to interface: the minmod above one is the minmod below the
    // next (here the curvatures at -3 and -2, around the first interface's
    // lower side)
    float cp = dp1 - d0;
    float kh = curv_minmod(d0 - dm1, cp);
    float lam_mu = 0.0f;
    const int J = M + 4;                 // interfaces j = -2 .. M+1
#pragma unroll 1
    for (int j0 = 0; j0 < J; j0 += CH) {
        float xc[CH], lc[CH];
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            xc[q] = xn[q];
            lc[q] = ln[q];
        }
        if (j0 + CH < J) {
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                xn[q] = rx.next();
                ln[q] = rl.next();
            }
        }
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const int j = j0 + q - 2;
            if (j > M + 1) break;
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = w[k + 1];
            w[4] = xc[q];
            dm2 = dm1; dm1 = d0; d0 = dp1; dp1 = w[4] - w[3];
            const float cn = dp1 - d0;
            const float kl = kh;
            kh = curv_minmod(cp, cn);
            cp = cn;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = acc[k + 1];
            acc[4] = lc[q];
            const float ps = lb - la;
            la = lb;
            lb = lc[q];
            const bool count = !PER || (j >= 0 && j < M);
            const bool ghost = !PER && (j < 0 || j >= M);
            flux_scatter<SIDE, MU>(Stencil{w[0], w[1], w[2], w[3], w[4], dm2, dm1, d0, dp1}, sh, L,
                                   kl, kh, ps, acc, ghost, count, lam_mu);
            if (j >= 2) put(j - 2, acc[0]);
        }
    }
    return lam_mu;
}

// UNI: the line's shift is the same in every lane of the wave (its constants
// are then scalars, and the side of the limiter is one branch per line).
template <bool UNI, bool MU, bool PER, class R, class Put>
__device__ __forceinline__ float line_adjoint(const R& rx, const R& rl, Put&& put, int M,
                                              const LineShift& sh, const AdjLine& L)
{
    if constexpr (UNI) {
        if (sh.comp) return line_adjoint_side<kComp, MU, PER>(rx, rl, put, M, sh, L);
        return line_adjoint_side<kPlain, MU, PER>(rx, rl, put, M, sh, L);
    }
    return line_adjoint_side<kPerLane, MU, PER>(rx, rl, put, M, sh, L);
}

}  // namespace

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_position_tan(const float* __restrict__ f,
                                                      const float* __restrict__ v,
                                                      float* __restrict__ out, PosArgs a)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= a.O * a.I) return;
    const long o = t / a.I, k = t - (t / a.I) * a.I;
    const int jl = (int)(((k % a.Nu) / a.pst) % a.nshift);
    const LineShift sh = split_shift(a.shift[jl], a.M, true);
    const int dir = sh.neg ? -1 : 1;
    const long base = o * (long)a.M * a.I + k;
    Reader32 rx{f + base, nullptr, a.I, 0, a.M, dir, true, 0};
    Reader32 rv{v + base, nullptr, a.I, 0, a.M, dir, true, 0};
    line_tangent(rx, rv, out + base, a.I, a.M, dir, sh, true, 0.0f);
}

// Whether the y adjoint's waves can take one u_y each (k_position_adj's
// permutation); pst = nu_z identifies the y sweep.
__host__ __device__ __forceinline__ bool adj_gathered(const PosArgs& a)
{
    return a.pst == a.nuz && a.nshift > 1 && a.nshift * a.nuz * a.nux == a.Nu && a.nuz <= 64 &&
           64 % a.nuz == 0 && a.nux % (64 / a.nuz) == 0;
}

// UNI: the lanes of every wave share the shift (the launcher checks)
template <bool UNI>
__global__ void __launch_bounds__(256) k_position_adj(const float* __restrict__ f,
                                                      const float* __restrict__ lam,
                                                      float* __restrict__ lam_in, PosArgs a)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= a.O * a.I) return;
    const long o = t / a.I;
    long k = t - o * a.I;
    // y sweeps (the shift follows u_y, pst = nu_z): consecutive lanes would
    // cover 64 / nu_z values of u_y, and a wave would run both sides of every
    // branch on the shift.  Instead each wave takes one u_y: 64 / nu_z whole
    // uz-lines from consecutive u_x rows -- a permutation of k within groups
    // of 64 nu_y elements (64 / nu_z u_x rows), which tile every row
    if (adj_gathered(a)) {
        const long G = 64L * a.nshift;
        const long l = k & 63;
        const long rr = l / a.nuz;
        k = (k / G) * G + (rr * a.nshift + (k % G) / 64) * a.nuz + (l - rr * a.nuz);
    }
    int jl = (int)(((k % a.Nu) / a.pst) % a.nshift);
    if (UNI) jl = uniform_sgpr(jl);
    LineShift sh = split_shift(a.shift[jl], a.M, true);
    AdjLine L = adj_line(sh);
    if constexpr (UNI) {
        sh = uniform_shift(sh);
        L = uniform_adj(L);
    }
    const int dir = sh.neg ? -1 : 1;
    // the wave's first element (lane 0's, its smallest) and this lane's offset
    // from it; without a common walk every lane has its own row pointer
    const long base = o * (long)a.M * a.I + k;
    const long b0 = UNI ? uniform_long(base) : base;
    const unsigned lane = (unsigned)((base - b0) * (long)sizeof(float));
    const long top = dir > 0 ? 0 : (long)(a.M - 1) * a.I;       // frame row 0
    const long step = dir * a.I * (long)sizeof(float);
    const RowStream<true> rx(reinterpret_cast<const char*>(f + b0 + top), lane, step, a.M);
    const RowStream<true> rl(reinterpret_cast<const char*>(lam + b0 + top), lane, step, a.M);
    char* out = reinterpret_cast<char*>(lam_in + b0 + top);
    line_adjoint<UNI, false, true>(rx, rl, [&](int r, float v) {
        *reinterpret_cast<float*>(out + r * step + lane) = v;
    }, a.M, sh, L);
}

// Velocity sweeps: one work-group per spatial cell; lines of the cell are
// (sub, k) with line start ((cell*nsub + sub) * M) * I + k.
__global__ void __launch_bounds__(256) k_velocity_tan(const float* __restrict__ f,
                                                      const float* __restrict__ v,
                                                      float* __restrict__ out,
                                                      const float* __restrict__ g_dot, VelArgs a)
{
    const long cell = blockIdx.x;
    const double s = (double)a.g[cell] * a.factor;
    const LineShift sh = split_shift(s, a.M, a.periodic);
    const int dir = sh.neg ? -1 : 1;
    // d mu / d s = +1 (rightward) or -1 (walked mirrored); s_dot = g_dot dt / du
    const float s_dot = g_dot != nullptr ? (float)((double)g_dot[cell] * a.factor) : 0.0f;
    const float mu_dot = sh.neg ? -s_dot : s_dot;
    const long lpc = a.nsub * a.I;
    for (long l = threadIdx.x; l < lpc; l += blockDim.x) {
        const long sub = l / a.I, k = l - (l / a.I) * a.I;
        const long base = ((cell * a.nsub + sub) * a.M) * a.I + k;
        Reader32 rx{f + base, nullptr, a.I, 0, a.M, dir, a.periodic, 0};
        Reader32 rv{v + base, nullptr, a.I, 0, a.M, dir, a.periodic, 0};
        line_tangent(rx, rv, out + base, a.I, a.M, dir, sh, a.periodic, mu_dot);
    }
}

// Constants of the velocity lines of a work-group's cells, made once per cell
// by one lane each (split_shift and adj_line are about 300 vector
// instructions, a tenth of the work of a 16-cell line if every wave repeats
// them) and read back as scalars.
constexpr int kAdjCells = 8;             // most cells per work-group

struct AdjEntry {
    LineShift sh;
    AdjLine L;
};

// Cells of a work-group: eight, fewer where that would leave CUs idle.
static int adj_cells_per_group(long cells)
{
    const long q = cells / 2048;
    return (int)(q < 1 ? 1 : (q > kAdjCells ? kAdjCells : q));
}

__device__ __forceinline__ void adj_entries(AdjEntry* tab, const VelArgs& a, long cell0, int nc)
{
    if ((int)threadIdx.x < nc) {
        const double s = (double)a.g[cell0 + threadIdx.x] * a.factor;
        tab[threadIdx.x].sh = split_shift(s, a.M, a.periodic);
        tab[threadIdx.x].L = adj_line(tab[threadIdx.x].sh);
    }
    __syncthreads();
}

// FAR: the lines of one wave lie up to 4 GiB apart or more (velocity blocks of
// 2^30 cells), so every lane keeps its own row pointer.
template <bool PER, bool FAR>
__global__ void __launch_bounds__(256) k_velocity_adj(const float* __restrict__ f,
                                                      const float* __restrict__ lam,
                                                      float* __restrict__ lam_in,
                                                      float* __restrict__ lam_g, VelArgs a, int cpg)
{
    __shared__ AdjEntry tab[kAdjCells];
    __shared__ double red[4];
    const long cell0 = (long)blockIdx.x * cpg;
    const int nc = (int)(a.cells - cell0 < cpg ? a.cells - cell0 : cpg);
    adj_entries(tab, a, cell0, nc);
    // within a velocity block, at most 2^31 - 1 (unsigned: a counter passes its
    // bound by up to a work-group)
    const unsigned I = (unsigned)a.I, lpc = (unsigned)(a.nsub * a.I);
    for (int c = 0; c < nc; ++c) {
        const long cell = cell0 + c;
        const LineShift sh = uniform_shift(tab[c].sh);
        const AdjLine L = uniform_adj(tab[c].L);
        const int dir = sh.neg ? -1 : 1;
        double mine = 0.0;
        // frame row 0 of the cell's first line
        const long top = cell * a.nsub * a.M * a.I + (dir > 0 ? 0 : (long)(a.M - 1) * a.I);
        const long step = dir * a.I * (long)sizeof(float);
        for (unsigned l = threadIdx.x; l < lpc; l += blockDim.x) {
            const unsigned sub = l / I, k = l - sub * I;
            const long off = (long)sub * a.M * I + k;
            const long o0 = FAR ? off : uniform_long(off);   // lane 0's line, the wave's first
            const unsigned lane = (unsigned)((off - o0) * (long)sizeof(float));
            const RowStream<PER> rx(reinterpret_cast<const char*>(f + top + o0), lane, step, a.M);
            const RowStream<PER> rl(reinterpret_cast<const char*>(lam + top + o0), lane, step, a.M);
            char* out = reinterpret_cast<char*>(lam_in + top + o0);
            mine += (double)line_adjoint<true, true, PER>(rx, rl, [&](int r, float v) {
                *reinterpret_cast<float*>(out + r * step + lane) = v;
            }, a.M, sh, L);
        }
        if (lam_g != nullptr) {
            const double tot = block_sum(mine, red);
            // lam_s = +lam_mu (rightward) or -lam_mu (mirrored); ds/dg = dt/du
            if (threadIdx.x == 0) lam_g[cell] += (float)((sh.neg ? -tot : tot) * a.factor);
        }
    }
}

// Adjoint of the uz sweep: the lines are contiguous (M values), so a
// work-group stages NT whole lines of f and of lam through LDS with 16-byte
// loads, each thread walks one line out of LDS into a third tile, and the
// results leave with 16-byte stores.  lam_mu is summed per cell as in
// k_velocity_adj (per thread over its lines, then over the work-group).
template <int MT, int NT, bool PER>
__global__ void __launch_bounds__(NT) k_velocity_adj_uz(const float* __restrict__ f,
                                                        const float* __restrict__ lam,
                                                        float* __restrict__ lam_in,
                                                        float* __restrict__ lam_g, VelArgs a, int cpg)
{
    constexpr int LS = MT + 1;                  // padded line stride in LDS
    // a vacuum walk writes row j-2 when it has read past it, so the result may
    // take the input's place; a periodic one reads its first rows again
    __shared__ float tf[NT * LS], tl[NT * LS], per[PER ? NT * LS : 1];
    float* to = PER ? per : tf;
    __shared__ AdjEntry tab[kAdjCells];
    __shared__ double red[NT / 64];
    const long cell0 = (long)blockIdx.x * cpg;
    const int nc = (int)(a.cells - cell0 < cpg ? a.cells - cell0 : cpg);
    adj_entries(tab, a, cell0, nc);
    const long lpc = a.nsub;                    // lines per cell = nux * nuy
    for (int c = 0; c < nc; ++c) {
        const long cell = cell0 + c;
        const LineShift sh = uniform_shift(tab[c].sh);
        const AdjLine L = uniform_adj(tab[c].L);
        const int dir = sh.neg ? -1 : 1;
        const long cbase = cell * lpc;
        double mine = 0.0;
        for (long l0 = 0; l0 < lpc; l0 += NT) {
            const int nl = (int)((lpc - l0) < NT ? (lpc - l0) : NT);
            const long off0 = (cbase + l0) * MT;
            for (int e = threadIdx.x * 4; e < nl * MT; e += NT * 4) {
                const int ln = e / MT;
                const int off = e - ln * MT;
                const float4 x = *reinterpret_cast<const float4*>(f + off0 + e);
                const float4 y = *reinterpret_cast<const float4*>(lam + off0 + e);
                float* df = tf + ln * LS + off;
                float* dl = tl + ln * LS + off;
                df[0] = x.x; df[1] = x.y; df[2] = x.z; df[3] = x.w;
                dl[0] = y.x; dl[1] = y.y; dl[2] = y.z; dl[3] = y.w;
            }
            __syncthreads();
            if (threadIdx.x < nl) {
                const int top = threadIdx.x * LS + (dir > 0 ? 0 : MT - 1);
                const LdsStream<PER> rx(tf + top, dir, MT), rl(tl + top, dir, MT);
                float* out = to + top;
                mine += (double)line_adjoint<true, true, PER>(rx, rl, [&](int r, float v) {
                    out[r * dir] = v;
                }, MT, sh, L);
            }
            __syncthreads();
            for (int e = threadIdx.x * 4; e < nl * MT; e += NT * 4) {
                const int ln = e / MT;
                const int off = e - ln * MT;
                const float* src = to + ln * LS + off;
                *reinterpret_cast<float4*>(lam_in + off0 + e) = make_float4(src[0], src[1], src[2], src[3]);
            }
            __syncthreads();
        }
        if (lam_g != nullptr) {
            const double tot = block_sum(mine, red);
            if (threadIdx.x == 0) lam_g[cell] += (float)((sh.neg ? -tot : tot) * a.factor);
        }
    }
}

hipError_t launch_position_tan(const float* f, const float* v, float* out, const PosArgs& a,
                               hipStream_t st)
{
    const long total = a.O * a.I;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_position_tan, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, f,
                       v, out, a);
    return hipGetLastError();
}

hipError_t launch_position_adj(const float* f, const float* lam, float* lam_in, const PosArgs& a,
                               hipStream_t st)
{
    const long total = a.O * a.I;
    if (total == 0) return hipSuccess;
    const dim3 grid((unsigned)((total + 255) / 256));
    // whole waves of one shift: x sweeps whose u_x rows are whole waves, y
    // sweeps whose waves can be gathered; rows of whole waves, so that none
    // straddles two of them
    const bool uni = a.I % 64 == 0 && (adj_gathered(a) || a.pst % 64 == 0);
    if (uni) hipLaunchKernelGGL(k_position_adj<true>, grid, dim3(256), 0, st, f, lam, lam_in, a);
    else hipLaunchKernelGGL(k_position_adj<false>, grid, dim3(256), 0, st, f, lam, lam_in, a);
    return hipGetLastError();
}

static unsigned vel_block(const VelArgs& a)
{
    long bs = ((a.nsub * a.I + 63) / 64) * 64;
    return (unsigned)(bs > 256 ? 256 : bs);
}

hipError_t launch_velocity_tan(const float* f, const float* v, float* out, const float* g_dot,
                               const VelArgs& a, hipStream_t st)
{
    if (a.cells == 0) return hipSuccess;
    hipLaunchKernelGGL(k_velocity_tan, dim3((unsigned)a.cells), dim3(vel_block(a)), 0, st, f, v,
                       out, g_dot, a);
    return hipGetLastError();
}

hipError_t launch_velocity_adj(const float* f, const float* lam, float* lam_in, float* lam_g,
                               const VelArgs& a, hipStream_t st)
{
    if (a.cells == 0) return hipSuccess;
    // uz (contiguous lines of 16, 32 or 64 values, 16-byte aligned cells):
    // LDS tiles of 4096 values per array
    const bool al = ((uintptr_t)f | (uintptr_t)lam | (uintptr_t)lam_in) % 16 == 0;
    const int cpg = adj_cells_per_group(a.cells);
    const dim3 grid((unsigned)((a.cells + cpg - 1) / cpg));
    if (a.I == 1 && al) {
#define VL_UZ(MTV, NTV)                                                                          \
    if (a.periodic)                                                                             \
        hipLaunchKernelGGL((k_velocity_adj_uz<MTV, NTV, true>), grid, dim3(NTV), 0, st, f, lam,   \
                           lam_in, lam_g, a, cpg);                                              \
    else                                                                                        \
        hipLaunchKernelGGL((k_velocity_adj_uz<MTV, NTV, false>), grid, dim3(NTV), 0, st, f, lam,  \
                           lam_in, lam_g, a, cpg);                                              \
    return hipGetLastError()
        switch (a.M) {
            case 16: VL_UZ(16, 256);
            case 32: VL_UZ(32, 128);
            case 64: VL_UZ(64, 64);
            default: break;
        }
#undef VL_UZ
    }
    // a wave's lines lie within M (64 + I) elements
    const bool far = (double)a.M * (64.0 + (double)a.I) >= 1073741824.0;
    auto kern = a.periodic ? (far ? k_velocity_adj<true, true> : k_velocity_adj<true, false>)
                           : (far ? k_velocity_adj<false, true> : k_velocity_adj<false, false>);
    hipLaunchKernelGGL(kern, grid, dim3(vel_block(a)), 0, st, f, lam, lam_in, lam_g, a, cpg);
    return hipGetLastError();
}

}  // namespace vlasov
