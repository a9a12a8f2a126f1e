// Butterfly factorization of a 2D discrete FIO on gfx950 (Section 2.2 on a
// quadtree, the phases of Sections 5.2 and 5.3), for the levels where the outermost factors
// meet at the middle level (L' = h, no B or C factor): K~ = U M V.
//
// Trees: n = 2^L points per dimension, N = n^2, h = ceil(L/2), lc = L - h.
//   V side: pairs (tau' at spatial level lc, sigma at frequency level h),
//           pair index tau' * 4^h + sigma;
//   U side: pairs (tau at spatial level h, sigma' at frequency level lc),
//           pair index tau * 4^lc + sigma';
//   M couples U pair (tau, sigma') with the V pairs (parent^(h-lc)(tau), sigma)
//   for the rr = 4^(h-lc) frequency boxes sigma of level h inside sigma'.
// Box indices are Morton codes of the box coordinates (first coordinate on the
// odd bits), so the points of a box are contiguous in Morton order and the
// children of box v are 4v .. 4v+3.
//
// Factor layout (complex entries, column-major blocks; the import/export layout):
//   V: block p (V pair), q^2 x b^2, entry (i, s) at p q^2 b^2 + s q^2 + i
//   M: block u * 4^h + sigma (u, sigma at level h), q^2 x q^2, entry (i, j) at
//      blk q^4 + j q^2 + i
//   U: block p (U pair), b^2 x q^2, entry (s, i) at p q^2 b^2 + i b^2 + s
// with s the Morton index of a point inside its box and i = i1 q + i2 the
// tensor Chebyshev index.  The adjoint applies read conjugate-transposed copies
// (built on the device from the forward factors) so that every step streams its
// factor with consecutive lanes on consecutive rows:
//   Vadj block sigma * 4^lc + tau' = V_{tau',sigma}^*  (b^2 x q^2)
//   Madj block (tau' * 4^h + sigma) * rr + d = M_{tau' rr + d, sigma}^*  (q^2 x q^2)
//   Uadj block p = U_p^*  (q^2 x b^2)
//
// Apply: one kernel per factor (k2_mm).  A wave owns up to 6 x 16 rows of one output block (a pair's
// q^2 coefficients, or a leaf box's b^2 values) for 8 or 16 right-hand sides and runs the products on the
// matrix cores.  The leaf-box sums over 4^lc blocks are split over waves and reduced in a fixed
// order; every column is summed in the same order at any width and split of rows (deterministic
// results).  Few columns: the factor stream bounds it (n = 128, 8 columns: 9.6 GB in 1.83 ms, 5.2 TB/s; one
// lane per row took 1.89 ms, no more than runs differ by).  Many columns: the FP64 matrix rate (n = 64, 144 columns: 46 of 75
// TFLOP/s with the 81 rows padded to 96; one lane per row reached 24).  In between the launches of few, long waves: n = 8
// 105 -> 27 us, n = 16 80 -> 26 us at 8 columns.
//
// Coefficient buffers: entry (pair p, coefficient i, column c) at (p q^2 + i) * ldc + c with ldc = nrhs
// rounded up to the columns of a wave; the adjoint steps store their pairs in the order in which
// the next step sums them.
#include <cmath>

#include "bf.h"
#include "ddmath.h"
#include "mat4.h"
#include "timing.h"

namespace fio {

namespace {

struct G2 {
    int n, L, h, lc, b, hb, q, q2, b2;
    long S, T, rr;                // 4^h, 4^lc, 4^(h-lc)
    double a0, a1;                // phase parameters
    int iso;                      // Section 5.3's isotropic phase (c2 = c1)
    int hankel;                   // Section 5.3's amplitude
};

G2 g2_of(const fio_bf_s *bf) {
    G2 g;
    g.n = (int)bf->n1;
    g.L = bf->L;
    g.h = bf->h;
    g.lc = bf->lc;
    g.b = bf->b;
    g.hb = bf->hb;
    g.q = bf->q;
    g.q2 = bf->q * bf->q;
    g.b2 = bf->b * bf->b;
    g.S = 1L << (2 * bf->h);
    g.T = 1L << (2 * bf->lc);
    g.rr = g.S / g.T;
    g.a0 = bf->desc.c0;
    g.a1 = bf->desc.c1;
    g.iso = bf->desc.phase_kind == FIO_PHASE2_ISO;
    g.hankel = bf->desc.amp_kind == FIO_AMP_HANKEL;
    return g;
}

// --- geometry and phase (Sections 5.2 and 5.3) ---------------------------------------------
__device__ __forceinline__ void demorton(long m, int bits, int &j1, int &j2) {
    j1 = 0;
    j2 = 0;
    for (int k = 0; k < bits; ++k) {
        j1 |= (int)((m >> (2 * k + 1)) & 1) << k;
        j2 |= (int)((m >> (2 * k)) & 1) << k;
    }
}

// user (lexicographic) index of the point with Morton code m
__device__ __forceinline__ long lex_of(long m, int L, int n) {
    int j1, j2;
    demorton(m, L, j1, j2);
    return (long)j1 * n + j2;
}

// Phases are formed in double-double arithmetic from exact points (ddmath.h; box corners and
// grid points are binary fractions or integers, Chebyshev points are center + (w/2) t_i) and
// reduced modulo 1 before the single rounding of an entry; Lagrange values are taken in the
// reference coordinate of the point in its box, which is the same for every box: lag[s][i] = q_i(point s
// of the b on a side).
__global__ void gen2_lagrange(Nodes tn, int b, double *lag) {
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= b * tn.q) return;
    const double hw = 0.5 * b;
    lag[id] = dd_lagrange(dd_of((id / tn.q - hw) / hw), id % tn.q, tn);
}

__device__ dd rho2_dd(const G2 &g, dd x1, dd x2, dd k1, dd k2) {
    dd s1, co1, s2, co2;
    dd_sincospi(dd_ldexp(x1, 2.0), s1, co1);
    dd_sincospi(dd_ldexp(x2, 2.0), s2, co2);
    const dd c1 = dd_add(dd_of(g.a0), dd_mul_d(dd_mul(s1, s2), g.a1));
    const dd c2 = g.iso ? c1 : dd_add(dd_of(g.a0), dd_mul_d(dd_mul(co1, co2), g.a1));
    const dd t1 = dd_mul(c1, k1), t2 = dd_mul(c2, k2);
    return dd_sqrt(dd_add(dd_mul(t1, t1), dd_mul(t2, t2)));
}

// box geometry: spatial box j at level l is [j1 2^-l, (j1 + 1) 2^-l] x [..];
// frequency box j at level l is [-n/2 + j1 n 2^-l, ..] x [..]
__device__ __forceinline__ void s_box(int l, long box, double &lo1, double &lo2, double &w) {
    int j1, j2;
    demorton(box, l, j1, j2);
    w = ldexp(1.0, -l);
    lo1 = j1 * w;
    lo2 = j2 * w;
}

__device__ __forceinline__ void f_box(const G2 &g, int l, long box, double &lo1, double &lo2, double &w) {
    int j1, j2;
    demorton(box, l, j1, j2);
    w = ldexp((double)g.n, -l);
    lo1 = -0.5 * g.n + j1 * w;
    lo2 = -0.5 * g.n + j2 * w;
}

// --- factor generation ------------------------------------------------------------
// V(i, s) of pair p = tau' * S + sigma:
//   exp(2 pi i (y.(xi_s - gamma_i) + rho(y, xi_s) - rho(y, gamma_i))) q_i(xi_s)
__global__ void gen2_V(G2 g, Nodes tn, const double *lag, double2 *out) {
    const size_t nV = (size_t)g.T * g.S * g.q2 * g.b2;
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= nV) return;
    const int i = (int)(id % g.q2);
    const int s = (int)((id / g.q2) % g.b2);
    const long p = (long)(id / ((size_t)g.q2 * g.b2));
    const long tau = p / g.S, sigma = p % g.S;
    double y1, y2, ws, f1, f2, wf;
    s_box(g.lc, tau, y1, y2, ws);
    y1 += 0.5 * ws;
    y2 += 0.5 * ws;
    f_box(g, g.h, sigma, f1, f2, wf);
    int a1, a2;
    demorton(s, g.hb, a1, a2);
    const double k1 = f1 + a1, k2 = f2 + a2;                   // xi_s (integers)
    const int i1 = i / g.q, i2 = i % g.q;
    const double c1 = f1 + 0.5 * wf, c2 = f2 + 0.5 * wf, hw = 0.5 * wf;
    const dd g1 = dd_add(dd_of(c1), dd_ldexp(tn.t(i1), hw)), g2 = dd_add(dd_of(c2), dd_ldexp(tn.t(i2), hw));
    const dd lin = dd_add(dd_frac(dd_mul_d(dd_sub(dd_of(k1), g1), y1)), dd_frac(dd_mul_d(dd_sub(dd_of(k2), g2), y2)));
    const dd nl = dd_sub(rho2_dd(g, dd_of(y1), dd_of(y2), dd_of(k1), dd_of(k2)), rho2_dd(g, dd_of(y1), dd_of(y2), g1, g2));
    const double w = lag[a1 * g.q + i1] * lag[a2 * g.q + i2];
    const double2 e = dd_expi2pi(dd_add(lin, dd_frac(nl)));
    out[id] = zc(e.x * w, e.y * w);
}

// M(i, j) of block u * S + sigma: k(z_u,i, gamma_sigma,j)
__global__ void gen2_M(G2 g, Nodes tn, double2 *out) {
    const size_t nM = (size_t)g.S * g.S * g.q2 * g.q2;
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= nM) return;
    const int i = (int)(id % g.q2);
    const int j = (int)((id / g.q2) % g.q2);
    const long blk = (long)(id / ((size_t)g.q2 * g.q2));
    const long u = blk / g.S, sigma = blk % g.S;
    double z1, z2, ws, f1, f2, wf;
    s_box(g.h, u, z1, z2, ws);
    f_box(g, g.h, sigma, f1, f2, wf);
    const double hs = 0.5 * ws, hf = 0.5 * wf;
    const dd x1 = dd_add(dd_of(z1 + hs), dd_ldexp(tn.t(i / g.q), hs));
    const dd x2 = dd_add(dd_of(z2 + hs), dd_ldexp(tn.t(i % g.q), hs));
    const dd k1 = dd_add(dd_of(f1 + hf), dd_ldexp(tn.t(j / g.q), hf));
    const dd k2 = dd_add(dd_of(f2 + hf), dd_ldexp(tn.t(j % g.q), hf));
    const dd r = rho2_dd(g, x1, x2, k1, k2);
    const dd lin = dd_add(dd_frac(dd_mul(x1, k1)), dd_frac(dd_mul(x2, k2)));
    const double2 e = dd_expi2pi(dd_add(lin, dd_frac(r)));
    if (!g.hankel) {
        out[id] = e;
        return;
    }
    // a = H0^(1)(t) exp(-i t), t = 2 pi rho (H0^(1) = J0 + i Y0): a is smooth in t, so t is taken
    // rounded once; the oscillation of H0^(1) cancels against exp(-i t) at the same t.
    // Chebyshev points never fall on xi = 0, so rho > 0 here.
    const double t = 2.0 * M_PI * dd_val(r);
    double st, ct;
    sincos(t, &st, &ct);
    const double jr = j0(t), yi = y0(t);
    const double ar = jr * ct + yi * st, ai = yi * ct - jr * st;    // (J0 + i Y0)(cos t - i sin t)
    out[id] = zc(ar * e.x - ai * e.y, ar * e.y + ai * e.x);
}

// U(s, i) of pair p = tau * T + sigma':
//   exp(2 pi i ((x_s - z_i).eta + rho(x_s, eta) - rho(z_i, eta))) p_i(x_s)
__global__ void gen2_U(G2 g, Nodes tn, const double *lag, double2 *out) {
    const size_t nU = (size_t)g.S * g.T * g.q2 * g.b2;
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= nU) return;
    const int s = (int)(id % g.b2);
    const int i = (int)((id / g.b2) % g.q2);
    const long p = (long)(id / ((size_t)g.q2 * g.b2));
    const long tau = p / g.T, sig = p % g.T;
    double t1, t2, ws, e1, e2, wf;
    s_box(g.h, tau, t1, t2, ws);
    f_box(g, g.lc, sig, e1, e2, wf);
    e1 += 0.5 * wf;
    e2 += 0.5 * wf;                                            // eta_sigma'
    int a1, a2;
    demorton(s, g.hb, a1, a2);
    const double hs = 0.5 * ws, c1 = t1 + hs, c2 = t2 + hs;
    const double x1 = t1 + a1 * (1.0 / g.n), x2 = t2 + a2 * (1.0 / g.n);   // grid points, exact
    const int i1 = i / g.q, i2 = i % g.q;
    const dd z1 = dd_add(dd_of(c1), dd_ldexp(tn.t(i1), hs)), z2 = dd_add(dd_of(c2), dd_ldexp(tn.t(i2), hs));
    const dd lin = dd_add(dd_frac(dd_mul_d(dd_sub(dd_of(x1), z1), e1)), dd_frac(dd_mul_d(dd_sub(dd_of(x2), z2), e2)));
    const dd nl = dd_sub(rho2_dd(g, dd_of(x1), dd_of(x2), dd_of(e1), dd_of(e2)), rho2_dd(g, z1, z2, dd_of(e1), dd_of(e2)));
    const double w = lag[a1 * g.q + i1] * lag[a2 * g.q + i2];
    const double2 e = dd_expi2pi(dd_add(lin, dd_frac(nl)));
    out[id] = zc(e.x * w, e.y * w);
}

// conjugate-transposed copies of the three factors (layout in the file header)
__global__ void adj2_V(G2 g, const double2 *V, double2 *Va) {
    const size_t nV = (size_t)g.T * g.S * g.q2 * g.b2;
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= nV) return;
    // destination order: block sigma * T + tau, entry (s, i) at i b2 + s
    const int s = (int)(id % g.b2);
    const int i = (int)((id / g.b2) % g.q2);
    const long blk = (long)(id / ((size_t)g.q2 * g.b2));
    const long sigma = blk / g.T, tau = blk % g.T;
    const double2 v = V[((size_t)(tau * g.S + sigma) * g.b2 + s) * g.q2 + i];
    Va[id] = zc(v.x, -v.y);
}

__global__ void adj2_M(G2 g, const double2 *M, double2 *Ma) {
    const size_t nM = (size_t)g.S * g.S * g.q2 * g.q2;
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= nM) return;
    // destination block (tau' * S + sigma) * rr + d holds M_{tau' rr + d, sigma}^*: entry (j, i) at i q2 + j
    const int j = (int)(id % g.q2);
    const int i = (int)((id / g.q2) % g.q2);
    const long blk = (long)(id / ((size_t)g.q2 * g.q2));
    const long d = blk % g.rr, p = blk / g.rr;
    const long taup = p / g.S, sigma = p % g.S;
    const long u = taup * g.rr + d;
    const double2 v = M[((size_t)(u * g.S + sigma) * g.q2 + j) * g.q2 + i];
    Ma[id] = zc(v.x, -v.y);
}

__global__ void adj2_U(G2 g, const double2 *U, double2 *Ua) {
    const size_t nU = (size_t)g.S * g.T * g.q2 * g.b2;
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= nU) return;
    // destination: block p, entry (i, s) at s q2 + i
    const int i = (int)(id % g.q2);
    const int s = (int)((id / g.q2) % g.b2);
    const long p = (long)(id / ((size_t)g.q2 * g.b2));
    const double2 v = U[((size_t)p * g.q2 + i) * g.b2 + s];
    Ua[id] = zc(v.x, -v.y);
}

__global__ void cvt2_f32(const double2 *in, float2 *out, size_t n) {
    size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id < n) {
        double2 v = in[id];
        out[id] = make_float2((float)v.x, (float)v.y);
    }
}

// --- apply -------------------------------------------------------------------------
enum Step { VF, MF, UF, UA, MA, VA };

template <typename T> struct K2Args {
    G2 g;
    const cpx<T> *A;        // factor blocks of this step
    const cpx<T> *cin;      // input coefficients (MF, UF, MA, VA)
    const double2 *X;       // input vector (VF: frequency side, UA: spatial side)
    long ldx;
    cpx<T> *cout;           // output coefficients (VF, MF, UA, MA) or partial sums (UF, VA, nsplit > 1)
    double2 *Y;             // output vector (UF: spatial side, VA: frequency side), when nsplit == 1
    long ldy;
    int nrhs, ldc;          // right-hand sides, coefficient row stride
    int nb, nsplit;         // blocks per output, splits of the block range
    int fint;               // frequency-side vectors in Morton order (no index map)
    int step, rows, cols;   // the Step, rows and columns of a factor block
    int rgroups, cgroups;   // row and column groups (waves) of an output
    unsigned nwave;         // waves of the launch: output blocks x splits x groups
};

__device__ __forceinline__ double2 to_z(double2 v) { return v; }
__device__ __forceinline__ double2 to_z(float2 v) { return zc(v.x, v.y); }

// One step of an apply: each wave forms NR x 16 rows of an output block for 8 NC right-hand sides on
// the matrix cores.  The real and imaginary parts of 8 columns are the 16 columns of one real tile, so that
// A_r X and A_i X are two products, combined once at the end, and a block of 8 columns wastes
// nothing.  The blocks of one output and the coefficients they act on are consecutive in memory, so the
// product runs over all their columns as one inner dimension, 4 at a time; entries go straight from
// memory to registers, D steps ahead, at a wave-uniform address plus a lane offset that does not change.
// The bound on waves per SIMD keeps the accumulators in the same 96 registers as the rest for 3 row tiles (5
// waves; 4 without it: n = 64, 70 columns 1040 -> 1002 us).
template <typename T, int NR, int NC, bool VEC, int D>
__global__ void __launch_bounds__(256, NR * NC <= 3 ? 5 : NR * NC == 4 ? 4 : 2) k2_mm(K2Args<T> a) {
    using C = cpx<T>;
    using M = Mat4<T>;
    using V = typename M::V;
    const G2 &g = a.g;
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    // consecutive workgroups run on one XCD, whose L2 then serves the column groups of an output
    const unsigned wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const unsigned W = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (W >= a.nwave) return;
    const unsigned tiles = a.rgroups * a.cgroups;
    const int os = (int)(W / tiles), tile = (int)(W - os * tiles), o = os / a.nsplit, split = os - o * a.nsplit;
    const int lS = 2 * g.h, lT = 2 * g.lc, S = 1 << lS, TT = 1 << lT, lrr = lS - lT;   // S, T and rr = S / T
    const int rg = tile / a.cgroups, c0 = (tile - rg * a.cgroups) * 8 * NC, r0 = rg * 16 * NR;
    const int R = a.rows, nbs = a.nb / a.nsplit, K = nbs * a.cols, nfull = K >> 2, rem = K & 3;
    // factor entries: rows beyond the block repeat its last one and are not stored
    const char *pa = reinterpret_cast<const char *>(a.A + ((size_t)o * a.nb + (size_t)split * nbs) * R * a.cols);
    const int astep = 4 * R * (int)sizeof(C);
    unsigned va[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        const int r = r0 + 16 * t + lr;
        va[t] = (unsigned)(lk * R + (r < R ? r : R - 1)) * (unsigned)sizeof(C);
    }
    // inputs: the points of one leaf box (VEC) or the coefficients of the output's partner pairs
    const char *pb;
    unsigned bstep = 0;
    size_t vb[NC];
    bool inner = false;
    if (VEC) {
        const int box = a.step == VF ? o & (S - 1) : o >> lT;
        inner = a.step == VF && a.fint;
        pb = reinterpret_cast<const char *>(a.X + (inner ? (long)box * g.b2 : lex_of((long)box * g.b2, g.L, g.n)));
        // the lane's point among 4: Morton bits 1 and 0
        const long pt = inner ? lk : (long)(lk >> 1) * g.n + (lk & 1);
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int c = c0 + 8 * u + (lr & 7);
            vb[u] = (pt + (size_t)(c < a.nrhs ? c : a.nrhs - 1) * a.ldx) * sizeof(double2) + (lr >> 3) * sizeof(double);
        }
    } else {
        int pair = split * nbs;                // the first partner pair, as stored (see the end), or leaf box
        if (a.step == VF)
            pair = o & (S - 1);
        else if (a.step == UA)
            pair = o >> lT;
        else if (a.step == MF)
            pair += ((o >> lS) << lS) + ((o & (TT - 1)) << lrr);
        else if (a.step == MA)
            pair += (((o >> lS) << lT) + ((o & (S - 1)) >> lrr)) << lrr;
        else
            pair += o << lT;
        pb = reinterpret_cast<const char *>(a.cin + (size_t)pair * a.cols * a.ldc + c0);
        bstep = 4 * a.ldc * (unsigned)sizeof(C);
#pragma unroll
        for (int u = 0; u < NC; ++u)
            vb[u] = (unsigned)((lk * a.ldc + 8 * u + (lr & 7)) * sizeof(C) + (lr >> 3) * sizeof(T));
    }
    // offset of the inputs of step k (wave-uniform)
    auto boff = [&](int k) -> size_t {
        if (!VEC) return (size_t)k * bstep;
        if (inner) return (size_t)k * 4 * sizeof(double2);
        const int j1 = ((k >> 1) & 1) | ((k >> 2) & 2), j2 = (k & 1) | ((k >> 1) & 2);   // hb <= 3
        return ((size_t)2 * j1 * g.n + 2 * j2) * sizeof(double2);
    };
    auto bval = [&](const char *p) -> T {
        if (VEC) return (T) * reinterpret_cast<const double *>(p);
        return *reinterpret_cast<const T *>(p);
    };
    C fa[D][NR], ta[NR];
    T fb[D][NC], tb[NC];
    auto load = [&](C(&xa)[NR], T(&xb)[NC], int k) {
        const char *qa = pa + (size_t)k * astep, *qb = pb + boff(k);
#pragma unroll
        for (int t = 0; t < NR; ++t) xa[t] = *reinterpret_cast<const C *>(qa + va[t]);
#pragma unroll
        for (int u = 0; u < NC; ++u) xb[u] = bval(qb + vb[u]);
    };
    V P[NR][NC], Q[NR][NC];
#pragma unroll
    for (int t = 0; t < NR; ++t)
#pragma unroll
        for (int u = 0; u < NC; ++u) P[t][u] = Q[t][u] = V{0, 0, 0, 0};
    auto mac = [&](const C(&xa)[NR], const T(&xb)[NC]) {
#pragma unroll
        for (int t = 0; t < NR; ++t)
#pragma unroll
            for (int u = 0; u < NC; ++u) {
                P[t][u] = M::mac(xa[t].x, xb[u], P[t][u]);
                Q[t][u] = M::mac(xa[t].y, xb[u], Q[t][u]);
            }
    };
    if (!VEC && rem) {
        // the K mod 4 last columns first: lanes beyond them read the first of these and count zero (a leaf box
        // has a multiple of 4 points)
        const bool in = lk < rem;
        const char *qa = pa + (size_t)nfull * astep - (in ? 0 : (size_t)lk * R * sizeof(C));
        const char *qb = pb + boff(nfull);
        if (!in) qb -= (size_t)lk * a.ldc * sizeof(C);
#pragma unroll
        for (int t = 0; t < NR; ++t) {
            ta[t] = *reinterpret_cast<const C *>(qa + va[t]);
            if (!in) ta[t] = czero<C>();
        }
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            tb[u] = bval(qb + vb[u]);
            if (!in) tb[u] = T(0);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < nfull) load(fa[d], fb[d], d);
    if (!VEC && rem) mac(ta, tb);
    int k = 0;
    for (; k + D <= nfull; k += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            mac(fa[d], fb[d]);
            if (k + d + D < nfull) load(fa[d], fb[d], k + d + D);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (k + d < nfull) mac(fa[d], fb[d]);
    // lanes of columns 0 .. 7 hold A_r X_r and A_i X_r, the others A_r X_i and A_i X_i
    const bool im = lr >= 8;
    // where the pair is stored: in the order in which the next step reads
    int at = os;
    if (a.step == UA)
        at = ((((o >> lT) >> lrr << lT) + (o & (TT - 1))) << lrr) + ((o >> lT) & ((1 << lrr) - 1));
    else if (a.step == MA)
        at = ((o & (S - 1)) << lT) + (o >> lS);
    C *out = a.cout ? a.cout + (size_t)at * R * a.ldc + c0 : nullptr;
    const long ybase = (a.step == VA && a.fint) ? (long)o * g.b2 : lex_of((long)o * g.b2, g.L, g.n);
#pragma unroll
    for (int t = 0; t < NR; ++t)
#pragma unroll
        for (int u = 0; u < NC; ++u)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                // a lane gets the entry of row i, the lane 8 on that of row i + 2
                const T tp = row_half(im ? P[t][u][i] : P[t][u][i + 2]), tq = row_half(im ? Q[t][u][i] : Q[t][u][i + 2]);
                C v;
                v.x = im ? tp - Q[t][u][i + 2] : P[t][u][i] - tq;
                v.y = im ? P[t][u][i + 2] + tq : tp + Q[t][u][i];
                const int r = r0 + 16 * t + M::row(lane, i) + (im ? M::row(0, 2) : 0), c = 8 * u + (lr & 7);
                if (r >= R) continue;
                if (out) {
                    out[(unsigned)(r * a.ldc + c)] = v;
                } else if (c0 + c < a.nrhs) {
                    int j1, j2;
                    demorton(r, g.hb, j1, j2);
                    const long row = ybase + ((a.step == VA && a.fint) ? r : (long)j1 * g.n + j2);
                    a.Y[row + (size_t)(c0 + c) * a.ldy] = to_z(v);
                }
            }
}

// P(m, c) = X(point m, c): an input block in internal point order, columns fastest, padded to ldc
template <typename T>
__global__ void k2_pack(G2 g, const double2 *X, long ldx, int nrhs, int ldc, int inner, cpx<T> *P) {
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= (size_t)g.S * g.b2 * ldc) return;
    const int c = (int)(id % ldc);
    const long m = (long)(id / ldc);
    const double2 x = X[(inner ? m : lex_of(m, g.L, g.n)) + (size_t)(c < nrhs ? c : nrhs - 1) * ldx];
    cpx<T> v;
    v.x = (T)x.x;
    v.y = (T)x.y;
    P[id] = v;
}

// fixed-order sum of the split partials, scattered to the user vector
template <typename T>
__global__ void k2_reduce(G2 g, const cpx<T> *part, int nsplit, int ldc, int nrhs, int frequency, int fint, double2 *Y, long ldy) {
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const size_t tot = (size_t)g.S * g.b2 * nrhs;
    if (id >= tot) return;
    const int c = (int)(id % nrhs);
    const long m = (long)(id / nrhs);               // o * b2 + r
    const cpx<T> *p = part + ((size_t)(m / g.b2) * nsplit * g.b2 + m % g.b2) * ldc + c;
    cpx<T> s = czero<cpx<T>>();
    for (int k = 0; k < nsplit; ++k) s = cadd(s, p[(size_t)k * g.b2 * ldc]);
    const long row = (frequency && fint) ? m : lex_of(m, g.L, g.n);
    Y[row + (size_t)c * ldy] = to_z(s);
}

__global__ void k_perm2(int n, int L, int to_int, const double2 *X, long ldx, double2 *Y, long ldy, int nrhs) {
    const size_t N = (size_t)n * n;
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= N * nrhs) return;
    const long m = (long)(id % N);
    const size_t c = id / N;
    const long l = lex_of(m, L, n);
    if (to_int)
        Y[m + c * ldy] = X[l + c * ldx];
    else
        Y[l + c * ldy] = X[m + c * ldx];
}


int nsplit_of(long nb) { return (int)(nb < 16 ? nb : 16); }

constexpr long kFewWaves = 2048;

template <typename T, int NR, int NC, bool VEC, int D> void launch_mm(K2Args<T> &a, long nout, hipStream_t s) {
    const int nrt = (a.rows + 15) / 16;
    a.rgroups = (nrt + NR - 1) / NR;
    const long nwave = nout * a.nsplit * a.rgroups * a.cgroups, wgs = (nwave + 3) / 4;
    if (nwave > (1L << 31)) throw Err{FIO_ERR_UNSUPPORTED};
    a.nwave = (unsigned)nwave;
    k2_mm<T, NR, NC, VEC, D><<<dim3((unsigned)((wgs + 7) / 8 * 8)), 256, 0, s>>>(a);
}

// Rows per wave.  At most 4 tiles (2 waves per SIMD hide little, fewer rows read the inputs more often), in the
// fewest equal groups; fewer when that leaves the card without 2 waves per SIMD (n = 16, 8 columns: 40.0 us
// with 3 tiles, 28.8 us with 1 or 2, which also look 4 steps ahead); the 6 tiles of q = 9 in one wave when
// a single column group streams the factors (n = 128, 8 columns: 2006 us with 3 + 3 tiles, 1900 us).
template <typename T, int NC, bool VEC> void run_step(K2Args<T> &a, long nout, hipStream_t s) {
    a.cgroups = a.ldc / (8 * NC);
    const int nrt = (a.rows + 15) / 16, groups = (nrt + 3) / 4, nr = (nrt + groups - 1) / groups;
    const long waves = nout * a.nsplit * a.cgroups;            // per row group
    if constexpr (sizeof(T) == 4 && NC == 2) {
        if (nrt == 7 && waves >= kFewWaves) return launch_mm<T, 7, NC, VEC, 1>(a, nout, s);
        if (nrt == 8 && waves >= kFewWaves) return launch_mm<T, 8, NC, VEC, 1>(a, nout, s);
    }
    if (nr == 1 || waves * ((nrt + 1) / 2) < kFewWaves)
        launch_mm<T, 1, NC, VEC, 4>(a, nout, s);
    else if (nr == 2 || waves * groups < kFewWaves)
        launch_mm<T, 2, NC, VEC, 4>(a, nout, s);
    else if (NC == 1 && (nrt == 5 || nrt == 6) && a.cgroups == 1 && waves >= 4 * kFewWaves)
        launch_mm<T, 6, 1, VEC, 2>(a, nout, s);
    else if (nr == 3)
        launch_mm<T, 3, NC, VEC, 2>(a, nout, s);
    else
        launch_mm<T, 4, NC, VEC, 2>(a, nout, s);
}

// NC x 8 columns per wave
template <typename T, int NC>
void apply2k(fio_bf_s *bf, bool adj, const double2 *X, long ldx, double2 *Y, long ldy, int nrhs, const cpx<T> *F,
             const cpx<T> *Fa, void *ws, bool fint, int nsplit, hipStream_t s) {
    using C = cpx<T>;
    const G2 g = g2_of(bf);
    constexpr int KC = 8 * NC;
    const int ldc = (nrhs + KC - 1) / KC * KC;
    const size_t ncoef = (size_t)bf->N * g.q2 * ldc;
    C *c1 = reinterpret_cast<C *>(ws);
    C *c2 = c1 + ncoef;
    C *part = c2 + ncoef;
    const bool f64 = sizeof(T) == 8;
    const long NP = bf->N;                            // pairs on either side
    // reduction split of the U / V^* steps: a power of two dividing the T partner blocks, at most
    // nsplit_of(T) (the workspace holds that many partial sums)
    int nsp = nsplit_of(g.T);
    if (nsplit > 0 && nsplit < nsp && g.T % nsplit == 0) nsp = nsplit;
    K2Args<T> a{};
    a.g = g;
    a.nrhs = nrhs;
    a.ldc = ldc;
    a.fint = fint ? 1 : 0;
    a.X = X;
    a.ldx = ldx;
    a.Y = Y;
    a.ldy = ldy;
    // leaf-input, middle and leaf-output step of the direction
    auto first = [&](int step, const C *A, C *out, C *spare) {
        K2Args<T> v = a;
        v.step = step; v.A = A; v.cin = spare; v.cout = out; v.nb = 1; v.nsplit = 1; v.rows = g.q2; v.cols = g.b2;
        // the columns of a user vector are gathered once into rows when 64 or more outputs read a box (n = 64:
        // 70 columns 1087 -> 1031 us, 8 columns 267 -> 263 us; n = 32, 16 partners: 8 columns 117 -> 120 us)
        if (nrhs < 8 || g.T < 64) {
            run_step<T, NC, true>(v, NP, s);
        } else {
            k2_pack<T><<<grid1d((size_t)bf->N * ldc, 256), 256, 0, s>>>(g, X, ldx, nrhs, ldc, step == VF && fint, spare);
            run_step<T, NC, false>(v, NP, s);
        }
    };
    auto middle = [&](int step, const C *A, const C *in, C *out) {
        K2Args<T> v = a;
        v.step = step; v.A = A; v.cin = in; v.cout = out; v.nb = (int)g.rr; v.nsplit = 1; v.rows = v.cols = g.q2;
        run_step<T, NC, false>(v, NP, s);
    };
    auto last = [&](int step, const C *A, const C *in) {
        K2Args<T> v = a;
        v.step = step; v.A = A; v.cin = in; v.cout = nsp > 1 ? part : nullptr; v.nb = (int)g.T; v.nsplit = nsp;
        v.rows = g.b2; v.cols = g.q2;
        run_step<T, NC, false>(v, g.S, s);
        if (nsp > 1)
            k2_reduce<T><<<grid1d((size_t)g.S * g.b2 * nrhs, 256), 256, 0, s>>>(g, part, nsp, ldc, nrhs, step == VA,
                                                                              a.fint, Y, ldy);
    };
    if (!adj) {
        const C *V = F + bf->offV, *M = F + bf->offM, *U = F + bf->offU;
        {
            FIO_TIMED(f64 ? "bf2_V_f64" : "bf2_V_f32", s);
            first(VF, V, c1, c2);
        }
        {
            FIO_TIMED(f64 ? "bf2_M_f64" : "bf2_M_f32", s);
            middle(MF, M, c1, c2);
        }
        {
            FIO_TIMED(f64 ? "bf2_U_f64" : "bf2_U_f32", s);
            last(UF, U, c2);
        }
    } else {
        const C *Va = Fa + bf->offV, *Ma = Fa + bf->offM, *Ua = Fa + bf->offU;
        {
            FIO_TIMED(f64 ? "bf2_U_f64" : "bf2_U_f32", s);
            first(UA, Ua, c2, c1);
        }
        {
            FIO_TIMED(f64 ? "bf2_M_f64" : "bf2_M_f32", s);
            middle(MA, Ma, c2, c1);
        }
        {
            FIO_TIMED(f64 ? "bf2_V_f64" : "bf2_V_f32", s);
            last(VA, Va, c1);
        }
    }
    FIO_HIP(hipGetLastError());
}

template <typename T>
void apply2(fio_bf_s *bf, bool adj, const double2 *X, long ldx, double2 *Y, long ldy, int nrhs, const cpx<T> *F,
            const cpx<T> *Fa, void *ws, bool fint, hipStream_t s) {
    // Columns per wave and reduction split: tuned (fio_bf_autotune), or 8 columns, which pad least (n = 64, 70 columns:
    // 1002 us against 1064 us with 16; where no column is added the tuner takes 16 for large blocks: n = 128, 64
    // columns 7010 against 6320 us).  FP32 with 7 or 8 row tiles (see run_step): 16, except on the smallest
    // operators and where a third or more of the columns would be padding.
    const TileCfg c = bf_tile(bf, adj, sizeof(T) == 8 ? FIO_PREC_FP64 : FIO_PREC_FP32, nrhs);
    const int c8 = (nrhs + 7) / 8;
    const bool wide32 = sizeof(T) == 4 && bf->q >= 10 && bf->n1 >= 32 && c8 != 1 && c8 != 3;
    if (c.kc == 16 || (c.kc == 0 && wide32))
        apply2k<T, 2>(bf, adj, X, ldx, Y, ldy, nrhs, F, Fa, ws, fint, c.nsplit, s);
    else
        apply2k<T, 1>(bf, adj, X, ldx, Y, ldy, nrhs, F, Fa, ws, fint, c.nsplit, s);
}

}  // namespace

// ---------------------------------------------------------------------------
fio_status bf2d_plan(const fio_bf_desc *d, fio_bf_s *bf) {
    if (d->n < 4 || d->n > (1L << 15) || (d->n & (d->n - 1))) return FIO_ERR_ARG;
    if (d->phase_kind < FIO_PHASE2_ANISO || d->phase_kind > FIO_PHASE2_ISO) return FIO_ERR_ARG;
    if (d->amp_kind < FIO_AMP_ONE || d->amp_kind > FIO_AMP_HANKEL) return FIO_ERR_ARG;
    if (d->amp_kind == FIO_AMP_GAUSSIAN_SUM) return FIO_ERR_UNSUPPORTED;   // 1D amplitude only
    if (d->q < 2 || d->q > 16 || d->level_offset < 1) return FIO_ERR_ARG;
    int L = 0;
    while ((1L << L) < d->n) ++L;
    const int h = (L + 1) / 2;
    if (L - d->level_offset > h) return FIO_ERR_UNSUPPORTED;   // transfer levels are not built in 2D
    const int b = (int)(d->n >> h);
    if (b * b > 128) return FIO_ERR_UNSUPPORTED;                // a leaf box must fit one workgroup
    if (h > 7) return FIO_ERR_UNSUPPORTED;                      // 4^h leaf boxes on one grid axis
    if (d->q * d->q > 128) return FIO_ERR_UNSUPPORTED;
    bf->desc = *d;
    bf->desc.amp_centers = nullptr;          // not used in 2D
    bf->dim = 2;
    bf->n1 = d->n;
    bf->N = d->n * d->n;
    bf->L = L;
    bf->h = h;
    bf->lc = L - h;
    bf->Lp = h;
    bf->nl = 0;
    bf->q = d->q;
    bf->b = b;
    bf->hb = 0;
    while ((1 << bf->hb) < b) ++bf->hb;
    const size_t q2 = (size_t)d->q * d->q, b2 = (size_t)b * b;
    const size_t S = 1UL << (2 * h), T = 1UL << (2 * bf->lc);
    bf->offV = 0;
    bf->offM = T * S * q2 * b2;
    bf->offU = bf->offM + S * S * q2 * q2;
    bf->total = bf->offU + S * T * q2 * b2;
    return FIO_OK;
}

size_t bf2d_ws_bytes(const fio_bf_s *bf, int nrhs, fio_prec prec) {
    if (prec == FIO_PREC_SPLIT_FP16) return 0;
    const size_t es = prec == FIO_PREC_FP64 ? sizeof(double2) : sizeof(float2);
    const size_t ldc = (size_t)(nrhs + 15) / 16 * 16;     // the larger of the two column chunkings
    const size_t T = 1UL << (2 * bf->lc);
    const size_t ns = (size_t)nsplit_of((long)T);
    return (2 * (size_t)bf->N * bf->q * bf->q * ldc + (ns > 1 ? ns * (size_t)bf->N * ldc : 0)) * es;
}

void bf2d_generate(fio_bf_s *bf, hipStream_t s) {
    const G2 g = g2_of(bf);
    double2 *base = bf->f64.as<double2>();
    const size_t nV = bf->offM - bf->offV, nM = bf->offU - bf->offM, nU = bf->total - bf->offU;
    const Nodes tn = make_nodes(bf->q);
    DevBuf lagb(bf->b * bf->q * sizeof(double));
    const double *lag = lagb.as<double>();
    gen2_lagrange<<<grid1d(bf->b * bf->q, 64), 64, 0, s>>>(tn, bf->b, lagb.as<double>());
    gen2_V<<<grid1d(nV, 256), 256, 0, s>>>(g, tn, lag, base + bf->offV);
    gen2_M<<<grid1d(nM, 256), 256, 0, s>>>(g, tn, base + bf->offM);
    gen2_U<<<grid1d(nU, 256), 256, 0, s>>>(g, tn, lag, base + bf->offU);
    FIO_HIP(hipGetLastError());
    FIO_HIP(hipStreamSynchronize(s));        // the table is released here
}

// adjoint copies and the single-precision copies of both
void bf2d_finish(fio_bf_s *bf, hipStream_t s) {
    const G2 g = g2_of(bf);
    const size_t nV = bf->offM - bf->offV, nM = bf->offU - bf->offM, nU = bf->total - bf->offU;
    bf->adj64.alloc(bf->total * sizeof(double2));
    const double2 *F = bf->f64.as<double2>();
    double2 *A = bf->adj64.as<double2>();
    adj2_V<<<grid1d(nV, 256), 256, 0, s>>>(g, F + bf->offV, A + bf->offV);
    adj2_M<<<grid1d(nM, 256), 256, 0, s>>>(g, F + bf->offM, A + bf->offM);
    adj2_U<<<grid1d(nU, 256), 256, 0, s>>>(g, F + bf->offU, A + bf->offU);
    if (bf->desc.prec_mask & (1u << FIO_PREC_FP32)) {
        bf->f32.alloc(bf->total * sizeof(float2));
        bf->adj32.alloc(bf->total * sizeof(float2));
        cvt2_f32<<<grid1d(bf->total, 256), 256, 0, s>>>(F, bf->f32.as<float2>(), bf->total);
        cvt2_f32<<<grid1d(bf->total, 256), 256, 0, s>>>(A, bf->adj32.as<float2>(), bf->total);
    }
    FIO_HIP(hipGetLastError());
}

void bf2d_apply(fio_bf_s *bf, bool adj, const double2 *X, long ldx, double2 *Y, long ldy, int nrhs, fio_prec prec,
                void *ws, bool fint, hipStream_t s) {
    if (prec == FIO_PREC_FP64)
        apply2<double>(bf, adj, X, ldx, Y, ldy, nrhs, bf->f64.as<double2>(), bf->adj64.as<double2>(), ws, fint, s);
    else if (prec == FIO_PREC_FP32)
        apply2<float>(bf, adj, X, ldx, Y, ldy, nrhs, bf->f32.as<float2>(), bf->adj32.as<float2>(), ws, fint, s);
    else
        throw Err{FIO_ERR_UNSUPPORTED};
}

void permute2d(int n, bool to_internal, const double2 *X, long ldx, double2 *Y, long ldy, int nrhs, hipStream_t s) {
    int L = 0;
    while ((1 << L) < n) ++L;
    const size_t tot = (size_t)n * n * nrhs;
    if (tot == 0) return;
    k_perm2<<<grid1d(tot, 256), 256, 0, s>>>(n, L, to_internal ? 1 : 0, X, ldx, Y, ldy, nrhs);
    FIO_HIP(hipGetLastError());
}

}  // namespace fio

extern "C" fio_status fio_permute2d(long n, int to_internal, const void *X, long ldx, void *Y, long ldy, int nrhs,
                                    void *stream) {
    FIO_CHECK_ARG(n >= 1 && n <= (1L << 15) && (n & (n - 1)) == 0 && nrhs >= 0);
    if (nrhs == 0) return FIO_OK;
    FIO_CHECK_ARG(X && Y && X != Y && ldx >= n * n && ldy >= n * n);
    return fio::guarded([&] {
        fio::permute2d((int)n, to_internal != 0, (const double2 *)X, ldx, (double2 *)Y, ldy, nrhs,
                       fio::as_stream(stream));
        return FIO_OK;
    });
}
