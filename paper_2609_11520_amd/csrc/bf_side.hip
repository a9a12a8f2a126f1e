// Side passes of the 1D structured butterfly (see bf_side.h): table generation and kernels.
#include "bf_side.h"

#include <algorithm>

#include "bf_apply.h"
#include "ddmath.h"

namespace fio {

// ---------------------------------------------------------------------------
// tables
SideOff side_off(const fio_bf_s *bf) {
    SideOff o;
    const size_t N = bf->N;
    o.amp = bf->amp.m > 0;
    o.V = kSideHead;
    o.C = o.V + 8 * 2 * kSideEV;
    o.M = o.C + ((size_t)(16 << bf->nl) - 16) * 2 * kSideRow;
    o.B = o.M + (o.amp ? N * kSideEMamp : ((size_t)1 << bf->h) * 2 * kSideEM);
    o.U = o.B + ((size_t)(2L << (bf->h + bf->nl)) - (2L << bf->h)) * 2 * kSideRow;
    o.total = o.U + N * kSideEU;
    return o;
}

bool side_built(const fio_bf_s *bf) { return bf->side64.p != nullptr; }

__device__ __forceinline__ unsigned rev_bits(unsigned v, int bits) { return bits ? __brev(v) >> (32 - bits) : 0u; }

// kappa(x) = x + sgn c(x)
__device__ __forceinline__ dd kappa(const Geo &g, dd x, double sgn) { return dd_add(x, dd_mul_d(c_dd(g, x), sgn)); }

// C twiddles b(0, t) of (tau, sign) at every level j: alpha at spatial level 3 + j, children of width w
__global__ void gen_side_C(Geo g, Nodes tn, int nl, double2 *out) {
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const long row = id / kSideRow + 32;                        // 2 (tau + 2^(4+j)), the levels one after another
    if (row >= (32L << nl)) return;
    const int t = id % kSideRow;
    if (t >= kSideQ) {
        out[id] = zc(0.0, 0.0);
        return;
    }
    const int lev = 63 - __clzll(row >> 1);                     // spatial level of tau, 4 + j
    const long tau = (row >> 1) - (1L << lev);
    const double sgn = (row & 1) ? 1.0 : -1.0;
    const double yt = (tau + 0.5) / (double)(1L << lev), ya = ((tau >> 1) + 0.5) / (double)(1L << (lev - 1));
    const double hw = 0.5 * (double)g.N / (double)(1L << (g.L + 1 - lev));       // beta at frequency level L + 1 - lev
    const dd kt = kappa(g, dd_of(yt), sgn), dk = dd_sub(kt, kappa(g, dd_of(ya), sgn));
    const dd ph = dd_sub(dd_frac(dd_mul(dk, dd_ldexp(tn.t(t), hw))), dd_frac(dd_mul_d(kt, hw)));
    out[id] = dd_expi2pi(ph);
}

// B twiddles a(0, i) of (tau, sign) at every level j: tau at spatial level h + 1 + j
__global__ void gen_side_B(Geo g, Nodes tn, int nl, double2 *out) {
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const long row = id / kSideRow + (4L << g.h);
    if (row >= (4L << (g.h + nl))) return;
    const int i = id % kSideRow;
    if (i >= kSideQ) {
        out[id] = zc(0.0, 0.0);
        return;
    }
    const int lev = 63 - __clzll(row >> 1);                     // spatial level of tau
    const long tau = (row >> 1) - (1L << lev);
    const double sgn = (row & 1) ? 1.0 : -1.0, wt = 1.0 / (double)(1L << lev);
    const double hw = 0.5 * (double)g.N / (double)(1L << (g.L + 1 - lev));       // half the width of beta
    const dd z = dd_add(dd_of((tau + 0.5) * wt), dd_ldexp(tn.t(i), 0.5 * wt));
    out[id] = dd_expi2pi(dd_frac(dd_mul_d(kappa(g, z, sgn), -hw)));
}

__global__ void gen_side_V(Geo g, double2 *out) {
    const int id = threadIdx.x;
    if (id >= 8 * 2 * kSideEV) return;
    const int e = id % kSideEV, row = id / kSideEV;
    const dd kap = kappa(g, dd_of(((row >> 1) + 0.5) / 8.0), (row & 1) ? 1.0 : -1.0);
    out[id] = dd_expi2pi(dd_frac(dd_mul_d(kap, e < 3 ? e + 1.0 : -4.0)));
}

// leaf entry s of (box, partner) sits at ((box / 8) 8 + s) 64 + partner 8 + box % 8
__device__ __forceinline__ size_t leaf_pos(unsigned box, unsigned partner) {
    return (size_t)(box >> 3) * kSideEU * 64 + partner * 8 + (box & 7u);
}

__global__ void gen_side_U(Geo g, double2 *out) {
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id >= (size_t)g.N * kSideEU) return;
    const int lane = id & 63, s = (int)((id >> 6) % kSideEU);
    const long box = (long)((id >> 6) / kSideEU) * 8 + (lane & 7);
    const double eta = -0.5 * g.N + ((lane >> 3) + 0.5) * ((double)g.N / 8.0);
    const dd x = dd_of((double)(box * 8 + s) / (double)g.N);
    const dd lin = dd_frac(dd_mul_d(x, eta)), non = dd_frac(dd_mul_d(c_dd(g, x), fabs(eta)));
    out[id] = dd_expi2pi(dd_add(lin, non));
}

// Y_ij of (tau, sign) at level h; with an amplitude, of every pair p = tau 2^h + sigma (blocks of 64 pairs)
__global__ void gen_side_M(Geo g, Nodes tn, Amp am, int full, double2 *out) {
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const long H = 1L << g.h;
    if (id >= (full ? (size_t)g.N * kSideEMamp : (size_t)H * 2 * kSideEM)) return;
    long tau, sigma = 0;
    int e;
    double sgn;
    const double wf = (double)g.N / (double)H;
    double eta = 0.0;
    if (full) {
        e = (int)((id >> 6) % kSideEMamp);
        const long p = (long)((id >> 6) / kSideEMamp) * 64 + (id & 63);
        tau = p / H;
        sigma = p % H;
        eta = -0.5 * g.N + (sigma + 0.5) * wf;
        sgn = eta > 0 ? 1.0 : -1.0;
    } else {
        e = (int)(id % kSideEM);
        tau = (long)(id / kSideEM) >> 1;
        sgn = ((id / kSideEM) & 1) ? 1.0 : -1.0;
    }
    const int i = full ? e / 9 : e / 4, j = full ? e % 9 : e % 4;
    const dd y = dd_of((tau + 0.5) / (double)H), z = dd_add(y, dd_ldexp(tn.t(i), 0.5 / (double)H));
    const dd dk = dd_sub(kappa(g, z, sgn), kappa(g, y, sgn)), dg = dd_ldexp(tn.t(j), 0.5 * wf);
    const double2 v = dd_expi2pi(dd_frac(dd_mul(dk, dg)));
    const double av = full ? amp_at(am, dd_val(z), eta + dd_val(dg), (double)g.N) : 1.0;
    out[id] = zc(v.x * av, v.y * av);
}

// The matrices at the head of the tables, rows of 9 reals.  Rows 0..8, row t of P_0 in halves:
// (P_0(t, r) + P_0(t, q-1-r)) / 2 for r < 4, P_0(t, 4), the half differences for r < 4, with
// P_0(t, r) = p_r(-1/2 + t_t / 2) (P_1(i, t) = P_0(q-1-i, q-1-t)).  Row 9: the leaf values P(0, i); rows
// 10..12: P(4 + m, .), m = 1..3, in the same halves (P(s, i) = p_i((s - 4) / 4), P(4 - m, i) = P(4 + m, q-1-i)
// and P(4, i) = [i = 4]).
__global__ void gen_side_head(Nodes tn, double *out) {
    const int id = threadIdx.x;
    if (id >= 2 * kSideHead) return;
    const int row = id / 9, c = id % 9, r = c < 5 ? c : c - 5;
    if (row >= 13) {
        out[id] = 0.0;
        return;
    }
    const dd u = row < 9 ? dd_add(dd_of(-0.5), dd_ldexp(tn.t(row), 0.5)) : dd_of(row == 9 ? -1.0 : (row - 9) / 4.0);
    if (row == 9) {
        out[id] = dd_lagrange(u, c, tn);
        return;
    }
    const double p = dd_lagrange(u, r, tn), m = dd_lagrange(u, 8 - r, tn);
    out[id] = c == 4 ? p : 0.5 * (c < 4 ? p + m : p - m);
}

__global__ void cvt_side_f32(const double2 *in, float2 *out, size_t n) {
    const size_t id = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (id < n) out[id] = make_float2((float)in[id].x, (float)in[id].y);
}

void side_generate(fio_bf_s *bf, hipStream_t s) {
    const SideOff o = side_off(bf);
    const Geo g = geo_of(bf);
    const Nodes tn = make_nodes(bf->q);
    bf->side64.alloc(o.total * sizeof(double2));
    double2 *t = bf->side64.as<double2>();
    const unsigned T = 256;
    gen_side_head<<<1, 2 * kSideHead, 0, s>>>(tn, reinterpret_cast<double *>(t));
    gen_side_V<<<1, 64, 0, s>>>(g, t + o.V);
    gen_side_C<<<grid1d(o.M - o.C, T), T, 0, s>>>(g, tn, bf->nl, t + o.C);
    gen_side_M<<<grid1d(o.B - o.M, T), T, 0, s>>>(g, tn, bf->amp, o.amp, t + o.M);
    gen_side_B<<<grid1d(o.U - o.B, T), T, 0, s>>>(g, tn, bf->nl, t + o.B);
    gen_side_U<<<grid1d(o.total - o.U, T), T, 0, s>>>(g, t + o.U);
    FIO_HIP(hipGetLastError());
}

void side_make_f32(fio_bf_s *bf, hipStream_t s) {
    const size_t n = side_off(bf).total;
    bf->side32.alloc(n * sizeof(float2));
    cvt_side_f32<<<grid1d(n, 256), 256, 0, s>>>(bf->side64.as<double2>(), bf->side32.as<float2>(), n);
    FIO_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// kernels
template <typename T> struct SideArgs {
    const cpx<T> *TW;        // transfer table of the side
    const cpx<T> *LF;        // leaf table of the side
    const cpx<T> *M;         // middle table
    const T *mat;            // matrix rows at the head of the tables
    const double2 *X;        // input vectors (null: coefficients from `in`)
    long ldx;
    const cpx<T> *in;
    cpx<T> *out;
    double2 *Y;              // output vectors (leaf factor applied at the end)
    long ldy;
    const double2 *Ysub;     // not null: Y = Ysub - the result
    long ldsub;
    int nrhs, kc, nch;       // columns, columns per workgroup, column chunks
    int nset, nsb;           // workgroup sets, and sub-butterflies (or leaf boxes) per workgroup
    int j0, kl;              // first level of the side and levels of this pass
    int L, h, Lp;
    int mid;                 // 0: no middle factor, kSideEM or kSideEMamp: its table form
};

#define FIO_SIDE_FN __device__ __forceinline__

template <typename C> FIO_SIDE_FN C smul(C a, C b) {
    C r;
    r.x = fma(-a.y, b.y, a.x * b.x);
    r.y = fma(a.y, b.x, a.x * b.y);
    return r;
}
template <typename C> FIO_SIDE_FN C smulc(C a, C b) {   // conj(a) b
    C r;
    r.x = fma(a.y, b.y, a.x * b.x);
    r.y = fma(-a.y, b.x, a.x * b.y);
    return r;
}
// acc + m v with a real m (set for the first term)
template <typename T> FIO_SIDE_FN void racc(cpx<T> &acc, T m, cpx<T> v, bool first) {
    acc.x = first ? m * v.x : fma(m, v.x, acc.x);
    acc.y = first ? m * v.y : fma(m, v.y, acc.y);
}

// Values that are uniform over the wave and constant while a kernel runs, read through the scalar
// cache (the constant address space).
template <typename V> using scalar_ptr = const __attribute__((address_space(4))) V *;

// Row r of the matrices, read one row ahead of its use: with the offset opaque the compiler does not
// hold the whole matrix in scalar registers.
template <typename T> struct MatRow {
    T v[9];
    FIO_SIDE_FN void read(const T *m, int r) {
        int o = r * 9;
        asm volatile("" : "+s"(o));
        const scalar_ptr<T> p = (scalar_ptr<T>)(uintptr_t)m + o;
#pragma unroll
        for (int i = 0; i < 9; ++i) v[i] = p[i];
    }
};

// Keeps the loads of the next part of a kernel behind this point: without it the compiler
// issues every load of a level at once and spills the registers they return to.
FIO_SIDE_FN void load_fence() { asm volatile("" ::: "memory"); }

// One transfer group for the lane's column: x0, x1 the two children's coefficients in, the two
// children's coefficients out.  With the mirror symmetry of P_0, P_1 the two outputs of one input
// child (B forward, C adjoint) and the two inputs of one output child (C forward, B adjoint) share
// one product with the symmetric and antisymmetric halves (81 real multiply-adds per component),
// and the conjugate pairs of the twiddles turn their products into real scalings of sums and
// differences.  A scalar row of the matrix feeds both children: 36 multiply-adds.
//   The 9 twiddles of child c sit at tw + c 2 kSideRow; FP32 loads them all ahead (two per load),
// FP64 kAhead rows ahead of use.
template <typename T, bool CS, bool ADJ> struct SideGroup {
    using C = cpx<T>;
    static constexpr bool D = sizeof(T) == 8;
    static constexpr int kAhead = 4;   // rows
    C w[2][10];

    // twiddle of row t and child c (the second child's rows run down on the B side)
    static FIO_SIDE_FN constexpr int ent(int t, int c) { return !CS && c ? 8 - t : t; }
    template <int t> FIO_SIDE_FN void load_row(const C *tw) {
        w[0][ent(t, 0)] = tw[ent(t, 0)];
        w[1][ent(t, 1)] = tw[2 * kSideRow + ent(t, 1)];
    }
    FIO_SIDE_FN void prefetch(const C *tw) {
        load_fence();
        if constexpr (D) {
            load_row<0>(tw);
            load_row<1>(tw);
            load_row<2>(tw);
            load_row<3>(tw);
        } else {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const float4 v = reinterpret_cast<const float4 *>(tw + c * 2 * kSideRow)[i];
                    w[c][2 * i] = cmake<C>(v.x, v.y);
                    w[c][2 * i + 1] = cmake<C>(v.z, v.w);
                }
        }
        load_fence();
    }
    template <int t> FIO_SIDE_FN void advance(const C *tw) {
        if constexpr (D && t + kAhead < 9) {
            load_fence();
            load_row<t + kAhead>(tw);
            load_fence();
        }
    }

    // row t of the sums into e (symmetric half) and f (antisymmetric half): [0], [1] are the children
    // on the C side, the real and imaginary parts of the twiddles on the B side
    template <int t> FIO_SIDE_FN void out_row(const T *mat, const C *tw, const C (&x0)[9], const C (&x1)[9],
                                              const MatRow<T> &row, C (&e)[2][5], C (&f)[2][4]) {
        if constexpr (t < 9) {
            MatRow<T> next;
            if constexpr (t < 8) next.read(mat, t + 1);
            advance<t>(tw);
            C s[2], d[2];
            if constexpr (CS) {
                const C u = cadd(x0[t], x1[8 - t]), v = csub(x0[t], x1[8 - t]);
#pragma unroll
                for (int c = 0; c < 2; ++c) {      // b x_0 +- conj(b) x_1
                    const C b = w[c][t];
                    s[c].x = fma(-b.y, v.y, b.x * u.x);
                    s[c].y = fma(b.y, v.x, b.x * u.y);
                    d[c].x = fma(-b.y, u.y, b.x * v.x);
                    d[c].y = fma(b.y, u.x, b.x * v.y);
                }
            } else {
                const C a0 = w[0][t], a1 = w[1][8 - t];
                const C p = cscale(x0[t], a0.x), q = cscale(x1[8 - t], a1.x);
                const C pi = cscale(x0[t], a0.y), qi = cscale(x1[8 - t], a1.y);
                s[0] = cadd(p, q);
                d[0] = csub(p, q);
                s[1] = cadd(pi, qi);
                d[1] = csub(pi, qi);
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int r = 0; r < 5; ++r) racc(e[c][r], row.v[r], s[c], t == 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) racc(f[c][r], row.v[5 + r], d[c], t == 0);
            }
            out_row<t + 1>(mat, tw, x0, x1, next, e, f);
        }
    }
    // row r of both outputs from the halves of both inputs (C side) or of their sum and difference (B side)
    template <int r> FIO_SIDE_FN void in_row(const T *mat, const C *tw, const C (&s)[2][4], const C (&d)[2][4],
                                             const C (&mid)[2], const MatRow<T> &row, C (&y0)[9], C (&y1)[9]) {
        if constexpr (r < 9) {
            MatRow<T> next;
            if constexpr (r < 8) next.read(mat, r + 1);
            advance<r>(tw);
            C p[2], q[2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                C u, v;
                racc(u, row.v[4], mid[o], true);
                racc(v, row.v[5], d[o][0], true);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    racc(u, row.v[t], s[o][t], false);
                    if (t) racc(v, row.v[5 + t], d[o][t], false);
                }
                p[o] = cadd(u, v);
                q[o] = csub(u, v);
            }
            if constexpr (CS) {
                C y = smulc(w[0][r], p[0]), z = smul(w[0][r], q[0]);
                cfmac(y, w[1][r], p[1]);
                cfma(z, w[1][r], q[1]);
                y0[r] = y;
                y1[8 - r] = z;
            } else {
                const C a0 = w[0][r], a1 = w[1][8 - r];
                y0[r].x = fma(-a0.y, p[1].y, a0.x * p[0].x);
                y0[r].y = fma(a0.y, p[1].x, a0.x * p[0].y);
                y1[8 - r].x = fma(-a1.y, q[1].y, a1.x * q[0].x);
                y1[8 - r].y = fma(a1.y, q[1].x, a1.x * q[0].y);
            }
            in_row<r + 1>(mat, tw, s, d, mid, next, y0, y1);
        }
    }

    FIO_SIDE_FN void apply(const T *mat, const C *tw, C (&x0)[9], C (&x1)[9]) {
        MatRow<T> row;
        row.read(mat, 0);
        if constexpr (CS != ADJ) {
            C e[2][5], f[2][4];
            out_row<0>(mat, tw, x0, x1, row, e, f);
            if constexpr (CS) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    x0[r] = cadd(e[0][r], f[0][r]);
                    x0[8 - r] = csub(e[0][r], f[0][r]);
                    x1[r] = cadd(e[1][r], f[1][r]);
                    x1[8 - r] = csub(e[1][r], f[1][r]);
                }
                x0[4] = e[0][4];
                x1[4] = e[1][4];
            } else {
                // conj(a) = re - i im for the first child, a for the second
                auto put = [&](int r, C p, C q) {
                    x0[r] = cmake<C>(p.x + q.y, p.y - q.x);
                    x1[r] = cmake<C>(p.x - q.y, p.y + q.x);
                };
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    put(r, cadd(e[0][r], f[0][r]), cadd(e[1][r], f[1][r]));
                    put(8 - r, csub(e[0][r], f[0][r]), csub(e[1][r], f[1][r]));
                }
                put(4, e[0][4], e[1][4]);
            }
        } else {
            C s[2][4], d[2][4], mid[2];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const C a = x0[t], b = x0[8 - t], c = x1[t], g = x1[8 - t];
                if constexpr (CS) {
                    s[0][t] = cadd(a, b);
                    d[0][t] = csub(a, b);
                    s[1][t] = cadd(c, g);
                    d[1][t] = csub(c, g);
                } else {
                    const C p = cadd(a, c), q = csub(a, c), p2 = cadd(b, g), q2 = csub(b, g);
                    s[0][t] = cadd(p, p2);
                    d[0][t] = csub(p, p2);
                    s[1][t] = cadd(q, q2);
                    d[1][t] = csub(q, q2);
                }
            }
            mid[0] = CS ? x0[4] : cadd(x0[4], x1[4]);
            mid[1] = CS ? x1[4] : csub(x0[4], x1[4]);
            in_row<0>(mat, tw, s, d, mid, row, x0, x1);
        }
    }
};

// The leaf factor on 8 input rows: V (lf: its 4 entries) or U^* (lf: the block's 8 entries, 64 apart)
template <typename T, bool USIDE>
FIO_SIDE_FN void side_leaf_fwd(const T *mat, const cpx<T> *lf, cpx<T> (&w)[8], cpx<T> (&c)[9]) {
    using C = cpx<T>;
    MatRow<T> row;
    row.read(mat, 9);
    if constexpr (USIDE) {
#pragma unroll
        for (int s = 0; s < 8; ++s) w[s] = smulc(lf[s * 64], w[s]);
    } else {
        w[0] = smul(lf[3], w[0]);
#pragma unroll
        for (int m = 1; m < 4; ++m) {
            const C e = lf[m - 1];
            w[4 + m] = smul(e, w[4 + m]);
            w[4 - m] = smulc(e, w[4 - m]);
        }
    }
    C E[5], O[4];
#pragma unroll
    for (int i = 0; i < 9; ++i) racc(c[i], row.v[i], w[0], true);
#pragma unroll
    for (int m = 1; m < 4; ++m) {
        row.read(mat, 9 + m);
        const C S = cadd(w[4 + m], w[4 - m]), Df = csub(w[4 + m], w[4 - m]);
#pragma unroll
        for (int i = 0; i < 5; ++i) racc(E[i], row.v[i], S, m == 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) racc(O[i], row.v[5 + i], Df, m == 1);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c[i] = cadd(c[i], cadd(E[i], O[i]));
        c[8 - i] = cadd(c[8 - i], csub(E[i], O[i]));
    }
    c[4] = cadd(cadd(c[4], E[4]), w[4]);
}

// its adjoint: 8 rows from 9 coefficients, handed to emit(row, value) as they are formed
template <typename T, bool USIDE, typename Emit>
FIO_SIDE_FN void side_leaf_bwd(const T *mat, const cpx<T> *lf, cpx<T> (&c)[9], Emit &&emit) {
    using C = cpx<T>;
    MatRow<T> row, next;
    row.read(mat, 9);
    next.read(mat, 10);
    C y;
#pragma unroll
    for (int i = 0; i < 9; ++i) racc(y, row.v[i], c[i], i == 0);
    emit(0, USIDE ? smul(lf[0], y) : smulc(lf[3], y));
    if constexpr (USIDE)
        emit(4, smul(lf[4 * 64], c[4]));
    else
        emit(4, c[4]);
    // sums and differences of the mirrored coefficients in place
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const C p = c[i], q = c[8 - i];
        c[i] = cadd(p, q);
        c[8 - i] = csub(p, q);
    }
#pragma unroll
    for (int m = 1; m < 4; ++m) {
        load_fence();
        row = next;
        if (m < 3) next.read(mat, 10 + m);
        C u, v;
        racc(u, row.v[4], c[4], true);
        racc(v, row.v[5], c[8], true);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            racc(u, row.v[i], c[i], false);
            if (i) racc(v, row.v[5 + i], c[8 - i], false);
        }
        const C p = cadd(u, v), q = csub(u, v);
        if constexpr (USIDE) {
            emit(4 + m, smul(lf[(4 + m) * 64], p));
            emit(4 - m, smul(lf[(4 - m) * 64], q));
        } else {
            const C e = lf[m - 1];
            emit(4 + m, smulc(e, p));
            emit(4 - m, smul(e, q));
        }
    }
}

// Middle factor of the thread's two pairs for a = 1 (one block: they share the spatial box and the
// sign; V is scalar_ptr when the whole workgroup does): x <- Y x, or Y^* x
template <typename T, bool ADJ, typename V> FIO_SIDE_FN void side_middle(V m, cpx<T> (&xa)[9], cpx<T> (&xb)[9]) {
    using C = cpx<T>;
    if constexpr (!ADJ) {
        // y_i = x_4 + sum_j Y_ij x_j + conj(Y_ij) x_(8-j)
        C E[2][4], Df[2][4], mid[2] = {xa[4], xb[4]};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            E[0][j] = cadd(xa[j], xa[8 - j]);
            Df[0][j] = csub(xa[j], xa[8 - j]);
            E[1][j] = cadd(xb[j], xb[8 - j]);
            Df[1][j] = csub(xb[j], xb[8 - j]);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            T yr[4], yi[4];
            load_fence();
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                yr[j] = m[2 * (i * 4 + j)];
                yi[j] = m[2 * (i * 4 + j) + 1];
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                C s = mid[b];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    s.x = fma(yr[j], E[b][j].x, s.x);
                    s.y = fma(yr[j], E[b][j].y, s.y);
                    s.x = fma(-yi[j], Df[b][j].y, s.x);
                    s.y = fma(yi[j], Df[b][j].x, s.y);
                }
                if (b)
                    xb[i] = s;
                else
                    xa[i] = s;
            }
        }
    } else {
        // conj(Y) w = p w - i q w, Y w = p w + i q w with Y = p + i q
        C pv[2][4], qv[2][4], sum[2];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            T yr[4], yi[4];
            load_fence();
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                yr[j] = m[2 * (i * 4 + j)];
                yi[j] = m[2 * (i * 4 + j) + 1];
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const C v = b ? xb[i] : xa[i];
                sum[b] = i ? cadd(sum[b], v) : v;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    racc(pv[b][j], yr[j], v, i == 0);
                    racc(qv[b][j], yi[j], v, i == 0);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            xa[j] = cmake<C>(pv[0][j].x + qv[0][j].y, pv[0][j].y - qv[0][j].x);
            xa[8 - j] = cmake<C>(pv[0][j].x - qv[0][j].y, pv[0][j].y + qv[0][j].x);
            xb[j] = cmake<C>(pv[1][j].x + qv[1][j].y, pv[1][j].y - qv[1][j].x);
            xb[8 - j] = cmake<C>(pv[1][j].x - qv[1][j].y, pv[1][j].y + qv[1][j].x);
        }
        xa[4] = sum[0];
        xb[4] = sum[1];
    }
}

// Middle blocks of the thread's two pairs with an amplitude: entries 64 apart at m, those of the second pair next to
// the first's (in FP32 one load for both).  The loads bound it: one pair after the other, N = 2^16 forward, 64
// columns, took 1430 us in FP64 (1370 with 64-column tiles and scalar loads), both at once 1280 us.
template <typename T> struct MidPair {
    cpx<T> a, b;
};
FIO_SIDE_FN MidPair<float> mid_pair(const float2 *m) {
    const float4 v = *reinterpret_cast<const float4 *>(m);
    return {make_float2(v.x, v.y), make_float2(v.z, v.w)};
}
FIO_SIDE_FN MidPair<double> mid_pair(const double2 *m) { return {m[0], m[1]}; }

template <typename T, bool ADJ> FIO_SIDE_FN void side_middle_full(const cpx<T> *m, cpx<T> (&x0)[9], cpx<T> (&x1)[9]) {
    using C = cpx<T>;
    C y0[9], y1[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) y0[i] = y1[i] = czero<C>();
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        load_fence();
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            const MidPair<T> v = mid_pair(m + (i * 9 + j) * 64);
            if constexpr (ADJ) {
                cfmac(y0[j], v.a, x0[i]);
                cfmac(y1[j], v.b, x1[i]);
            } else {
                cfma(y0[i], v.a, x0[j]);
                cfma(y1[i], v.b, x1[j]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        x0[i] = y0[i];
        x1[i] = y1[i];
    }
}

template <typename T, bool ADJ>
FIO_SIDE_FN void side_apply_mid(const SideArgs<T> &a, unsigned box, unsigned neg, size_t pair, cpx<T> (&x0)[9],
                                cpx<T> (&x1)[9]) {
    if (a.mid == kSideEMamp) {
        const cpx<T> *m = a.M + (pair >> 6) * kSideEMamp * 64 + (pair & 63);
        side_middle_full<T, ADJ>(m, x0, x1);
    } else if (a.nsb == 1) {
        const int o = __builtin_amdgcn_readfirstlane((int)(box * 2 + neg) * kSideEM);
        side_middle<T, ADJ>((scalar_ptr<T>)(uintptr_t)(a.M + o), x0, x1);
    } else {
        side_middle<T, ADJ>(reinterpret_cast<const T *>(a.M + (size_t)(box * 2 + neg) * kSideEM), x0, x1);
    }
}

// A workgroup owns nsb closed sub-butterflies of 2^kl pairs and kc columns; a thread owns one group
// (two pairs) and one column through all kl levels.  At level j the thread's two pairs are the
// slots that differ in bit j; its thread number g holds the other slot bits, bit j + 1 at position j
// (for the next level; the adjoint runs the levels down).  Between two levels that position takes
// over bit j: the thread keeps one of its two pairs and swaps the other with the thread that
// differs there, so the exchange needs LDS for one pair per thread only.  The first level reads HBM
// (or the leaf factor's output) straight into registers and the last one stores from registers.
// FP64 runs 2 waves per SIMD (up to 256 registers), FP32 3.
//   A vector load costs the L1 16 cycles whatever its lanes share, and FP64 multiply-adds issue every 5.3
// cycles at 2 waves per SIMD: with per-pair twiddles (54 loads per B group) the loads bound the pass; with the
// shared tables of bf_side.h (18 per group) the vector units do.  N = 2^18, one apply, FP64 / FP32 ms, against
// the 3-level passes with 64 columns per workgroup that this kernel replaced: 1 column 0.10 / 0.07 against
// 4.07 / 2.18, 8 columns 0.48 / 0.25 against 4.06 / 2.21, 64 columns 3.5 / 1.8 against 5.73 / 2.98.
//   OUT (B forward, C adjoint, whole sides): the workgroup runs the 8 coarse partners of its leaf boxes one
// after another and sums the leaf factor's rows in registers, so that the leaf coefficients never
// reach memory.
template <typename T, bool CS, bool ADJ, bool OUT>
__global__ void __launch_bounds__(256, sizeof(T) == 8 ? 2 : 3) k_side_pass(SideArgs<T> a) {
    using C = cpx<T>;
    static_assert(!OUT || CS == ADJ, "leaf output: B forward, C adjoint");
    extern __shared__ double2 side_lds[];
    C *xch = reinterpret_cast<C *>(side_lds);                 // one pair per thread
    const int kl = a.kl, kc = a.kc;
    const unsigned G = 1u << (kl - 1);
    // Workgroups go round-robin over the 8 XCDs: an XCD gets runs of 8 consecutive sets, every column
    // chunk of a set in a row, so that what neighbours share (input rows, tables) comes from its L2.
    const unsigned b = blockIdx.x;
    unsigned set, chunk;
    if ((a.nset & 63) == 0) {
        const unsigned i = b >> 3, q = i / a.nch;
        chunk = i % a.nch;
        set = (q >> 3) * 64 + (b & 7u) * 8 + (q & 7u);
    } else {
        chunk = b % a.nch;
        set = b / a.nch;
    }
    const unsigned tid = threadIdx.x, gl = tid / kc, c = tid - gl * kc;
    const unsigned sub = set * a.nsb + (gl >> (kl - 1)), g = gl & (G - 1u);
    // alpha and sigma boxes of the pass's sub-butterflies (log2 of their numbers).  Sub-butterflies with
    // the same leaf boxes and different coarse partners follow one another; OUT counts leaf box sets.
    const int lA = CS ? 3 + a.j0 : a.h + a.j0, lS = a.L - lA - kl;
    unsigned A = 0, S = 0;
    if constexpr (OUT) {
        (CS ? S : A) = sub;
    } else if constexpr (CS) {
        A = sub & ((1u << lA) - 1u);
        S = sub >> lA;
    } else {
        S = sub & ((1u << lS) - 1u);
        A = sub >> lS;
    }
    const int col0 = chunk * kc + c;
    const bool act = col0 < a.nrhs;
    const int col = act ? col0 : a.nrhs - 1;
    const size_t ld = a.nrhs;
    const unsigned gr = rev_bits(g, kl - 1);
    // the thread's first pair before the first and after the last forward level (the other one: + 1, + 2^lS)
    auto pair_in = [&]() { return ((size_t)A << (lS + kl)) + ((size_t)S << kl) + 2 * g; };
    auto pair_out = [&]() { return ((((size_t)A << kl) + 2 * gr) << lS) + S; };
    auto load = [&](C (&x0)[9], C (&x1)[9]) {
        const size_t p0 = ADJ ? pair_out() : pair_in(), p1 = ADJ ? p0 + ((size_t)1 << lS) : p0 + 1;
        // (an opaque stride: the row addresses are formed here, not kept in registers across OUT's loop)
        size_t ld = a.nrhs;
        asm volatile("" : "+s"(ld));
        const C *i0 = a.in + p0 * 9 * ld + col, *i1 = a.in + p1 * 9 * ld + col;
        load_fence();
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            x0[i] = i0[i * ld];
            x1[i] = i1[i * ld];
        }
        load_fence();
    };
    // sign of the frequency: the top bit of sigma
    auto neg = [&]() { return S >> (lS - 1); };
    // twiddles of the thread's group at the st-th level of the pass
    auto table = [&](int st) {
        const int j = ADJ ? kl - 1 - st : st;
        const unsigned alpha = (A << j) | rev_bits(g & ((1u << j) - 1u), j);
        const size_t first = CS ? ((size_t)16 << (a.j0 + j)) - 16 : ((size_t)2 << (a.h + a.j0 + j)) - ((size_t)2 << a.h);
        return a.TW + ((first + 2 * alpha) * 2 + neg()) * kSideRow;
    };
    SideGroup<T, CS, ADJ> grp;
    C *own = xch + tid * 9;
    // the levels of one sub-butterfly; the first level's twiddles are prefetched
    auto levels = [&](C (&x0)[9], C (&x1)[9]) {
        const C *tw = table(0);
#pragma unroll 1
        for (int st = 0;; ++st) {
            grp.apply(a.mat, tw, x0, x1);
            if (st + 1 == kl) break;
            tw = table(st + 1);
            grp.prefetch(tw);
            const int pos = ADJ ? kl - 2 - st : st;          // thread bit that changes its slot bit
            const bool one = (g >> pos) & 1u;
            const C *peer = xch + (int)(tid + (one ? -(kc << pos) : kc << pos)) * 9;
            if (st || OUT) __syncthreads();                  // the last exchange has been read
            // (the empty asm keep the two sides apart: merged, they would index the pairs through memory)
            if (one) {
                asm volatile("; send 0" ::: "memory");
#pragma unroll
                for (int i = 0; i < 9; ++i) own[i] = x0[i];
                asm volatile("; send 0 done" ::: "memory");
            } else {
                asm volatile("; send 1" ::: "memory");
#pragma unroll
                for (int i = 0; i < 9; ++i) own[i] = x1[i];
                asm volatile("; send 1 done" ::: "memory");
            }
            __syncthreads();
            if (one) {
                asm volatile("; take 0" ::: "memory");
#pragma unroll
                for (int i = 0; i < 9; ++i) x0[i] = peer[i];
                asm volatile("; take 0 done" ::: "memory");
            } else {
                asm volatile("; take 1" ::: "memory");
#pragma unroll
                for (int i = 0; i < 9; ++i) x1[i] = peer[i];
                asm volatile("; take 1 done" ::: "memory");
            }
        }
    };
    // the thread's two neighbouring leaf boxes: before the first level (C), after the last (B)
    auto leaf_box = [&]() { return CS ? (S << kl) + 2 * g : (A << kl) + 2 * gr; };
    auto leaf_tab = [&](unsigned box) {
        return CS ? a.LF + (A * 2 + neg()) * kSideEV : a.LF + leaf_pos(box, S);
    };
    if constexpr (OUT) {
        const unsigned box = leaf_box();
        C ya[8], yb[8], x0[9], x1[9];
#pragma unroll
        for (int s = 0; s < 8; ++s) ya[s] = yb[s] = czero<C>();
        load(x0, x1);
        grp.prefetch(table(0));
#pragma unroll 1
        for (int p = 0;; ++p) {
            if constexpr (!CS) {
                if (a.mid) side_apply_mid<T, false>(a, A, neg(), pair_in(), x0, x1);
            }
            levels(x0, x1);
            const C *lf = leaf_tab(box);
            load_fence();
            side_leaf_bwd<T, !CS>(a.mat, lf, x0, [&](int s, C v) { ya[s] = cadd(ya[s], v); });
            load_fence();
            side_leaf_bwd<T, !CS>(a.mat, CS ? lf : lf + 1, x1, [&](int s, C v) { yb[s] = cadd(yb[s], v); });
            load_fence();
            if (p == 7) break;
            (CS ? A : S) = p + 1;
            load(x0, x1);
            grp.prefetch(table(0));
        }
        if (act) {
            double2 *yp = a.Y + (size_t)box * 8 + (size_t)col * a.ldy;
            const double2 *up = a.Ysub ? a.Ysub + (size_t)box * 8 + (size_t)col * a.ldsub : nullptr;
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const C v = s < 8 ? ya[s & 7] : yb[s & 7];
                double2 z = zc((double)v.x, (double)v.y);
                if (up) {
                    const double2 u = up[s];
                    z = zc(u.x - z.x, u.y - z.y);
                }
                yp[s] = z;
            }
        }
    } else {
        C x0[9], x1[9];
        if (CS != ADJ && a.X) {
            const unsigned box = leaf_box();
            const double2 *xp = a.X + (size_t)box * 8 + (size_t)col * a.ldx;
            C xa[8], xb[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const double2 u = xp[s], v = xp[8 + s];
                xa[s] = cmake<C>((T)u.x, (T)u.y);
                xb[s] = cmake<C>((T)v.x, (T)v.y);
            }
            const C *lf = leaf_tab(box);
            side_leaf_fwd<T, !CS>(a.mat, lf, xa, x0);
            load_fence();
            side_leaf_fwd<T, !CS>(a.mat, CS ? lf : lf + 1, xb, x1);
        } else {
            load(x0, x1);
        }
        grp.prefetch(table(0));
        if constexpr (!CS && !ADJ) {
            if (a.mid) side_apply_mid<T, false>(a, A, neg(), pair_in(), x0, x1);
        }
        levels(x0, x1);
        if constexpr (!CS && ADJ) {
            if (a.mid) side_apply_mid<T, true>(a, A, neg(), pair_in(), x0, x1);
        }
        if (act) {
            const size_t p0 = ADJ ? pair_in() : pair_out(), p1 = ADJ ? p0 + 1 : p0 + ((size_t)1 << lS);
            C *o0 = a.out + p0 * 9 * ld + col, *o1 = a.out + p1 * 9 * ld + col;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                o0[i * ld] = x0[i];
                o1[i * ld] = x1[i];
            }
        }
    }
}

// Leaf factors on their own.  A thread owns one (box, partner, column); IN writes the pair's
// coefficients, out sums the 8 partners of a box in order through LDS and writes rows.
// Pair of (box, partner): U side box 8 + partner, V side partner 2^L' + box.
template <typename T, bool USIDE> FIO_SIDE_FN const cpx<T> *leaf_entries(const SideArgs<T> &a, unsigned box, unsigned partner) {
    return USIDE ? a.LF + leaf_pos(box, partner) : a.LF + (partner * 2 + (box >> (a.Lp - 1))) * kSideEV;
}

template <typename T, bool USIDE>
__global__ void __launch_bounds__(256) k_side_leaf_in(SideArgs<T> a) {
    using C = cpx<T>;
    const unsigned tid = threadIdx.x, kc = a.kc, u = tid / kc, c = tid - u * kc;
    const unsigned chunk = blockIdx.x % a.nch, box = (blockIdx.x / a.nch) * a.nsb + (u >> 3), partner = u & 7u;
    const int col = chunk * kc + c;
    if (col >= a.nrhs) return;
    const double2 *xp = a.X + (size_t)box * 8 + (size_t)col * a.ldx;
    C x[8], v[9];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const double2 t = xp[s];
        x[s] = cmake<C>((T)t.x, (T)t.y);
    }
    side_leaf_fwd<T, USIDE>(a.mat, leaf_entries<T, USIDE>(a, box, partner), x, v);
    const size_t p = USIDE ? (size_t)box * 8 + partner : ((size_t)partner << a.Lp) + box, ld = a.nrhs;
    C *op = a.out + p * 9 * ld + col;
#pragma unroll
    for (int i = 0; i < 9; ++i) op[i * ld] = v[i];
}

template <typename T, bool USIDE>
__global__ void __launch_bounds__(256) k_side_leaf_out(SideArgs<T> a) {
    using C = cpx<T>;
    extern __shared__ double2 side_lds[];
    C *part = reinterpret_cast<C *>(side_lds);       // [unit][column][9], 8 rows used
    const unsigned tid = threadIdx.x, kc = a.kc, u = tid / kc, c = tid - u * kc;
    const unsigned chunk = blockIdx.x % a.nch, box0 = (blockIdx.x / a.nch) * a.nsb, box = box0 + (u >> 3),
                   partner = u & 7u;
    const int col0 = chunk * kc;
    const int col = col0 + (int)c < a.nrhs ? col0 + c : a.nrhs - 1;
    const size_t p = USIDE ? (size_t)box * 8 + partner : ((size_t)partner << a.Lp) + box, ld = a.nrhs;
    const C *ip = a.in + p * 9 * ld + col;
    C v[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) v[i] = ip[i * ld];
    C *pp = part + (size_t)tid * 9;
    side_leaf_bwd<T, USIDE>(a.mat, leaf_entries<T, USIDE>(a, box, partner), v, [&](int s, C y) { pp[s] = y; });
    __syncthreads();
    // one output row and column per thread, rows on consecutive lanes
    const unsigned nrow = (unsigned)a.nsb * 8, r = tid % nrow, cc = tid / nrow;
    if (col0 + (int)cc >= a.nrhs) return;
    const C *q = part + ((r >> 3) * 8 * kc + cc) * 9 + (r & 7u);
    C t = czero<C>();
#pragma unroll
    for (int k = 0; k < 8; ++k) t = cadd(t, q[k * kc * 9]);
    double2 z = zc((double)t.x, (double)t.y);
    const size_t row = (size_t)box0 * 8 + r;
    if (a.Ysub) {
        const double2 w = a.Ysub[row + (size_t)(col0 + cc) * a.ldsub];
        z = zc(w.x - z.x, w.y - z.y);
    }
    a.Y[row + (size_t)(col0 + cc) * a.ldy] = z;
}

// ---------------------------------------------------------------------------
// launchers
template <typename T> static SideArgs<T> side_args(const fio_bf_s *bf, bool cside, int nrhs) {
    const SideOff o = side_off(bf);
    const cpx<T> *t = reinterpret_cast<const cpx<T> *>(sizeof(T) == 8 ? bf->side64.p : bf->side32.p);
    if (!t) throw Err{FIO_ERR_ARG};
    SideArgs<T> a{};
    a.TW = t + (cside ? o.C : o.B);
    a.LF = t + (cside ? o.V : o.U);
    a.M = t + o.M;
    a.mat = reinterpret_cast<const T *>(t);
    a.mid = o.amp ? kSideEMamp : kSideEM;
    a.nrhs = nrhs;
    // columns per workgroup: at most 8 (see side_pass), the same for every chunk
    a.nch = (nrhs + 7) / 8;
    a.kc = (nrhs + a.nch - 1) / a.nch;
    a.L = bf->L;
    a.h = bf->h;
    a.Lp = bf->Lp;
    return a;
}

// nlev transfer levels of one side starting at level j0 of the side (counted from the leaf level on
// the C side, from level h on the B side; the adjoint runs them in the reverse order).  a.X: the pass
// starts from the input vectors (C forward, B adjoint); a.Y: it ends in the output vectors (B forward,
// C adjoint).
template <typename T>
static void side_pass(SideArgs<T> a, bool cside, bool adj, int j0, int nlev, hipStream_t s) {
    a.j0 = j0;
    a.kl = nlev;
    if (cside || j0 > 0) a.mid = 0;      // M follows the C side: before the first level of the B side
    const int G = 1 << (nlev - 1);
    // A shorter pass moves the coefficients more often and has threads to spare: 256 bytes of a row per workgroup
    // instead of 8 columns (as long as it has 256 threads).  One level per pass in FP32, 64 columns, N = 2^16 / 2^18:
    // 1430 / 6770 -> 1255 / 5810 us, three levels with the leaf factors apart 850 / 3510 -> 765 / 3140 us.
    const int cap = std::min((int)(256 / sizeof(cpx<T>)), 256 / G);
    if (nlev < a.Lp - a.h && cap > 8) {
        a.nch = (a.nrhs + cap - 1) / cap;
        a.kc = (a.nrhs + a.nch - 1) / a.nch;
    }
    // sub-butterflies per workgroup: enough for one full wave
    a.nsb = 1;
    while (a.nsb * G * a.kc < 64) a.nsb *= 2;
    a.nset = (int)((1L << (a.L - nlev - (a.Y ? 3 : 0))) / a.nsb);
    const unsigned block = (unsigned)(a.nsb * G * a.kc), grid = (unsigned)a.nset * a.nch;
    const size_t lds = nlev > 1 ? (size_t)block * 9 * sizeof(cpx<T>) : 0;
    FIO_TIMED(sizeof(T) == 8 ? (a.Y ? "bf_side_out_f64" : a.X ? "bf_side_in_f64" : "bf_side_f64")
                             : (a.Y ? "bf_side_out_f32" : a.X ? "bf_side_in_f32" : "bf_side_f32"), s);
    if (a.Y) {
        if (cside)
            k_side_pass<T, true, true, true><<<grid, block, lds, s>>>(a);
        else
            k_side_pass<T, false, false, true><<<grid, block, lds, s>>>(a);
    } else if (cside) {
        if (adj)
            k_side_pass<T, true, true, false><<<grid, block, lds, s>>>(a);
        else
            k_side_pass<T, true, false, false><<<grid, block, lds, s>>>(a);
    } else if (adj) {
        k_side_pass<T, false, true, false><<<grid, block, lds, s>>>(a);
    } else {
        k_side_pass<T, false, false, false><<<grid, block, lds, s>>>(a);
    }
    FIO_HIP(hipGetLastError());
}

// boxes per workgroup of the leaf kernels (a power of two) and their launch shape
template <typename T> static void leaf_shape(SideArgs<T> &a, unsigned &grid, unsigned &block) {
    a.nsb = 1;
    while (2 * a.nsb * 8 * a.kc <= 256) a.nsb *= 2;
    block = (unsigned)(a.nsb * 8 * a.kc);
    grid = (unsigned)((1L << a.Lp) / a.nsb) * a.nch;
}

template <typename T> static void side_leaf_in(SideArgs<T> a, bool uside, hipStream_t s) {
    unsigned grid, block;
    leaf_shape(a, grid, block);
    FIO_TIMED(sizeof(T) == 8 ? "bf_leaf_in_f64" : "bf_leaf_in_f32", s);
    if (uside)
        k_side_leaf_in<T, true><<<grid, block, 0, s>>>(a);
    else
        k_side_leaf_in<T, false><<<grid, block, 0, s>>>(a);
    FIO_HIP(hipGetLastError());
}

template <typename T> static void side_leaf_out(SideArgs<T> a, bool uside, hipStream_t s) {
    unsigned grid, block;
    leaf_shape(a, grid, block);
    const size_t lds = (size_t)block * 9 * sizeof(cpx<T>);
    FIO_TIMED(sizeof(T) == 8 ? "bf_leaf_out_f64" : "bf_leaf_out_f32", s);
    if (uside)
        k_side_leaf_out<T, true><<<grid, block, lds, s>>>(a);
    else
        k_side_leaf_out<T, false><<<grid, block, lds, s>>>(a);
    FIO_HIP(hipGetLastError());
}

template <typename T>
void side_apply(const fio_bf_s *bf, bool adj, const double2 *X, long ldx, double2 *Y, long ldy, int nrhs, cpx<T> *c0,
                cpx<T> *c1, int kmax, bool leaf_sep, const double2 *Ysub, long ldsub, hipStream_t s) {
    const int nl = bf->nl;
    cpx<T> *cur = c0, *nxt = c1;
    int step = kSideMaxLevels;
    if (kmax > 0 && kmax < step) step = kmax;
    if (kmax == 0) {
        const int parts = (nl + step - 1) / step;
        step = (nl + parts - 1) / parts;
    }
    // forward C^[L'] .. C^[h+1], M, B^[h+1] .. B^[L']; adjoint B^[L']* .. B^[h+1]*, M*, C^[h+1]* .. C^[L']*:
    // both run a first side from the leaves to level h and a second one back
    SideArgs<T> a = side_args<T>(bf, !adj, nrhs), o = side_args<T>(bf, adj, nrhs);
    a.X = X;
    a.ldx = ldx;
    o.ldy = ldy;
    o.Ysub = Ysub;
    o.ldsub = ldsub;
    if (leaf_sep) {
        a.out = cur;
        side_leaf_in<T>(a, adj, s);
        a.X = nullptr;
    }
    for (int done = 0; done < nl;) {
        const int n = nl - done < step ? nl - done : step;
        a.in = cur;
        a.out = nxt;
        side_pass<T>(a, !adj, adj, adj ? nl - done - n : done, n, s);
        a.X = nullptr;
        std::swap(cur, nxt);
        done += n;
    }
    // The second side in one pass can end in the output rows itself: its workgroups then run the 8
    // coarse partners in turn, so it needs enough of them to keep the card busy.  Measured in-pass against
    // a leaf kernel of its own (FP64 / FP32 ms of an apply, 64 columns unless noted): adjoint N = 2^18 3.42 /
    // 1.80 against 4.02 / 2.08, 2^16 0.78 / 0.43 against 0.84 / 0.49, 2^18 with 16 columns (1024 workgroups)
    // 0.88 / 0.50 against 0.96 / 0.53, 2^14 (4 levels, 1024 one-wave workgroups) 0.20 / 0.13 against 0.21 / 0.12,
    // the same: hence at least 5 levels; forward 2^18 3.49 / 1.83 against 3.60 / 2.01, 2^16 (2048 workgroups)
    // 0.87 / 0.46 against 0.80 / 0.46, 2^18 with 32 columns 1.80 / 0.94 against 1.78 / 1.01.  The in-pass forms
    // hold 16 row sums beside the two pairs and spill: forward 99 registers a lane in FP64 and 30 in FP32, adjoint
    // 75 and 10 (of the others, the FP64 adjoint B side 14 and the FP32 forward B side 4).
    // With an amplitude the FP32 forward one also reads two blocks of 81 entries per partner and column chunk: 2^16
    // with 64 / 150 columns 0.91 / 1.83 against 0.54 / 1.33, 2^18 3.17 against 2.29: never.
    const long groups = ((long)1 << bf->h) * o.nch;
    const bool out = !leaf_sep && step >= nl && nl >= 5 && groups >= (adj ? 1024 : sizeof(T) == 8 ? 4096 : 2048) &&
                     (adj || sizeof(T) == 8 || o.mid != kSideEMamp);
    for (int done = 0; done < nl;) {
        const int n = nl - done < step ? nl - done : step;
        o.in = cur;
        o.out = nxt;
        o.Y = out ? Y : nullptr;
        side_pass<T>(o, adj, adj, adj ? nl - done - n : done, n, s);
        std::swap(cur, nxt);
        done += n;
    }
    if (!out) {
        o.in = cur;
        o.Y = Y;
        side_leaf_out<T>(o, !adj, s);
    }
}

#define FIO_SIDE_INST(T)                                                                                        \
    template void side_apply<T>(const fio_bf_s *, bool, const double2 *, long, double2 *, long, int, cpx<T> *,  \
                                cpx<T> *, int, bool, const double2 *, long, hipStream_t);
FIO_SIDE_INST(double)
FIO_SIDE_INST(float)
#undef FIO_SIDE_INST

}  // namespace fio
