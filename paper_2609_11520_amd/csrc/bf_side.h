// Side passes of the 1D structured butterfly (q = 9): the tables they read and their launchers.
//
// On a frequency half line the phase is linear in xi: Phi(x, xi) = kappa(x) xi with
// kappa(x) = x + sgn c(x).  With the coefficients of every pair rescaled by unit factors,
//   C side, pair (tau, sigma):  c_j = exp(-2 pi i kappa(y_tau) (gamma_j - eta_sigma)) chat_j,
//   B side, pair (tau, sigma):  chat_i = exp(-2 pi i kappa(z_tau,i) eta_sigma) c_i,
// the factors of eq. bf become
//   V: chat_j = sum_s P(s, j) exp(2 pi i kappa(y_tau) (xi_s - eta_sigma)) f_s,
//   C: chat_j = sum_(c_in, t) P_(c_in)(t, j) b(c_in, t) chat_(beta, t),  with, for the parent alpha of tau,
//      b(0, t) = exp(2 pi i ((kappa(y_tau) - kappa(y_alpha)) (w/2) t_t - kappa(y_tau) w/2)), w the width of
//      beta, and b(1, q-1-t) = conj(b(0, t)),
//   M: chat_i = sum_j Y_ij chat_j, Y_ij = a exp(2 pi i (kappa(z_i) - kappa(y_tau)) (w/2) t_j); for a = 1
//      Y_i,4 = 1 and Y_i,q-1-j = conj(Y_ij),
//   B: chat_i = sum_(c_in) a(c_in, i) sum_t P_(c_out)(i, t) chat_(beta, t),
//      a(0, i) = exp(-2 pi i kappa(z_tau,i) w/2) = conj(a(1, i)),
//   U: y_s = sum_sigma exp(2 pi i Phi(x_s, eta_sigma)) sum_i P(s, i) chat_i
// (P_c, P: the Lagrange values of child and leaf points).  The transfer and middle diagonals depend on
// the spatial box and the sign of the frequency only, not on the pair: all tables together are small
// enough for the caches, so a pass moves little more than its coefficients.
#pragma once
#include "bf.h"

namespace fio {

constexpr int kSideQ = 9;
constexpr int kSideHead = 60;      // 81 + 36 real matrix entries (see gen_side_head), as complex entries
constexpr int kSideRow = 10;       // complex entries per (box, sign) of a transfer table, 9 used
constexpr int kSideEV = 4;         // V: exp(2 pi i kappa d), d = 1, 2, 3, -4, per (coarse box, sign)
constexpr int kSideEU = 8;         // U: exp(2 pi i Phi(x_s, eta)), per (leaf box, coarse partner)
constexpr int kSideEM = 36;        // M for a = 1: Y_ij, j < 4, per (box, sign)
constexpr int kSideEMamp = 81;     // M with a variable amplitude: per pair
constexpr int kSideMaxLevels = 6;  // levels per pass: a workgroup of 256 threads holds 2^6 pairs x 8 columns

// element offsets of the tables of a handle
struct SideOff {
    size_t V, C, M, B, U, total;
    bool amp;
};
SideOff side_off(const fio_bf_s *bf);
bool side_built(const fio_bf_s *bf);
void side_generate(fio_bf_s *bf, hipStream_t s);          // FP64 tables
void side_make_f32(fio_bf_s *bf, hipStream_t s);          // their FP32 copy

// A whole apply: Y = K~ X or K~^* X (with Ysub: Y = Ysub - K~ X) through the coefficient buffers c0,
// c1.  kmax: at most that many levels per pass (0: kSideMaxLevels), leaf_sep: the leaf factors as
// their own kernels; the result is bitwise the same for every choice and column count.
template <typename T>
void side_apply(const fio_bf_s *bf, bool adj, const double2 *X, long ldx, double2 *Y, long ldy, int nrhs, cpx<T> *c0,
                cpx<T> *c1, int kmax, bool leaf_sep, const double2 *Ysub, long ldsub, hipStream_t s);

}  // namespace fio
