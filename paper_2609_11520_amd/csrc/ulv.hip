// ULV factorization of an HPD HSS matrix and its solve (Section 2.4) on gfx950.
//
// Factor (offline, level by level from the leaves):
//   QL basis elimination U = Q [0; Uhat2] with Householder reflectors taken from
//   the bottom of each column; Dchk = Q^* D Q; Cholesky Dchk11 = L11 L11^*;
//   Dhat21 = Dchk21 L11^{-*}; Dhat22 = Dchk22 - Dhat21 Dhat21^*; then the merge
//   of eq. ulv_merge for every parent and a Cholesky of the root block.
// The two solve sweeps of Section 2.4 are stored per node as one m x m matrix
//   W = [L11^{-1} Q1^*; Q2^* - Dhat21 L11^{-1} Q1^*]
// so that the bottom-up step is [bhat1; yhat2] = W y_tau and the top-down step is
// c_tau = W^* [bhat1; chat2]; the root keeps Linv = L_rho^{-1}.  The online solve
// is therefore one batched product per level and direction (k_ulv_leaf for leaves of up to 64 rows,
// k_ulv_mm for larger nodes, k_ulv_wide for wide blocks and many nodes), with the levels of small nodes
// in bands of up to four (k_ulv_band).
#include "hss.h"
#include "hss_qr.h"
#include "mat4.h"
#include "timing.h"

#include <cmath>
#include <cstring>

struct hss_ulv_s {
    long N = 0;
    int leaf = 0, Lh = 0, m0 = 0;
    std::vector<std::vector<int>> m, k, r;      // per level (1..Lh)
    std::vector<std::vector<size_t>> woff;
    std::vector<std::vector<long>> yoff, roff;  // rows of a node in its level vector / parent vector
    std::vector<long> rows;                     // rows of the level-l vector (l = 0..Lh)
    fio::DevBuf W;                              // all W slots
    fio::DevBuf Linv;                           // m0 x m0
    fio::DevBuf meta;                           // device copies of the per-level tables
    std::vector<size_t> meta_woff, meta_m, meta_k, meta_yoff, meta_roff;   // byte offsets into meta
    fio::DevBuf ws;
    std::mutex ws_mu;
};

namespace fio {

constexpr int kUlvMaxM = 2048;   // largest node size of the factorization
// one workgroup per node; large nodes (upper levels of 2D trees) get 16 waves
inline unsigned ulv_threads(int m) { return m >= 192 ? 1024u : 256u; }

__device__ __forceinline__ double wsum(double v, double *sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
    return t;
}

// In-place Cholesky (lower) of the leading n x n block of A (column-major, lda).
// Returns false (on every thread) when a pivot is not positive.
__device__ bool wg_potrf(double2 *A, int lda, int n, double *sh, int *s_flag) {
    const int tid = threadIdx.x, nt = blockDim.x;
    if (tid == 0) *s_flag = 0;
    __syncthreads();
    for (int c = 0; c < n; ++c) {
        double d = A[c + (size_t)c * lda].x;
        if (!(d > 0.0) || !isfinite(d)) {
            if (tid == 0) *s_flag = 1;
            __syncthreads();
            return false;
        }
        d = sqrt(d);
        __syncthreads();
        for (int i = c + tid; i < n; i += nt) {
            double2 v = A[i + (size_t)c * lda];
            A[i + (size_t)c * lda] = i == c ? zc(d, 0.0) : zc(v.x / d, v.y / d);
        }
        __syncthreads();
        // trailing update of the lower triangle: A(i, j) -= L(i, c) conj(L(j, c)), c < j <= i
        const int rem = n - c - 1;
        for (int e = tid; e < rem * rem; e += nt) {
            int i = c + 1 + e % rem, j = c + 1 + e / rem;
            if (j > i) continue;
            double2 li = A[i + (size_t)c * lda], lj = A[j + (size_t)c * lda];
            double2 &a = A[i + (size_t)j * lda];
            a.x -= li.x * lj.x + li.y * lj.y;
            a.y -= li.y * lj.x - li.x * lj.y;
        }
        __syncthreads();
    }
    // clear the strict upper triangle (not part of L)
    for (int e = tid; e < n * n; e += nt) {
        int i = e % n, j = e / n;
        if (j > i) A[i + (size_t)j * lda] = zc(0.0, 0.0);
    }
    __syncthreads();
    (void)sh;
    return true;
}

struct FactArgs {
    // inputs per node of the level
    const double2 *D;       // node diagonal blocks
    const size_t *doff;
    const double2 *U;       // node bases
    const size_t *uoff;
    const int *msz, *rsz;
    // outputs
    double2 *W;             // m x m per node
    const size_t *woff;
    double2 *D22;           // r x r per node (slot m x m)
    double2 *U2;            // r x r per node (slot m x m)
    const size_t *soff;
    double2 *scratch;       // 3 m^2 per node
    const size_t *scoff;
    int *fail;
};

// Basis elimination, partial Cholesky and the node's W (one workgroup per node), in two
// phases around the two dense products Dchk = Q^* D Q, which run as batched GEMMs over
// all nodes of the level:
//   PHASE 0: QL of U_tau (Householder), explicit Q, the reduced basis U2;
//   PHASE 1: Cholesky of Dchk11, Dhat21, Dhat22 and W = [L11^{-1} Q1^*; Q2^* - Dhat21 L11^{-1} Q1^*].
template <int PHASE>
__global__ void __launch_bounds__(1024) k_ulv_node(FactArgs a) {
    __shared__ double sh[16];
    __shared__ double s_tau[kUlvMaxM];
    __shared__ int s_flag;
    const int node = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int m = a.msz[node], r = a.rsz[node], k = m - r;
    if (m == 0) return;
    double2 *Uw = a.scratch + a.scoff[node];        // m x r working copy, then reflectors
    double2 *Q = Uw + (size_t)m * m;                 // m x m explicit Q
    double2 *T = Q + (size_t)m * m;                  // m x m: Dchk = Q^* D Q (batched GEMMs)
    const double2 *Uin = a.U + a.uoff[node];
    double2 *Wm = a.W + a.woff[node];
    if constexpr (PHASE == 0) {
        for (int e = tid; e < m * r; e += nt) Uw[e] = Uin[e];
        __syncthreads();
        // QL: for column jj = r-1..0 eliminate rows 0..p-1 (p = k + jj) into row p
        for (int jj = r - 1; jj >= 0; --jj) {
            const int p = k + jj, n = p + 1;
            double2 *x = Uw + (size_t)jj * m;            // rows 0..p
            const double2 al = x[p];
            double part = 0.0;
            for (int i = tid; i < n; i += nt) part += x[i].x * x[i].x + x[i].y * x[i].y;
            const double sigma = sqrt(wsum(part, sh));
            double tau = 0.0;
            if (sigma != 0.0) {                  // a NaN goes on into every column
                const double aa = sqrt(al.x * al.x + al.y * al.y);
                double2 ph = aa > 0.0 ? zc(al.x / aa, al.y / aa) : zc(1.0, 0.0);
                double2 beta = zc(-ph.x * sigma, -ph.y * sigma);
                double2 den = csub(al, beta);
                double dn = den.x * den.x + den.y * den.y;
                double2 inv = zc(den.x / dn, -den.y / dn);
                for (int i = tid; i < p; i += nt) x[i] = cmul(x[i], inv);
                __syncthreads();
                if (tid == 0) x[p] = beta;
                tau = 1.0 + aa / sigma;
            }
            if (tid == 0) s_tau[jj] = tau;
            __syncthreads();
            // apply H = I - tau v v^*, v = [x[0..p); 1], to columns 0..jj-1 (rows 0..p)
            if (tau != 0.0) {
                for (int c = tid; c < jj; c += nt) {
                    double2 *col = Uw + (size_t)c * m;
                    double2 w = col[p];
                    for (int i = 0; i < p; ++i) cfmac(w, x[i], col[i]);
                    double2 tw = zc(tau * w.x, tau * w.y);
                    col[p] = csub(col[p], tw);
                    for (int i = 0; i < p; ++i) col[i] = csub(col[i], cmul(x[i], tw));
                }
            }
            __syncthreads();
        }
        // Q = H_{r-1} ... H_0 I: apply H_0 first
        for (int e = tid; e < m * m; e += nt) Q[e] = zc((e % m) == (e / m) ? 1.0 : 0.0, 0.0);
        __syncthreads();
        for (int jj = 0; jj < r; ++jj) {
            const double tau = s_tau[jj];
            if (tau == 0.0) continue;
            const int p = k + jj;
            const double2 *x = Uw + (size_t)jj * m;
            for (int c = tid; c < m; c += nt) {
                double2 *col = Q + (size_t)c * m;
                double2 w = col[p];
                for (int i = 0; i < p; ++i) cfmac(w, x[i], col[i]);
                double2 tw = zc(tau * w.x, tau * w.y);
                col[p] = csub(col[p], tw);
                for (int i = 0; i < p; ++i) col[i] = csub(col[i], cmul(x[i], tw));
            }
            __syncthreads();
        }
        // Uhat2: rows k..m-1 of the transformed U (lower triangular r x r: entries j >= i of the
        // reflector-free part); the transformed U is [0; L] with L(i, c) at row k + i, column c
        double2 *U2 = a.U2 + a.soff[node];
        for (int e = tid; e < r * r; e += nt) {
            int i = e % r, c = e / r;
            U2[e] = (c <= i) ? Uw[(k + i) + (size_t)c * m] : zc(0.0, 0.0);
        }
        return;
    }
    // T holds Dchk = (Q^* D) Q (the W slot held Q^* D); Cholesky of Dchk11 (k x k) in place
    if (!wg_potrf(T, m, k, sh, &s_flag)) {
        if (tid == 0) atomicAdd(a.fail, 1);
        return;
    }
    // X = Dhat21^* = L11^{-1} Dchk12 (k x r; Dchk is Hermitian, so Dchk12 = Dchk21^*), in place
    // in T(0..k, k..m), forward substitution per column
    for (int c = tid; c < r; c += nt) {
        double2 *col = T + (size_t)(k + c) * m;
        for (int i = 0; i < k; ++i) {
            double2 acc = col[i];
            for (int l = 0; l < i; ++l) acc = csub(acc, cmul(T[i + (size_t)l * m], col[l]));
            const double d = T[i + (size_t)i * m].x;
            col[i] = zc(acc.x / d, acc.y / d);
        }
    }
    // Dhat22 starts as Dchk22; the level's batched GEMM subtracts X^* X
    double2 *D22 = a.D22 + a.soff[node];
    for (int e = tid; e < r * r; e += nt) {
        const int i = e % r, j = e / r;
        D22[e] = T[(k + i) + (size_t)(k + j) * m];
    }
    // W1 = L11^{-1} Q1^* (k x m), forward substitution per column c of Q1^*
    for (int c = tid; c < m; c += nt) {
        for (int i = 0; i < k; ++i) {
            double2 q = Q[c + (size_t)i * m];            // Q1^*(i, c) = conj(Q(c, i))
            double2 acc = zc(q.x, -q.y);
            for (int l = 0; l < i; ++l) {
                double2 t = cmul(T[i + (size_t)l * m], Wm[l + (size_t)c * m]);
                acc = csub(acc, t);
            }
            double d = T[i + (size_t)i * m].x;
            Wm[i + (size_t)c * m] = zc(acc.x / d, acc.y / d);
        }
    }
    // W2 starts as Q2^* (r x m); the level's batched GEMM subtracts X^* W1 (= Dhat21 W1)
    for (int e = tid; e < r * m; e += nt) {
        const int i = e % r, c = e / r;
        const double2 q = Q[c + (size_t)(k + i) * m];
        Wm[(k + i) + (size_t)c * m] = zc(q.x, -q.y);
    }
}

// ---------------------------------------------------------------------------
// Levels of larger nodes: the same two phases spread over the card.
//
// Phase 0: with the rows and columns of U in reverse order the QL elimination is a QR, and Q is the
// product of its reflectors applied to the identity: both run in the blocks of hss_qr.h.
// Phase 1: Dchk11 = L11 L11^*, X = L11^{-1} Dchk12 and W1 = L11^{-1} Q1^* are one forward
// substitution on the rows [Dchk11 Dchk12 | Q1^*] (the rows of Dchk11 become L11^*), 32 rows a step:
// k_fact_diag brings the diagonal block up to date and factors it, k_fact_rows the rest of the rows.
// Both are chains of small dependent steps on data in cache.  With a launch per reflector and one
// workgroup per node for the substitutions the factorization of 2D n = 64 (nodes of 64 to 784 rows, a
// root of 832) took 212 ms, with these kernels 29.6 ms.
struct TriNode {
    double2 *T, *W;         // m x m each: the matrix and the right-hand sides of its row sweep
    int m, k;               // k rows are factored
};

constexpr int kFact = 32;

// Uw <- U in reverse order (m x r), T <- I
__global__ void k_ubig_init(FactArgs a) {
    const int node = blockIdx.y, m = a.msz[node], r = a.rsz[node];
    if (m == 0) return;
    double2 *Uw = a.scratch + a.scoff[node], *T = Uw + (size_t)2 * m * m;
    const double2 *Uin = a.U + a.uoff[node];
    for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < (long)m * m; e += (long)gridDim.x * blockDim.x) {
        const int i = (int)(e % m), j = (int)(e / m);
        if (j < r) Uw[e] = Uin[(m - 1 - i) + (size_t)(r - 1 - j) * m];
        T[e] = zc(i == j ? 1.0 : 0.0, 0.0);
    }
}

// Q and Uhat2 back in order
__global__ void k_ubig_finish(FactArgs a) {
    const int node = blockIdx.y, m = a.msz[node], r = a.rsz[node];
    if (m == 0) return;
    const double2 *Uw = a.scratch + a.scoff[node], *T = Uw + (size_t)2 * m * m;
    double2 *Q = a.scratch + a.scoff[node] + (size_t)m * m, *U2 = a.U2 + a.soff[node];
    for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < (long)m * m; e += (long)gridDim.x * blockDim.x) {
        Q[e] = T[(size_t)m * m - 1 - e];
        if (e < (long)r * r) {
            const int i = (int)(e % r), c = (int)(e / r);
            U2[e] = c <= i ? Uw[(r - 1 - i) + (size_t)(r - 1 - c) * m] : zc(0.0, 0.0);
        }
    }
}

// W <- Q^*, D22 <- Dchk22, one 32 x 32 tile per workgroup
__global__ void __launch_bounds__(256) k_fact_prep(FactArgs a) {
    __shared__ double2 t[32][33];
    const int node = blockIdx.z, m = a.msz[node], r = a.rsz[node], k = m - r;
    const int i0 = blockIdx.x * 32, j0 = blockIdx.y * 32;
    if (i0 >= m || j0 >= m) return;
    const double2 *Q = a.scratch + a.scoff[node] + (size_t)m * m, *T = Q + (size_t)m * m;
    double2 *W = a.W + a.woff[node], *D22 = a.D22 + a.soff[node];
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
    for (int q = y; q < 32; q += 8)
        if (i0 + x < m && j0 + q < m) {
            const double2 v = Q[i0 + x + (size_t)(j0 + q) * m];
            t[q][x] = zc(v.x, -v.y);
            const int i = i0 + x - k, j = j0 + q - k;
            if (i >= 0 && j >= 0) D22[i + (size_t)j * r] = T[i0 + x + (size_t)(j0 + q) * m];
        }
    __syncthreads();
    for (int q = y; q < 32; q += 8)
        if (j0 + x < m && i0 + q < m) W[j0 + x + (size_t)(i0 + q) * m] = t[x][q];
}

// 32 x 32 tile sum over rows l0 <= l < l1 of conj(R(l, rows)) X(l, columns); R has nb columns, X nc
__device__ __forceinline__ void fact_tile(const double2 *R, const double2 *X, int m, int l0, int l1, int nb, int nc,
                                          double2 (*As)[33], double2 (*Bs)[33], double2 (&acc)[2][2]) {
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = zc(0.0, 0.0);
    for (int l = l0; l < l1; l += 16) {
        double2 ta[2], tb[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = tid + 256 * q, kk = l + (e & 15), c = e >> 4;
            const bool oa = kk < l1 && c < nb, ob = kk < l1 && c < nc;
            ta[q] = R[(oa ? kk : 0) + (size_t)(oa ? c : 0) * m];
            tb[q] = X[(ob ? kk : 0) + (size_t)(ob ? c : 0) * m];
            if (!oa) ta[q] = zc(0.0, 0.0);
            if (!ob) tb[q] = zc(0.0, 0.0);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = tid + 256 * q;
            As[e & 15][e >> 4] = zc(ta[q].x, -ta[q].y);
            Bs[e & 15][e >> 4] = tb[q];
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            const double2 a0 = As[kk][tx], a1 = As[kk][tx + 16], b0 = Bs[kk][ty], b1 = Bs[kk][ty + 16];
            cfma(acc[0][0], a0, b0);
            cfma(acc[0][1], a0, b1);
            cfma(acc[1][0], a1, b0);
            cfma(acc[1][1], a1, b1);
        }
    }
}

// Diagonal block k0 of a node: R_kk (upper, R_kk^* R_kk = the updated block) into T and R_kk^{-*} into
// Li.  The elimination runs on [block | I] in registers: thread (column, row mod 4), one barrier per row.
__global__ void __launch_bounds__(256) k_fact_diag(const TriNode *__restrict__ nodes, int k0, double2 *Li, int *fail) {
    __shared__ double2 As[16][33], Bs[16][33], Cs[kFact][kFact + 1];
    __shared__ double2 row[2][64];
    const TriNode d = nodes[blockIdx.x];
    if (k0 >= d.k) return;
    const int m = d.m, nb = d.k - k0 < kFact ? d.k - k0 : kFact, tid = threadIdx.x;
    double2 *T = d.T + (size_t)k0 * m;
    double2 acc[2][2];
    fact_tile(T, T, m, 0, k0, nb, nb, As, Bs, acc);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int i = (tid & 15) + 16 * u, j = (tid >> 4) + 16 * v;
            double2 c = zc(i == j ? 1.0 : 0.0, 0.0);
            if (i < nb && j < nb) c = csub(T[k0 + i + (size_t)j * m], acc[u][v]);
            Cs[i][j] = c;
        }
    __syncthreads();
    const int j = tid & 63, w = tid >> 6;
    double ax[8], ay[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int i = w + 4 * q;
        const double2 c = j < kFact ? Cs[i][j & 31] : zc(j - kFact == i ? 1.0 : 0.0, 0.0);
        ax[q] = c.x;
        ay[q] = c.y;
    }
    bool bad = false;
#pragma unroll
    for (int c = 0; c < kFact; ++c) {
        if ((c & 3) == w) {
            double p = __shfl(ax[c >> 2], c);
            if (!(p > 0.0) || !isfinite(p)) {
                bad = true;
                p = 1.0;
            }
            p = sqrt(p);
            ax[c >> 2] /= p;
            ay[c >> 2] = j == c ? 0.0 : ay[c >> 2] / p;
            row[c & 1][j] = zc(ax[c >> 2], ay[c >> 2]);
        }
        __syncthreads();
        const double2 rj = row[c & 1][j];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = w + 4 * q;
            if (4 * q + 3 > c) {
                const double2 ri = row[c & 1][i];
                if (i > c) {
                    ax[q] -= ri.x * rj.x + ri.y * rj.y;
                    ay[q] -= ri.x * rj.y - ri.y * rj.x;
                }
            }
        }
    }
    if (bad && j == 0) atomicAdd(fail, 1);
    double2 *O = Li + (size_t)blockIdx.x * kFact * kFact;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int i = w + 4 * q;
        if (j >= kFact)
            O[i + (j - kFact) * kFact] = zc(ax[q], ay[q]);
        else if (i <= j && j < nb)
            T[k0 + i + (size_t)j * m] = zc(ax[q], ay[q]);
    }
}

// The other columns of rows k0 .. k0 + 31 of [T | W], 32 columns per workgroup.  UNIT: W started as
// the identity, so that only its columns up to the block are not zero.
template <bool UNIT>
__global__ void __launch_bounds__(256) k_fact_rows(const TriNode *__restrict__ nodes, int k0,
                                                  const double2 *__restrict__ Li) {
    __shared__ double2 As[16][33], Bs[16][33], Cs[kFact][kFact + 1], Ls[kFact][kFact + 1];
    const TriNode d = nodes[blockIdx.y];
    if (k0 >= d.k) return;
    const int m = d.m, nb = d.k - k0 < kFact ? d.k - k0 : kFact, tid = threadIdx.x;
    const int ct = m - k0 - nb, nt = (ct + 31) / 32;
    const bool inT = (int)blockIdx.x < nt;
    const int c0 = inT ? k0 + nb + 32 * blockIdx.x : 32 * (blockIdx.x - nt), cend = inT ? m : UNIT ? k0 + nb : m;
    if (c0 >= cend) return;
    const int nc = cend - c0 < 32 ? cend - c0 : 32;
    double2 *X = (inT ? d.T : d.W) + (size_t)c0 * m;
    for (int e = tid; e < kFact * kFact; e += 256) Ls[e / kFact][e % kFact] = Li[(size_t)blockIdx.y * kFact * kFact + e];
    double2 acc[2][2];
    fact_tile(d.T + (size_t)k0 * m, X, m, UNIT && !inT ? c0 : 0, k0, nb, nc, As, Bs, acc);
    const int tx = tid & 15, ty = tid >> 4;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int i = tx + 16 * u, j = ty + 16 * v;
            double2 c = zc(0.0, 0.0);
            if (i < nb && j < nc) c = csub(X[k0 + i + (size_t)j * m], acc[u][v]);
            Cs[i][j] = c;
        }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int i = tx + 16 * u, j = ty + 16 * v;
            if (i >= nb || j >= nc) continue;
            double2 x = zc(0.0, 0.0);
            for (int l = 0; l <= i; ++l) cfma(x, Ls[l][i], Cs[l][j]);
            X[k0 + i + (size_t)j * m] = x;
        }
}

// device buffers of the level steps, kept over the levels of a factorization
struct UlvWork {
    WyWork wy;
    DevBuf Li;
    Uploads up;
    explicit UlvWork(hipStream_t s) : up(s) {}
};

// the row sweep over all nodes of a list (mmax, kmax: the largest m and k)
static void fact_sweep(const std::vector<TriNode> &nodes, int mmax, int kmax, bool unit, int *fail, UlvWork &w,
                       hipStream_t s) {
    const unsigned nn = (unsigned)nodes.size();
    w.Li.ensure((size_t)nn * kFact * kFact * sizeof(double2));
    const TriNode *d = w.up.put(nodes);
    w.up.flush();
    double2 *Li = w.Li.as<double2>();
    for (int k0 = 0; k0 < kmax; k0 += kFact) {
        k_fact_diag<<<nn, 256, 0, s>>>(d, k0, Li, fail);
        // a node with few rows left in this block has more columns to its right
        const unsigned tiles = (unsigned)((mmax - k0 + 31) / 32 + ((unit ? k0 + kFact : mmax) + 31) / 32);
        if (unit)
            k_fact_rows<true><<<dim3(tiles, nn), 256, 0, s>>>(d, k0, Li);
        else
            k_fact_rows<false><<<dim3(tiles, nn), 256, 0, s>>>(d, k0, Li);
    }
    FIO_HIP(hipGetLastError());
}

// Levels whose largest node has at least this many rows take these kernels: with 1024 leaves of 64 rows (N = 2^16)
// the factorization takes 3.87 ms with them and 4.84 ms with one workgroup per node, for 2D n = 64 29.6 and
// 30.6 ms (54.6 from 256 rows on); the levels of 8 rows above the leaves of 1D trees lose with them (4.46 ms).
constexpr int kUlvBig = 64;
static int g_ulv_big = kUlvBig;

static void ulv_phase0_big(const FactArgs &fa, const std::vector<int> &ms, const std::vector<int> &rs,
                           const std::vector<size_t> &scoff, UlvWork &w, hipStream_t s) {
    const unsigned y = (unsigned)ms.size();
    k_ubig_init<<<dim3(16, y), 256, 0, s>>>(fa);
    std::vector<WyNode> un(ms.size()), qn(ms.size());
    for (size_t j = 0; j < ms.size(); ++j) {
        double2 *Uw = fa.scratch + scoff[j];
        un[j] = WyNode{Uw, Uw, ms[j], ms[j], ms[j], rs[j], rs[j]};
        qn[j] = WyNode{Uw, Uw + (size_t)2 * ms[j] * ms[j], ms[j], ms[j], ms[j], rs[j], ms[j]};
    }
    wy_qr(un, w.wy, w.up, s);
    wy_apply(qn, w.wy, true, w.up, s);
    k_ubig_finish<<<dim3(16, y), 256, 0, s>>>(fa);
    FIO_HIP(hipGetLastError());
}

static void ulv_phase1_big(const FactArgs &fa, const std::vector<int> &ms, const std::vector<int> &rs,
                           const std::vector<size_t> &scoff, const std::vector<size_t> &woff, UlvWork &w,
                           hipStream_t s) {
    std::vector<TriNode> tn(ms.size());
    int mmax = 0, kmax = 0;
    for (size_t j = 0; j < ms.size(); ++j) {
        tn[j] = TriNode{fa.scratch + scoff[j] + (size_t)2 * ms[j] * ms[j], fa.W + woff[j], ms[j], ms[j] - rs[j]};
        mmax = ms[j] > mmax ? ms[j] : mmax;
        kmax = tn[j].k > kmax ? tn[j].k : kmax;
    }
    const unsigned t = (unsigned)((mmax + 31) / 32);
    k_fact_prep<<<dim3(t, t, (unsigned)ms.size()), 256, 0, s>>>(fa);
    fact_sweep(tn, mmax, kmax, false, fa.fail, w, s);
}

// Merge of eq. ulv_merge for every parent (one workgroup per parent):
//   D+ = [[D22(a1), (U2(a2) B U2(a1)^*)^*], [U2(a2) B U2(a1)^*, D22(a2)]],
//   U+ = diag(U2(a1), U2(a2)) U_parent  (skipped at the root).
struct MergeArgs {
    const double2 *D22, *U2;
    const size_t *soff;      // child slots
    const int *rch;          // child ranks
    const double2 *B;        // B_{a2,a1} of each parent
    const size_t *boff;
    const double2 *Upar;     // parent bases (m x r_par slots), or null at the root
    const size_t *upoff;
    const int *rpar;
    double2 *Dout;           // merged D (m x m per parent)
    const size_t *dooff;
    double2 *Uout;           // merged U (m x r_par per parent)
    const size_t *uooff;
    double2 *tmp;            // per parent: T (r2 x r1), then U2(a1)^* (r1 x r1)
    const size_t *toff;
};

// Merge, around four batched GEMMs over the parents of the level:
//   k_ulv_merge_prep: diagonal blocks D22(a1), D22(a2) into D+, and U2(a1)^* next to T;
//   GEMMs: T = U2(a2) B, lower-left block of D+ = T U2(a1)^*, U+ = diag(U2(a1), U2(a2)) U_parent;
//   k_ulv_merge_fill: upper-right block of D+ = conj transpose of the lower-left block.
__global__ void __launch_bounds__(1024) k_ulv_merge_prep(MergeArgs a) {
    const int par = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int c1 = 2 * par, c2 = 2 * par + 1;
    const int r1 = a.rch[c1], r2 = a.rch[c2], m = r1 + r2;
    if (m == 0) return;
    const double2 *Da = a.D22 + a.soff[c1], *Db = a.D22 + a.soff[c2];
    const double2 *Ua = a.U2 + a.soff[c1];
    double2 *UaH = a.tmp + a.toff[par] + (size_t)r1 * r2;
    double2 *D = a.Dout + a.dooff[par];
    for (int e = tid; e < r1 * r1; e += nt) {
        const int i = e % r1, j = e / r1;
        D[i + (size_t)j * m] = Da[e];
        const double2 u = Ua[j + (size_t)i * r1];
        UaH[e] = zc(u.x, -u.y);
    }
    for (int e = tid; e < r2 * r2; e += nt) {
        const int i = e % r2, j = e / r2;
        D[(r1 + i) + (size_t)(r1 + j) * m] = Db[e];
    }
}

__global__ void __launch_bounds__(1024) k_ulv_merge_fill(MergeArgs a) {
    const int par = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int r1 = a.rch[2 * par], r2 = a.rch[2 * par + 1], m = r1 + r2;
    double2 *D = a.Dout + a.dooff[par];
    for (int e = tid; e < r1 * r2; e += nt) {
        const int i = e % r1, j = e / r1;          // upper-right (i, r1 + j) = conj(lower-left (r1 + j, i))
        const double2 v = D[(r1 + j) + (size_t)i * m];
        D[i + (size_t)(r1 + j) * m] = zc(v.x, -v.y);
    }
}

__global__ void k_root_eye(double2 *X, int m) {
    for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < (long)m * m; e += (long)gridDim.x * blockDim.x)
        X[e] = zc(e % m == e / m ? 1.0 : 0.0, 0.0);
}

// Root: the row sweep on [D+ | I] leaves Linv = L_rho^{-1}
static void ulv_root_factor(double2 *D, int m, double2 *Linv, int *fail, UlvWork &w, hipStream_t s) {
    k_root_eye<<<256, 256, 0, s>>>(Linv, m);
    const std::vector<TriNode> tn{TriNode{D, Linv, m, m}};
    fact_sweep(tn, m, m, true, fail, w, s);
}

// One level of the ULV solve.  UP: z = W y_tau, rows < k to Bh, rows >= k to the parent's
// vector (Ylo).  DOWN: c_tau = W^* [Bh rows; Ylo rows].
struct LevelArgs {
    const double2 *W;
    const size_t *woff;
    const int *m, *k;
    const long *yoff, *roff;
};

// the vectors of a level: Y its own (input of UP, output of DOWN; accum != 0 adds, the update f += G~^{-1} y of
// a refinement step), Bh its eliminated rows, Ylo its parents'
struct LevelVecs {
    const double2 *Yin;
    double2 *Yout, *Bh, *Ylo;
    long ldy, ldb, ldlo;
    int nrhs, accum;
};

// row gm of a node's result, column gc
template <bool DOWN>
__device__ __forceinline__ void ulv_put(const LevelVecs &v, long yo, long ro, int k, int gm, int gc, double2 z) {
    if (DOWN) {
        double2 *p = v.Yout + (yo + gm) + (size_t)gc * v.ldy;
        if (v.accum) z = cadd(*p, z);
        *p = z;
    } else if (gm < k) {
        v.Bh[(yo + gm) + (size_t)gc * v.ldb] = z;
    } else {
        v.Ylo[(ro + gm - k) + (size_t)gc * v.ldlo] = z;
    }
}

// The complex entries of a 16-row tile: lanes of columns 0 .. 7 hold A_r X_r and A_i X_r, the others A_r X_i and
// A_i X_i (W^* has -A_i); a lane gets the entry of row i, the lane 8 on that of row i + 2.
template <bool DOWN, typename F>
__device__ __forceinline__ void ulv_tile(Mat4<double>::V P, Mat4<double>::V Q, int lane, F &&put) {
    const bool im = (lane & 15) >= 8;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double tp = row_half(im ? P[i] : P[i + 2]), p = im ? P[i + 2] : P[i];
        double tq = row_half(im ? Q[i] : Q[i + 2]), q = im ? Q[i + 2] : Q[i];
        if (DOWN) {
            tq = -tq;
            q = -q;
        }
        put(i, Mat4<double>::row(lane, i) + (im ? Mat4<double>::row(0, 2) : 0), im ? zc(tp - q, p + tq) : zc(p - tq, tp + q));
    }
}

// Nodes of more than 64 rows (2D trees have 2 to 32 of them in a level): a workgroup forms 16 NR rows for 8 columns
// on the matrix cores, entries straight from memory to registers, D steps of 4 inner indices ahead; each of
// its 8 waves takes an eighth of the inner dimension, summed in order through LDS.
// 4 nodes of 242 rows, 8 columns: 35.5 -> 8.2 us; a root of 424 rows 137 -> 20 us (one lane per row with
// partial sums in memory, tiles of 32 x 32 through LDS: 8 to 40 workgroups in all).  The load latency of a
// wave's 8 to 14 steps bounds it.
template <bool DOWN, int NR>
__global__ void __launch_bounds__(512) k_ulv_mm(LevelArgs a, LevelVecs v, int rgroups, int cgroups, unsigned nwork) {
    using M = Mat4<double>;
    using V = M::V;
    constexpr int KS = 8, D = 4;
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // consecutive workgroups run on one XCD, whose L2 then serves the column groups of a node
    const unsigned work = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (work >= nwork) return;
    const int cg = work % cgroups, rn = work / cgroups, r0 = rn % rgroups * 16 * NR, node = rn / rgroups;
    const int m = a.m[node], k = a.k[node];
    if (r0 >= m) return;
    const long yo = a.yoff[node], ro = a.roff[node];
    const int c = cg * 8 + (lr & 7), cc = c < v.nrhs ? c : v.nrhs - 1;
    const int ns = (m + 3) >> 2, per = (ns + KS - 1) / KS, s0 = wave * per;
    const int s1 = s0 + per < ns ? s0 + per : ns;
    const double2 *W = a.W + a.woff[node];
    int row[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        const int r = r0 + 16 * t + lr;
        row[t] = r < m ? r : m - 1;                 // rows beyond the node repeat its last one and are not stored
    }
    const double *y1 = reinterpret_cast<const double *>(DOWN ? v.Bh + yo + (size_t)cc * v.ldb
                                                             : v.Yin + yo + (size_t)cc * v.ldy) + (lr >> 3);
    const double *y2 = reinterpret_cast<const double *>(v.Ylo + ro - k + (size_t)cc * v.ldlo) + (lr >> 3);
    double2 fa[D][NR];
    double fb[D];
    auto load = [&](int d, int s) {
        const int l = 4 * s + lk, lc = l < m ? l : m - 1;
#pragma unroll
        for (int t = 0; t < NR; ++t) fa[d][t] = DOWN ? W[lc + (size_t)row[t] * m] : W[row[t] + (size_t)lc * m];
        const double x = (DOWN && lc >= k ? y2 : y1)[2 * (size_t)lc];
        fb[d] = l < m ? x : 0.0;
    };
    V P[NR], Q[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) P[t] = Q[t] = V{0, 0, 0, 0};
    auto mac = [&](int d) {
#pragma unroll
        for (int t = 0; t < NR; ++t) {
            P[t] = M::mac(fa[d][t].x, fb[d], P[t]);
            Q[t] = M::mac(fa[d][t].y, fb[d], Q[t]);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (s0 + d < s1) load(d, s0 + d);
    int s = s0;
    for (; s + D <= s1; s += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            mac(d);
            if (s + d + D < s1) load(d, s + d + D);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (s + d < s1) mac(d);
    __shared__ double2 part[KS * NR * 128];
#pragma unroll
    for (int t = 0; t < NR; ++t)
        ulv_tile<DOWN>(P[t], Q[t], lane, [&](int, int r, double2 z) { part[(wave * 16 * NR + 16 * t + r) * 8 + (lr & 7)] = z; });
    __syncthreads();
    for (int e = threadIdx.x; e < 128 * NR; e += 512) {
        const int gm = r0 + (e >> 3), gc = cg * 8 + (e & 7);
        if (gm >= m || gc >= v.nrhs) continue;
        double2 z = part[e];
#pragma unroll
        for (int w = 1; w < KS; ++w) z = cadd(z, part[w * 128 * NR + e]);
        ulv_put<DOWN>(v, yo, ro, k, gm, gc, z);
    }
}

// Nodes of at most 64 rows (the leaves): a workgroup takes a node for 8 CW columns, staged in LDS (a column of
// a node is contiguous, and the vectors' columns are far apart) and written back through it; a wave forms 4 / RG
// row tiles of 8 columns, W straight from memory.  Inner indices in order, whatever the split.
// The stream of W bounds it: 4096 leaves of N = 2^18, 8 columns, 268 MB in 61 (down) and 69 us (up); 1024 of
// N = 2^16, 16 columns: 48 -> 23 us a direction (tiles of 64 x 64 on the vector units before).
template <bool DOWN, int CW, int RG>
__global__ void __launch_bounds__(64 * CW * RG) k_ulv_leaf(LevelArgs a, LevelVecs v, int cgroups, unsigned nwork) {
    using M = Mat4<double>;
    using V = M::V;
    constexpr int NR = 4 / RG, NW = CW * RG, LD = 65, NCOL = 8 * CW, D = 2;
    __shared__ double2 xs[NCOL * LD];
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned work = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (work >= nwork) return;
    const int node = work / cgroups, c0 = (work - node * cgroups) * NCOL;
    const int m = a.m[node], k = a.k[node];
    if (m == 0) return;
    const long yo = a.yoff[node], ro = a.roff[node];
    const double2 *W = a.W + a.woff[node];
    const int r0 = wave / CW * 16 * NR, xc = wave % CW * 8;
    const int ns = (m + 7) >> 3;
    int row[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        const int r = r0 + 16 * t + lr;
        row[t] = r < m ? r : m - 1;
    }
    // a step takes 8 inner indices, two per lane, so that W^* uses a whole cache line at once
    double2 fa[D][2][NR];
    auto load = [&](int d, int s) {
#pragma unroll
        for (int t = 0; t < NR; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int l = 8 * s + 2 * lk + u, lc = l < m ? l : m - 1;
                fa[d][u][t] = DOWN ? W[lc + row[t] * m] : W[row[t] + lc * m];
            }
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < ns) load(d, d);
#pragma unroll
    for (int j = 0; j < NCOL / NW; ++j) {
        const int l = lane, c = wave + NW * j, gc = c0 + c < v.nrhs ? c0 + c : v.nrhs - 1, lc = l < m ? l : m - 1;
        const double2 *p = DOWN ? (lc < k ? v.Bh + (yo + lc) + (size_t)gc * v.ldb : v.Ylo + (ro + lc - k) + (size_t)gc * v.ldlo)
                                : v.Yin + (yo + lc) + (size_t)gc * v.ldy;
        const double2 x = *p;
        xs[c * LD + l] = l < m ? x : zc(0.0, 0.0);
    }
    __syncthreads();
    V P[NR], Q[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) P[t] = Q[t] = V{0, 0, 0, 0};
    const double *xb = reinterpret_cast<const double *>(xs + (xc + (lr & 7)) * LD + 2 * lk) + (lr >> 3);
    auto mac = [&](int d, int s) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const double x = xb[16 * s + 2 * u];
#pragma unroll
            for (int t = 0; t < NR; ++t) {
                P[t] = M::mac(fa[d][u][t].x, x, P[t]);
                Q[t] = M::mac(fa[d][u][t].y, x, Q[t]);
            }
        }
    };
    if (r0 < m) {
        int s = 0;
        for (; s + D <= ns; s += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                mac(d, s + d);
                if (s + d + D < ns) load(d, s + d + D);
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (s + d < ns) mac(d, s + d);
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NR; ++t)
        ulv_tile<DOWN>(P[t], Q[t], lane, [&](int, int r, double2 z) { xs[(xc + (lr & 7)) * LD + r0 + 16 * t + r] = z; });
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NCOL / NW; ++j) {
        const int c = wave + NW * j;
        if (lane < m && c0 + c < v.nrhs) ulv_put<DOWN>(v, yo, ro, k, lane, c0 + c, xs[c * LD + lane]);
    }
}

// The same for wider blocks and for levels of many nodes: a workgroup of RG x CG waves forms 16 NR RG rows for 8 CG
// columns of a node, W and the vectors through LDS in chunks of 32 inner indices, the next chunk on its way to
// registers while one is used, so that waves share what they read and W^* is read along its columns.  Inner
// indices in the order of k_ulv_leaf, or (SPLIT) of k_ulv_mm, its 8 slices one after another.
// N = 2^16 with 512 leaves of 128 rows, a solve of 64 columns: 467 us with k_ulv_mm (which reads W once per 8
// columns), 300 us with tiles of 32 x 32 on the vector units, 235 us; 8 columns 109, 170 and 93 us.  4096 leaves of 64
// rows, 64 columns: 613 us with W in halves of 32 inner indices and the whole vectors in LDS, 549 us; 33 columns 563 ->
// 420 us, 1024 leaves and 512 columns 1086 -> 980 us, 512 leaves of 32 rows and 512 columns 433 -> 241 us (whose rows
// beyond the node and columns beyond the block were multiplied too).
template <bool DOWN, int NR, int RG, int CG, bool SPLIT>
__global__ void __launch_bounds__(64 * RG * CG) k_ulv_wide(LevelArgs a, LevelVecs v, int rgroups, int cgroups, unsigned nwork) {
    using M = Mat4<double>;
    using V = M::V;
    constexpr int RT = 16 * NR * RG, CT = 8 * CG, NT = 64 * RG * CG, KC = 32, LW = KC + 1, LX = KC + 2, LD = RT + 1;
    constexpr int EW = RT * KC / NT, EX = CT * KC / NT, EO = RT * CT / NT;
    __shared__ double2 lds[RT * LW + CT * LX];
    static_assert(CT * LD <= RT * LW + CT * LX, "the results are staged in the same LDS");
    double2 *ws = lds, *xs = lds + RT * LW;                    // [row][inner], [column][inner]
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive workgroups run on one XCD, whose L2 then serves the column groups of a node
    const unsigned work = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (work >= nwork) return;
    const int c0 = work % cgroups * CT, rn = work / cgroups, g0 = rn % rgroups * RT, node = rn / rgroups;
    const int m = a.m[node], k = a.k[node];
    if (g0 >= m) return;
    const long yo = a.yoff[node], ro = a.roff[node];
    const double2 *W = a.W + a.woff[node];
    const int r0 = wave / CG * 16 * NR, xc = wave % CG * 8;
    const bool act = g0 + r0 < m && c0 + xc < v.nrhs;
    double wr[EW], wi[EW], xr[EX], xi[EX];                     // (arrays of pairs would be kept in memory)
    auto fetch = [&](int l0) {
#pragma unroll
        for (int j = 0; j < EW; ++j) {
            const int e = tid + NT * j, r = g0 + (DOWN ? e / KC : e % RT), l = l0 + (DOWN ? e % KC : e / RT);
            const int rc = r < m ? r : m - 1, lc = l < m ? l : m - 1;
            const double2 w = W[DOWN ? lc + (size_t)rc * m : rc + (size_t)lc * m];
            wr[j] = w.x;
            wi[j] = w.y;
        }
#pragma unroll
        for (int j = 0; j < EX; ++j) {
            const int e = tid + NT * j, c = c0 + e / KC, l = l0 + e % KC;
            const int cc = c < v.nrhs ? c : v.nrhs - 1, lc = l < m ? l : m - 1;
            const double2 *p = DOWN ? (lc < k ? v.Bh + (yo + lc) + (size_t)cc * v.ldb : v.Ylo + (ro + lc - k) + (size_t)cc * v.ldlo)
                                    : v.Yin + (yo + lc) + (size_t)cc * v.ldy;
            const double2 x = *p;
            xr[j] = l < m ? x.x : 0.0;
            xi[j] = l < m ? x.y : 0.0;
        }
    };
    V P[NR], Q[NR];
    double2 sum[NR][2];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        P[t] = Q[t] = V{0, 0, 0, 0};
        sum[t][0] = sum[t][1] = zc(-0.0, -0.0);
    }
    // adds the slice's products to the sums
    auto flush = [&]() {
#pragma unroll
        for (int t = 0; t < NR; ++t) {
            ulv_tile<DOWN>(P[t], Q[t], lane, [&](int i, int, double2 z) { sum[t][i] = cadd(sum[t][i], z); });
            P[t] = Q[t] = V{0, 0, 0, 0};
        }
    };
    // steps of 4 inner indices, and of a slice
    const int ns = SPLIT ? (m + 3) >> 2 : 2 * ((m + 7) >> 3), per = SPLIT ? (ns + 7) >> 3 : ns;
    const double2 *wb = ws + (r0 + lr) * LW + (SPLIT ? lk : 2 * lk);
    const double *xb = reinterpret_cast<const double *>(xs + (xc + (lr & 7)) * LX + (SPLIT ? lk : 2 * lk)) + (lr >> 3);
    int left = per;
    for (int s0 = -KC / 4;; s0 += KC / 4) {
        const bool more = s0 + KC / 4 < ns;
        if (more) fetch(4 * s0 + KC);
        if (act && s0 >= 0) {
#pragma unroll
            for (int q = 0; q < KC / 4; ++q) {
                if (s0 + q >= ns) break;
                const int l = SPLIT ? 4 * q : 8 * (q >> 1) + (q & 1);
                const double x = xb[2 * l];
#pragma unroll
                for (int t = 0; t < NR; ++t) {
                    const double2 w = wb[16 * t * LW + l];
                    P[t] = M::mac(w.x, x, P[t]);
                    Q[t] = M::mac(w.y, x, Q[t]);
                }
                if (SPLIT && --left == 0) {
                    flush();
                    left = per;
                }
            }
        }
        __syncthreads();
        if (!more) break;
#pragma unroll
        for (int j = 0; j < EW; ++j) {
            const int e = tid + NT * j;
            ws[DOWN ? e / KC * LW + e % KC : e % RT * LW + e / RT] = zc(wr[j], wi[j]);
        }
#pragma unroll
        for (int j = 0; j < EX; ++j) {
            const int e = tid + NT * j;
            xs[e / KC * LX + e % KC] = zc(xr[j], xi[j]);
        }
        __syncthreads();
    }
    if (!SPLIT || left != per) flush();
#pragma unroll
    for (int t = 0; t < NR; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            lds[(xc + (lr & 7)) * LD + r0 + 16 * t + M::row(lane, i) + (lr >= 8 ? M::row(0, 2) : 0)] = sum[t][i];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < EO; ++j) {
        const int e = tid + NT * j, r = g0 + e % RT, c = e / RT;
        if (r < m && c0 + c < v.nrhs) ulv_put<DOWN>(v, yo, ro, k, r, c0 + c, lds[c * LD + e % RT]);
    }
}

// ---------------------------------------------------------------------------
// Bands: consecutive levels whose nodes have at most kBandRows rows (the upper levels of 1D trees, 8 rows
// at rank 4) in one launch.  A workgroup takes the subtree below one node of the band's top level (or,
// at the top of the tree, all its nodes and the root: up, root and down in one launch) for 8 columns.
// Its W, vectors and tables are read into LDS at once; the levels then run one barrier apart.  A launch
// per level is 4.7 us whatever it does: N = 2^14, 5 columns, the 7 upper levels and the root took
// 75 us of a solve, 33 us in 3 launches.
constexpr int kBandRows = 8, kBandLevels = 4, kBandNodes = 30, kBandRoot = 2 * kBandRows;

struct BandArgs {
    LevelArgs lv[kBandLevels];   // levels la .. la + nlev - 1
    int nlev;
    const double2 *Yin;          // vectors of the lowest level (UP)
    double2 *Yout;               // vectors of the lowest level (DOWN)
    long ldin, ldout;
    double2 *Bh[kBandLevels];
    long ldb[kBandLevels];
    double2 *Ylo;                // vectors of the level above (not TOP)
    long ldlo;
    const double2 *Linv;         // TOP
    int m0, nrhs, accum;
};

enum BandMode { BAND_UP, BAND_DOWN, BAND_TOP };

template <int MODE> __global__ void __launch_bounds__(256) k_ulv_band(BandArgs a) {
    constexpr int NN = MODE == BAND_TOP ? kBandNodes : kBandNodes / 2;
    __shared__ double2 Ws[NN][64];                             // column-major 8 x 8
    __shared__ double2 ys[NN][64];                             // [row][column]
    __shared__ double2 bs[MODE == BAND_UP ? 1 : NN][64];
    __shared__ double2 rs[kBandRoot][8], rt[MODE == BAND_TOP ? kBandRoot : 1][8];
    __shared__ double2 Ls[MODE == BAND_TOP ? kBandRoot * kBandRoot : 1];
    __shared__ int sm[NN], sk[NN], so[NN], slev[NN];           // rows, eliminated rows, row of the rest in the parent
    __shared__ long syo[NN];
    __shared__ size_t swo[NN];
    __shared__ long sro;
    const int tid = threadIdx.x, c0 = blockIdx.y * 8, top = MODE == BAND_TOP ? 2 : 1;
    const int nodes = top * ((1 << a.nlev) - 1);
    if (tid < nodes) {
        // node tid: level i, the j-th of the subtree there
        int i = 0;
        while (tid >= top * ((2 << i) - 1)) ++i;
        const int j = tid - top * ((1 << i) - 1), g = MODE == BAND_TOP ? j : ((int)blockIdx.x << i) + j;
        const LevelArgs &L = a.lv[i];
        slev[tid] = i;
        sm[tid] = L.m[g];
        sk[tid] = L.k[g];
        swo[tid] = L.woff[g];
        syo[tid] = L.yoff[g];
        // within the parent's rows: the first child's start there, the second's follow the first's
        so[tid] = i > 0 || MODE == BAND_TOP ? ((g & 1) ? L.m[g - 1] - L.k[g - 1] : 0) : 0;
        if (MODE != BAND_TOP && i == 0) sro = L.roff[g];
    }
    __syncthreads();
    const int low = top * ((1 << (a.nlev - 1)) - 1);          // first node of the lowest level
#pragma unroll 4
    for (int e = tid; e < nodes * 64; e += 256) {
        // entries outside the node read its first one (the load has no condition of its own)
        const int n = e >> 6, r = e & 7, q = (e >> 3) & 7, m = sm[n];
        const bool in = r < m && q < m;
        const double2 w = a.lv[0].W[in ? swo[n] + r + (size_t)q * m : 0];
        Ws[n][e & 63] = in ? w : zc(0.0, 0.0);
    }
    for (int e = (MODE != BAND_DOWN ? low : 0) * 64 + tid; e < nodes * 64; e += 256) {
        const int n = e >> 6, r = e & 7, q = (e >> 3) & 7, m = sm[n];
        // vectors: rows on neighbouring lanes
        const int c = c0 + q;
        if (MODE != BAND_DOWN && n >= low) {
            double2 y = zc(0.0, 0.0);
            if (r < m && c < a.nrhs) y = a.Yin[syo[n] + r + (size_t)c * a.ldin];
            ys[n][r * 8 + q] = y;
        }
        if (MODE == BAND_DOWN) {
            double2 b = zc(0.0, 0.0);
            if (r < sk[n] && c < a.nrhs) b = a.Bh[slev[n]][syo[n] + r + (size_t)c * a.ldb[slev[n]]];
            bs[n][r * 8 + q] = b;
        }
    }
    if (MODE == BAND_DOWN) {
        if (tid < 64) {
            const int r = tid & 7, q = tid >> 3;
            double2 y = zc(0.0, 0.0);
            if (r < sm[0] - sk[0] && c0 + q < a.nrhs) y = a.Ylo[sro + r + (size_t)(c0 + q) * a.ldlo];
            rs[r][q] = y;
        }
    }
    if (MODE == BAND_TOP)
        for (int e = tid; e < a.m0 * a.m0; e += 256) Ls[e] = a.Linv[e];
    __syncthreads();
    if (MODE != BAND_DOWN) {
        for (int i = a.nlev - 1; i >= 0; --i) {
            const int first = top * ((1 << i) - 1), cnt = top << i;
            for (int e = tid; e < cnt * 64; e += 256) {
                const int j = e >> 6, n = first + j, r = (e >> 3) & 7, q = e & 7, m = sm[n], k = sk[n];
                if (r >= m) continue;
                double2 z = zc(0.0, 0.0);
#pragma unroll
                for (int l = 0; l < 8; ++l) {
                    // W is zero from column m on, the rows there may hold anything
                    const double2 y = ys[n][l * 8 + q];
                    cfma(z, Ws[n][l * 8 + r], zc(l < m ? y.x : 0.0, l < m ? y.y : 0.0));
                }
                if (r < k) {
                    if (MODE == BAND_TOP)
                        bs[n][r * 8 + q] = z;
                    else if (c0 + q < a.nrhs)
                        a.Bh[i][syo[n] + r + (size_t)(c0 + q) * a.ldb[i]] = z;
                } else if (i > 0) {
                    ys[top * ((1 << (i - 1)) - 1) + (j >> 1)][(so[n] + r - k) * 8 + q] = z;
                } else if (MODE == BAND_TOP) {
                    rs[so[n] + r - k][q] = z;
                } else if (c0 + q < a.nrhs) {
                    a.Ylo[sro + r - k + (size_t)(c0 + q) * a.ldlo] = z;
                }
            }
            __syncthreads();
        }
    }
    if (MODE == BAND_UP) return;
    if (MODE == BAND_TOP) {
        // Y0 <- Linv^* Linv Y0
        const int r = tid >> 3, q = tid & 7, m = a.m0;
        double2 z = zc(0.0, 0.0);
        if (r < m)
            for (int l = 0; l < m; ++l) cfma(z, Ls[r + l * m], rs[l][q]);
        if (r < m) rt[r][q] = z;
        __syncthreads();
        z = zc(0.0, 0.0);
        if (r < m)
            for (int l = 0; l < m; ++l) cfmac(z, Ls[l + r * m], rt[l][q]);
        if (r < m) rs[r][q] = z;
        __syncthreads();
    }
    for (int i = 0; i < a.nlev; ++i) {
        const int first = top * ((1 << i) - 1), cnt = top << i;
        for (int e = tid; e < cnt * 64; e += 256) {
            const int j = e >> 6, n = first + j, r = (e >> 3) & 7, q = e & 7, m = sm[n], k = sk[n];
            if (r >= m) continue;
            const double2 *up = i > 0 ? &ys[top * ((1 << (i - 1)) - 1) + (j >> 1)][so[n] * 8 + q] : &rs[so[n]][q];
            const double2 *bn = &bs[n][q];
            double2 z = zc(0.0, 0.0);
#pragma unroll
            for (int l = 0; l < 8; ++l) {
                const double2 y = l >= k && l < m ? up[(l - k) * 8] : bn[l * 8];
                cfmac(z, Ws[n][r * 8 + l], zc(l < m ? y.x : 0.0, l < m ? y.y : 0.0));
            }
            ys[n][r * 8 + q] = z;
        }
        __syncthreads();
    }
    for (int e = tid; e < (nodes - low) * 64; e += 256) {
        const int n = low + (e >> 6), r = e & 7, q = (e >> 3) & 7;
        if (r < sm[n] && c0 + q < a.nrhs) {
            double2 *p = a.Yout + syo[n] + r + (size_t)(c0 + q) * a.ldout;
            const double2 y = ys[n][r * 8 + q];
            *p = a.accum ? cadd(*p, y) : y;
        }
    }
}

template <typename T> static size_t put(std::vector<char> &blob, const std::vector<T> &v) {
    size_t off = (blob.size() + 255) & ~(size_t)255;
    blob.resize(off + v.size() * sizeof(T) + 8);
    if (!v.empty()) std::memcpy(blob.data() + off, v.data(), v.size() * sizeof(T));
    return off;
}

static fio_status factor_impl(hss_s *h, hipStream_t s, hss_ulv_t *out) {
    hss_ulv_s *f = new hss_ulv_s();
    const int Lh = h->Lh;
    f->N = h->N;
    f->leaf = h->leaf;
    f->Lh = Lh;
    f->m.assign(Lh + 1, {});
    f->k.assign(Lh + 1, {});
    f->r.assign(Lh + 1, {});
    f->woff.assign(Lh + 1, {});
    f->yoff.assign(Lh + 1, {});
    f->roff.assign(Lh + 1, {});
    f->rows.assign(Lh + 1, 0);
    fio_status st = guarded([&] {
        size_t wtot = 0;
        for (int l = Lh; l >= 1; --l) {
            const int nn = h->nodes(l);
            long yo = 0, ro = 0;
            for (int j = 0; j < nn; ++j) {
                int m = h->m[l][j], r = h->rank[l][j];
                f->m[l].push_back(m);
                f->r[l].push_back(r);
                f->k[l].push_back(m - r);
                f->woff[l].push_back(wtot);
                wtot += (size_t)m * m;
                f->yoff[l].push_back(yo);
                f->roff[l].push_back(ro);
                yo += m;
                ro += r;
            }
            f->rows[l] = yo;
            f->rows[l - 1] = ro;
        }
        f->m0 = h->m[0][0];
        f->W.alloc(wtot * sizeof(double2) + 16);
        f->Linv.alloc((size_t)f->m0 * f->m0 * sizeof(double2) + 16);
        DevBuf failb(sizeof(int));
        FIO_HIP(hipMemsetAsync(failb.p, 0, sizeof(int), s));
        // level-by-level factorization
        DevBuf Dcur, Ucur, Dn, Un, D22, U2, scr, tmp;
        UlvWork uw(s);
        Uploads &up = uw.up;
        const double2 *Din = h->Dbuf.as<double2>();
        std::vector<size_t> din_off(h->nodes(Lh)), uin_off = h->uoff[Lh];
        for (int j = 0; j < h->nodes(Lh); ++j) din_off[j] = (size_t)j * h->leaf * h->leaf;
        const double2 *Uin = h->Ubuf[Lh]->as<double2>();
        for (int l = Lh; l >= 1; --l) {
            const int nn = h->nodes(l);
            std::vector<size_t> soff(nn), scoff(nn);
            size_t stot = 0, sctot = 0;
            int mlev = 0;
            for (int j = 0; j < nn; ++j) {
                int m = f->m[l][j];
                mlev = m > mlev ? m : mlev;
                soff[j] = stot;
                stot += (size_t)m * m;
                scoff[j] = sctot;
                sctot += (size_t)3 * m * m;
                if (m > kUlvMaxM) throw Err{FIO_ERR_UNSUPPORTED};
            }
            D22.ensure(stot * sizeof(double2) + 16);
            U2.ensure(stot * sizeof(double2) + 16);
            scr.ensure(sctot * sizeof(double2) + 16);
            FactArgs fa;
            fa.D = Din;
            fa.doff = up.put(din_off);
            fa.U = Uin;
            fa.uoff = up.put(uin_off);
            fa.msz = up.put(f->m[l]);
            fa.rsz = up.put(f->r[l]);
            fa.W = f->W.as<double2>();
            fa.woff = up.put(f->woff[l]);
            fa.D22 = D22.as<double2>();
            fa.U2 = U2.as<double2>();
            fa.soff = up.put(soff);
            fa.scratch = scr.as<double2>();
            fa.scoff = up.put(scoff);
            fa.fail = failb.as<int>();
            up.flush();
            if (mlev < g_ulv_big) {
                k_ulv_node<0><<<nn, ulv_threads(mlev), 0, s>>>(fa);
                FIO_HIP(hipGetLastError());
            } else {
                ulv_phase0_big(fa, f->m[l], f->r[l], scoff, uw, s);
            }
            {
                // Dchk = Q^* D Q for every node of the level: W slot <- Q^* D, T <- (Q^* D) Q
                ZgemmBatch g1, g2;
                double2 *sc = scr.as<double2>();
                double2 *W = f->W.as<double2>();
                for (int j = 0; j < nn; ++j) {
                    const int m = f->m[l][j];
                    double2 *Q = sc + scoff[j] + (size_t)m * m, *T = Q + (size_t)m * m;
                    g1.add(Q, m, Din + din_off[j], m, W + f->woff[l][j], m, m, m, m);
                    g2.add(W + f->woff[l][j], m, Q, m, T, m, m, m, m);
                }
                g1.put(up);
                g2.put(up);
                up.flush();
                g1.run(true, zc(1.0, 0.0), zc(0.0, 0.0), s);
                g2.run(false, zc(1.0, 0.0), zc(0.0, 0.0), s);
            }
            if (mlev < g_ulv_big) {
                k_ulv_node<1><<<nn, ulv_threads(mlev), 0, s>>>(fa);
                FIO_HIP(hipGetLastError());
            } else {
                ulv_phase1_big(fa, f->m[l], f->r[l], scoff, f->woff[l], uw, s);
            }
            {
                // Dhat22 = Dchk22 - X^* X and W2 = Q2^* - X^* W1 for every node of the level, with
                // X = Dhat21^* (k x r) left in T(0..k, k..m) by the node kernel
                ZgemmBatch g3, g4;
                double2 *sc = scr.as<double2>();
                double2 *W = f->W.as<double2>();
                double2 *D22b = fa.D22;
                for (int j = 0; j < nn; ++j) {
                    const int m = f->m[l][j], r = f->r[l][j], k = m - r;
                    if (m == 0 || r == 0 || k == 0) continue;
                    double2 *T = sc + scoff[j] + 2 * (size_t)m * m;
                    const double2 *X = T + (size_t)k * m;
                    g3.add(X, m, X, m, D22b + soff[j], r, r, r, k);
                    g4.add(X, m, W + f->woff[l][j], m, W + f->woff[l][j] + k, m, r, m, k);
                }
                g3.put(up);
                g4.put(up);
                up.flush();
                g3.run(true, zc(-1.0, 0.0), zc(1.0, 0.0), s);
                g4.run(true, zc(-1.0, 0.0), zc(1.0, 0.0), s);
            }
            // merge into level l-1
            const int np = h->nodes(l - 1);
            std::vector<size_t> dooff(np), uooff(np), toff(np), upoff(np, 0);
            std::vector<int> rpar(np, 0);
            size_t dt = 0, ut = 0, tt = 0;
            for (int j = 0; j < np; ++j) {
                int r1 = f->r[l][2 * j], r2 = f->r[l][2 * j + 1], m = r1 + r2;
                dooff[j] = dt;
                dt += (size_t)m * m;
                toff[j] = tt;
                tt += (size_t)r1 * r2 + (size_t)r1 * r1;      // T, then U2(a1)^*
                if (l - 1 >= 1) {
                    rpar[j] = h->rank[l - 1][j];
                    upoff[j] = h->uoff[l - 1][j];
                }
                uooff[j] = ut;
                ut += (size_t)m * rpar[j];
            }
            Dn.ensure(dt * sizeof(double2) + 16);
            Un.ensure(ut * sizeof(double2) + 16);
            tmp.ensure(tt * sizeof(double2) + 16);
            const std::vector<size_t> &boff = h->boff[l - 1];
            MergeArgs ma;
            ma.D22 = D22.as<double2>();
            ma.U2 = U2.as<double2>();
            ma.soff = fa.soff;
            ma.rch = fa.rsz;
            ma.B = h->Bbuf.as<double2>();
            ma.boff = up.put(boff);
            ma.Upar = (l - 1 >= 1) ? h->Ubuf[l - 1]->as<double2>() : nullptr;
            ma.upoff = up.put(upoff);
            ma.rpar = up.put(rpar);
            ma.Dout = Dn.as<double2>();
            ma.dooff = up.put(dooff);
            ma.Uout = Un.as<double2>();
            ma.uooff = up.put(uooff);
            ma.tmp = tmp.as<double2>();
            ma.toff = up.put(toff);
            {
                ZgemmBatch g1, g2, g3, g4;
                const double2 *U2b = U2.as<double2>();
                for (int j = 0; j < np; ++j) {
                    const int r1 = f->r[l][2 * j], r2 = f->r[l][2 * j + 1], m = r1 + r2, rp = rpar[j];
                    if (m == 0) continue;
                    const double2 *Ua = U2b + soff[2 * j], *Ub = U2b + soff[2 * j + 1];
                    double2 *T = tmp.as<double2>() + toff[j], *UaH = T + (size_t)r1 * r2;
                    double2 *Dp = Dn.as<double2>() + dooff[j];
                    g1.add(Ub, r2, h->Bbuf.as<double2>() + boff[j], r2, T, r2, r2, r1, r2);   // T = U2(a2) B
                    g2.add(T, r2, UaH, r1, Dp + r1, m, r2, r1, r1);                          // lower-left
                    if (l - 1 >= 1) {
                        const double2 *Up = h->Ubuf[l - 1]->as<double2>() + upoff[j];
                        double2 *Uo = Un.as<double2>() + uooff[j];
                        g3.add(Ua, r1, Up, m, Uo, m, r1, rp, r1);                            // rows of a1
                        g4.add(Ub, r2, Up + r1, m, Uo + r1, m, r2, rp, r2);                  // rows of a2
                    }
                }
                for (ZgemmBatch *g : {&g1, &g2, &g3, &g4}) g->put(up);
                up.flush();
                k_ulv_merge_prep<<<np, ulv_threads(mlev), 0, s>>>(ma);
                FIO_HIP(hipGetLastError());
                for (ZgemmBatch *g : {&g1, &g2, &g3, &g4}) g->run(false, zc(1.0, 0.0), zc(0.0, 0.0), s);
                k_ulv_merge_fill<<<np, ulv_threads(mlev), 0, s>>>(ma);
                FIO_HIP(hipGetLastError());
            }
            Dcur.swap(Dn);
            Ucur.swap(Un);
            Din = Dcur.as<double2>();
            Uin = Ucur.as<double2>();
            din_off = dooff;
            uin_off = uooff;
        }
        if (f->m0 > 0) ulv_root_factor(Dcur.as<double2>(), f->m0, f->Linv.as<double2>(), failb.as<int>(), uw, s);
        // a level that fails leaves values that are not numbers to the levels above, and one count here
        int fail = 0;
        FIO_HIP(hipMemcpyAsync(&fail, failb.p, sizeof(int), hipMemcpyDeviceToHost, s));
        FIO_HIP(hipStreamSynchronize(s));
        if (fail) throw Err{FIO_ERR_NOT_HPD};
        // device tables for the solve
        std::vector<char> blob;
        f->meta_woff.assign(Lh + 1, 0);
        f->meta_m.assign(Lh + 1, 0);
        f->meta_k.assign(Lh + 1, 0);
        f->meta_yoff.assign(Lh + 1, 0);
        f->meta_roff.assign(Lh + 1, 0);
        // level 0: the root as one node of Linv without eliminated rows
        f->meta_woff[0] = put(blob, std::vector<size_t>{0});
        f->meta_m[0] = put(blob, std::vector<int>{f->m0});
        f->meta_k[0] = put(blob, std::vector<int>{0});
        f->meta_yoff[0] = f->meta_roff[0] = put(blob, std::vector<long>{0});
        for (int l = 1; l <= Lh; ++l) {
            f->meta_woff[l] = put(blob, f->woff[l]);
            f->meta_m[l] = put(blob, f->m[l]);
            f->meta_k[l] = put(blob, f->k[l]);
            f->meta_yoff[l] = put(blob, f->yoff[l]);
            f->meta_roff[l] = put(blob, f->roff[l]);
        }
        f->meta.alloc(blob.size() + 16);
        FIO_HIP(hipMemcpy(f->meta.p, blob.data(), blob.size(), hipMemcpyHostToDevice));
        return FIO_OK;
    });
    if (st != FIO_OK) {
        delete f;
        return st;
    }
    *out = f;
    return FIO_OK;
}

static size_t ulv_ws_bytes(const hss_ulv_s *f, int nrhs) {
    // level vectors l = 0..Lh-1, Bh for l = 1..Lh, root temporary
    size_t rows = 0;
    for (int l = 0; l < f->Lh; ++l) rows += f->rows[l];
    for (int l = 1; l <= f->Lh; ++l) rows += f->rows[l];
    rows += f->m0;
    return (rows + 8 * (size_t)(f->Lh + 2)) * (size_t)nrhs * sizeof(double2) + 8192;
}

// One level of nn nodes of at most mmax rows.  A column is summed in an order that depends on the level alone; the
// rows and columns of a workgroup only split the work.
template <bool DOWN> static void ulv_level(const LevelArgs &a, const LevelVecs &v, int nn, int mmax, hipStream_t s) {
    auto wgs = [](long n) {
        if (n > (1L << 31)) throw Err{FIO_ERR_UNSUPPORTED};
        return dim3((unsigned)((n + 7) / 8 * 8));
    };
    const int rt = (mmax + 15) / 16, r64 = (mmax + 63) / 64, c8 = (v.nrhs + 7) / 8, c16 = (v.nrhs + 15) / 16,
              c32 = (v.nrhs + 31) / 32;
    // 16 columns per workgroup where 32 would leave half of one's columns empty (4096 leaves of 64 rows, 33 columns:
    // 508 -> 420 us)
    const bool by16 = c16 & 1;
    const long n8 = (long)nn * r64 * c8, n16 = (long)nn * r64 * c16, n32 = (long)nn * r64 * c32;
    if (mmax > 64 && nn < 128) {
        // Few nodes: the inner dimension is split over the waves of a workgroup.  64 nodes of 256 rows take 56 us a
        // solve of one column split and 60 us with the kernels of many nodes, 128 of 128 rows 52 and 52 us, but 64
        // columns 108 and 89 us.  Two workgroups per CU of the wide form are enough: 2D n = 64, 256 columns
        // 749 us, with k_ulv_mm 806 us.
        const int r2 = (rt + 1) / 2;
        const long m2 = (long)nn * c8 * r2, m1 = (long)nn * c8 * rt;
        if (n32 >= 512)
            k_ulv_wide<DOWN, 2, 2, 4, true><<<wgs(n32), 512, 0, s>>>(a, v, r64, c32, (unsigned)n32);
        else if (m2 >= 512)
            k_ulv_mm<DOWN, 2><<<wgs(m2), 512, 0, s>>>(a, v, r2, c8, (unsigned)m2);
        else
            k_ulv_mm<DOWN, 1><<<wgs(m1), 512, 0, s>>>(a, v, rt, c8, (unsigned)m1);
    } else if (mmax > 64) {
        if (v.nrhs <= 8)
            k_ulv_wide<DOWN, 1, 4, 1, false><<<wgs(n8), 256, 0, s>>>(a, v, r64, c8, (unsigned)n8);
        else if (by16)
            k_ulv_wide<DOWN, 1, 4, 2, false><<<wgs(n16), 512, 0, s>>>(a, v, r64, c16, (unsigned)n16);
        else
            k_ulv_wide<DOWN, 2, 2, 4, false><<<wgs(n32), 512, 0, s>>>(a, v, r64, c32, (unsigned)n32);
    } else if (v.nrhs > 16 && n32 >= 512) {
        if (mmax <= 16)
            k_ulv_wide<DOWN, 1, 1, 4, false><<<wgs(n32), 256, 0, s>>>(a, v, 1, c32, (unsigned)n32);
        else if (mmax <= 32)
            k_ulv_wide<DOWN, 1, 2, 4, false><<<wgs(n32), 512, 0, s>>>(a, v, 1, c32, (unsigned)n32);
        else if (by16)
            k_ulv_wide<DOWN, 1, 4, 2, false><<<wgs(n16), 512, 0, s>>>(a, v, 1, c16, (unsigned)n16);
        else
            k_ulv_wide<DOWN, 2, 2, 4, false><<<wgs(n32), 512, 0, s>>>(a, v, 1, c32, (unsigned)n32);
    } else if (v.nrhs > 8 && n16 >= 512) {
        k_ulv_leaf<DOWN, 2, 2><<<wgs(n16), 256, 0, s>>>(a, v, c16, (unsigned)n16);
    } else {
        k_ulv_leaf<DOWN, 1, 4><<<wgs(n8), 256, 0, s>>>(a, v, c8, (unsigned)n8);
    }
}

// C = G~^{-1} Y, or C += G~^{-1} Y with accumulate (the last level adds to C)
void ulv_solve_impl(hss_ulv_s *f, const double2 *Y, long ldy, double2 *C, long ldc, int nrhs, void *ws,
                    hipStream_t s, bool accumulate = false) {
    if (nrhs <= 0) return;
    const int Lh = f->Lh;
    double2 *base = reinterpret_cast<double2 *>(ws);
    std::vector<double2 *> Yl(Lh + 1, nullptr), Bl(Lh + 1, nullptr);
    size_t off = 0;
    auto take = [&](long rows) {
        double2 *p = base + off;
        off += ((size_t)rows * nrhs + 7) & ~(size_t)7;
        return p;
    };
    for (int l = 0; l < Lh; ++l) Yl[l] = take(f->rows[l]);
    for (int l = 1; l <= Lh; ++l) Bl[l] = take(f->rows[l]);
    double2 *rt = take(f->m0);
    const char *mb = f->meta.as<char>();
    auto args = [&](int l) {
        LevelArgs a;
        a.W = f->W.as<double2>();
        a.woff = (const size_t *)(mb + f->meta_woff[l]);
        a.m = (const int *)(mb + f->meta_m[l]);
        a.k = (const int *)(mb + f->meta_k[l]);
        a.yoff = (const long *)(mb + f->meta_yoff[l]);
        a.roff = (const long *)(mb + f->meta_roff[l]);
        return a;
    };
    auto mmax = [&](int l) {
        int v = 0;
        for (int x : f->m[l]) v = x > v ? x : v;
        return v;
    };
    auto vecs = [&](int l) {
        LevelVecs v;
        v.Yin = l == Lh ? Y : Yl[l];
        v.Yout = l == Lh ? C : Yl[l];
        v.Bh = Bl[l];
        v.Ylo = Yl[l - 1];
        v.ldy = f->rows[l];
        v.ldb = f->rows[l];
        v.ldlo = f->rows[l - 1];
        v.nrhs = nrhs;
        v.accum = l == Lh && accumulate ? 1 : 0;
        return v;
    };
    // levels 1 .. lt run in bands, the first of them with the root
    int lt = 0;
    while (lt < Lh && mmax(lt + 1) <= kBandRows) ++lt;
    std::vector<std::pair<int, int>> bands;      // (top level, levels)
    if (lt > 0) {
        const int nt = lt < kBandLevels ? lt : kBandLevels;
        bands.push_back({1, nt});
        const int rest = lt - nt, nb = (rest + kBandLevels - 1) / kBandLevels;
        for (int b = 0, l = nt + 1; b < nb; ++b) {
            const int n = rest / nb + (b < rest % nb ? 1 : 0);
            bands.push_back({l, n});
            l += n;
        }
    }
    auto band = [&](size_t b) {
        const int la = bands[b].first, n = bands[b].second, ll = la + n - 1;
        BandArgs a{};
        a.nlev = n;
        for (int i = 0; i < n; ++i) {
            a.lv[i] = args(la + i);
            a.Bh[i] = Bl[la + i];
            a.ldb[i] = f->rows[la + i];
        }
        a.Yin = ll == Lh ? Y : Yl[ll];
        a.Yout = ll == Lh ? C : Yl[ll];
        a.ldin = ll == Lh ? ldy : f->rows[ll];
        a.ldout = ll == Lh ? ldc : f->rows[ll];
        a.Ylo = Yl[la - 1];
        a.ldlo = f->rows[la - 1];
        a.Linv = f->Linv.as<double2>();
        a.m0 = f->m0;
        a.nrhs = nrhs;
        a.accum = ll == Lh && accumulate ? 1 : 0;
        return a;
    };
    const unsigned cg = (unsigned)((nrhs + 7) / 8);
    // bottom-up
    for (int l = Lh; l > lt; --l) {
        if (mmax(l) == 0) continue;
        FIO_TIMED("ulv_up", s);
        LevelVecs v = vecs(l);
        if (l == Lh) v.ldy = ldy;
        ulv_level<false>(args(l), v, (int)f->m[l].size(), mmax(l), s);
    }
    for (size_t b = bands.size(); b-- > 1;) {
        FIO_TIMED("ulv_up", s);
        k_ulv_band<BAND_UP><<<dim3(1u << bands[b].first, cg), 256, 0, s>>>(band(b));
    }
    // root: Y0 <- Linv^* Linv Y0
    if (lt > 0) {
        FIO_TIMED("ulv_root", s);
        k_ulv_band<BAND_TOP><<<dim3(1, cg), 256, 0, s>>>(band(0));
    } else if (f->m0 > 0) {
        FIO_TIMED("ulv_root", s);
        LevelArgs a = args(0);
        a.W = f->Linv.as<double2>();
        LevelVecs v{Yl[0], Yl[0], nullptr, rt, f->m0, 0, f->m0, nrhs, 0};
        ulv_level<false>(a, v, 1, f->m0, s);
        ulv_level<true>(a, v, 1, f->m0, s);
    }
    // top-down
    for (size_t b = 1; b < bands.size(); ++b) {
        FIO_TIMED("ulv_down", s);
        k_ulv_band<BAND_DOWN><<<dim3(1u << bands[b].first, cg), 256, 0, s>>>(band(b));
    }
    for (int l = lt + 1; l <= Lh; ++l) {
        if (mmax(l) == 0) continue;
        FIO_TIMED("ulv_down", s);
        LevelVecs v = vecs(l);
        if (l == Lh) v.ldy = ldc;
        ulv_level<true>(args(l), v, (int)f->m[l].size(), mmax(l), s);
    }
    FIO_HIP(hipGetLastError());
}

size_t ulv_ws_bytes_pub(const hss_ulv_s *f, int nrhs) { return ulv_ws_bytes(f, nrhs); }

}  // namespace fio

using namespace fio;

extern "C" fio_status hss_ulv_factor(hss_t h, void *stream, hss_ulv_t *out) {
    PoolScope scope;
    FIO_CHECK_ARG(h && out);
    return factor_impl(h, as_stream(stream), out);
}

extern "C" fio_status hss_ulv_workspace_size(hss_ulv_t f, int nrhs, size_t *bytes) {
    FIO_CHECK_ARG(f && bytes && nrhs >= 0);
    *bytes = ulv_ws_bytes(f, nrhs);
    return FIO_OK;
}

extern "C" fio_status hss_ulv_solve(hss_ulv_t f, const void *Y, long ldy, void *C, long ldc, int nrhs, void *ws,
                                    size_t ws_bytes, void *stream) {
    FIO_CHECK_ARG(f && nrhs >= 0);
    if (nrhs == 0) return FIO_OK;
    FIO_CHECK_ARG(Y && C && ldy >= f->N && ldc >= f->N);
    if (Y == C) FIO_CHECK_ARG(ldy == ldc);
    size_t need = ulv_ws_bytes(f, nrhs);
    return guarded([&] {
        hipStream_t s = as_stream(stream);
        if (ws) {
            if (ws_bytes < need) return FIO_ERR_ARG;
            ulv_solve_impl(f, (const double2 *)Y, ldy, (double2 *)C, ldc, nrhs, ws, s);
        } else {
            std::lock_guard<std::mutex> lk(f->ws_mu);
            if (f->ws.bytes < need) {
                FIO_HIP(hipStreamSynchronize(s));
                f->ws.alloc(need);
            }
            ulv_solve_impl(f, (const double2 *)Y, ldy, (double2 *)C, ldc, nrhs, f->ws.p, s);
        }
        return FIO_OK;
    });
}

extern "C" void hss_ulv_destroy(hss_ulv_t f) {
    PoolScope scope;
    delete f;
}

extern "C" void fio_ulv_set_big_node(int rows) { fio::g_ulv_big = rows > 0 ? rows : fio::kUlvBig; }
