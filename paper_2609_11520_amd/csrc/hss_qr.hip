// Batched blocked Householder factorizations (see hss_qr.h).
//
// A reflector per launch re-reads the whole node for every column; here kWyBlock columns are factored
// by one workgroup with the panel in registers, and their product I - V T V^* is applied to the
// other columns in one pass over them.  Over the levels of 2D n = 64 (up to 832 columns of 1594 rows, and as
// many more to update) the panels take 23 us and the updates 35 us per block on average: 22 ms in
// all, where a reflector per launch took 570 ms.  The panel is one workgroup's chain of 8 reductions;
// an update reads its columns twice, the second time from cache.
#include "hss_qr.h"

#include <algorithm>

namespace fio {

// Sums 16 values over the wave: on return the lane holds the total of value
// ((lane >> 2) & 15) reversed in its bits (wave_sum16_index).
template <int half> __device__ __forceinline__ void wave_fold(double (&v)[16], bool up, int m) {
#pragma unroll
    for (int i = 0; i < half; ++i) {
        const double send = up ? v[i] : v[i + half], keep = up ? v[i + half] : v[i];
        v[i] = keep + __shfl_xor(send, m);
    }
}
__device__ __forceinline__ double wave_sum16(double (&v)[16]) {
    const int lane = threadIdx.x & 63;
    wave_fold<8>(v, lane & 32, 32);
    wave_fold<4>(v, lane & 16, 16);
    wave_fold<2>(v, lane & 8, 8);
    wave_fold<1>(v, lane & 4, 4);
    double t = v[0];
    t += __shfl_xor(t, 2);
    t += __shfl_xor(t, 1);
    return t;
}
__device__ __forceinline__ int wave_sum16_index() {
    const int lane = threadIdx.x & 63;
    return ((lane >> 5) & 1) * 8 + ((lane >> 4) & 1) * 4 + ((lane >> 3) & 1) * 2 + ((lane >> 2) & 1);
}

// orders a wave's own LDS accesses across its lanes
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Panel of columns j0 .. j0 + NB - 1 of every node: one workgroup holds rows j0 + tid + q blockDim in
// registers.  Per column one reduction gives the norm, the products with the later columns of the
// panel and those with its earlier reflectors (for T).
template <int RPT, int NB>
__global__ void __launch_bounds__(NB == 8 ? 1024 : 512) k_qr_panel(const WyNode *__restrict__ nodes, int j0, double *tau, int kt,
                                                  double2 *T) {
    static_assert(2 * NB <= 16, "one value per reduction slot");
    const WyNode d = nodes[blockIdx.x];
    if (j0 >= d.k) return;
    const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6, lane = tid & 63, wave = tid >> 6;
    const int nb = d.k - j0 < NB ? d.k - j0 : NB;
    __shared__ double part[16][16], tot[16];
    __shared__ double2 sr[2][NB], sg[NB][NB];      // sr by turns: a wave may be one column ahead
    __shared__ double stau[NB];
    double2 a[RPT][NB];
    double2 *P = d.C + (size_t)j0 * d.ldc + j0;          // row j0, column j0
    const int rows = d.n - j0;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = tid + q * nt;
#pragma unroll
        for (int c = 0; c < NB; ++c) a[q][c] = r < rows && c < nb ? P[r + (size_t)c * d.ldc] : zc(0.0, 0.0);
    }
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        if (c < nb) {
            double2 *srow = sr[c & 1];
            // slot 0: |x|^2 below the pivot; slots 2 k + 2, 2 k + 3 (k skipping c): products
            double v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = 0.0;
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const bool below = q > 0 || tid > c;
                const double2 x = below ? a[q][c] : zc(0.0, 0.0);
                v[0] = fma(x.x, x.x, fma(x.y, x.y, v[0]));
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    if (k == c) continue;
                    // conj(x) a_k for the later columns, conj(v_k) x for the earlier reflectors
                    const int sl = 2 * (k < c ? k : k - 1) + 2;
                    const double2 y = a[q][k];
                    v[sl] = fma(x.x, y.x, fma(x.y, y.y, v[sl]));
                    const double im = k > c ? fma(x.x, y.y, -x.y * y.x) : fma(y.x, x.y, -y.y * x.x);
                    v[sl + 1] += im;
                }
            }
            const double t = wave_sum16(v);
            if ((lane & 3) == 0) part[wave][wave_sum16_index()] = t;
            if (tid == c) {
#pragma unroll
                for (int k = 0; k < NB; ++k) srow[k] = a[0][k];
            }
            __syncthreads();
            if (tid < 64) {
                double u = 0.0;
                for (int w = tid >> 4; w < nw; w += 4) u += part[w][tid & 15];
                u += __shfl_xor(u, 16);
                u += __shfl_xor(u, 32);
                if (tid < 16) tot[tid] = u;
            }
            __syncthreads();
            const double2 x0 = srow[c];
            const double a2 = x0.x * x0.x + x0.y * x0.y, sigma = sqrt(a2 + tot[0]);
            if (sigma != 0.0) {                  // a NaN goes on into every column
                const double aa = sqrt(a2);
                const double2 ph = aa > 0.0 ? zc(x0.x / aa, x0.y / aa) : zc(1.0, 0.0);
                const double2 beta = zc(-ph.x * sigma, -ph.y * sigma);
                const double2 den = csub(x0, beta);
                const double dn = den.x * den.x + den.y * den.y;
                const double2 inv = zc(den.x / dn, -den.y / dn);
                const double ta = 1.0 + aa / sigma;
#pragma unroll
                for (int q = 0; q < RPT; ++q)
                    if (q > 0 || tid > c) a[q][c] = cmul(a[q][c], inv);
#pragma unroll
                for (int k = c + 1; k < NB; ++k) {
                    const double2 dk = zc(tot[2 * (k - 1) + 2], tot[2 * (k - 1) + 3]);
                    double2 wk = srow[k];
                    cfmac(wk, inv, dk);                      // v^* a_k = a_k(j) + conj(inv) sum conj(x) a_k
                    const double2 tw = zc(ta * wk.x, ta * wk.y);
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        if (q > 0 || tid > c)
                            a[q][k] = csub(a[q][k], cmul(a[q][c], tw));
                        else if (tid == c)
                            a[q][k] = csub(a[q][k], tw);
                    }
                }
                if (tid == c) a[0][c] = beta;
                if (tid < c) {
                    // v_i^* v_c, i = tid
                    double2 g = cconj(srow[tid]);
                    cfma(g, inv, zc(tot[2 * tid + 2], tot[2 * tid + 3]));
                    sg[tid][c] = g;
                }
                if (tid == 0) stau[c] = ta;
            } else {
                if (tid == c) a[0][c] = zc(0.0, 0.0);
                if (tid < c) sg[tid][c] = zc(0.0, 0.0);
                if (tid == 0) stau[c] = 0.0;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = tid + q * nt;
#pragma unroll
        for (int c = 0; c < NB; ++c)
            if (r < rows && c < nb) P[r + (size_t)c * d.ldc] = a[q][c];
    }
    __syncthreads();
    // T(i, c) = -tau_c sum_(i <= l < c) T(i, l) v_l^* v_c, one row per thread
    if (tid < nb) {
        double2 *Tb = T + (size_t)blockIdx.x * kt * kWyBlock + (size_t)j0 * kWyBlock;
        tau[(size_t)blockIdx.x * kt + j0 + tid] = stau[tid];
        double2 row[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            double2 t = zc(0.0, 0.0);
            if (c == tid) t = zc(stau[c], 0.0);
            if (c > tid && c < nb) {
#pragma unroll
                for (int l = 0; l < c; ++l)
                    if (l >= tid) cfma(t, row[l], sg[l][c]);
                t = zc(-stau[c] * t.x, -stau[c] * t.y);
            }
            row[c] = t;
            if (c < nb) Tb[tid + (size_t)c * kWyBlock] = t;
        }
    }
}

// A panel of one column, read from memory: nodes of more than kWyMaxRows rows
__global__ void __launch_bounds__(1024) k_qr_column(const WyNode *__restrict__ nodes, int j0, double *tau, int kt,
                                                   double2 *T) {
    __shared__ double part[16];
    const WyNode d = nodes[blockIdx.x];
    if (j0 >= d.k) return;
    const int tid = threadIdx.x, rows = d.n - j0;
    double2 *x = d.C + (size_t)j0 * d.ldc + j0;
    double p = 0.0;
    for (int r = 1 + tid; r < rows; r += 1024) p = fma(x[r].x, x[r].x, fma(x[r].y, x[r].y, p));
    for (int o = 32; o > 0; o >>= 1) p += __shfl_xor(p, o);
    if ((tid & 63) == 0) part[tid >> 6] = p;
    const double2 x0 = x[0];
    __syncthreads();
    p = 0.0;
    for (int w = 0; w < 16; ++w) p += part[w];
    const double a2 = x0.x * x0.x + x0.y * x0.y, sigma = sqrt(a2 + p), aa = sqrt(a2);
    double ta = 0.0;
    double2 beta = zc(0.0, 0.0);
    if (sigma != 0.0) {
        const double2 ph = aa > 0.0 ? zc(x0.x / aa, x0.y / aa) : zc(1.0, 0.0);
        beta = zc(-ph.x * sigma, -ph.y * sigma);
        const double2 den = csub(x0, beta);
        const double dn = den.x * den.x + den.y * den.y;
        const double2 inv = zc(den.x / dn, -den.y / dn);
        ta = 1.0 + aa / sigma;
        for (int r = 1 + tid; r < rows; r += 1024) x[r] = cmul(x[r], inv);
    }
    if (tid == 0) {
        x[0] = beta;
        tau[(size_t)blockIdx.x * kt + j0] = ta;
        T[(size_t)blockIdx.x * kt * kWyBlock + (size_t)j0 * kWyBlock] = zc(ta, 0.0);
    }
}

// T of the blocks of existing reflectors: workgroup (block, node), 28 products of reflectors over 4 waves
__global__ void __launch_bounds__(256) k_wy_factors(const WyNode *__restrict__ nodes, const double *__restrict__ tau,
                                                   int ldtau, int block, int kt, double2 *T) {
    constexpr int NB = kWyBlock;
    const WyNode d = nodes[blockIdx.y];
    const int j0 = blockIdx.x * block;
    if (j0 >= d.k) return;
    const int nb = d.k - j0 < block ? d.k - j0 : block;
    __shared__ double2 sg[NB][NB];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // pairs (i, c), i < c, numbered c (c - 1) / 2 + i: wave w takes 7 w .. 7 w + 6
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = 0.0;
    const double2 *P = d.V + (size_t)j0 * d.ldv + j0;
    auto at = [&](int r, int c) {
        return c >= nb || r < c ? zc(0.0, 0.0) : r == c ? zc(1.0, 0.0) : P[r + (size_t)c * d.ldv];
    };
    for (int r = lane; r < d.n - j0; r += 64) {
        for (int p = 0; p < 7; ++p) {
            const int e = wave * 7 + p;
            int c = 1;
            while (c * (c + 1) / 2 <= e) ++c;
            const double2 l = at(r, e - c * (c - 1) / 2), q = at(r, c);
            v[2 * p] = fma(l.x, q.x, fma(l.y, q.y, v[2 * p]));
            v[2 * p + 1] = fma(l.x, q.y, fma(-l.y, q.x, v[2 * p + 1]));
        }
    }
    const double t = wave_sum16(v);
    const int idx = wave_sum16_index();
    if ((lane & 3) == 0 && idx < 14) {
        const int e = wave * 7 + (idx >> 1);
        int c = 1;
        while (c * (c + 1) / 2 <= e) ++c;
        double *g = &sg[e - c * (c - 1) / 2][c].x;
        g[idx & 1] = t;
    }
    __syncthreads();
    const int tid = threadIdx.x;
    if (tid < nb) {
        double2 *Tb = T + (size_t)blockIdx.y * kt * NB + (size_t)j0 * NB;
        double2 row[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const double ta = c < nb ? tau[(size_t)blockIdx.y * ldtau + j0 + c] : 0.0;
            double2 x = zc(0.0, 0.0);
            if (c == tid) x = zc(ta, 0.0);
            if (c > tid && c < nb) {
#pragma unroll
                for (int l = 0; l < c; ++l)
                    if (l >= tid) cfma(x, row[l], sg[l][c]);
                x = zc(-ta * x.x, -ta * x.y);
            }
            row[c] = x;
            if (c < nb) Tb[tid + (size_t)c * NB] = x;
        }
    }
}

// Columns c0 .. nc - 1 of C <- (I - V T' V^*) C for the block of reflectors at j0, T' = T^* (FWD: the product
// H_(j0+NB-1) .. H_j0) or T (H_j0 .. H_(j0+NB-1)).  A wave owns CW columns, lanes run over the rows: one
// pass forms V^* C, a second one subtracts.  cmode 0: c0 = 0, 1: c0 = j0, 2: c0 = j0 + NB.
template <int CW, bool FWD>
__global__ void __launch_bounds__(256) k_wy_update(const WyNode *__restrict__ nodes, int j0, int block,
                                                  int cmode, const double2 *__restrict__ T, int kt) {
    constexpr int NB = kWyBlock;
    const WyNode d = nodes[blockIdx.y];
    if (j0 >= d.k) return;
    const int nb = d.k - j0 < block ? d.k - j0 : block;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = (cmode == 0 ? 0 : cmode == 1 ? j0 : j0 + nb) + (blockIdx.x * 4 + wave) * CW;
    if (col >= d.nc) return;
    __shared__ double sw[4][NB * CW * 2];
    const int nc = d.nc - col < CW ? d.nc - col : CW;
    const double2 *P = d.V + (size_t)j0 * d.ldv + j0;
    double2 *Cp = d.C + (size_t)col * d.ldc + j0;
    const int rows = d.n - j0;
    // rows of V inside the block's triangle
    auto vat = [&](int r, int c) {
        double2 x = P[r + (size_t)(c < nb ? c : 0) * d.ldv];
        if (c >= nb || r < c) x = zc(0.0, 0.0);
        if (c < nb && r == c) x = zc(1.0, 0.0);
        return x;
    };
    double acc[CW][NB * 2];
#pragma unroll
    for (int u = 0; u < CW; ++u)
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) acc[u][i] = 0.0;
    for (int r = lane; r < rows; r += 64) {
        double2 x[CW];
#pragma unroll
        for (int u = 0; u < CW; ++u) x[u] = Cp[r + (size_t)(u < nc ? u : 0) * d.ldc];
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const double2 v = vat(r, c);
#pragma unroll
            for (int u = 0; u < CW; ++u) {
                acc[u][2 * c] = fma(v.x, x[u].x, fma(v.y, x[u].y, acc[u][2 * c]));
                acc[u][2 * c + 1] = fma(v.x, x[u].y, fma(-v.y, x[u].x, acc[u][2 * c + 1]));
            }
        }
    }
#pragma unroll
    for (int u = 0; u < CW; ++u) {
        const double t = wave_sum16(acc[u]);
        if ((lane & 3) == 0) sw[wave][u * 2 * NB + wave_sum16_index()] = t;
    }
    wave_fence();
    // y = T' w, lane (u, c)
    double2 y = zc(0.0, 0.0);
    if (lane < CW * NB) {
        const int u = lane / NB, c = lane % NB;
        const double2 *Tb = T + (size_t)blockIdx.y * kt * NB + (size_t)j0 * NB;
        if (c < nb) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const double2 w = zc(sw[wave][u * 2 * NB + 2 * i], sw[wave][u * 2 * NB + 2 * i + 1]);
                if (FWD) {
                    if (i <= c) cfmac(y, Tb[i + (size_t)c * NB], w);
                } else if (i >= c && i < nb) {
                    cfma(y, Tb[c + (size_t)i * NB], w);
                }
            }
        }
    }
    wave_fence();
    if (lane < CW * NB) {
        sw[wave][2 * lane] = y.x;
        sw[wave][2 * lane + 1] = y.y;
    }
    wave_fence();
    double2 yv[CW][NB];
#pragma unroll
    for (int u = 0; u < CW; ++u)
#pragma unroll
        for (int c = 0; c < NB; ++c)
            yv[u][c] = zc(sw[wave][(u * NB + c) * 2], sw[wave][(u * NB + c) * 2 + 1]);
    for (int r = lane; r < rows; r += 64) {
        double2 x[CW];
#pragma unroll
        for (int u = 0; u < CW; ++u) x[u] = Cp[r + (size_t)(u < nc ? u : 0) * d.ldc];
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const double2 v = vat(r, c);
#pragma unroll
            for (int u = 0; u < CW; ++u) x[u] = csub(x[u], cmul(v, yv[u][c]));
        }
#pragma unroll
        for (int u = 0; u < CW; ++u)
            if (u < nc) Cp[r + (size_t)u * d.ldc] = x[u];
    }
}

namespace {

struct Extent {
    int n = 0, k = 0, nc = 0;
};

Extent extent(const std::vector<WyNode> &nodes) {
    Extent e;
    for (const WyNode &d : nodes) {
        e.n = std::max(e.n, d.n);
        e.k = std::max(e.k, d.k);
        e.nc = std::max(e.nc, d.nc);
    }
    return e;
}

void upload_nodes(const std::vector<WyNode> &nodes, WyWork &w, int nmax, int kmax, Uploads &up) {
    w.nodes = up.put(nodes);
    up.flush();
    w.block = nmax <= 2048 ? 8 : nmax <= kWyMaxRows ? 4 : 1;
    w.kt = (kmax + kWyBlock - 1) / kWyBlock * kWyBlock;
    w.tau.ensure(nodes.size() * (size_t)w.kt * sizeof(double));
    w.T.ensure(nodes.size() * (size_t)w.kt * kWyBlock * sizeof(double2));
}

void update(const WyWork &w, int nn, int j0, int cmode, int ncols, bool fwd, hipStream_t s) {
    if (ncols <= 0) return;
    const WyNode *nodes = w.nodes;
    const double2 *T = w.T.as<double2>();
    // 4 columns per wave read V less often; 2 fill the card when there are few
    if ((long)ncols * nn >= 16384) {
        const dim3 g((unsigned)(ncols + 15) / 16, (unsigned)nn);
        if (fwd)
            k_wy_update<4, true><<<g, 256, 0, s>>>(nodes, j0, w.block, cmode, T, w.kt);
        else
            k_wy_update<4, false><<<g, 256, 0, s>>>(nodes, j0, w.block, cmode, T, w.kt);
    } else {
        const dim3 g((unsigned)(ncols + 7) / 8, (unsigned)nn);
        if (fwd)
            k_wy_update<2, true><<<g, 256, 0, s>>>(nodes, j0, w.block, cmode, T, w.kt);
        else
            k_wy_update<2, false><<<g, 256, 0, s>>>(nodes, j0, w.block, cmode, T, w.kt);
    }
}

}  // namespace

void wy_qr(const std::vector<WyNode> &nodes, WyWork &w, Uploads &up, hipStream_t s) {
    const Extent e = extent(nodes);
    const int nn = (int)nodes.size();
    if (e.k == 0) return;
    upload_nodes(nodes, w, e.n, e.k, up);
    const WyNode *dn = w.nodes;
    for (int j0 = 0; j0 < e.k; j0 += w.block) {
        const int rows = e.n - j0;
        double *tau = w.tau.as<double>();
        double2 *T = w.T.as<double2>();
        auto threads = [&](int rpt) { return (unsigned)((rows + 64 * rpt - 1) / (64 * rpt) * 64); };
        if (w.block == 1)
            k_qr_column<<<nn, 1024, 0, s>>>(dn, j0, tau, w.kt, T);
        else if (w.block == 4)
            k_qr_panel<10, 4><<<nn, threads(10), 0, s>>>(dn, j0, tau, w.kt, T);
        else
            k_qr_panel<2, 8><<<nn, threads(2), 0, s>>>(dn, j0, tau, w.kt, T);
        update(w, nn, j0, 2, e.nc - j0, true, s);
    }
    FIO_HIP(hipGetLastError());
}

void wy_factors(const std::vector<WyNode> &nodes, const double *tau, int ldtau, WyWork &w, Uploads &up,
                hipStream_t s) {
    const Extent e = extent(nodes);
    if (e.k == 0) return;
    upload_nodes(nodes, w, e.n, e.k, up);
    k_wy_factors<<<dim3((unsigned)(w.kt / w.block), (unsigned)nodes.size()), 256, 0, s>>>(
        w.nodes, tau, ldtau, w.block, w.kt, w.T.as<double2>());
    FIO_HIP(hipGetLastError());
}

void wy_apply(const std::vector<WyNode> &nodes, WyWork &w, bool unit, Uploads &up, hipStream_t s) {
    const Extent e = extent(nodes);
    if (e.k == 0) return;
    upload_nodes(nodes, w, e.n, e.k, up);
    for (int j0 = w.kt - w.block; j0 >= 0; j0 -= w.block)
        update(w, (int)nodes.size(), j0, unit ? 1 : 0, e.nc - (unit ? j0 : 0), false, s);
    FIO_HIP(hipGetLastError());
}

}  // namespace fio
