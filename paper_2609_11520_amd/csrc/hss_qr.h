// Batched blocked Householder factorizations (compact WY form) of the nodes of one HSS level,
// shared by the construction (Section 3.1) and the ULV factorization (Section 2.4).
#pragma once
#include "common.h"

namespace fio {

// One node: k reflectors in the columns of V (n rows, leading dimension ldv; column c holds v below the
// diagonal, v(c) = 1 implied) and the nc columns of C that they act on.
struct WyNode {
    double2 *V, *C;
    int ldv, ldc, n, k, nc;
};

constexpr int kWyBlock = 8;             // reflectors per block
constexpr int kWyMaxRows = 5120;        // largest n the panel kernel holds in registers; beyond, one column a step

// Device buffers of a level's factorizations, kept over the levels
struct WyWork {
    DevBuf tau, T;
    const WyNode *nodes = nullptr;      // the device copy of the last node list
    int kt = 0;                         // reflectors per node in tau and T
    int block = kWyBlock;               // reflectors per block: kWyBlock, 4 beyond 2048 rows, 1 beyond kWyMaxRows
};

// Householder QR of the first k columns of every node's V (= C, ldv = ldc) with the reflectors applied to
// all nc columns: H_j of column j is the reflector of the convention beta = -(x0/|x0|) ||x||, tau = 1 +
// |x0|/||x||.  R replaces the upper triangle, v the rest; tau and the blocks' triangular factors T go to w.
void wy_qr(const std::vector<WyNode> &nodes, WyWork &w, Uploads &up, hipStream_t s);
// Triangular factors of existing reflectors with the scalars tau (ldtau per node) into w
void wy_factors(const std::vector<WyNode> &nodes, const double *tau, int ldtau, WyWork &w, Uploads &up,
                hipStream_t s);
// C <- H_0 H_1 ... H_(k-1) C for every node (after wy_qr or wy_factors on nodes with the
// same V, n and k); unit: the columns of C are those of [I; 0], so block j0 leaves the columns before j0 alone
void wy_apply(const std::vector<WyNode> &nodes, WyWork &w, bool unit, Uploads &up, hipStream_t s);

}  // namespace fio
