// Blocked Householder QR in 16 x 16 tiles and the solves on its factors (qr.hip).
#pragma once

#include "ftcg_internal.h"

namespace ftcg {

constexpr int QR_NB = 16;            // tile edge, columns per panel
constexpr int64_t QR_ROWS = 4096;    // rows a panel kernel holds in registers at most

inline int64_t qr_panels(int64_t c) { return (c + QR_NB - 1) / QR_NB; }

// QR of the first npanel tile columns of A (nrb x nct tiles, npanel <= nrb <=
// QR_ROWS / 16), reflected through the later tile columns too: R above the
// diagonal, R_jj in diag (16 npanel), unit reflectors below, T (npanel x 256)
// their compact forms. With f (16 npanel right-hand sides, overwritten) the
// forward substitution R^T y = f runs along.
void qr_factor(double* A, int nrb, int nct, int npanel, double* diag, double* T, double2* f, double2* y,
               hipStream_t s);
// R beta = the two columns after the c columns' tiles (real, imaginary part);
// *bad = 1 at a vanishing pivot (c <= QR_ROWS)
void qr_backsub_tiles(const double* A, int nrb, int c, const double* diag, double2* beta, int* bad, hipStream_t s);
// the same on a column-major matrix of r rows, right-hand sides in columns c and c + 1
void qr_backsub_cols(const double* A, int64_t r, int c, const double* diag, double2* beta, int* bad, hipStream_t s);
// beta = Q [y; 0] (r <= QR_ROWS; y from qr_factor)
void qr_minnorm(const double* A, int nrb, int r, int c, const double* diag, const double* T, const double2* y,
                double2* beta, int* bad, hipStream_t s);

}  // namespace ftcg
