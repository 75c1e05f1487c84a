// Sums of squared correlations of sector vectors (qsg_corr.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace qsg {

// With W_s the Walsh-Hadamard transform of v_s^2 over the n = L^2 - 1 index
// bits (s = e, o: the even and the odd vector) and R_s[S] = W_s[S] / W_s[0]
// the correlation of a set S of sites (the last site's bit left out):
//   out[3k + 0] = sum over pairs of R R',
//   out[3k + 1] = sum over pairs of R R' [cos(2 pi dx1/L) + cos(2 pi dx2/L)],
//   out[3k + 2] = sum over quadruples of R R'
// for R R' = R_e R_e (k = 0), R_e R_o (k = 1), R_o R_o (k = 2); without an odd
// vector (null) only k = 0.  L <= kTmMaxL.  ws: tm_corr_ws_doubles doubles.
// out: device.  Deterministic (fixed summation order).
constexpr int kCorrSums = 9;
size_t tm_corr_ws_doubles(uint32_t L, bool mixed);
hipError_t launch_tm_corr_sums(uint32_t L, const double* even, const double* odd, double* ws,
                               double* out, hipStream_t s);

}  // namespace qsg
