// The error bound of the exact search's bf16 screening, apart from the
// kernels so that it can be checked on the host too.
#pragma once

namespace ifvs {

// eps >= |dd - d| for every row of norm at most max_norm that its rounding to
// bf16 moves by at most max_err, and a query of norm qnorm that its rounding
// moves by q_err (all 2-norms, of the values as they are): dd = |x|^2 + |q|^2 -
// 2 x.q from the rounded values x', q', d the distance as defined (fp32, j order).
//  * x.q - x'.q' = (x - x').q + x'.(q - q'), so it is within max_err |q| +
//    |x'| q_err, and |x'| <= max_norm + max_err.  (Rows whose roundings all
//    point one way reach it: bf16 has 8 significant bits, so a value moves by
//    up to 2^-8 of itself.  By the largest movement of any row it is about half
//    as wide on ordinary data as with that 2^-8 for every value.)
//  * g covers, generously, the fp32 sums of dim terms: the accumulation of
//    x'.q', |x|^2, |q|^2, d, the comparison's own additions and the rounding of
//    max_norm.
__host__ __device__ inline float exact_eps(int dim, double max_norm, double max_err, double qnorm, double q_err) {
  const double g = (4.0 * dim + 16.0) * 0x1p-23;
  const double both = max_norm + qnorm;
  const double dot = max_err * qnorm + (max_norm + max_err) * q_err;
  const double e = 2.0 * (dot + g * (max_norm + max_err) * (qnorm + q_err) + g * both * both) + 1e-30;
  return static_cast<float>(e * (1.0 + 0x1p-20));
}

}  // namespace ifvs
