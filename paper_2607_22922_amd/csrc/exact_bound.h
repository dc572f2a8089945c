// The error bound of the exact search's bf16 screening, apart from the
// kernels so that it can be checked on the host too.
#pragma once

namespace ifvs {

// eps >= |dd - d| for every row of norm at most max_norm and a query of norm
// qnorm: dd = |x|^2 + |q|^2 - 2 x.q from the values rounded to bf16, d the
// distance as defined (fp32, j order).
//  * bf16 has 8 significant bits, so rounding to nearest is off by at most
//    u = 2^-8 of the value (1 + 2^-8 becomes 1).  A product of two rounded
//    values is within 2u + u^2 of the exact one, so x.q is within that times
//    |x| |q|, and 2 x.q within twice it; rows whose roundings all point one
//    way reach it.  (2u + u^2 = 2.004 u; 2.01 u leaves room for the rounding
//    of the norms themselves.)
//  * g covers, generously, the fp32 sums of dim terms: the accumulation of
//    x.q, |x|^2, |q|^2, d and the comparison's own additions.
__host__ __device__ inline float exact_eps(int dim, double max_norm, double qnorm) {
  const double u = 0x1p-8;
  const double g = (4.0 * dim + 16.0) * 0x1p-23;
  const double both = max_norm + qnorm;
  const double e = 2.0 * ((2.01 * u + g) * max_norm * qnorm + g * both * both) + 1e-30;
  return static_cast<float>(e * (1.0 + 0x1p-20));
}

}  // namespace ifvs
