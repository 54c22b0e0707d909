#pragma once

namespace dpmm {

// Bounds on the score of the uncentred BF16 form (label_mfma.hip, label_prune.hip).  l = c_k - q / 2 is the
// score of the FP32 record (W, mu, c_k), q = ||y||^2, y = W (x - mu).  With
// x' = x - c (c a centre common to all clusters) and beta = -W (mu - c),
// y = W x' + beta; the matrix cores form Y = bf16(W) bf16(x') + beta with exact
// products and FP32 sums.  Each rounding to BF16 is within 2^-8 relative, so
//   |Y_j - y_j| <= g sum_i |W_ji| |x'_i| + g2 sum_i |W_ji| (|x'_i| + |mu_i - c_i|)
// with g = 2^-7 (plus a margin) for the two BF16 roundings and g2 = 2^-14 for
// the FP32 sums and roundings of both this form and the FP32 draw it stands
// for ((3d + 5) 2^-24 at most, d <= 128).  By Cauchy-Schwarz
//   E = ||Y - y|| <= (g + g2) ||W||_F ||x'|| + g2 ||W||_F ||mu - c||.
// The share of W's rounding in g may be taken by its own norm, ||W - bf16(W)||_F in the
// place of g / 2 ||W||_F, and rows centred on the cluster's own mean have mu - c = 0.
// The computed s = sqrt(q_bf16) is within 2^-16 s of ||Y||, so with
// E' = E + 2^-16 s the exact q lies in [max(0, s - E')^2, (s + E')^2]: the
// score lies in [c_k - (s + E')^2 / 2, c_k - max(0, s - E')^2 / 2].
// The first r rows of W, which reach the first r coordinates only, bound their own part
// of q in the same way (W, x' and mu - c cut to them).
constexpr float UC_GAMMA = 1.02f / 128.0f;
constexpr float UC_GAMMA2 = 1.0f / 16384.0f;
constexpr float UC_EPSS = 1.0f / 65536.0f;

// The same for a bf16x3 score of a row centred on the cluster's own mean, v = x - mu:
// W = W_hi + W_lo and v = v_hi + v_lo up to 2^-16 relative, and the kernel forms
// W_hi v_hi + W_hi v_lo + W_lo v_hi.  Left out are W_lo v_lo and the two remainders, 3 * 2^-16
// sum_i |W_ji| |v_i|; the 3 d products are added in FP32 (3 d 2^-23 at most, d <= 128,
// should each sum be cut off), and the FP32 draw's d as well: 2^-13.3 in all, so
//   ||Y - y|| <= g3 ||W||_F ||v||,  g3 = 2^-13.
constexpr float X3_GAMMA = 1.0f / 8192.0f;
// A lower bound of the FP32 score c - q / 2 of a row with bf16x3 norm s = sqrt(q) and
// wv >= ||W||_F ||v||, the rounding of both scores and of the bound itself included.
constexpr float x3_lower(float c, float s, float wv) {
  const float e = s + (X3_GAMMA * wv + UC_EPSS * s), h = 0.5f * e * e;
  return c - h - 1e-6f * (h + (c < 0.0f ? -c : c));
}

}  // namespace dpmm
