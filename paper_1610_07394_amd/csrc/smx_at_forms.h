// The linear forms that split the Axilrod-Teller trace into scalars:
// tr(ABC) = sum_r l_r(A) l_r(B) l_r(C) for symmetric traceless 3 x 3 matrices, as
// tr(ABC) is symmetric in them and tr(A^3) = sum_r l_r(A)^3.
//
// The ten forms.  With Z = A_zz, u = (A_xx - A_yy) / 2, v = A_xy, s = A_xz,
// t = A_yz:  tr(A^3) = 3 det A =
//   3/4 Z^3 - 3 Z (u^2 + v^2) + 3/2 Z (s^2 + t^2) + 3 (u (s^2 - t^2) + 2 v s t).
// Take kappa Z, the three alpha Z + beta u', and the six gamma Z + delta u' +-
// epsilon t', where u' = u cos 2a + v sin 2a and t' = t cos a - s sin a for a = 0,
// 120, 240 degrees about z.  Summing their cubes and comparing:
//   gamma eps^2 = 1/6,  delta eps^2 = -2/3,  beta^3 + 2 delta^3 = 0,
//   9/2 alpha beta^2 + 9 gamma delta^2 = -3,  kappa^3 + 3 alpha^3 + 6 gamma^3 = 3/4,
// a family with one free parameter; gamma = 5/24 keeps the sum of |l_r|^3 (which
// is what rounding errors grow with) within 1% of its least value.  No nine real
// forms were found by numerical search; the tensor product itself needs 18.
#pragma once

namespace smx {

constexpr int kAtForms = 10;
constexpr double kAtKappa = 1.384271578456131, kAtAlpha = -0.8672456560109711, kAtBeta = 1.0499342082457277,
                 kAtGamma = 5.0 / 24.0, kAtDelta = -5.0 / 6.0, kAtEps = 0.8944271909999159,
                 kAtSin = 0.8660254037844386;  // sin 120
// coefficients of Z, u, v, s, t
constexpr double kAtForm[kAtForms][5] = {
    {kAtKappa, 0, 0, 0, 0},
    {kAtAlpha, kAtBeta, 0, 0, 0},
    {kAtAlpha, -0.5 * kAtBeta, -kAtSin * kAtBeta, 0, 0},
    {kAtAlpha, -0.5 * kAtBeta, kAtSin * kAtBeta, 0, 0},
    {kAtGamma, kAtDelta, 0, 0, kAtEps},
    {kAtGamma, kAtDelta, 0, 0, -kAtEps},
    {kAtGamma, -0.5 * kAtDelta, -kAtSin * kAtDelta, -kAtSin * kAtEps, -0.5 * kAtEps},
    {kAtGamma, -0.5 * kAtDelta, -kAtSin * kAtDelta, kAtSin * kAtEps, 0.5 * kAtEps},
    {kAtGamma, -0.5 * kAtDelta, kAtSin * kAtDelta, kAtSin * kAtEps, -0.5 * kAtEps},
    {kAtGamma, -0.5 * kAtDelta, kAtSin * kAtDelta, -kAtSin * kAtEps, 0.5 * kAtEps},
};

}  // namespace smx
