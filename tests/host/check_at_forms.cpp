// Host check of the pieces of the matrix form that are plain arithmetic: the
// linear forms reproduce tr(ABC) of symmetric traceless matrices, and the dealing
// of block runs to the XCDs is a bijection.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "smx_at_forms.h"
#include "smx_maps.h"

using namespace smx;

static void fail(const char *what) {
    std::printf("FAIL %s\n", what);
    std::exit(1);
}

// entries Z = A_zz, u = (A_xx - A_yy) / 2, v = A_xy, s = A_xz, t = A_yz
static void matrix(const double c[5], double A[3][3]) {
    const double xx = -0.5 * c[0] + c[1], yy = -0.5 * c[0] - c[1];
    const double m[3][3] = {{xx, c[2], c[3]}, {c[2], yy, c[4]}, {c[3], c[4], c[0]}};
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) A[i][j] = m[i][j];
}

int main() {
    unsigned s = 1;
    auto rnd = [&] {
        s = s * 1664525u + 1013904223u;
        return double(s >> 8) / double(1 << 23) - 1.0;
    };
    for (int t = 0; t < 1000; ++t) {
        double c[3][5], M[3][3][3];
        for (int q = 0; q < 3; ++q) {
            for (double &v : c[q]) v = rnd();
            matrix(c[q], M[q]);
        }
        double tr = 0.0, sum = 0.0;
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j)
                for (int k = 0; k < 3; ++k) tr += M[0][i][j] * M[1][j][k] * M[2][k][i];
        for (int r = 0; r < kAtForms; ++r) {
            double p = 1.0;
            for (int q = 0; q < 3; ++q) {
                double l = 0.0;
                for (int e = 0; e < 5; ++e) l += kAtForm[r][e] * c[q][e];
                p *= l;
            }
            sum += p;
        }
        // |entries| <= 1: both sides are sums of at most a few hundred products of that size
        if (!(std::fabs(sum - tr) <= 1e-13)) fail("tr(ABC)");
    }
    for (int lg : {3, 5})
        for (unsigned G : {1u, 7u, 63u, 64u, 65u, 255u, 256u, 257u, 1530u, 5280u}) {
            std::vector<char> seen(G, 0);
            for (unsigned b = 0; b < G; ++b) {
                const unsigned d = xcd_deal(b, G, lg);
                if (d >= G || seen[d]) fail("xcd_deal");
                seen[d] = 1;
            }
        }
    std::printf("ok\n");
    return 0;
}
