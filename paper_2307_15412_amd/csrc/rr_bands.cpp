// rr_bands.cpp -- interpolation of a band of path lengths over the samples of
// a chirp (host): the nodes and coefficients that k_band.hip and the product
// engine use.
//
// A path adds exp(-j 2 pi k gamma) to sample k, so the sum over paths whose
// gamma lies within +-h of a band's centre is, after taking the centre's own
// rotation out, band-limited: it is fixed by its values at few of the samples.
// For a class of n nodes r_0 .. r_{n-1} (Chebyshev points over the samples,
// rounded to whole ones, so that phases stay exact integers modulo 2^32) the
// coefficients are the least-squares prediction of a process of flat spectrum
// on [-h, h] (its covariance is the sinc kernel s(k) = sinc(2 h k)):
//     L = S[k, r] (S[r, r] + e I)^-1,   e = 1e-14.
// With z = pi h (K - 1), half the phase that the band's edge gathers over the
// chirp, the largest error of any path in the band is below 2e-7 for the z
// below at every K >= 5 n, and the coefficients of a sample have a 2-norm of
// about 1, so rounding in the node sums does not grow.
#include <cmath>
#include <vector>

#include "rr_internal.h"

namespace {
const int N_CLASS = 7;
const int CLASS_N[N_CLASS] = {8, 12, 16, 20, 24, 28, 32};
const float CLASS_Z[N_CLASS] = {1.4f, 4.2f, 8.0f, 11.5f, 15.0f, 19.0f, 22.5f};

// Chebyshev points over 0 .. K - 1, the first half rounded and mirrored
void class_nodes(int K, int n, int32_t *r)
{
    const double e0 = (1.0 - std::cos(M_PI * 0.5 / n)) / 2.0;
    for (int j = 0; 2 * j < n; j++) {
        const double x = (1.0 - std::cos(M_PI * (j + 0.5) / n)) / 2.0;
        r[j] = (int32_t)std::floor((x - e0) / (1.0 - 2.0 * e0) * (K - 1) + 0.5);
        if (j && r[j] <= r[j - 1]) r[j] = r[j - 1] + 1;
        r[n - 1 - j] = K - 1 - r[j];
    }
}

double sinc(double x) { return x == 0.0 ? 1.0 : std::sin(M_PI * x) / (M_PI * x); }
long double sinc_l(long double x)
{
    const long double pi = 3.14159265358979323846264338328L;
    return x == 0.0L ? 1.0L : sinl(pi * x) / (pi * x);
}
}  // namespace

int rr_band_nodes(int K)
{
    int n = 0;
    for (int q = 0; q < N_CLASS; q++)
        if (K >= 5 * CLASS_N[q]) n = CLASS_N[q];
    return n;
}

BandClasses rr_band_classes(int K, std::vector<int32_t> &nodes, std::vector<float> &coef)
{
    BandClasses c{};
    nodes.clear();
    coef.clear();
    for (int q = 0; q < N_CLASS; q++) {
        const int n = CLASS_N[q];
        if (K < 5 * n) break;
        std::vector<int32_t> r(RR_BAND_NMAX, 0);   // [RR_BAND_NMAX]
        class_nodes(K, n, r.data());
        const double h2 = 2.0 * CLASS_Z[q] / (M_PI * (K - 1));
        // Cholesky factor of S[r, r] + e I (in extended precision: its last
        // pivots are of the size of e), the inverse pivots on its diagonal
        long double F[RR_BAND_NMAX][RR_BAND_NMAX];
        double G[RR_BAND_NMAX][RR_BAND_NMAX];
        for (int i = 0; i < n; i++)
            for (int j = 0; j <= i; j++) {
                long double v = sinc_l((long double)h2 * (r[i] - r[j])) + (i == j ? 1e-14L : 0.0L);
                for (int k = 0; k < j; k++) v -= F[i][k] * F[j][k];
                F[i][j] = i == j ? 1.0L / sqrtl(v) : v * F[j][j];
                G[i][j] = (double)F[i][j];
            }
        c.n[q] = n;
        c.z[q] = CLASS_Z[q];
        c.coef[q] = (int32_t)coef.size();
        nodes.insert(nodes.end(), r.begin(), r.end());
        coef.resize(coef.size() + (size_t)n * K);
        float *L = coef.data() + c.coef[q];        // [node][sample]
        // the nodes are symmetric about the chirp's middle: half the samples
        for (int k = 0; 2 * k < K; k++) {
            double x[RR_BAND_NMAX];
            for (int i = 0; i < n; i++) {
                double v = sinc(h2 * (k - r[i]));
                for (int j = 0; j < i; j++) v -= G[i][j] * x[j];
                x[i] = v * G[i][i];
            }
            for (int i = n - 1; i >= 0; i--) {
                double v = x[i];
                for (int j = i + 1; j < n; j++) v -= G[j][i] * x[j];
                x[i] = v * G[i][i];
                L[(size_t)i * K + k] = (float)x[i];
                if (2 * k != K - 1) L[(size_t)(n - 1 - i) * K + K - 1 - k] = (float)x[i];
            }
        }
        c.count = q + 1;
    }
    return c;
}
