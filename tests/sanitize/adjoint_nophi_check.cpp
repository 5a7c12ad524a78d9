// adjoint_nophi_check.cpp -- test-only: the form of the step vector-Jacobian
// product that the kernels run (dp_step_vjp<false>: no phi component), compiled
// for the host, against
//   (1) the form with phi on a cotangent whose phi component is zero,
//   (2) central differences of the frozen-step map in the state and in (E, L, a),
//   (3) itself along a trajectory: 64-step segments from the four basis
//       cotangents, applied last segment first, against the sequential sweep.
// Entry 2 of its state and its cotangent is left unset, so that MemorySanitizer
// reports a read of it, and builds with variables initialised to a pattern and to
// zero would disagree.
#include <cmath>
#include <cstdio>

#include "kt_adjoint_math.h"

using namespace kt;
using namespace kt::adj;

static void step_map(double M, double a, double E, double L, const double y[5], double h, double out[5]) {
    double K[6][5], Y[5];
    for (int j = 0; j < 6; ++j) {
        for (int i = 0; i < 5; ++i) {
            double acc = 0.0;
            for (int l = 0; l < j; ++l) acc += dp_a(j, l) * K[l][i];
            Y[i] = y[i] + h * acc;
        }
        double s, c;
        field(M, a, E, L, Y, K[j], &s, &c);
    }
    for (int i = 0; i < 5; ++i) {
        double acc = 0.0;
        for (int j = 0; j < 6; ++j) acc += dp_b(j) * K[j][i];
        out[i] = y[i] + h * acc;
    }
}

static unsigned long long g_state = 88172645463325252ull;
static double uniform(double lo, double hi) {
    g_state ^= g_state << 13;
    g_state ^= g_state >> 7;
    g_state ^= g_state << 17;
    return lo + (hi - lo) * (static_cast<double>(g_state >> 11) * (1.0 / 9007199254740992.0));
}

static const int IDX[4] = {0, 1, 3, 4};

int main() {
    double checksum = 0.0, worst_form = 0.0, worst_fd = 0.0;
    for (int t = 0; t < 200; ++t) {
        const double M = 1.0, a = t % 5 == 0 ? 0.0 : uniform(-0.95, 0.95), E = uniform(0.8, 1.2),
                     L = t % 7 == 0 ? 0.0 : uniform(-4.0, 4.0);
        const double z[4] = {uniform(3.0, 60.0), uniform(0.3, 2.8), uniform(-1.0, 1.0), uniform(-3.0, 3.0)};
        const double h = uniform(0.01, 0.5) * z[0] * 0.05;
        double v[4];
        for (double& x : v) x = uniform(-1.0, 1.0);
        double y[5], b[5];  // entry 2 unset
        double yf[5] = {z[0], z[1], 0.7, z[2], z[3]}, bf[5] = {v[0], v[1], 0.0, v[2], v[3]};
        for (int i = 0; i < 4; ++i) {
            y[IDX[i]] = z[i];
            b[IDX[i]] = v[i];
        }
        ParBar p{0.0, 0.0, 0.0}, q{0.0, 0.0, 0.0};
        dp_step_vjp<false>(M, a, E, L, y, h, b, &p);
        dp_step_vjp<true>(M, a, E, L, yf, h, bf, &q);
        const double got[7] = {b[0], b[1], b[3], b[4], p.E, p.L, p.a}, full[7] = {bf[0], bf[1], bf[3], bf[4], q.E, q.L, q.a};
        if (bf[2] != 0.0) worst_form = 1.0;
        for (int i = 0; i < 7; ++i) {
            worst_form = std::fmax(worst_form, std::fabs(got[i] - full[i]) / (std::fabs(full[i]) + 1e-3));
            checksum += got[i];
        }
        // v . map in each component of the state and in E, L, a: fourth-order central
        // differences, whose rounding (1e-14 / 2e-4) is far below the bound
        for (int k = 0; k < 7; ++k) {
            const double weight[4] = {1.0 / 12.0, -2.0 / 3.0, 2.0 / 3.0, -1.0 / 12.0}, at[4] = {-2.0, -1.0, 1.0, 2.0};
            double fd = 0.0;
            for (int side = 0; side < 4; ++side) {
                double w[5] = {z[0], z[1], 0.7, z[2], z[3]}, par[3] = {E, L, a}, f[5];
                double& x = k < 4 ? w[IDX[k]] : par[k - 4];
                const double eps = 2e-4 * (std::fabs(x) + 1.0);
                x += at[side] * eps;
                step_map(M, par[2], par[0], par[1], w, h, f);
                for (int i = 0; i < 4; ++i) fd += weight[side] * v[i] * f[IDX[i]] / eps;
            }
            worst_fd = std::fmax(worst_fd, std::fabs(fd - got[k]) / (std::fabs(fd) + 1e-3));
        }
    }

    // a fall from r = 12M to 2.1M around an a = 0.7 hole (horizon at 1.71M)
    const double M = 1.0, a = 0.7, E = 1.0, L = 2.9;
    constexpr int N = 300, SEG = 64, NSEG = (N + SEG - 1) / SEG;
    static double Y[N][5], H[N];
    double y[5] = {12.0, 1.2, 0.0, -0.9, 0.5};
    for (int j = 0; j < N; ++j) {
        H[j] = 0.05 + 0.02 * std::sin(0.37 * j);
        for (int i = 0; i < 5; ++i) Y[j][i] = y[i];
        step_map(M, a, E, L, y, H[j], y);
    }
    const double seed[4] = {0.8, -1.3, 0.4, 2.1};
    double seq[5];
    for (int i = 0; i < 4; ++i) seq[IDX[i]] = seed[i];
    ParBar pb{0.0, 0.0, 0.0};
    for (int j = N - 1; j >= 0; --j) dp_step_vjp<false>(M, a, E, L, Y[j], H[j], seq, &pb);
    double v[4] = {seed[0], seed[1], seed[2], seed[3]}, par[3] = {0.0, 0.0, 0.0};
    for (int s = NSEG - 1; s >= 0; --s) {
        double nv[4] = {0.0, 0.0, 0.0, 0.0};
        for (int b = 0; b < 4; ++b) {
            double c[5];
            for (int i = 0; i < 4; ++i) c[IDX[i]] = i == b ? 1.0 : 0.0;
            ParBar q{0.0, 0.0, 0.0};
            for (int j = (s + 1) * SEG < N ? (s + 1) * SEG - 1 : N - 1; j >= s * SEG; --j)
                dp_step_vjp<false>(M, a, E, L, Y[j], H[j], c, &q);
            for (int i = 0; i < 4; ++i) nv[i] = std::fma(v[b], c[IDX[i]], nv[i]);
            par[0] = std::fma(v[b], q.E, par[0]);
            par[1] = std::fma(v[b], q.L, par[1]);
            par[2] = std::fma(v[b], q.a, par[2]);
        }
        for (int i = 0; i < 4; ++i) v[i] = nv[i];
    }
    const double one[7] = {seq[0], seq[1], seq[3], seq[4], pb.E, pb.L, pb.a};
    const double two[7] = {v[0], v[1], v[2], v[3], par[0], par[1], par[2]};
    double scale = 0.0, split = 0.0;
    for (int i = 0; i < 7; ++i) scale = std::fmax(scale, std::fabs(one[i]));
    for (int i = 0; i < 7; ++i) {
        split = std::fmax(split, std::fabs(two[i] - one[i]) / scale);
        checksum += two[i];
    }
    std::printf("checksum %.17g form %.3e fd %.3e split %.3e r_end %.3f\n", checksum, worst_form, worst_fd, split, y[0]);
    return 0;
}
