// Host test of the column form of the sinogram line sums (csrc/radon_cols.hpp):
// walks the strips as the kernel does, checks that every line is owned once,
// that every pixel lies inside the image and every line inside its lane's
// slots, and compares the sums with the direct sum over the line's bilinear
// samples.  Prints the worst relative difference.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <vector>

#include "../paper_1806_02637_amd/csrc/radon_cols.hpp"

using namespace ecc;

static double direct(const std::vector<float> &img, int W, int H, double sa, double ca, double t, double ds, int n_s) {
    const double c = 0.5 * (n_s - 1), u0 = 0.5 * (W - 1), v0 = 0.5 * (H - 1);
    double acc = 0.0;
    for (int j = 0; j < n_s; ++j) {
        const double s = (j - c) * ds, x = u0 + t * ca - s * sa, y = v0 + t * sa + s * ca;
        if (!(x > -1.0 && x < W && y > -1.0 && y < H)) continue;
        const int ix = (int)floor(x), iy = (int)floor(y);
        const double fx = x - ix, fy = y - iy;
        auto at = [&](int i, int k) { return i >= 0 && i < W && k >= 0 && k < H ? (double)img[k * W + i] : 0.0; };
        acc += (1 - fy) * ((1 - fx) * at(ix, iy) + fx * at(ix + 1, iy)) +
               fy * ((1 - fx) * at(ix, iy + 1) + fx * at(ix + 1, iy + 1));
    }
    return acc * ds;
}

#define CHECK(x)                                                              \
    do {                                                                      \
        if (!(x)) {                                                           \
            printf("FAILED %s (%dx%d n_t %d m %d)\n", #x, W, H, n_t, m);      \
            return 1;                                                         \
        }                                                                     \
    } while (0)

// Samples summed and the weight as the kernel chooses them.
static int n_weight(const RadonAngle &g) {
    const double ds = fabs(g.h) * sqrt(1.0 + g.s * g.s);
    const int N = radon_samples(g.inv_h), MT = ds >= 0.7072 ? 4 : ds >= 0.5657 ? 5 : ds >= 0.4715 ? 6 : 0;
    return MT > 0 ? std::max(std::min(N, MT), MT - 1) : N;
}
template <int N>
static float weight_n(const RadonAngle &g, float b, float psi, bool ends, int index, int n_s) {
    const RadonSteps<N> r = radon_steps<N>(g.s, g.h);
    return ends ? radon_weight<true>(b, psi, r, index, n_s) : radon_weight<false>(b, psi, r, 0, 0);
}
static float weight(const RadonAngle &g, int N, float b, float psi, bool ends, int index, int n_s) {
    const double ds = fabs(g.h) * sqrt(1.0 + g.s * g.s);
    if (ds < 0.4715)
        return ends ? radon_weight_any<true>(b, psi, (float)g.s, (float)g.h, N, index, n_s)
                    : radon_weight_any<false>(b, psi, (float)g.s, (float)g.h, N, 0, 0);
    switch (N) {
    case 3: return weight_n<3>(g, b, psi, ends, index, n_s);
    case 4: return weight_n<4>(g, b, psi, ends, index, n_s);
    case 5: return weight_n<5>(g, b, psi, ends, index, n_s);
    default: return weight_n<6>(g, b, psi, ends, index, n_s);
    }
}

static int run(int W, int H, int n_alpha, int n_t, double ds, double &worst) {
    std::vector<float> img((size_t)W * H);
    for (auto &x : img) x = (float)(0.2 + rand() / (double)RAND_MAX);
    const double t_max = 0.5 * sqrt((double)W * W + (double)H * H), dt = 2.0 * t_max / (n_t - 1);
    const int n_s = 2 * (int)ceil(t_max / ds) + 1;
    const double c = 0.5 * (n_s - 1);
    int R = dt < 0.601 ? (int)ceil(0.9014 / dt) : 1;
    const int NL = radon_lines_per_lane(R * dt);
    for (int m = 0; m < n_alpha; ++m) {
        const double alpha = m * (3.14159265358979323846 / n_alpha), sa = sin(alpha), ca = cos(alpha);
        std::vector<double> G(n_t, -1.0);
        std::vector<int> owned(n_t, 0);
        for (int r = 0; r < R; ++r) {
            const RadonAngle g = radon_angle(sa, ca, W, H, n_t, t_max, dt, ds, r, R);
            const double pc = 0.5 * (g.P - 1), zone = radon_end_zone(g.P, g.Q);
            const int N_min = radon_samples(g.inv_h);
            CHECK(0.5 * N_min >= fabs(g.inv_h) - 1e-9 && 0.5 * N_min < fabs(g.inv_h) + 0.5);
            for (int j = 0; strip_first_line(g, j) < g.n_lines; ++j) {
                const double Q0 = g.origin0 + (double)j * g.stride;
                const int k_lo = strip_first_line(g, j), k_hi = strip_first_line(g, j + 1);
                int p_lo, p_hi;
                strip_columns(g, j, p_lo, p_hi);
                CHECK(p_lo >= 0 && p_hi <= g.P);
                std::vector<double> acc(64 * NL, 0.0);
                for (int p = 0; p < g.P; ++p) {
                    const double sh = g.s * (p - pc), fl = floor(sh);
                    for (int i = 0; i < 64; ++i) {
                        const int q = (int)(Q0 + fl) + i;
                        const int first = lane_first_line(g, Q0, i);
                        if (q < 0 || q >= g.Q) continue;
                        CHECK(p >= p_lo && p < p_hi);
                        const double val = img[g.trans ? p * W + q : q * W + p];
                        // every line closer than rho is in the lane's slots
                        for (int k = first - 3; k < first + NL + 3; ++k) {
                            const double b = q - (g.kappa0 + k * g.dkappa) - sh;
                            const double tau = sample_at(g, k, p, c);
                            const int N = n_weight(g);
                            const float psi = psi_value(psi_bits(tau, N));
                            const float w = weight(g, N, (float)b, psi, fabs(p - pc) >= zone, radon_first_sample(tau, N), n_s);
                            if (k < first || k >= first + NL) CHECK(w < 1e-6f);
                            else acc[i * NL + k - first] += (double)w * val;
                        }
                    }
                }
                for (int k = k_lo; k < k_hi; ++k) {
                    const int real = r + R * k, kk = g.flip ? n_t - 1 - real : real;
                    CHECK(kk >= 0 && kk < n_t);
                    owned[kk]++;
                    int i_lo, i_hi;
                    line_lanes(g, Q0, k, i_lo, i_hi);
                    double sum = 0.0;
                    for (int i = i_lo; i <= i_hi; ++i) {
                        const int slot = k - lane_first_line(g, Q0, i);
                        if (slot >= 0 && slot < NL) sum += acc[i * NL + slot];
                    }
                    G[kk] = sum * ds;
                }
            }
        }
        double scale = 0.0, off = 0.0;
        for (int k = 0; k < n_t; ++k) {
            CHECK(owned[k] == 1);
            const double ref = direct(img, W, H, sa, ca, -t_max + k * dt, ds, n_s);
            scale = std::max(scale, fabs(ref));
            off = std::max(off, fabs(ref - G[k]));
        }
        worst = std::max(worst, off / scale);
        // one weight rounds to 2^-24 and positions to 2^-23 px, summed over the line
        CHECK(off <= 1e-6 * scale);
    }
    return 0;
}

int main() {
    double worst = 0.0;
    const struct { int W, H, n_alpha, n_t; double ds; } cases[] = {
        {64, 64, 24, 65, 0.5},  {128, 96, 19, 107, 0.5}, {2, 2, 8, 5, 1.0},    {97, 61, 16, 75, 0.7},
        {61, 130, 12, 300, 0.5}, {150, 3, 16, 99, 0.5},  {3, 150, 17, 99, 0.31}, {70, 70, 9, 1001, 1.0},
        {80, 60, 12, 40, 0.13}, {200, 150, 13, 43, 0.5}, {64, 90, 21, 80, 0.6}, {64, 90, 20, 80, 0.95},
    };
    for (auto &t : cases)
        if (run(t.W, t.H, t.n_alpha, t.n_t, t.ds, worst)) return 1;
    printf("ok worst %.2e\n", worst);
    return 0;
}
