// The histogram solver (csrc/histogram.hpp, one lane per row) on the host, for general alpha: stands in for the
// device's power functions and lane helpers with those of libm and a wave of one lane, and compares the returned
// root with a float64 bisection of the same histogram.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <random>
#include <type_traits>
#include <vector>

#define EA_DEV inline
static inline bool __any(bool x) { return x; }
static inline unsigned __lane_id() { return 0; }
static inline float __builtin_amdgcn_exp2f(float x) { return exp2f(x); }
static inline float __builtin_amdgcn_logf(float x) { return log2f(x); }
struct Pair { uint32_t v[2]; uint32_t operator[](int i) const { return v[i]; } };
static inline Pair __builtin_amdgcn_permlane32_swap(uint32_t a, uint32_t b, bool, bool) { return Pair{{a, b}}; }
using std::max;
using std::min;
namespace ea {
constexpr int ALPHA_15 = 0, ALPHA_20 = 1, ALPHA_GEN = 2;
static inline float xhalf_sum(float x) { return x; }
template <int AM> float pow_r1(float y, float r) { return exp2f((r - 1.f) * log2f(r < 1.f ? fmaxf(y, 1e-6f) : y)); }
}  // namespace ea
#include "histogram.hpp"

constexpr int SLOTS = 64, NB = 63;

int main() {
    std::mt19937 rng(7);
    std::normal_distribution<double> gauss;
    const double alphas[] = {1.001, 1.005, 1.01, 1.02, 1.03, 1.04, 1.05, 1.1, 1.25, 1.4, 1.6, 1.75, 1.9, 1.999};
    const int counts[] = {1, 2, 256, 1024, 8192, 131072};
    const double stds[] = {0.0, 1.0, 4.0, 9.0, 16.0, 40.0};
    double worst = 0.0;
    for (double alpha : alphas)
        for (int n : counts)
            for (double std : stds)
                for (int outliers = 0; outliers < 3; ++outliers) {
                    // scores, and the bins of one unit below their maximum, in a circular window
                    std::vector<double> x(n);
                    for (auto& v : x) v = (alpha - 1.0) * std * gauss(rng);
                    for (int i = 0; i < outliers && i < n; ++i) x[i] = *std::max_element(x.begin(), x.end()) + (i + 1) * 0.2;
                    const double m = *std::max_element(x.begin(), x.end()), h = 1.0 / NB;
                    const long top = (long)floor(m * NB), lo_bin = top - NB;
                    const int rot = (int)(rng() % SLOTS);
                    uint32_t H[SLOTS] = {0};
                    for (double v : x) {
                        const long a = (long)floor(v * NB);
                        if (a >= lo_bin) ++H[(rot + (a - lo_bin)) & (SLOTS - 1)];
                    }
                    const double origin = lo_bin * h, r = 1.0 / (double)(float)(alpha - 1.0);
                    auto f = [&](double tau) {
                        double s = -1.0;
                        for (int k = 0; k < SLOTS; ++k)
                            if (k * h > tau) s += H[(rot + k) & (SLOTS - 1)] * pow(k * h - tau, r);
                        return s;
                    };
                    double lo = -2.0 * h, hi = 1.0;
                    for (int i = 0; i < 60; ++i) { const double mid = 0.5 * (lo + hi); (f(mid) >= 0.0 ? lo : hi) = mid; }
                    const double want = std::max(lo, m - 1.0 - origin);
                    float gap;
                    const float got = ea::solve_histogram<ea::ALPHA_GEN, SLOTS, 32, false>(H, rot, 0, (float)h, (float)r, (float)(m - 1.0 - origin), gap);
                    const double err = got - want;
                    worst = std::max(worst, fabs(err));
                    // 5e-6: fp32 sums of up to 64 terms whose powers are off by r 2^-23 of themselves, over a slope of r
                    if (!(fabs(err) <= 5e-6) || !(gap >= 0.f && gap <= 5e-6f)) {
                        printf("alpha %g n %d std %g outliers %d: root %.7f, wanted %.7f, gap %g\n", alpha, n, std, outliers, got, want, gap);
                        return 1;
                    }
                }
    printf("worst %.2e\nok\n", worst);
    return 0;
}
