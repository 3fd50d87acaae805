// Checks of the tables that asn_host.cpp builds for the banded and the sparse step, read back here
// as the kernels read them.  Prints one line per finding; no line: all right.
//   host_tables band   levels azim dtype beta    the banded step's tables give K back, from each reach
//   host_tables defect levels azim dtype beta    ... and its row sums, where c(d) and c(-d) are neighbours
//   host_tables sparse levels azim order dtype beta width chunk   the sparse step's tables give K back
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "asn_host.hpp"

using namespace asn;

static float rounded(double k, int dtype) {
    const float f = (float)k;
    return dtype == 0 ? f : dtype == 1 ? bf16_to_float(float_to_bf16_rne(f)) : half_to_float(float_to_half_rne(f));
}
static std::vector<float> stored_kernel(const std::vector<double>& om, const std::vector<double>& w, double beta,
                                        int dtype) {
    std::vector<double> K;
    std::string err;
    const int Q = (int)w.size();
    if (!kernel_matrix(Q, om.data(), w.data(), beta / Q, 0, K, err)) std::exit(2);
    std::vector<float> k(K.size());
    for (size_t i = 0; i < K.size(); ++i) k[i] = rounded(K[i], dtype);
    return k;
}
// The next number of the stored type above v > 0.
static float above(float v, int dtype) {
    if (dtype == 0) return std::nextafterf(v, 2.f);
    const uint16_t h = dtype == 1 ? float_to_bf16_rne(v) : float_to_half_rne(v);
    return dtype == 1 ? bf16_to_float((uint16_t)(h + 1)) : half_to_float((uint16_t)(h + 1));
}

// K as the banded kernel's instance of reach R multiplies it, by source level and offset.
static std::vector<double> band_multiplied(int L, int A, int R, const std::vector<uint32_t>& desc,
                                           const std::array<std::vector<float>, 3>& coef) {
    const int N = 2 * R + 1, Q = L * A;
    std::vector<double> K((size_t)Q * Q, 0.0);
    for (int j = 0; j < L; ++j) {
        const uint32_t* d8 = &desc[8 * (size_t)j];
        const uint32_t first = R == 1 ? d8[7] : R == 2 ? d8[0] : d8[1], form = d8[2];
        const uint32_t steps = R == 1 ? d8[3] >> 4 : R == 2 ? d8[3] : d8[6];
        const std::vector<float>& c = coef[(size_t)R - 1];
        auto add = [&](int m, int d) {
            const size_t at = first + (size_t)d * N + m;
            if (at >= c.size()) {
                std::printf("reach %d level %d: offset %d beyond the table\n", R, j, d);
                return;
            }
            const int i = j + m - R;
            if (i < 0 || i >= L) {
                if (c[at] != 0.f) std::printf("reach %d level %d: output level %d\n", R, j, i);
                return;
            }
            for (int k = 0; k < A; ++k)
                for (int s = -1; s <= (d ? 1 : -1); s += 2)
                    K[(size_t)(i * A + k) * Q + j * A + ((k + s * d) % A + A) % A] += c[at];
        };
        for (int m = 0; m < N; ++m) {
            const bool outer = m < R - 1 || m > R + 1;
            add(m, 0);
            add(m, 1);
            if (!outer || (form & kBandOuter2)) add(m, 2);
            if (!(form & kBandBeyond2)) continue;
            if (!outer || (form & kBandOuter3)) {
                add(m, 3);
                add(m, 4);
            }
            for (int n = 1; n < (int)(form & kBandSteps); ++n)
                if ((int)((steps >> (4 * m)) & 15u) > n)
                    for (int d = 4 * n + 1; d <= 4 * n + 4; ++d) add(m, d);
        }
    }
    return K;
}

static int band(int L, int A, int dtype, double beta, bool defect) {
    std::vector<double> om, w;
    product_quadrature(L, A, om, w);
    std::vector<float> k = stored_kernel(om, w, beta, dtype);
    const int Q = L * A;
    int pairs = 0;
    if (defect)   // one offset of each pair of levels: c(-d) the number above c(d)
        for (int i = 0; i < L; ++i)
            for (int j = 0; j < L; ++j) {
                const int d = 1 + (i + j) % 3;
                const float c = k[(size_t)(i * A) * Q + j * A + d];
                if (c == 0.f || 2 * d == A) continue;
                ++pairs;
                for (int a = 0; a < A; ++a) k[(size_t)(i * A + a) * Q + j * A + (a - d + A) % A] = above(c, dtype);
            }
    BandForm bf;
    std::vector<uint32_t> desc;
    std::array<std::vector<float>, 3> coef;
    std::vector<double> gain;
    if (!band_form(L, A, k.data(), 3, 8, bf) || !band_scatter_tables(bf, dtype, desc, coef, gain)) {
        std::puts("no banded form");
        return 0;
    }
    if (defect && pairs == 0) std::puts("no pair of neighbours in this set");
    for (int R = std::max(1, bf.reach); R <= 3; ++R) {
        const std::vector<double> m = band_multiplied(L, A, R, desc, coef);
        for (int q = 0; q < Q; ++q) {
            double sum = 0.0, got = 0.0;
            for (int p = 0; p < Q; ++p) {
                sum += k[(size_t)q * Q + p];
                got += m[(size_t)q * Q + p];
                // (the entry at +d serves both where they are neighbouring numbers)
                const double e = k[(size_t)q * Q + p];
                const double tol = std::fmax(e * (dtype == 0 ? 0x1p-23 : dtype == 1 ? 0x1p-7 : 0x1p-10),
                                             dtype == 0 ? 0x1p-149 : dtype == 1 ? 0x1p-133 : 0x1p-24);
                const int i = q / A, j = p / A, d = ((p - q) % A + A) % A;
                const bool both = 2 * d > A && k[(size_t)q * Q + j * A + (q - i * A + A - d) % A] != (float)e;
                if (std::fabs(m[(size_t)q * Q + p] - e) > (both || 2 * d == A ? tol : 0.0)) {
                    std::printf("reach %d: K[%d][%d] %.9g, not %.9g\n", R, q, p, m[(size_t)q * Q + p],
                                (double)k[(size_t)q * Q + p]);
                    return 0;
                }
            }
            // (FP64 sums of at most 2048 terms of a row that sums to about 1)
            if (std::fabs(got - (sum + gain[(size_t)(q / A)])) > 1e-12) {
                std::printf("reach %d: row %d sums to %.9g, not %.9g\n", R, q, got, sum + gain[(size_t)(q / A)]);
                return 0;
            }
        }
    }
    return 0;
}

static int sparse(int L, int A, int order, int dtype, double beta, int width, int chunk) {
    std::vector<double> om, w;
    if (order) icosahedron_quadrature(order, om, w);
    else product_quadrature(L, A, om, w);
    const std::vector<float> k = stored_kernel(om, w, beta, dtype);
    const int Q = (int)w.size();
    SparseForm s;
    if (!sparse_form(Q, k.data(), width, chunk, (size_t)Q * Q, s)) {
        std::puts("no sparse form");
        return 0;
    }
    std::vector<double> m((size_t)Q * Q, 0.0);
    std::vector<int> seen((size_t)Q, 0);
    const size_t groups = s.first.size() - 1;
    if (groups != (size_t)((Q + width - 1) / width) || s.order.size() != groups * width ||
        s.src.size() != (size_t)s.first.back() * chunk || s.coef.size() != s.src.size() * width)
        std::puts("table sizes");
    for (size_t g = 0; g < groups; ++g)
        for (int o = 0; o < width; ++o) {
            const int q = s.order[g * width + o];
            const bool again = (int)g * width + o >= Q;   // fills the last group up
            if (!again) ++seen[(size_t)q];
            for (int c = s.first[g] * chunk; c < s.first[g + 1] * chunk && !again; ++c)
                m[(size_t)q * Q + s.src[(size_t)c]] += s.coef[(size_t)c * width + o];
        }
    for (int q = 0; q < Q; ++q) {
        if (seen[(size_t)q] != 1) std::printf("ordinate %d in %d groups\n", q, seen[(size_t)q]);
        for (int p = 0; p < Q; ++p)
            if (m[(size_t)q * Q + p] != (double)k[(size_t)q * Q + p]) {
                std::printf("K[%d][%d] %.9g, not %.9g\n", q, p, m[(size_t)q * Q + p], (double)k[(size_t)q * Q + p]);
                return 0;
            }
    }
    return 0;
}

int main(int argc, char** argv) {
    auto n = [&](int i) { return std::atoi(argv[i]); };
    if (argc == 6 && (!std::strcmp(argv[1], "band") || !std::strcmp(argv[1], "defect")))
        return band(n(2), n(3), n(4), std::atof(argv[5]), argv[1][0] == 'd');
    if (argc == 9 && !std::strcmp(argv[1], "sparse"))
        return sparse(n(2), n(3), n(4), n(5), std::atof(argv[6]), n(7), n(8));
    return 2;
}
