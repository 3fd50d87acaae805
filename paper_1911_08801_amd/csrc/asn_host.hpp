// Host-side set-up of an as-S_N problem: quadrature, kernel matrix, time step
// and operand rounding.  Plain C++ (no HIP), FP64 throughout.
#pragma once

#include <array>
#include <cstdint>
#include <string>
#include <vector>

namespace asn {

// Gauss-Legendre nodes x[n] (ascending) and weights w[n] on [-1, 1].
void gauss_legendre(int n, std::vector<double>& x, std::vector<double>& w);

// Product set: mu = Gauss-Legendre nodes, phi_k = (k + 1/2) 2 pi / n_azim,
// ordinate q = i * n_azim + k; omega is [Q][3], weights sum to 4 pi.
void product_quadrature(int n_polar, int n_azim, std::vector<double>& omega,
                        std::vector<double>& w);

// Icosahedron set of the given order (>= 2): N = 10 (order - 1)^2 + 2 ordinates on
// the subdivided faces of a regular icosahedron with a vertex at (0, 0, 1); the
// weight of a node is the area of the spherical polygon through the centres of
// its surrounding triangles.  Sorted by decreasing z, then increasing azimuth.
void icosahedron_quadrature(int order, std::vector<double>& omega, std::vector<double>& w);

// Normalised artificial in-scattering matrix K[Q][Q] (row-major) from
// S_qp = exp(-((1 - Omega_q . Omega_p)/eps)^2).  mode 0: symmetric scaling
// (rows and w-weighted columns sum to one); mode 1: row normalisation.
// Returns false (with a message) if the scaling does not converge.
bool kernel_matrix(int Q, const double* omega, const double* w, double eps, int mode,
                   std::vector<double>& K, std::string& err);

// Banded form of K for a product set of `levels` polar levels times `azim` azimuths
// (ordinate q = i * azim + k).  The set is invariant under rotations by 2 pi / azim
// about the polar axis, so K[(i, k), (j, k')] depends on i, j and (k' - k) mod azim
// only: per pair of levels one run of coefficients c_ij(delta) over azimuth offsets,
// nonzero for |delta| <= s_ij (cyclic distance).  Pair k of level i is level
// j = i + k - reach, k = 0 .. 2 reach.  A run either is symmetric, delta = -s .. s
// (2 s + 1 < azim), or covers the whole ring, delta = 1 - azim/2 .. azim/2; the runs
// of a level are stored one after the other, each zero-padded to a multiple of 4, at
// coef[range[2 i] .. range[2 i] + range[2 i + 1]).  desc[8 i .. 8 i + 7] describes
// level i: desc[8 i] is the number n of coupled pairs, desc[8 i + 1 + p] (p < n) the
// code of pair p:
//   bits 0-5   s (azim / 2 for a whole ring)       bit 6  wide: whole ring or s > narrow_max
//   bit 7      whole ring                          bits 8-10  k
//   bits 11-17 the run's start within the level, in units of 4 coefficients.
// reach is the largest |i - j| with a nonzero.  The padding and bit 6 are what asn_contraction_work
// counts an FP32 banded step by; the kernels' tables are made of the runs alone.
struct BandForm {
    int levels = 0, azim = 0, reach = 0;
    std::vector<uint32_t> desc;
    std::vector<int32_t> range;
    std::vector<float> coef;
};
// From the FP32 values K32[Q][Q] (row-major); false when the stored values are not
// exactly of that form (every row of a level equal to the level's first row shifted),
// when reach exceeds max_reach (at most 3) or a level has more than 508 coefficients.
// Even azim up to 126.
bool band_form(int levels, int azim, const float* K32, int max_reach, int narrow_max,
               BandForm& out);
// The tables the banded kernel reads, by source level: level j adds to the outputs of
// level i = j + m - 3, column m = 0 .. 6, the products c_ij(d) (psi[k + d] + psi[k - d]),
// d = 0 .. D (d = 0: the value itself once; d = azim / 2, where both are one ordinate: half
// the coefficient).  The set is symmetric under phi -> -phi, so c_ij(d) = c_ij(-d); where
// the two stored values round to neighbouring numbers the one at +d serves both (either is
// within half an ulp, plus the FP64 evaluation's error, of the exact entry), and gain[i] is what
// the sum of a row of level i so grows by (0 without such a pair): the row defect of a
// reduced-precision K is less by it.
// Per level rows d of N = 2 R + 1 floats, output levels j - R .. j + R (zero where nothing
// couples), in coef[R - 1] for every R from the set's reach (at least 1) to 3, padded with
// zeros to D = 2 or a multiple of 4.  desc, 8 words a level: its first float in coef[1] and
// coef[2]; its form (kBand flags below); ceil(D / 4) of each output, 4 bits each, for R = 2;
// two free words; the same for R = 3; its first float in coef[0].  dtype: the operand type the
// values were rounded to.  False on asymmetry beyond that.
constexpr uint32_t kBandSteps = 15;          // ceil(D / 4)
constexpr uint32_t kBandBeyond2 = 16;        // D > 2
constexpr uint32_t kBandOuter2 = 32;         // an output other than j - 1 .. j + 1 couples at d >= 2
constexpr uint32_t kBandOuter3 = 64;         // ... at d >= 3
bool band_scatter_tables(const BandForm& bf, int dtype, std::vector<uint32_t>& desc,
                         std::array<std::vector<float>, 3>& coef, std::vector<double>& gain);
// Whether the BF16 / FP16 banded step of this K is faster on the matrix cores, which multiply every
// coupled pair's whole circulant block, than by the tables above, whose time grows with K's width
// (desc: their descriptors).  The line, in products of the tables a level and ordinate, is fitted to
// 1039 timings of both (1 to 32 levels, 32 to 64 azimuths, 50^2 to 800^2 cells, K of one level to
// dense; 0.3 % above the faster of the two on average, 14 % at most): higher with more levels, whose
// operands wait in LDS, and with fewer azimuths, of which the tables sum fewer; lower up to 32 M
// cell-ordinates, where both states stay in the 256 MB cache, which the tables' kernel writes past;
// higher below about 15 M, where the matrix form's two further launches and its start count.  Us a
// step, tables and matrix: BF16 4 x 64 azimuths, 400^2 cells, 21 products 161 and 154, 33: 177 and
// 170, 51: 215 and 177, 101: 294 and 205; 8 x 64, 200^2, 19: 75 and 90, 66: 123 and 106; 16 x 32,
// 400^2, 22: 217 and 263, 50: 384 and 378; FP16 4 x 64, 400^2, 147 (reach 3): 385 and 201.
bool band_on_matrix_cores(const BandForm& bf, const std::vector<uint32_t>& desc, int64_t cells);
// The A operands of MFMA 16x16x32 for pair `pair` of level `level` of a banded form of
// the BF16 (dtype 1) or FP16 (dtype 2) K: the pair's circulant block C[a][a'] =
// c((a' - a) mod azim) sliced as 16 output x 32 input azimuths at the offsets 16 f,
// f = 0 .. azim / 16 - 1 (slice f: rows m, columns k hold c((16 f + k - m) mod azim)),
// each as 64 lanes x 8 values (lane l: row l % 16, columns 8 (l / 16) .. + 7), appended
// to `out` as operand bits.  azim 32, 48 or 64 (48: columns past the last azimuth meet
// zero operands in the kernel).
void band_lp_fragments(const BandForm& bf, int level, int pair, int dtype,
                       std::vector<uint16_t>& out);
// The tables of the sparse step: the ordinates in groups of `width` that share sources, in order
// (order; the last group filled up with its first ordinate), and per group the ordinates that any
// of its rows of K32[Q][Q] has a nonzero at, in `chunk`s, as rows of K in that order: src, and
// coef, width a source (zeros fill the last chunk up, at its first source).  first: the chunks
// before each group, and in all.  A group is an ordinate not taken yet and those of its sources
// that add the fewest sources of their own.  False when there would be more than max_chunks.
struct SparseForm {
    std::vector<int> order, src, first;
    std::vector<float> coef;
};
bool sparse_form(int Q, const float* K32, int width, int chunk, size_t max_chunks, SparseForm& out);
// The run of a pair code: first offset and length.
inline void band_run(uint32_t code, int azim, int& lo, int& len) {
    const int s = (int)(code & 63u);
    const bool ring = (code & 128u) != 0;
    lo = ring ? 1 - azim / 2 : -s;
    len = ring ? azim : 2 * s + 1;
}

// dt = t_final / n with n = ceil(t_final / dt_max), dt_max = cfl / max(|xi|/dx + |eta|/dy).
void cfl_time_step(int Q, const double* omega, double dx, double dy, double cfl, double t_final,
                   double& dt, int64_t& n);

// Decay rate bound of a cell-to-cell sawtooth mode in a uniform region:
//   2 max_q (|xi_q|/dx + |eta_q|/dy) + max_c (sigma_a + sigma_s + 2 (1 - min_q K_qq) sigma_as).
// K is Q x Q row-major.  dt times this is the stability number.
double stability_rate(int Q, const double* omega, const double* K, double dx, double dy, int64_t C,
                      const float* sigma_a, const float* sigma_s, const float* sigma_as);
// The streaming rule with dt_max further limited to 2 cfl / srate.
void stiff_time_step(int Q, const double* omega, double dx, double dy, double srate, double cfl,
                     double t_final, double& dt, int64_t& n);

// Round a float to bfloat16 / IEEE half bits, round to nearest, ties to even.
uint16_t float_to_bf16_rne(float f);
uint16_t float_to_half_rne(float f);
float bf16_to_float(uint16_t h);
float half_to_float(uint16_t h);

}  // namespace asn
