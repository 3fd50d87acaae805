// C ABI of the as-S_N library: problem set-up, device memory layout, stepping.
#include "../../include/asn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <map>
#include <memory>
#include <mutex>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "asn_host.hpp"
#include "asn_implicit.hpp"
#include "asn_kernels.hpp"

using asn::QInfo;
using asn::StepArgs;

namespace {

thread_local std::string g_last_error;

asn_status fail(asn_status s, const std::string& msg) {
    g_last_error = msg;
    return s;
}

#define HIP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail(ASN_E_HIP, std::string(#expr ": ") + hipGetErrorString(e_));         \
    } while (0)

inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

constexpr int kGmresRestart = 30;

struct Layout {
    int Q = 0, Qp = 0, G = 1, qchunk = 1, tiles_x = 1, tiles_y = 1, fin_blocks = 1;
    int64_t C = 0, P = 0;
    bool lowp = false, fused = false;
    bool flat = false;   // separate-kernel stencil over flat cell chunks (not column strips)
    bool banded = false; // banded step: one kernel per pass for a product ordinate set
    bool sparse = false; // sparse step: one kernel per pass for any set with a sparse K
    bool matrix = false; // the banded step, on the matrix cores
    // one launch a pass: 64-cell blocks of every ordinate that finish their cells' moments
    bool by_cells() const { return (banded && !matrix) || sparse; }
    int ktab_len = 0;
    size_t off_psi0, off_psi1, off_Y, off_Kt, off_Klp, off_rdef, off_ktab, off_qi, off_coef, off_iso,
        off_band, off_bcoef[3], off_bcxy, off_bfrag, off_sgroup, off_sord, off_srow, off_scoef,
        off_phi64, off_phipart, off_blk, off_fin, off_ypart, off_fix, off_delta, off_bmax0, off_bmax1, off_rec,
        off_tab, off_off, off_base, off_left, off_imp,
        total;
};

// Coefficients a table of band_scatter_tables can need at most for `levels` polar levels of
// `azim` azimuths: offsets 0 .. azim / 2 (a multiple of 4) of n outputs; and 16 more (the
// kernel reads whole scalar loads).
static size_t band_coef_capacity(int levels, int azim, int n) {
    return (size_t)levels * n * (size_t)(1 + round_up(azim / 2, 4)) + 16;
}

// log2 of an accepted operand scale block (0 selects the default), else -1.
int scale_block_log(int32_t n) {
    if (n == 0) n = asn::kScaleBlock;
    if (n < asn::kScaleBlockMin || n > asn::kScaleBlockMax || (n & (n - 1)) != 0) return -1;
    int l = 0;
    while ((1 << l) < n) ++l;
    return l;
}

// Pitch of an ordinate's plane in cells: the cells rounded up to a scale block of 256 (1 KiB).
// The banded step streams n_azim planes at once, and at a pitch of a multiple of 16 KiB (of 64
// KiB above all) their cells meet in fewer memory channels, so there the pitch is 6 KiB more:
// kernel at 256^2 x 2048 339 -> 314 us, 512^2 x 1152 777 -> 743, 640^2 x 512 453 -> 422, 768^2 x
// 512 631 -> 599, 1024^2 x 2048 5.26 -> 4.95 ms (pads of 2 to 37 KiB do as well but for a few:
// 1 KiB at 256^2 380 us, 9 at 768^2 643).  Not below 64 KiB, where the pad would cost memory
// for nothing.  azim: the planes the banded kernel reaches with one 31-bit byte offset (0:
// another form).
int64_t plane_pitch(int64_t C, int azim) {
    const int64_t u = round_up(C, asn::kScaleBlock) / asn::kScaleBlock, v = u + 6;
    const bool pad = azim > 0 && u >= 64 && u % 16 == 0 && azim * v * asn::kScaleBlock * 4 < (int64_t)1 << 31;
    return (pad ? v : u) * asn::kScaleBlock;
}

// Columns of K that a 128-row tile of the reduced-precision contraction multiplies, 32 at a time, mean.
double tile_columns(int Q, const std::vector<float>& K32) {
    const int bm = asn::kGemmBM, bk = asn::kBK_LP;
    int64_t n = 0;
    for (int q0 = 0; q0 < Q; q0 += bm)
        for (int k0 = 0; k0 < Q; k0 += bk) {
            bool any = false;
            for (int q = q0; q < std::min(Q, q0 + bm) && !any; ++q)
                for (int k = k0; k < std::min(Q, k0 + bk) && !any; ++k) any = K32[(size_t)q * Q + k] != 0.f;
            n += any;
        }
    return (double)(n * bk) / (double)(round_up(Q, bm) / bm);
}
// Mean sources of a group of the sparse step at most.  Its time goes with their number, the tiled
// contraction's with its nonzero blocks: 200^2 x 492, us a step, 33 sources 96 (tiled 155; BF16 96 and
// 137), 78 sources 144 (196; BF16 150 and 149), 177 sources 251 (235).  Up to 170 ordinates it is the
// faster one at a dense K too (200^2 x 162 70 and 86, BF16 73 and 77; x 92 28 and 45).
int sparse_sources(int Q) { return Q <= 170 ? Q : 64; }
// ... and at most in a large problem, where the tiled contraction's launches and its last wave of
// blocks no longer count: there the matrix cores are faster at a dense K.  A step of 1 M
// cell-ordinates takes the sparse kernel about 1.8 us (2.4 and 3.0 with two and one block a CU) and
// 0.033 to 0.042 for each source, the tiled one 4.4 to 7 us by its nonzero blocks (tiles: columns of
// K that a tile of 128 rows multiplies, mean; pad: of rows, 128 at a time).  Sparse over tiled time
// of a step at 5, 16, 31 and 80 M cell-ordinates (the fused form, square grids):
//   128 ordinates, dense: FP32 0.77 1.01 1.01 1.07, BF16 0.88 1.19 1.33 1.31, Heun 0.81 1.06 0.99 0.87
//   76 sources of 128: FP32 0.59 0.76 0.74 0.81, BF16 0.64 0.85 0.99 0.98
//   92 ordinates, dense: FP32 0.80 0.75 0.88 0.92, BF16 0.70 0.83 1.02 1.02
//   162 ordinates, dense: FP32 0.91 0.88 0.87 0.86, BF16 0.95 1.16 1.14 1.17, FP16 0.94 1.20 1.18 1.20
//   256, 60 sources, 192 columns: BF16 0.75 0.84 0.95 1.02; 252, 55, 224: 0.72 0.74 0.86 0.90
//   512, 45 sources, 224 columns: BF16 0.62 0.77 0.91 0.98 (1.04 at 128 M), 58: 0.70 0.87 1.01 1.09
//   492, 50 sources, 304 columns: BF16 0.67 0.69 0.79 0.85; 362, FP16, 31, 235: 0.45 0.77 0.98 0.94
double sparse_sources_large(int Q, int dtype, bool heun, int64_t cells, const std::vector<float>& K32) {
    const double m = 1e-6 * (double)cells * Q, pad = (double)round_up(Q, asn::kGemmBM) / Q;
    const double any = (double)round_up(sparse_sources(Q), asn::kSparseChunk);
    if (dtype == ASN_GEMM_F32) return Q <= 170 && m > 12.0 && (!heun || m <= 28.0) ? std::min(any, 118.0 * pad) : any;
    if (Q <= 170) return m > 8.0 ? std::min(any, 75.0 * pad) : any;
    const bool bf16 = dtype == ASN_GEMM_BF16;
    const double per_column = asn::sparse_waves(Q) == 8 ? (bf16 ? 0.29 : 0.26) : (bf16 ? 0.196 : 0.16);
    return m > 64.0 ? std::min(any, per_column * tile_columns(Q, K32) * pad) : any;
}
// Groups of the sparse step, and the chunks of sources it takes at most (the larger its K's
// unions, the less it is worth), with the one that the kernel loads beyond the last.
size_t sparse_groups(int Q) { return ((size_t)Q + asn::kBandO - 1) / asn::kBandO; }
size_t sparse_chunks(int Q) {
    return sparse_groups(Q) * ((sparse_sources(Q) + asn::kSparseChunk - 1) / asn::kSparseChunk) + 1;
}

Layout make_layout(int nx, int ny, int Q, int dtype, int scheme, bool fused, int band_levels = 0,
                   int band_azim = 0, bool sparse = false, bool matrix = false) {
    Layout L;
    L.banded = band_levels > 0;
    L.sparse = sparse;
    L.matrix = matrix;
    // the reduced-precision step of these forms keeps the fused form's pending correction
    if (L.banded || sparse) fused = dtype != ASN_GEMM_F32 && scheme == ASN_SCHEME_EULER;
    L.fused = fused;
    L.Q = Q;
    L.Qp = (int)round_up(Q, asn::kGemmBM);
    L.C = (int64_t)nx * ny;
    L.P = plane_pitch(L.C, band_azim);
    L.lowp = dtype != ASN_GEMM_F32;
    const int strip = scheme == ASN_SCHEME_HEUN ? asn::kStripXM : asn::kStripX;
    L.tiles_x = (nx + strip - 1) / strip;
    L.tiles_y = (ny + asn::kTileY - 1) / asn::kTileY;
    // Separate stencils up to a width run over flat cell chunks, wider grids over
    // column strips; the ordinates are split into chunks sized to the grid below.
    L.flat = !fused && !L.banded && !sparse && ((scheme == ASN_SCHEME_EULER && nx <= asn::kFlatMaxNx) ||
                                     (scheme == ASN_SCHEME_HEUN && nx <= asn::kFlatMaxNxM));
    if (L.flat) {
        L.tiles_x = (int)((L.P + asn::kFlatCells - 1) / asn::kFlatCells);
        L.tiles_y = 1;
    }
    int tiles = L.tiles_x * L.tiles_y;
    if (L.banded || sparse) {
        // one block per kBandCells cells, every ordinate: each cell's Phi
        // complete
        L.tiles_x = (int)((L.C + asn::kBandCells - 1) / asn::kBandCells);
        L.tiles_y = 1;
        tiles = L.tiles_x;
        L.qchunk = Q;
        L.G = 1;
    } else if (fused) {
        // the stencil runs in the contraction's epilogue: its blocks are the
        // contraction's 128 x 128 tiles, one Phi partial per ordinate tile
        L.tiles_x = (int)(L.P / asn::kGemmBN);
        L.tiles_y = 1;
        tiles = L.tiles_x;
        L.qchunk = asn::kGemmBM;
        L.G = L.Qp / asn::kGemmBM;
    } else {
        // strip blocks: about four rounds of the 1024 resident; flat-chunk blocks: one
        // round of the 512 resident (a partial last round would cost a whole one, and
        // fewer chunks leave fewer Phi partials to sum)
        int G = L.flat ? asn::kFlatResident / tiles : (int)std::lround(4096.0 / tiles);
        G = std::max(1, std::min(G, std::min(64, std::max(1, Q / 2))));
        L.qchunk = (Q + G - 1) / G;
        L.G = (Q + L.qchunk - 1) / L.qchunk;
    }
    L.fin_blocks = (int)((L.C + 255) / 256);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (size_t)round_up((int64_t)bytes, 256);
        return o;
    };
    const size_t plane = (size_t)L.P;
    L.off_psi0 = take((size_t)Q * plane * 4);
    L.off_psi1 = take((size_t)Q * plane * 4);
    // the fused, banded and sparse steps keep Y in registers
    L.off_Y = take(fused || L.banded || sparse ? 0 : (size_t)Q * plane * 4);
    L.off_Kt = take((size_t)L.Qp * L.Qp * 4);
    L.off_Klp = take(L.lowp ? (size_t)L.Qp * L.Qp * 2 : 0);
    L.off_rdef = take((size_t)L.Qp * 4);
    {
        const int mt = L.Qp / asn::kGemmBM;
        const int bk = L.lowp ? asn::kBK_LP : asn::kBK_F32;
        L.ktab_len = mt + 1 + 2 * mt * (L.Qp / bk);   // offsets, k-steps, sub-block masks
        L.off_ktab = take((size_t)L.ktab_len * 4);
    }
    // level descriptors, 8 words; the coefficient tables of each reach; (cx, cy)
    // (on the matrix cores: one level more, the operand table and 1 KiB after it)
    L.off_band = take(L.banded ? (size_t)(band_levels + (matrix ? 1 : 0)) * 32 : 0);
    for (int r = 0; r < 3; ++r)
        L.off_bcoef[r] = take(L.banded && !matrix ? band_coef_capacity(band_levels, band_azim, 2 * r + 3) * 4 : 0);
    L.off_bcxy = take(L.banded && !matrix ? (size_t)Q * 8 : 0);
    L.off_bfrag = take(matrix ? (size_t)(band_levels + 1) * asn::band_lp_block(band_azim) * 16 + 1024 : 0);
    const size_t groups = sparse ? sparse_groups(Q) : 0, chunks = sparse ? sparse_chunks(Q) : 0;
    L.off_sgroup = take(groups * sizeof(asn::SparseGroup));
    L.off_sord = take(groups * asn::kBandO * sizeof(asn::SparseOrdinate));
    L.off_srow = take(chunks * asn::kSparseChunk * 4);
    L.off_scoef = take(chunks * asn::kSparseChunk * asn::kBandO * 4);
    L.off_qi = take((size_t)Q * sizeof(QInfo));
    L.off_coef = take(plane * 16);
    L.off_iso = take(plane * 4);
    L.off_phi64 = take(plane * 8);
    L.off_phipart = take((size_t)L.G * plane * 8);
    // (these forms) the partials of a step are read in the next one, so once per state buffer
    const size_t sets = L.by_cells() ? 2 : 1;
    L.off_blk = take(sets * tiles * L.G * 2 * 8);
    L.off_fin = take(sets * std::max<size_t>(L.fin_blocks, L.by_cells() ? tiles : 0) * 4 * 8);
    L.off_ypart = take(L.lowp && !L.by_cells() ? (size_t)(L.Qp / asn::kGemmBM) * plane * 8 : 0);
    L.off_fix = take(L.lowp && !fused ? plane * 4 : 0);
    L.off_delta = take(L.lowp && fused ? sets * plane * 4 : 0);   // (sets: follows the state buffer)
    // block maxima for the smallest scale block (any block size a problem takes fits)
    L.off_bmax0 = take((size_t)asn::scale_blocks(L.P, scale_block_log(asn::kScaleBlockMin)) * 4);
    L.off_bmax1 = take((size_t)asn::scale_blocks(L.P, scale_block_log(asn::kScaleBlockMin)) * 4);
    L.off_rec = take(asn::REC_LEN * 8);
    // the problem as a batch of one: step arguments for both buffers, block offsets,
    // buffer base and step counter
    L.off_tab = take(2 * sizeof(StepArgs));
    L.off_off = take(asn::KT_COUNT * 2 * sizeof(int));
    L.off_base = take(sizeof(int));
    L.off_left = take(sizeof(int));
    // FP64 state and iteration vectors of the implicit scheme
    size_t imp = 0;
    if (scheme == ASN_SCHEME_IMPLICIT) {
        asn::ImplicitParams ip{};
        ip.nx = nx;
        ip.ny = ny;
        ip.Q = Q;
        ip.C = L.C;
        ip.P = L.P;
        ip.gmres_restart = kGmresRestart;
        imp = asn::ImplicitSolver::bytes(ip);
    }
    L.off_imp = take(imp);
    L.total = off;
    return L;
}

}  // namespace

struct asn_problem_s {
    int nx = 0, ny = 0;
    Layout L;
    double dx = 0, dy = 0, dt = 0, W = 0, eps = 0, stability = 0;
    int64_t n_to_tfinal = 0, steps_done = 0;
    int dtype = 0, norm = 0, scheme = 0;
    int sb_log = 8;   // log2 of the cells per operand scale block
    hipStream_t stream = nullptr;
    int device = 0;
    bool owns = false;
    char* base = nullptr;
    int cur = 0;  // which psi buffer holds the current state
    std::vector<double> w;
    double tile_entries = 0;  // K entries inside the multiplied tiles (real rows/cols)
    double nonzero_entries = 0;   // nonzero entries of K in the stored operand type
    StepArgs tab[2];          // step arguments when psi buffer 0 / 1 holds the state
    int blocks[asn::KT_COUNT];
    std::unique_ptr<asn::ImplicitSolver> imp;   // the implicit scheme's solver (else null)
    int band_levels = 0, band_azim = 0, band_reach = 0;   // banded step (else 0)
    bool fuses = false;   // what asn_step_form reports of a sparse step: the form it replaces
    bool flat = false;    // whether that form's stencil runs over flat cell chunks
    // a step's block as if of a product set with so many azimuths, kBandO a wave
    // (with matrix cores: its azimuth count)
    int block_az() const { return L.sparse ? asn::sparse_waves(L.Q) * asn::kBandO : band_azim; }
    size_t band_lds() const {
        if (L.sparse) return asn::sparse_lds_bytes(L.Q);
        return asn::band_lds_bytes(band_azim, dtype, scheme == ASN_SCHEME_HEUN);
    }
};

// Problems that share their launches: a batch is up to five such groups (the problems whose steps
// are banded, banded on the matrix cores, sparse with blocks of 8 or of 16 waves, and the others).
struct Group {
    int first = 0, n = 0;    // of the batch's problems in launch order
    int scheme = 0;          // launch scheme (the flat-chunk, strip or banded form)
    int band_az = 0;         // banded: the largest azimuth count, LDS bytes per block and reach
    size_t band_lds = 0;
    int band_reach = 0;
    int grid[asn::KT_COUNT] = {};
    asn::BatchArgs args{};
};
constexpr int kMaxGroups = 5;
struct Plan {
    int n = 0, n_groups = 0;
    asn_problem order[asn::kMaxArm];
    Group groups[kMaxGroups];
};

struct asn_batch_s {
    Plan plan;
    int dtype = 0, scheme = 0;
    int index[asn::kMaxArm];   // problem order[i] is the caller's problem index[i]
    hipStream_t stream = nullptr;
    char* dev = nullptr;
    std::map<int64_t, std::pair<hipGraph_t, hipGraphExec_t>> graphs;
};

namespace {

StepArgs make_args(asn_problem p, int cur) {
    const Layout& L = p->L;
    char* b = p->base;
    StepArgs a{};
    a.nx = p->nx;
    a.ny = p->ny;
    a.Q = L.Q;
    a.Qp = L.Qp;
    a.C = L.C;
    a.P = L.P;
    a.G = L.G;
    a.qchunk = L.qchunk;
    a.tiles_x = L.tiles_x;
    a.tiles_y = L.tiles_y;
    a.fin_blocks = L.fin_blocks;
    a.dtype = p->dtype;
    a.sb_log = p->sb_log;
    a.fused = L.fused ? 1 : 0;
    a.W = p->W;
    a.area = p->dx * p->dy;
    float* psi0 = reinterpret_cast<float*>(b + L.off_psi0);
    float* psi1 = reinterpret_cast<float*>(b + L.off_psi1);
    a.psi = cur == 0 ? psi0 : psi1;
    a.psi_new = cur == 0 ? psi1 : psi0;
    a.Y = reinterpret_cast<float*>(b + L.off_Y);
    a.Kt = reinterpret_cast<const float*>(b + L.off_Kt);
    a.Klp = reinterpret_cast<const uint16_t*>(b + L.off_Klp);
    a.rdef = reinterpret_cast<const float*>(b + L.off_rdef);
    a.ktab = reinterpret_cast<const int*>(b + L.off_ktab);
    a.qi = reinterpret_cast<const QInfo*>(b + L.off_qi);
    a.coef = reinterpret_cast<const float4*>(b + L.off_coef);
    a.iso = reinterpret_cast<float*>(b + L.off_iso);
    a.phi64 = reinterpret_cast<double*>(b + L.off_phi64);
    a.phi_part = reinterpret_cast<double*>(b + L.off_phipart);
    a.blk_part = reinterpret_cast<double*>(b + L.off_blk);
    a.fin_part = reinterpret_cast<double*>(b + L.off_fin);
    a.ypart = reinterpret_cast<double*>(b + L.off_ypart);
    a.fix = reinterpret_cast<float*>(b + L.off_fix);
    a.delta = reinterpret_cast<float*>(b + L.off_delta);
    unsigned* bm0 = reinterpret_cast<unsigned*>(b + L.off_bmax0);
    unsigned* bm1 = reinterpret_cast<unsigned*>(b + L.off_bmax1);
    a.bmax_cur = cur == 0 ? bm0 : bm1;
    a.bmax_next = cur == 0 ? bm1 : bm0;
    a.rec = reinterpret_cast<double*>(b + L.off_rec);
    if (L.by_cells() && L.lowp) {
        a.delta_next = a.delta + (cur ? 0 : L.P);
        a.delta += cur ? L.P : 0;
    }
    if (L.by_cells() && cur) {
        a.blk_part += 2 * (size_t)L.tiles_x;
        a.fin_part += 4 * (size_t)L.tiles_x;
    }
    if (L.banded) {
        (L.matrix ? a.bpairs : a.band) = reinterpret_cast<const uint4*>(b + L.off_band);   // two per level
        a.bfrag = L.matrix ? reinterpret_cast<const uint4*>(b + L.off_bfrag) : nullptr;
        a.bcoef3 = reinterpret_cast<const float*>(b + L.off_bcoef[0]);
        a.bcoef5 = reinterpret_cast<const float*>(b + L.off_bcoef[1]);
        a.bcoef7 = reinterpret_cast<const float*>(b + L.off_bcoef[2]);
        a.bcxy = reinterpret_cast<const float2*>(b + L.off_bcxy);
        a.n_lev = p->band_levels;
        a.n_az = p->band_azim;
        a.reach = p->band_reach;
    }
    if (L.sparse) {
        a.sp_group = reinterpret_cast<const asn::SparseGroup*>(b + L.off_sgroup);
        a.sp_ord = reinterpret_cast<const asn::SparseOrdinate*>(b + L.off_sord);
        a.sp_row = reinterpret_cast<const uint32_t*>(b + L.off_srow);
        a.sp_coef = reinterpret_cast<const float*>(b + L.off_scoef);
        a.band = reinterpret_cast<const uint4*>(a.sp_group);
        a.n_az = p->block_az();
    }
    return a;
}

// The problem as a batch of one (tables in its workspace).
asn::BatchArgs single_batch(asn_problem p) {
    const Layout& L = p->L;
    asn::BatchArgs b{};
    b.tab = reinterpret_cast<const StepArgs*>(p->base + L.off_tab);
    b.off = reinterpret_cast<const int*>(p->base + L.off_off);
    b.base = reinterpret_cast<const int*>(p->base + L.off_base);
    b.limit = reinterpret_cast<const int*>(p->base + L.off_left);
    b.n = 1;
    return b;
}

hipError_t arm_single(asn_problem p, int64_t limit) {
    asn::ArmArgs v{};
    v.limit[0] = (int)std::min<int64_t>(limit, 1 << 30);
    v.cur[0] = p->cur;
    const Layout& L = p->L;
    return asn::launch_arm(reinterpret_cast<int*>(p->base + L.off_left),
                           reinterpret_cast<int*>(p->base + L.off_base), 1, v, p->stream);
}

// K of a quadrature/width/normalisation, cached across problems (set-up is O(Q^2)
// with a scaling loop; serving creates many problems with the same ordinates).
bool cached_kernel(int Q, const std::vector<double>& om, const std::vector<double>& w, double eps,
                   int mode, std::vector<double>& K, std::string& err) {
    static std::mutex mu;
    static std::vector<std::pair<std::vector<double>, std::vector<double>>> cache;  // key, K
    std::vector<double> key(om);
    key.insert(key.end(), w.begin(), w.end());
    key.push_back(eps);
    key.push_back((double)mode);
    {
        std::lock_guard<std::mutex> g(mu);
        for (auto& e : cache)
            if (e.first == key) {
                K = e.second;
                return true;
            }
    }
    if (!asn::kernel_matrix(Q, om.data(), w.data(), eps, mode, K, err)) return false;
    std::lock_guard<std::mutex> g(mu);
    if (cache.size() >= 8) cache.erase(cache.begin());
    cache.emplace_back(std::move(key), K);
    return true;
}

asn_status check_grid(const asn_grid* g) {
    if (!g) return fail(ASN_E_INVALID, "grid is NULL");
    if (g->nx < 1 || g->ny < 1) return fail(ASN_E_INVALID, "nx and ny must be >= 1");
    if (!(g->x_max > g->x_min) || !(g->y_max > g->y_min) || !std::isfinite(g->x_max - g->x_min) ||
        !std::isfinite(g->y_max - g->y_min))
        return fail(ASN_E_INVALID, "empty or non-finite domain");
    // plane byte offsets are 32-bit in the stencil's buffer addressing
    if ((int64_t)g->nx * g->ny > (int64_t)1 << 29) return fail(ASN_E_INVALID, "grid too large");
    return ASN_OK;
}

asn_status resolve_quadrature(const asn_quadrature* q, std::vector<double>& om,
                              std::vector<double>& w) {
    if (!q) return fail(ASN_E_INVALID, "quadrature is NULL");
    if (q->q_custom > 0) {
        if (!q->omega_xyz || !q->weights)
            return fail(ASN_E_INVALID, "custom quadrature needs omega_xyz and weights");
        const int Q = q->q_custom;
        om.assign(q->omega_xyz, q->omega_xyz + 3 * (size_t)Q);
        w.assign(q->weights, q->weights + Q);
        for (int i = 0; i < Q; ++i) {
            const double n = std::sqrt(om[3 * i] * om[3 * i] + om[3 * i + 1] * om[3 * i + 1] +
                                       om[3 * i + 2] * om[3 * i + 2]);
            if (!(std::fabs(n - 1.0) <= 1e-12)) return fail(ASN_E_INVALID, "ordinate not unit length");
            if (!(w[i] > 0.0) || !std::isfinite(w[i])) return fail(ASN_E_INVALID, "weight must be > 0");
        }
        return ASN_OK;
    }
    if (q->icosahedron_order > 0) {
        if (q->icosahedron_order < 2 || q->icosahedron_order > 41)
            return fail(ASN_E_INVALID, "icosahedron_order must be in [2, 41]");
        asn::icosahedron_quadrature(q->icosahedron_order, om, w);
        return ASN_OK;
    }
    if (q->n_polar < 1 || q->n_azim < 1) return fail(ASN_E_INVALID, "n_polar and n_azim must be >= 1");
    if ((int64_t)q->n_polar * q->n_azim > 16384) return fail(ASN_E_INVALID, "too many ordinates");
    asn::product_quadrature(q->n_polar, q->n_azim, om, w);
    return ASN_OK;
}

// T(fp32(K)) as 16-bit patterns in a ld x ld zero-padded row-major array, and the
// row defects r_q = fp32(1 - sum_p T(K)_qp) with the sum taken in FP64.
void quantise_kernel(int Q, const double* K, int dtype, int ld, uint16_t* out, float* rdef) {
    for (int q = 0; q < Q; ++q) {
        double sum = 0.0;
        for (int k = 0; k < Q; ++k) {
            const float f = (float)K[(size_t)q * Q + k];
            uint16_t h;
            double back;
            if (dtype == ASN_GEMM_BF16) {
                h = asn::float_to_bf16_rne(f);
                back = asn::bf16_to_float(h);
            } else {
                h = asn::float_to_half_rne(f);
                back = asn::half_to_float(h);
            }
            out[(size_t)q * ld + k] = h;
            sum += back;
        }
        rdef[q] = (float)(1.0 - sum);
    }
}

int quad_size(const asn_quadrature* q) {
    if (q->q_custom > 0) return q->q_custom;
    if (q->icosahedron_order > 0) return 10 * (q->icosahedron_order - 1) * (q->icosahedron_order - 1) + 2;
    return q->n_polar * q->n_azim;
}

asn_status check_field(const float* f, int64_t n, const char* name, bool allow_null) {
    if (!f) return allow_null ? ASN_OK : fail(ASN_E_INVALID, std::string(name) + " is NULL");
    for (int64_t i = 0; i < n; ++i)
        if (!(f[i] >= 0.f) || !std::isfinite(f[i]))
            return fail(ASN_E_INVALID, std::string(name) + " must be finite and >= 0");
    return ASN_OK;
}

// Whether forward-Euler steps run fused (stencil in the contraction's epilogue).
// ASN_FORM_AUTO: 16-bit operands always fuse; FP32 fuses problems below 2^25
// cell-ordinates and runs the separate contraction (four blocks per CU) and flat
// stencil above, where they are faster (400^2 x 512: 0.48 vs 0.50 ms per step;
// 700^2 x 1152: 2.98 vs 3.32 ms; 1024^2 x 2048: 11.9 vs 15.8 ms; 128^2 x 512: 0.093 vs
// 0.078 ms).  Wider grids than the flat stencil takes fuse.
bool use_fused(int dtype, int scheme, int form, int nx, int ny, int Q) {
    if (!asn::can_fuse(dtype, scheme) || form == ASN_FORM_SEPARATE) return false;
    if (form == ASN_FORM_BANDED) return false;
    if (form == ASN_FORM_FUSED || dtype != ASN_GEMM_F32) return true;
    return !(nx <= asn::kFlatMaxNx && (double)nx * ny * Q >= 33554432.0);
}

// Whether a problem may take the banded step: forward Euler, or Heun in FP32 unless separate
// kernels were asked for (its form is reported as separate either way), on a product set whose
// azimuth count has a kernel instance (FP32: 8 .. 64 in steps of 8; BF16 / FP16: 32, 48 or
// 64) (ASN_FORM_AUTO or ASN_FORM_BANDED); the stored K must then also have the banded
// form (band_form).
bool band_candidate(int dtype, int scheme, int form, const asn_quadrature* q, int64_t C) {
    // the kernel addresses one polar level of planes (n_azim * P floats) with byte
    // offsets below 2^31
    const int64_t P = round_up(C, asn::kScaleBlock);
    const bool az_ok = asn::band_azimuths_supported(q->n_azim, dtype);
    const bool scheme_ok = scheme == ASN_SCHEME_EULER
                               ? form == ASN_FORM_AUTO || form == ASN_FORM_BANDED
                               : scheme == ASN_SCHEME_HEUN && dtype == ASN_GEMM_F32 &&
                                     (form == ASN_FORM_AUTO || form == ASN_FORM_FUSED);
    return az_ok && scheme_ok && (int64_t)std::max(q->n_azim, 1) * P * 4 < ((int64_t)1 << 31) &&
           q->q_custom == 0 && q->icosahedron_order == 0 && q->n_polar >= 1;
}

// Whether the Heun passes of a product set of few levels leave the banded kernel, which takes two
// levels' time beyond the set's and whose blocks of n_azim / 4 waves leave a CU's 16 wave slots empty
// (24, 40 to 56 azimuths) or start and end at once (64), to the sparse one: from 2 M cell-ordinates on
// that is the faster one, and the banded one slower than separate kernels at large grids.  Us a step
// banded, sparse, separate: 2 x 64, 400^2, beta 4.5 240, 138, 209, beta 20 324, 247, 252; 800^2 dense
// 1343, 973, 1110; 2 x 40 dense, 800^2 842, 481, 683; 1 x 24, 800^2 288, 153, 202; 3 x 40 dense, 800^2
// 1189, 884, 1044.  2 x 32 (dense, 800^2 435, 366, 544), 3 x 32 (596, 618, 805), 3 x 48 (1351, 1166, 1641)
// and more levels stay banded.
bool heun_few_levels(const asn_quadrature* q, int64_t C) {
    const int l = q->n_polar, az = q->n_azim;
    return (double)C * l * az >= 2e6 && az >= 24 && (l == 1 || (l == 2 && az != 32) || (l == 3 && az == 40));
}

// Bytes that either layout of the banded step needs.
size_t band_layouts(const asn_grid& g, const asn_quadrature& q, int Q, int dtype, int scheme) {
    size_t bytes = make_layout(g.nx, g.ny, Q, dtype, scheme, false, q.n_polar, q.n_azim).total;
    if (dtype != ASN_GEMM_F32)
        bytes = std::max(bytes, make_layout(g.nx, g.ny, Q, dtype, scheme, false, q.n_polar, q.n_azim, false, true).total);
    return bytes;
}

// Whether a problem that does not take the banded step may take the sparse one (unless separate
// kernels were asked for; it reports the form it replaces): its LDS rows fit a block, and a
// plane's bytes 31 bits.  K must then also be sparse enough (sparse_form).
bool sparse_candidate(int dtype, int scheme, int form, int Q, int64_t C) {
    const bool heun = scheme == ASN_SCHEME_HEUN;
    const bool ok = (form == ASN_FORM_AUTO || form == ASN_FORM_FUSED) &&
                    (heun ? dtype == ASN_GEMM_F32 : scheme == ASN_SCHEME_EULER);
    return ok && asn::sparse_lds_bytes(Q) + asn::kSparseSums <= asn::kLds &&
           round_up(C, asn::kScaleBlock) * 4 < ((int64_t)1 << 31);
}

}  // namespace

extern "C" {

asn_status asn_options_default(asn_options* opt) {
    if (!opt) return fail(ASN_E_INVALID, "options is NULL");
    std::memset(opt, 0, sizeof(*opt));
    opt->gemm_dtype = ASN_GEMM_F32;
    opt->normalization = ASN_NORM_SYM;
    opt->cfl = 0.95;
    opt->scale_block = asn::kScaleBlock;
    return ASN_OK;
}

asn_status asn_workspace_size(const asn_grid* grid, const asn_quadrature* quad,
                              const asn_options* opt, size_t* bytes) {
    asn_status s = check_grid(grid);
    if (s != ASN_OK) return s;
    if (!quad || !bytes) return fail(ASN_E_INVALID, "NULL argument");
    const int Q = quad_size(quad);
    if (Q < 1) return fail(ASN_E_INVALID, "Q must be >= 1");
    asn_options d;
    asn_options_default(&d);
    const int dtype = opt ? opt->gemm_dtype : d.gemm_dtype;
    const int scheme = opt ? opt->scheme : d.scheme;
    const int form = opt ? opt->step_form : d.step_form;
    if (scale_block_log(opt ? opt->scale_block : d.scale_block) < 0)
        return fail(ASN_E_INVALID, "scale_block must be a power of two from 64 to 4096 (or 0)");
    if (form < ASN_FORM_AUTO || form > ASN_FORM_BANDED)
        return fail(ASN_E_INVALID, "step_form must be ASN_FORM_AUTO, _SEPARATE, _FUSED or _BANDED");
    if (form == ASN_FORM_BANDED) {
        if (!band_candidate(dtype, scheme, form, quad, (int64_t)grid->nx * grid->ny))
            return fail(ASN_E_UNSUPPORTED, "ASN_FORM_BANDED needs forward Euler on a product set "
                                           "with n_azim in {8, 16, ..., 64} (FP32) or {32, 48, 64} "
                                           "(BF16, FP16)");
        *bytes = band_layouts(*grid, *quad, Q, dtype, scheme);
        return ASN_OK;
    }
    const bool fused = use_fused(dtype, scheme, form, grid->nx, grid->ny, Q);
    size_t total = make_layout(grid->nx, grid->ny, Q, dtype, scheme, fused).total;
    // which of the forms a K has is known only once it is built: cover every layout
    if (band_candidate(dtype, scheme, form, quad, (int64_t)grid->nx * grid->ny))
        total = std::max(total, band_layouts(*grid, *quad, Q, dtype, scheme));
    if (sparse_candidate(dtype, scheme, form, Q, (int64_t)grid->nx * grid->ny))
        total = std::max(total, make_layout(grid->nx, grid->ny, Q, dtype, scheme, false, 0, 0, true).total);
    *bytes = total;
    return ASN_OK;
}

asn_status asn_create(const asn_grid* grid, const asn_quadrature* quad, const float* sigma_s,
                      const float* sigma_a, const float* sigma_as, const float* source,
                      double kernel_beta, double t_final, const asn_options* opt_in,
                      void* hip_stream, void* workspace, size_t workspace_bytes,
                      asn_problem* out) {
    if (!out) return fail(ASN_E_INVALID, "out is NULL");
    *out = nullptr;
    asn_status s = check_grid(grid);
    if (s != ASN_OK) return s;
    asn_options opt;
    if (opt_in) opt = *opt_in;
    else asn_options_default(&opt);
    if (opt.gemm_dtype < ASN_GEMM_F32 || opt.gemm_dtype > ASN_GEMM_F16)
        return fail(ASN_E_INVALID, "unknown gemm_dtype");
    if (opt.normalization != ASN_NORM_SYM && opt.normalization != ASN_NORM_ROW)
        return fail(ASN_E_INVALID, "unknown normalization");
    const int sb_log = scale_block_log(opt.scale_block);
    if (sb_log < 0)
        return fail(ASN_E_INVALID, "scale_block must be a power of two from 64 to 4096 (or 0)");
    if (opt.scheme != ASN_SCHEME_EULER && opt.scheme != ASN_SCHEME_HEUN &&
        opt.scheme != ASN_SCHEME_IMPLICIT)
        return fail(ASN_E_INVALID, "unknown scheme");
    const bool implicit = opt.scheme == ASN_SCHEME_IMPLICIT;
    if (opt.step_form < ASN_FORM_AUTO || opt.step_form > ASN_FORM_BANDED)
        return fail(ASN_E_INVALID, "step_form must be ASN_FORM_AUTO, _SEPARATE, _FUSED or _BANDED");
    if (opt.source_test != ASN_SOURCE_TEST_ABSOLUTE && opt.source_test != ASN_SOURCE_TEST_RELATIVE)
        return fail(ASN_E_INVALID, "source_test must be ASN_SOURCE_TEST_ABSOLUTE or ASN_SOURCE_TEST_RELATIVE");
    if (opt.dt_rule != ASN_DT_STREAMING && opt.dt_rule != ASN_DT_STIFF)
        return fail(ASN_E_INVALID, "unknown dt_rule");
    if (!(opt.cfl > 0.0)) return fail(ASN_E_INVALID, "cfl must be > 0");
    if (opt.cfl > 1.0 && !implicit)
        return fail(ASN_E_UNSTABLE, "cfl above 1 is unstable for the explicit step");
    if (!(t_final > 0.0) || !std::isfinite(t_final)) return fail(ASN_E_INVALID, "t_final must be > 0");
    if (!(kernel_beta > 0.0) && !(opt.eps_override > 0.0))
        return fail(ASN_E_INVALID, "kernel_beta must be > 0");

    std::vector<double> om, w;
    s = resolve_quadrature(quad, om, w);
    if (s != ASN_OK) return s;
    const int Q = (int)w.size();
    const int64_t C = (int64_t)grid->nx * grid->ny;
    if ((s = check_field(sigma_s, C, "sigma_s", false)) != ASN_OK) return s;
    if ((s = check_field(sigma_a, C, "sigma_a", false)) != ASN_OK) return s;
    if ((s = check_field(sigma_as, C, "sigma_as", false)) != ASN_OK) return s;
    if ((s = check_field(source, C, "source", true)) != ASN_OK) return s;

    auto* p = new asn_problem_s();
    p->nx = grid->nx;
    p->ny = grid->ny;
    p->dx = (grid->x_max - grid->x_min) / grid->nx;
    p->dy = (grid->y_max - grid->y_min) / grid->ny;
    p->dtype = opt.gemm_dtype;
    p->sb_log = sb_log;
    p->norm = opt.normalization;
    p->scheme = opt.scheme;
    p->stream = reinterpret_cast<hipStream_t>(hip_stream);
    p->w = w;
    double W = 0.0;
    for (double v : w) W += v;
    p->W = W;
    p->eps = opt.eps_override > 0.0 ? opt.eps_override : kernel_beta / Q;

    // kernel matrix
    std::vector<double> K;
    std::string err;
    if (!cached_kernel(Q, om, w, p->eps, p->norm == ASN_NORM_SYM ? 0 : 1, K, err)) {
        delete p;
        return fail(ASN_E_UNSUPPORTED, err);
    }

    // time step
    const double srate = asn::stability_rate(Q, om.data(), K.data(), p->dx, p->dy, C, sigma_a,
                                             sigma_s, sigma_as);
    if (opt.dt_rule == ASN_DT_STIFF)
        asn::stiff_time_step(Q, om.data(), p->dx, p->dy, srate, opt.cfl, t_final, p->dt,
                             p->n_to_tfinal);
    else
        asn::cfl_time_step(Q, om.data(), p->dx, p->dy, opt.cfl, t_final, p->dt, p->n_to_tfinal);
    if (opt.dt_override > 0.0) {
        double rate = 0.0;
        for (int q = 0; q < Q; ++q)
            rate = std::fmax(rate, std::fabs(om[3 * q]) / p->dx + std::fabs(om[3 * q + 1]) / p->dy);
        if (!implicit && opt.dt_override * rate > opt.cfl * (1.0 + 1e-12)) {
            delete p;
            return fail(ASN_E_UNSTABLE, "dt_override exceeds the CFL bound");
        }
        p->dt = opt.dt_override;
        p->n_to_tfinal = (int64_t)std::llround(t_final / p->dt);
    }
    p->stability = p->dt * srate;

    // banded step when K has that form (ASN_FORM_AUTO) or on request (ASN_FORM_BANDED)
    asn::BandForm bf;
    bool banded = false, matrix = false;
    std::vector<uint32_t> ddesc;   // its level descriptors and coefficients
    std::array<std::vector<float>, 3> bcoef;
    std::vector<double> gain;
    asn::SparseForm sf;
    bool sparse = sparse_candidate(p->dtype, p->scheme, opt.step_form, Q, C);
    const bool may_band = band_candidate(p->dtype, p->scheme, opt.step_form, quad, C) &&
                          !(p->scheme == ASN_SCHEME_HEUN && heun_few_levels(quad, C));
    const int Qp = (int)round_up(Q, asn::kGemmBM);
    std::vector<uint16_t> Klp;   // BF16 / FP16 K and its row defects
    std::vector<float> rdef((size_t)Qp, 0.f);
    if (p->dtype != ASN_GEMM_F32) {
        Klp.assign((size_t)Qp * Qp, 0);
        quantise_kernel(Q, K.data(), p->dtype, Qp, Klp.data(), rdef.data());
    }
    if (may_band || sparse) {
        // the values the kernels multiply: FP32 K, or its BF16 / FP16 rounding
        std::vector<float> K32((size_t)Q * Q);
        for (int q = 0; q < Q; ++q)
            for (int k = 0; k < Q; ++k) {
                const size_t i = (size_t)q * Q + k, j = (size_t)q * Qp + k;
                K32[i] = p->dtype == ASN_GEMM_F32    ? (float)K[i]
                         : p->dtype == ASN_GEMM_BF16 ? asn::bf16_to_float(Klp[j])
                                                     : asn::half_to_float(Klp[j]);
            }
        banded = may_band &&
                 asn::band_form(quad->n_polar, quad->n_azim, K32.data(), asn::kBandMaxReach, asn::kBandNarrow, bf);
        banded = banded && asn::band_supported(bf.azim, p->dtype, bf.reach, p->scheme == ASN_SCHEME_HEUN) &&
                 asn::band_scatter_tables(bf, p->dtype, ddesc, bcoef, gain);
        // the kernel takes one row defect per level (the rows of a level hold the same values, so
        // their FP64 sums agree; checked)
        for (int q = 0; banded && p->dtype != ASN_GEMM_F32 && q < Q; ++q)
            if (rdef[(size_t)q] != rdef[(size_t)(q / quad->n_azim) * quad->n_azim]) banded = false;
        matrix = banded && p->dtype != ASN_GEMM_F32 && asn::band_on_matrix_cores(bf, ddesc, C);
        // ... of the coefficients it multiplies
        for (int q = 0; banded && !matrix && p->dtype != ASN_GEMM_F32 && q < Q; ++q)
            rdef[(size_t)q] = (float)((double)rdef[(size_t)q] - gain[(size_t)(q / quad->n_azim)]);
        sparse = sparse && !banded &&
                 asn::sparse_form(Q, K32.data(), asn::kBandO, asn::kSparseChunk, sparse_chunks(Q) - 1, sf) &&
                 (double)sf.first.back() * asn::kSparseChunk <=
                     (double)sparse_groups(Q) * sparse_sources_large(Q, p->dtype, p->scheme == ASN_SCHEME_HEUN, C, K32);
    }
    if (opt.step_form == ASN_FORM_BANDED && !banded) {
        delete p;
        return fail(ASN_E_UNSUPPORTED,
                    "ASN_FORM_BANDED needs forward Euler on a product set with n_azim in "
                    "{8, 16, ..., 64} (FP32) or {32, 48, 64} (BF16, FP16), n_azim * cells below 2^29, "
                    "and a stored K that couples polar levels at most 3 apart (BF16 at 48 or "
                    "64 azimuths: 2) and is circulant along the azimuth");
    }
    if (banded) {
        p->band_levels = bf.levels;
        p->band_azim = bf.azim;
        p->band_reach = bf.reach;
        p->L = make_layout(p->nx, p->ny, Q, p->dtype, p->scheme, false, bf.levels, bf.azim, false, matrix);
    } else {
        p->L = make_layout(p->nx, p->ny, Q, p->dtype, p->scheme,
                           use_fused(p->dtype, p->scheme, opt.step_form, p->nx, p->ny, Q));
        p->fuses = p->L.fused;
        p->flat = p->L.flat;
        if (sparse) p->L = make_layout(p->nx, p->ny, Q, p->dtype, p->scheme, false, 0, 0, true);
    }
    const Layout& L = p->L;
    if (workspace) {
        if (workspace_bytes < L.total) {
            delete p;
            return fail(ASN_E_OOM, "workspace smaller than asn_workspace_size");
        }
        p->base = static_cast<char*>(workspace);
        p->owns = false;
    } else {
        void* m = nullptr;
        if (hipMalloc(&m, L.total) != hipSuccess) {
            delete p;
            return fail(ASN_E_OOM, "hipMalloc of the problem memory failed");
        }
        p->base = static_cast<char*>(m);
        p->owns = true;
    }
    (void)hipGetDevice(&p->device);

    // host-side tables
    std::vector<float> Kt((size_t)L.Qp * L.Qp, 0.f);
    for (int q = 0; q < Q; ++q)
        for (int k = 0; k < Q; ++k) Kt[(size_t)k * L.Qp + q] = (float)K[(size_t)q * Q + k];
    // k-steps per M-tile whose tile of the stored K (FP32 or 16-bit) has a nonzero entry.
    // Steps inside the tile's own ordinate range come last: the fused epilogue then
    // reads rows that the block (and its neighbours) has just streamed through L2.
    // After the k-step list, one mask per entry.  FP32: bit 4 s + g is set when rows
    // m0 + 16 s .. m0 + 16 s + 15 and columns k0 + 4 g .. k0 + 4 g + 3 of the step's K tile
    // (one MFMA operand block) have a nonzero entry; the kernel skips the products of the
    // other blocks.  16-bit operands: bit s for the 16-row sub-block (the kernel
    // multiplies whole tiles).
    std::vector<int> ktab((size_t)L.ktab_len, 0);
    {
        const int mt_n = L.Qp / asn::kGemmBM;
        const int bk = L.lowp ? asn::kBK_LP : asn::kBK_F32;
        const int nk = (Q + bk - 1) / bk;
        std::vector<int> entries, masks;
        double cover = 0;
        for (int mt = 0; mt < mt_n; ++mt) {
            ktab[mt] = (int)entries.size();
            const int m0 = mt * asn::kGemmBM, m1 = std::min(Q, m0 + asn::kGemmBM);
            std::vector<int> own, own_mask;
            for (int kt = 0; kt < nk; ++kt) {
                const int k0 = kt * bk, k1 = std::min(Q, k0 + bk);
                uint32_t mask = 0;
                for (int m = m0; m < m1; ++m)
                    for (int k = k0; k < k1; ++k)
                        if (L.lowp ? (Klp[(size_t)m * L.Qp + k] & 0x7FFFu) != 0
                                   : Kt[(size_t)k * L.Qp + m] != 0.f)
                            mask |= L.lowp ? 1u << ((m - m0) / 16) : 1u << (4 * ((m - m0) / 16) + (k - k0) / 4);
                if (mask) {
                    const bool is_own = L.fused && k0 >= m0 && k0 < m0 + asn::kGemmBM;
                    (is_own ? own : entries).push_back(kt);
                    (is_own ? own_mask : masks).push_back((int)mask);
                    // K entries the kernel multiplies: whole tiles (16-bit operands) or
                    // the nonzero 16 x 4 blocks (FP32)
                    if (L.lowp) {
                        cover += (double)(m1 - m0) * (k1 - k0);
                    } else {
                        for (int b = 0; b < 32; ++b) {
                            if (!(mask & (1u << b))) continue;
                            const int r0 = m0 + 16 * (b / 4), c0 = k0 + 4 * (b % 4);
                            cover += (double)std::max(0, std::min(m1, r0 + 16) - r0) *
                                     std::max(0, std::min(k1, c0 + 4) - c0);
                        }
                    }
                }
            }
            entries.insert(entries.end(), own.begin(), own.end());
            masks.insert(masks.end(), own_mask.begin(), own_mask.end());
        }
        ktab[mt_n] = (int)entries.size();
        std::copy(entries.begin(), entries.end(), ktab.begin() + mt_n + 1);
        std::copy(masks.begin(), masks.end(), ktab.begin() + mt_n + 1 + entries.size());
        p->tile_entries = cover;
    }
    {   // the method's own products: nonzeros of the stored K
        double nz = 0;
        for (int q = 0; q < Q; ++q)
            for (int k = 0; k < Q; ++k)
                nz += L.lowp ? ((Klp[(size_t)q * L.Qp + k] & 0x7FFFu) != 0)
                             : (Kt[(size_t)k * L.Qp + q] != 0.f);
        p->nonzero_entries = nz;
    }
    if (banded) {   // the banded step multiplies each pair's run (wide runs padded to 4);
                    // the reduced-precision one each pair's whole n_az x n_az block
        double ex = 0;
        for (int i = 0; i < bf.levels; ++i) {
            const int n = (int)bf.desc[(size_t)i * 8];
            for (int t = 0; t < n; ++t) {
                const uint32_t code = bf.desc[(size_t)i * 8 + 1 + t];
                int lo = 0, len = 0;
                asn::band_run(code, bf.azim, lo, len);
                ex += L.lowp ? (double)bf.azim * bf.azim
                             : (double)bf.azim * ((code & 64u) ? (len + 3) / 4 * 4 : len);
            }
        }
        p->tile_entries = ex;
    }
    std::vector<QInfo> qi(Q);
    for (int q = 0; q < Q; ++q) {
        const double xi = om[3 * q], eta = om[3 * q + 1];
        qi[q].cx = (float)(p->dt * std::fabs(xi) / p->dx);
        qi[q].cy = (float)(p->dt * std::fabs(eta) / p->dy);
        qi[q].wf = (float)w[q];
        qi[q].dir = (xi > 0 ? 1 : 0) | (xi < 0 ? 2 : 0) | (eta > 0 ? 4 : 0) | (eta < 0 ? 8 : 0);
        qi[q].w = w[q];
    }
    std::vector<float4> coef((size_t)L.P, make_float4(0.f, 0.f, 0.f, 0.f));
    for (int64_t c = 0; c < C; ++c) {
        coef[c].x = (float)(p->dt * (double)sigma_a[c]);
        coef[c].y = (float)(p->dt * (double)sigma_s[c]);
        coef[c].z = (float)(p->dt * (double)sigma_as[c]);
        coef[c].w = source ? (float)(p->dt * (double)source[c]) : 0.f;
    }

    std::vector<float> dcxy;   // banded kernel: (cx, cy) per ordinate
    std::vector<uint16_t> bfrag;   // (on the matrix cores) its operand table
    if (matrix) {
        // Per level the coupled pairs of level l first, then zero operands whose partner is the level
        // itself (the kernel runs the first 2 reach + 1 slots of its launch's largest reach, with no
        // count); then (cx, cy) of level l - 1's ordinates (its update runs a level behind); the last
        // block holds only the last level's.
        constexpr int slots = 2 * asn::kBandMaxReach + 1;
        const size_t block = asn::band_lp_block(bf.azim), pairs = block - (size_t)bf.azim / 2;   // uint4
        ddesc.assign((size_t)(bf.levels + 1) * 8, 0u);
        for (int i = 0; i <= bf.levels; ++i) {
            const int n = i < bf.levels ? (int)bf.desc[(size_t)i * 8] : 0;
            uint32_t kc = 0;
            for (int t = 0; t < slots; ++t)
                kc |= (t < n ? ((bf.desc[(size_t)i * 8 + 1 + t] >> 8) & 7u) : (uint32_t)bf.reach) << (4 * t);
            ddesc[(size_t)i * 8] = (uint32_t)n;
            ddesc[(size_t)i * 8 + 1] = (uint32_t)(i * block);
            ddesc[(size_t)i * 8 + 2] = kc;
            for (int t = 0; t < n; ++t) asn::band_lp_fragments(bf, i, t, p->dtype, bfrag);
            bfrag.resize((i * block + pairs) * 8, 0);
            for (int az = 0; az < bf.azim; ++az) {
                float c[2] = {0.f, 0.f};
                if (i > 0) {
                    c[0] = qi[(size_t)(i - 1) * bf.azim + az].cx;
                    c[1] = qi[(size_t)(i - 1) * bf.azim + az].cy;
                }
                uint16_t w[4];
                std::memcpy(w, c, sizeof(c));
                bfrag.insert(bfrag.end(), w, w + 4);
            }
        }
    } else if (banded) {
        for (int i = 0; i < bf.levels; ++i)   // the FP64 weight of a level's ordinates
            std::memcpy(&ddesc[8 * (size_t)i + 4], &qi[(size_t)i * bf.azim].w, 8);
        for (const QInfo& v : qi) {
            dcxy.push_back(v.cx);
            dcxy.push_back(v.cy);
        }
    }
    std::vector<asn::SparseGroup> sgroup;   // sparse kernel
    std::vector<asn::SparseOrdinate> sord;
    std::vector<uint32_t> srow;
    if (sparse) {
        for (size_t g = 0; g + 1 < sf.first.size(); ++g) {
            asn::SparseGroup v{};
            for (int o = 0; o < asn::kBandO; ++o) {
                const int q = sf.order[g * asn::kBandO + o];
                v.ord[o] = (uint32_t)q << 4 | (uint32_t)qi[q].dir;
                const bool again = (int)g * asn::kBandO + o >= Q;
                sord.push_back({qi[q].cx, qi[q].cy, rdef[q], 0.f, again ? 0.0 : qi[q].w, 0.0});
            }
            v.first = sf.first[g];
            v.chunks = sf.first[g + 1] - sf.first[g];
            sgroup.push_back(v);
        }
        for (int k : sf.src) srow.push_back(4u * (uint32_t)(k * asn::kBandCells));
    }
    auto bail = [&](asn_status st) {
        if (p->owns) (void)hipFree(p->base);
        delete p;
        return st;
    };
    char* b = p->base;
    auto copy_tables = [&] {
        auto copy = [&](size_t off, const void* from, size_t bytes) {
            return hipMemcpyAsync(b + off, from, bytes, hipMemcpyHostToDevice, p->stream);
        };
        hipError_t e = copy(L.off_band, ddesc.data(), ddesc.size() * 4);
        if (matrix) {
            if (e == hipSuccess) e = copy(L.off_bfrag, bfrag.data(), bfrag.size() * 2);
            return e == hipSuccess ? asn::prepare_banded_lp(bf.azim, p->dtype, bf.reach) : e;
        }
        for (int r = 0; r < 3 && e == hipSuccess; ++r)
            if (!bcoef[r].empty()) e = copy(L.off_bcoef[r], bcoef[r].data(), bcoef[r].size() * 4);
        if (e == hipSuccess) e = copy(L.off_bcxy, dcxy.data(), dcxy.size() * 4);
        return e == hipSuccess ? asn::prepare_banded(bf.azim, p->dtype, bf.reach, p->scheme == ASN_SCHEME_HEUN) : e;
    };
    if (hipMemsetAsync(b, 0, L.total, p->stream) != hipSuccess ||
        hipMemcpyAsync(b + L.off_Kt, Kt.data(), Kt.size() * 4, hipMemcpyHostToDevice, p->stream) !=
            hipSuccess ||
        hipMemcpyAsync(b + L.off_qi, qi.data(), qi.size() * sizeof(QInfo), hipMemcpyHostToDevice,
                       p->stream) != hipSuccess ||
        hipMemcpyAsync(b + L.off_rdef, rdef.data(), rdef.size() * 4, hipMemcpyHostToDevice,
                       p->stream) != hipSuccess ||
        hipMemcpyAsync(b + L.off_ktab, ktab.data(), ktab.size() * 4, hipMemcpyHostToDevice,
                       p->stream) != hipSuccess ||
        (banded && copy_tables() != hipSuccess) ||
        (sparse &&
         (hipMemcpyAsync(b + L.off_sgroup, sgroup.data(), sgroup.size() * sizeof(sgroup[0]), hipMemcpyHostToDevice,
                         p->stream) != hipSuccess ||
          hipMemcpyAsync(b + L.off_sord, sord.data(), sord.size() * sizeof(sord[0]), hipMemcpyHostToDevice,
                         p->stream) != hipSuccess ||
          hipMemcpyAsync(b + L.off_srow, srow.data(), srow.size() * 4, hipMemcpyHostToDevice, p->stream) !=
              hipSuccess ||
          hipMemcpyAsync(b + L.off_scoef, sf.coef.data(), sf.coef.size() * 4, hipMemcpyHostToDevice, p->stream) !=
              hipSuccess ||
          asn::prepare_sparse(asn::sparse_waves(Q), p->dtype, p->scheme == ASN_SCHEME_HEUN) != hipSuccess)) ||
        (L.lowp && hipMemcpyAsync(b + L.off_Klp, Klp.data(), Klp.size() * 2,
                                  hipMemcpyHostToDevice, p->stream) != hipSuccess) ||
        hipMemcpyAsync(b + L.off_coef, coef.data(), coef.size() * 16, hipMemcpyHostToDevice,
                       p->stream) != hipSuccess)
        return bail(fail(ASN_E_HIP, "copying the problem tables to the device failed"));
    p->cur = 0;
    p->steps_done = 0;
    p->tab[0] = make_args(p, 0);
    p->tab[1] = make_args(p, 1);
    asn::blocks_per_kind(p->tab[0], p->blocks);
    int off1[asn::KT_COUNT * 2];
    for (int k = 0; k < asn::KT_COUNT; ++k) {
        off1[2 * k] = 0;
        off1[2 * k + 1] = p->blocks[k];
    }
    if (hipMemcpyAsync(b + L.off_tab, p->tab, sizeof(p->tab), hipMemcpyHostToDevice, p->stream) !=
            hipSuccess ||
        hipMemcpyAsync(b + L.off_off, off1, sizeof(off1), hipMemcpyHostToDevice, p->stream) !=
            hipSuccess)
        return bail(fail(ASN_E_HIP, "copying the step tables to the device failed"));
    if (arm_single(p, 1) != hipSuccess ||
        asn::launch_init(p->tab[0], single_batch(p), p->stream) != hipSuccess)
        return bail(fail(ASN_E_HIP, "initial moment kernels failed to launch"));
    if (implicit) {
        asn::ImplicitParams ip{};
        ip.nx = p->nx;
        ip.ny = p->ny;
        ip.Q = Q;
        ip.C = C;
        ip.P = L.P;
        ip.dx = p->dx;
        ip.dy = p->dy;
        ip.dt = p->dt;
        ip.W = p->W;
        ip.gmres_tol = opt.implicit_tol > 0.0 ? opt.implicit_tol : 1.5e-8;
        ip.source_tol = opt.source_tol > 0.0 ? opt.source_tol : 1e-4;
        ip.source_relative = opt.source_test == ASN_SOURCE_TEST_RELATIVE;
        ip.gmres_restart = kGmresRestart;
        p->imp.reset(new asn::ImplicitSolver());
        std::string ierr;
        if (!p->imp->init(ip, om.data(), w.data(), K.data(), sigma_s, sigma_a, sigma_as, source,
                          b + L.off_imp, p->stream, ierr))
            return bail(fail(ierr.find("nx must") != std::string::npos ? ASN_E_UNSUPPORTED : ASN_E_HIP,
                             ierr));
        if (!p->imp->set_state(reinterpret_cast<const float*>(b + L.off_psi0),
                               reinterpret_cast<double*>(b + L.off_phi64), ierr))
            return bail(fail(ASN_E_HIP, ierr));
    }
    if (hipStreamSynchronize(p->stream) != hipSuccess)
        return bail(fail(ASN_E_HIP, "synchronising after set-up failed"));
    *out = p;
    return ASN_OK;
}

// cell: as launch_init.
static asn_status finish_set_state(asn_problem p, const float* cell = nullptr) {
    p->steps_done = 0;
    HIP_TRY(arm_single(p, 1));
    HIP_TRY(asn::launch_init(p->tab[p->cur], single_batch(p), p->stream, cell));
    if (p->imp) {
        const Layout& L = p->L;
        std::string ierr;
        if (!p->imp->set_state(reinterpret_cast<const float*>(p->base + (p->cur == 0 ? L.off_psi0 : L.off_psi1)),
                               reinterpret_cast<double*>(p->base + L.off_phi64), ierr))
            return fail(ASN_E_HIP, ierr);
    }
    return ASN_OK;
}

asn_status asn_set_state(asn_problem p, const float* psi, int32_t on_device) {
    if (!p || !psi) return fail(ASN_E_INVALID, "NULL argument");
    const Layout& L = p->L;
    float* dst = reinterpret_cast<float*>(p->base + (p->cur == 0 ? L.off_psi0 : L.off_psi1));
    HIP_TRY(hipMemcpy2DAsync(dst, L.P * 4, psi, L.C * 4, L.C * 4, L.Q,
                             on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                             p->stream));
    if (!on_device) HIP_TRY(hipStreamSynchronize(p->stream));
    return finish_set_state(p);
}

asn_status asn_set_state_isotropic(asn_problem p, const float* cell, int32_t on_device) {
    if (!p || !cell) return fail(ASN_E_INVALID, "NULL argument");
    const Layout& L = p->L;
    float* dst = reinterpret_cast<float*>(p->base + (p->cur == 0 ? L.off_psi0 : L.off_psi1));
    // stage the cell values in the iso buffer (recomputed from the new state below)
    float* stage = reinterpret_cast<float*>(p->base + L.off_iso);
    HIP_TRY(hipMemcpyAsync(stage, cell, L.C * 4,
                           on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, p->stream));
    HIP_TRY(asn::launch_broadcast(dst, stage, L.Q, L.C, L.P, p->stream));
    if (!on_device) HIP_TRY(hipStreamSynchronize(p->stream));
    return finish_set_state(p, stage);
}

asn_status asn_get_state(asn_problem p, float* psi, int32_t on_device) {
    if (!p || !psi) return fail(ASN_E_INVALID, "NULL argument");
    const Layout& L = p->L;
    if (p->L.lowp && p->L.fused)   // fold the pending correction into the stored state
        HIP_TRY(asn::launch_materialize(p->tab[p->cur], p->stream));
    if (p->imp) {          // the implicit state is FP64: round it into the FP32 buffer first
        std::string ierr;
        if (!p->imp->get_state(reinterpret_cast<float*>(p->base + (p->cur == 0 ? L.off_psi0 : L.off_psi1)),
                               ierr))
            return fail(ASN_E_HIP, ierr);
    }
    const float* src = reinterpret_cast<const float*>(p->base + (p->cur == 0 ? L.off_psi0 : L.off_psi1));
    HIP_TRY(hipMemcpy2DAsync(psi, L.C * 4, src, L.P * 4, L.C * 4, L.Q,
                             on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, p->stream));
    HIP_TRY(hipStreamSynchronize(p->stream));
    return ASN_OK;
}

// The scheme the kernels are launched with: a separate-kernel step whose stencil
// runs over flat cell chunks (Euler or Heun) has a launch form of its own.
static int launch_scheme(asn_problem p) {
    if (p->L.sparse) return p->scheme == ASN_SCHEME_HEUN ? asn::SCHEME_HEUN_SPARSE : asn::SCHEME_EULER_SPARSE;
    if (p->L.matrix) return asn::SCHEME_EULER_BANDED_LP;
    if (p->L.banded) return p->scheme == ASN_SCHEME_HEUN ? asn::SCHEME_HEUN_BANDED : asn::SCHEME_EULER_BANDED;
    if (!p->L.flat) return p->scheme;
    return p->scheme == ASN_SCHEME_HEUN ? asn::SCHEME_HEUN_FLAT : asn::SCHEME_EULER_FLAT;
}

// An Euler step moves the state to the other buffer; a Heun step brings it back.
static int state_flip(int scheme, int64_t n_steps) {
    return scheme == ASN_SCHEME_HEUN ? 0 : (int)(n_steps & 1);
}

asn_status asn_step(asn_problem p, int64_t n_steps) {
    if (!p) return fail(ASN_E_INVALID, "problem is NULL");
    if (n_steps < 0 || n_steps > (1 << 30)) return fail(ASN_E_INVALID, "n_steps must be in [0, 2^30]");
    if (n_steps == 0) return ASN_OK;
    if (p->imp) {
        std::string ierr;
        if (!p->imp->step(n_steps, reinterpret_cast<double*>(p->base + p->L.off_phi64), ierr))
            return fail(ASN_E_HIP, ierr);
        p->steps_done += n_steps;
        return ASN_OK;
    }
    HIP_TRY(arm_single(p, n_steps));
    asn::BatchArgs b = single_batch(p);
    const size_t lds = p->L.by_cells() ? p->band_lds() : 0;
    for (int64_t i = 0; i < n_steps; ++i) {
        b.step = (int)i;
        b.s_par = (int)(i & 1);
        HIP_TRY(asn::launch_step(b, p->blocks, p->dtype, launch_scheme(p), p->stream, nullptr,
                                 p->block_az(), lds, p->band_reach));
    }
    HIP_TRY(asn::launch_last_budget(b, (int)n_steps, launch_scheme(p), p->stream));
    p->cur ^= state_flip(p->scheme, n_steps);
    p->steps_done += n_steps;
    return ASN_OK;
}

asn_status asn_step_timed(asn_problem p, int64_t n_steps, double kernel_ms[5]) {
    if (!p || !kernel_ms) return fail(ASN_E_INVALID, "NULL argument");
    if (n_steps < 1 || n_steps > (1 << 20)) return fail(ASN_E_INVALID, "n_steps must be in [1, 2^20]");
    if (p->imp) {          // iterative steps: only the span of a whole step is reported
        hipEvent_t e0 = nullptr, e1 = nullptr;
        HIP_TRY(hipEventCreate(&e0));
        HIP_TRY(hipEventCreate(&e1));
        HIP_TRY(hipEventRecord(e0, p->stream));
        const asn_status st = asn_step(p, n_steps);
        HIP_TRY(hipEventRecord(e1, p->stream));
        HIP_TRY(hipEventSynchronize(e1));
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        if (st != ASN_OK) return st;
        for (int k = 0; k < 4; ++k) kernel_ms[k] = 0.0;
        kernel_ms[4] = ms / (double)n_steps;
        return ASN_OK;
    }
    const int passes = asn::passes_per_step(p->scheme);
    const size_t per = 5 * (size_t)passes;
    std::vector<hipEvent_t> ev((size_t)n_steps * per, nullptr);
    asn_status st = ASN_OK;
    for (auto& e : ev)
        if (hipEventCreate(&e) != hipSuccess) {
            st = fail(ASN_E_HIP, "hipEventCreate failed");
            break;
        }
    if (st == ASN_OK && arm_single(p, n_steps) != hipSuccess)
        st = fail(ASN_E_HIP, "arming the step counter failed");
    asn::BatchArgs bt = single_batch(p);
    for (int64_t i = 0; st == ASN_OK && i < n_steps; ++i) {
        bt.step = (int)i;
        bt.s_par = (int)(i & 1);
        const hipError_t e = asn::launch_step(
            bt, p->blocks, p->dtype, launch_scheme(p), p->stream, &ev[(size_t)i * per], p->block_az(),
            p->L.by_cells() ? p->band_lds() : 0, p->band_reach);
        if (e != hipSuccess) {
            st = fail(ASN_E_HIP, std::string("step launch failed: ") + hipGetErrorString(e));
            break;
        }
    }
    if (st == ASN_OK && asn::launch_last_budget(bt, (int)n_steps, launch_scheme(p), p->stream) != hipSuccess)
        st = fail(ASN_E_HIP, "budget launch failed");
    if (st == ASN_OK) {
        p->cur ^= state_flip(p->scheme, n_steps);
        p->steps_done += n_steps;
    }
    double acc[5] = {0, 0, 0, 0, 0};
    if (st == ASN_OK && hipEventSynchronize(ev.back()) != hipSuccess)
        st = fail(ASN_E_HIP, "hipEventSynchronize failed");
    for (int64_t i = 0; st == ASN_OK && i < n_steps; ++i)
        for (int pass = 0; st == ASN_OK && pass < passes; ++pass) {
            hipEvent_t* e = &ev[(size_t)i * per + 5 * (size_t)pass];
            for (int k = 0; k < 5; ++k) {
                float ms = 0.f;
                if (hipEventElapsedTime(&ms, e[k == 4 ? 0 : k], e[k == 4 ? 4 : k + 1]) != hipSuccess) {
                    st = fail(ASN_E_HIP, "hipEventElapsedTime failed");
                    break;
                }
                acc[k] += ms;
            }
        }
    for (auto& e : ev)
        if (e) (void)hipEventDestroy(e);
    if (st != ASN_OK) return st;
    for (int k = 0; k < 5; ++k) kernel_ms[k] = acc[k] / (double)n_steps;
    return ASN_OK;
}

// Whether problems may step together (shared operand type, scheme, kernel form,
// stream; no repeats, no implicit problems).
static asn_status check_batch(asn_problem* probs, int32_t n) {
    if (!probs || n < 1 || n > asn::kMaxArm)
        return fail(ASN_E_INVALID, "a batch holds 1 to 64 problems");
    for (int32_t i = 0; i < n; ++i) {
        if (!probs[i]) return fail(ASN_E_INVALID, "NULL problem in batch");
        if (probs[i]->dtype != probs[0]->dtype)
            return fail(ASN_E_INVALID, "problems of a batch must share the operand type");
        if (probs[i]->scheme != probs[0]->scheme)
            return fail(ASN_E_INVALID, "problems of a batch must share the time scheme");
        if (probs[i]->imp)
            return fail(ASN_E_UNSUPPORTED, "implicit problems step alone (asn_step)");
        auto fused = [&](int32_t k) { return probs[k]->L.sparse ? probs[k]->fuses : probs[k]->L.fused; };
        if (fused(i) != fused(0))
            return fail(ASN_E_INVALID, "problems of a batch must share the kernel form "
                                       "(asn_step_form; ask for ASN_FORM_FUSED or ASN_FORM_SEPARATE "
                                       "when their sizes differ)");
        if (probs[0]->scheme == ASN_SCHEME_EULER && (probs[i]->L.banded != probs[0]->L.banded ||
                                                     probs[i]->band_azim != probs[0]->band_azim))
            return fail(ASN_E_INVALID, "problems of a banded batch must share the azimuth count "
                                       "(and a batch is banded for all its problems or none)");
        // (Heun: by the grid's width, also where the banded passes run)
        if (probs[0]->scheme == ASN_SCHEME_HEUN
                ? (probs[i]->nx <= asn::kFlatMaxNxM) != (probs[0]->nx <= asn::kFlatMaxNxM)
                : probs[i]->flat != probs[0]->flat)
            return fail(ASN_E_INVALID, std::string("problems of a batch must share the stencil form: ") +
                                       "separate-kernel steps use flat cell chunks up to nx = " +
                                       std::to_string(asn::kFlatMaxNx) + " (Euler) or " +
                                       std::to_string(asn::kFlatMaxNxM) + " (Heun), strips beyond");
        if (probs[i]->stream != probs[0]->stream)
            return fail(ASN_E_INVALID, "problems of a batch must share the HIP stream");
        for (int32_t j = 0; j < i; ++j)
            if (probs[j] == probs[i]) return fail(ASN_E_INVALID, "a problem appears twice");
    }
    return ASN_OK;
}

// The groups of a checked batch, and the device tables behind them as one block: step arguments
// of both buffers, block offsets per kernel kind and group, buffer bases, limits.
static size_t plan_bytes(int n) {
    return 2 * (size_t)n * sizeof(StepArgs) + (size_t)asn::KT_COUNT * (n + kMaxGroups) * sizeof(int) +
           2 * (size_t)asn::kMaxArm * sizeof(int);
}
static int group_kind(asn_problem p) {
    return p->L.matrix ? 4 : p->L.banded ? 0 : p->L.sparse ? (asn::sparse_waves(p->L.Q) == 8 ? 1 : 2) : 3;
}
static void make_plan(asn_problem* probs, int32_t n, char* dev, Plan& p, int* index, StepArgs* tab, int* off) {
    p.n = n;
    int at = 0;
    for (int kind = 0; kind < kMaxGroups; ++kind) {
        const int first = at;
        for (int32_t i = 0; i < n; ++i)
            if (group_kind(probs[i]) == kind) {
                if (index) index[at] = i;
                p.order[at++] = probs[i];
            }
        if (at == first) continue;
        Group& g = p.groups[p.n_groups++];
        g.first = first;
        g.n = at - first;
        g.scheme = launch_scheme(p.order[first]);
    }
    int* o = off;
    const size_t tab_b = 2 * (size_t)n * sizeof(StepArgs);
    for (int k = 0; k < p.n_groups; ++k) {
        Group& g = p.groups[k];
        g.args.tab = reinterpret_cast<const StepArgs*>(dev) + 2 * g.first;
        g.args.off = reinterpret_cast<const int*>(dev + tab_b) + (o - off);
        int* tail = reinterpret_cast<int*>(dev + tab_b) + asn::KT_COUNT * (n + kMaxGroups);
        g.args.base = tail + g.first;
        g.args.limit = tail + asn::kMaxArm + g.first;
        g.args.n = g.n;
        for (int i = 0; i < g.n; ++i) {
            asn_problem q = p.order[g.first + i];
            tab[2 * (g.first + i)] = q->tab[0];
            tab[2 * (g.first + i) + 1] = q->tab[1];
            for (int kind = 0; kind < asn::KT_COUNT; ++kind) {
                int* row = o + kind * (g.n + 1);
                if (i == 0) row[0] = 0;
                row[i + 1] = row[i] + q->blocks[kind];
            }
            if (q->L.by_cells()) g.band_lds = std::max(g.band_lds, q->band_lds());
            g.band_az = std::max(g.band_az, q->block_az());
            g.band_reach = std::max(g.band_reach, q->band_reach);
        }
        for (int kind = 0; kind < asn::KT_COUNT; ++kind) g.grid[kind] = o[kind * (g.n + 1) + g.n];
        o += asn::KT_COUNT * (g.n + 1);
    }
}
static hipError_t arm_plan(const Plan& p, const asn::ArmArgs& v, hipStream_t s) {
    return asn::launch_arm(const_cast<int*>(p.groups[0].args.limit), const_cast<int*>(p.groups[0].args.base), p.n, v,
                           s);
}
// n_steps steps of every group, and what follows the last.
static hipError_t launch_plan(const Plan& p, int64_t n_steps, int dtype, hipStream_t s) {
    hipError_t e = hipSuccess;
    for (int k = 0; k < p.n_groups && e == hipSuccess; ++k) {
        const Group& g = p.groups[k];
        asn::BatchArgs args = g.args;
        for (int64_t j = 0; j < n_steps && e == hipSuccess; ++j) {
            args.step = (int)j;
            args.s_par = (int)(j & 1);
            e = asn::launch_step(args, g.grid, dtype, g.scheme, s, nullptr, g.band_az, g.band_lds, g.band_reach);
        }
        if (e == hipSuccess) e = asn::launch_last_budget(args, (int)n_steps, g.scheme, s);
    }
    return e;
}

asn_status asn_batch_create(asn_problem* probs, int32_t n, asn_batch* out) {
    if (!out) return fail(ASN_E_INVALID, "out is NULL");
    *out = nullptr;
    const asn_status cs = check_batch(probs, n);
    if (cs != ASN_OK) return cs;
    auto* b = new asn_batch_s();
    b->dtype = probs[0]->dtype;
    b->scheme = probs[0]->scheme;
    b->stream = probs[0]->stream;
    std::vector<StepArgs> tab(2 * (size_t)n);
    std::vector<int> off((size_t)asn::KT_COUNT * (n + kMaxGroups), 0);
    void* m = nullptr;
    if (hipMalloc(&m, plan_bytes(n)) != hipSuccess) {
        delete b;
        return fail(ASN_E_OOM, "hipMalloc of the batch tables failed");
    }
    b->dev = static_cast<char*>(m);
    make_plan(probs, n, b->dev, b->plan, b->index, tab.data(), off.data());
    const size_t tab_b = tab.size() * sizeof(StepArgs);
    if (hipMemcpyAsync(b->dev, tab.data(), tab_b, hipMemcpyHostToDevice, b->stream) != hipSuccess ||
        hipMemcpyAsync(b->dev + tab_b, off.data(), off.size() * sizeof(int), hipMemcpyHostToDevice, b->stream) !=
            hipSuccess ||
        hipStreamSynchronize(b->stream) != hipSuccess) {
        (void)hipFree(b->dev);
        delete b;
        return fail(ASN_E_HIP, "copying the batch tables failed");
    }
    *out = b;
    return ASN_OK;
}

asn_status asn_batch_step(asn_batch b, int64_t n_steps, const int64_t* limit) {
    if (!b) return fail(ASN_E_INVALID, "batch is NULL");
    if (n_steps < 0 || n_steps > (1 << 20)) return fail(ASN_E_INVALID, "n_steps must be in [0, 2^20]");
    asn::ArmArgs v{};
    int64_t take[asn::kMaxArm];
    bool any = false;
    for (int i = 0; i < b->plan.n; ++i) {
        take[i] = limit ? std::max<int64_t>(0, std::min<int64_t>(limit[b->index[i]], n_steps)) : n_steps;
        v.limit[i] = (int)take[i];
        v.cur[i] = b->plan.order[i]->cur;
        any = any || take[i] > 0;
    }
    if (!any) return ASN_OK;
    HIP_TRY(arm_plan(b->plan, v, b->stream));
    if (b->stream != nullptr && n_steps >= 2) {
        // Capture the step sequence once per length; later calls replay it.
        auto it = b->graphs.find(n_steps);
        if (it == b->graphs.end()) {
            hipGraph_t g = nullptr;
            hipGraphExec_t ge = nullptr;
            HIP_TRY(hipStreamBeginCapture(b->stream, hipStreamCaptureModeRelaxed));
            const hipError_t e = launch_plan(b->plan, n_steps, b->dtype, b->stream);
            const hipError_t e2 = hipStreamEndCapture(b->stream, &g);
            if (e != hipSuccess || e2 != hipSuccess) {
                if (g) (void)hipGraphDestroy(g);
                return fail(ASN_E_HIP, std::string("capturing the step graph failed: ") +
                                           hipGetErrorString(e != hipSuccess ? e : e2));
            }
            if (hipGraphInstantiate(&ge, g, nullptr, nullptr, 0) != hipSuccess) {
                (void)hipGraphDestroy(g);
                return fail(ASN_E_HIP, "instantiating the step graph failed");
            }
            it = b->graphs.emplace(n_steps, std::make_pair(g, ge)).first;
        }
        HIP_TRY(hipGraphLaunch(it->second.second, b->stream));
    } else {
        HIP_TRY(launch_plan(b->plan, n_steps, b->dtype, b->stream));
    }
    for (int i = 0; i < b->plan.n; ++i) {
        b->plan.order[i]->cur ^= state_flip(b->scheme, take[i]);
        b->plan.order[i]->steps_done += take[i];
    }
    return ASN_OK;
}

asn_status asn_batch_destroy(asn_batch b) {
    if (!b) return ASN_OK;
    asn_status st = ASN_OK;
    if (hipStreamSynchronize(b->stream) != hipSuccess)
        st = fail(ASN_E_HIP, "synchronising before destroying the batch failed");
    for (auto& kv : b->graphs) {
        (void)hipGraphExecDestroy(kv.second.second);
        (void)hipGraphDestroy(kv.second.first);
    }
    if (b->dev) (void)hipFree(b->dev);
    delete b;
    return st;
}

// asn_step_batch_noalloc: the batch tables (step arguments of both buffers, block
// offsets per kernel kind, buffer bases, step counters) live in this file-scope device
// array instead of a hipMalloc'd block.  In host code the array's name is no device
// address: each device's copy is reached through the pointer hipGetSymbolAddress
// returns for it (kept per device at the first call there).
constexpr size_t kNoAllocBytes = 64 * 1024;
static __device__ __align__(256) unsigned char noalloc_scratch[kNoAllocBytes];

static std::mutex g_scratch_mu;
static std::map<int, char*> g_scratch_ptr;

static asn_status scratch_on_device(char** out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> g(g_scratch_mu);
    auto it = g_scratch_ptr.find(dev);
    if (it == g_scratch_ptr.end()) {
        void* ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(noalloc_scratch)));
        it = g_scratch_ptr.emplace(dev, static_cast<char*>(ptr)).first;
    }
    *out = it->second;
    return ASN_OK;
}

asn_status asn_step_batch_noalloc(asn_problem* probs, int32_t n, int64_t n_steps) {
    const asn_status cs = check_batch(probs, n);
    if (cs != ASN_OK) return cs;
    if (n_steps < 0 || n_steps > (1 << 20)) return fail(ASN_E_INVALID, "n_steps must be in [0, 2^20]");
    // the tables, laid out as in asn_batch_create, in host arrays of fixed size
    constexpr int kN = asn::kMaxArm;
    StepArgs tab[2 * kN];
    int off[asn::KT_COUNT * (kN + kMaxGroups)];
    if (plan_bytes(n) > kNoAllocBytes)
        return fail(ASN_E_INVALID, "batch tables exceed the no-allocation scratch (" +
                                       std::to_string(kNoAllocBytes) + " bytes)");
    if (n_steps == 0) return ASN_OK;
    char* dev = nullptr;
    const asn_status ss = scratch_on_device(&dev);
    if (ss != ASN_OK) return ss;
    Plan plan;
    make_plan(probs, n, dev, plan, nullptr, tab, off);
    hipStream_t stream = probs[0]->stream;
    // stream order: earlier work on this stream that read the tables has finished
    // before the copies land; the host arrays must outlive the copies, hence the wait
    const size_t tab_b = 2 * (size_t)n * sizeof(StepArgs);
    HIP_TRY(hipMemcpyAsync(dev, tab, tab_b, hipMemcpyHostToDevice, stream));
    HIP_TRY(hipMemcpyAsync(dev + tab_b, off, (size_t)asn::KT_COUNT * (n + kMaxGroups) * sizeof(int),
                           hipMemcpyHostToDevice, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    asn::ArmArgs v{};
    for (int i = 0; i < n; ++i) {
        v.limit[i] = (int)n_steps;
        v.cur[i] = plan.order[i]->cur;
    }
    HIP_TRY(arm_plan(plan, v, stream));
    HIP_TRY(launch_plan(plan, n_steps, probs[0]->dtype, stream));
    for (int i = 0; i < n; ++i) {
        probs[i]->cur ^= state_flip(probs[i]->scheme, n_steps);
        probs[i]->steps_done += n_steps;
    }
    // the next call overwrites the tables: let this one's kernels finish first
    HIP_TRY(hipStreamSynchronize(stream));
    return ASN_OK;
}

asn_status asn_step_batch(asn_problem* probs, int32_t n, int64_t n_steps) {
    asn_batch b = nullptr;
    asn_status s = asn_batch_create(probs, n, &b);
    if (s != ASN_OK) return s;
    s = asn_batch_step(b, n_steps, nullptr);
    const asn_status s2 = asn_batch_destroy(b);
    return s != ASN_OK ? s : s2;
}

asn_status asn_scalar_flux(asn_problem p, double* phi_host) {
    if (!p || !phi_host) return fail(ASN_E_INVALID, "NULL argument");
    HIP_TRY(hipMemcpyAsync(phi_host, p->base + p->L.off_phi64, p->L.C * 8, hipMemcpyDeviceToHost,
                           p->stream));
    HIP_TRY(hipStreamSynchronize(p->stream));
    return ASN_OK;
}

asn_status asn_mass_budget(asn_problem p, double out[ASN_BUDGET_LEN]) {
    if (!p || !out) return fail(ASN_E_INVALID, "NULL argument");
    if (p->imp) {
        HIP_TRY(hipStreamSynchronize(p->stream));
        for (int k = 0; k < ASN_BUDGET_LEN; ++k) out[k] = p->imp->budget[k];
        if (!std::isfinite(out[0])) return fail(ASN_E_UNSTABLE, "mass is not finite");
        return ASN_OK;
    }
    double rec[asn::REC_LEN];
    HIP_TRY(hipMemcpyAsync(rec, p->base + p->L.off_rec, sizeof(rec), hipMemcpyDeviceToHost, p->stream));
    HIP_TRY(hipStreamSynchronize(p->stream));
    out[0] = rec[asn::REC_MASS];
    out[1] = rec[asn::REC_MASS0];
    out[2] = rec[asn::REC_ABS];
    out[3] = rec[asn::REC_OUT];
    out[4] = rec[asn::REC_SRC];
    out[5] = rec[asn::REC_DEF];
    out[6] = rec[asn::REC_RES];
    out[7] = rec[asn::REC_STEPS];
    if (!std::isfinite(out[0])) return fail(ASN_E_UNSTABLE, "mass is not finite");
    return ASN_OK;
}

asn_status asn_info(asn_problem p, double* dt, int64_t* steps_done, int64_t* steps_to_tfinal,
                    int32_t* q) {
    if (!p) return fail(ASN_E_INVALID, "problem is NULL");
    if (dt) *dt = p->dt;
    if (steps_done) *steps_done = p->steps_done;
    if (steps_to_tfinal) *steps_to_tfinal = p->n_to_tfinal;
    if (q) *q = p->L.Q;
    return ASN_OK;
}

asn_status asn_step_form(asn_problem p, int32_t* form) {
    if (!p || !form) return fail(ASN_E_INVALID, "NULL argument");
    *form = p->L.banded && p->scheme == ASN_SCHEME_EULER       ? ASN_FORM_BANDED
            : (p->L.sparse ? p->fuses : p->L.fused) ? ASN_FORM_FUSED
                                                    : ASN_FORM_SEPARATE;
    return ASN_OK;
}

asn_status asn_step_kernel(asn_problem p, char* name, int32_t len) {
    if (!p || !name || len < 1) return fail(ASN_E_INVALID, "NULL argument");
    if (p->imp) name[0] = 0;
    else asn::contraction_kernel(p->dtype, launch_scheme(p), p->L.fused, p->block_az(), p->band_reach, name, (size_t)len);
    return ASN_OK;
}

asn_status asn_iteration_counts(asn_problem p, int64_t* sweeps, int64_t* matvecs) {
    if (!p) return fail(ASN_E_INVALID, "problem is NULL");
    if (sweeps) *sweeps = p->imp ? p->imp->sweeps : 0;
    if (matvecs) *matvecs = p->imp ? p->imp->matvecs : 0;
    return ASN_OK;
}

asn_status asn_stability(asn_problem p, double* z) {
    if (!p || !z) return fail(ASN_E_INVALID, "NULL argument");
    *z = p->stability;
    return ASN_OK;
}

asn_status asn_contraction_work(asn_problem p, double* dense_flops, double* tile_flops) {
    if (!p) return fail(ASN_E_INVALID, "problem is NULL");
    const double C = (double)p->L.C, Q = (double)p->L.Q;
    if (dense_flops) *dense_flops = 2.0 * Q * Q * C;
    if (tile_flops) *tile_flops = 2.0 * p->tile_entries * C;
    return ASN_OK;
}

asn_status asn_contraction_nonzero(asn_problem p, double* nonzero_flops) {
    if (!p || !nonzero_flops) return fail(ASN_E_INVALID, "NULL argument");
    *nonzero_flops = 2.0 * p->nonzero_entries * (double)p->L.C;
    return ASN_OK;
}

asn_status asn_destroy(asn_problem p) {
    if (!p) return ASN_OK;
    asn_status s = ASN_OK;
    if (hipStreamSynchronize(p->stream) != hipSuccess)
        s = fail(ASN_E_HIP, "synchronising before destroy failed");
    if (p->owns && p->base) (void)hipFree(p->base);
    delete p;
    return s;
}

const char* asn_status_string(asn_status s) {
    switch (s) {
        case ASN_OK: return "ok";
        case ASN_E_INVALID: return "invalid argument";
        case ASN_E_OOM: return "out of memory";
        case ASN_E_HIP: return "HIP runtime error";
        case ASN_E_UNSTABLE: return "unstable";
        case ASN_E_STATE: return "invalid state";
        case ASN_E_UNSUPPORTED: return "unsupported";
    }
    return "unknown status";
}

const char* asn_last_error(void) { return g_last_error.c_str(); }

asn_status asn_build_quadrature(int32_t n_polar, int32_t n_azim, double* omega_xyz,
                                double* weights) {
    if (n_polar < 1 || n_azim < 1 || !omega_xyz || !weights)
        return fail(ASN_E_INVALID, "invalid quadrature request");
    std::vector<double> om, w;
    asn::product_quadrature(n_polar, n_azim, om, w);
    std::memcpy(omega_xyz, om.data(), om.size() * 8);
    std::memcpy(weights, w.data(), w.size() * 8);
    return ASN_OK;
}

asn_status asn_build_icosahedron(int32_t order, double* omega_xyz, double* weights) {
    if (order < 2 || order > 41 || !omega_xyz || !weights)
        return fail(ASN_E_INVALID, "invalid icosahedron request");
    std::vector<double> om, w;
    asn::icosahedron_quadrature(order, om, w);
    std::memcpy(omega_xyz, om.data(), om.size() * 8);
    std::memcpy(weights, w.data(), w.size() * 8);
    return ASN_OK;
}

asn_status asn_build_kernel(int32_t q, const double* omega_xyz, const double* weights, double eps,
                            int32_t normalization, double* k_out) {
    if (q < 1 || !omega_xyz || !weights || !k_out || !(eps > 0.0))
        return fail(ASN_E_INVALID, "invalid kernel request");
    if (normalization != ASN_NORM_SYM && normalization != ASN_NORM_ROW)
        return fail(ASN_E_INVALID, "unknown normalization");
    std::vector<double> K;
    std::string err;
    if (!asn::kernel_matrix(q, omega_xyz, weights, eps, normalization == ASN_NORM_SYM ? 0 : 1, K, err))
        return fail(ASN_E_UNSUPPORTED, err);
    std::memcpy(k_out, K.data(), K.size() * 8);
    return ASN_OK;
}

asn_status asn_build_kernel_lowp(int32_t q, const double* k_in, int32_t gemm_dtype,
                                 uint16_t* k_bits, float* row_defect) {
    if (q < 1 || !k_in || !k_bits || !row_defect)
        return fail(ASN_E_INVALID, "invalid reduced-precision kernel request");
    if (gemm_dtype != ASN_GEMM_BF16 && gemm_dtype != ASN_GEMM_F16)
        return fail(ASN_E_INVALID, "gemm_dtype must be ASN_GEMM_BF16 or ASN_GEMM_F16");
    quantise_kernel(q, k_in, gemm_dtype, q, k_bits, row_defect);
    return ASN_OK;
}

asn_status asn_band_expand(int32_t n_polar, int32_t n_azim, const double* k_in, float* k_out,
                           int32_t* reach) {
    if (n_polar < 1 || n_azim < 1 || (int64_t)n_polar * n_azim > 16384 || !k_in || !k_out || !reach)
        return fail(ASN_E_INVALID, "invalid band request");
    const int Q = n_polar * n_azim;
    std::vector<float> K32((size_t)Q * Q);
    for (size_t i = 0; i < K32.size(); ++i) K32[i] = (float)k_in[i];
    asn::BandForm bf;
    if (!asn::band_form(n_polar, n_azim, K32.data(), asn::kBandMaxReach, asn::kBandNarrow, bf))
        return fail(ASN_E_UNSUPPORTED, "K has no banded form");
    // decode the per-level runs that the kernels' tables are made of
    std::fill(k_out, k_out + (size_t)Q * Q, 0.f);
    auto put_run = [&](int i, int k, int lo, int len, int first) {
        const int j = i + k - bf.reach;
        for (int t = 0; t < len; ++t) {
            const int delta = lo + t;
            for (int kk = 0; kk < n_azim; ++kk) {
                const int kp = ((kk + delta) % n_azim + n_azim) % n_azim;
                k_out[(size_t)(i * n_azim + kk) * Q + j * n_azim + kp] = bf.coef[first + t];
            }
        }
    };
    for (int i = 0; i < n_polar; ++i) {
        const int n = (int)bf.desc[(size_t)i * 8];
        for (int p = 0; p < n; ++p) {
            const uint32_t c = bf.desc[(size_t)i * 8 + 1 + p];
            int lo = 0, len = 0;
            asn::band_run(c, n_azim, lo, len);
            put_run(i, (int)((c >> 8) & 7u), lo, len, bf.range[2 * (size_t)i] + 4 * (int)(c >> 11));
        }
    }
    *reach = bf.reach;
    return ASN_OK;
}

asn_status asn_time_step(const asn_grid* grid, int32_t q, const double* omega_xyz, double cfl,
                         double t_final, double* dt, int64_t* n_steps) {
    asn_status s = check_grid(grid);
    if (s != ASN_OK) return s;
    if (q < 1 || !omega_xyz || !dt || !n_steps || !(t_final > 0.0) || !(cfl > 0.0))
        return fail(ASN_E_INVALID, "invalid time-step request");
    if (cfl > 1.0) return fail(ASN_E_UNSTABLE, "cfl above 1 is unstable for the explicit step");
    const double dx = (grid->x_max - grid->x_min) / grid->nx;
    const double dy = (grid->y_max - grid->y_min) / grid->ny;
    asn::cfl_time_step(q, omega_xyz, dx, dy, cfl, t_final, *dt, *n_steps);
    return ASN_OK;
}

}  // extern "C"
