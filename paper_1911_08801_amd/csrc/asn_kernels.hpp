// Device kernels of the as-S_N step and their launchers (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace asn {

// Per-ordinate constants of the streaming update, read with uniform (scalar) loads.
struct QInfo {
    float cx;     // dt |xi_q| / dx
    float cy;     // dt |eta_q| / dy
    float wf;     // w_q in FP32
    int32_t dir;  // bit0 xi > 0, bit1 xi < 0, bit2 eta > 0, bit3 eta < 0
    double w;     // w_q in FP64 (moment and budget accumulation)
};

// Device-side particle budget record (FP64), updated once per step.
enum {
    REC_MASS = 0,      // M at the current level
    REC_MASS0 = 1,     // M at set_state
    REC_ABS = 2,       // cumulative absorption increments
    REC_OUT = 3,       // cumulative outflow increments
    REC_SRC = 4,       // cumulative source increments
    REC_DEF = 5,       // cumulative collision defect increments
    REC_RES = 6,       // max relative residual
    REC_STEPS = 7,     // steps covered
    REC_ABS_NEXT = 8,  // absorption increment of the current level
    REC_SRC_STEP = 9,  // source increment per step (constant)
    REC_HALF = 10,     // Heun: half of the first stage's mass increment
    REC_ABS_STAGE = 11,  // Heun: absorption increment of the intermediate level
    REC_LEN = 16
};

// Time schemes: forward Euler + donor cell; Heun + minmod-limited fluxes.
enum { SCHEME_EULER = 0, SCHEME_HEUN = 1 };
// Launch form of a forward-Euler step with separate kernels whose stencil runs over
// flat cell chunks (see kFlatCells); the scheme is Euler.
constexpr int SCHEME_EULER_FLAT = 3;

// Separate forward-Euler stencil over flat chunks of kFlatCells consecutive cells (512
// threads, 4 cells each): each ordinate's plane segment, with the row below or above it,
// is staged in LDS in rounds of 2048 floats, at most kFlatRounds.  Used when
// nx <= kFlatMaxNx.
constexpr int kFlatThreads = 512;
constexpr int kFlatCells = 4 * kFlatThreads;
constexpr int kFlatRounds = 3;
constexpr int kFlatMaxNx = kFlatRounds * kFlatCells - kFlatCells - 8;
// Heun passes in the same form: the limited stencil reads two rows on one side and one
// on the other, so the segment is kFlatCells + 3 nx + 8 floats.
constexpr int SCHEME_HEUN_FLAT = 4;
// Flat-chunk stencil blocks the chip keeps resident at once: 256 CUs x 2 blocks of
// 8 waves (at most 4 waves per SIMD at their register use, 48 KB of LDS each).
constexpr int kFlatResident = 512;
constexpr int kFlatMaxNxM = (kFlatRounds * kFlatCells - kFlatCells - 8) / 3;

// Banded forward-Euler step (product ordinate sets): one kernel per step does the
// contraction, the stream + collide update, the moments and the budget partials.
// A block owns kBandCells consecutive cells (flat index) and every ordinate and walks
// the polar levels in order; a wave owns kBandO consecutive azimuths of every level, a
// lane one cell, so a block has n_az / kBandO waves.  LDS holds two levels: n_az rows of
// band_row floats (the cells, with the neighbour on either side at the ends), for BF16 /
// FP16 operands followed by as many rows of the rounded operands.
constexpr int SCHEME_EULER_BANDED = 5;
// Both passes of the FP32 Heun + minmod scheme in the same form.
constexpr int SCHEME_HEUN_BANDED = 6;
constexpr int kBandCells = 64;
constexpr int kBandO = 4;
// (Heun passes: two neighbours on either side)
__host__ __device__ constexpr int band_row(bool heun) { return kBandCells + (heun ? 4 : 2); }
constexpr int kBandMaxReach = 3;
// Largest half-width of the pair codes that band_form (asn_host.hpp) marks narrow.
constexpr int kBandNarrow = 8;
// Azimuth counts the step takes: FP32 8 .. 64 in steps of 8, BF16 / FP16 32, 48 or 64; BF16
// at 48 or 64 azimuths couples levels at most 2 apart.
constexpr int kBandMaxAzim = 64;
inline bool band_azimuths_supported(int az, int dtype) {
    return dtype == 0 ? az >= 8 && az <= kBandMaxAzim && az % 8 == 0 : az == 32 || az == 48 || az == 64;
}
// The Heun passes are FP32, reach 2 at most.
inline bool band_supported(int az, int dtype, int reach, bool heun) {
    return band_azimuths_supported(az, dtype) && (!heun || dtype == 0) &&
           reach <= (heun || (dtype == 1 && az > 32) ? 2 : kBandMaxReach);
}
// Dynamic LDS of a banded block (the final sums reuse it).
inline size_t band_lds_bytes(int az, int dtype, bool heun) {
    return (size_t)(dtype == 0 ? 2 : 4) * az * band_row(heun) * 4;
}

// The banded BF16 / FP16 step on the matrix cores (MFMA 16x16x32, FP32 accumulate): a block owns
// kBandCells consecutive cells and every ordinate; wave (m, n) produces azimuths 16 m .. 16 m + 15
// of cells 16 n .. 16 n + 15.  Per level pair (i, j) the circulant block of the stored K is
// multiplied as A operands of 16 x 32 (one per 16-azimuth offset, built on the host:
// band_lp_fragments) with the quantised partner level as B operand.
constexpr int SCHEME_EULER_BANDED_LP = 9;
// k-steps of 32 azimuths a level pair takes (48 azimuths: two, the second half-padded)
__host__ __device__ constexpr int band_lp_ksteps(int az) { return (az + 31) / 32; }
__host__ __device__ constexpr int band_lp_threads(int az) { return (az / 16) * (kBandCells / 16) * 64; }
// 16-bit elements of a slot of the quantised-level ring (one level, one operand term): the
// 8-azimuth chunks of every k-step (the padding past n_az held at zero), each chunk the
// block's cells in a row ([chunk][cell][8]: 16 lanes reading one chunk of 16 cells read
// 256 contiguous bytes)
__host__ __device__ constexpr int band_lp_slot(int az) { return 4 * band_lp_ksteps(az) * kBandCells * 8; }
// Dynamic LDS of its block (at most 152 KB, for any reach that band_supported takes): the ring of
// 2 reach + 2 quantised levels (two operand terms for BF16), two buffers of a level's A operands (at
// most 2 reach + 1 pairs, n_az / 16 fragments of 1 KiB each, and the previous level's (cx, cy)), the
// ring of tile-edge values (reach + 3 levels).
inline size_t band_lp_lds_bytes(int az, int reach, int dtype) {
    const int terms = dtype == 1 ? 2 : 1, mt = az / 16, nt = kBandCells / 16;
    return (size_t)(2 * reach + 2) * terms * band_lp_slot(az) * 2 +
           (size_t)2 * ((2 * reach + 1) * mt * 1024 + az * 8) + (size_t)(reach + 3) * 2 * nt * az * 4;
}
// uint4 of a level's block in its operand table: 2 kBandMaxReach + 1 pair slots, the (cx, cy) of
// the level before.
inline size_t band_lp_block(int az) { return (size_t)(2 * kBandMaxReach + 1) * (az / 16) * 64 + az / 2; }

// A step's form for any ordinate set with a sparse K, also one kernel a pass (Heun: FP32).  A block
// owns kBandCells cells and every ordinate, whose values (BF16 / FP16: rounded operands) are all in
// LDS, a row each, so their number is bounded by it.  Tables: sparse_form (asn_host.hpp).
constexpr int SCHEME_EULER_SPARSE = 7;
constexpr int SCHEME_HEUN_SPARSE = 8;
constexpr int kSparseChunk = 8;   // sources multiplied at a time
// LDS of a CU, and what a sparse block takes beside its rows (1072 bytes of sums).
constexpr size_t kLds = 160 * 1024, kSparseSums = 2048;
// Waves of a block: 8, and 16 where LDS has room for one block a CU (200^2 x 492: 142 -> 96 us; at
// 252 ordinates, two blocks a CU, 54.7 and 54.8; at 288 in BF16 70 and 74).
inline int sparse_waves(int Q) { return 2 * ((size_t)Q * kBandCells * 4 + kSparseSums) > kLds ? 16 : 8; }
inline size_t sparse_lds_bytes(int Q) {
    const size_t rows = (size_t)Q * kBandCells * 4;
    const size_t sums = (size_t)sparse_waves(Q) * (kBandCells * 16 + 4);   // finish_cells
    return rows > sums ? rows : sums;
}
struct SparseGroup {
    uint32_t ord[kBandO];     // ordinate << 4 | its direction bits (the last group: repeated)
    int first, chunks;        // its chunks of sources
    int pad[2];
};
struct SparseOrdinate {
    float cx, cy, rdef, pad;
    double w;
    double pad2;
};

// Modes of the budget kernel.
enum { BUD_STEP = 0, BUD_INIT = 1, BUD_STAGE1 = 2, BUD_STAGE2 = 3 };

// Cells per block of the reduced-precision operand scale: the default, and the range
// of powers of two a problem may choose (StepArgs::sb_log).  A block holds at least 64
// cells, so the 64 cells of one wave of the contraction's epilogue or of a flat-chunk
// stencil lie in one block.
constexpr int kScaleBlock = 256;
constexpr int kScaleBlockMin = 64;
constexpr int kScaleBlockMax = 4096;
// Blocks of 2^sb_log cells covering a plane of P cells.
__host__ __device__ inline int64_t scale_blocks(int64_t P, int sb_log) { return (P + (1 << sb_log) - 1) >> sb_log; }
// Scaled operands satisfy |x| < 2^(kScaleExp + 1).
constexpr int kScaleExp = 14;

// GEMM tiles (rows of K x cells x contraction step).
constexpr int kGemmBM = 128;
constexpr int kGemmBN = 128;

// Contraction depth per k-step: FP32 path and reduced-precision path.
constexpr int kBK_F32 = 16;
constexpr int kBK_LP = 32;

// Stencil tile: a strip of 62 updated columns (one wavefront of 64 lanes, the two
// outer lanes read the neighbouring columns) x 4 wavefronts x kRows rows each.
constexpr int kRows = 4;
constexpr int kStripX = 62;
// The limited (two-cell) stencil: 60 updated columns, two halo lanes per side.
constexpr int kStripXM = 60;
constexpr int kTileY = 4 * kRows;

struct StepArgs {
    // geometry
    int nx, ny, Q, Qp;
    int64_t C, P;  // cells, plane pitch (multiple of 256 cells)
    // stencil decomposition
    int G, qchunk, tiles_x, tiles_y;
    int fin_blocks;
    // operand type: 0 FP32, 1 BF16, 2 FP16
    int dtype;
    // log2 of the cells per block of the reduced-precision operand scale
    int sb_log;
    // 1: the stencil runs in the contraction's epilogue (forward Euler); the
    // stencil decomposition is then the contraction's: tiles_x = P / kGemmBN cell
    // tiles, tiles_y = 1, G = Qp / kGemmBM ordinate tiles
    int fused;
    double W, area;
    // buffers
    const float* psi;
    float* psi_new;
    float* Y;
    const float* Kt;        // FP32 K transposed, [Qp][Qp]
    const uint16_t* Klp;    // reduced-precision K, [Qp][Qp] row-major (K[m][k])
    const float* rdef;      // row defect of the reduced-precision K, [Qp]
    const int* ktab;        // per M-tile k-steps with a nonzero K tile: offsets[mtiles + 1],
                            // then the k-step indices (steps of kBK_F32 or kBK_LP ordinates)
    const QInfo* qi;
    const float4* coef;     // per cell {dt sigma_a, dt sigma_s, dt sigma_as, dt q}
    float* iso;             // Phi / W (FP32)
    double* phi64;          // Phi (FP64)
    double* phi_part;       // [G][P]
    double* blk_part;       // stencil block partials [G * tiles][2]
    double* fin_part;       // finalize block partials [fin_blocks][4] (banded: [tiles][4], and both
                            // kinds once per state buffer)
    double* ypart;          // [Qp / kGemmBM][P] weighted row sums of Y (reduced precision)
    float* fix;             // [P] per-cell particle correction of the reduced-precision Y
    float* delta;           // [P] fused reduced precision: pending isotropic correction of the
                            // stored state (true state = psi + delta); iso then holds Phi^ / W
                            // of the stored state and phi64 the true Phi
    float* delta_next;      // [P] banded: that of the new state (delta follows the psi buffer)
    unsigned* bmax_cur;     // block max |psi^n| (read by the GEMM), follows the psi buffer; per
                            // scale block, banded and sparse: per 64 cells
    unsigned* bmax_next;    // block max |psi^{n+1}| (written by the stencil)
    double* rec;
    // banded step (product ordinate sets): n_lev levels of n_az azimuths, coupling
    // levels up to `reach` apart; per level a descriptor (band, two uint4) and its coefficients for
    // the kernel's instances of reach 1, 2 and 3 (bcoef3, bcoef5, bcoef7) as built by
    // band_scatter_tables (asn_host.hpp), and per ordinate (cx, cy) (bcxy)
    const uint4* band;
    const float* bcoef3;
    const float* bcoef5;
    const float* bcoef7;
    const float2* bcxy;
    int n_lev, n_az, reach;
    // on the matrix cores (then `band` is not set): per level and one more, two uint4 {pairs, first
    // uint4 of its block in bfrag, the level offsets k of its pair slots (4 bits each), 0}; per level
    // pair and 16-azimuth offset the A operand of MFMA 16x16x32 as 64 lanes x 8 16-bit values
    // (band_lp_fragments)
    const uint4* bpairs;
    const uint4* bfrag;
    // sparse step (then also `band` is set and n_az such that the budget's fold has its threads):
    // groups of ordinates, per position in them what the step takes of an ordinate, LDS byte
    // offsets of the sources' rows and their coefficients, kBandO a source
    const SparseGroup* sp_group;
    const SparseOrdinate* sp_ord;
    const uint32_t* sp_row;
    const float* sp_coef;
};

// Kernel kinds of one step, each with its own block decomposition.
enum { KT_GEMM = 0, KT_FIX = 1, KT_SC = 2, KT_FIN = 3, KT_COUNT = 4 };

// Launch view of a batch of problems that share Q, K and the operand type.
// Every kernel covers all problems in one launch: block b of kernel kind k
// belongs to problem i with off[k * (n + 1) + i] <= b < off[k * (n + 1) + i + 1].
// tab[2 i + c] are the step arguments of problem i when psi buffer c holds its
// current state; at batch step s problem i uses c = base[i] ^ s_par.  A problem takes the
// steps below limit[i]; at later ones its blocks exit at once.  A single problem is a
// batch of one, so a problem computes bitwise the same alone and in a batch.
struct BatchArgs {
    const StepArgs* tab;
    const int* off;
    const int* base;
    const int* limit;
    int n;
    int step;    // steps of the call before this one
    int s_par;   // buffer parity: of the step (Euler), of the pass (Heun)
};

// Blocks of each kernel kind for one problem.
void blocks_per_kind(const StepArgs& a, int out[KT_COUNT]);

// Whether a problem runs the stencil inside the FP32 contraction.
inline bool can_fuse(int dtype, int scheme) { (void)dtype; return scheme == SCHEME_EULER; }

// One step for every problem of the batch.  Euler: one pass of contraction,
// stream + collide, finalize and budget, on the buffers selected by b.s_par.
// Heun: two such passes (s_par 0, then 1), so the state returns to its buffer.
// If ev is given, ev[5 k .. 5 k + 4] are recorded before, between and after
// the four kernels of pass k.
// band_az / band_lds: the banded step's azimuth count and dynamic LDS bytes (the largest of
// the batch); band_reach: the reach the banded
// kernel is instantiated for (at least every problem's).
hipError_t launch_step(const BatchArgs& b, const int* grid, int dtype, int scheme, hipStream_t s,
                       hipEvent_t* ev = nullptr, int band_az = 0, size_t band_lds = 0,
                       int band_reach = 0);
// Raise the dynamic LDS limit of the banded kernel that serves an azimuth count, operand type
// and reach, to the most that any problem of that instance takes (a limit set for one problem
// would hold for a larger one that is still alive).
hipError_t prepare_banded(int band_az, int dtype, int reach, bool heun);
// The same of the banded kernel on the matrix cores and of the sparse kernel of so many waves.
hipError_t prepare_banded_lp(int band_az, int dtype, int reach);
hipError_t prepare_sparse(int waves, int dtype, bool heun);
// Passes per step of a scheme.
inline int passes_per_step(int scheme) {
    return scheme == SCHEME_HEUN || scheme == SCHEME_HEUN_FLAT || scheme == SCHEME_HEUN_BANDED ||
                   scheme == SCHEME_HEUN_SPARSE
               ? 2
               : 1;
}
// The name of the kernel that launch_step contracts with (Heun: in the first pass).
void contraction_kernel(int dtype, int scheme, bool fused, int band_az, int band_reach, char* out, size_t n);
// After the last of a call's n_steps steps: what the next step's launch would do for it (the
// banded step's budget).
hipError_t launch_last_budget(const BatchArgs& b, int n_steps, int scheme, hipStream_t s);
// Arm a batch: limit[i] and base[i] = cur[i], i < n <= kMaxArm.
constexpr int kMaxArm = 64;
struct ArmArgs {
    int limit[kMaxArm];
    int cur[kMaxArm];
};
hipError_t launch_arm(int* limit, int* base, int n, const ArmArgs& v, hipStream_t s);
// Moments of the current state (after set_state): phi64, iso, bmax, budget record.
hipError_t launch_init(const StepArgs& a, const BatchArgs& one, hipStream_t s, const float* cell = nullptr);
// Fused reduced precision: fold the pending correction into the stored state.
hipError_t launch_materialize(const StepArgs& a, hipStream_t s);
// psi[q][c] = cell[c] for all q (pitch P), zero padding.
hipError_t launch_broadcast(float* psi, const float* cell, int Q, int64_t C, int64_t P,
                            hipStream_t s);

}  // namespace asn
