// Device kernels of the explicit as-S_N step (gfx950, wave64).
//
// One step (paper Section 3.2, eq. asSNeq; forward Euler + donor cell, or the
// paper's Heun + minmod scheme of Section 3.1 as two such passes):
//   1. contraction  Y = K Psi  over ordinates, every cell      (MFMA, gemm_*)
//   2. stream + collide psi^{n+1} from psi^n, Y, Phi^n          (HBM, stream_collide)
//      also emits partial moments Phi^{n+1} and budget partials
//   3. finalize: Phi^{n+1} = sum of partials, Phi/W, mass partials
//   4. budget: one block folds the partials into the FP64 record
// All reductions have a fixed order (no floating-point atomics), so a step is
// bitwise reproducible.
#include "asn_kernels.hpp"

#include <cstdio>
#include <type_traits>

#include "asn_host.hpp"

namespace asn {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Buffers are reached through pointers stored in the device argument table, which
// carry no address space; qualifying them as global keeps loads and stores on the
// global path (flat accesses would also tie up the LDS counter).
#if defined(__HIP_DEVICE_COMPILE__)
#define ASN_G __attribute__((address_space(1)))
#else
#define ASN_G
#endif
template <typename T>
__device__ __forceinline__ ASN_G T* gp(T* p) {
    return (ASN_G T*)p;
}

// Consecutive workgroups are dispatched round-robin over the 8 XCDs.  Map the
// hardware block id to a logical tile id so that logical neighbours share an
// XCD (and its L2): XCD x receives logical ids [start_x, start_x + count_x).
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    constexpr int X = 8;
    const int per = nb / X, rem = nb % X;
    const int xcd = bid % X, slot = bid / X;
    return xcd * per + (xcd < rem ? xcd : rem) + slot;
}

// Problem i and its local block for hardware block b of kernel kind `kind`;
// false if that problem takes no such step in this batch.
__device__ __forceinline__ bool locate(const BatchArgs& B, int kind, int b, int& i, int& local) {
    const ASN_G int* off = gp(B.off) + kind * (B.n + 1);
    int lo = 0, hi = B.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    i = lo;
    local = b - off[lo];
    return gp(B.limit)[lo] > B.step;
}

__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, off, 64));
    return v;
}

__device__ __forceinline__ StepArgs args_of(const BatchArgs& B, int i) {
    return gp(B.tab)[2 * i + (gp(B.base)[i] ^ B.s_par)];
}

// ---------------------------------------------------------------------------
// 1a. FP32 contraction Y[q][c] = sum_p K[q][p] psi[p][c] on MFMA 16x16x4 f32.
//     Block tile 128 (ordinates) x 128 (cells), k-step 16, 4 waves of 64x64.
//     Kt is K transposed and zero-padded to Qp x Qp; psi rows >= Q meet zero rows
//     of Kt.  Only k-steps whose K tile has a nonzero are visited, and in those
//     each wave multiplies only the 16-ordinate x 4 blocks of its 64 rows that
//     have one.  The products are taken with the operands swapped (Y^T = Psi^T
//     K^T), so each lane's accumulator holds four consecutive cells of one
//     ordinate: Y is stored as float4 rows.
//     FUSED: the forward-Euler stream + collide update is applied in the
//     epilogue instead of storing Y: the lane reads the old values and upwind
//     neighbours of its cells as aligned float4 rows, writes psi^{n+1} as a float4
//     (two cell groups, the halves of one 128-byte line, stored together), and
//     the block emits the Phi partial of its 128 ordinates for its 128 cells
//     plus its budget partials.  Y never reaches memory.
// ---------------------------------------------------------------------------
constexpr int kBK = kBK_F32;
constexpr int kLdsPad = 16;

template <int NV, typename OutPtr>
__device__ __forceinline__ void block_sum_256(double (&v)[NV], OutPtr out);

#ifndef ASN_F32_FUSED_WAVES
#define ASN_F32_FUSED_WAVES 2
#endif
// The fused epilogue needs more registers (two resident blocks per CU); the plain
// contraction fits four, whose loads then hide behind the others' products.
template <bool FUSED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FUSED ? ASN_F32_FUSED_WAVES : 4)))
void gemm_f32_kernel(BatchArgs B) {
    __shared__ float As[2][kBK][kGemmBM + kLdsPad];
    __shared__ float Bs[2][kBK][kGemmBN + kLdsPad];
    int pi, tile;
    if (!locate(B, KT_GEMM, xcd_remap(blockIdx.x, gridDim.x), pi, tile)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const ASN_G float* __restrict__ Kt = gp(a.Kt);
    const ASN_G float* __restrict__ psi = gp(a.psi);
    ASN_G float* __restrict__ Y = gp(a.Y);
    const ASN_G int* __restrict__ ktab = gp(a.ktab);
    const int Q = a.Q, Qp = a.Qp;
    const int64_t P = a.P;
    const int mtiles = Qp / kGemmBM;
    const int mt = tile % mtiles;
    const int nt = tile / mtiles;
    const int m0 = mt * kGemmBM;
    const int64_t n0 = (int64_t)nt * kGemmBN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave & 1) * 64, wn = (wave >> 1) * 64;

    // Staging of one k-step (kBK ordinates): thread t moves float4 number t + 256 r
    // (r < kBK / 8) of the A tile (Kt rows) and of the B tile (psi rows).  Steps past
    // row Q - 1 of psi read that row again: the matching rows of Kt are zero, so they
    // add exact zeros (a conditional overwrite of the loaded value would make the
    // wait for it count all loads in flight).
    constexpr int kNR = kBK / 8;
    const int kk0 = tid >> 5, c4 = (tid & 31) << 2;
#define ASN_GL1(S, r, k0)                                                                      \
    do {                                                                                       \
        const int ka = (k0) + kk0 + 8 * (r);                                                   \
        ra##S##r = *reinterpret_cast<const ASN_G float4*>(Kt + (size_t)ka * Qp + m0 + c4);     \
        rb##S##r = *reinterpret_cast<const ASN_G float4*>(psi + (size_t)min(ka, Q - 1) * P + n0 + c4); \
    } while (0)
#define ASN_LS1(S, r, b)                                                                       \
    do {                                                                                       \
        *reinterpret_cast<float4*>(&As[b][kk0 + 8 * (r)][c4]) = ra##S##r;                      \
        *reinterpret_cast<float4*>(&Bs[b][kk0 + 8 * (r)][c4]) = rb##S##r;                      \
    } while (0)
    static_assert(kNR == 2, "staging of 16-row k-steps");
    // register set X, and (plain contraction) set Y for a second step in flight
    float4 raX0, raX1, rbX0, rbX1, raY0, raY1, rbY0, rbY1;
    auto gloadX = [&](int k0) { ASN_GL1(X, 0, k0); ASN_GL1(X, 1, k0); };
    auto gloadY = [&](int k0) { ASN_GL1(Y, 0, k0); ASN_GL1(Y, 1, k0); };
    auto lstoreX = [&](int b) { ASN_LS1(X, 0, b); ASN_LS1(X, 1, b); };
    auto lstoreY = [&](int b) { ASN_LS1(Y, 0, b); ASN_LS1(Y, 1, b); };
#undef ASN_GL1
#undef ASN_LS1

    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Only k-steps whose K tile has a nonzero entry, and in those only the 16 x 4 operand
    // blocks of the wave with a nonzero entry (the skipped products are +0).
    const ASN_G int* __restrict__ klist = ktab + (mtiles + 1) + ktab[mt];
    const ASN_G int* __restrict__ mlist = klist + ktab[mtiles];
    const int nkt = ktab[mt + 1] - ktab[mt];
    // products of visited step kt from LDS buffer b (none for kt = nkt, the padding
    // step of an odd count)
    // mask of visited step kt (0 for the padding step kt = nkt)
    auto step_mask = [&](int kt) { return kt < nkt ? (unsigned)mlist[kt] : 0u; };
    auto mma = [&](unsigned m, int b) {
        // this wave's 64 ordinates: bit 4 i + g for sub-block i and k-group g (4 k each)
        // (wave-uniform: kept in a scalar register, tested with scalar branches)
        const unsigned wmask =
            (unsigned)__builtin_amdgcn_readfirstlane((int)((m >> (16 * (wave & 1))) & 0xFFFFu));
#pragma unroll
        for (int kk = 0; kk < kBK; kk += 4) {
            float av[4], bv[4];
            const int kr = kk + (lane >> 4), cl = lane & 15;
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = As[b][kr][wm + i * 16 + cl];
#pragma unroll
            for (int j = 0; j < 4; ++j) bv[j] = Bs[b][kr][wn + j * 16 + cl];
            // rows = cells (bv), columns = ordinates (av): acc[i][j] holds cells block i of
            // ordinate block j, four consecutive cells of one ordinate per lane
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (wmask & (1u << (4 * j + kk / 4)))
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[i], av[j], acc[i][j], 0, 0, 0);
        }
    };
    if constexpr (FUSED) {
        // one step in flight: loaded during the products of the previous one
        if (nkt > 0) {
            gloadX(klist[0] * kBK);
            lstoreX(0);
        }
        __syncthreads();
        for (int kt = 0; kt < nkt; ++kt) {
            const int b = kt & 1;
            if (kt + 1 < nkt) gloadX(klist[kt + 1] * kBK);
            mma(step_mask(kt), b);
            if (kt + 1 < nkt) lstoreX(b ^ 1);
            __syncthreads();
        }
    } else {
        // two steps in flight: set X holds even steps, set Y odd ones; a step's
        // registers are loaded two product phases before they go to LDS.  The loop is
        // entered, and goes round, with both sets in flight, the one stored next the
        // older, and has no conditional store or exit, so every wait counts only the
        // older set.  Loads past the last step repeat it; an odd count ends with a
        // padding step that multiplies nothing.
        // The step numbers and masks (scalar loads) are fetched one use ahead, so no
        // step waits on a scalar load issued in it.
        if (nkt > 0) {
            gloadX(klist[0] * kBK);
            gloadY(klist[min(1, nkt - 1)] * kBK);
        }
        int kx = klist[min(2, max(nkt - 1, 0))], ky = klist[min(3, max(nkt - 1, 0))];
        unsigned mx = step_mask(0), my = step_mask(1);
        for (int kt = 0; kt < nkt; kt += 2) {
            lstoreX(0);
            __syncthreads();
            gloadX(kx * kBK);
            kx = klist[min(kt + 4, nkt - 1)];
            mma(mx, 0);
            mx = step_mask(kt + 2);
            lstoreY(1);
            __syncthreads();
            gloadY(ky * kBK);
            ky = klist[min(kt + 5, nkt - 1)];
            mma(my, 1);
            my = step_mask(kt + 3);
        }
    }
    // D layout of the 16x16 MFMA: lane holds rows 4 (lane / 16) + v, column lane % 16, so
    // acc[i][j] is cells n0 + wn + 16 i + 4 (lane / 16) + v of ordinate m0 + wm + 16 j +
    // lane % 16.
    if constexpr (!FUSED) {
        // one float4 store per cell group; groups i and i + 1 (the halves of a 128-byte
        // line of the ordinate's row) back to back
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = m0 + wm + j * 16 + (lane & 15);
            if (q < Q) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t c0 = n0 + wn + i * 16 + 4 * (lane >> 4);
                    *reinterpret_cast<ASN_G float4*>(Y + (size_t)q * P + c0) =
                        make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
                }
            }
        }
    } else {
        const int nx = a.nx, ny = a.ny;
        const int64_t C = a.C;
        const ASN_G QInfo* __restrict__ qtab = gp(a.qi);
        const ASN_G float* __restrict__ isop = gp(a.iso);
        const ASN_G float4* __restrict__ coef = gp(a.coef);
        ASN_G float* __restrict__ out = gp(a.psi_new);
        const bool rows4 = (nx & 3) == 0;   // then a float4 of cells never crosses a grid row
        // The lane's four ordinates (columns j).  Padding ordinates (q >= Q) read row 0
        // and store nothing.
        QInfo qi[4];
        bool qok[4];
        const ASN_G float* rowp[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = m0 + wm + j * 16 + (lane & 15);
            qok[j] = q < Q;
            qi[j] = qtab[qok[j] ? q : 0];
            rowp[j] = psi + (size_t)(qok[j] ? q : 0) * P;
        }
        __shared__ double phred[2][kGemmBN];
        double defect = 0.0, outflow = 0.0;
        float4 held[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // four consecutive cells c0 .. c0 + 3 (c0 a multiple of 4, c0 + 3 < P)
            const int64_t c0 = n0 + wn + i * 16 + 4 * (lane >> 4);
            // All loads of this cell group first, at clamped in-range addresses, so that
            // they are in flight together; ghost and padding values are masked below.
            const float4 iso4 = *reinterpret_cast<const ASN_G float4*>(isop + c0);
            float4 cf[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) cf[k] = coef[c0 + k];
            float4 v4[4], u4[4];
            float xs[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const ASN_G float* row = rowp[j];
                v4[j] = *reinterpret_cast<const ASN_G float4*>(row + c0);
                // the x-upwind cell outside the float4: just before (xi > 0) or after it
                const int64_t xi = (qi[j].dir & 1) ? c0 - 1 : c0 + 4;
                xs[j] = row[min(max(xi, (int64_t)0), P - 1)];
                // the y-upwind row: below (eta > 0) or above; one aligned float4 when nx
                // is a multiple of 4, else four scalars
                const int64_t yi = c0 + ((qi[j].dir & 4) ? -(int64_t)nx : (int64_t)nx);
                if (rows4) {
                    u4[j] = *reinterpret_cast<const ASN_G float4*>(row + min(max(yi, (int64_t)0), P - 4));
                } else {
                    u4[j].x = row[min(max(yi, (int64_t)0), P - 1)];
                    u4[j].y = row[min(max(yi + 1, (int64_t)0), P - 1)];
                    u4[j].z = row[min(max(yi + 2, (int64_t)0), P - 1)];
                    u4[j].w = row[min(max(yi + 3, (int64_t)0), P - 1)];
                }
            }
            // Per cell: live (a grid cell, not padding) and its boundary faces as the bits
            // of the direction code (bit0 x = 0, bit1 x = nx - 1, bit2 y = 0, bit3
            // y = ny - 1): the upwind neighbour of ordinate class d is a ghost where
            // d & in_edge != 0 and the cell has an outflow face where d & out_edge != 0.
            int in_edge[4], out_edge[4];
            bool ck[4];
            {
                const int y0 = (int)(c0 / nx);
                int x = (int)(c0 - (int64_t)y0 * nx), y = y0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    ck[k] = c0 + k < C;
                    const int e = (x == 0 ? 1 : 0) | (x == nx - 1 ? 2 : 0) | (y == 0 ? 4 : 0) |
                                  (y == ny - 1 ? 8 : 0);
                    in_edge[k] = e;
                    out_edge[k] = ((e & 5) << 1) | ((e & 10) >> 1);
                    x = x + 1 == nx ? 0 : x + 1;
                    y = x == 0 ? y + 1 : y;
                }
            }
            const float isv[4] = {iso4.x, iso4.y, iso4.z, iso4.w};
            double ph[4] = {0.0, 0.0, 0.0, 0.0};
            // An interior group (four live cells off the domain boundary) needs no ghost,
            // padding or outflow handling.
            bool interior = true;
#pragma unroll
            for (int k = 0; k < 4; ++k) interior = interior && ck[k] && in_edge[k] == 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const QInfo& qj = qi[j];
                const int d = qj.dir;
                const float vv[4] = {v4[j].x, v4[j].y, v4[j].z, v4[j].w};
                const float uu[4] = {u4[j].x, u4[j].y, u4[j].z, u4[j].w};
                const float lft[4] = {xs[j], vv[0], vv[1], vv[2]};
                const float rgt[4] = {vv[1], vv[2], vv[3], xs[j]};
                float nv[4];
                float colsum = 0.f, o = 0.f;
                if (interior) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        // (cx = 0 when d & 3 = 0 and cy = 0 when d & 12 = 0)
                        const float ux = (d & 1) ? lft[k] : rgt[k];
                        const float v = vv[k];
                        const float col = cf[k].z * (acc[i][j][k] - v) + cf[k].y * (isv[k] - v);
                        nv[k] = v - qj.cx * (v - ux) - qj.cy * (v - uu[k]) - cf[k].x * v + col + cf[k].w;
                        colsum += col;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int gi = d & in_edge[k], go = d & out_edge[k];
                        const float ux = (gi & 3) ? 0.f : ((d & 1) ? lft[k] : rgt[k]);
                        const float uy = (gi & 12) ? 0.f : uu[k];
                        const float v = vv[k];
                        const float col = cf[k].z * (acc[i][j][k] - v) + cf[k].y * (isv[k] - v);
                        const float r = v - qj.cx * (v - ux) - qj.cy * (v - uy) - cf[k].x * v + col + cf[k].w;
                        nv[k] = ck[k] ? r : 0.f;   // padding cells stay zero
                        colsum += ck[k] ? col : 0.f;
                        o += ck[k] ? ((go & 3) ? qj.cx * v : 0.f) + ((go & 12) ? qj.cy * v : 0.f) : 0.f;
                    }
                }
                const double wj = qok[j] ? qj.w : 0.0;   // padding ordinates add nothing
#pragma unroll
                for (int k = 0; k < 4; ++k) ph[k] += wj * (double)nv[k];
                // Groups i and i + 1 are the two halves of a 128-byte line of the row: the
                // even group's result is held and both are stored together.
                const float4 res = make_float4(nv[0], nv[1], nv[2], nv[3]);
                if ((i & 1) == 0) {
                    held[j] = res;
                } else if (qok[j]) {
                    ASN_G float* o = out + (size_t)(m0 + wm + j * 16 + (lane & 15)) * P + c0;
                    *reinterpret_cast<ASN_G float4*>(o - 16) = held[j];
                    *reinterpret_cast<ASN_G float4*>(o) = res;
                }
                defect += wj * (double)colsum;
                outflow += wj * (double)o;
            }
            // Phi partial of this wave's 64 ordinates: the 16 lanes of a row group
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                ph[k] += __shfl_xor(ph[k], 1, 64);
                ph[k] += __shfl_xor(ph[k], 2, 64);
                ph[k] += __shfl_xor(ph[k], 4, 64);
                ph[k] += __shfl_xor(ph[k], 8, 64);
                if ((lane & 15) == 0) phred[wave & 1][wn + i * 16 + 4 * (lane >> 4) + k] = ph[k];
            }
        }
        // then the two waves that share the cells (fixed order)
        double sums[2] = {defect, outflow};
        block_sum_256<2>(sums, gp(a.blk_part) + 2 * (size_t)tile);   // synchronises the block
        if (tid < kGemmBN)
            gp(a.phi_part)[(size_t)mt * P + n0 + tid] = phred[0][tid] + phred[1][tid];
    }
}

// ---------------------------------------------------------------------------
// 1b. Reduced-precision contraction (BF16 or FP16 operands, FP32 accumulate) on
//     MFMA 16x16x32.  Only the anisotropic part of psi is rounded:
//       iso_c = Phi_c / W,  dev = psi - iso,  s = dev * 2^(E - e_b)
//       x = T(s) for FP16; for BF16 x = hi + lo, hi = T(s), lo = T(s - hi), two
//       MFMAs per k-step (a single BF16 term biases quasi-steady regions)
//       Y = iso + 2^(e_b - E) (T(K) x) + r_q dev,   r_q = 1 - sum_p T(K)_qp
//     with e_b the exponent of the block max |psi| over 256 cells (the N tile
//     lies inside one such block).  The epilogue also writes, per cell, the
//     w-weighted sum of this tile's Y rows (FP64) for the per-cell particle fix
//     applied in stream + collide.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kBKL = kBK_LP;
constexpr int kRowL = kBKL + 8;  // LDS row length in 16-bit elements (padded)

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Two FP32 values rounded to nearest even in the operand type, packed (lo in bits
// 0..15): one v_cvt_pk_bf16_f32 / v_cvt_pk_f16_f32 on gfx950.
template <int DT>
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const f32x2_t w = {lo, hi};
    if constexpr (DT == 1) return __builtin_bit_cast(uint32_t, __builtin_convertvector(w, bf16x2_t));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(w, f16x2_t));
}

// BF16 residual terms of a packed pair p = pack2<1>(lo, hi): s - T(s) is exact in FP32;
// the residuals are rounded to BF16 and packed as well.
__device__ __forceinline__ uint32_t bf16_residual2(uint32_t p, float lo, float hi) {
    return pack2<1>(lo - __uint_as_float(p << 16), hi - __uint_as_float(p & 0xFFFF0000u));
}

template <int DT>
__device__ __forceinline__ f32x4 mfma_lp(const uint4& av, const uint4& bv, const f32x4& c) {
    if constexpr (DT == 1)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                       __builtin_bit_cast(bf16x8, bv), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, av),
                                                      __builtin_bit_cast(f16x8, bv), c, 0, 0, 0);
}

template <int DT, bool FUSED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((FUSED || DT == 1) ? 2 : 3, 3)))
void gemm_lp_kernel(BatchArgs B) {
    __shared__ __attribute__((aligned(16))) uint16_t As[2][kGemmBM][kRowL];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][kGemmBN][kRowL];
    __shared__ __attribute__((aligned(16))) uint16_t Bl[DT == 1 ? 2 : 1][DT == 1 ? kGemmBN : 1][kRowL];
    __shared__ double red[2][kGemmBN];
    __shared__ double yred[FUSED ? 2 : 1][FUSED ? kGemmBN : 1];
    int pi, tile;
    if (!locate(B, KT_GEMM, xcd_remap(blockIdx.x, gridDim.x), pi, tile)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const ASN_G uint16_t* __restrict__ Klp = gp(a.Klp);
    const ASN_G float* __restrict__ psi = gp(a.psi);
    const ASN_G float* __restrict__ iso = gp(a.iso);
    const ASN_G float* __restrict__ rdef = gp(a.rdef);
    const ASN_G QInfo* __restrict__ qinfo = gp(a.qi);
    const ASN_G int* __restrict__ ktab = gp(a.ktab);
    ASN_G float* __restrict__ Yo = gp(a.Y);
    ASN_G double* __restrict__ ypart = gp(a.ypart);
    const int mtiles = a.Qp / kGemmBM;
    const int mt = tile % mtiles;
    const int nt = tile / mtiles;
    const int m0 = mt * kGemmBM;
    const int64_t n0 = (int64_t)nt * kGemmBN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave & 1) * 64, wn = (wave >> 1) * 64;
    const int Q = a.Q, Qp = a.Qp;
    const int64_t P = a.P;

    // Operand scale 2^(E - e_b) of scale block b (at least 64 cells): the four cells a
    // thread stages (n0 + 4 cg ..) lie in one block, and so do the 64 output cells of a
    // wave (n0 + wn ..); with blocks of 128 or more the tile has one scale.
    auto block_exp = [&](int64_t c) {
        const float bm = __uint_as_float(gp(a.bmax_cur)[c >> a.sb_log]);
        int e = 0;
        if (bm > 0.f) (void)frexpf(bm, &e);
        return max(e, -100);
    };
    const float s_in = ldexpf(1.f, kScaleExp - block_exp(n0 + 4 * (tid & 31)));
    const float s_out = ldexpf(1.f, block_exp(n0 + __builtin_amdgcn_readfirstlane(wn)) - kScaleExp);

    // Staging of one k-step (32 ordinates).  A: thread t moves 16-byte pieces t and
    // t + 256 of the T(K) tile.  B: thread t loads ordinates k0 + 4 kg .. + 3 of cells
    // n0 + 4 cg .. + 3 (four float4), subtracts iso, scales, rounds, and writes each
    // cell's four values as one 8-byte group of its LDS row.
    const int arow0 = tid >> 2, arow1 = arow0 + 64, akq = (tid & 3) * 8;
    const int cg = tid & 31, kg = tid >> 5;
    const float4 iso4 = *reinterpret_cast<const ASN_G float4*>(iso + n0 + 4 * cg);
    uint4 ra0, ra1;
    float4 rb[4];
#define ASN_GLOAD_LP(k0)                                                                       \
    do {                                                                                       \
        ra0 = *reinterpret_cast<const ASN_G uint4*>(Klp + (size_t)(m0 + arow0) * Qp + (k0) + akq); \
        ra1 = *reinterpret_cast<const ASN_G uint4*>(Klp + (size_t)(m0 + arow1) * Qp + (k0) + akq); \
        _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                        \
            const int kr = (k0) + 4 * kg + j;                                                  \
            rb[j] = *reinterpret_cast<const ASN_G float4*>(psi + (size_t)min(kr, Q - 1) * P +  \
                                                           n0 + 4 * cg);                       \
            if (kr >= Q) rb[j] = iso4; /* T(K) is zero there; keep the operand finite */       \
        }                                                                                      \
    } while (0)
    auto lstore = [&](int b) {
        *reinterpret_cast<uint4*>(&As[b][arow0][akq]) = ra0;
        *reinterpret_cast<uint4*>(&As[b][arow1][akq]) = ra1;
        // (v - iso) 2^(E - e_b): the scale is a power of two, so one FMA with the
        // scaled iso rounds exactly as the difference would
        const float ivs[4] = {iso4.x * s_in, iso4.y * s_in, iso4.z * s_in, iso4.w * s_in};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float v = c == 0 ? rb[j].x : c == 1 ? rb[j].y : c == 2 ? rb[j].z : rb[j].w;
                x[j] = __builtin_fmaf(v, s_in, -ivs[c]);
            }
            uint2 pk;
            pk.x = pack2<DT>(x[0], x[1]);
            pk.y = pack2<DT>(x[2], x[3]);
            *reinterpret_cast<uint2*>(&Bs[b][4 * cg + c][4 * kg]) = pk;
            if constexpr (DT == 1) {
                uint2 pl;
                pl.x = bf16_residual2(pk.x, x[0], x[1]);
                pl.y = bf16_residual2(pk.y, x[2], x[3]);
                *reinterpret_cast<uint2*>(&Bl[b][4 * cg + c][4 * kg]) = pl;
            }
        }
    };

    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Only k-steps whose T(K) tile has a nonzero entry (whole tiles are multiplied:
    // tests per operand block cost more issue slots than the products they skip).
    const ASN_G int* __restrict__ klist = ktab + (mtiles + 1) + ktab[mt];
    const int nkt = ktab[mt + 1] - ktab[mt];
    if (nkt > 0) {
        ASN_GLOAD_LP(klist[0] * kBKL);
        lstore(0);
    }
    __syncthreads();
    for (int kt = 0; kt < nkt; ++kt) {
        const int b = kt & 1;
        if (kt + 1 < nkt) ASN_GLOAD_LP(klist[kt + 1] * kBKL);
        const int r16 = lane & 15, kofs = 8 * (lane >> 4);
        uint4 av[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) av[i] = *reinterpret_cast<const uint4*>(&As[b][wm + i * 16 + r16][kofs]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint4 bv = *reinterpret_cast<const uint4*>(&Bs[b][wn + j * 16 + r16][kofs]);
            // FUSED: rows = cells (bv), columns = ordinates (av): acc[cell block][ordinate block]
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (FUSED) acc[j][i] = mfma_lp<DT>(bv, av[i], acc[j][i]);
                else acc[i][j] = mfma_lp<DT>(av[i], bv, acc[i][j]);
            }
            if constexpr (DT == 1) {
                const uint4 bl = *reinterpret_cast<const uint4*>(&Bl[b][wn + j * 16 + r16][kofs]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (FUSED) acc[j][i] = mfma_lp<DT>(bl, av[i], acc[j][i]);
                    else acc[i][j] = mfma_lp<DT>(av[i], bl, acc[i][j]);
                }
            }
        }
        if (kt + 1 < nkt) lstore(b ^ 1);
        __syncthreads();
    }
#undef ASN_GLOAD_LP

    if constexpr (!FUSED) {
    double part[4] = {0.0, 0.0, 0.0, 0.0};
    #pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t n = n0 + wn + j * 16 + (lane & 15);
            const float iso_n = iso[n];
    #pragma unroll
            for (int i = 0; i < 4; ++i)
    #pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = m0 + wm + i * 16 + 4 * (lane >> 4) + v;
                    if (m < Q) {
                        const float dev = psi[(size_t)m * P + n] - iso_n;
                        const float y = iso_n + s_out * acc[i][j][v] + rdef[m] * dev;
                        Yo[(size_t)m * P + n] = y;
                        part[j] += qinfo[m].w * (double)y;
                    }
                }
            part[j] += __shfl_xor(part[j], 16, 64);
            part[j] += __shfl_xor(part[j], 32, 64);
            if (lane < 16) red[wave & 1][wn + j * 16 + lane] = part[j];
        }
        __syncthreads();
        if (tid < kGemmBN) ypart[(size_t)mt * P + n0 + tid] = red[0][tid] + red[1][tid];
    } else {
        // Stream + collide with the stored state psi^ and the per-cell pending particle
        // correction delta: the true state is psi^ + delta (delta is isotropic, so it
        // drops out of the quantised deviation psi^ - iso^; iso^ = Phi^ / W).
        //   Y^  = (iso^ + delta) + 2^(e - E) T(K) x + r_q (psi^ - iso^)
        //   new = psi - cx (psi - up_x) - cy (psi - up_y) - dt sigma_a psi + col^ + dt q
        //   col^ = dt sigma_as (Y^ - psi) + dt sigma_s (iso - psi)
        // The block writes psi^{n+1} without its own correction and the per-cell
        // partials of Phi^, of sum_q w_q Y^ (for the next correction) and the budget.
        const int nx = a.nx, ny = a.ny;
        const int64_t C = a.C;
        ASN_G float* __restrict__ out = gp(a.psi_new);
        const ASN_G float* __restrict__ dl = gp(a.delta);
        const bool rows4 = (nx & 3) == 0;
        float rq[4], cxq[4], cyq[4];
        int dq[4];
        double wq[4];
        bool qok[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = m0 + wm + j * 16 + (lane & 15);
            qok[j] = q < Q;
            const QInfo qi = qinfo[qok[j] ? q : 0];
            rq[j] = rdef[qok[j] ? q : 0];
            cxq[j] = qi.cx;
            cyq[j] = qi.cy;
            dq[j] = qi.dir;
            wq[j] = qi.w;
        }
        double defect = 0.0, outflow = 0.0;
        float mx = 0.f;
        const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 held[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t c0 = n0 + wn + i * 16 + 4 * (lane >> 4);
            // Groups i and i + 1 are the two halves of a 128-byte line of the row: the
            // even group's result is held and both are stored together.
            auto emit = [&](int j, int q, const float4& res) {
                if ((i & 1) == 0) {
                    held[j] = res;
                } else {
                    ASN_G float* o = out + (size_t)q * P + c0;
                    *reinterpret_cast<ASN_G float4*>(o - 16) = held[j];
                    *reinterpret_cast<ASN_G float4*>(o) = res;
                }
            };
            float aa[4], bs[4], gs[4], ss[4];
            int xk[4], yk[4];
            bool ck[4];
            const float4 ih4 = *reinterpret_cast<const ASN_G float4*>(iso + c0);
            const float4 d4 = *reinterpret_cast<const ASN_G float4*>(dl + c0);
            const float ihv[4] = {ih4.x, ih4.y, ih4.z, ih4.w};
            const float dv[4] = {d4.x, d4.y, d4.z, d4.w};
            {
                const int y0 = (int)(c0 / nx);
                int x = (int)(c0 - (int64_t)y0 * nx), y = y0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    ck[k] = c0 + k < C;
                    xk[k] = x;
                    yk[k] = y;
                    if (++x == nx) {
                        x = 0;
                        ++y;
                    }
                    const float4 cf = ck[k] ? gp(a.coef)[c0 + k] : z4;
                    aa[k] = cf.x;
                    bs[k] = cf.y;
                    gs[k] = cf.z;
                    ss[k] = cf.w;
                }
            }
            // pending corrections of the neighbouring cells
            const float dprev = c0 >= 4 ? dl[c0 - 1] : 0.f;
            const float dnext = c0 + 4 < P ? dl[c0 + 4] : 0.f;
            double ph[4] = {0.0, 0.0, 0.0, 0.0}, yp[4] = {0.0, 0.0, 0.0, 0.0};
            // An interior group (four live cells of one grid row, off the domain
            // boundary) needs no ghost, padding or outflow handling.
            const bool interior = ck[3] && xk[0] >= 1 && xk[3] == xk[0] + 3 && xk[3] <= nx - 2 &&
                                  yk[0] >= 1 && yk[0] <= ny - 2;
            if (interior) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!qok[j]) continue;
                const int q = m0 + wm + j * 16 + (lane & 15);
                const ASN_G float* row = psi + (size_t)q * P;
                const float4 v4 = *reinterpret_cast<const ASN_G float4*>(row + c0);
                const float vh[4] = {v4.x, v4.y, v4.z, v4.w};
                // x-upwind value outside the group (before it for xi > 0, else after it)
                // and the y-upwind row; for xi = 0 (eta = 0) cx (cy) is 0 and any finite
                // value serves
                const bool xp = dq[j] & 1;
                const float xsv = row[xp ? c0 - 1 : c0 + 4] + (xp ? dprev : dnext);
                const int64_t sh = (dq[j] & 4) ? -(int64_t)nx : (int64_t)nx;
                float uy[4];
                if (rows4) {
                    const float4 u4 = *reinterpret_cast<const ASN_G float4*>(row + c0 + sh);
                    const float4 e4 = *reinterpret_cast<const ASN_G float4*>(dl + c0 + sh);
                    uy[0] = u4.x + e4.x;
                    uy[1] = u4.y + e4.y;
                    uy[2] = u4.z + e4.z;
                    uy[3] = u4.w + e4.w;
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) uy[k] = row[c0 + k + sh] + dl[c0 + k + sh];
                }
                float tv[4];   // true state psi^ + delta
#pragma unroll
                for (int k = 0; k < 4; ++k) tv[k] = vh[k] + dv[k];
                const float lft[4] = {xsv, tv[0], tv[1], tv[2]};
                const float rgt[4] = {tv[1], tv[2], tv[3], xsv};
                float nv[4];
                float colsum = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float v = tv[k];
                    const float ux = xp ? lft[k] : rgt[k];
                    const float dev = vh[k] - ihv[k];
                    const float ya = s_out * acc[i][j][k] + rq[j] * dev;   // Y^ - iso
                    const float col = gs[k] * ((ihv[k] + ya) - vh[k]) + bs[k] * (ihv[k] - vh[k]);
                    nv[k] = v - cxq[j] * (v - ux) - cyq[j] * (v - uy[k]) - aa[k] * v + col + ss[k];
                    ph[k] += wq[j] * (double)nv[k];
                    yp[k] += wq[j] * ((double)(ihv[k] + dv[k]) + (double)ya);
                    colsum += col;
                    mx = fmaxf(mx, fabsf(nv[k]));
                }
                emit(j, q, make_float4(nv[0], nv[1], nv[2], nv[3]));
                defect += wq[j] * (double)colsum;
            }
            } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!qok[j]) continue;
                const int q = m0 + wm + j * 16 + (lane & 15);
                const ASN_G float* row = psi + (size_t)q * P;
                const float4 v4 = *reinterpret_cast<const ASN_G float4*>(row + c0);
                const float vh[4] = {v4.x, v4.y, v4.z, v4.w};
                float ux[4] = {0.f, 0.f, 0.f, 0.f};
                if (dq[j] & 1) {
                    ux[0] = (c0 >= 4 ? row[c0 - 1] : 0.f) + dprev;
#pragma unroll
                    for (int k = 1; k < 4; ++k) ux[k] = vh[k - 1] + dv[k - 1];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (xk[k] == 0) ux[k] = 0.f;
                } else if (dq[j] & 2) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) ux[k] = vh[k + 1] + dv[k + 1];
                    ux[3] = (c0 + 4 < P ? row[c0 + 4] : 0.f) + dnext;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (xk[k] == nx - 1) ux[k] = 0.f;
                }
                float uy[4] = {0.f, 0.f, 0.f, 0.f};
                if (dq[j] & 12) {
                    const int64_t sh = (dq[j] & 4) ? -(int64_t)nx : (int64_t)nx;
                    if (rows4) {
                        const bool has = (dq[j] & 4) ? yk[0] > 0 : yk[0] < ny - 1;
                        if (has && ck[0]) {
                            const float4 u4 = *reinterpret_cast<const ASN_G float4*>(row + c0 + sh);
                            const float4 e4 = *reinterpret_cast<const ASN_G float4*>(dl + c0 + sh);
                            uy[0] = u4.x + e4.x;
                            uy[1] = u4.y + e4.y;
                            uy[2] = u4.z + e4.z;
                            uy[3] = u4.w + e4.w;
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const bool has = ck[k] && ((dq[j] & 4) ? yk[k] > 0 : yk[k] < ny - 1);
                            uy[k] = has ? row[c0 + k + sh] + dl[c0 + k + sh] : 0.f;
                        }
                    }
                }
                float nv[4];
                float colsum = 0.f, o = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float v = vh[k] + dv[k];
                    const float dev = vh[k] - ihv[k];
                    const float ya = s_out * acc[i][j][k] + rq[j] * dev;   // Y^ - iso
                    const float col = gs[k] * ((ihv[k] + ya) - vh[k]) + bs[k] * (ihv[k] - vh[k]);
                    const float r = v - cxq[j] * (v - ux[k]) - cyq[j] * (v - uy[k]) - aa[k] * v + col + ss[k];
                    nv[k] = ck[k] ? r : 0.f;
                    ph[k] += wq[j] * (double)nv[k];
                    yp[k] += ck[k] ? wq[j] * ((double)(ihv[k] + dv[k]) + (double)ya) : 0.0;
                    colsum += ck[k] ? col : 0.f;
                    mx = fmaxf(mx, fabsf(nv[k]));
                    if (ck[k]) {
                        if (((dq[j] & 1) && xk[k] == nx - 1) || ((dq[j] & 2) && xk[k] == 0)) o += cxq[j] * v;
                        if (((dq[j] & 4) && yk[k] == ny - 1) || ((dq[j] & 8) && yk[k] == 0)) o += cyq[j] * v;
                    }
                }
                emit(j, q, make_float4(nv[0], nv[1], nv[2], nv[3]));
                defect += wq[j] * (double)colsum;
                outflow += wq[j] * (double)o;
            }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
#pragma unroll
                for (int sft = 1; sft < 16; sft <<= 1) {
                    ph[k] += __shfl_xor(ph[k], sft, 64);
                    yp[k] += __shfl_xor(yp[k], sft, 64);
                }
                if ((lane & 15) == 0) {
                    red[wave & 1][wn + i * 16 + 4 * (lane >> 4) + k] = ph[k];
                    yred[wave & 1][wn + i * 16 + 4 * (lane >> 4) + k] = yp[k];
                }
            }
        }
        // block max |psi^{n+1}| of the next operand scale: the wave's 64 cells lie in
        // one block
        const unsigned mbits = wave_max_u32(__float_as_uint(mx));
        if (lane == 0 && mbits) atomicMax(&a.bmax_next[(n0 + wn) >> a.sb_log], mbits);
        double sums[2] = {defect, outflow};
        block_sum_256<2>(sums, gp(a.blk_part) + 2 * (size_t)tile);   // synchronises the block
        if (tid < kGemmBN) {
            gp(a.phi_part)[(size_t)mt * P + n0 + tid] = red[0][tid] + red[1][tid];
            ypart[(size_t)mt * P + n0 + tid] = yred[0][tid] + yred[1][tid];
        }
    }
}

// ---------------------------------------------------------------------------
// Block-level FP64 sum in a fixed order (wave butterflies, then wave 0).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int NV, typename OutPtr>
__device__ __forceinline__ void block_sum_256(double (&v)[NV], OutPtr out) {
    __shared__ double red[4][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) red[wave][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) out[k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
}
// The same for a block of NW waves (block size 64 NW).
template <int NW, int NV, typename OutPtr>
__device__ __forceinline__ void block_sum_waves(double (&v)[NV], OutPtr out) {
    __shared__ double red[NW][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) red[wave][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double t = red[0][k];
#pragma unroll
            for (int w = 1; w < NW; ++w) t += red[w][k];
            out[k] = t;
        }
}

// The same for a block of nw <= MAXW waves.
template <int MAXW, int NV, typename OutPtr>
__device__ __forceinline__ void block_sum_n(double (&v)[NV], int nw, OutPtr out) {
    __shared__ double red[MAXW][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) red[wave][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double t = red[0][k];
            for (int w = 1; w < nw; ++w) t += red[w][k];
            out[k] = t;
        }
}

// ---------------------------------------------------------------------------
// 2. Stream + collide.  Block = 4 waves; wave w owns rows y0 + w R .. + R - 1
//    of a strip of 62 columns: lane l holds column x0 + l - 1, lanes 0 and 63
//    only read the neighbouring columns (halo), lanes 1..62 update.  The block
//    loops over a chunk of ordinates and loads plane q + 1 while it updates
//    plane q.  Upwind neighbour along y: the lane's previous (or next) row, plus
//    one halo row per wave; along x: the neighbouring lane (shuffle).
//    Memory goes through buffer descriptors of one ordinate plane each: offsets
//    outside the grid read as 0 (the vacuum ghost value) and stores to them are
//    dropped, so the loop has no per-cell branches.  Runs for grids wider than the
//    flat-chunk form takes (stream_collide_flat_kernel, below).
//      col  = dt sigma_as (Y - fix - psi) + dt sigma_s (Phi/W - psi)
//      new  = psi - cx (psi - up_x) - cy (psi - up_y) - dt sigma_a psi + col + dt q
//    LP: fix is the per-cell particle correction of the reduced-precision Y, and
//    the block max |new| for the next step's operand scale is reduced per wave.
// ---------------------------------------------------------------------------
constexpr uint32_t kOOB = 0x80000000u;   // byte offset beyond every plane
constexpr int kRsrcWord3 = 0x00020000;   // raw buffer, 32-bit data (gfx9 family)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const float* base, int64_t C) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)(C * 4),
                                             kRsrcWord3);
}

// The raw buffer builtins move 32-bit patterns; reinterpret, never convert.
__device__ __forceinline__ float load_plane(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ void store_plane(float v, __amdgpu_buffer_rsrc_t r, uint32_t off) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, 0, 0);
}
// Non-temporal forms (cache policy NT) for data the kernel touches once and that no
// later kernel of the step reads from the caches (the flat stencil's Y and new state:
// 400^2 x 512 0.193 -> 0.186 ms, 700^2 x 1152 1.26 -> 1.22 ms; its staged state rows
// stay cached, a neighbouring block reads them again).
constexpr int kCachePolicyNT = 2;
__device__ __forceinline__ float load_plane_nt(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kCachePolicyNT));
}
__device__ __forceinline__ void store_plane_nt(float v, __amdgpu_buffer_rsrc_t r, uint32_t off) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, 0, kCachePolicyNT);
}


// Block barrier that orders LDS only (the stencil waves exchange their rows through LDS;
// a full barrier would also wait for the next plane's global loads in flight).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <bool LP>
__global__ __launch_bounds__(256) void stream_collide_kernel(BatchArgs B) {
    constexpr int R = kRows;
    int pi, local;
    if (!locate(B, KT_SC, blockIdx.x, pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int bx = local % a.tiles_x;
    const int by = (local / a.tiles_x) % a.tiles_y;
    const int g = local / (a.tiles_x * a.tiles_y);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nx = a.nx, ny = a.ny;
    const int64_t P = a.P, C = a.C;
    const int x = bx * kStripX + lane - 1;
    const int ybase = by * kTileY + wave * R;
    const int q0 = g * a.qchunk;
    const int q1 = min(a.Q, q0 + a.qchunk);
    const bool xok = x >= 0 && x < nx;
    const bool outl = xok && lane >= 1 && lane <= 62;

    float aa[R], bs[R], gs[R], ss[R], isov[R], fix[R], mx[R];
    double phacc[R];
    bool in[R];
    uint32_t off_ld[R], off_st[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = ybase + r;
        const bool yok = y < ny;
        const uint32_t c = (uint32_t)(y * nx + x);
        in[r] = outl && yok;
        off_ld[r] = (xok && yok) ? 4u * c : kOOB;
        off_st[r] = in[r] ? 4u * c : kOOB;
        aa[r] = bs[r] = gs[r] = ss[r] = isov[r] = fix[r] = 0.f;
        mx[r] = 0.f;
        phacc[r] = 0.0;
        if (in[r]) {
            const float4 cf = gp(a.coef)[c];
            aa[r] = cf.x;
            bs[r] = cf.y;
            gs[r] = cf.z;
            ss[r] = cf.w;
            isov[r] = gp(a.iso)[c];
            if (LP) fix[r] = gp(a.fix)[c];
        }
    }
    const uint32_t off_hlo =
        (xok && ybase >= 1 && ybase - 1 < ny) ? 4u * (uint32_t)((ybase - 1) * nx + x) : kOOB;
    const uint32_t off_hhi = (xok && ybase + R < ny) ? 4u * (uint32_t)((ybase + R) * nx + x) : kOOB;
    const bool edge = bx == 0 || bx == a.tiles_x - 1 || by == 0 || by == a.tiles_y - 1;
    double defect = 0.0, outflow = 0.0;

    struct Plane {
        float v[R], y[R], hy;
    };
    auto load = [&](int q, int dir, Plane& pn) {
        const __amdgpu_buffer_rsrc_t rp = plane_rsrc(a.psi + (size_t)q * P, C);
        const __amdgpu_buffer_rsrc_t ry = plane_rsrc(a.Y + (size_t)q * P, C);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pn.v[r] = load_plane(rp, off_ld[r]);
            pn.y[r] = load_plane(ry, off_ld[r]);
        }
        // only the block's outer halo rows come from memory (wave 0 the row below the
        // tile for eta > 0, wave 3 the row above it for eta < 0); the others are the
        // neighbouring waves' own rows, exchanged through LDS
        const uint32_t oh = ((dir & 4) && wave == 0) ? off_hlo : (((dir & 8) && wave == 3) ? off_hhi : kOOB);
        pn.hy = load_plane(rp, oh);
    };
    // xr[q & 1][row of the tile][lane]: the tile's 16 rows of plane q; hr[q & 1][wave]: the
    // halo row each wave loaded (only waves 0 and 3 load one; every wave stores its
    // slot so that no store depends on the wave index)
    __shared__ float xr[2][kTileY][64];
    __shared__ float hr[2][4][64];

    // Ordinate q updates from plane slot q & 1 while the next plane loads into the
    // other slot.  The slots are fixed per unrolled half and every load is issued
    // unconditionally (the last ordinate of the chunk is loaded again at the end), so
    // no slot is ever copied or merged across a branch, which would wait for the
    // loads in flight.
    const ASN_G QInfo* __restrict__ qtab = gp(a.qi);
    auto body = [&](int q, const QInfo& qc, const Plane& cur) {
        const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.psi_new + (size_t)q * P, C);
        float (*xq)[64] = xr[q & 1];
#pragma unroll
        for (int r = 0; r < R; ++r) xq[wave * R + r][lane] = cur.v[r];
        hr[q & 1][wave][lane] = cur.hy;
        lds_barrier();
        // the row below the wave's rows (eta > 0) or above them (eta < 0)
        const float* hsrc = (qc.dir & 4) ? (wave == 0 ? &hr[q & 1][0][0] : &xq[wave * R - 1][0])
                                         : (wave == 3 ? &hr[q & 1][3][0] : &xq[(wave + 1) * R][0]);
        const float hy = hsrc[lane];
        float colsum = 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float v = cur.v[r];
            float uy = 0.f;
            if (qc.dir & 4) uy = (r == 0) ? hy : cur.v[r - 1];
            else if (qc.dir & 8) uy = (r == R - 1) ? hy : cur.v[r + 1];
            float ux = 0.f;
            if (qc.dir & 1) ux = __shfl_up(v, 1, 64);
            else if (qc.dir & 2) ux = __shfl_down(v, 1, 64);
            const float col = gs[r] * ((cur.y[r] - fix[r]) - v) + bs[r] * (isov[r] - v);
            const float nv = v - qc.cx * (v - ux) - qc.cy * (v - uy) - aa[r] * v + col + ss[r];
            store_plane(nv, ro, off_st[r]);
            phacc[r] += qc.w * (double)nv;
            colsum += in[r] ? col : 0.f;
            if (LP) mx[r] = fmaxf(mx[r], in[r] ? fabsf(nv) : 0.f);
        }
        defect += qc.w * (double)colsum;
        if (edge) {
            // Mass leaving through the boundary this step: the donor flux of the
            // last cell before a boundary face, for the directions that exit there.
            float o = 0.f;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!in[r]) continue;
                const int y = ybase + r;
                if (((qc.dir & 1) && x == nx - 1) || ((qc.dir & 2) && x == 0)) o += qc.cx * cur.v[r];
                if (((qc.dir & 4) && y == ny - 1) || ((qc.dir & 8) && y == 0)) o += qc.cy * cur.v[r];
            }
            outflow += qc.w * (double)o;
        }
    };
    Plane pa, pb;
    QInfo qa = qtab[min(q0, a.Q - 1)], qb;
    load(min(q0, a.Q - 1), qa.dir, pa);
    for (int q = q0; q < q1; q += 2) {
        const int qn = min(q + 1, q1 - 1);
        qb = qtab[qn];
        load(qn, qb.dir, pb);
        body(q, qa, pa);
        if (q + 1 >= q1) break;
        const int qn2 = min(q + 2, q1 - 1);
        qa = qtab[qn2];
        load(qn2, qa.dir, pa);
        body(q + 1, qb, pb);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (in[r]) gp(a.phi_part)[(size_t)g * P + (uint32_t)((ybase + r) * nx + x)] = phacc[r];
    if (LP) {
        // The updating lanes of one row (at most 62 cells) cover at most two scale blocks.
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int y = ybase + r;
            const int64_t c_first = (int64_t)y * nx + bx * kStripX;
            const int64_t b0 = c_first >> a.sb_log;
            const int64_t cb = ((int64_t)y * nx + x) >> a.sb_log;
            const unsigned bits = in[r] ? __float_as_uint(mx[r]) : 0u;
            const unsigned m0 = wave_max_u32(cb == b0 ? bits : 0u);
            const unsigned m1 = wave_max_u32(cb != b0 ? bits : 0u);
            if (lane == 0 && y < ny) {
                if (m0) atomicMax(&a.bmax_next[b0], m0);
                if (m1) atomicMax(&a.bmax_next[b0 + 1], m1);
            }
        }
    }
    double sums[2] = {defect, outflow};
    block_sum_256<2>(sums, gp(a.blk_part) + 2 * (size_t)local);
}

// ---------------------------------------------------------------------------
// 2'. Stream + collide over flat cell chunks (separate forward-Euler stencil).
//     Block (chunk bt, ordinate chunk g) updates cells b0 .. b0 + kFlatCells - 1 for
//     the ordinates of chunk g.  Per ordinate the plane segment [b0 - 1, b0 + L + 1)
//     plus the row below it (eta > 0) or above it (eta < 0) is staged in LDS (float4
//     loads from a 16-byte aligned start, so every row segment is read as whole
//     128-byte lines; cells outside the planes read as 0 through the buffer bounds),
//     the x- and y-upwind values are read from there with ghost masks at the domain
//     boundary, and the next ordinate's segment is fetched meanwhile into the other
//     register slot.  Thread t updates cells b0 + t + 512 j, j = 0..3: a wave's 64
//     lanes read 64 consecutive LDS words (no bank conflicts) and store 256 contiguous
//     bytes.  Same arithmetic and partials as stream_collide_kernel.
// ---------------------------------------------------------------------------
template <bool LP>
__global__ __launch_bounds__(kFlatThreads) void stream_collide_flat_kernel(BatchArgs B) {
    constexpr int T = kFlatThreads, L = kFlatCells, NR = kFlatRounds, J = L / T;
    int pi, local;
    // consecutive chunks on one XCD: the rows a chunk stages beyond its own cells are
    // its neighbours' cells, read at about the same time through the same L2
    if (!locate(B, KT_SC, xcd_remap(blockIdx.x, gridDim.x), pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int tiles = a.tiles_x;
    const int bt = local % tiles, g = local / tiles;
    const int tid = threadIdx.x, lane = tid & 63;
    const int nx = a.nx, ny = a.ny;
    const int C = (int)a.C, Pi = (int)a.P;
    const int b0 = bt * L;
    const int q0 = g * a.qchunk;
    const int q1 = min(a.Q, q0 + a.qchunk);

    // the thread's cells b0 + tid + T j
    float aa[J], bs[J], gs[J], ss[J], isov[J], fix[J], mx[J];
    uint32_t off[J];   // byte offset of the cell in a plane, out of range beyond the pitch
    double phacc[J];
    int e_in = 0;      // 4 bits per cell: boundary faces as the bits of the direction code
    int live = 0;      // bit j: cell j is a grid cell (not padding)
    int wedge = 0;     // bit j: some lane of the wave holds a boundary cell j (uniform)
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int c = b0 + tid + T * j;
        const bool in = c < C;
        const int y = c / nx, x = c - y * nx;
        float4 cf = make_float4(0.f, 0.f, 0.f, 0.f);
        if (in) cf = gp(a.coef)[c];
        aa[j] = cf.x;
        bs[j] = cf.y;
        gs[j] = cf.z;
        ss[j] = cf.w;
        isov[j] = in ? gp(a.iso)[c] : 0.f;
        fix[j] = (LP && in) ? gp(a.fix)[c] : 0.f;
        mx[j] = 0.f;
        phacc[j] = 0.0;
        off[j] = c < Pi ? 4u * (uint32_t)c : kOOB;
        // bit0 x = 0, bit1 x = nx - 1, bit2 y = 0, bit3 y = ny - 1: the upwind
        // neighbour of direction d is a ghost where d & e != 0
        const int e = (x == 0 ? 1 : 0) | (x == nx - 1 ? 2 : 0) | (y == 0 ? 4 : 0) |
                      (y == ny - 1 ? 8 : 0);
        e_in |= e << (4 * j);
        live |= in ? 1 << j : 0;
        wedge |= __ballot(in && e != 0) ? 1 << j : 0;
    }
    double defect = 0.0, outflow = 0.0;

    // staged segment start (16-byte aligned, may be negative)
    auto seg_start = [&](int dir) { return (dir & 4) ? ((b0 - nx - 1) & ~3) : ((b0 - 1) & ~3); };
    struct Plane {
        float4 r[NR];
        float y[J];
    };
    auto load = [&](int q, int dir, Plane& pn) {
        // bounds at the pitch (cells C .. P - 1 hold zeros), so a float4 never straddles
        const __amdgpu_buffer_rsrc_t rp = plane_rsrc(a.psi + (size_t)q * a.P, a.P);
        const __amdgpu_buffer_rsrc_t ry = plane_rsrc(a.Y + (size_t)q * a.P, a.P);
        const int st = seg_start(dir);
        const int seg_len = L + nx + 8;   // floats the update reads (rounds past it are not fetched)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int i = 4 * (tid + T * r);
            const int c = st + i;
            const uint32_t o = (c >= 0 && i < seg_len) ? 4u * (uint32_t)c : kOOB;
            pn.r[r] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rp, o, 0, 0));
        }
#pragma unroll
        for (int j = 0; j < J; ++j) pn.y[j] = load_plane_nt(ry, off[j]);
    };
    __shared__ float4 seg[2][NR * T];
    const ASN_G QInfo* __restrict__ qtab = gp(a.qi);
    // stage: the plane's segment into LDS buffer q & 1 (consumes the slot's segment)
    auto stage = [&](int q, const Plane& cur) {
        float4* sq = seg[q & 1];
#pragma unroll
        for (int r = 0; r < NR; ++r) sq[tid + T * r] = cur.r[r];
    };
    // compute: the update of plane q from LDS buffer q & 1 and the slot's Y values
    auto compute = [&](int q, const QInfo& qc, const Plane& cur) {
        lds_barrier();
        const int d = qc.dir;
        const float* sf = reinterpret_cast<const float*>(seg[q & 1]) + (b0 - seg_start(d) + tid);
        const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.psi_new + (size_t)q * a.P, a.P);
        const int ysh = (d & 4) ? -nx : nx;   // y-upwind cell (cy = 0 when d & 12 = 0)
        const int xsh = (d & 1) ? -1 : 1;     // x-upwind cell (cx = 0 when d & 3 = 0)
        const int dout = ((d & 5) << 1) | ((d & 10) >> 1);   // outflow faces of d
        float colsum = 0.f, o = 0.f;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const float* pc = sf + T * j;
            const int e = (e_in >> (4 * j)) & 15;
            const bool in = (live >> j) & 1;
            const float v = pc[0];
            const float ux = (d & e & 3) ? 0.f : pc[xsh];
            const float uy = (d & e & 12) ? 0.f : pc[ysh];
            const float col = gs[j] * ((cur.y[j] - fix[j]) - v) + bs[j] * (isov[j] - v);
            const float r = v - qc.cx * (v - ux) - qc.cy * (v - uy) - aa[j] * v + col + ss[j];
            const float nv = in ? r : 0.f;   // padding cells stay zero
            store_plane_nt(nv, ro, off[j]);
            phacc[j] += qc.w * (double)nv;
            colsum += in ? col : 0.f;
            if ((wedge >> j) & 1) {   // only waves holding a boundary cell j
                const int go = dout & e;
                o += in ? ((go & 3) ? qc.cx * v : 0.f) + ((go & 12) ? qc.cy * v : 0.f) : 0.f;
            }
            if (LP) mx[j] = fmaxf(mx[j], fabsf(nv));
        }
        defect += qc.w * (double)colsum;
        outflow += qc.w * (double)o;
    };
    // two plane slots used alternately, loads unconditional (as in stream + collide).
    // Loads and stores share one counter, so the wait for a slot also waits for loads
    // issued after it: more slots or planes per wait did not help (measured).
    const int ql = max(q1 - 1, 0);
    Plane pa, pb;
    QInfo qa = qtab[min(q0, ql)], qb;
    load(min(q0, ql), qa.dir, pa);
    for (int q = q0; q < q1; q += 2) {
        const int qn = min(q + 1, ql);
        qb = qtab[qn];
        load(qn, qb.dir, pb);
        stage(q, pa);
        compute(q, qa, pa);
        if (q + 1 >= q1) break;
        const int qn2 = min(q + 2, ql);
        qa = qtab[qn2];
        load(qn2, qa.dir, pa);
        stage(q + 1, pb);
        compute(q + 1, qb, pb);
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
        if ((live >> j) & 1) gp(a.phi_part)[(size_t)g * a.P + b0 + tid + T * j] = phacc[j];
    if (LP) {
        // a wave's 64 cells j lie in one scale block of the next operand
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const unsigned m = wave_max_u32(__float_as_uint(mx[j]));
            const int cw = b0 + (tid & ~63) + T * j;
            if (lane == 0 && m && cw < Pi) atomicMax(&a.bmax_next[cw >> a.sb_log], m);
        }
    }
    double sums[2] = {defect, outflow};
    block_sum_waves<T / 64, 2>(sums, gp(a.blk_part) + 2 * (size_t)local);
}

// ---------------------------------------------------------------------------
// 2b. Heun stage with limited second-order upwind fluxes (paper Section 3.1).
//     Per ordinate and axis a cell's slope is minmod(psi_i - psi_{i-1},
//     psi_{i+1} - psi_i); a face carries the value reconstructed on its upwind
//     side, psi_i + s_i / 2 or psi_{i+1} - s_{i+1} / 2, and cells outside the
//     grid read 0 (vacuum, also for their slopes).  Same block shape as
//     stream_collide_kernel, with a strip of 60 columns: lane l holds column
//     x0 + l - 2, lanes 2..61 update, and each wave reads two halo rows on each side.
//     Runs for grids wider than the flat-chunk form takes (muscl_flat_kernel).
//       STAGE 1: out = psi + dt R(psi)                 (psi^n  -> psi^1)
//       STAGE 2: out = (old + psi + dt R(psi)) / 2     (psi^1, old = psi^n)
//     In stage 2 the output buffer holds psi^n: every lane reads its own cell
//     of it before overwriting that cell, and no other lane reads it.
// ---------------------------------------------------------------------------
// minmod(a, b) is the median of a, b and 0: the operand of smaller magnitude when the
// signs agree, else 0 (one v_med3_f32).
__device__ __forceinline__ float minmod(float a, float b) {
    return __builtin_amdgcn_fmed3f(a, b, 0.f);
}

template <bool LP, int STAGE>
__global__ __launch_bounds__(256) void muscl_kernel(BatchArgs B) {
    constexpr int R = kRows;
    int pi, local;
    if (!locate(B, KT_SC, blockIdx.x, pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int bx = local % a.tiles_x;
    const int by = (local / a.tiles_x) % a.tiles_y;
    const int g = local / (a.tiles_x * a.tiles_y);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nx = a.nx, ny = a.ny;
    const int64_t P = a.P, C = a.C;
    const int x = bx * kStripXM + lane - 2;
    const int ybase = by * kTileY + wave * R;
    const int q0 = g * a.qchunk;
    const int q1 = min(a.Q, q0 + a.qchunk);
    const bool xok = x >= 0 && x < nx;
    const bool outl = xok && lane >= 2 && lane <= 61;

    float aa[R], bs[R], gs[R], ss[R], isov[R], fix[R], mx[R];
    double phacc[R];
    bool in[R];
    uint32_t off_ld[R], off_st[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = ybase + r;
        const bool yok = y < ny;
        const uint32_t c = (uint32_t)(y * nx + x);
        in[r] = outl && yok;
        off_ld[r] = (xok && yok) ? 4u * c : kOOB;
        off_st[r] = in[r] ? 4u * c : kOOB;
        aa[r] = bs[r] = gs[r] = ss[r] = isov[r] = fix[r] = 0.f;
        mx[r] = 0.f;
        phacc[r] = 0.0;
        if (in[r]) {
            const float4 cf = gp(a.coef)[c];
            aa[r] = cf.x;
            bs[r] = cf.y;
            gs[r] = cf.z;
            ss[r] = cf.w;
            isov[r] = gp(a.iso)[c];
            if (LP) fix[r] = gp(a.fix)[c];
        }
    }
    // halo rows ybase - 2, ybase - 1, ybase + R, ybase + R + 1
    uint32_t off_h[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int yy = k < 2 ? ybase - 2 + k : ybase + R + (k - 2);
        off_h[k] = (xok && yy >= 0 && yy < ny) ? 4u * (uint32_t)(yy * nx + x) : kOOB;
    }
    const bool edge = bx == 0 || bx == a.tiles_x - 1 || by == 0 || by == a.tiles_y - 1;
    double defect = 0.0, outflow = 0.0;

    struct Plane {
        float v[R], y[R], h[4], o[R];
    };
    auto load = [&](int q, int dir, Plane& pn) {
        const __amdgpu_buffer_rsrc_t rp = plane_rsrc(a.psi + (size_t)q * P, C);
        const __amdgpu_buffer_rsrc_t ry = plane_rsrc(a.Y + (size_t)q * P, C);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pn.v[r] = load_plane(rp, off_ld[r]);
            pn.y[r] = load_plane(ry, off_ld[r]);
        }
        // eta > 0 takes two rows below and one above, eta < 0 the mirror image; only
        // the block's outer halo rows come from memory (wave 0 below the tile, wave 3
        // above it), the others are the neighbouring waves' own rows, through LDS
        pn.h[0] = load_plane(rp, ((dir & 4) && wave == 0) ? off_h[0] : kOOB);
        pn.h[1] = load_plane(rp, ((dir & 12) && wave == 0) ? off_h[1] : kOOB);
        pn.h[2] = load_plane(rp, ((dir & 12) && wave == 3) ? off_h[2] : kOOB);
        pn.h[3] = load_plane(rp, ((dir & 8) && wave == 3) ? off_h[3] : kOOB);
        if (STAGE == 2) {
            const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.psi_new + (size_t)q * P, C);
#pragma unroll
            for (int r = 0; r < R; ++r) pn.o[r] = load_plane(ro, off_st[r]);
        }
    };

    // Two plane slots used alternately, loads unconditional (as in stream + collide).
    const ASN_G QInfo* __restrict__ qtab = gp(a.qi);
    // xr[q & 1][row of the tile][lane]: the tile's 16 rows of plane q; hr[q & 1][wave][k]:
    // the halo rows each wave loaded (only waves 0 and 3 load any; every wave stores its
    // slots so that no store depends on the wave index)
    __shared__ float xr[2][kTileY][64];
    __shared__ float hr[2][4][4][64];
    auto body = [&](int q, const QInfo& qc, const Plane& cur) {
        const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.psi_new + (size_t)q * P, C);
        float (*xq)[64] = xr[q & 1];
#pragma unroll
        for (int r = 0; r < R; ++r) xq[wave * R + r][lane] = cur.v[r];
#pragma unroll
        for (int k = 0; k < 4; ++k) hr[q & 1][wave][k][lane] = cur.h[k];
        lds_barrier();
        // column e[k] = row ybase - 2 + k: two rows below the wave's rows (the tile's
        // outer halo for wave 0), its own rows, two rows above (outer halo for wave 3)
        const float* lo = wave == 0 ? &hr[q & 1][0][0][0] : &xq[wave * R - 2][0];
        const float* hi = wave == 3 ? &hr[q & 1][3][2][0] : &xq[(wave + 1) * R][0];
        float e[R + 4];
        e[0] = lo[lane];
        e[1] = lo[64 + lane];
#pragma unroll
        for (int r = 0; r < R; ++r) e[r + 2] = cur.v[r];
        e[R + 2] = hi[lane];
        e[R + 3] = hi[64 + lane];
        // upwind face values along y: fy[k] = value on the face above row k - 2
        // (eta > 0, k = 1..R+1 used) or below row k - 2 (eta < 0, k = 2..R+2 used)
        float fy[R + 4];
#pragma unroll
        for (int k = 1; k < R + 3; ++k) {
            const float sl = minmod(e[k] - e[k - 1], e[k + 1] - e[k]);
            fy[k] = (qc.dir & 4) ? e[k] + 0.5f * sl : e[k] - 0.5f * sl;
        }
        float colsum = 0.f, o = 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float v = cur.v[r];
            const float vl = __shfl_up(v, 1, 64);
            const float vr = __shfl_down(v, 1, 64);
            const float sx = minmod(v - vl, vr - v);
            float dfx = 0.f, fout_x = 0.f;
            if (qc.dir & 1) {
                const float f = v + 0.5f * sx;
                dfx = f - __shfl_up(f, 1, 64);
                fout_x = f;
            } else if (qc.dir & 2) {
                const float gl = v - 0.5f * sx;
                dfx = gl - __shfl_down(gl, 1, 64);
                fout_x = gl;
            }
            float dfy = 0.f, fout_y = 0.f;
            if (qc.dir & 4) {
                dfy = fy[r + 2] - fy[r + 1];
                fout_y = fy[r + 2];
            } else if (qc.dir & 8) {
                dfy = fy[r + 2] - fy[r + 3];
                fout_y = fy[r + 2];
            }
            const float col = gs[r] * ((cur.y[r] - fix[r]) - v) + bs[r] * (isov[r] - v);
            const float nv = v - qc.cx * dfx - qc.cy * dfy - aa[r] * v + col + ss[r];
            const float res = STAGE == 2 ? 0.5f * (cur.o[r] + nv) : nv;
            store_plane(res, ro, off_st[r]);
            phacc[r] += qc.w * (double)res;
            colsum += in[r] ? col : 0.f;
            if (LP) mx[r] = fmaxf(mx[r], in[r] ? fabsf(res) : 0.f);
            if (edge && in[r]) {
                // particles leaving through a boundary face: the reconstructed
                // value on the face of the last cell, for directions that exit there
                const int y = ybase + r;
                if (((qc.dir & 1) && x == nx - 1) || ((qc.dir & 2) && x == 0)) o += qc.cx * fout_x;
                if (((qc.dir & 4) && y == ny - 1) || ((qc.dir & 8) && y == 0)) o += qc.cy * fout_y;
            }
        }
        defect += qc.w * (double)colsum;
        outflow += qc.w * (double)o;
    };
    Plane pa, pb;
    QInfo qa = qtab[min(q0, a.Q - 1)], qb;
    load(min(q0, a.Q - 1), qa.dir, pa);
    for (int q = q0; q < q1; q += 2) {
        const int qn = min(q + 1, q1 - 1);
        qb = qtab[qn];
        load(qn, qb.dir, pb);
        body(q, qa, pa);
        if (q + 1 >= q1) break;
        const int qn2 = min(q + 2, q1 - 1);
        qa = qtab[qn2];
        load(qn2, qa.dir, pa);
        body(q + 1, qb, pb);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (in[r]) gp(a.phi_part)[(size_t)g * P + (uint32_t)((ybase + r) * nx + x)] = phacc[r];
    if (LP) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int y = ybase + r;
            const int64_t c_first = (int64_t)y * nx + bx * kStripXM;
            const int64_t b0 = c_first >> a.sb_log;
            const int64_t cb = ((int64_t)y * nx + x) >> a.sb_log;
            const unsigned bits = in[r] ? __float_as_uint(mx[r]) : 0u;
            const unsigned m0 = wave_max_u32(cb == b0 ? bits : 0u);
            const unsigned m1 = wave_max_u32(cb != b0 ? bits : 0u);
            if (lane == 0 && y < ny) {
                if (m0) atomicMax(&a.bmax_next[b0], m0);
                if (m1) atomicMax(&a.bmax_next[b0 + 1], m1);
            }
        }
    }
    double sums[2] = {defect, outflow};
    block_sum_256<2>(sums, gp(a.blk_part) + 2 * (size_t)local);
}

// Per-cell particle correction of the reduced-precision Y: the w-weighted sum of
// Y over all ordinates (from the per-tile partials, fixed order) minus Phi, over W.
__global__ __launch_bounds__(256) void particle_fix_kernel(BatchArgs B) {
    int pi, local;
    if (!locate(B, KT_FIX, blockIdx.x, pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int64_t c = (int64_t)local * 256 + threadIdx.x;
    if (c >= a.C) return;
    double m = -gp(a.phi64)[c];
    const int nparts = a.Qp / kGemmBM;
    const ASN_G double* yp = gp(a.ypart);
    for (int t = 0; t < nparts; ++t) m += yp[(size_t)t * a.P + c];
    gp(a.fix)[c] = (float)(m / a.W);
}

// ---------------------------------------------------------------------------
// 2c. Heun pass over flat cell chunks: the MUSCL update of muscl_kernel (same
//     arithmetic) in the flat-chunk form of stream_collide_flat_kernel.  The staged
//     segment holds the chunk with two cells of x context and the two rows below and
//     one above it (eta > 0) or the mirror image (eta < 0).  Cells beyond the grid's
//     rows read as zero; x ghosts (two per side) are masked from the cell's x.  Thread
//     t updates cells b0 + t + 512 j, j = 0..3, so that the 64 lanes of a wave read
//     64 consecutive LDS words (no bank conflicts) and store 256 contiguous bytes.
// ---------------------------------------------------------------------------
template <bool LP, int STAGE>
__global__ __launch_bounds__(kFlatThreads) void muscl_flat_kernel(BatchArgs B) {
    constexpr int T = kFlatThreads, L = kFlatCells, NR = kFlatRounds, J = L / T;
    int pi, local;
    // consecutive chunks on one XCD: the rows a chunk stages beyond its own cells are
    // its neighbours' cells, read at about the same time through the same L2
    if (!locate(B, KT_SC, xcd_remap(blockIdx.x, gridDim.x), pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int tiles = a.tiles_x;
    const int bt = local % tiles, g = local / tiles;
    const int tid = threadIdx.x, lane = tid & 63;
    const int nx = a.nx, ny = a.ny;
    const int C = (int)a.C, Pi = (int)a.P;
    const int b0 = bt * L;
    const int q0 = g * a.qchunk;
    const int q1 = min(a.Q, q0 + a.qchunk);

    float aa[J], bs[J], gs[J], ss[J], isov[J], fix[J], mx[J];
    int xk[J];
    uint32_t off[J];   // byte offset of the cell in a plane, out of range beyond the pitch
    double phacc[J];
    int live = 0;      // bit j: cell j is a grid cell (not padding)
    unsigned ex = 0;   // 4 bits per cell: the direction bits that leave the grid there
    int wexit = 0;     // bit j: some lane of the wave holds a boundary cell j (uniform)
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int c = b0 + tid + T * j;
        const bool in = c < C;
        const int y = c / nx, x = c - y * nx;
        float4 cf = make_float4(0.f, 0.f, 0.f, 0.f);
        if (in) cf = gp(a.coef)[c];
        aa[j] = cf.x;
        bs[j] = cf.y;
        gs[j] = cf.z;
        ss[j] = cf.w;
        isov[j] = in ? gp(a.iso)[c] : 0.f;
        fix[j] = (LP && in) ? gp(a.fix)[c] : 0.f;
        mx[j] = 0.f;
        phacc[j] = 0.0;
        xk[j] = x;
        off[j] = c < Pi ? 4u * (uint32_t)c : kOOB;
        live |= in ? 1 << j : 0;
        // +x leaves at x = nx - 1, -x at x = 0, +y at y = ny - 1, -y at y = 0
        const unsigned e = in ? (unsigned)(x == nx - 1) | (unsigned)(x == 0) << 1 |
                                    (unsigned)(y == ny - 1) << 2 | (unsigned)(y == 0) << 3
                              : 0u;
        ex |= e << (4 * j);
        wexit |= __ballot(e != 0) ? 1 << j : 0;
    }
    double defect = 0.0, outflow = 0.0;

    // staged segment start (16-byte aligned, may be negative)
    auto seg_start = [&](int dir) {
        return (dir & 4) ? ((b0 - 2 * nx - 2) & ~3) : ((dir & 8) ? ((b0 - nx - 2) & ~3) : ((b0 - 2) & ~3));
    };
    struct Plane {
        float4 r[NR];
        float y[J], o[J];
    };
    auto load = [&](int q, int dir, Plane& pn) {
        // bounds at the pitch (cells C .. P - 1 hold zeros), so a float4 never straddles
        const __amdgpu_buffer_rsrc_t rp = plane_rsrc(a.psi + (size_t)q * a.P, a.P);
        const __amdgpu_buffer_rsrc_t ry = plane_rsrc(a.Y + (size_t)q * a.P, a.P);
        const int st = seg_start(dir);
        const int seg_len = L + 3 * nx + 8;   // floats the update reads
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int i = 4 * (tid + T * r);
            const int c = st + i;
            const uint32_t o = (c >= 0 && i < seg_len) ? 4u * (uint32_t)c : kOOB;
            pn.r[r] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rp, o, 0, 0));
        }
#pragma unroll
        for (int j = 0; j < J; ++j) pn.y[j] = load_plane(ry, off[j]);
        if (STAGE == 2) {   // the old level, stored where the result goes
            const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.psi_new + (size_t)q * a.P, a.P);
#pragma unroll
            for (int j = 0; j < J; ++j) pn.o[j] = load_plane(ro, off[j]);
        } else {
#pragma unroll
            for (int j = 0; j < J; ++j) pn.o[j] = 0.f;
        }
    };
    __shared__ float4 seg[2][NR * T];
    const ASN_G QInfo* __restrict__ qtab = gp(a.qi);
    auto body = [&](int q, const QInfo& qc, const Plane& cur) {
        float4* sq = seg[q & 1];
#pragma unroll
        for (int r = 0; r < NR; ++r) sq[tid + T * r] = cur.r[r];
        lds_barrier();
        const int d = qc.dir;
        const float* sf = reinterpret_cast<const float*>(sq) + (b0 - seg_start(d) + tid);
        const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.psi_new + (size_t)q * a.P, a.P);
        float colsum = 0.f, o = 0.f;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const float* pc = sf + T * j;
            const int x = xk[j];
            const float v = pc[0];
            // x neighbours, zero ghosts outside the row
            const float vm1 = x >= 1 ? pc[-1] : 0.f;
            const float vp1 = x <= nx - 2 ? pc[1] : 0.f;
            const float sx = minmod(v - vm1, vp1 - v);
            float dfx = 0.f, fout_x = 0.f;
            if (d & 1) {
                const float vm2 = x >= 2 ? pc[-2] : 0.f;
                const float f = v + 0.5f * sx;
                const float fl = vm1 + 0.5f * minmod(vm1 - vm2, v - vm1);
                dfx = f - fl;
                fout_x = f;
            } else if (d & 2) {
                const float vp2 = x <= nx - 3 ? pc[2] : 0.f;
                const float gl = v - 0.5f * sx;
                const float gr = vp1 - 0.5f * minmod(vp1 - v, vp2 - vp1);
                dfx = gl - gr;
                fout_x = gl;
            }
            // y neighbours (rows beyond the grid read as zero)
            float dfy = 0.f, fout_y = 0.f;
            if (d & 4) {
                const float ym2 = pc[-2 * nx], ym1 = pc[-nx], yp1 = pc[nx];
                const float f = v + 0.5f * minmod(v - ym1, yp1 - v);
                const float fb = ym1 + 0.5f * minmod(ym1 - ym2, v - ym1);
                dfy = f - fb;
                fout_y = f;
            } else if (d & 8) {
                const float ym1 = pc[-nx], yp1 = pc[nx], yp2 = pc[2 * nx];
                const float gb = v - 0.5f * minmod(v - ym1, yp1 - v);
                const float ga = yp1 - 0.5f * minmod(yp1 - v, yp2 - yp1);
                dfy = gb - ga;
                fout_y = gb;
            }
            const bool in = (live >> j) & 1;
            const float col = gs[j] * ((cur.y[j] - fix[j]) - v) + bs[j] * (isov[j] - v);
            const float nv = v - qc.cx * dfx - qc.cy * dfy - aa[j] * v + col + ss[j];
            const float res = STAGE == 2 ? 0.5f * (cur.o[j] + nv) : nv;
            const float rv = in ? res : 0.f;   // padding cells stay zero
            store_plane(rv, ro, off[j]);
            phacc[j] += qc.w * (double)rv;
            colsum += in ? col : 0.f;
            if (LP) mx[j] = fmaxf(mx[j], fabsf(rv));
            if ((wexit >> j) & 1) {
                // particles leaving through a boundary face: the reconstructed value on
                // the face of the last cell, for directions that exit there
                const unsigned e = (ex >> (4 * j)) & (unsigned)d;
                if (e & 3u) o += qc.cx * fout_x;
                if (e & 12u) o += qc.cy * fout_y;
            }
        }
        defect += qc.w * (double)colsum;
        outflow += qc.w * (double)o;
    };
    // two plane slots used alternately, loads unconditional (as in stream + collide)
    Plane pa, pb;
    QInfo qa = qtab[min(q0, a.Q - 1)], qb;
    load(min(q0, a.Q - 1), qa.dir, pa);
    for (int q = q0; q < q1; q += 2) {
        const int qn = min(q + 1, q1 - 1);
        qb = qtab[qn];
        load(qn, qb.dir, pb);
        body(q, qa, pa);
        if (q + 1 >= q1) break;
        const int qn2 = min(q + 2, q1 - 1);
        qa = qtab[qn2];
        load(qn2, qa.dir, pa);
        body(q + 1, qb, pb);
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
        if ((live >> j) & 1) gp(a.phi_part)[(size_t)g * a.P + b0 + tid + T * j] = phacc[j];
    if (LP) {
        // a wave's 64 cells j lie in one scale block of the next operand
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const unsigned m = wave_max_u32(__float_as_uint(mx[j]));
            const int cw = b0 + (tid & ~63) + T * j;
            if (lane == 0 && m && cw < Pi) atomicMax(&a.bmax_next[cw >> a.sb_log], m);
        }
    }
    double sums[2] = {defect, outflow};
    block_sum_waves<T / 64, 2>(sums, gp(a.blk_part) + 2 * (size_t)local);
}

// ---------------------------------------------------------------------------
// 3. Finalize: Phi = sum of the G partials (fixed order), Phi/W, mass partials.
// ---------------------------------------------------------------------------
// sum over g < G of p[g P + c], added in the order g = 0, 1, ...; the loads of eight
// partials are issued together (one memory round trip per eight, not per partial)
__device__ __forceinline__ double sum_partials(const ASN_G double* p, int G, int64_t P,
                                               int64_t c) {
    double s = 0.0;
    for (int g0 = 0; g0 < G; g0 += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(size_t)min(g0 + u, G - 1) * P + c];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (g0 + u < G) s += v[u];
    }
    return s;
}

__global__ __launch_bounds__(256) void finalize_kernel(BatchArgs B, int init) {
    int pi, local;
    if (!locate(B, KT_FIN, blockIdx.x, pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int G = init ? 1 : a.G;
    ASN_G unsigned* bmax_zero = init ? nullptr : gp(a.bmax_cur);
    const int64_t c = (int64_t)local * 256 + threadIdx.x;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (c < a.C) {
        const float4 cf = gp(a.coef)[c];
        const bool lp_fused = a.dtype != 0 && a.fused;
        const double phi_old = lp_fused && !init ? gp(a.phi64)[c] : 0.0;
        double phi = sum_partials(gp(a.phi_part), G, a.P, c);
        double corr = 0.0;   // W delta: particles of the pending correction (fused BF16 / FP16)
        if (lp_fused) {
            if (init) {
                gp(a.delta)[c] = 0.f;
            } else {
                // the particle correction of this step's reduced-precision Y: every
                // ordinate of the cell gets delta = -dt sigma_as (sum_q w_q Y^ - Phi^n) / W
                const double ys = sum_partials(gp(a.ypart), G, a.P, c);
                const float d = (float)(-(double)cf.z * (ys - phi_old) / a.W);
                gp(a.delta)[c] = d;
                corr = a.W * (double)d;
            }
        }
        // iso holds Phi^ / W of the stored state; phi64 the true Phi
        gp(a.iso)[c] = (float)(phi / a.W);
        phi += corr;
        gp(a.phi64)[c] = phi;
        s[0] = phi;
        s[1] = (double)cf.x * phi;
        s[2] = (double)cf.w;
        s[3] = corr;
    }
    if (bmax_zero != nullptr && c < scale_blocks(a.P, a.sb_log)) bmax_zero[c] = 0u;
    block_sum_256<4>(s, gp(a.fin_part) + 4 * (size_t)local);
}

// The stored state of a fused reduced-precision problem plus its pending per-cell
// correction becomes the plain state: psi[q][c] += delta[c], delta = 0, iso = Phi / W.
// Four cells (P is a multiple; delta is 0 beyond C) and eight planes a thread: 700^2 x 1152 1.27 ->
// 0.90 ms (5.0 TB/s).
constexpr int kMaterialize = 8;
__global__ __launch_bounds__(256) void materialize_kernel(StepArgs a, float* psi) {
    const int64_t c = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
    if (c >= a.P) return;
    const f32x4 d = *reinterpret_cast<const ASN_G f32x4*>(gp(a.delta) + c);
    const int q0 = blockIdx.y * kMaterialize;
    f32x4 v[kMaterialize];
#pragma unroll
    for (int u = 0; u < kMaterialize; ++u)
        v[u] = *reinterpret_cast<const ASN_G f32x4*>(gp(psi) + (size_t)min(q0 + u, a.Q - 1) * a.P + c);
#pragma unroll
    for (int u = 0; u < kMaterialize; ++u)
        if (q0 + u < a.Q) *reinterpret_cast<ASN_G f32x4*>(gp(psi) + (size_t)(q0 + u) * a.P + c) = v[u] + d;
}

__global__ void materialize_done_kernel(StepArgs a) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.C) return;
    a.delta[c] = 0.f;
    a.iso[c] = (float)(a.phi64[c] / a.W);
}

// ---------------------------------------------------------------------------
// 4. Budget: fold block partials into the record (one block, fixed order).
// ---------------------------------------------------------------------------
//    BUD_STEP    Euler step: M^{n+1} against M^n - A^n - O + S + D.
//    BUD_STAGE1  Heun, first pass: checks the intermediate level M^1 against
//                M^n + its full increment, and keeps half of that increment.
//    BUD_STAGE2  Heun, second pass: M^{n+1} against M^n + half of each pass's
//                increment (the new level is the mean of psi^n and psi^1 +
//                dt R(psi^1)).
//    BUD_INIT    after set_state: M^0.
// One block of 1024 threads per problem.  Each thread folds a strided share of the
// partials, the loads of both kinds issued together, four of each at a time (one
// round trip per four partials instead of per partial), then the block folds the
// threads in a fixed order.  Thread 0 reads the record while the partials arrive and
// writes it back whole.
constexpr int kBudgetThreads = 1024;
// T: threads of the block (at most kBudgetThreads); n_fin, n_blk: partials of either kind; U: of
// each in flight a thread (1: and the record loaded after them, for the fewest registers).
template <int U = 4>
__device__ __forceinline__ void budget_fold(const StepArgs& a, int n_fin, int n_blk, int T, int mode) {
#pragma clang fp contract(off)   // (the same bits from each kernel it is part of)
    const bool init = mode == BUD_INIT;
    ASN_G double* rec = gp(a.rec);
    double r[REC_LEN];
    auto record = [&] {
#pragma unroll
        for (int k = 0; k < REC_LEN; ++k) r[k] = rec[k];
    };
    if (U > 1 && threadIdx.x == 0) record();
    double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const ASN_G double4* fp = reinterpret_cast<const ASN_G double4*>(gp(a.fin_part));
    const ASN_G double2* bp = reinterpret_cast<const ASN_G double2*>(gp(a.blk_part));
    for (int i0 = threadIdx.x; i0 < max(n_fin, n_blk); i0 += T * U) {
        double4 v[U];
        double2 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * T;
            v[u] = fp[min(i, n_fin - 1)];
            w[u] = double2{0.0, 0.0};
            if (n_blk > 0) w[u] = bp[min(i, n_blk - 1)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * T;
            if (i < n_fin) {
                s[0] += v[u].x;
                s[1] += v[u].y;
                s[2] += v[u].z;
                s[5] += v[u].w;
            }
            if (i < n_blk) {
                s[3] += w[u].x;
                s[4] += w[u].y;
            }
        }
    }
    __shared__ double tot[6];
    block_sum_n<kBudgetThreads / 64, 6>(s, T / 64, tot);
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (U == 1) record();
    const double m_next = a.area * tot[0];
    const double abs_next = a.area * tot[1];
    auto store = [&]() {
#pragma unroll
        for (int k = 0; k < REC_LEN; ++k) rec[k] = r[k];
    };
    if (init) {
#pragma unroll
        for (int k = 0; k < REC_LEN; ++k) r[k] = 0.0;
        r[REC_MASS] = m_next;
        r[REC_MASS0] = m_next;
        r[REC_ABS_NEXT] = abs_next;
        r[REC_SRC_STEP] = a.area * a.W * tot[2];
        store();
        return;
    }
    // collision defect: the stencil's increments plus the pending correction's particles
    const double def = a.area * (tot[3] + tot[5]);
    const double out = a.area * tot[4];
    const double ref = fmax(r[REC_MASS0], r[REC_MASS]);
    auto residual = [&](double got, double pred) {
        const double rel = ref > 0.0 ? fabs(got - pred) / ref : fabs(got - pred);
        r[REC_RES] = fmax(r[REC_RES], rel);
    };
    if (mode == BUD_STEP) {
        residual(m_next, r[REC_MASS] - r[REC_ABS_NEXT] - out + r[REC_SRC_STEP] + def);
        r[REC_ABS] += r[REC_ABS_NEXT];
        r[REC_OUT] += out;
        r[REC_SRC] += r[REC_SRC_STEP];
        r[REC_DEF] += def;
        r[REC_STEPS] += 1.0;
        r[REC_MASS] = m_next;
        r[REC_ABS_NEXT] = abs_next;
        store();
        return;
    }
    // Heun passes: each contributes half of its increment to the step
    const double abs_in = mode == BUD_STAGE1 ? r[REC_ABS_NEXT] : r[REC_ABS_STAGE];
    const double inc = -abs_in - out + r[REC_SRC_STEP] + def;
    r[REC_ABS] += 0.5 * abs_in;
    r[REC_OUT] += 0.5 * out;
    r[REC_SRC] += 0.5 * r[REC_SRC_STEP];
    r[REC_DEF] += 0.5 * def;
    if (mode == BUD_STAGE1) {
        residual(m_next, r[REC_MASS] + inc);
        r[REC_HALF] = 0.5 * inc;
        r[REC_ABS_STAGE] = abs_next;
    } else {
        residual(m_next, r[REC_MASS] + r[REC_HALF] + 0.5 * inc);
        r[REC_STEPS] += 1.0;
        r[REC_MASS] = m_next;
        r[REC_ABS_NEXT] = abs_next;
    }
    store();
}

// One block per problem.  A banded pass's partials are one of either kind per block of the
// pass; its fold takes band_fold_threads(n_az) threads here and in the next pass's launch, so
// that a record does not depend on which of the two did it.
__device__ __forceinline__ int band_fold_threads(int n_az) { return n_az / kBandO * 64; }
__global__ __launch_bounds__(kBudgetThreads) void budget_kernel(BatchArgs B, int mode, bool banded) {
    const int pi = blockIdx.x;
    if (gp(B.limit)[pi] <= B.step) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    if (banded) {
        if ((int)threadIdx.x >= band_fold_threads(a.n_az)) return;
        budget_fold(a, a.tiles_x, a.tiles_x, band_fold_threads(a.n_az), mode);
    } else
        budget_fold(a, a.fin_blocks, mode == BUD_INIT ? 0 : a.tiles_x * a.tiles_y * a.G, kBudgetThreads, mode);
}

// Tables that the host writes before any step and the kernels only read: reached through the
// constant address space, their uniform loads are scalar (SMEM) loads, which do not wait behind
// the vector memory counter.
#if defined(__HIP_DEVICE_COMPILE__)
#define ASN_K __attribute__((address_space(4)))
#else
#define ASN_K
#endif
template <typename T>
__device__ __forceinline__ const ASN_K T* kp(const T* p) {
    return (const ASN_K T*)p;
}

// ---------------------------------------------------------------------------
// Moments of a freshly set state: Phi partial (G = 1) and block max |psi|.  `cell`: the value
// of every ordinate of a cell where the state is isotropic (the same sum, without reading the
// state), or NULL.  A call that sets an isotropic state, with four cells and eight planes a thread
// in broadcast_kernel: 1024^2 x 2048 4.97 -> 2.53 ms (3.4 TB/s of writes), 700^2 x 1152 1.35 ->
// 0.79 ms, 50^2 x 128 93 -> 70 us; one that sets any, 311 x 173 x 288 154 -> 118 us.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void moments_kernel(StepArgs a, const float* cell) {
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= a.C) return;
    double phi = 0.0;
    float mx = 0.f;
    const ASN_K QInfo* qi = kp(a.qi);
    if (cell) {
        const float v = gp(cell)[c];
        for (int q = 0; q < a.Q; ++q) phi += qi[q].w * (double)v;
        mx = fabsf(v);
    } else {
        constexpr int U = 16;   // planes in flight: a thread's reads are a chain otherwise
        for (int q0 = 0; q0 < a.Q; q0 += U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = q0 + u < a.Q ? gp(a.psi)[(size_t)(q0 + u) * a.P + c] : 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (q0 + u < a.Q) phi += qi[q0 + u].w * (double)v[u];
                mx = fmaxf(mx, fabsf(v[u]));
            }
        }
    }
    a.phi_part[c] = phi;
    atomicMax(&a.bmax_cur[c >> (a.band ? 6 : a.sb_log)], __float_as_uint(mx));
}

__global__ void fill_u32_kernel(unsigned* p, int64_t n, unsigned v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Four cells and kBroadcast planes a thread (P is a multiple of four).
constexpr int kBroadcast = 8;
__global__ __launch_bounds__(256) void broadcast_kernel(float* psi, const float* cell, int Q, int64_t C, int64_t P) {
    const int64_t c = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
    if (c >= P) return;
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = c + i < C ? cell[c + i] : 0.f;
    for (int q = blockIdx.y * kBroadcast; q < min(Q, ((int)blockIdx.y + 1) * kBroadcast); ++q)
        *reinterpret_cast<f32x4*>(psi + (size_t)q * P + c) = v;
}

// ---------------------------------------------------------------------------
// 5. Banded step for product ordinate sets (forward Euler; FP32 Heun).
//    The set is invariant under rotations by 2 pi / n_az about the polar axis and under
//    reflection of the azimuth, so Y_(i,k) = sum_j sum_d c_ij(d) (psi_(j, k + d) + psi_(j, k - d)):
//    per pair of levels a short symmetric circular convolution along the azimuth.  The
//    kernel goes by source level: level j's sums over +-d are formed once and serve
//    every output level within `reach`, whose partial sums stay in registers until their
//    last source has passed.  That halves the multiplications of the direct form, reads
//    each LDS row once per source level instead of once per level pair, and keeps two
//    levels in LDS.  Block = kBandCells consecutive cells (flat index) x every ordinate;
//    wave w owns azimuths 4 w .. 4 w + 3 of every level, lane c cell c, so coefficients,
//    (cx, cy) and the flow direction are uniform over a wave (scalar registers).
//    Pass j: convolve level j (LDS slot j & 1); its stream + collide terms but for the
//    in-scattering (x-upwind values from the slot); write level j + 1 into the other slot;
//    finish and store level j - RT; load level j + 2 and the y-upwind values of level
//    j + 1; one LDS barrier.  A pass's scalar loads come in one round trip with its LDS
//    rows (awaited one by one they cost a tenth).  The value and the terms of a level wait in
//    registers for its in-scattering; the pass is written 2 RT + 1 times, so that these
//    and the partial sums rotate by renaming.
//    What bounds it: memory and VALU issue together.  At 1024^2 x 2048 the pass without its
//    loads and stores takes 3.7 ms (203 VALU instructions a wave and level, half of them in
//    the four levels at either pole, which couple up to the whole ring), without its
//    convolution 4.4 ms, as a whole 5.2 ms (all three before the planes' pitch was padded, 5.0 ms
//    with that: 3.4 TB/s on 8 B per update; a 4 GiB copy reaches 4.9, and the y-upwind rows, which
//    the L2 no longer holds at this width, make it 10.0 B moved: 4.3 TB/s); 400^2 x 512 0.172 ms
//    (3.8 TB/s), 700^2 x 1152 1.36 ms.  The direct form (gathering per output level, all levels
//    within reach in LDS) took 6.85, 0.289 and 2.23 ms.  The instances of reach 3 for more than 32
//    azimuths spill, 13 registers in FP32 and 43 in FP16: 32 x 64 azimuths beta 9, 256^2 cells, FP32
//    554 us (reach 2 at beta 4.5: 319; the direct form 884 and 441).  Two levels of loads in flight, flags between neighbouring waves instead of
//    the barrier, and loads issued at the start of a pass instead of its end were all
//    slower: what they add in registers and instructions costs more than they hide.
//    BF16 / FP16 operands: the recipe of the fused reduced-precision form (the state is
//    stored without its pending per-cell correction delta, only the anisotropic part is
//    rounded: x = T((psi^ - iso^) 2^(E - e_b)), Y^ - iso^ = 2^(e_b - E) sum T(K) x + r_q
//    (psi^ - iso^)), its products in FP32: a rounded operand, both BF16 terms together, is an
//    FP32 number.  Where K is narrow the vector units, which skip its zeros, finish before the
//    matrix cores do with each level pair's whole circulant block (the kernel below, for wide K):
//    400^2 x 512 BF16 0.242 -> 0.196 ms, 700^2 x 1152 FP16 1.63 -> 1.34 ms.
//    Heun + minmod, FP32: both passes in this form, instead of a contraction, stencil, finalize
//    and budget kernel each.  A pass without its contraction's round trip through Y reads psi
//    (its three y neighbours from L2) and writes it, the second also reads psi^n, where its
//    result goes.  400^2 x 512 981 -> 531 us a step, 700^2 x 1152 6.78 -> 4.32 ms, 50^2 x 128
//    70 -> 33 us, 2000 x 1000 x 32 0.81 -> 0.41 ms.  Registers bound it, 128 a lane: 16 waves in
//    a CU, with about 120 vector instructions more a wave and level than forward Euler.
// ---------------------------------------------------------------------------
// Awaits scalar loads here (and what is in flight in LDS), so that they are issued together
// and not one by one where each is used.
template <int M>
__device__ __forceinline__ void await(const float (&k)[M]) {
#pragma unroll
    for (int i = 0; i < M; ++i) asm volatile("" ::"s"(k[i]));
}

// The convolution of one source level j: acc[i mod N] += c_ij(d) (v[k + d] + v[k - d]) for
// the output levels i = j - RT .. j + RT (N = 2 RT + 1; P = j mod N, so nothing moves from
// level to level).  Most levels couple the three middle outputs to azimuths at most 2 apart
// and the others to at most 1: those products always; the rest by the level's flags, offsets
// beyond 4 in steps of four, each output as many as it needs (steps: 4 bits each).  lo / hi:
// the lane's column in the four rows before / after its wave's; col: in row 0.
template <int RT, int P, int ROW>
__device__ __forceinline__ void scatter(float (&acc)[2 * RT + 1][kBandO], const float (&v)[kBandO],
                                        const float (&near)[4], const float (&k0)[3 * (2 * RT + 1)],
                                        const float* lo, const float* hi, const float* col, int a0,
                                        int A, uint32_t form, uint32_t steps, const ASN_K float* kc) {
    constexpr int O = kBandO, N = 2 * RT + 1;
    auto add = [&](int m, float k, const float (&s)[O]) {
        const int r = (P + m - RT + N) % N;
#pragma unroll
        for (int o = 0; o < O; ++o) acc[r][o] = fmaf(k, s[o], acc[r][o]);
    };
    auto outer = [](int m) { return m < RT - 1 || m > RT + 1; };
    float up[2 * O], dn[2 * O];   // azimuths a0 .. a0 + 7 and a0 - 4 .. a0 + 3
    auto sum = [&](int d, float (&s)[O]) {
#pragma unroll
        for (int o = 0; o < O; ++o) s[o] = up[o + d] + dn[O + o - d];
    };
#pragma unroll
    for (int o = 0; o < O; ++o) up[o] = dn[O + o] = v[o];
    dn[O - 2] = near[0];
    dn[O - 1] = near[1];
    up[O] = near[2];
    up[O + 1] = near[3];
#pragma unroll
    for (int m = 0; m < N - 1; ++m) add(m, k0[m], v);
#pragma unroll
    for (int o = 0; o < O; ++o) acc[(P + RT) % N][o] = k0[N - 1] * v[o];   // its first source
    float s[O];
    sum(1, s);
#pragma unroll
    for (int m = 0; m < N; ++m) add(m, k0[N + m], s);
    sum(2, s);
#pragma unroll
    for (int m = RT - 1; m <= RT + 1; ++m) add(m, k0[2 * N + m], s);
    if (form & kBandOuter2)
#pragma unroll
        for (int m = 0; m < N; ++m)
            if (outer(m)) add(m, k0[2 * N + m], s);
    if (form & kBandBeyond2) {
        float k[2 * N], s4[O];
#pragma unroll
        for (int i = 0; i < 2 * N; ++i) k[i] = kc[3 * N + i];
        up[O + 2] = hi[2 * ROW];
        up[O + 3] = hi[3 * ROW];
        dn[1] = lo[ROW];
        dn[0] = lo[0];
        await(k);
        sum(3, s);
        sum(4, s4);
#pragma unroll
        for (int m = RT - 1; m <= RT + 1; ++m) {
            add(m, k[m], s);
            add(m, k[N + m], s4);
        }
        if (form & kBandOuter3)
#pragma unroll
            for (int m = 0; m < N; ++m)
                if (outer(m)) {
                    add(m, k[m], s);
                    add(m, k[N + m], s4);
                }
        // the window's halves change roles from step to step
        const int ns = (int)(form & kBandSteps);
        int ah = a0 + O, al = a0 - O;
        float ua[O], ub[O], da[O], db[O];
#pragma unroll
        for (int o = 0; o < O; ++o) {
            ua[o] = up[O + o];
            da[o] = dn[o];
        }
        auto step = [&](int n, float (&u0)[O], float (&u1)[O], float (&d0)[O], float (&d1)[O]) {
            ah = ah >= A - O ? ah + O - A : ah + O;
            al = al < O ? al - O + A : al - O;
            kc += 4 * N;
            const float* ph = col + ah * ROW;
            const float* pl = col + al * ROW;
            float kw[4 * N];
#pragma unroll
            for (int i = 0; i < 4 * N; ++i) kw[i] = kc[N + i];
#pragma unroll
            for (int o = 0; o < O; ++o) {
                u1[o] = ph[o * ROW];
                d1[o] = pl[o * ROW];
            }
            await(kw);
#pragma unroll
            for (int d = 1; d <= 3; d += 2) {
#pragma unroll
                for (int o = 0; o < O; ++o) {
                    s[o] = (o + d < O ? u0[(o + d) % O] : u1[(o + d) % O]) + (o >= d ? d0[(o - d + O) % O] : d1[(o - d + O) % O]);
                    s4[o] = (o + d + 1 < O ? u0[(o + d + 1) % O] : u1[(o + d + 1) % O]) +
                            (o >= d + 1 ? d0[(o - d - 1 + O) % O] : d1[(o - d - 1 + O) % O]);
                }
#pragma unroll
                for (int m = 0; m < N; ++m)
                    if ((int)((steps >> (4 * m)) & 15u) > n) {
                        add(m, kw[(d - 1) * N + m], s);
                        add(m, kw[d * N + m], s4);
                    }
            }
        };
        for (int n = 1; n < ns; n += 2) {
            step(n, ua, ub, da, db);
            if (n + 1 >= ns) break;
            step(n + 1, ub, ua, db, da);
        }
    }
}

// A level's descriptor: the first of its coefficients, the form of its convolution, the
// steps of four offsets of each output level (band_scatter_tables).
struct BandLevel {
    uint32_t coef, form, steps;
};
template <int RT>
__device__ __forceinline__ BandLevel band_level(const uint4* band, int l) {
    const ASN_K uint4* p = kp(band) + 2 * l;
    return {RT == 1 ? p[1].w : RT == 2 ? p[0].x : p[0].y, p[0].z, RT == 1 ? p[0].w >> 4 : RT == 2 ? p[0].w : p[1].z};
}
// ... and the weight of its ordinates.
__device__ __forceinline__ double band_weight(const uint4* band, int l) {
    return *reinterpret_cast<const ASN_K double*>(kp(band) + 2 * l + 1);
}

// The rounded operand of the reduced-precision contraction, x = T(s) for s = dev 2^(E - e_b)
// (BF16: hi + lo), as the FP32 number it is: a lo term ends within s's 24 bits.
template <int DT>
__device__ __forceinline__ void round_pair(float s0, float s1, float& x0, float& x1) {
    if constexpr (DT == 1) {
        const uint32_t p = pack2<1>(s0, s1), r = bf16_residual2(p, s0, s1);
        x0 = __uint_as_float(p << 16) + __uint_as_float(r << 16);
        x1 = __uint_as_float(p & 0xFFFF0000u) + __uint_as_float(r & 0xFFFF0000u);
    } else {
        x0 = (float)(_Float16)s0;
        x1 = (float)(_Float16)s1;
    }
}

// E - e_b of the operand scale of the 64 cells from c0, from the maxima of the 64-cell blocks of
// their scale block.
__device__ __forceinline__ int operand_scale(const StepArgs& a, int c0, int lane) {
    const int first = (c0 >> a.sb_log) << (a.sb_log - 6), b = first + lane;
    unsigned bits = 0u;
    if (lane < 1 << (a.sb_log - 6) && b < a.tiles_x) bits = gp(a.bmax_cur)[b];
    const float bm = __uint_as_float(wave_max_u32(bits));
    int e = 0;
    if (bm > 0.f) (void)frexpf(bm, &e);
    return __builtin_amdgcn_readfirstlane(kScaleExp - max(e, -100));
}

// The end of a 64-cell block of NW waves, each with some of the ordinates of every cell (slots:
// LDS that is free again).
template <bool LP>
__device__ __forceinline__ void finish_cells(const StepArgs& a, float* slots, int NW, int wave, int lane,
                                             int local, const float4& cf, float isov, float dv, double phacc,
                                             double ypacc, float mx, double defect, double outflow) {
    const int cell = local * kBandCells + lane;
    const bool in = cell < (int)a.C;
    // Phi^{n+1} of each cell: the waves' partials in a fixed order.  Wave 0 holds the block's
    // cells, so it takes over what finalize_kernel does for the other forms: Phi, Phi / W and
    // the mass partials.
    // Reduced precision also sums Y and turns its particle defect into the new state's pending
    // correction (the neighbours read the old one, so there are two buffers), and takes the
    // block's maximum for the next operand scale.
    double* red = reinterpret_cast<double*>(slots);
    double* redy = red + NW * kBandCells;
    red[wave * kBandCells + lane] = phacc;
    if constexpr (LP) {
        redy[wave * kBandCells + lane] = ypacc;
        const unsigned m = wave_max_u32(__float_as_uint(mx));
        if (lane == 0) reinterpret_cast<unsigned*>(redy + NW * kBandCells)[wave] = m;
    }
    lds_barrier();
    if (wave == 0) {
        double fin[4] = {0.0, 0.0, 0.0, 0.0};
        if (in) {
            double phi = red[lane];
            for (int g = 1; g < NW; ++g) phi += red[g * kBandCells + lane];
            // Phi of psi^n, in FP64; and of its stored values
            const double old = gp(a.phi64)[cell], stored = LP ? old - a.W * (double)dv : old;
            // the physical scattering's part of the collision defect, sum_q w_q bs (iso -
            // psi_q) = bs (W iso - Phi), once per cell
            defect += (double)cf.y * (a.W * (double)isov - stored);
            gp(a.iso)[cell] = (float)(phi / a.W);
            if constexpr (LP) {
                double ys = redy[lane];
                for (int g = 1; g < NW; ++g) ys += redy[g * kBandCells + lane];
                ys += a.W * (double)(isov + dv);   // sum_q w_q Y, Y = iso^ + delta + (Y^ - iso^)
                const float d = (float)(-(double)cf.z * (ys - old) / a.W);
                gp(a.delta_next)[cell] = d;
                fin[3] = a.W * (double)d;
                phi += fin[3];
            }
            gp(a.phi64)[cell] = phi;
            fin[0] = phi;
            fin[1] = (double)cf.x * phi;
            fin[2] = (double)cf.w;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) fin[k] = wave_sum(fin[k]);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) gp(a.fin_part)[4 * (size_t)local + k] = fin[k];
            if constexpr (LP) {
                const unsigned* m = reinterpret_cast<const unsigned*>(redy + NW * kBandCells);
                unsigned t = m[0];
                for (int g = 1; g < NW; ++g) t = max(t, m[g]);
                gp(a.bmax_next)[local] = t;
            }
        }
    }
    double sums[2] = {defect, outflow};
    block_sum_n<16, 2>(sums, NW, gp(a.blk_part) + 2 * (size_t)local);
}

// T: the largest block (512 threads up to 32 azimuths: the reach-3 instance then keeps its
// queue in registers).  DT: operand type of the contraction.  HS: 0 forward Euler, 1 / 2 the
// first / second pass of the Heun + minmod scheme (FP32; muscl_kernel's fluxes, so the rows hold
// two cells beyond each end and three y neighbours are loaded).
template <int RT, int T, int DT, int HS>
__global__ __launch_bounds__(T) void banded_euler_kernel(BatchArgs B) {
    constexpr int O = kBandO, ROW = band_row(HS != 0), LEFT = HS ? 2 : 1;   // LEFT: the first cell's column
    constexpr bool LP = DT != 0;
    extern __shared__ float slots[];
    int pi, local;
    if ((int)blockIdx.x < B.n) {   // the last pass's budget, one block per problem
        pi = blockIdx.x;
        const int last = HS == 2 ? B.step : B.step - 1;   // its step
        if (last < 0 || gp(B.limit)[pi] <= last) return;
        BatchArgs P = B;
        P.s_par ^= 1;
        const StepArgs a = args_of(P, pi);
        if ((int)threadIdx.x >= band_fold_threads(a.n_az)) return;
        budget_fold(a, a.tiles_x, a.tiles_x, band_fold_threads(a.n_az),
                    HS == 0 ? BUD_STEP : HS == 1 ? BUD_STAGE2 : BUD_STAGE1);
        return;
    }
    if (!locate(B, KT_SC, xcd_remap(blockIdx.x - B.n, gridDim.x - B.n), pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int A = a.n_az, NW = A / O, a0 = wave * O;
    if (wave >= NW) return;   // a Heun batch's problems may have different azimuth counts
    const int nx = a.nx, ny = a.ny, L = a.n_lev, C = (int)a.C;
    const int c0 = local * kBandCells, cell = c0 + lane;
    const bool in = cell < C;
    const ASN_K float* bcoef = kp(RT == 1 ? a.bcoef3 : RT == 2 ? a.bcoef5 : a.bcoef7);
    const ASN_K float2* bcxy = kp(a.bcxy) + a0;

    float4 cf = make_float4(0.f, 0.f, 0.f, 0.f);
    float isov = 0.f;
    if (in) {
        cf = gp(a.coef)[cell];
        isov = gp(a.iso)[cell];
    }
    // reduced precision: the pending correction of the cell, and E - e_b of its operand scale
    float dv = 0.f;
    int sc = 0;
    if constexpr (LP) {
        if (in) dv = gp(a.delta)[cell];
        sc = operand_scale(a, c0, lane);
    }
    // boundary of the lane's cell: 1 / 2 first / last column, 4 / 8 first / last row; 16 a
    // padding cell
    const int y = cell / nx, x = cell - y * nx;
    int at = in ? (x == 0 ? 1 : 0) | (x == nx - 1 ? 2 : 0) | (y == 0 ? 4 : 0) | (y == ny - 1 ? 8 : 0) : 16;
    // (Heun: 32 / 64 also where the second cell that way is a ghost)
    if (HS) at |= in ? (x <= 1 ? 32 : 0) | (x >= nx - 2 ? 64 : 0) : 0;
    const bool edge = __ballot(at != 0) != 0;
    // Memory is reached through one buffer descriptor per level, a lane's byte offset in a
    // plane and the (uniform) offset of the plane; kOOB reads 0 (the vacuum ghost).
    const uint32_t pb = (uint32_t)(a.P * 4);   // bytes of an azimuth plane
    const uint32_t lvl_bytes = (uint32_t)A * pb, s0 = (uint32_t)a0 * pb;
    const size_t lvl_floats = (size_t)A * (size_t)a.P;
    const uint32_t voff = 4u * (uint32_t)cell;
    // n_az / 4 is even, so the flow direction is the same for azimuths 0, 1 and for 2, 3 of the
    // wave (reduced precision: n_az / 16 is whole, it is the same for all four): index o / G.
    // yd, xd: the pending corrections of the upwind cells (0 for a ghost)
    constexpr int G = LP ? 4 : 2, NG = O / G;
    uint32_t dir[NG], yoff[NG], yoff2[HS ? NG : 1], ydn[HS ? NG : 1];   // Heun: also the cell
                                                                      // beyond, the downwind one
    float yd = 0.f, xd = 0.f;
#pragma unroll
    for (int h = 0; h < NG; ++h) {
        dir[h] = (uint32_t)kp(a.qi)[a0 + G * h].dir;
        const int yc = (dir[h] & 4) ? cell - nx : cell + nx;
        const bool yv = in && yc >= 0 && yc < C;
        yoff[h] = yv ? 4u * (uint32_t)yc : kOOB;
        if constexpr (HS != 0) {
            const int y2 = (dir[h] & 4) ? cell - 2 * nx : cell + 2 * nx, y1 = 2 * cell - yc;
            yoff2[h] = (in && y2 >= 0 && y2 < C) ? 4u * (uint32_t)y2 : kOOB;
            ydn[h] = (in && y1 >= 0 && y1 < C) ? 4u * (uint32_t)y1 : kOOB;
        }
        if constexpr (LP) {
            if (yv) yd = gp(a.delta)[yc];
            if (!(at & ((dir[h] & 1) ? 17 : 18))) xd = gp(a.delta)[(dir[h] & 1) ? cell - 1 : cell + 1];
        }
    }
    // lane l also fetches azimuth a0 + l % 4's upwind cell beyond the block's end, and keeps it
    // in the column before / after the cells of that row (every lane: no branch on lanes, so
    // the kernel's branches all stay scalar).  Heun: lanes of l / 4 % 4 = 1 the second cell
    // upwind, 2 the one downwind.
    const int hd = gp(a.qi)[a0 + (lane & 3)].dir;
    const int hk = HS ? (lane >> 2) & 3 : 0;
    const bool hleft = (hd & 1) ? hk != 2 : hk == 2;
    const int hcol = hleft ? (hk == 1 ? -2 : -1) : kBandCells + (hk == 1 ? 1 : 0);   // from the first cell
    const int hc = c0 + hcol;
    const uint32_t hoff = hc >= 0 ? (uint32_t)(lane & 3) * pb + 4u * (uint32_t)hc : kOOB;
    const int hrow = (a0 + (lane & 3)) * ROW + LEFT + hcol;
    const int SF = A * ROW;
    const int own = a0 * ROW + LEFT + lane;
    const int lo = (a0 == 0 ? A - O : a0 - O) * ROW + LEFT + lane;
    const int hi = (a0 + O == A ? 0 : a0 + O) * ROW + LEFT + lane;
    int xup[NG];
#pragma unroll
    for (int h = 0; h < NG; ++h) xup[h] = own + ((dir[h] & 1) ? -1 : 1);
    // (reduced precision: the rounded operands of a level follow its values)
    const int XO = LP ? SF : 0, SS = SF + XO;

    struct Entry {
        float v[O], t[O];     // value, terms but the in-scattering
    };
    float pre[O], preh;   // the next level, on its way into LDS (lanes 0 .. 3: a halo value)
    float uy[O];          // its y-upwind values
    float uy2[HS ? O : 1], dy1[HS ? O : 1], old[HS == 2 ? O : 1];   // Heun: the other two; psi^n
    auto level_rsrc = [&](const float* base) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)lvl_bytes,
                                                 kRsrcWord3);
    };
    auto load = [&](__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t plane) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, plane, 0));
    };
    auto fetch = [&](const float* base) {
        const __amdgpu_buffer_rsrc_t r = level_rsrc(base);
#pragma unroll
        for (int o = 0; o < O; ++o) pre[o] = load(r, voff, s0 + (uint32_t)o * pb);
        preh = load(r, hoff, s0);
    };
    auto put = [&](int slot) {
        float* s = slots + slot * SS;
#pragma unroll
        for (int o = 0; o < O; ++o) s[own + o * ROW] = pre[o];
        s[hrow] = preh;
        if constexpr (LP) {
            float x[O];
#pragma unroll
            for (int o = 0; o < O; o += 2)
                round_pair<DT>(ldexpf(pre[o] - isov, sc), ldexpf(pre[o + 1] - isov, sc), x[o], x[o + 1]);
#pragma unroll
            for (int o = 0; o < O; ++o) s[XO + own + o * ROW] = x[o];
        }
    };
    auto fetch_y = [&](const float* base) {
        const __amdgpu_buffer_rsrc_t r = level_rsrc(base);
#pragma unroll
        for (int o = 0; o < O; ++o) {
            uy[o] = load(r, yoff[o / G], s0 + (uint32_t)o * pb);
            if constexpr (HS != 0) {
                uy2[o] = load(r, yoff2[o / G], s0 + (uint32_t)o * pb);
                dy1[o] = load(r, ydn[o / G], s0 + (uint32_t)o * pb);
            }
        }
    };
    auto fetch_old = [&](const float* base) {   // psi^n, where the result goes
        const __amdgpu_buffer_rsrc_t r = level_rsrc(base);
#pragma unroll
        for (int o = 0; o < O; ++o) old[o] = load(r, voff, s0 + (uint32_t)o * pb);
    };

    // (level j's at j mod N, of which RT + 1 are in use at a time)
    constexpr int N = 2 * RT + 1;
    Entry q[N];
    float acc[N][O];
#pragma unroll
    for (int m = 0; m < N; ++m)
#pragma unroll
        for (int o = 0; o < O; ++o) acc[m][o] = 0.f;
    double phacc = 0.0, defect = 0.0, outflow = 0.0, ypacc = 0.0;
    float mx = 0.f;
    const float* pf = a.psi;   // planes of the level fetched next
    const float* py = a.psi;   // and of the one whose y-upwind values are
    float* po = a.psi_new;     // planes of the level finished next
    BandLevel d = band_level<RT>(a.band, 0);   // of level j
    fetch(pf);
    fetch_y(py);
    put(0);
    if (L > 1) {
        pf += lvl_floats;
        fetch(pf);
    }
    lds_barrier();

    auto pass = [&](int j, auto phase) {   // phase: j mod N
        constexpr int PJ = decltype(phase)::value;
        Entry& e = q[PJ];                   // level j
        Entry& n = q[(PJ + N - RT) % N];    // level j - RT
        BandLevel dn = d;
        // the weight of the level finished here, and its row defect
        const double w = band_weight(a.band, max(j - RT, 0));
        const float rq = LP ? kp(a.rdef)[max(j - RT, 0) * A] : 0.f;
        if (j < L) {
            const float* s = slots + (j & 1) * SS;
            float ux[O], xv[O], ux2[HS ? O : 1], dx1[HS ? O : 1];
#pragma unroll
            for (int o = 0; o < O; ++o) {
                e.v[o] = s[own + o * ROW];
                if constexpr (HS == 0) ux[o] = s[xup[o / G] + o * ROW];
            }
            s += XO;
#pragma unroll
            for (int o = 0; o < O; ++o) xv[o] = LP ? s[own + o * ROW] : e.v[o];
            const float near[4] = {s[lo + 2 * ROW], s[lo + 3 * ROW], s[hi], s[hi + ROW]};
            // the level's uniform values, in one round trip with the LDS rows
            const ASN_K float* kc = bcoef + d.coef;
            const ASN_K float* kcc = reinterpret_cast<const ASN_K float*>(bcxy + j * A);
            float k0[3 * N], cc[2 * O];
#pragma unroll
            for (int i = 0; i < 3 * N; ++i) k0[i] = kc[i];
#pragma unroll
            for (int i = 0; i < 2 * O; ++i) cc[i] = kcc[i];
            dn = band_level<RT>(a.band, min(j + 1, L - 1));
            await(k0);
            await(cc);
            asm volatile("" ::"s"(w), "s"(rq));
            scatter<RT, PJ, ROW>(acc, xv, near, k0, s + lo, s + hi, s + LEFT + lane, a0, A, d.form, d.steps, kc);
            if constexpr (HS != 0) {   // (after the convolution: registers)
#pragma unroll
                for (int o = 0; o < O; ++o) {   // xup = own -+ 1: the second cell upwind, the downwind one
                    ux[o] = s[xup[o / G] + o * ROW];
                    ux2[o] = s[2 * xup[o / G] - own + o * ROW];
                    dx1[o] = s[2 * own - xup[o / G] + o * ROW];
                }
            }
            // stream + collide without the in-scattering, one chain of FMAs:
            //   psi' = psi + [bs (iso - psi) + ss - aa psi + cy (uy - psi) + cx (ux - psi) + gs (Y - psi)]
            // (aa = dt sigma_a, bs = dt sigma_s, gs = dt sigma_as, ss = dt q); no coefficient
            // of psi is folded into a per-cell constant, whose rounding would bias every
            // ordinate of the cell alike.  A padding cell (not in) has psi = 0, zero
            // coefficients and zero upwind values, so it stays zero.  Reduced precision: psi is
            // the stored value plus the pending correction in the streaming and absorption
            // terms, the stored one in the collision (the correction is isotropic).
            if (edge) {   // ghosts along x, outflow through the faces on the boundary
                asm volatile("" : "+v"(at));   // (evaluated here, not kept in masks)
                float ob = 0.f;
#pragma unroll
                for (int o = 0; o < O; ++o) {
                    const int dx = (dir[o / G] & 1) ? 1 : 2, dy = (dir[o / G] & 4) ? 8 : 4;
                    if (at & (dx | 16)) ux[o] = 0.f;
                    float vx = e.v[o] + dv, vy = vx;   // the value on an outflow face
                    if constexpr (HS != 0) {
                        if (at & (32 * dx | 16)) ux2[o] = 0.f;
                        if (at & ((3 - dx) | 16)) dx1[o] = 0.f;
                        vx += 0.5f * minmod(vx - ux[o], dx1[o] - vx);
                        vy += 0.5f * minmod(vy - uy[o], dy1[o] - vy);
                    }
                    ob += (at & (3 - dx) ? cc[2 * o] * vx : 0.f) + (at & dy ? cc[2 * o + 1] * vy : 0.f);
                }
                outflow += band_weight(a.band, j) * (double)ob;
            }
#pragma unroll
            for (int o = 0; o < O; ++o) {
                float t = fmaf(cf.y, isov - e.v[o], cf.w);
                const float v = LP ? e.v[o] + dv : e.v[o];
                t = fmaf(-cf.x, v, t);
                if constexpr (HS != 0) {
                    // upwind flux differences with minmod-limited slopes, (v + s/2) - (u + s_u/2)
                    // with s = minmod(v - u, d - v), s_u = minmod(u - u2, v - u)
                    auto flux = [&](float u, float u2, float d1) {
                        const float g = v - u;
                        return fmaf(0.5f, minmod(g, d1 - v) - minmod(u - u2, g), g);
                    };
                    t = fmaf(-cc[2 * o + 1], flux(uy[o], uy2[o], dy1[o]), t);
                    e.t[o] = fmaf(-cc[2 * o], flux(ux[o], ux2[o], dx1[o]), t);
                    continue;
                }
                t = fmaf(cc[2 * o + 1], (LP ? uy[o] + yd : uy[o]) - v, t);
                e.t[o] = fmaf(cc[2 * o], (LP ? ux[o] + xd : ux[o]) - v, t);
            }
            if (j + 1 < L) put((j + 1) & 1);   // this slot's readers passed the last barrier
        }
        if (j >= RT) {
            // finish level j - RT (entry n); Phi takes each new value in FP64; the
            // in-scattering's sum over the outputs, gs sum (Y - psi), is formed in FP32
            // (small terms) and added once per level
            const __amdgpu_buffer_rsrc_t r = level_rsrc(po);
            po += lvl_floats;
            float sd = 0.f, ys = 0.f;
#pragma unroll
            for (int o = 0; o < O; ++o) {
                const float sum = acc[(PJ + N - RT) % N][o];
                float dy, v = n.v[o];
                if constexpr (LP) {   // Y^ - iso^ = 2^(e_b - E) sum + r_q dev, dev = psi^ - iso^
                    const float dev = v - isov, ya = fmaf(rq, dev, ldexpf(sum, -sc));
                    ys += ya;
                    dy = ya - dev;
                    v += dv;
                } else {
                    dy = sum - v;
                }
                float nv = v + fmaf(cf.z, dy, n.t[o]);
                if constexpr (HS == 2) nv = 0.5f * (old[o] + nv);
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(nv), r, voff, s0 + (uint32_t)o * pb,
                                                      kCachePolicyNT);   // read next step, not from L2
                phacc += w * (double)nv;
                sd += dy;
                if constexpr (LP) mx = fmaxf(mx, fabsf(nv));
            }
            defect += w * (double)(cf.z * sd);
            if constexpr (LP) ypacc += w * (double)ys;
        }
        if constexpr (HS == 2)
            if (j + 1 >= RT && j + 1 < L + RT) fetch_old(po);
        if (j + 1 < L) {
            py += lvl_floats;
            fetch_y(py);
        }
        if (j + 2 < L) {
            pf += lvl_floats;
            fetch(pf);
        }
        d = dn;
        lds_barrier();
    };
    for (int j = 0; j < L + RT; j += N) {
        pass(j, std::integral_constant<int, 0>{});
        if (j + 1 >= L + RT) break;
        pass(j + 1, std::integral_constant<int, 1>{});
        if (j + 2 >= L + RT) break;
        pass(j + 2, std::integral_constant<int, 2>{});
        if constexpr (N > 3) {
            if (j + 3 >= L + RT) break;
            pass(j + 3, std::integral_constant<int, 3>{});
            if (j + 4 >= L + RT) break;
            pass(j + 4, std::integral_constant<int, 4>{});
        }
        if constexpr (N > 5) {
            if (j + 5 >= L + RT) break;
            pass(j + 5, std::integral_constant<int, 5>{});
            if (j + 6 >= L + RT) break;
            pass(j + 6, std::integral_constant<int, 6>{});
        }
    }

    finish_cells<LP>(a, slots, NW, wave, lane, local, cf, isov, dv, phacc, ypacc, mx, defect, outflow);
}

// ---------------------------------------------------------------------------
// 6. The banded BF16 / FP16 step on the matrix cores (FP32 accumulate), for product sets of 32,
//    48 or 64 azimuths whose K is wide (band_on_matrix_cores, asn_host.hpp).  As in the fused reduced-precision form the state is
//    stored without its pending per-cell particle correction delta (isotropic, so it
//    drops out of the rounded deviation), and only the anisotropic part is rounded:
//      x = T((psi^ - iso^) 2^(E - e_b))  (BF16: hi + lo),
//      Y^ - iso^ = 2^(e_b - E) sum_j T(C_ij) x_j + r_q (psi^ - iso^),
//    T(C_ij) the circulant block of level pair (i, j) of the stored K.  Block =
//    kBandCells cells x every ordinate; wave (m-tile mt, n-tile nt) owns azimuths
//    16 mt .. + 15 of cells 16 nt .. + 15, lane l the four azimuths 16 mt + 4 (l / 16) ..
//    of cell 16 nt + l % 16, which is where MFMA 16x16x32 leaves them.  Per level pair
//    and k-step of 32 azimuths one MFMA per operand term: A is the block's 16 x 32 slice
//    at the wave's azimuth offset (host-built, staged in LDS a level ahead), B eight
//    consecutive azimuths of one cell of the partner level from a ring of quantised
//    levels ([8-azimuth chunk][cell], 16-byte reads).  The ring is filled from registers
//    loaded a level before; the unrounded values of the lane's own cell wait in registers
//    (reach + 1 levels) for the level's update, which runs one level behind the products
//    and is interleaved with them; x neighbours come from the adjacent lanes (DPP) or, at
//    the edges of a 16-cell tile, from a small ring the neighbouring waves (or the block's
//    halo loads) fill at the same time.  Outputs as the fused form:
//    psi^{n+1} without its correction, per cell Phi^ and sum_q w_q Y^, budget partials,
//    block maxima of the next operand scale; finalize and budget kernels follow.
//    Its time hardly depends on K's width: BF16 4 x 64, 400^2, 154 us with one level coupled and
//    205 with whole rings of three to four (294 by the tables of the kernel above), 2 x 64, dense 116
//    (152), 4 x 32, dense 122 (174), 8 x 64, 200^2, a fifth of K 106 (123); FP16 4 x 64, 400^2, dense
//    201 (385).  What bounds it: each B operand is read from LDS by n_az / 16 waves.
// ---------------------------------------------------------------------------
// (lanes at the row's edge get 0; the kernel takes their value from the edge ring)
__device__ __forceinline__ float dpp_from_left(float v) {   // lane l gets lane l - 1 (row of 16)
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x111, 0xF, 0xF, true));
}
__device__ __forceinline__ float dpp_from_right(float v) {  // lane l gets lane l + 1 (row of 16)
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x101, 0xF, 0xF, true));
}

template <int A, int DT, int R>
__global__ __launch_bounds__(band_lp_threads(A)) void banded_lp_kernel(BatchArgs B) {
    constexpr int MT = A / 16, NT = kBandCells / 16, KS = band_lp_ksteps(A), TERMS = DT == 1 ? 2 : 1;
    constexpr int NW = MT * NT, T = NW * 64;
    constexpr int KC = 4 * KS;                // 16-byte chunks of 8 azimuths a cell holds
    constexpr int NS = 2 * R + 2, NE = R + 3, NP = 2 * R + 1;
    constexpr int XSLOT = band_lp_slot(A);    // elements per ring slot and term:
                                              // [chunk][cell][8 azimuths]
    constexpr int FR = NP * MT * 64;          // uint4 of A operands (NP pair slots)
    constexpr int FRX = FR + A / 2;           // and the (cx, cy) table: uint4 per buffer
    constexpr int FSL = (2 * kBandMaxReach + 1) * MT * 64;   // uint4 of a level's slots
    constexpr int CPT = (FRX + T - 1) / T;    // uint4 staged per thread
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    uint16_t* xr = reinterpret_cast<uint16_t*>(lds_raw);
    uint4* fr = reinterpret_cast<uint4*>(lds_raw + (size_t)NS * TERMS * XSLOT * 2);
    float* edge = reinterpret_cast<float*>(lds_raw + (size_t)NS * TERMS * XSLOT * 2 + (size_t)2 * FRX * 16);
    int pi, local;
    if (!locate(B, KT_SC, xcd_remap(blockIdx.x, gridDim.x), pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mt = wave % MT, nt = wave / MT;
    const int g = lane >> 4, cl = lane & 15;
    const int a0 = 16 * mt + 4 * g;      // the lane's first azimuth
    const int cc = 16 * nt + cl;         // its cell within the block
    const int nx = a.nx, ny = a.ny, L = a.n_lev, RE = a.reach;
    const int C = (int)a.C;
    const int64_t P = a.P;
    const int cell = local * kBandCells + cc;
    const bool in = cell < C;
    const ASN_G QInfo* __restrict__ qtab = gp(a.qi);
    const ASN_K QInfo* qk = kp(a.qi);
    const ASN_K uint4* ldesc = kp(a.bpairs);
    const ASN_G uint4* __restrict__ frag = gp(a.bfrag);
    const ASN_K float* rdk = kp(a.rdef);   // r_q, the same for every ordinate of a level

    float4 cf = make_float4(0.f, 0.f, 0.f, 0.f);
    float ihv = 0.f, dv = 0.f;   // iso^ = Phi^ / W and the pending correction of the cell
    if (in) {
        cf = gp(a.coef)[cell];
        ihv = gp(a.iso)[cell];
        dv = gp(a.delta)[cell];
    }
    float s_in, s_out;   // the cell's operand scale 2^(E - e_b) and its inverse
    {
        const float bm = in ? __uint_as_float(gp(a.bmax_cur)[cell >> a.sb_log]) : 0.f;
        int e = 0;
        if (bm > 0.f) (void)frexpf(bm, &e);
        e = max(e, -100);
        s_in = ldexpf(1.f, kScaleExp - e);
        s_out = ldexpf(1.f, e - kScaleExp);
    }
    const float ivs = ihv * s_in;
    const int y = cell / nx, x = cell - y * nx;
    const int e = in ? ((x == 0 ? 1 : 0) | (x == nx - 1 ? 2 : 0) | (y == 0 ? 4 : 0) |
                        (y == ny - 1 ? 8 : 0))
                     : 0;
    const bool wedge = __ballot(e != 0) != 0;
    const uint32_t lvl_bytes = (uint32_t)(A * P * 4), pb = (uint32_t)(P * 4);
    const uint32_t off0 = 4u * (uint32_t)(a0 * P) + 4u * (uint32_t)cell;
    // the lane's four azimuths lie in one quadrant (n_az / 4 is a multiple of 4): one
    // y-upwind cell; its offsets yoff + o pb (from kOOB they stay past every plane: a
    // level holds under 2^31 bytes, and 3 pb more stays below 2^32)
    uint32_t yoff;
    float ydl;   // pending correction of the y-upwind cell
    bool tl[4], tr[4], ox[4], oy[4];
    {
        const int d = qtab[a0].dir;
        const int yc = (d & 4) ? cell - nx : cell + nx;
        const bool yv = in && yc >= 0 && yc < C;
        ydl = yv ? gp(a.delta)[yc] : 0.f;
        yoff = yv ? off0 + 4u * (uint32_t)(yc - cell) : kOOB;
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        const int d = qtab[a0 + o].dir;
        const bool gx = !in || (d & e & 3) != 0;
        tl[o] = !gx && (d & 1);
        tr[o] = !gx && !(d & 1);
        const int go = (((d & 5) << 1) | ((d & 10) >> 1)) & e;   // outflow faces of d
        ox[o] = in && (go & 3);
        oy[o] = in && (go & 12);
    }
    // the block's halo cells, one value a lane: in tile 0 lanes 0 .. 3 of each row of 16
    // read azimuth a0 + cl of the cell before the block, in the last tile lanes 12 .. 15
    // azimuth a0 + cl - 12 of the cell after it (the other lanes' halo offsets read 0)
    const bool hlo = nt == 0 && cl < 4, hhi = nt == NT - 1 && cl >= 12;
    const int hcell = hlo ? local * kBandCells - 1 : local * kBandCells + kBandCells;
    const int haz = a0 + (hlo ? cl : cl - 12);
    const bool hvalid = (hlo || hhi) && hcell >= 0 && hcell < (int)P;
    const float hdl = (hvalid && hcell < C) ? gp(a.delta)[hcell] : 0.f;
    const uint32_t hoff = hvalid ? 4u * (uint32_t)(haz * P) + 4u * (uint32_t)hcell : kOOB;
    const int hslot = hlo ? haz : (NT + NT - 1) * A + haz;   // its place in an edge slot
    const size_t lvl_floats = (size_t)A * (size_t)P;
    auto level_rsrc = [&](const float* base) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)lvl_bytes, kRsrcWord3);
    };

    struct Fill {
        float v[4], h;
    };
    auto fetch = [&](int l, Fill& f) {
        const __amdgpu_buffer_rsrc_t r = level_rsrc(a.psi + (size_t)l * lvl_floats);
#pragma unroll
        for (int o = 0; o < 4; ++o) f.v[o] = load_plane(r, off0 + (uint32_t)o * pb);
        f.h = load_plane(r, hoff);
    };
    // the lane's four azimuths of level l into the ring (rounded operand terms) and the
    // tile-edge values (true state psi^ + delta) its neighbours need
    auto put = [&](int l, const Fill& f) {
        uint16_t* xs = xr + (size_t)(l % NS) * TERMS * XSLOT + ((a0 >> 3) * kBandCells + cc) * 8 + (a0 & 7);
        float xv[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) xv[o] = __builtin_fmaf(f.v[o], s_in, -ivs);
        uint2 pk;
        pk.x = pack2<DT>(xv[0], xv[1]);
        pk.y = pack2<DT>(xv[2], xv[3]);
        *reinterpret_cast<uint2*>(xs) = pk;
        if constexpr (DT == 1) {
            uint2 pl;
            pl.x = bf16_residual2(pk.x, xv[0], xv[1]);
            pl.y = bf16_residual2(pk.y, xv[2], xv[3]);
            *reinterpret_cast<uint2*>(xs + XSLOT) = pl;
        }
        float* es = edge + (size_t)(l % NE) * 2 * NT * A;
        if (cl == 15 && nt < NT - 1) {   // the left neighbour of the next tile
            float* d = es + (nt + 1) * A + a0;
#pragma unroll
            for (int o = 0; o < 4; ++o) d[o] = f.v[o] + dv;
        }
        if (cl == 0 && nt > 0) {         // the right neighbour of the previous tile
            float* d = es + (NT + nt - 1) * A + a0;
#pragma unroll
            for (int o = 0; o < 4; ++o) d[o] = f.v[o] + dv;
        }
        if (hlo || hhi) es[hslot] = f.h + hdl;   // the block's halo
    };
    // block l of the operand table into buffer l & 1 (thread t moves uint4 t and t + T):
    // level l's A operands (2 kBandMaxReach + 1 pair slots, the coupled pairs first; the
    // kernel runs the first NP, those past a problem's pairs hold zero operands), then the
    // (cx, cy) of level l - 1's ordinates, read by the update that runs one level behind.
    // Block n_lev holds the last level's (cx, cy).
    static_assert(CPT <= 2, "at most two staged uint4 per thread");
    auto src_of = [&](int x) { return x < FR ? x : FSL + (x - FR); };
    auto fetch_frag = [&](int l, uint4& f0, uint4& f1) {
        const ASN_G uint4* src = frag + ldesc[2 * l].y;
        f0 = src[src_of(FRX >= T ? tid : min(tid, FRX - 1))];
        if constexpr (CPT > 1) f1 = src[src_of(min(tid + T, FRX - 1))];
    };
    auto put_frag = [&](int l, const uint4& f0, const uint4& f1) {
        uint4* dst = fr + (size_t)(l & 1) * FRX;
        if (FRX >= T || tid < FRX) dst[tid] = f0;
        if constexpr (CPT > 1) if (tid + T < FRX) dst[tid + T] = f1;
    };
    // the next update's inputs: the lane's own four values (from the register queue), the
    // y-upwind values and the level's r_q and weight (its (cx, cy) come from LDS)
    struct Ahead {
        float v[4], y[4];
        float rq;
        double w;
    };
    auto fetch_ahead = [&](int l, Ahead& ah) {
        const __amdgpu_buffer_rsrc_t r = level_rsrc(a.psi + (size_t)l * lvl_floats);
        const int q0 = l * A;
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            ah.y[o] = load_plane(r, yoff + (uint32_t)o * pb);
        }
        ah.rq = rdk[q0];
        ah.w = qk[q0].w;
    };

    // n_az not a multiple of 32: the last k-step reads azimuths past n_az, which the ring
    // holds at zero (the A operands' wrapped values there multiply zeros)
    if constexpr (A % 32 != 0) {
        uint4* z = reinterpret_cast<uint4*>(xr);
        constexpr int NZ = NS * TERMS * XSLOT * 2 / 16;
        for (int t = tid; t < NZ; t += T) z[t] = make_uint4(0u, 0u, 0u, 0u);
        lds_barrier();
    }
    // The level loop runs one level behind in its update: pass i contracts level i and
    // updates level i - 1 with the products of the pass before, two independent streams
    // (LDS reads and MFMA; VALU, DPP and stores) interleaved in one schedule.  The edge
    // ring is reach + 3 levels deep: a level's edges stay until its lagging update has
    // read them.
    // the lane's own unrounded values of the levels in the ring ahead of the update
    // (levels i + 1 .. i + R + 1 at the end of pass i)
    float fifo[R + 1][4];
    {   // prologue: levels 0 .. R into the ring and the queue, level 0's operands
        Fill f;
#pragma unroll
        for (int l = 0; l <= R; ++l) {
            fetch(min(l, L - 1), f);
            if (l < L) put(l, f);
#pragma unroll
            for (int o = 0; o < 4; ++o) fifo[l][o] = f.v[o];
        }
        uint4 g0, g1;
        fetch_frag(0, g0, g1);
        put_frag(0, g0, g1);
    }
    Fill pre;
    fetch(min(R + 1, L - 1), pre);
    uint4 fp0, fp1;
    fetch_frag(1, fp0, fp1);
    Ahead ah;
    lds_barrier();

    double phacc = 0.0, ypacc = 0.0, defect = 0.0, outflow = 0.0;
    float mx = 0.f;
    const int mtk0 = ((0 - mt) % MT + MT) % MT;   // fragment of k-step 0: offset (32 kt - 16 mt) mod A
    // B operand of k-step kt: chunk g + 4 kt of the lane's cell (16 lanes of a row read
    // 256 contiguous bytes)
    const uint16_t* xl = xr + (g * kBandCells + cc) * 8;
    static_assert(KC * kBandCells * 8 == XSLOT, "ring slot layout");
    static_assert(A * 256 <= NS * TERMS * XSLOT * 2, "the final partials fit in the ring");
    // level i's products: every pair slot, k-steps of 32 azimuths, operand terms
    struct Ops {
        uint4 a[KS], b[KS];
        const uint16_t* xs;
    };
    struct Pass {
        uint32_t kcodes;
        int sb;
        const uint4* fl;
    };
    auto pass_of = [&](int i) {
        Pass ps;
        ps.kcodes = ldesc[2 * i].z;
        ps.fl = fr + (size_t)(i & 1) * FRX + lane;
        // ring slot of level i - RE (k = 0); a pair's partner i - RE + k sits k slots on
        ps.sb = ((i - RE) % NS + NS) % NS;
        return ps;
    };
    // a pair's A operands and its first operand term; the second term (BF16) is read
    // into the same registers after the first term's products
    auto load_pair = [&](const Pass& ps, int p, Ops& op) {
        int sl = ps.sb + (int)((ps.kcodes >> (4 * p)) & 15u);
        sl = sl >= NS ? sl - NS : sl;
        op.xs = xl + (size_t)sl * TERMS * XSLOT;
#pragma unroll
        for (int kt = 0; kt < KS; ++kt) op.a[kt] = ps.fl[(p * MT + (mtk0 + 2 * kt) % MT) * 64];
#pragma unroll
        for (int kt = 0; kt < KS; ++kt)
            op.b[kt] = *reinterpret_cast<const uint4*>(op.xs + 4 * kBandCells * 8 * kt);
    };
    auto load_term = [&](int t, Ops& op) {
#pragma unroll
        for (int kt = 0; kt < KS; ++kt)
            op.b[kt] = *reinterpret_cast<const uint4*>(op.xs + t * XSLOT + 4 * kBandCells * 8 * kt);
    };
    auto mul_term = [&](const Ops& op, f32x4& acc) {
#pragma unroll
        for (int kt = 0; kt < KS; ++kt) acc = mfma_lp<DT>(op.a[kt], op.b[kt], acc);
    };
    auto mul_pair = [&](Ops& op, f32x4& acc) {   // (no overlap with other work)
        mul_term(op, acc);
#pragma unroll
        for (int t = 1; t < TERMS; ++t) {
            load_term(t, op);
            mul_term(op, acc);
        }
    };
    // the update of the lane's four outputs of level j (as the fused reduced-precision form):
    //   v = psi^ + delta, dev = psi^ - iso^, Y^ - iso^ = s_out acc + r_q dev
    //   col = gs ((iso^ + Y^ - iso^) - psi^) + bs (iso^ - psi^)
    //   new = v - cx (v - ux) - cy (v - uy) - aa v + col + ss
    // (the look-ahead values hold level j)
    struct Upd {
        __amdgpu_buffer_rsrc_t ro;
        const float* es;   // the level's edge slot at the lane's tile and azimuths
        const float2* cxy;   // the level's (cx, cy) at the lane's azimuths
        float colsum, yas;
        double ph;
    };
    auto upd_begin = [&](int j, Upd& u) {
        u.es = edge + (size_t)(j % NE) * 2 * NT * A + nt * A + a0;
        u.cxy = reinterpret_cast<const float2*>(fr + (size_t)((j + 1) & 1) * FRX + FR) + a0;
        u.ro = level_rsrc(a.psi_new + (size_t)j * lvl_floats);
        u.colsum = 0.f;
        u.yas = 0.f;
        u.ph = 0.0;
    };
    auto upd_out = [&](int o, const f32x4& acc, Upd& u) {
        const float vh = ah.v[o];
        const float v = vh + dv;
        // the row shifts run in every lane (a lane whose neighbour is inactive would read
        // 0), then the row's edge lanes (0 and 15) take the edge ring's value
        const float dl = dpp_from_left(v), dr = dpp_from_right(v);
        const float left = cl == 0 ? u.es[o] : dl;
        const float right = cl == 15 ? u.es[NT * A + o] : dr;
        const float ux = tl[o] ? left : (tr[o] ? right : 0.f);
        const float uy = ah.y[o] + ydl;
        const float dev = vh - ihv;
        const float ya = s_out * acc[o] + ah.rq * dev;
        const float col = cf.z * ((ihv + ya) - vh) + cf.y * (ihv - vh);
        // a padding cell (not in) has psi^ = delta = iso^ = 0, zero coefficients, zero
        // operands and ghosts: its update is 0 without a select
        const float2 c = u.cxy[o];
        const float nv = v - c.x * (v - ux) - c.y * (v - uy) - cf.x * v + col + cf.w;
        // a wave writes half of each 128-byte line, a sibling wave the other half: the L2
        // joins them (non-temporal stores wrote 1.4x the bytes)
        store_plane(nv, u.ro, off0 + (uint32_t)o * pb);
        u.ph += (double)nv;
        u.yas += ya;
        u.colsum += col;
        mx = fmaxf(mx, fabsf(nv));
    };
    auto upd_end = [&](const Upd& u) {
        phacc += ah.w * u.ph;
        // sum over the four outputs of Y^ = iso^ + delta + (Y^ - iso^); the deviations,
        // small against iso^, summed in FP32
        ypacc += ah.w * ((in ? 4.0 * (double)(ihv + dv) : 0.0) + (double)u.yas);
        defect += ah.w * (double)u.colsum;
    };
    // the outflow of the level just updated (the look-ahead values still hold it)
    auto outflow_of = [&](const Upd& u) {
        if (wedge) {
            float ob = 0.f;
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const float v = ah.v[o] + dv;
                const float2 c = u.cxy[o];
                ob += (ox[o] ? c.x * v : 0.f) + (oy[o] ? c.y * v : 0.f);
            }
            outflow += ah.w * (double)ob;
        }
    };
    // the end of pass i: level i + R + 1 goes into the ring slot level i - R - 1 held and
    // the queue, level i leaves the queue for the next pass's update, loads for the next
    // passes
    auto advance = [&](int i) {
        if (i + R + 1 < L) put(i + R + 1, pre);
        fetch_ahead(i, ah);
#pragma unroll
        for (int o = 0; o < 4; ++o) ah.v[o] = fifo[0][o];
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int o = 0; o < 4; ++o) fifo[q][o] = fifo[q + 1][o];
#pragma unroll
        for (int o = 0; o < 4; ++o) fifo[R][o] = pre.v[o];
        fetch(min(i + R + 2, L - 1), pre);
        lds_barrier();
    };

    f32x4 accp = {0.f, 0.f, 0.f, 0.f};
    {   // pass 0: products only
        put_frag(1, fp0, fp1);
        fetch_frag(min(2, L), fp0, fp1);
        const Pass ps = pass_of(0);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            Ops op;
            load_pair(ps, p, op);
            mul_pair(op, accp);
        }
        advance(0);
    }
    for (int i = 1; i < L; ++i) {
        // block i + 1 of the operand table (its buffer's last readers passed the barrier)
        put_frag(i + 1, fp0, fp1);
        fetch_frag(min(i + 2, L), fp0, fp1);
        // pass i in chunks the scheduler may not merge: chunk p reads pair p's operands,
        // updates output p of level i - 1 while they arrive, then multiplies pair p (the
        // MFMAs run on while the next chunk issues)
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        const Pass ps = pass_of(i);
        Upd u;
        upd_begin(i - 1, u);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            __builtin_amdgcn_sched_barrier(0);
            Ops op;
            load_pair(ps, p, op);
            if (p < 4) upd_out(p, accp, u);
            mul_term(op, acc);
#pragma unroll
            for (int t = 1; t < TERMS; ++t) {
                load_term(t, op);
                mul_term(op, acc);
            }
        }
#pragma unroll
        for (int o = NP; o < 4; ++o) upd_out(o, accp, u);
        __builtin_amdgcn_sched_barrier(0);
        upd_end(u);
        accp = acc;
        outflow_of(u);
        advance(i);
    }
    {
        Upd u;
        upd_begin(L - 1, u);
#pragma unroll
        for (int o = 0; o < 4; ++o) upd_out(o, accp, u);
        upd_end(u);
        outflow_of(u);
    }

    // per cell Phi^ and sum_q w_q Y^: the (n_az / 4) lane groups' partials in a fixed order
    double* red = reinterpret_cast<double*>(lds_raw);
    red[(4 * mt + g) * kBandCells + cc] = phacc;
    red[(A / 4 + 4 * mt + g) * kBandCells + cc] = ypacc;
    lds_barrier();
    if (tid < kBandCells) {
        const int c = local * kBandCells + tid;
        if (c < C) {
            double s = red[tid], sy = red[(A / 4) * kBandCells + tid];
#pragma unroll
            for (int k = 1; k < A / 4; ++k) {
                s += red[k * kBandCells + tid];
                sy += red[(A / 4 + k) * kBandCells + tid];
            }
            gp(a.phi_part)[c] = s;
            gp(a.ypart)[c] = sy;
        }
    }
    // block max |psi^{n+1}| of the next operand scale: the block's cells lie in one block
    const unsigned mbits = wave_max_u32(__float_as_uint(mx));
    if (lane == 0 && mbits) atomicMax(&a.bmax_next[(local * kBandCells) >> a.sb_log], mbits);
    double sums[2] = {defect, outflow};
    block_sum_waves<NW, 2>(sums, gp(a.blk_part) + 2 * (size_t)local);
}

// ---------------------------------------------------------------------------
// 7. Step for any ordinate set whose K is sparse and whose values at 64 cells fit LDS
//    (forward Euler; FP32 Heun).
//    A K with 13 % nonzeros (162 ordinates of the icosahedron: 21 a row) leaves the matrix cores
//    nearly all zeros whatever the tile, and few ordinates leave most of a 128-row tile empty.
//    Block = kBandCells consecutive cells x every ordinate, all their values (reduced precision:
//    rounded operands) in LDS; a wave takes groups of kBandO ordinates that share most of their
//    sources (sparse_form: 32 for those four) and multiplies the union of their rows' nonzeros:
//    an LDS value serves four outputs, coefficients are scalar.  The neighbours' values are loaded
//    beside the products, from L2.  The rest of the step as in the banded kernel.
//    What bounds it: 280^2 x 162 takes 46 us (2.2 TB/s on 8 B per update); without the products
//    26 us, without scalar misses the products alone would be 21 us of VALU issue.  The two
//    overlap only between a CU's blocks (three at 162 ordinates), which start together.  A chunk
//    of eight sources a trip to the scalar tables instead of four: 55 -> 47 us; ten waves a block
//    59 (the tables' 35 KB outrun the scalar cache sooner); neighbours or a group's constants
//    fetched a group ahead: no gain; halo columns in LDS instead of loads: 58, and reduced
//    precision 42 -> 33 us with the LDS that saves.  Against a contraction over 128 x 128 tiles
//    with the step in its epilogue, us a step: 280^2 x 162 FP32 117 -> 46, BF16 108 -> 50;
//    50^2 x 12 25 -> 4.5; 400^2 x 492 505 -> 322, BF16 442 -> 329; 200^2 x 128 (16 azimuths) BF16
//    52 -> 27; Heun 280^2 x 162 217 -> 95.
// ---------------------------------------------------------------------------
template <int DT, int HS, int T>
__global__ __launch_bounds__(T, T == 512 ? 6 : 4) void sparse_step_kernel(BatchArgs B) {
    constexpr int O = kBandO, ROW = kBandCells, NW = T / 64;
    constexpr bool LP = DT != 0;
    extern __shared__ float slots[];
    int pi, local;
    if ((int)blockIdx.x < B.n) {   // the last pass's budget, one block per problem
        pi = blockIdx.x;
        const int last = HS == 2 ? B.step : B.step - 1;   // its step
        if (last < 0 || gp(B.limit)[pi] <= last) return;
        BatchArgs P = B;
        P.s_par ^= 1;
        const StepArgs a = args_of(P, pi);
        budget_fold<1>(a, a.tiles_x, a.tiles_x, T,
                       HS == 0 ? BUD_STEP : HS == 1 ? BUD_STAGE2 : BUD_STAGE1);
        return;
    }
    if (!locate(B, KT_SC, xcd_remap(blockIdx.x - B.n, gridDim.x - B.n), pi, local)) return;
    const StepArgs a = args_of(B, pi);   // by value: no reloads after stores
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nx = a.nx, ny = a.ny, Q = a.Q, C = (int)a.C;
    const int c0 = local * kBandCells, cell = c0 + lane;
    const bool in = cell < C;

    float4 cf = make_float4(0.f, 0.f, 0.f, 0.f);
    float isov = 0.f;
    if (in) {
        cf = gp(a.coef)[cell];
        isov = gp(a.iso)[cell];
    }
    // 1 / 2 first / last column, 4 / 8 first / last row; 16 a padding cell
    const int y = cell / nx, x = cell - y * nx;
    int at = in ? (x == 0 ? 1 : 0) | (x == nx - 1 ? 2 : 0) | (y == 0 ? 4 : 0) | (y == ny - 1 ? 8 : 0) : 16;
    const bool edge = __ballot(at != 0) != 0;
    // reduced precision: the pending corrections of the cell and its four neighbours (0 for a
    // ghost), the operand scale
    float dv = 0.f, dl = 0.f, dr = 0.f, dd = 0.f, du = 0.f;
    int sc = 0;
    if constexpr (LP) {
        if (in) {
            const float* dp = a.delta + cell;
            dv = gp(dp)[0];
            if (!(at & 1)) dl = gp(dp)[-1];
            if (!(at & 2)) dr = gp(dp)[1];
            if (!(at & 4)) dd = gp(dp)[-nx];
            if (!(at & 8)) du = gp(dp)[nx];
        }
        sc = operand_scale(a, c0, lane);
    }
    // one buffer descriptor per plane; kOOB reads 0 (the vacuum ghost)
    const uint32_t voff = 4u * (uint32_t)cell;
    auto plane = [&](const float* base, int q) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + (size_t)q * (size_t)a.P), 0,
                                                 (int)(uint32_t)(a.P * 4), kRsrcWord3);
    };
    auto load = [&](__amdgpu_buffer_rsrc_t r, uint32_t off) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    };
    // byte offsets in a plane of the cells 1 (and for Heun 2) columns and rows away
    auto x_off = [&](int d) { return in && x + d >= 0 && x + d < nx ? voff + 4u * (uint32_t)d : kOOB; };
    auto y_off = [&](int d) {
        return in && y + d >= 0 && y + d < ny ? voff + 4u * (uint32_t)(d * nx) : kOOB;
    };
    const uint32_t x_m = x_off(-1), x_p = x_off(1), x_mm = HS ? x_off(-2) : 0u, x_pp = HS ? x_off(2) : 0u;
    const uint32_t y_m = y_off(-1), y_p = y_off(1), y_mm = HS ? y_off(-2) : 0u, y_pp = HS ? y_off(2) : 0u;

    // the block's values, straight into LDS, all in flight; reduced precision: through registers,
    // the rounded operands
    if constexpr (LP) {
        constexpr int U = 16;
        for (int q0 = wave; q0 < Q; q0 += U * NW) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = load(plane(a.psi, min(q0 + u * NW, Q - 1)), voff);
#pragma unroll
            for (int u = 0; u < U; u += 2) {
                float x0, x1;
                round_pair<DT>(ldexpf(v[u] - isov, sc), ldexpf(v[u + 1] - isov, sc), x0, x1);
                const int q = q0 + u * NW;
                if (q < Q) slots[q * ROW + lane] = x0;
                if (q + NW < Q) slots[(q + NW) * ROW + lane] = x1;
            }
        }
    } else {
        using Lds = __attribute__((address_space(3))) void;
        for (int q = wave; q < Q; q += NW)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(plane(a.psi, q), (Lds*)(slots + q * ROW), 4, voff, 0, 0, 0);
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    }
    lds_barrier();

    double phacc = 0.0, defect = 0.0, outflow = 0.0, ypacc = 0.0;
    float mx = 0.f;
    const int groups = (Q + O - 1) / O;
    for (int g = wave; g < groups; g += NW) {
        const ASN_K SparseGroup* d = kp(a.sp_group) + g;
        uint32_t od[O];
#pragma unroll
        for (int o = 0; o < O; ++o) od[o] = d->ord[o];   // ordinate << 4 | its direction bits
        // its own value (FP32: in LDS) and its neighbours' (Heun: the second ones upwind, the ones
        // downwind; psi^n)
        float v0[O], ux[O], uy[O], ux2[HS ? O : 1], uy2[HS ? O : 1], dx1[HS ? O : 1], dy1[HS ? O : 1],
            old[HS == 2 ? O : 1];
#pragma unroll
        for (int o = 0; o < O; ++o) {
            const int q = (int)(od[o] >> 4);
            const __amdgpu_buffer_rsrc_t r = plane(a.psi, q);
            if constexpr (LP) v0[o] = load(r, voff);
            ux[o] = load(r, od[o] & 1 ? x_m : x_p);
            uy[o] = load(r, od[o] & 4 ? y_m : y_p);
            if constexpr (HS != 0) {
                ux2[o] = load(r, od[o] & 1 ? x_mm : x_pp);
                dx1[o] = load(r, od[o] & 1 ? x_p : x_m);
                uy2[o] = load(r, od[o] & 4 ? y_mm : y_pp);
                dy1[o] = load(r, od[o] & 4 ? y_p : y_m);
            }
            if constexpr (HS == 2) old[o] = load(plane(a.psi_new, q), voff);
            if constexpr (!LP) v0[o] = slots[q * ROW + lane];
        }
        float acc[O];
#pragma unroll
        for (int o = 0; o < O; ++o) acc[o] = 0.f;
        constexpr int S = kSparseChunk;
        const char* lds = reinterpret_cast<const char*>(slots + lane);
        // The coefficients of all groups are more than the scalar cache holds, and scalar loads return
        // in no order, so each chunk waits for one trip to L2: chunks of as many coefficients as
        // there are registers, and the next chunk's row offsets with them.
        const ASN_K uint32_t* rp = kp(a.sp_row) + S * d->first;
        const ASN_K float* kc = kp(a.sp_coef) + S * O * d->first;
        uint32_t row[S];
#pragma unroll
        for (int i = 0; i < S; ++i) row[i] = rp[i];
        for (int c = d->chunks; c > 0; --c) {
            float v[S], k[S * O];
#pragma unroll
            for (int i = 0; i < S * O; ++i) k[i] = kc[i];
#pragma unroll
            for (int i = 0; i < S; ++i) v[i] = *reinterpret_cast<const float*>(lds + row[i]);
            kc += S * O;
            rp += S;
#pragma unroll
            for (int i = 0; i < S; ++i) row[i] = rp[i];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < S; ++i)
#pragma unroll
                for (int o = 0; o < O; ++o) acc[o] = fmaf(k[i * O + o], v[i], acc[o]);
            asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));
#pragma unroll
            for (int i = 0; i < S; ++i) asm volatile("" : "+s"(row[i]));   // (a value, not a load to move)
        }
        float cx[O], cy[O], rq[O];
        double w[O];   // (0 where the last group repeats an ordinate)
#pragma unroll
        for (int o = 0; o < O; ++o) {
            const ASN_K SparseOrdinate* t = kp(a.sp_ord) + (O * g + o);
            cx[o] = t->cx;
            cy[o] = t->cy;
            rq[o] = t->rdef;
            w[o] = t->w;
        }
#pragma unroll
        for (int o = 0; o < O; ++o) {
            const int q = (int)(od[o] >> 4), right = od[o] & 1, up = od[o] & 4;
            const float v = v0[o] + dv;
            if (edge) {   // outflow through the faces on the boundary
                float vx = v, vy = v;   // the value there
                if constexpr (HS != 0) {
                    vx += 0.5f * minmod(v - ux[o], dx1[o] - v);
                    vy += 0.5f * minmod(v - uy[o], dy1[o] - v);
                }
                outflow += w[o] * (double)((at & (right ? 2 : 1) ? cx[o] * vx : 0.f) + (at & (up ? 8 : 4) ? cy[o] * vy : 0.f));
            }
            // the banded kernel's chain
            float t1 = fmaf(cf.y, isov - v0[o], cf.w);
            t1 = fmaf(-cf.x, v, t1);
            if constexpr (HS != 0) {
                auto flux = [&](float u, float u2, float d1) {
                    const float gr = v - u;
                    return fmaf(0.5f, minmod(gr, d1 - v) - minmod(u - u2, gr), gr);
                };
                t1 = fmaf(-cy[o], flux(uy[o], uy2[o], dy1[o]), t1);
                t1 = fmaf(-cx[o], flux(ux[o], ux2[o], dx1[o]), t1);
            } else if constexpr (LP) {
                t1 = fmaf(cy[o], uy[o] + (up ? dd : du) - v, t1);
                t1 = fmaf(cx[o], ux[o] + (right ? dl : dr) - v, t1);
            } else {
                t1 = fmaf(cy[o], uy[o] - v, t1);
                t1 = fmaf(cx[o], ux[o] - v, t1);
            }
            float dy;
            if constexpr (LP) {   // Y^ - iso^ = 2^(e_b - E) sum + r_q dev, dev = psi^ - iso^
                const float dev = v0[o] - isov, ya = fmaf(rq[o], dev, ldexpf(acc[o], -sc));
                ypacc += w[o] * (double)ya;
                dy = ya - dev;
            } else {
                dy = acc[o] - v0[o];
            }
            float nv = v + fmaf(cf.z, dy, t1);
            if constexpr (HS == 2) nv = 0.5f * (old[o] + nv);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(nv), plane(a.psi_new, q), voff, 0, 0);
            phacc += w[o] * (double)nv;
            defect += w[o] * (double)(cf.z * dy);
            if constexpr (LP) mx = fmaxf(mx, fabsf(nv));
        }
    }
    lds_barrier();
    finish_cells<LP>(a, slots, NW, wave, lane, local, cf, isov, dv, phacc, ypacc, mx, defect, outflow);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static inline unsigned div_up(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

void blocks_per_kind(const StepArgs& a, int out[KT_COUNT]) {
    const bool banded = a.band != nullptr || a.bfrag != nullptr;
    out[KT_GEMM] = banded ? 0 : (a.Qp / kGemmBM) * (int)(a.P / kGemmBN);
    out[KT_FIX] = (a.dtype != 0 && !a.fused) ? a.fin_blocks : 0;
    out[KT_SC] = (a.fused && !banded) ? 0 : a.tiles_x * a.tiles_y * a.G;
    out[KT_FIN] = a.fin_blocks;
}

// One launch per step: each block finishes its cells' moments, and the fold of a step's budget
// partials, which nothing in the next step waits for, runs in n more blocks of that step's
// launch (the partials alternate with the state buffers; the call's last fold is a launch of
// its own, launch_last_budget).  With finalize_kernel and budget_kernel after every step
// 24 steps of 50^2 x 128, set-up and results included, took 726 us instead of 516, 40 steps of
// 311 x 173 x 288 3.13 ms instead of 2.76, a step of 400^2 x 512 187 us instead of 175.
// (f takes the instance: its kernel, and its name as a profiler prints it)
template <int RT, int T, int DT, int HS>
struct BandedInstance {
    static constexpr auto kernel = banded_euler_kernel<RT, T, DT, HS>;
    static void name(char* out, size_t n) { std::snprintf(out, n, "banded_euler_kernel<%d, %d, %d, %d>", RT, T, DT, HS); }
};
template <typename F>
static hipError_t with_banded(int az, int dtype, int reach, int heun, F&& f) {
    const bool small = az <= 32;   // at most 512 threads
    if (reach < 0 || !band_supported(az, dtype, reach, heun != 0)) return hipErrorInvalidValue;
    // FP32: the instance for reach 2 also serves smaller reaches (zero coefficients)
    if (heun == 1) return f(BandedInstance<2, 1024, 0, 1>{});
    if (heun == 2) return f(BandedInstance<2, 1024, 0, 2>{});
    if (dtype == 0) {
        if (reach <= 2) return f(BandedInstance<2, 1024, 0, 0>{});
        return small ? f(BandedInstance<3, 512, 0, 0>{}) : f(BandedInstance<3, 1024, 0, 0>{});
    }
    if (dtype == 1) {
        if (reach <= 1) return f(BandedInstance<1, 1024, 1, 0>{});
        return reach == 2 ? f(BandedInstance<2, 1024, 1, 0>{}) : f(BandedInstance<3, 512, 1, 0>{});
    }
    if (reach <= 1) return f(BandedInstance<1, 1024, 2, 0>{});
    if (reach == 2) return f(BandedInstance<2, 1024, 2, 0>{});
    return small ? f(BandedInstance<3, 512, 2, 0>{}) : f(BandedInstance<3, 1024, 2, 0>{});
}

// The same of the banded step on the matrix cores.
template <int A, int DT, int R>
struct BandedLpInstance {
    static constexpr auto kernel = banded_lp_kernel<A, DT, R>;
    static void name(char* out, size_t n) { std::snprintf(out, n, "banded_lp_kernel<%d, %d, %d>", A, DT, R); }
};
template <int A, int DT, typename F>
static hipError_t with_banded_lp_a(int reach, F&& f) {
    if (reach < 0 || !band_supported(A, DT, reach, false)) return hipErrorInvalidValue;
    if (reach == 0) return f(BandedLpInstance<A, DT, 0>{});
    if (reach == 1) return f(BandedLpInstance<A, DT, 1>{});
    if (reach == 2) return f(BandedLpInstance<A, DT, 2>{});
    if constexpr (DT == 2 || A == 32) return f(BandedLpInstance<A, DT, 3>{});
    return hipErrorInvalidValue;
}
template <typename F>
static hipError_t with_banded_lp(int az, int dtype, int reach, F&& f) {
    if (az == 32) return dtype == 1 ? with_banded_lp_a<32, 1>(reach, f) : with_banded_lp_a<32, 2>(reach, f);
    if (az == 48) return dtype == 1 ? with_banded_lp_a<48, 1>(reach, f) : with_banded_lp_a<48, 2>(reach, f);
    if (az == 64) return dtype == 1 ? with_banded_lp_a<64, 1>(reach, f) : with_banded_lp_a<64, 2>(reach, f);
    return hipErrorInvalidValue;
}
static hipError_t launch_banded_lp(const BatchArgs& b, int blocks, int az, int dtype, hipStream_t s, int reach) {
    return with_banded_lp(az, dtype, reach, [&](auto i) {
        i.kernel<<<blocks, band_lp_threads(az), band_lp_lds_bytes(az, reach, dtype), s>>>(b);
        return hipSuccess;
    });
}
hipError_t prepare_banded_lp(int az, int dtype, int reach) {
    return with_banded_lp(az, dtype, reach, [&](auto i) {
        return hipFuncSetAttribute((const void*)i.kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)band_lp_lds_bytes(az, reach, dtype));
    });
}

// heun: 0, or the pass.
static hipError_t launch_banded(const BatchArgs& b, int blocks, int az, int dtype, size_t lds, hipStream_t s,
                                int reach, int heun) {
    return with_banded(az, dtype, reach, heun, [&](auto i) {
        i.kernel<<<blocks + b.n, az / kBandO * 64, lds, s>>>(b);
        return hipSuccess;
    });
}

hipError_t prepare_banded(int az, int dtype, int reach, bool heun) {
    const size_t lds = band_lds_bytes(kBandMaxAzim, dtype, heun);
    hipError_t e = hipSuccess;
    for (int pass = heun ? 1 : 0; pass <= (heun ? 2 : 0) && e == hipSuccess; ++pass)
        e = with_banded(az, dtype, reach, pass, [&](auto i) {
            return hipFuncSetAttribute((const void*)i.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        });
    return e;
}

template <int DT, int HS, int T>
struct SparseInstance {
    static constexpr auto kernel = sparse_step_kernel<DT, HS, T>;
    static void name(char* out, size_t n) { std::snprintf(out, n, "sparse_step_kernel<%d, %d, %d>", DT, HS, T); }
};
template <int T, typename F>
static hipError_t with_sparse_t(int dtype, int heun, F&& f) {
    if (heun == 1) return f(SparseInstance<0, 1, T>{});
    if (heun == 2) return f(SparseInstance<0, 2, T>{});
    if (dtype == 0) return f(SparseInstance<0, 0, T>{});
    return dtype == 1 ? f(SparseInstance<1, 0, T>{}) : f(SparseInstance<2, 0, T>{});
}
template <typename F>
static hipError_t with_sparse(int waves, int dtype, int heun, F&& f) {
    return waves == 8 ? with_sparse_t<512>(dtype, heun, f) : with_sparse_t<1024>(dtype, heun, f);
}

static hipError_t launch_sparse(const BatchArgs& b, int blocks, int waves, int dtype, size_t lds, hipStream_t s,
                                int heun) {
    return with_sparse(waves, dtype, heun, [&](auto i) {
        i.kernel<<<blocks + b.n, waves * 64, lds, s>>>(b);
        return hipSuccess;
    });
}

hipError_t prepare_sparse(int waves, int dtype, bool heun) {
    hipError_t e = hipSuccess;
    for (int pass = heun ? 1 : 0; pass <= (heun ? 2 : 0) && e == hipSuccess; ++pass)
        e = with_sparse(waves, dtype, pass, [&](auto i) {
            return hipFuncSetAttribute((const void*)i.kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(kLds - kSparseSums));
        });
    return e;
}

// Stencil kinds of a pass: 0 donor-cell strips, 1 / 2 Heun stages (strips), 3 donor-cell
// flat chunks, 4 / 5 Heun stages (flat chunks), kStencilBanded the banded Euler step and + 1,
// + 2 the banded Heun passes (contraction and stencil in one kernel), kStencilSparse likewise,
// kStencilBandedLp the banded step on the matrix cores (in one kernel too, then finalize and budget).
constexpr int kStencilBanded = 16, kStencilSparse = 32, kStencilBandedLp = 64;

// One pass: contraction, stencil, finalize, budget.
static hipError_t launch_pass(const BatchArgs& b, const int* grid, int dtype, int stencil,
                              int bud, hipStream_t s, hipEvent_t* ev, int band_az = 0,
                              size_t band_lds = 0, int band_reach = 0) {
    hipError_t e = hipSuccess;
    auto mark = [&](int k) {
        if (ev && e == hipSuccess) e = hipEventRecord(ev[k], s);
    };
    if (stencil == kStencilBandedLp) {
        mark(0);
        e = launch_banded_lp(b, grid[KT_SC], band_az, dtype, s, band_reach);
        mark(1);
        mark(2);
        if (e == hipSuccess) finalize_kernel<<<grid[KT_FIN], 256, 0, s>>>(b, 0);
        mark(3);
        if (e == hipSuccess) budget_kernel<<<b.n, kBudgetThreads, 0, s>>>(b, bud, false);
        mark(4);
        return e != hipSuccess ? e : hipGetLastError();
    }
    if (stencil >= kStencilBanded) {   // contraction and stencil in one kernel
        mark(0);
        e = stencil >= kStencilSparse
                ? launch_sparse(b, grid[KT_SC], band_az / kBandO, dtype, band_lds, s, stencil - kStencilSparse)
                : launch_banded(b, grid[KT_SC], band_az, dtype, band_lds, s, band_reach, stencil - kStencilBanded);
        for (int k = 1; k < 5; ++k) mark(k);
        if (e != hipSuccess) return e;
        return hipGetLastError();
    }
    // a batch whose stencil grid is empty runs the stencil inside the contraction
    const bool fused = grid[KT_SC] == 0;
    mark(0);
    if (dtype == 0 && fused)
        gemm_f32_kernel<true><<<grid[KT_GEMM], 256, 0, s>>>(b);
    else if (dtype == 0)
        gemm_f32_kernel<false><<<grid[KT_GEMM], 256, 0, s>>>(b);
    else if (dtype == 1 && fused)
        gemm_lp_kernel<1, true><<<grid[KT_GEMM], 256, 0, s>>>(b);
    else if (dtype == 1)
        gemm_lp_kernel<1, false><<<grid[KT_GEMM], 256, 0, s>>>(b);
    else if (fused)
        gemm_lp_kernel<2, true><<<grid[KT_GEMM], 256, 0, s>>>(b);
    else
        gemm_lp_kernel<2, false><<<grid[KT_GEMM], 256, 0, s>>>(b);
    if (dtype != 0 && !fused) particle_fix_kernel<<<grid[KT_FIX], 256, 0, s>>>(b);
    mark(1);
    const bool lp = dtype != 0;
    if (!fused && stencil == 0) {
        if (lp) stream_collide_kernel<true><<<grid[KT_SC], 256, 0, s>>>(b);
        else stream_collide_kernel<false><<<grid[KT_SC], 256, 0, s>>>(b);
    } else if (!fused && stencil == 3) {
        if (lp) stream_collide_flat_kernel<true><<<grid[KT_SC], kFlatThreads, 0, s>>>(b);
        else stream_collide_flat_kernel<false><<<grid[KT_SC], kFlatThreads, 0, s>>>(b);
    } else if (!fused && stencil == 1) {
        if (lp) muscl_kernel<true, 1><<<grid[KT_SC], 256, 0, s>>>(b);
        else muscl_kernel<false, 1><<<grid[KT_SC], 256, 0, s>>>(b);
    } else if (!fused && stencil == 2) {
        if (lp) muscl_kernel<true, 2><<<grid[KT_SC], 256, 0, s>>>(b);
        else muscl_kernel<false, 2><<<grid[KT_SC], 256, 0, s>>>(b);
    } else if (!fused && stencil == 4) {
        if (lp) muscl_flat_kernel<true, 1><<<grid[KT_SC], kFlatThreads, 0, s>>>(b);
        else muscl_flat_kernel<false, 1><<<grid[KT_SC], kFlatThreads, 0, s>>>(b);
    } else if (!fused && stencil == 5) {
        if (lp) muscl_flat_kernel<true, 2><<<grid[KT_SC], kFlatThreads, 0, s>>>(b);
        else muscl_flat_kernel<false, 2><<<grid[KT_SC], kFlatThreads, 0, s>>>(b);
    }
    mark(2);
    finalize_kernel<<<grid[KT_FIN], 256, 0, s>>>(b, 0);
    mark(3);
    budget_kernel<<<b.n, kBudgetThreads, 0, s>>>(b, bud, false);
    mark(4);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

hipError_t launch_step(const BatchArgs& b, const int* grid, int dtype, int scheme, hipStream_t s,
                       hipEvent_t* ev, int band_az, size_t band_lds, int band_reach) {
    if (scheme == SCHEME_EULER_BANDED || scheme == SCHEME_EULER_SPARSE)
        return launch_pass(b, grid, dtype, scheme == SCHEME_EULER_SPARSE ? kStencilSparse : kStencilBanded,
                           BUD_STEP, s, ev, band_az, band_lds, band_reach);
    if (scheme == SCHEME_EULER_BANDED_LP)
        return launch_pass(b, grid, dtype, kStencilBandedLp, BUD_STEP, s, ev, band_az, band_lds, band_reach);
    if (passes_per_step(scheme) == 1)
        return launch_pass(b, grid, dtype, scheme == SCHEME_EULER_FLAT ? 3 : 0, BUD_STEP, s, ev);
    // stencil of the first pass
    const int st = scheme == SCHEME_HEUN_BANDED   ? kStencilBanded + 1
                   : scheme == SCHEME_HEUN_SPARSE ? kStencilSparse + 1
                   : scheme == SCHEME_HEUN_FLAT   ? 4
                                                  : 1;
    BatchArgs b1 = b;
    b1.s_par = 0;
    hipError_t e = launch_pass(b1, grid, dtype, st, BUD_STAGE1, s, ev, band_az, band_lds, band_reach);
    if (e != hipSuccess) return e;
    b1.s_par = 1;
    return launch_pass(b1, grid, dtype, st + 1, BUD_STAGE2, s, ev ? ev + 5 : nullptr, band_az, band_lds, band_reach);
}

void contraction_kernel(int dtype, int scheme, bool fused, int band_az, int band_reach, char* out, size_t n) {
    const int heun = passes_per_step(scheme) == 2 ? 1 : 0;
    auto name = [&](auto i) {
        i.name(out, n);
        return hipSuccess;
    };
    if (scheme == SCHEME_EULER_BANDED || scheme == SCHEME_HEUN_BANDED)
        (void)with_banded(band_az, dtype, band_reach, heun, name);
    else if (scheme == SCHEME_EULER_BANDED_LP)
        (void)with_banded_lp(band_az, dtype, band_reach, name);
    else if (scheme == SCHEME_EULER_SPARSE || scheme == SCHEME_HEUN_SPARSE)
        (void)with_sparse(band_az / kBandO, dtype, heun, name);
    else if (dtype == 0)
        std::snprintf(out, n, "gemm_f32_kernel<%s>", fused ? "true" : "false");
    else
        std::snprintf(out, n, "gemm_lp_kernel<%d, %s>", dtype, fused ? "true" : "false");
}

hipError_t launch_last_budget(const BatchArgs& b, int n_steps, int scheme, hipStream_t s) {
    if (scheme < SCHEME_EULER_BANDED || scheme == SCHEME_EULER_BANDED_LP || n_steps < 1) return hipSuccess;
    const bool heun = passes_per_step(scheme) == 2;
    BatchArgs l = b;
    l.step = n_steps - 1;
    l.s_par = heun ? 1 : l.step & 1;
    budget_kernel<<<l.n, kBudgetThreads, 0, s>>>(l, heun ? BUD_STAGE2 : BUD_STEP, true);
    return hipGetLastError();
}

__global__ void arm_kernel(int* limit, int* base, int n, ArmArgs v) {
    const int i = threadIdx.x;
    if (i < n) {
        limit[i] = v.limit[i];
        base[i] = v.cur[i];
    }
}

hipError_t launch_arm(int* limit, int* base, int n, const ArmArgs& v, hipStream_t s) {
    if (n < 1 || n > kMaxArm) return hipErrorInvalidValue;
    arm_kernel<<<1, kMaxArm, 0, s>>>(limit, base, n, v);
    return hipGetLastError();
}

hipError_t launch_init(const StepArgs& a, const BatchArgs& one, hipStream_t s, const float* cell) {
    const int64_t nb = scale_blocks(a.P, a.band ? 6 : a.sb_log);
    fill_u32_kernel<<<div_up(nb, 256), 256, 0, s>>>(a.bmax_cur, nb, 0u);
    fill_u32_kernel<<<div_up(nb, 256), 256, 0, s>>>(a.bmax_next, nb, 0u);
    moments_kernel<<<div_up(a.C, 256), 256, 0, s>>>(a, cell);
    finalize_kernel<<<a.fin_blocks, 256, 0, s>>>(one, 1);
    budget_kernel<<<1, kBudgetThreads, 0, s>>>(one, BUD_INIT, false);
    return hipGetLastError();
}

hipError_t launch_materialize(const StepArgs& a, hipStream_t s) {
    dim3 g(div_up(a.P, 1024), div_up(a.Q, kMaterialize));
    materialize_kernel<<<g, 256, 0, s>>>(a, const_cast<float*>(a.psi));
    materialize_done_kernel<<<div_up(a.C, 256), 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_broadcast(float* psi, const float* cell, int Q, int64_t C, int64_t P,
                            hipStream_t s) {
    dim3 g(div_up(P, 1024), div_up(Q, kBroadcast));
    broadcast_kernel<<<g, 256, 0, s>>>(psi, cell, Q, C, P);
    return hipGetLastError();
}

}  // namespace asn
