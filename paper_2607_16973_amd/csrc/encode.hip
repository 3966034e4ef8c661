// Rotation + quantisation of float32 rows on gfx950 (section II-B, steps 1-5).
//
// Pipeline per chunk of rows:
//  0. split_rows_kernel: the row norm n = sqrt(sum_k x_k^2) (float64, see
//     kSumEps), a report of non-finite inputs, and every row scaled by
//     a power of two 2^e (n 2^e in [2^15, 2^16) / 1.02) and split into two
//     float16 parts, x 2^e = xh + xl (1 + eps).  The rotation is split the
//     same way once, R 2^15 = Rh + Rl (1 + eps).
//  1. encode_gemm: Y = X R^T on the float16 matrix cores
//     (v_mfma_f32_32x32x16_f16, sixteen times the float32 rate): xh Rh, xh Rl
//     and xl Rh, whose products are exact in float32.  The xh Rh partials of
//     each 32-wide slab of k are rounded into 32-bit integer accumulators, the
//     two small sums stay in float32.  The epilogue turns every y into a code
//     by comparing it with fl64(t_i * n) and flags the coordinate when y lies
//     within tau of a threshold, where tau bounds |y - S| for S the float64
//     sequential dot product of the definition.  With u = 2^-23 (twice the
//     unit roundoff, for additions that truncate), ||R_j|| <= 1 + 1e-6 and
//     A = sum_k |R_jk x_k| <= n (1 + 1e-6), relative to n:
//       xh Rh: 32 products per slab, added from 0 in any order: 33 u A
//              (1 + 2^-10)^2; rounded to the integer unit, at most 1.02 2^-30 n
//              (n 2^e may be as small as 2^15 / 1.02), once per slab: d/32 1.02 2^-31;
//       xh Rl + xl Rh: 2d products of which the absolute sum is at most
//              2^-10 A (1 + 2^-10), in any order: (2d + 1) u 2^-10 (1 + 2^-9);
//       xl Rl left out, and xl and Rl rounded: 2^-22 A each;
//       parts below the smallest normal float16 (2^-14, 2^-29 relative to
//              the scales, 1.02 2^-29 for x) if the matrix cores flush them: 4.08
//              sqrt(d) 2^-29;
//       the float64 reference itself: < 3e-13; the float32 arithmetic of
//              the epilogue: 5 2^-24.
//     tau_rel sums these: 5.6e-6 at d = 1536.
//  2. fixup: every flagged coordinate is recomputed as the sequential float64
//     sum sum_{k=0}^{d-1} R[j][k] x_k (every product of two float32 values is
//     exact in float64) and re-coded.  Flags are kept per list tile; with
//     few flags per tile (b <= 4) one wave per flag sums in parallel and only
//     falls back to the sequential order where that decides the code, with
//     many (b = 8, about 3% of coordinates) each tile stages its X and R
//     slabs in LDS once for all of its flags.
//  3. pack: per row, scale = n / sqrt(sum_j fl64(c_code_j^2)) (float64, as by
//     sequential sums: kSumEps) and the codes are written in the canonical bitstream
//     and/or the index's blocked layout.
// With TQ+ calibration (section II-B) coordinate j is coded against its own
// thresholds fl64(a_ij n), a_ij = fl64(mu_j + fl64(kappa_j t_i)), and the
// scale uses yhat_j = fl64(mu_j + fl64(kappa_j c_code_j)); both tables are
// computed on the host in float64 and passed in (CalibDev).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "kernels.h"
#include "lds_dma.h"

namespace tq {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int BM = 128;                 // rows of X per workgroup
constexpr int BN = 128;                 // rows of R (output columns) per workgroup
constexpr int KB = 32;                  // k per slab
constexpr int LDS_STRIDE = KB + 4;      // floats per staged row (conflict-free b128 reads)
constexpr int GEMM_THREADS = 512;       // 8 waves: 2 along rows x 4 along columns
constexpr int RC_PANEL = 32;            // rows of a split panel (an MFMA tile)

// The bound tau / n above.
double tau_rel(int d) {
    const double u = std::ldexp(1.0, -23);
    const double hh = 33 * u * (1 + std::ldexp(1.0, -10)) * (1 + std::ldexp(1.0, -10)) +
                      (d / 32) * 1.02 * std::ldexp(1.0, -31);
    const double small = (2 * d + 1) * u * std::ldexp(1.0, -10) * (1 + std::ldexp(1.0, -9));
    const double rest = 3 * std::ldexp(1.0, -22) + 4.08 * std::sqrt((double)d) * std::ldexp(1.0, -29) + 3e-13 +
                        5 * std::ldexp(1.0, -24);
    return (hh + small + rest) * (1 + 3e-6);
}

struct QuantArgs {
    const double *bounds;   // device copy of the thresholds t_i (levels-1)
    // TQ+ calibration: per-coordinate thresholds a_ij = mu_j + kappa_j t_i,
    // [levels-1][d] (null: the shared t_i)
    const double *athr;
    int levels;
    uint8_t *codes_tmp;     // [rows][d] unpacked codes of this chunk
    const float *inv;       // [rows] 1 / (n 2^(e + 15)): y / n per unit of the products; 0 for a zero row
    float tau;              // bound on |y - S| relative to the norm
    double bin_width;       // of the epilogue's table
    uint16_t *flags;        // per list tile, one slot per output: flagged (local row << 7 | local col)
    unsigned int *tile_count;   // flags of each list tile
};

// XCD-aware tile order: the d/BN column tiles of one row tile go to the same
// XCD (workgroups are dealt to the 8 XCDs round-robin), so the X tile is read
// from HBM once and then served by that XCD's L2.
__device__ inline void tile_of(int bid, int ncol, int &rt, int &ct) {
    const int x = bid & 7;
    const int rest = bid >> 3;
    ct = rest % ncol;
    rt = (rest / ncol) * 8 + x;
}

// Y = X R^T in float32 (query rotation).  Each 32-wide k-slab is
// accumulated on the matrix cores (v_mfma_f32_16x16x4f32, lane (l16, g4)
// feeding k = 16 sub + 4 g4 + st to step st of sub-slab sub) and then added
// into float64 accumulators in slab order; the result is rounded to float32
// once.  rot_small_kernel repeats exactly this arithmetic.
__global__ __launch_bounds__(GEMM_THREADS) void rot_gemm(
    const float *__restrict__ X, int64_t m, const float *__restrict__ R, int d,
    int n_row_tiles, float *__restrict__ Y) {
    __shared__ __attribute__((aligned(16))) float As[2][BM * LDS_STRIDE];
    __shared__ __attribute__((aligned(16))) float Bs[2][BN * LDS_STRIDE];

    const int ncol = (d + BN - 1) / BN;
    int rt, ct;
    tile_of(blockIdx.x, ncol, rt, ct);
    if (rt >= n_row_tiles) return;
    const int64_t row0 = (int64_t)rt * BM;
    const int col0 = ct * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wr = wave >> 2;     // 0..1 : 64-row half
    const int wc = wave & 3;      // 0..3 : 32-column quarter
    const int l16 = lane & 15;
    const int g4 = lane >> 4;

    // global -> register prefetch: 2 float4 of A and 2 of B per thread per slab
    f4 pa[2], pb[2];
    auto load_slab = [&](int k0) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int e = tid + r * GEMM_THREADS;
            const int row = e >> 3;
            const int kq = (e & 7) * 4;
            const int64_t gr = row0 + row;
            if (gr < m)
                pa[r] = *reinterpret_cast<const f4 *>(X + gr * d + k0 + kq);
            else
                pa[r] = f4{0.f, 0.f, 0.f, 0.f};
            if (col0 + row < d)
                pb[r] = *reinterpret_cast<const f4 *>(R + (int64_t)(col0 + row) * d + k0 + kq);
            else
                pb[r] = f4{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto store_slab = [&](int buf) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int e = tid + r * GEMM_THREADS;
            const int row = e >> 3;
            const int kq = (e & 7) * 4;
            *reinterpret_cast<f4 *>(&As[buf][row * LDS_STRIDE + kq]) = pa[r];
            *reinterpret_cast<f4 *>(&Bs[buf][row * LDS_STRIDE + kq]) = pb[r];
        }
    };

    f4 acc[4][2];
    double accd[4][2][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < 4; ++v) accd[i][j][v] = 0.0;
        }

    const int nslab = d / KB;
    load_slab(0);
    store_slab(0);
    __syncthreads();
    for (int s = 0; s < nslab; ++s) {
        const int buf = s & 1;
        if (s + 1 < nslab) load_slab((s + 1) * KB);
#pragma unroll
        for (int sub = 0; sub < KB / 16; ++sub) {
            f4 af[4], bf[2];
#pragma unroll
            for (int ti = 0; ti < 4; ++ti)
                af[ti] = *reinterpret_cast<const f4 *>(
                    &As[buf][(wr * 64 + ti * 16 + l16) * LDS_STRIDE + sub * 16 + g4 * 4]);
#pragma unroll
            for (int tj = 0; tj < 2; ++tj)
                bf[tj] = *reinterpret_cast<const f4 *>(
                    &Bs[buf][(wc * 32 + tj * 16 + l16) * LDS_STRIDE + sub * 16 + g4 * 4]);
#pragma unroll
            for (int st = 0; st < 4; ++st)
#pragma unroll
                for (int ti = 0; ti < 4; ++ti)
#pragma unroll
                    for (int tj = 0; tj < 2; ++tj)
                        acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            af[ti][st], bf[tj][st], acc[ti][tj], 0, 0, 0);
        }
        // fold the slab's float32 partials into float64
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int v = 0; v < 4; ++v) accd[i][j][v] += (double)acc[i][j][v];
                acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
            }
        if (s + 1 < nslab) store_slab(buf ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int lr = wr * 64 + ti * 16 + g4 * 4 + v;
            const int64_t gr = row0 + lr;
            if (gr >= m) continue;
#pragma unroll
            for (int tj = 0; tj < 2; ++tj) {
                const int col = col0 + wc * 32 + tj * 16 + l16;
                if (col < d) Y[gr * d + col] = (float)accd[ti][tj][v];
            }
        }
}

// ------------------------------------------------------ norms and splitting
// Split panels: 32 rows of a matrix in the operand order of
// v_mfma_f32_32x32x16_f16, [panel][k / 16][part][lane] with 16 bytes (8
// float16) per lane: lane l holds row 32 panel + (l & 31), k = 16 (k / 16) +
// 8 (l >> 5) .. +7; part 0 is the high part, part 1 the low one.  A panel's
// k-step is 2 KiB.
__device__ inline int64_t split_at(int64_t row, int ks, int h, int part, int d) {
    return (((row >> 5) * (d / 16) + ks) * 2 + part) * 64 + 32 * h + (row & 31);
}
// Splits the 8 values v (scaled by 2^e) and stores both parts.
__device__ inline void split_store(const f4 &v0, const f4 &v1, int e, uint4 *planes, int64_t at) {
    union {
        _Float16 f[8];
        uint4 u;
    } hi, lo;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float x = ldexpf(i < 4 ? v0[i & 3] : v1[i & 3], e);
        hi.f[i] = (_Float16)x;
        lo.f[i] = (_Float16)(x - (float)hi.f[i]);   // the difference is exact
    }
    planes[at] = hi.u;
    planes[at + 64] = lo.u;
}

constexpr int kRotScale = 15;           // R is scaled by 2^15

__global__ __launch_bounds__(256) void split_rotation_kernel(const float *__restrict__ R, int d,
                                                             uint4 *__restrict__ planes) {
    // consecutive threads: 8 rows of one 8-wide piece (128 bytes of a plane)
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t per8 = 8 * (d / 8);
    if (e >= (int64_t)d / 8 * per8) return;
    const int64_t row = e / per8 * 8 + (e & 7);
    const int piece = (int)(e % per8 >> 3);
    const f4 *src = reinterpret_cast<const f4 *>(R + row * d + piece * 8);
    split_store(src[0], src[1], kRotScale, planes, split_at(row, piece >> 1, piece & 1, 0, d));
}

// Norms.  The definition's norm n is the square root of the sum of squares
// added in k order in float64, a chain of d dependent additions.  A sum in any
// other order is within d 2^-53 (2.3e-13 at most) of the exact one like it (all
// terms are positive), so the two norms are within 2.3e-13 of each other
// relatively, and scales, with two such sums, within kSumEps.  The encoder works with parallel sums and
// repeats the chains where a result could depend on it: a scale whose
// float32 rounding differs within the margin (scale_of; about one row in
// 60,000), a coordinate as close to a threshold (fixup).  The chains took 5 us
// of latency per group of rows, 11 where one wave converted for them.
constexpr double kSumEps = 5e-13;

// The definition's norm of a row.
__device__ inline double exact_norm(const float *__restrict__ x, int d) {
    constexpr int B = 16;   // pieces of 4 loaded together (d is a multiple of 64)
    double s2 = 0.0;
    for (int k = 0; k < d; k += 4 * B) {
        f4 v[B];
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = *reinterpret_cast<const f4 *>(x + k + 4 * u);
#pragma unroll
        for (int u = 0; u < B; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c)   // the square is exact: fused or not
                s2 = __builtin_fma((double)v[u][c], (double)v[u][c], s2);
    }
    return std::sqrt(s2);
}
// n / sqrt(h2) as float32, and whether every pair within kSumEps of these
// rounds to the same.
__device__ inline bool scale_of(double n, double h2, float &s) {
    const double q = n / std::sqrt(h2);
    s = (float)q;
    return (float)(q * (1.0 - kSumEps)) == (float)(q * (1.0 + kSumEps));
}

// Norms and split panels of 8 rows per workgroup (rows m .. up to a multiple
// of 32: zeros).  The rows are read once into LDS (padded by one 16-byte
// piece, so that the 8 rows' pieces lie in distinct banks), a wave sums two
// rows, and all split: bound by the 8 bytes that are read and written per
// coordinate (32,768 rows at d = 1536: 68 us, 5.9 TB/s; 110 us with the
// norm's chain in the kernel).  A non-finite input makes the sum non-finite (x^2 of a finite
// float32 cannot overflow float64), which sets *status.
constexpr int SR_ROWS = 8;
constexpr int SR_THREADS = 256;
__global__ __launch_bounds__(SR_THREADS) void split_rows_kernel(
    const float *__restrict__ X, int64_t m, int d, uint4 *__restrict__ planes,
    double *__restrict__ norms, float *__restrict__ inv, int *__restrict__ status) {
    extern __shared__ __attribute__((aligned(16))) float xs[];   // [SR_ROWS][d + 4]
    __shared__ int exps[SR_ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * SR_ROWS;
    const int ps = d + 4, pq = d / 4;   // LDS row stride; 16-byte pieces of a row
    constexpr int LD = SR_ROWS * (2048 / 4) / SR_THREADS;   // loads per thread, d <= 2048
    {
        f4 v[LD];
        const int total = SR_ROWS * pq;
#pragma unroll
        for (int u = 0; u < LD; ++u) {
            const int e = tid + u * SR_THREADS;
            const int r = e / pq;
            v[u] = f4{0.f, 0.f, 0.f, 0.f};
            if (e < total && r0 + r < m)
                v[u] = *reinterpret_cast<const f4 *>(X + (r0 + r) * d + (e - r * pq) * 4);
        }
#pragma unroll
        for (int u = 0; u < LD; ++u) {
            const int e = tid + u * SR_THREADS;
            const int r = e / pq;
            if (e < total) *reinterpret_cast<f4 *>(xs + r * ps + (e - r * pq) * 4) = v[u];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 2 * wave + i;
        double s = 0.0;
        for (int q = lane; q < pq; q += 64) {
            const f4 v = *reinterpret_cast<const f4 *>(xs + r * ps + 4 * q);
#pragma unroll
            for (int c = 0; c < 4; ++c) s = __builtin_fma((double)v[c], (double)v[c], s);
        }
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) {
            const double n = std::sqrt(s);
            const bool ok = n > 0.0 && std::isfinite(n);
            const int e = ok ? 15 - ilogb(n * 1.02) : 0;
            exps[r] = e;
            if (r0 + r < m) {
                norms[r0 + r] = n;
                if (!std::isfinite(s)) atomicOr(status, 1);
            }
            if (r0 + r < m) inv[r0 + r] = ok ? (float)(1.0 / ldexp(n, e + kRotScale)) : 0.f;
        }
    }
    __syncthreads();
    for (int e = tid; e < SR_ROWS * (d / 8); e += SR_THREADS) {
        const int r = e & 7, piece = e >> 3;
        const f4 *x = reinterpret_cast<const f4 *>(xs + r * ps + piece * 8);
        split_store(x[0], x[1], exps[r], planes, split_at(r0 + r, piece >> 1, piece & 1, 0, d));
    }
}

// ------------------------------------------------------------- encode_gemm
// Y = X R^T with the quantiser epilogue, for the encode.  WR x WC waves of TM
// x TN tiles of 32 x 32 outputs:
//  - both operands are split panels, staged by direct global -> LDS loads of
//    1 KiB pieces into a ring of ST k-steps of 16, ST - 1 k-steps ahead,
//    one barrier per k-step; operand reads are 16 bytes per lane at
//    consecutive addresses;
//  - three products per tile and k-step.  The integer fold of the previous
//    slab's xh Rh partials (round, convert, add) is interleaved with them and
//    is hidden behind them: 24 products and the fold of four tiles run at the
//    rate of the products alone (2.0 to 2.1 PFLOP/s in a register-only loop),
//    which a fold into float64 does not (it has twice the registers).
// Large shape (TM = TN = 2, 2 x 2 waves, 128 x 128 outputs, two workgroups per
// compute unit): 224 registers of accumulators and operands leave two waves
// per SIMD.  Each operand register is read again for the next k-step as soon as
// its last product is issued; the column order alternates so that the next
// k-step starts with the pair that was read first.  32,768 rows at d = 1536
// take 530 us, 870 TFLOP/s of products (1,409 us with float32 products); of
// the time, without the loads into LDS it would be 160 us less, without the
// reads from it 70 us, without the fold 45 us.  256 x 128 outputs and one
// workgroup of 8 waves move a quarter less through the L2 and take as long,
// but 83 instead of 56 us where one round of tiles is all there is.
// Small shape (TM = TN = 1, 2 x 2 waves, 64 x 64 outputs) for row counts
// whose large tiles would leave compute units idle: see kEncodeSmallOutputs.
//
// The epilogue's table of the thresholds t_0 .. t_{L-2}: EG_BINS bins of equal
// width over [t_0, t_{L-2}] (values outside take the end ones), each with the
// threshold next to its centre and the number of thresholds below that one.
// Two thresholds are at least 1/519 of the range apart (over all dimensions
// and widths, at b = 8), almost two bins, so that no other threshold lies in
// the bin or within tau of it.
constexpr int EG_BINS = 1024;

typedef float f16v __attribute__((ext_vector_type(16)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

template <int TM, int TN, int WR, int WC, int ST>
struct EgShape {
    static constexpr int STAGES = ST;
    static constexpr int WAVES = WR * WC;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int RP = TM * WR, CP = TN * WC;     // panels of rows and columns
    static constexpr int ROWS = 32 * RP, COLS = 32 * CP;
    static constexpr int PIECES = 2 * (RP + CP);         // 1 KiB pieces of a k-step
    static constexpr int PW = PIECES / WAVES;            // of which a wave loads
    static constexpr int STEP_B = PIECES * 1024;
    static constexpr int SIDE = COLS;                    // of a workgroup's outputs and list
    static_assert(ROWS == COLS, "square tiles");
    static constexpr size_t lds = (size_t)ST * STEP_B + ROWS * 4 + EG_BINS * 8 + 8;
    static_assert(PIECES % WAVES == 0, "whole pieces per wave");
};
using EgLarge = EgShape<2, 2, 2, 2, 4>;
using EgSmall = EgShape<1, 1, 2, 2, 6>;

template <int TM, int TN, int WR, int WC, int ST>
__global__ __launch_bounds__(64 * WR * WC, 2) void encode_gemm(
    const uint4 *__restrict__ Xp, int64_t m, const uint4 *__restrict__ Rp, int d, int n_row_tiles,
    QuantArgs qa) {
    using S = EgShape<TM, TN, WR, WC, ST>;
    static_assert((TM == 1 && TN == 1) || (TM == 2 && TN == 2), "operand schedules below");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    char *stg = smem;
    float *inv_s = reinterpret_cast<float *>(smem + ST * S::STEP_B);      // [ROWS]
    float2 *bin_s = reinterpret_cast<float2 *>(inv_s + S::ROWS);                 // [EG_BINS]
    unsigned int *nflag_s = reinterpret_cast<unsigned int *>(bin_s + EG_BINS);

    const int ncol = (d + S::COLS - 1) / S::COLS;
    int rt, ct;
    tile_of(blockIdx.x, ncol, rt, ct);
    if (rt >= n_row_tiles) return;
    const int64_t row0 = (int64_t)rt * S::ROWS;
    const int col0 = ct * S::COLS;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WC, wc = wave % WC;
    const int l32 = lane & 31;
    const int h = lane >> 5;
    const int KS = d / 16;        // even: d is a multiple of 64

    // This wave's pieces of a k-step: piece p is part p & 1 of row panel
    // p >> 1 (p < 2 RP), then of the column panels.  Panels past the last row
    // or column are clamped to the last one: they only feed outputs that the
    // epilogue drops.
    const int64_t last_rp = (m - 1) >> 5;
    const int last_cp = (d >> 5) - 1;
    const char *src[S::PW];
#pragma unroll
    for (int j = 0; j < S::PW; ++j) {
        const int p = wave * S::PW + j;
        const bool is_r = p < 2 * S::RP;
        int64_t panel = is_r ? (row0 >> 5) + (p >> 1) : (col0 >> 5) + ((p - 2 * S::RP) >> 1);
        const int64_t last = is_r ? last_rp : last_cp;
        panel = panel < last ? panel : last;
        src[j] = reinterpret_cast<const char *>(is_r ? Xp : Rp) + panel * KS * 2048 + (p & 1) * 1024;
    }
    const uint32_t stg_lds = (uint32_t)(uintptr_t)stg;
    int rq = 0, rq_st = 0;        // next k-step to request (the last one again past the end), its stage
    auto request = [&]() {
        const uint32_t base = stg_lds + rq_st * S::STEP_B + wave * (S::PW * 1024);
        const int64_t off = (int64_t)(rq < KS ? rq : KS - 1) * 2048;
#pragma unroll
        for (int j = 0; j < S::PW; ++j) lds_dma16_s((uint32_t)lane * 16, src[j] + off, base + j * 1024);
        ++rq;
        rq_st = rq_st + 1 == ST ? 0 : rq_st + 1;
    };

    const int L = qa.levels;
    if (!qa.athr)
        for (int e = tid; e < EG_BINS; e += S::THREADS) {
            const double centre = qa.bounds[0] + (e + 0.5) * qa.bin_width;
            int c = 0;   // thresholds at most the centre
            for (int step = L / 2; step >= 1; step >>= 1) c += qa.bounds[c + step - 1] <= centre ? step : 0;
            const bool up = c == 0 || (c < L - 1 && qa.bounds[c] - centre < centre - qa.bounds[c - 1]);
            const int i = up ? c : c - 1;
            bin_s[e] = make_float2((float)qa.bounds[i], __int_as_float(i));
        }
    if (tid == 0) *nflag_s = 0;
    for (int r = tid; r < S::ROWS; r += S::THREADS) inv_s[r] = row0 + r < m ? qa.inv[row0 + r] : 0.f;
    wait_vmem<0>();   // the counts below are of the pieces alone
#pragma unroll
    for (int i = 0; i < ST - 1; ++i) request();

    const f16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                       0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f16v hh[TM][TN], sm[TM][TN];   // xh Rh of the current slab; xh Rl + xl Rh
    int tot[TM][TN][16];           // xh Rh of the slabs before
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            hh[i][j] = zero;
            sm[i][j] = zero;
#pragma unroll
            for (int e = 0; e < 16; ++e) tot[i][j][e] = 0;
        }
    // operands [set][tile][part]; the small shape has two sets in turn
    constexpr int SETS = TM == 1 ? 2 : 1;
    half8 a[SETS][TM][2], b[SETS][TN][2];
    int rd_st = 0;                // stage of the operands read next
    const char *a_at = stg + wr * TM * 2048 + lane * 16;
    const char *b_at = stg + S::RP * 2048 + wc * TN * 2048 + lane * 16;
    auto load_a = [&](int set, int i) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
            a[set][i][p] = *reinterpret_cast<const half8 *>(a_at + rd_st * S::STEP_B + i * 2048 + p * 1024);
    };
    auto load_b = [&](int set, int j) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
            b[set][j][p] = *reinterpret_cast<const half8 *>(b_at + rd_st * S::STEP_B + j * 2048 + p * 1024);
    };
    auto fold = [&](int i, int j, int half) {
#pragma unroll
        for (int e = 8 * half; e < 8 * half + 8; ++e) tot[i][j][e] += (int)__builtin_rintf(hh[i][j][e]);
    };
    // the three products of tile (i, j); an even k-step starts a slab
    auto products = [&](int set, int i, int j, bool even) {
        sm[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[set][i][1], b[set][j][0], sm[i][j], 0, 0, 0);
        if (even) {
            __builtin_amdgcn_sched_barrier(0);
            fold(i, j, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        sm[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[set][i][0], b[set][j][1], sm[i][j], 0, 0, 0);
        if (even) {
            __builtin_amdgcn_sched_barrier(0);
            fold(i, j, 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        hh[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[set][i][0], b[set][j][0], even ? zero : hh[i][j],
                                                          0, 0, 0);
    };
    // Publishes the k-step after the current one (own pieces landed, then
    // everyone's) and requests the k-step ST - 1 ahead into the stage of the
    // previous one, which every wave is past.  Operand reads in flight need
    // not complete here: their stage is not written before the next
    // publication but one.
    auto publish = [&]() {
        wait_vmem<(ST - 3) * S::PW>();
        asm volatile("s_barrier" ::: "memory");
        request();
    };
    wait_vmem<(ST - 2) * S::PW>();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i) load_a(0, i);
#pragma unroll
    for (int j = 0; j < TN; ++j) load_b(0, j);
    rd_st = 1;
    auto step = [&](auto PAR) {
        constexpr int par = decltype(PAR)::value;
        constexpr bool even = par == 0;
        if constexpr (TM == 1) {
            publish();
            load_a(par ^ 1, 0);
            load_b(par ^ 1, 0);
            __builtin_amdgcn_sched_barrier(0);
            products(par, 0, 0, even);
        } else {
            constexpr int c0 = par, c1 = par ^ 1;   // column order
            products(0, 0, c0, even);
            __builtin_amdgcn_sched_barrier(0);
            publish();
            __builtin_amdgcn_sched_barrier(0);
            products(0, 0, c1, even);
            __builtin_amdgcn_sched_barrier(0);
            load_a(0, 0);
            products(0, 1, c1, even);
            __builtin_amdgcn_sched_barrier(0);
            load_b(0, c1);
            products(0, 1, c0, even);
            __builtin_amdgcn_sched_barrier(0);
            load_a(0, 1);
            load_b(0, c0);
        }
        __builtin_amdgcn_sched_barrier(0);
        rd_st = rd_st + 1 == ST ? 0 : rd_st + 1;
    };
    for (int ks = 0; ks < KS; ks += 2) {
        step(std::integral_constant<int, 0>());
        step(std::integral_constant<int, 1>());
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            fold(i, j, 0);
            fold(i, j, 1);
        }
    wait_vmem<0>();    // the pieces requested past the end have landed:
    __syncthreads();   // the stages are free
    // TQ+ thresholds of the tile's columns, b <= 4, in the stages
    float *athr_s = reinterpret_cast<float *>(stg);
    const bool athr_lds = qa.athr && qa.levels <= 16;
    if (athr_lds) {
        for (int e = tid; e < (qa.levels - 1) * S::COLS; e += S::THREADS) {
            const int i = e / S::COLS, c = col0 + e % S::COLS;
            athr_s[e] = c < d ? (float)qa.athr[(int64_t)i * d + c] : 0.f;
        }
        __syncthreads();
    }

    const int lrow = wr * 32 * TM;                 // the wave's first row in the workgroup's tile
    const int64_t tile = (int64_t)rt * ncol + ct;
    uint16_t *tflags = qa.flags + tile * (S::SIDE * S::SIDE);
    // Code and flag of the lane's 16 outputs of a tile (one column, 16 rows),
    // from z = y / n in float32: the float32 rounding of the two sums, of
    // 1 / n, of the product and of the threshold is at most 4 2^-24 (|z| <= 1
    // up to tau), part of tau.  find(lc, z, c, flag) gives the number c of
    // thresholds at most z and whether one lies within tau of z.
    const bool whole = row0 + S::ROWS <= m && col0 + S::COLS <= d;
    uint8_t *cbase = qa.codes_tmp + row0 * d + col0;
    auto epilogue = [&](int ti, int tj, auto find) {
        const int lc = wc * 32 * TN + tj * 32 + l32;
        const int r0 = lrow + ti * 32 + 4 * h;   // row of output i: r0 + 8 (i >> 2) + (i & 3)
        const uint32_t at = (uint32_t)(r0 * d + lc);
        uint32_t flagged = 0u;   // bit i: output i
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int dr = 8 * (i >> 2) + (i & 3);
            const float z = ((float)tot[ti][tj][i] + sm[ti][tj][i]) * inv_s[r0 + dr];
            int c;
            bool flag;
            find(lc, z, c, flag);
            flagged |= flag ? 1u << i : 0u;
            if (whole || (row0 + r0 + dr < m && col0 + lc < d)) cbase[at + (uint32_t)(dr * d)] = (uint8_t)c;
        }
        while (flagged) {   // rare: a slot of this tile's list each (an LDS counter)
            const int i = __builtin_ctz(flagged);
            flagged &= flagged - 1u;
            const int r = r0 + 8 * (i >> 2) + (i & 3);
            if (row0 + r >= m || col0 + lc >= d) continue;
            if (inv_s[r] == 0.f)   // a zero row
                cbase[(uint32_t)(r * d + lc)] = (uint8_t)(L / 2);
            else
                tflags[atomicAdd(nflag_s, 1u)] = (uint16_t)((r << 7) | lc);
        }
    };
    if (!qa.athr) {
        const float t0 = (float)qa.bounds[0], inv_w = (float)(1.0 / qa.bin_width);
        auto find = [&](int, float z, int &c, bool &flag) {
            const float x = fminf(fmaxf((z - t0) * inv_w, 0.f), (float)(EG_BINS - 1));
            const float2 b = bin_s[(int)x];
            c = __float_as_int(b.y) + (b.x <= z ? 1 : 0);
            flag = fabsf(z - b.x) <= qa.tau;
        };
#pragma unroll
        for (int ti = 0; ti < TM; ++ti)
#pragma unroll
            for (int tj = 0; tj < TN; ++tj) epilogue(ti, tj, find);
    } else {
        // TQ+: a binary search of the column's own thresholds (L is a power
        // of two: c + step - 1 <= L - 2); zero rows may lie away from all of
        // them and are always flagged
        auto find = [&](int lc, float z, int &c, bool &flag) {
            const int col = col0 + lc < d ? col0 + lc : d - 1;
            auto thr = [&](int q) { return athr_lds ? athr_s[q * S::COLS + lc] : (float)qa.athr[(int64_t)q * d + col]; };
            c = 0;
            for (int step = L / 2; step >= 1; step >>= 1) c += thr(c + step - 1) <= z ? step : 0;
            flag = fabsf(z - thr(c > 0 ? c - 1 : 0)) <= qa.tau ||
                   fabsf(thr(c < L - 1 ? c : L - 2) - z) <= qa.tau || z == 0.f;
        };
#pragma unroll
        for (int ti = 0; ti < TM; ++ti)
#pragma unroll
            for (int tj = 0; tj < TN; ++tj) epilogue(ti, tj, find);
    }
    __syncthreads();
    if (tid == 0) qa.tile_count[tile] = *nflag_s;
}

// The code of coordinate j of a row with norm nrm whose exact sum is S.
__device__ inline int exact_code(double S, double nrm, int j, int d, const double *bounds,
                                 const double *athr, int levels) {
    int c = 0;
    for (int t = 0; t < levels - 1; ++t) {
        const double th = (athr ? athr[(int64_t)t * d + j] : bounds[t]) * nrm;
        c += (th <= S) ? 1 : 0;
    }
    return c;
}

// Exact recomputation of flagged coordinates (b <= 4).  One wave per flag
// (the list tile's flags w, w + 4, ... for wave w) adds the coordinate's
// products in float64 in parallel: every product is exact, so that sum and
// the definition's sequential one differ by at most 2 gamma_d n < kSumEps n.
// If no threshold lies that close, both give the same code; otherwise (about
// one flag in a million) the wave repeats the sum, and the norm's, in k order
// from its registers.  Bound by the 12 KiB of X and R a flag reads (68,000 flags of
// 32,768 rows at d = 1536: 128 us, 6.4 TB/s); one lane per flag summing in k
// order took 47 us for 400 flags, this takes 11.
constexpr int FX_WAVES = 4;
constexpr int FX_PC = 2048 / 256;            // 16-byte pieces of a row per lane at most

__global__ __launch_bounds__(FX_WAVES * 64) void fixup_flag_kernel(
    const float *__restrict__ X, const float *__restrict__ R, int d, int side, int nrow, int ncol,
    const double *__restrict__ bounds, const double *__restrict__ athr, int levels,
    const double *__restrict__ norms,
    const uint16_t *__restrict__ flags, const unsigned int *__restrict__ tile_count,
    uint8_t *__restrict__ codes_tmp) {
    int rt, ct;   // the column tiles of a row tile on one XCD: they share X rows
    tile_of(blockIdx.x, ncol, rt, ct);
    if (rt >= nrow) return;
    const int tile = rt * ncol + ct;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)rt * side;
    const int col0 = ct * side;
    const int cnt = (int)tile_count[tile];
    const uint16_t *tflags = flags + (int64_t)tile * (side * side);
    const int pq = d / 4;
    for (int f = wave; f < cnt; f += FX_WAVES) {
        const uint32_t fl = tflags[f];
        const int64_t row = row0 + (fl >> 7);
        const int j = col0 + (int)(fl & 127);
        const float *xr = X + row * d, *rr = R + (int64_t)j * d;
        f4 x[FX_PC], r[FX_PC];
#pragma unroll
        for (int u = 0; u < FX_PC; ++u) {
            const int q = lane + 64 * u;
            x[u] = r[u] = f4{0.f, 0.f, 0.f, 0.f};
            if (q < pq) {
                x[u] = *reinterpret_cast<const f4 *>(xr + 4 * q);
                r[u] = *reinterpret_cast<const f4 *>(rr + 4 * q);
            }
        }
        double nrm = norms[row];
        double S = 0.0;
#pragma unroll
        for (int u = 0; u < FX_PC; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) S = __builtin_fma((double)r[u][c], (double)x[u][c], S);
        for (int o = 32; o > 0; o >>= 1) S += __shfl_xor(S, o, 64);
        const double eps = 2 * kSumEps * nrm;   // of S, and of the thresholds' norm
        int code = exact_code(S + eps, nrm, j, d, bounds, athr, levels);
        if (code != exact_code(S - eps, nrm, j, d, bounds, athr, levels) || !std::isfinite(S)) {
            double T = 0.0, T2 = 0.0;
#pragma unroll
            for (int u = 0; u < FX_PC; ++u) {
                double p[4], p2[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    p[c] = (double)r[u][c] * (double)x[u][c];
                    p2[c] = (double)x[u][c] * (double)x[u][c];
                }
                const int nl = pq - 64 * u < 64 ? pq - 64 * u : 64;
                for (int l = 0; l < nl; ++l)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        T = T + __shfl(p[c], l, 64);
                        T2 = T2 + __shfl(p2[c], l, 64);
                    }
            }
            nrm = std::sqrt(T2);
            code = exact_code(T, nrm, j, d, bounds, athr, levels);
        }
        if (lane == 0) codes_tmp[row * d + j] = (uint8_t)code;
    }
}

// The same recomputation for tiles with many flags: the tile's X rows and R
// rows pass through LDS in slabs of KB (once per 512 flags), and each
// thread adds its flag's products in k order from there.  List tiles have
// `side` rows and columns (128 or 64).
__global__ __launch_bounds__(GEMM_THREADS) void fixup_tile_kernel(
    const float *__restrict__ X, int64_t m, const float *__restrict__ R, int d, int side, int ncol,
    const double *__restrict__ bounds, const double *__restrict__ athr, int levels,
    const double *__restrict__ norms,
    const uint16_t *__restrict__ flags, const unsigned int *__restrict__ tile_count,
    uint8_t *__restrict__ codes_tmp) {
    __shared__ __attribute__((aligned(16))) float As[BM * LDS_STRIDE];
    __shared__ __attribute__((aligned(16))) float Bs[BN * LDS_STRIDE];
    const int tile = blockIdx.x;
    const int64_t row0 = (int64_t)(tile / ncol) * side;
    const int col0 = (tile % ncol) * side;
    const unsigned int cnt = tile_count[tile];
    if (cnt == 0) return;
    const uint16_t *tflags = flags + (int64_t)tile * (side * side);
    const int tid = threadIdx.x;
    for (unsigned int e0 = 0; e0 < cnt; e0 += GEMM_THREADS) {
        const unsigned int e = e0 + tid;
        const bool active = e < cnt;
        const uint32_t f = active ? tflags[e] : 0u;
        const int lr = (int)(f >> 7), lc = (int)(f & 127);
        double S = 0.0;
        for (int k0 = 0; k0 < d; k0 += KB) {
            __syncthreads();   // the previous slab has been read
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int q = tid + r * GEMM_THREADS;
                const int row = q >> 3;
                const int kq = (q & 7) * 4;
                if (row >= side) continue;
                const int64_t gr = row0 + row;
                const f4 a = gr < m ? *reinterpret_cast<const f4 *>(X + gr * d + k0 + kq)
                                    : f4{0.f, 0.f, 0.f, 0.f};
                const f4 b = col0 + row < d
                                 ? *reinterpret_cast<const f4 *>(R + (int64_t)(col0 + row) * d + k0 + kq)
                                 : f4{0.f, 0.f, 0.f, 0.f};
                *reinterpret_cast<f4 *>(&As[row * LDS_STRIDE + kq]) = a;
                *reinterpret_cast<f4 *>(&Bs[row * LDS_STRIDE + kq]) = b;
            }
            __syncthreads();
            if (active) {
                const float *xa = &As[lr * LDS_STRIDE];
                const float *rb = &Bs[lc * LDS_STRIDE];
#pragma unroll
                for (int q = 0; q < KB; q += 4) {
                    const f4 a = *reinterpret_cast<const f4 *>(rb + q);
                    const f4 b = *reinterpret_cast<const f4 *>(xa + q);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const double prod = (double)a[c] * (double)b[c];
                        S = S + prod;
                    }
                }
            }
        }
        if (active) {
            const int64_t row = row0 + lr;
            const int j = col0 + lc;
            const double nrm = norms[row], eps = kSumEps * nrm;
            int code = exact_code(S + eps, nrm, j, d, bounds, athr, levels);
            if (code != exact_code(S - eps, nrm, j, d, bounds, athr, levels))   // the norm's last bits decide
                code = exact_code(S, exact_norm(X + row * d, d), j, d, bounds, athr, levels);
            codes_tmp[row * d + j] = (uint8_t)code;
        }
    }
}

// Packs 16 rows per workgroup, for the bit widths whose 16-byte blocked chunk
// holds 128 / BITS codes as 4 words of 32 / BITS codes (BITS in {1, 2, 4, 8};
// the canonical words are the same words): thread (row, c) takes the row's
// chunks c, c + 16, ..., adds their part of the scale's sum of fl64(c_code^2)
// (or the calibrated reconstruction's square) and writes each chunk's 16
// bytes to the canonical and blocked layouts (there 16 rows are 256 adjacent
// bytes).  The 16 parts are added in LDS.  For a row whose scale could depend
// on the order the workgroup stages the terms in LDS and one thread each
// repeats the definition's two chains.  257 rows at d = 1536 and 4 bits take
// 8 us (22 us with a row's chain per thread); 32,768 rows 39, of which about 15
// are such a row's chains in every second chunk of rows (30).
constexpr int PR_ROWS = 16;
template <int BITS>
__global__ __launch_bounds__(256) void pack_rows_kernel(
    const uint8_t *__restrict__ codes_tmp, const float *__restrict__ X, int64_t m, int d,
    const double *__restrict__ cent_sq, const double *__restrict__ ysq,
    const double *__restrict__ norms,
    uint8_t *__restrict__ canon, float *__restrict__ scales,
    uint8_t *__restrict__ blocked, float *__restrict__ blocked_scales, int64_t base,
    int chunks) {
    constexpr int L = 1 << BITS;
    constexpr int CPC = 128 / BITS;   // codes per chunk
    constexpr int LPC = CPC / 16;     // 16-byte loads of one-byte codes per chunk
    constexpr int PER = 32 / BITS;    // codes per word
    __shared__ double csq_s[L];
    __shared__ double part[16][PR_ROWS];
    __shared__ double sq_s[2048];   // a row's terms
    __shared__ float x_s[2048];
    __shared__ double chain_s[2];
    __shared__ int nredo;
    __shared__ int redo[PR_ROWS];
    const int tid = threadIdx.x, rl = tid & (PR_ROWS - 1), cg = tid / PR_ROWS;
    for (int i = tid; i < L; i += 256) csq_s[i] = ysq ? 0.0 : cent_sq[i];
    __syncthreads();
    const int64_t r = (int64_t)blockIdx.x * PR_ROWS + rl;
    const uint8_t *row = codes_tmp + (r < m ? r : 0) * d;
    const uint4 *src = reinterpret_cast<const uint4 *>(row);
    const int64_t v = base + r;
    uint8_t *bdst = blocked && r < m ? blocked + (v >> 6) * chunks * 1024 + (v & 63) * 16 : nullptr;
    uint8_t *cdst = canon && r < m ? canon + r * (int64_t)(d * BITS / 8) : nullptr;
    double h2 = 0.0;
    auto square = [&](int j, uint32_t code) { return ysq ? ysq[(int64_t)j * L + code] : csq_s[code]; };
    for (int ch = cg; ch < chunks; ch += 16) {
        uint4 cur[LPC];
#pragma unroll
        for (int i = 0; i < LPC; ++i) cur[i] = src[ch * LPC + i];
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < CPC; ++t) {
            const uint4 &q = cur[t >> 4];
            const int u = (t >> 2) & 3;
            const uint32_t word = u == 0 ? q.x : u == 1 ? q.y : u == 2 ? q.z : q.w;
            const uint32_t code = (word >> (8 * (t & 3))) & 255u;
            w[t / PER] |= code << (BITS * (t % PER));
            h2 = h2 + square(ch * CPC + t, code);
        }
        if (cdst) *reinterpret_cast<uint4 *>(cdst + ch * 16) = make_uint4(w[0], w[1], w[2], w[3]);
        if (bdst) {
            if (blocked_rotated(BITS))
                for (int u = 0; u < 4; ++u) w[u] = rotl2(w[u]);
            *reinterpret_cast<uint4 *>(bdst + ch * 1024) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    part[cg][rl] = h2;
    if (tid == 0) nredo = 0;
    __syncthreads();
    auto put = [&](int64_t row_, float s) {
        if (scales) scales[row_] = s;
        if (blocked_scales) blocked_scales[base + row_] = s;
    };
    if (cg == 0 && r < m) {
        for (int c = 1; c < 16; ++c) h2 += part[c][rl];
        const double nrm = norms[r];
        float s = 0.f;
        if (nrm != 0.0 && !scale_of(nrm, h2, s)) redo[atomicAdd(&nredo, 1)] = rl;
        else put(r, s);
    }
    __syncthreads();
    const int nr = nredo;
    for (int i = 0; i < nr; ++i) {
        const int64_t rr = (int64_t)blockIdx.x * PR_ROWS + redo[i];
        for (int j = tid; j < d; j += 256) {
            x_s[j] = X[rr * d + j];
            sq_s[j] = square(j, codes_tmp[rr * d + j]);
        }
        __syncthreads();
        if (tid == 0) {
            double s2 = 0.0;
            for (int j = 0; j < d; j += 32) {   // 32 terms read together (d is a multiple of 64)
                float t[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) t[u] = x_s[j + u];
#pragma unroll
                for (int u = 0; u < 32; ++u) s2 = __builtin_fma((double)t[u], (double)t[u], s2);
            }
            chain_s[0] = std::sqrt(s2);
        }
        if (tid == 64) {
            double s2 = 0.0;
            for (int j = 0; j < d; j += 16) {
                double t[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) t[u] = sq_s[j + u];
#pragma unroll
                for (int u = 0; u < 16; ++u) s2 = s2 + t[u];
            }
            chain_s[1] = std::sqrt(s2);
        }
        __syncthreads();
        if (tid == 0) put(rr, (float)(chain_s[0] / chain_s[1]));
    }
}

// Packs PACK_ROWS rows per workgroup (3-bit codes): scale, canonical
// bitstream, blocked layout.
// The codes are staged in LDS with a row stride of d + 16 bytes, so that the
// scale threads (one per row, reading 16 codes at a time) meet different
// banks.
constexpr int PACK_ROWS = 32;   // PACK_ROWS * (d + 16) bytes of LDS (66 KiB at d = 2048)

__global__ __launch_bounds__(256) void pack_kernel(
    const uint8_t *__restrict__ codes_tmp, const float *__restrict__ X, int64_t m, int d,
    const double *__restrict__ cent_sq, const double *__restrict__ ysq,
    const double *__restrict__ norms,
    uint8_t *__restrict__ canon, float *__restrict__ scales,
    uint8_t *__restrict__ blocked, float *__restrict__ blocked_scales, int64_t base,
    int chunks) {
    extern __shared__ __attribute__((aligned(16))) uint8_t cs_raw[];   // [PACK_ROWS][d + 16]
    __shared__ double csq_s[8];
    const int64_t r0 = (int64_t)blockIdx.x * PACK_ROWS;
    const int rows = (int)((m - r0) < PACK_ROWS ? (m - r0) : PACK_ROWS);
    const int tid = threadIdx.x;
    constexpr int L = 8;
    const int ps = d + 16;           // LDS row stride
    if (!ysq)
        for (int i = tid; i < L; i += blockDim.x) csq_s[i] = cent_sq[i];
    // stage codes, 16 B per piece; each thread's pieces are loaded together
    const int vec_per_row = d / 16;
    const int total = rows * vec_per_row;
    constexpr int PIECES = PACK_ROWS * (2048 / 16) / 256;   // at most 16 per thread
    uint4 v[PIECES];
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
        const int e = min(tid + u * 256, total - 1);   // rows >= 1: a valid piece
        const int r = e / vec_per_row, q = e % vec_per_row;
        v[u] = reinterpret_cast<const uint4 *>(codes_tmp + (r0 + r) * d)[q];
    }
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
        const int e = tid + u * 256;
        if (e < total) {
            const int r = e / vec_per_row, q = e % vec_per_row;
            reinterpret_cast<uint4 *>(cs_raw + r * ps)[q] = v[u];
        }
    }
    __syncthreads();
    // scale: one thread per row, j in order
    if (tid < rows) {
        const uint8_t *c = cs_raw + tid * ps;
        // sum_j fl64(yhat_j^2): c[code]^2, or with TQ+ the calibrated
        // reconstruction's square, per coordinate ([d][levels])
        double h2 = 0.0;
        if (ysq) {
            for (int j = 0; j < d; ++j) h2 = h2 + ysq[(int64_t)j * L + c[j]];
        } else {
            for (int j = 0; j < d; j += 16) {
                const uint4 w = *reinterpret_cast<const uint4 *>(c + j);
#pragma unroll
                for (int q = 0; q < 4; ++q) h2 = h2 + csq_s[(w.x >> (8 * q)) & 255];
#pragma unroll
                for (int q = 0; q < 4; ++q) h2 = h2 + csq_s[(w.y >> (8 * q)) & 255];
#pragma unroll
                for (int q = 0; q < 4; ++q) h2 = h2 + csq_s[(w.z >> (8 * q)) & 255];
#pragma unroll
                for (int q = 0; q < 4; ++q) h2 = h2 + csq_s[(w.w >> (8 * q)) & 255];
            }
        }
        const double nrm = norms[r0 + tid];
        float s = 0.f;
        if (nrm != 0.0 && !scale_of(nrm, h2, s))
            s = (float)(exact_norm(X + (r0 + tid) * d, d) / std::sqrt(h2));
        if (scales) scales[r0 + tid] = s;
        if (blocked_scales) blocked_scales[base + r0 + tid] = s;
    }
    // canonical rows: 32-bit words, bits LSB-first
    const int wpr = d * 3 / 32;   // words per canonical row
    if (canon) {
        for (int e = tid; e < rows * wpr; e += blockDim.x) {
            const int r = e / wpr, w = e % wpr;
            const uint8_t *c = cs_raw + r * ps;
            uint32_t word = 0;
            const int b0 = w * 32;
            for (int t = 0; t < 32; ++t) {
                const int bit = b0 + t;
                const int j = bit / 3, sh = bit % 3;
                word |= (uint32_t)((c[j] >> sh) & 1) << t;
            }
            reinterpret_cast<uint32_t *>(canon + (r0 + r) * (int64_t)(d * 3 / 8))[w] = word;
        }
    }
    // blocked layout: 16-byte chunk ch of vector v at ((v/64)*chunks + ch)*1024 + (v%64)*16
    if (blocked) {
        for (int e = tid; e < rows * chunks * 4; e += blockDim.x) {
            const int r = e / (chunks * 4), rem = e % (chunks * 4);
            const int ch = rem >> 2, wq = rem & 3;
            const uint8_t *c = cs_raw + r * ps;
            uint32_t word = 0;
            const int j0 = (ch * 4 + wq) * 10;
            for (int t = 0; t < 10; ++t) {
                const int j = j0 + t;
                if (j < d) word |= (uint32_t)c[j] << (3 * t);
            }
            const int64_t v = base + r0 + r;
            uint8_t *dst = blocked + ((v >> 6) * chunks + ch) * 1024 + (v & 63) * 16;
            reinterpret_cast<uint32_t *>(dst)[wq] = word;
        }
    }
}

// Y = X R^T for a few rows (m <= kSmallRows), with exactly the arithmetic of
// rot_gemm: every output element goes through the same
// v_mfma_f32_16x16x4f32 sequence per 32-wide slab (the same k in the same
// operand slots, sub and step order, from zero), the slab partials are
// folded into float64 in slab order and rounded to float32 at the end, so a
// row rotates to the same bits in either kernel.  The slab partials do not
// depend on each other, so they are computed in parallel: one workgroup per
// 16 x 16 output block, its 16 waves taking every 16th slab with all their
// loads issued at once; the partials meet in LDS and 256 threads fold them
// in order.  For short batches this is a few microseconds of latency (one
// round of loads) instead of 48 dependent slab steps.
constexpr int kSmallRows = 64;
constexpr int SPLIT_WAVES = 16;
constexpr int SPLIT_SLABS = 2048 / KB / SPLIT_WAVES;   // slabs per wave at most

__global__ __launch_bounds__(SPLIT_WAVES * 64) void rot_small_kernel(
    const float *__restrict__ X, int64_t m, int d, const float *__restrict__ R,
    float *__restrict__ Y, int *__restrict__ fill, int nfill, int fill_value) {
    __shared__ f4 part[2048 / KB][64];   // [slab][lane]: the 16 x 16 partial of a slab
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = threadIdx.x; i < nfill; i += SPLIT_WAVES * 64) fill[i] = fill_value;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int l16 = lane & 15;
    const int g4 = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.y * 16;
    const int c0 = blockIdx.x * 16;
    const int64_t gr = r0 + l16;   // the row of X this lane loads
    const bool rowok = gr < m;
    const float *xa = X + (rowok ? gr : 0) * d + g4 * 4;
    const float *rb = R + (int64_t)(c0 + l16) * d + g4 * 4;
    const int nslab = d / KB;
    f4 fa[SPLIT_SLABS][2], fb[SPLIT_SLABS][2];
#pragma unroll
    for (int u = 0; u < SPLIT_SLABS; ++u) {
        const int s = wave + u * SPLIT_WAVES;
        if (s < nslab) {
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) {
                fa[u][sub] = rowok ? *reinterpret_cast<const f4 *>(xa + s * KB + sub * 16)
                                   : f4{0.f, 0.f, 0.f, 0.f};
                fb[u][sub] = *reinterpret_cast<const f4 *>(rb + s * KB + sub * 16);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < SPLIT_SLABS; ++u) {
        const int s = wave + u * SPLIT_WAVES;
        if (s < nslab) {
            f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                for (int st = 0; st < 4; ++st)
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][sub][st], fb[u][sub][st],
                                                               acc, 0, 0, 0);
            part[s][lane] = acc;
        }
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        // output (row g4*4 + v, column l16) of the block: element v of lane (l16, g4)
        const int ln = threadIdx.x & 63;
        const int v = threadIdx.x >> 6;
        double accd = 0.0;
        for (int s = 0; s < nslab; ++s) accd += (double)part[s][ln][v];
        const int64_t row = r0 + (ln >> 4) * 4 + v;
        if (row < m) Y[row * d + c0 + (ln & 15)] = (float)accd;
    }
}

// Y = X R^T for kSmallRows < m <= kMidRows rows, again with exactly the
// arithmetic of rot_gemm (the same products in the same order per output).
// Tiles of 32 x 32 outputs, four waves with a 16 x 16 block each, so that a few
// hundred rows fill the chip: 256 rows at d = 1536 are 384 workgroups instead
// of 24.  Slabs of 32 k come by direct global -> LDS loads into a ring of
// RM_STAGES, five slabs ahead, one barrier per slab.  A 1 KiB piece holds 8
// rows of 8 16-byte quads, quad q of row r at place q ^ r, so that a read of
// one quad of 8 consecutive rows meets distinct banks.
constexpr int kMidRows = 2048;
constexpr int RM_STAGES = 6;
constexpr int RM_STAGE_B = 8 * 1024;     // four pieces of X, four of R

__global__ __launch_bounds__(256) void rot_mid_kernel(const float *__restrict__ X, int64_t m,
                                                      const float *__restrict__ R, int d,
                                                      float *__restrict__ Y) {
    __shared__ __attribute__((aligned(1024))) char stg[RM_STAGES * RM_STAGE_B];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g4 = lane >> 4;
    const int wr = wave >> 1, wc = wave & 1;
    const int64_t row0 = (int64_t)blockIdx.y * 32;
    const int col0 = blockIdx.x * 32;
    const int nslab = d / KB;   // even
    // piece `wave` of X and of R: row 8 wave + lane / 8, quad (lane & 7) ^ (row & 7)
    const int pr = 8 * wave + (lane >> 3), pq = (lane & 7) ^ (lane >> 3);
    const int64_t xr = row0 + pr < m ? row0 + pr : m - 1;   // rows past m feed dropped outputs
    const uint32_t xo = (uint32_t)((xr * d + pq * 4) * 4);
    const uint32_t ro = (uint32_t)(((col0 + pr) * d + pq * 4) * 4);
    const uint32_t stg_lds = (uint32_t)(uintptr_t)stg + wave * 1024;
    int rq = 0, rq_st = 0;      // next slab to request (the last one again past the end), its stage
    auto request = [&]() {
        const int s = rq < nslab ? rq : nslab - 1;
        lds_dma16_s(xo, X + s * KB, stg_lds + rq_st * RM_STAGE_B);
        lds_dma16_s(ro, R + s * KB, stg_lds + rq_st * RM_STAGE_B + 4096);
        ++rq;
        rq_st = rq_st + 1 == RM_STAGES ? 0 : rq_st + 1;
    };
#pragma unroll
    for (int i = 0; i < RM_STAGES - 1; ++i) request();
    // this lane's quads of a slab: row 16 wr (or column 16 wc) + l16, quad 4 sub + g4
    const char *ab = stg + (16 * wr + l16) * 128, *bb = stg + 4096 + (16 * wc + l16) * 128;
    const int q0 = (g4 ^ (l16 & 7)) * 16, q1 = ((4 + g4) ^ (l16 & 7)) * 16;
    double accd[4] = {0.0, 0.0, 0.0, 0.0};
    int st = 0;
    for (int s = 0; s < nslab; ++s) {
        wait_vmem<(RM_STAGES - 2) * 2>();   // slab s, then everyone's
        lds_barrier();                      // ... and every wave is past slab s - 1
        request();                          // slab s + 5, into its stage
        const char *A = ab + st * RM_STAGE_B, *B = bb + st * RM_STAGE_B;
        const f4 a[2] = {*reinterpret_cast<const f4 *>(A + q0), *reinterpret_cast<const f4 *>(A + q1)};
        const f4 b[2] = {*reinterpret_cast<const f4 *>(B + q0), *reinterpret_cast<const f4 *>(B + q1)};
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[sub][t], b[sub][t], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) accd[v] += (double)acc[v];
        st = st + 1 == RM_STAGES ? 0 : st + 1;
    }
    wait_vmem<0>();   // the slabs requested past the end
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int64_t gr = row0 + 16 * wr + 4 * g4 + v;
        if (gr < m) Y[gr * d + col0 + 16 * wc + l16] = (float)accd[v];
    }
}

}  // namespace

// Workspace of a chunk of `rows` rows.
struct EncodeLayout {
    size_t codes, planes, norms, inv, flags, counts, bounds, total;
};
static EncodeLayout encode_layout(int64_t rows, int d) {
    EncodeLayout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += (bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t r = (size_t)((rows + EgLarge::ROWS - 1) / EgLarge::ROWS * EgLarge::ROWS);
    const size_t c = (size_t)((d + BN - 1) / BN * BN);
    L.codes = take(r * (size_t)d);                // unpacked codes
    L.planes = take(r * (size_t)d * 4);           // split rows
    L.norms = take(r * sizeof(double));
    L.inv = take(r * sizeof(float));
    L.flags = take(r * c * sizeof(uint16_t));     // worst case: every coordinate
    L.counts = take(r / EgSmall::SIDE * (c / EgSmall::SIDE) * sizeof(unsigned int));
    L.bounds = take(255 * sizeof(double) + 256 * sizeof(double));   // bounds, cent_sq
    L.total = o;
    return L;
}

// Rows of the next chunk of n: a last chunk of few rows, which would leave
// most compute units idle through five launches (113 us for 1,696 rows at
// d = 1536, 34 a thousand for full ones), joins the one before.
static int64_t chunk_rows(int64_t n, int chunk) {
    return n <= chunk + kEncodeChunkSlack ? n : chunk;
}

// Rows that any chunk of n holds at most.
static int64_t layout_rows(int64_t n, int chunk) {
    return n <= chunk ? n : chunk + kEncodeChunkSlack;
}

size_t encode_workspace_bytes(int64_t n, int d, int chunk) {
    return encode_layout(layout_rows(n, chunk), d).total;
}

size_t split_rotation_bytes(int d) { return (size_t)d * d * 4; }

hipError_t split_rotation(const float *R, int d, void *planes, hipStream_t stream) {
    const int64_t items = (int64_t)d * (d / 8);
    hipLaunchKernelGGL(split_rotation_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, stream, R, d,
                       static_cast<uint4 *>(planes));
    return hipGetLastError();
}

// Outputs of a chunk up to which the small tiles are faster: 257, 1,696 and
// 4,096 rows at d = 1536 take 25, 53 and 106 us with small tiles, 56, 62 and
// 92 with large ones.
constexpr int64_t kEncodeSmallOutputs = 3 << 20;

// The tables of codebooks of up to 16 levels travel as kernel arguments (a
// copy from pageable host memory costs the stream about 10 us each), with
// the status word's reset.
struct SmallTables {
    double bounds[16], cent_sq[16];
};
__global__ void small_tables_kernel(SmallTables t, double *bounds, double *cent_sq, int *status) {
    const int i = threadIdx.x;
    if (i < 16) {
        bounds[i] = t.bounds[i];
        cent_sq[i] = t.cent_sq[i];
    }
    if (i == 0) *status = 0;
}

template <int TM, int TN, int WR, int WC, int ST>
static hipError_t launch_encode_gemm(const uint4 *Xp, int64_t m, const uint4 *Rp, int d, const QuantArgs &qa,
                                     hipStream_t stream) {
    using S = EgShape<TM, TN, WR, WC, ST>;
    static bool attr = false;
    if (!attr) {
        const hipError_t e = hipFuncSetAttribute((const void *)encode_gemm<TM, TN, WR, WC, ST>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::lds);
        if (e != hipSuccess) return e;
        attr = true;
    }
    const int nrt = (int)((m + S::ROWS - 1) / S::ROWS);
    const int ncol = (d + S::COLS - 1) / S::COLS;
    hipLaunchKernelGGL((encode_gemm<TM, TN, WR, WC, ST>), dim3((nrt + 7) / 8 * 8 * ncol), dim3(S::THREADS), S::lds,
                       stream, Xp, m, Rp, d, nrt, qa);
    return hipGetLastError();
}

hipError_t encode_rows(const float *X, int64_t n, int d, const float *R, const void *Rsplit,
                       const CodebookDev &cb, const EncodeOut &out, void *ws,
                       int *status_dev, hipStream_t stream, int chunk, const CalibDev &calib) {
    const EncodeLayout L = encode_layout(layout_rows(n, chunk), d);
    uint8_t *p = static_cast<uint8_t *>(ws);
    uint8_t *codes_tmp = p + L.codes;
    uint4 *planes = reinterpret_cast<uint4 *>(p + L.planes);
    double *norms = reinterpret_cast<double *>(p + L.norms);
    float *inv = reinterpret_cast<float *>(p + L.inv);
    uint16_t *flags = reinterpret_cast<uint16_t *>(p + L.flags);
    unsigned int *tile_count = reinterpret_cast<unsigned int *>(p + L.counts);
    double *bounds = reinterpret_cast<double *>(p + L.bounds);
    double *cent_sq = bounds + 255;

    hipError_t e;
    if (cb.levels <= 16) {
        SmallTables t{};
        std::copy(cb.bounds, cb.bounds + cb.levels - 1, t.bounds);
        std::copy(cb.cent_sq, cb.cent_sq + cb.levels, t.cent_sq);
        hipLaunchKernelGGL(small_tables_kernel, dim3(1), dim3(64), 0, stream, t, bounds, cent_sq, status_dev);
        e = hipGetLastError();
    } else {
        e = hipMemsetAsync(status_dev, 0, sizeof(int), stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(bounds, cb.bounds, sizeof(double) * (cb.levels - 1), hipMemcpyHostToDevice, stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(cent_sq, cb.cent_sq, sizeof(double) * cb.levels, hipMemcpyHostToDevice, stream);
    }
    if (e != hipSuccess) return e;

    const int chunks = chunks_per_vector(d, cb.bits);
    const size_t split_lds = (size_t)SR_ROWS * (d + 4) * sizeof(float);
    static bool attr = false;
    if (!attr) {
        e = hipFuncSetAttribute((const void *)split_rows_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                SR_ROWS * (2048 + 4) * (int)sizeof(float));
        if (e != hipSuccess) return e;
        attr = true;
    }
    for (int64_t r0 = 0, m; r0 < n; r0 += m) {
        m = chunk_rows(n - r0, chunk);
        // every list tile of the chunk's rows gets its flag count
        QuantArgs qa{bounds, calib.athr, cb.levels, codes_tmp, inv, (float)tau_rel(d),
                     (cb.bounds[cb.levels - 2] - cb.bounds[0]) / EG_BINS, flags, tile_count};
        hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)((m + 31) / 32 * (32 / SR_ROWS))), dim3(SR_THREADS),
                           split_lds, stream, X + r0 * d, m, d, planes, norms, inv, status_dev);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        const bool large = m * (int64_t)d > kEncodeSmallOutputs;
        const int side = large ? EgLarge::SIDE : EgSmall::SIDE;
        const uint4 *Rp = static_cast<const uint4 *>(Rsplit);
        e = large ? launch_encode_gemm<2, 2, 2, 2, 4>(planes, m, Rp, d, qa, stream)
                  : launch_encode_gemm<1, 1, 2, 2, 6>(planes, m, Rp, d, qa, stream);
        if (e != hipSuccess) return e;
        const int ncol = (d + side - 1) / side;
        const int nrow = (int)((m + side - 1) / side);
        // 8-bit codes flag about 3% of coordinates (thresholds ~4e-4 apart
        // at d = 1536): tiles then share their staged rows
        if (cb.levels > 16)
            hipLaunchKernelGGL(fixup_tile_kernel, dim3(nrow * ncol), dim3(GEMM_THREADS), 0, stream,
                               X + r0 * d, m, R, d, side, ncol, bounds, calib.athr, cb.levels, norms,
                               flags, tile_count, codes_tmp);
        else
            hipLaunchKernelGGL(fixup_flag_kernel, dim3((nrow + 7) / 8 * 8 * ncol), dim3(FX_WAVES * 64), 0, stream,
                               X + r0 * d, R, d, side, nrow, ncol, bounds, calib.athr, cb.levels, norms, flags, tile_count,
                               codes_tmp);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        uint8_t *canon_p = out.canonical ? out.canonical + r0 * (int64_t)(d * cb.bits / 8) : nullptr;
        float *scales_p = out.scales ? out.scales + r0 : nullptr;
        const dim3 prow((unsigned)((m + PR_ROWS - 1) / PR_ROWS));
        if (cb.bits == 3) {
            const int packs = (int)((m + PACK_ROWS - 1) / PACK_ROWS);
            hipLaunchKernelGGL(pack_kernel, dim3(packs), dim3(256), PACK_ROWS * (d + 16), stream,
                               codes_tmp, X + r0 * d, m, d, cent_sq, calib.ysq, norms, canon_p, scales_p,
                               out.blocked, out.blocked_scales, out.base + r0, chunks);
        } else if (cb.bits == 1) {
            hipLaunchKernelGGL(pack_rows_kernel<1>, prow, dim3(256), 0, stream, codes_tmp, X + r0 * d, m, d, cent_sq,
                               calib.ysq, norms, canon_p, scales_p, out.blocked, out.blocked_scales,
                               out.base + r0, chunks);
        } else if (cb.bits == 2) {
            hipLaunchKernelGGL(pack_rows_kernel<2>, prow, dim3(256), 0, stream, codes_tmp, X + r0 * d, m, d, cent_sq,
                               calib.ysq, norms, canon_p, scales_p, out.blocked, out.blocked_scales,
                               out.base + r0, chunks);
        } else if (cb.bits == 4) {
            hipLaunchKernelGGL(pack_rows_kernel<4>, prow, dim3(256), 0, stream, codes_tmp, X + r0 * d, m, d, cent_sq,
                               calib.ysq, norms, canon_p, scales_p, out.blocked, out.blocked_scales,
                               out.base + r0, chunks);
        } else {
            hipLaunchKernelGGL(pack_rows_kernel<8>, prow, dim3(256), 0, stream, codes_tmp, X + r0 * d, m, d, cent_sq,
                               calib.ysq, norms, canon_p, scales_p, out.blocked, out.blocked_scales,
                               out.base + r0, chunks);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

__global__ void fill_ints(int *p, int64_t n, int v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t rotate_rows_f32(const float *X, int64_t m, int d, const float *R, float *Y,
                           hipStream_t stream, int *fill, int64_t nfill, int fill_value) {
    if (!fill) nfill = 0;
    if (m > 0 && m <= kSmallRows && nfill <= kSmallRows) {
        const dim3 grid((unsigned)(d / 16), (unsigned)((m + 15) / 16));
        hipLaunchKernelGGL(rot_small_kernel, grid, dim3(SPLIT_WAVES * 64), 0, stream, X, m, d, R, Y,
                           fill, (int)nfill, fill_value);
        return hipGetLastError();
    }
    if (nfill > 0) {
        hipLaunchKernelGGL(fill_ints, dim3(1), dim3(256), 0, stream, fill, nfill, fill_value);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (m <= 0) return hipSuccess;
    // the direct loads into LDS want rows on 16-byte boundaries (d is a multiple
    // of 64); rows elsewhere take the ordinary loads of rot_gemm
    if (m <= kMidRows && (reinterpret_cast<uintptr_t>(X) & 15) == 0) {
        hipLaunchKernelGGL(rot_mid_kernel, dim3((unsigned)(d / 32), (unsigned)((m + 31) / 32)), dim3(256), 0,
                           stream, X, m, R, d, Y);
        return hipGetLastError();
    }
    const int ncol = (d + BN - 1) / BN;
    const int nrt = (int)((m + BM - 1) / BM);
    const int groups = (nrt + 7) / 8;
    hipLaunchKernelGGL(rot_gemm, dim3(groups * 8 * ncol), dim3(GEMM_THREADS), 0, stream, X, m, R,
                       d, nrt, Y);
    return hipGetLastError();
}

}  // namespace tq
