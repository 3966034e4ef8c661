// Batched search on the matrix cores (section II-B step 5 for a tile of
// queries at once, with the filter of section III-B).
//
// Per tile of up to 32 queries:
//  1. prep_kernel: q' scaled by a power of two and rounded to float16, with
//     the per-query constants below.
//  2. mfma_scores_kernel: one pass over the code store.  Each 16-byte chunk
//     of 64 vectors (32 coordinates each) is turned into float16 centroid
//     values and multiplied with the query tile on v_mfma_f32_16x16x32_f16;
//     after a block's last chunk the approximate scores s_v <c_hat, q'> are
//     written, scaled to a float16 range, as a [query][vector] matrix, and
//     each query's largest score in the block as a [query][block] matrix.
//  3. Selection of at most KC candidates per query (KC = eight per result,
//     64 to 512) with a bound amin on the approximate score of every other
//     vector.  Unfiltered: block_select_kernel.  The R-th largest block
//     maximum (R = KC - 32) is a score of R distinct vectors, so at least R
//     vectors reach it, and every vector that does lies in a block whose
//     maximum reaches it: a radix selection over the block maxima lists
//     those blocks, and their vectors that reach it are the candidates
//     (about R when vectors sit at random positions; if more than KC, a
//     radix selection over the listed scores keeps the KC best).
//     Filtered: filter_kernel lists the blocks that some query of the tile
//     may need (tenant summary against the union of the allowlists, live
//     slots) and turns the allowlists into a bit mask over the tile's queries
//     per tenant; only listed blocks are read, and a vector that a query may
//     not return scores -inf for it.
//  4. rescore_kernel: the exact score of each candidate with the
//     single-query scan's integer table (bit-identical scores), the top k of
//     them, and a certificate: with E a rigorous bound on |approximate -
//     exact| for every vector, a vector outside the candidates scores at
//     most amin + E; if that is below the k-th exact score the top k is
//     proven, otherwise the query's row joins the device list of queries
//     that the single-query scan, launched behind the batched kernels,
//     answers (it leaves at once when the list is empty: no host round trip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "kernels.h"
#include "lds_dma.h"
#include "lut.h"
#include "stream.h"
#include "topk.h"

namespace tq {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int kTile = 32;          // queries per pass over the codes: two MFMA row tiles of 16
constexpr int kCandMax = 512;      // candidates per query kept for exact rescoring (KC <= this)
constexpr int kCandMin = 64;
constexpr int kMaxBatchK = 256;    // largest k of the batched path
constexpr int BS_THREADS = 1024;   // block_select_kernel
constexpr int BS_WAVES = BS_THREADS / 64;
constexpr int kListMaxB = 8192;    // blocks a query's selection may list
constexpr int kHistCopies = 4;     // histogram copies (lane & 3), against atomic conflicts
constexpr int kHistStride = 257;   // words between copies: copies in different banks
// Selection outcome per query.
constexpr int kSelBound = 0;       // candidates + a bound amin on every other vector
constexpr int kSelOverflow = 1;    // no usable candidates: the query is not certified
constexpr int kSelAll = 2;         // every vector is a candidate
constexpr int MF_THREADS = 768;    // 12 waves: three per SIMD, 168 registers each
constexpr int SEL_THREADS = 256;
constexpr int kTicketStride = 32;  // ints between two workgroups' ticket counters (own 128 B line)
// Last word of a raw buffer resource (stride 0, byte offsets): 32-bit data
// format, so untyped loads, stores and atomics are bounds-checked by bytes.
constexpr int kBufferWord3 = 0x00020000;
constexpr int kKeepVmemB = 0x1 | 0x2 | 0x4 | 0x8 | 0x80 | 0x100 | 0x200 | 0x400;

// fn(std::integral_constant<int, i>) for i = 0 .. N-1.
template <int N, class Fn, int... I>
__device__ inline void static_for_impl(Fn &&fn, std::integer_sequence<int, I...>) {
    (fn(std::integral_constant<int, I>()), ...);
}
template <int N, class Fn>
__device__ inline void static_for(Fn &&fn) {
    static_for_impl<N>(fn, std::make_integer_sequence<int, N>());
}

// Per-query constants written by prep_kernel.
struct QInfo {
    float f;      // stored approximate score = s_v (acc f + c) (acc: MFMA sum of the scaled query)
    float norm;   // approximate score = stored * norm  (s_max ||q'||_2)
    float err;    // bound on |approximate - exact| before the float16 storage
    float c;      // TQ+ constant term / norm (0 without calibration)
};

// ------------------------------------------------------------------- prep
// The query is scaled by alpha = 2^e with max|alpha q'_j| in [2^14, 2^15)
// and rounded to float16: alpha q'_j + eps_j.  With the float16 centroids
// c_l + delta_l (|delta_l| <= dmax, |c_l + delta_l| <= cmax16), the MFMA sum
// is alpha sum_j c q'_j + sum_j (alpha delta q'_j + (c + delta) eps_j), so
//   |acc / alpha - <c, q'>| <= dmax ||q'||_1 + cmax16 ||eps||_1 / alpha
// plus the float32 accumulation of d products in any order,
//   gamma_d cmax16 (||q'||_1 + ||eps||_1 / alpha),  gamma_d = d u / (1 - d u),
// u = 2^-24, and a few float32 roundings when scaling and adding the
// constant term C (4 * 2^-23 of the same magnitude and of |C|).
// The exact score of b <= 4 (the integer tables of lut.h, at most d rows)
// differs from s_v (<c, q'> + C) by the table's rounding: each entry is
// within 1/2 unit plus 2 * 2^-24 of its products, the constant within 1/2
// unit, the integer sum is exact, and its float conversion and the product
// with s_v add 2^-24 each.  The table builder picks 2^sh > (2^31 - 1 - 2d) /
// (2 B'), B' = (cmax tot + |C|) (1 + 1e-5) with tot its float sum of |q'_j|
// (within 1e-6 of ||q'||_1), so the (d + 1)/2 units are below rho (cmax
// ||q'||_1 + |C|) in score units, rho = (d + 1) (1 + 2e-5) / (2^31 - 1 - 2d);
// with the 2^-24 terms the exact score is within (rho + 8 * 2^-24) s_v (cmax
// ||q'||_1 + |C|) of s_v (<c, q'> + C) (cmax <= cmax16 (1 + 2^-10): float16
// rounding moves a value by at most 2^-11 of it).  At b = 8 the exact score
// is a float32 sum of d products from C on: gamma_{d+8} takes rho's place.
// The sum of all terms times s_max is the error before storage (the factor
// 1.1 is margin only); the float16 storage of the approximate score adds at
// most 2^-11 of its magnitude plus 2^-25 norm, accounted for where the
// certificate is checked.  Relative errors say nothing about subnormal
// results: a query whose norm is not within 2^+-100 (and not 0, where every
// score is the exact 0 or s_v C) has an infinite bound, proves nothing and is
// answered by the scan.
__global__ void prep_kernel(const float *__restrict__ Q, const float *__restrict__ qconst, int nq,
                            int d, int bits, const float *smax_p,
                            float cmax16, float dmax, _Float16 *__restrict__ q16,
                            QInfo *__restrict__ info, int *__restrict__ zero, int nzero,
                            int *__restrict__ zero1) {
    __shared__ float red_m[SEL_THREADS / 64];
    __shared__ double red_1[SEL_THREADS / 64], red_2[SEL_THREADS / 64];
    const int q = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (q == 0) {
        for (int i = tid; i < nzero; i += SEL_THREADS) zero[i] = 0;   // the score kernel's tickets
        if (zero1 && tid == 0) *zero1 = 0;                            // the search's uncertified count
    }
    const float *row = Q + (int64_t)q * d;
    float m = 0.f;
    double s1 = 0.0, s2 = 0.0;
    for (int j = tid; j < d; j += SEL_THREADS) {
        const float v = row[j];
        m = fmaxf(m, fabsf(v));
        s1 += fabs((double)v);
        s2 += (double)v * v;
    }
    for (int o = 32; o > 0; o >>= 1) {
        m = fmaxf(m, __shfl_xor(m, o, 64));
        s1 += __shfl_xor(s1, o, 64);
        s2 += __shfl_xor(s2, o, 64);
    }
    if (lane == 0) {
        red_m[wave] = m;
        red_1[wave] = s1;
        red_2[wave] = s2;
    }
    __syncthreads();
    m = 0.f;
    s1 = 0.0;
    s2 = 0.0;
    for (int w = 0; w < SEL_THREADS / 64; ++w) {
        m = fmaxf(m, red_m[w]);
        s1 += red_1[w];
        s2 += red_2[w];
    }
    __syncthreads();   // red_1 is reused below
    const int e = m > 0.f ? 14 - ilogbf(m) : 0;
    const float alpha = ldexpf(1.0f, e);
    double se = 0.0;   // ||eps||_1
    for (int j = tid; j < d; j += SEL_THREADS) {
        const float a = row[j] * alpha;   // exact: alpha is a power of two
        const _Float16 h = (_Float16)a;
        q16[(int64_t)q * d + j] = h;
        se += fabs((double)(float)h - (double)a);
    }
    for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o, 64);
    if (lane == 0) red_1[wave] = se;
    __syncthreads();
    if (tid == 0) {
        se = 0.0;
        for (int w = 0; w < SEL_THREADS / 64; ++w) se += red_1[w];
        const double smax = (double)*smax_p;
        double norm = smax * sqrt(s2);
        // Below and above these the bounds do not hold as derived: subnormal
        // scores are rounded to multiples of 2^-149, largest ones overflow
        const bool in_range = norm == 0.0 || (norm >= ldexp(1.0, -100) && norm <= ldexp(1.0, 100));
        if (!(norm > 0.0)) norm = 1.0;
        const double u = ldexp(1.0, -24);
        const double gd = d * u / (1.0 - d * u);
        const double mag = (double)cmax16 * (s1 + se / alpha);
        const double rho = (d + 1) * (1.0 + 2e-5) / (2147483647.0 - 2.0 * d);
        const double gx = (d + 8) * u / (1.0 - (d + 8) * u);
        const double C = qconst ? (double)qconst[q] : 0.0;
        const double tab = ((bits == 8 ? gx : rho) + 8 * u) *
                           ((double)cmax16 * (1.0 + ldexp(1.0, -10)) * s1 + fabs(C));
        const double E = (double)dmax * s1 + (double)cmax16 * se / alpha + gd * mag +
                         4 * ldexp(1.0, -23) * (mag + fabs(C)) + tab;
        QInfo qi;
        qi.f = (float)(1.0 / ((double)alpha * norm));
        qi.norm = (float)norm;
        qi.err = in_range ? (float)(1.1 * smax * E) : INFINITY;
        qi.c = (float)(C / norm);
        info[q] = qi;
    }
}

// ----------------------------------------------------------------- filters
// Whether the single-query scan answers a pass's queries faster: it skips
// blocks by each query's own allowlist, the batched kernels by the union
// (tiles) or not at all (wide passes).  counts[0]: blocks of the union,
// counts[1]: blocks over all queries, from every kSampleB-th block.  The
// kernels of the pass leave at once then and the rescoring hands every query
// over.  Decided on the device: the host does not know the allowlists.
constexpr int kSampleB = 8;
struct Gate {
    const int *counts;         // null: never
    float scan_us, block_us;   // scan: per query, per block
    float pass_us, read_us;    // batched: per pass, per union block
};
// tile: of the group (counts per tile), nqt: its queries.
__device__ inline bool scan_is_faster(const Gate &g, int tile, int nqt) {
    if (!g.counts) return false;
    const int *c = g.counts + 2 * tile;
    return (float)nqt * g.scan_us + (float)c[1] * (float)kSampleB * g.block_us <
           g.pass_us + (float)c[0] * g.read_us;
}
// The same for query q of a launch of nqt queries in passes of tq queries.
__device__ inline bool scan_is_faster_for(const Gate &g, int q, int nqt, int tq) {
    const int t = q / tq;
    return scan_is_faster(g, t, nqt - t * tq < tq ? nqt - t * tq : tq);
}

struct FilterParams {
    const uint64_t *allow;     // [nqt][W] or null
    const uint64_t *live;      // [nblk] or null
    const uint64_t *summaries; // [nblk][W]
    int64_t nblk;
    int W, nqt;
    int words;                 // 32-query words per tenant
    uint32_t *tmask;           // [64 W][words]: bit q of a tenant's mask: query q admits it
    int *counts;               // see Gate; zero at launch
    int *list;                 // tiles: union blocks (order not fixed), or null
    uint16_t *bmax;            // tiles: [32][nblk], -inf for blocks that are not listed
    // Tile blockIdx.y of a group: its queries and its part of every output.
    __device__ void to_tile(int t) {
        if (allow) allow += (int64_t)t * kTile * W;
        nqt = nqt - t * kTile < kTile ? nqt - t * kTile : kTile;
        tmask += (int64_t)t * 64 * W * words;
        counts += 2 * t;
        list += t * nblk;
        bmax += (int64_t)t * kTile * nblk;
    }
};

// Workgroups of one thread per (tenant, mask word), then of one thread per
// block.  The latter stage the allowlists in LDS, 32 queries at a time
// (their words read one by one from L2 made the kernel 40 us at 1,000
// tenants), and share out the (sampled block, query) tests.
constexpr int FK_THREADS = 256;
constexpr int FK_SAMPLES = FK_THREADS / kSampleB;
__global__ __launch_bounds__(FK_THREADS) void filter_kernel(FilterParams p) {
    __shared__ uint64_t allow_s[32 * 64];            // [query][W] of 32 queries
    __shared__ uint64_t sum_s[FK_SAMPLES * 64];      // [sampled block][W]
    __shared__ unsigned long long any_s[64];         // union of the allowlists (W <= 64)
    const int tid = threadIdx.x, lane = tid & 63, W = p.W;
    if (p.list) p.to_tile(blockIdx.y);
    const int mask_items = 64 * W * p.words;
    const int mask_wgs = (mask_items + FK_THREADS - 1) / FK_THREADS;
    if ((int)blockIdx.x < mask_wgs) {
        const int e = blockIdx.x * FK_THREADS + tid;
        if (e < mask_items) {
            const int t = e / p.words, q0 = e % p.words * 32;
            uint32_t m = p.allow ? 0u : ~0u;
            if (p.allow) {
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    const int q = q0 + i < p.nqt ? q0 + i : 0;
                    const uint64_t a = p.allow[(int64_t)q * W + (t >> 6)] >> (t & 63);
                    m |= q0 + i < p.nqt ? (uint32_t)(a & 1ull) << i : 0u;
                }
            }
            p.tmask[e] = m;
        }
        return;
    }
    const int64_t b0 = (int64_t)(blockIdx.x - mask_wgs) * FK_THREADS;
    const int64_t b = b0 + tid;
    bool hit = b < p.nblk && (!p.live || p.live[b] != 0);
    int sum = 0;
    if (!p.allow) {
        sum = hit && b % kSampleB == 0 ? p.nqt : 0;
    } else {
        // summaries of the sampled blocks (b0 + kSampleB i), zero where dead
        for (int e = tid; e < FK_SAMPLES * W; e += FK_THREADS) {
            const int64_t sb = b0 + kSampleB * (e / W);
            const bool in = sb < p.nblk && (!p.live || p.live[sb] != 0);
            sum_s[e] = in ? p.summaries[sb * W + e % W] : 0ull;
        }
        if (tid < 64) any_s[tid] = 0;
        for (int q0 = 0; q0 < p.nqt; q0 += 32) {
            const int nq = p.nqt - q0 < 32 ? p.nqt - q0 : 32;
            __syncthreads();   // the previous queries' rows have been read
            for (int e = tid; e < nq * W; e += FK_THREADS) {
                const uint64_t a = p.allow[(int64_t)q0 * W + e];
                allow_s[e] = a;
                if (a) atomicOr(&any_s[e % W], (unsigned long long)a);
            }
            __syncthreads();
            for (int e = tid; e < FK_SAMPLES * nq; e += FK_THREADS) {
                const uint64_t *sm = sum_s + e / nq * W, *al = allow_s + e % nq * W;
                bool h = false;
                for (int w = 0; w < W; ++w) h |= (sm[w] & al[w]) != 0;
                sum += h;
            }
        }
        if (hit) {
            const uint64_t *sm = p.summaries + b * W;
            hit = false;
            for (int w = 0; w < W; ++w) hit |= (sm[w] & any_s[w]) != 0;
        }
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    const uint64_t m = __ballot(hit);
    int at = 0;
    if (lane == 0) {
        if (sum) atomicAdd(p.counts + 1, sum);
        if (m) at = atomicAdd(p.counts, (int)__popcll(m));
    }
    if (!p.list) return;
    at = __shfl(at, 0, 64);
    if (hit) {
        p.list[at + __popcll(m & ((1ull << lane) - 1))] = (int)b;
    } else if (b < p.nblk) {
        for (int q = 0; q < kTile; ++q) p.bmax[(int64_t)q * p.nblk + b] = 0xFC00u;   // -inf
    }
}

// ------------------------------------------------------------ MFMA scores
struct ScoreParams {
    const uint4 *codes;        // blocked store
    const float *scales;
    const _Float16 *q16;       // [nqt][d]
    const QInfo *info;         // [nqt]
    const float *cents;        // 2^b levels
    _Float16 *out;             // [kTile][npad] approximate scores / norm (rows >= nqt: 0)
    _Float16 *bmax;            // [kTile][nblk] per-block maximum of out (vectors < n)
    int *tickets;              // [workgroup * kTicketStride] block ticket counters, zero at launch
    int64_t n, nblk, npad;
    int d, chunks, nqt;
    int tiles;                 // of the group; the arrays above and below hold one part per tile
    // filtered tiles
    const int *list;           // blocks to score, counts[0] of them
    const int *counts;
    const uint32_t *tmask;     // [tenant] queries that admit it
    const uint16_t *tenants;
    const uint64_t *live;      // [nblk] or null
    int W;
    Gate gate;
    __device__ void to_tile(int t) {
        q16 += (int64_t)t * kTile * d;
        info += t * kTile;
        out += (int64_t)t * kTile * npad;
        bmax += (int64_t)t * kTile * nblk;
        nqt = nqt - t * kTile < kTile ? nqt - t * kTile : kTile;
        list += t * nblk;
        counts += 2 * t;
        tmask += (int64_t)t * 64 * W;
    }
};

// Float16 centroids of the 8 4-bit fields of a stored word w (the canonical
// word rotated left by 2): element t is coordinate t of the word.  The byte
// table holds, for every byte value e, the pair (c[e & 15], c[e >> 4]) as
// two float16 -- one lookup per two coordinates.  It is replicated NR times
// so that the lanes of a read meet distinct LDS banks whatever bytes they
// look up (entry e of replica i is the 32-bit word e * NR + i, read by lane
// i mod NR).
//  NR = 64: the word address e * 256 + 4 * lane has the byte e in byte 1 and
//    the lane's offset `lb` = 4 * lane in byte 0, so one byte permute of the
//    canonical word and lb forms it (64 KiB of table).
//  NR = 32: ((e << 7) | lb), lb = 4 * (lane mod 32), takes a shift or
//    field extract and an and-or per lookup (32 KiB of table).
// The other widths use tables of the same kind: an entry per pair of 2-bit
// codes (16) or of 3-bit codes (64), or per 8-bit code (256, the centroid in
// both halves).
typedef __attribute__((address_space(3))) const uint32_t lds_u32;

// Entry (byte B of w), for w whose bytes are entry numbers.
template <int NR, int B>
__device__ inline uint32_t table_byte(uint32_t w, uint32_t lb) {
    if constexpr (NR == 64) {
        // v_perm selector: byte 0 <- lb byte 0, byte 1 <- w byte B, bytes 2, 3 <- 0
        return *(lds_u32 *)(uintptr_t)__builtin_amdgcn_perm(w, lb, 0x0C0C0400u + (B << 8));
    } else {
        const uint32_t at = B == 0 ? w << 7 : w >> (8 * B - 7);
        return *(lds_u32 *)(uintptr_t)((at & 0x7F80u) | lb);
    }
}
// Entry of the SH / 6-th 6-bit field of w (64 replicas).
template <int SH>
__device__ inline uint32_t table_six(uint32_t w, uint32_t lb) {
    return *(lds_u32 *)(uintptr_t)((__builtin_amdgcn_ubfe(w, SH, 6) << 8) | lb);
}
// Low halves of two 8-bit entries as a pair.
__device__ inline uint32_t pair_of(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, 0x07060100u);   // bytes 0, 1 of a, bytes 2, 3 of b
}

union Half8 {
    uint32_t u[4];
    half8 h;
};

template <int NR>
__device__ inline half8 dequant8_canonical(uint32_t cw, uint32_t lb) {
    Half8 r;
    r.u[0] = table_byte<NR, 0>(cw, lb);
    r.u[1] = table_byte<NR, 1>(cw, lb);
    r.u[2] = table_byte<NR, 2>(cw, lb);
    r.u[3] = table_byte<NR, 3>(cw, lb);
    return r.h;
}
template <int NR>
__device__ inline half8 dequant8(uint32_t w, uint32_t lb) {
    return dequant8_canonical<NR>(__builtin_amdgcn_alignbit(w, w, 2), lb);   // canonical word
}

// How the codes of one width are fed to the MFMAs (k = 32 per step).  The
// lane exchanges leave lane row kq of a chunk with word kq of its vector;
// U consecutive chunks give the lane U words, and ST steps of 8 of their
// codes.  coord(u, st, kq, t): the coordinate that step st of unit u takes
// in slot t of lane row kq (the queries are laid out alike).
template <int BITS> struct Feed;
template <> struct Feed<4> {
    static constexpr int U = 1, ST = 1, ENTRIES = 256;
    __host__ __device__ static int coord(int u, int, int kq, int t) { return 32 * u + 8 * kq + t; }
};
template <> struct Feed<2> {
    static constexpr int U = 1, ST = 2, ENTRIES = 16;
    __host__ __device__ static int coord(int u, int st, int kq, int t) {
        return 64 * u + 16 * kq + 8 * st + t;
    }
};
template <> struct Feed<8> {
    static constexpr int U = 2, ST = 1, ENTRIES = 256;
    __host__ __device__ static int coord(int u, int, int kq, int t) {
        return 32 * u + 16 * (t >> 2) + 4 * kq + (t & 3);
    }
};
// b = 3: ten codes per word, 40 per chunk; the lane's four words hold 20
// pairs, four to a step (coordinates past d are zero in the queries).
template <> struct Feed<3> {
    static constexpr int U = 4, ST = 5, ENTRIES = 64;
    __host__ __device__ static int coord(int u, int st, int kq, int t) {
        const int p = 4 * st + (t >> 1);
        return 160 * u + 40 * (p / 5) + 10 * kq + 2 * (p % 5) + (t & 1);
    }
};
template <int BITS>
__device__ inline uint32_t table_entry(const float *cents, int e) {
    constexpr int M = (1 << BITS) - 1;
    const float lo = cents[e & M], hi = BITS == 8 ? lo : cents[e >> BITS & M];
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)lo) |
           (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)hi) << 16;
}
// B operand of step st from the lane's U words (w[0..U-1], as stored).
template <int BITS, int NR, int ST>
__device__ inline half8 feed_operand(const uint32_t *w, uint32_t lb) {
    if constexpr (BITS == 4) {
        return dequant8<NR>(w[0], lb);
    } else if constexpr (BITS == 2) {
        const uint32_t cw = __builtin_amdgcn_alignbit(w[0], w[0], 2);
        const uint32_t lo = cw & 0x0F0F0F0Fu, hi = (cw >> 4) & 0x0F0F0F0Fu;
        Half8 r;
        r.u[0] = table_byte<NR, 2 * ST>(lo, lb);
        r.u[1] = table_byte<NR, 2 * ST>(hi, lb);
        r.u[2] = table_byte<NR, 2 * ST + 1>(lo, lb);
        r.u[3] = table_byte<NR, 2 * ST + 1>(hi, lb);
        return r.h;
    } else if constexpr (BITS == 8) {
        Half8 r;
        r.u[0] = pair_of(table_byte<NR, 0>(w[0], lb), table_byte<NR, 1>(w[0], lb));
        r.u[1] = pair_of(table_byte<NR, 2>(w[0], lb), table_byte<NR, 3>(w[0], lb));
        r.u[2] = pair_of(table_byte<NR, 0>(w[1], lb), table_byte<NR, 1>(w[1], lb));
        r.u[3] = pair_of(table_byte<NR, 2>(w[1], lb), table_byte<NR, 3>(w[1], lb));
        return r.h;
    } else {
        Half8 r;
        r.u[0] = table_six<(4 * ST + 0) % 5 * 6>(w[(4 * ST + 0) / 5], lb);
        r.u[1] = table_six<(4 * ST + 1) % 5 * 6>(w[(4 * ST + 1) / 5], lb);
        r.u[2] = table_six<(4 * ST + 2) % 5 * 6>(w[(4 * ST + 2) / 5], lb);
        r.u[3] = table_six<(4 * ST + 3) % 5 * 6>(w[(4 * ST + 3) / 5], lb);
        return r.h;
    }
}
// Steps of a vector of `chunks` chunks.
__host__ __device__ constexpr int feed_steps(int bits, int chunks) {
    return bits == 4 ? chunks : bits == 2 ? 2 * chunks : bits == 8 ? chunks / 2 : chunks / 4 * 5;
}
__host__ __device__ constexpr int feed_entries(int bits) { return bits == 2 ? 16 : bits == 3 ? 64 : 256; }

// Copies of a ring slot's four words into registers of their own.  The
// exchanges below overwrite their operands in place; on the slot itself they
// make the register allocator move the slot's refill into other registers
// and copy it back at the loop's back edge, which waits for every load in
// flight (the ring drains once per eight chunks).  An opaque copy frees the
// slot for its refill at once.
__device__ inline void copy4(const uint4 &v, uint32_t &a, uint32_t &b, uint32_t &c, uint32_t &d) {
    asm volatile("v_mov_b32 %0, %4\n\tv_mov_b32 %1, %5\n\tv_mov_b32 %2, %6\n\tv_mov_b32 %3, %7"
                 : "=v"(a), "=v"(b), "=v"(c), "=v"(d)
                 : "v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w));
}

// Replicas of the score kernel's table: 64 where the table (64 KiB at b = 4
// and 8) and the query tile (2 KiB a step) fit the 160 KiB of LDS together.
// At b = 2 and 3 the table leaves room for the queries' factors in LDS; the
// feeds of these widths leave no registers for them.
__host__ __device__ constexpr bool factors_in_lds(int bits) { return bits == 2 || bits == 3; }
__host__ __device__ constexpr size_t score_lds(int bits, int chunks, int nr) {
    return (size_t)feed_entries(bits) * nr * 4 + (size_t)feed_steps(bits, chunks) * 2048 +
           (factors_in_lds(bits) ? 2 * kTile * 4 : 0);
}
__host__ __device__ constexpr int score_replicas(int bits, int chunks) {
    return score_lds(bits, chunks, 64) <= 160 * 1024 ? 64 : 32;
}

// One workgroup of 12 waves per compute unit.  The table and the query
// tile stay in LDS; the tile is stored in the A-operand order of the MFMAs
// (step, row tile t: 64 lanes x 16 bytes, lane 16 kq + i holding row
// 16 t + i, slots 0..7 of lane row kq), so each operand read is one 16-byte
// read per lane at consecutive addresses.  Waves claim the workgroup's
// 64-vector blocks one at a time from the workgroup's ticket counter in
// memory (one ahead, so the ring of RING chunk loads runs on into the next
// block; RING = 4 for chunk counts that 8 does not divide).  The kernel is
// bound by the code stream: 1,000,000 vectors at d = 1536 and 4 bits take
// 152 to 178 us, 4.3 to 5.1 TB/s, whatever the number of queries in the tile.
// FILT: the blocks of p.list, with the tile's allowlists and the live slots
// applied to the stored scores.  A block's tenant ids are loaded a block
// ahead and its query masks at its start, so neither wait drains the ring.
template <int BITS, int NR, int RING, bool FILT>
__global__ __launch_bounds__(MF_THREADS) void mfma_scores_kernel(ScoreParams p) {
    using F = Feed<BITS>;
    static_assert(RING % F::U == 0 && (RING == 4 || RING == 8), "whole units in the ring");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint32_t *T = reinterpret_cast<uint32_t *>(smem);                               // table, at 0
    uint4 *Qf = reinterpret_cast<uint4 *>(smem + (size_t)NR * F::ENTRIES * 4);      // [step][2][64]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // G workgroups per tile; the tiles' workgroups of one share of the codes
    // are 8 apart, on one XCD, where G allows
    const int G = gridDim.x / p.tiles;
    int g = blockIdx.x / p.tiles, tile = blockIdx.x % p.tiles;
    if (G % 8 == 0) {
        const int r = blockIdx.x >> 3;
        tile = r % p.tiles;
        g = r / p.tiles * 8 + (blockIdx.x & 7);
    }
    p.to_tile(tile);
    const int CH = p.chunks;   // multiple of RING
    if (FILT && scan_is_faster(p.gate, tile, p.nqt)) return;
    const int64_t nb = FILT ? (int64_t)*p.counts : p.nblk;
    const int64_t gb0 = nb * g / G, gb1 = nb * (g + 1) / G;
    const int nbw = (int)(gb1 - gb0);
    if (FILT && nbw == 0) return;
    // the block of this workgroup's share entry i (scalar loads of the list)
    typedef const __attribute__((address_space(4))) int *const_int;
    typedef const __attribute__((address_space(4))) uint64_t *const_u64;
    auto block_of = [&](int i) -> int64_t {
        if constexpr (FILT) return ((const_int)(uintptr_t)p.list)[gb0 + i];
        else return gb0 + i;
    };

    // query tile in operand order, zero rows past nqt
    for (int e = tid; e < feed_steps(BITS, CH) * 128; e += MF_THREADS) {
        const int st = e >> 7, t = (e >> 6) & 1, l = e & 63;
        const int r = 16 * t + (l & 15), kq = l >> 4;
        union {
            uint4 v;
            _Float16 h[8];
            uint2 w[2];
        } q;
        q.v = make_uint4(0, 0, 0, 0);
        if (r < p.nqt) {
            const _Float16 *row = p.q16 + (int64_t)r * p.d;
            const int u = st / F::ST, sub = st % F::ST;
            if constexpr (BITS == 8) {
                q.w[0] = *reinterpret_cast<const uint2 *>(row + F::coord(u, sub, kq, 0));
                q.w[1] = *reinterpret_cast<const uint2 *>(row + F::coord(u, sub, kq, 4));
            } else if constexpr (BITS == 3) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int j = F::coord(u, sub, kq, i);
                    q.h[i] = j < p.d ? row[j] : (_Float16)0.f;
                }
            } else {
                q.v = *reinterpret_cast<const uint4 *>(row + F::coord(u, sub, kq, 0));
            }
        }
        Qf[e] = q.v;
    }
    for (int e = tid; e < F::ENTRIES * NR; e += MF_THREADS)
        T[e] = table_entry<BITS>(p.cents, e / NR);   // e % NR is the replica
    const uint32_t lb = (uint32_t)(lane & (NR - 1)) * 4;
    // per-lane query factors: tile t, rows 4*(lane/16) + r
    constexpr bool FL = factors_in_lds(BITS);
    float qf[2][4], qc[2][4];
    float *fl = reinterpret_cast<float *>(Qf + feed_steps(BITS, CH) * 128);   // [2][32]: f, c
    if constexpr (FL) {
        if (tid < kTile) {
            const QInfo qi = p.info[tid < p.nqt ? tid : 0];
            fl[tid] = tid < p.nqt ? qi.f : 0.f;
            fl[kTile + tid] = tid < p.nqt ? qi.c : 0.f;
        }
    } else {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int q = 16 * t + 4 * (lane >> 4) + r;
                const QInfo qi = p.info[q < p.nqt ? q : 0];
                qf[t][r] = q < p.nqt ? qi.f : 0.f;
                qc[t][r] = q < p.nqt ? qi.c : 0.f;
            }
    }
    __syncthreads();

    // The ticket is a buffer atomic issued by every lane, of which only lane
    // 0's lies inside the 4-byte buffer: bounds checking drops the others'
    // adds (their value is 0).  An atomic under a branch on lane 0 instead
    // leaves the wait-count pass unsure of the loads in flight, and it then
    // drains the chunk ring inside the chunk loop.
    const __amdgpu_buffer_rsrc_t trs =
        __builtin_amdgcn_make_buffer_rsrc(p.tickets + (tile * G + g) * kTicketStride, 0, 4, kBufferWord3);
    auto take = [&]() {
        return __builtin_amdgcn_raw_ptr_buffer_atomic_add_i32(1, trs, lane == 0 ? 0 : 4, 0, 0);
    };
    int cur = __builtin_amdgcn_readfirstlane(take());
    if (cur >= nbw) return;
    int nxt = __builtin_amdgcn_readfirstlane(take());
    int64_t blk = block_of(cur);
    const uint4 *bsrc = p.codes + blk * CH * 64;   // uniform: the block's chunk 0
    const int qrow = lane & 15, kq = lane >> 4;
    int ten[4] = {0, 0, 0, 0};   // filtered: tenants of the current block's vectors 16m + qrow
    auto load_tenants = [&](int64_t b) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int64_t v = b * 64 + 16 * m + qrow;
            ten[m] = p.tenants[v < p.n ? v : 0];
        }
    };
    if (FILT) load_tenants(blk);
    // the ring: named registers (an array would end up in scratch)
    uint4 rb0, rb1, rb2, rb3, rb4, rb5, rb6, rb7;
    auto ring = [&](auto I) -> uint4 & {
        constexpr int i = decltype(I)::value;
        if constexpr (i == 0) return rb0;
        else if constexpr (i == 1) return rb1;
        else if constexpr (i == 2) return rb2;
        else if constexpr (i == 3) return rb3;
        else if constexpr (i == 4) return rb4;
        else if constexpr (i == 5) return rb5;
        else if constexpr (i == 6) return rb6;
        else return rb7;
    };
    static_for<RING>([&](auto I) {
        ring(I) = load_stream(bsrc + decltype(I)::value * 64 + lane);
        __builtin_amdgcn_sched_barrier(kKeepVmemB);
    });
    const uint4 *qa = Qf + lane;
    // a wave scores at most the workgroup's nbw blocks: the bound ends the
    // loop even if the tickets were to stop advancing
    for (int iter = 1;; ++iter) {
        // the block after this one (or this one again past the end: cache hits)
        const int64_t nblk_ = nxt < nbw ? block_of(nxt) : blk;
        const uint4 *nsrc = p.codes + nblk_ * CH * 64;
        const int ticket = take();
        uint32_t ok[4] = {0u, 0u, 0u, 0u};   // filtered: queries that may return vector 16m + qrow
        if constexpr (FILT) {
#pragma unroll
            for (int m = 0; m < 4; ++m) ok[m] = p.tmask[ten[m]];
            load_tenants(nblk_);
        }
        // unconditional loads (clamped index): a load under a branch makes the
        // wait-count pass drain the chunk ring in the loop below
        float scl[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int64_t v = blk * 64 + 16 * m + qrow;
            scl[m] = p.scales[v < p.n ? v : 0];
        }
        float4v acc[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int m = 0; m < 4; ++m) acc[t][m] = float4v{0.f, 0.f, 0.f, 0.f};
        // one unit of U chunks from c on, in ring slots I, I + 1, ...; the
        // ring index is a compile-time constant at every call
        auto unit = [&](const int c, auto I) {
            constexpr int i0 = decltype(I)::value;
            uint32_t w[4][F::U];   // [m][chunk]: this lane row's words of vector 16m + i
            static_for<F::U>([&](auto J) {
                constexpr int j = decltype(J)::value;
                uint4 &slot = ring(std::integral_constant<int, i0 + j>());
                // W_q (row m) = word q of vector 16m+i.  permlane32_swap(a, b)
                // exchanges a's rows 2, 3 with b's rows 0, 1; permlane16_swap(a, b)
                // exchanges a's rows 1, 3 with b's rows 0, 2.  After both levels
                // w[m] (row q) = W_q (row m): word q of vectors i, 16+i, 32+i,
                // 48+i in lane 16q+i, the B operands (lane row q, column i) of
                // the four 16-vector MFMAs.  The exchanges work on copies, and
                // the slot is refilled right after the copy.
                uint32_t cx, cy, cz, cw;
                copy4(slot, cx, cy, cz, cw);
                // refill RING chunks ahead: this block, then the next one
                {
                    const int nc = c + j + RING;
                    slot = load_stream((nc < CH ? bsrc + nc * 64 : nsrc + (nc - CH) * 64) + lane);
                    __builtin_amdgcn_sched_barrier(kKeepVmemB);
                }
                const auto s02 = __builtin_amdgcn_permlane32_swap(cx, cz, false, false);
                const auto s13 = __builtin_amdgcn_permlane32_swap(cy, cw, false, false);
                const auto t01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
                const auto t23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
                w[0][j] = t01[0];
                w[1][j] = t01[1];
                w[2][j] = t23[0];
                w[3][j] = t23[1];
            });
            const int s0 = c / F::U * F::ST;
            static_for<F::ST>([&](auto S) {
                constexpr int st = decltype(S)::value;
                const half8 a0 = __builtin_bit_cast(half8, qa[(s0 + st) * 128]);
                const half8 a1 = __builtin_bit_cast(half8, qa[(s0 + st) * 128 + 64]);
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const half8 b = feed_operand<BITS, NR, st>(w[m], lb);
                    acc[0][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, b, acc[0][m], 0, 0, 0);
                    acc[1][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, b, acc[1][m], 0, 0, 0);
                }
            });
        };
        for (int c0 = 0; c0 < CH; c0 += RING)
            static_for<RING / F::U>([&](auto I) {
                constexpr int i = decltype(I)::value * F::U;
                unit(c0 + i, std::integral_constant<int, i>());
            });
        if constexpr (FILT) {
            const uint64_t lv = p.live ? ((const_u64)(uintptr_t)p.live)[blk] : ~0ull;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int64_t v = blk * 64 + 16 * m + qrow;
                const bool may = v < p.n && ((lv >> (16 * m + qrow)) & 1ull);
                ok[m] = may ? ok[m] >> (4 * kq) : 0u;   // bit 16t + r: query 16t + 4kq + r
            }
        }
        // lane holds vectors 16m + qrow, queries 16t + 4*kq + r.  The stores
        // are unconditional (rows past nqt are zero scores in rows that the
        // workspace holds and nothing reads; the 16 lanes of a row store the
        // same block maximum): a store under a branch leaves the wait-count
        // pass unsure of the loads in flight, and it then drains the chunk
        // ring inside the chunk loop.  Stored scores are at least -65504:
        // -inf marks a vector that the query may not return.
        if constexpr (FL) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    qf[t][r] = fl[16 * t + 4 * kq + r];
                    qc[t][r] = fl[kTile + 16 * t + 4 * kq + r];
                }
        }
        float mx[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx[t][r] = -INFINITY;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int64_t v = blk * 64 + 16 * m + qrow;
            const bool vin = v < p.n;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int q = 16 * t + 4 * kq + r;
                    const float a = fmaf(acc[t][m][r], qf[t][r], qc[t][r]) * scl[m];
                    float c = fmaxf(a, -65504.f);
                    if constexpr (FILT) c = (ok[m] >> (16 * t + r)) & 1u ? c : -INFINITY;
                    const _Float16 h = (_Float16)c;
                    p.out[(int64_t)q * p.npad + v] = h;
                    mx[t][r] = fmaxf(mx[t][r], FILT || vin ? (float)h : -INFINITY);
                }
        }
        // block maxima: the 16 lanes of a DPP row hold the block's 64 vectors
        // of the same queries
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float x = mx[t][r];
                x = fmaxf(x, dpp_f<kDppRowRor8>(x));
                x = fmaxf(x, dpp_f<kDppRowRor4>(x));
                x = fmaxf(x, dpp_f<kDppRowRor2>(x));
                x = fmaxf(x, dpp_f<kDppRowRor1>(x));
                const int q = 16 * t + 4 * kq + r;
                p.bmax[(int64_t)q * p.nblk + blk] = (_Float16)x;
            }
        if (nxt >= nbw || iter >= nbw) break;
        blk = nblk_;
        nxt = __builtin_amdgcn_readfirstlane(ticket);
        bsrc = nsrc;
    }
}

// -------------------------------------------------------------- selection
// ------------------------------------------- selection by block maxima
// Order-preserving map of float16 bit patterns onto 16-bit keys.
__device__ inline uint32_t hkey(uint32_t h) { return (h & 0x8000u) ? (~h & 0xFFFFu) : (h | 0x8000u); }
// ... with 0 for -inf, the mark of vectors that the query may not return.
__device__ inline uint32_t present_key(uint32_t h) { return h == 0xFC00u ? 0u : hkey(h); }
__device__ inline float hkey_value(uint32_t key) {
    const uint32_t h = (key & 0x8000u) ? (key & 0x7FFFu) : (~key & 0xFFFFu);
    return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

// Run by one whole wave once the histogram copies of a digit (256 bins) are
// complete: the digit d with (#keys whose digit > d) < K <= (#keys whose
// digit >= d), for 1 <= K <= #keys; out[0] = d, out[1] = #keys whose digit
// > d.  Lane l holds bins 4l .. 4l+3.
__device__ inline void find_digit(const int *hist, int K, int *out) {
    const int lane = threadIdx.x & 63;
    int c[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        int v = 0;
#pragma unroll
        for (int h = 0; h < kHistCopies; ++h) v += hist[h * kHistStride + 4 * lane + j];
        c[j] = v;
    }
    const int s = (c[0] + c[1]) + (c[2] + c[3]);
    int S = s;   // keys in the bins of lanes >= this one
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_down(S, o, 64);
        if (lane + o < 64) S += t;
    }
    const uint64_t ge = __ballot(S >= K);
    const int L = 63 - __builtin_clzll(ge);
    if (lane == L) {
        int above = S - s;
        int d = 4 * lane;
        for (int j = 3; j >= 0; --j) {
            if (above + c[j] >= K) {
                d = 4 * lane + j;
                break;
            }
            above += c[j];
        }
        out[0] = d;
        out[1] = above;
    }
}

struct BlockSelParams {
    const uint16_t *approx;    // [nqt][npad] float16 bit patterns
    const uint16_t *bmax;      // [nqt][nblk]
    int *top_i;                // [nqt][KC] candidate ids (INT_MAX: none)
    float *top_s;              // [nqt][KC] and stored scores
    float *amin;               // [nqt] bound on the approximate score of non-candidates
    int *state;                // [nqt] kSel*
    int64_t n, nblk, npad;
    int KC;
    int nqt;
    Gate gate;
};

// One workgroup per query, as described at the top of the
// file.  Keys are the float16 bit patterns mapped by hkey; a radix
// selection takes the high byte, then the low byte, with LDS histograms.
__global__ __launch_bounds__(BS_THREADS) void block_select_kernel(BlockSelParams p) {
    __shared__ int hist[kHistCopies * kHistStride];
    __shared__ int list[kListMaxB];
    __shared__ int sh[8];
    const int q = blockIdx.x;
    if (scan_is_faster_for(p.gate, q, p.nqt, kTile)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int KC = p.KC, R = KC - 32;
    const uint16_t *bm = p.bmax + (int64_t)q * p.nblk;
    const uint16_t *row = p.approx + (int64_t)q * p.npad;
    int *out_i = p.top_i + (int64_t)q * KC;
    float *out_s = p.top_s + (int64_t)q * KC;
    auto put = [&](int pos, int64_t v, uint32_t key) {
        out_i[pos] = (int)v;
        out_s[pos] = hkey_value(key);
    };
    int *hc = hist + (lane & 3) * kHistStride;
    auto clear_hist = [&]() {
        for (int i = tid; i < kHistCopies * kHistStride; i += BS_THREADS) hist[i] = 0;
    };
    // Visitors of the keys: block maxima (thread t: blocks t + 1024 u) and
    // the scores of the listed blocks (wave w: listed blocks w + 16 u, lane =
    // vector).  Up to BB block keys per thread and LB listed-block keys per
    // lane stay in registers across the passes (one round of loads); beyond
    // that the keys are loaded again, in rounds of RB, for every pass.
    // A round's loads are unconditional, from clamped indices, and all
    // issued before any is used (the empty asm keeps the compiler from
    // moving a load under the branch that uses it, where it would be waited
    // for on the spot and a round would run one load at a time).
    constexpr int BB = 16, LB = 40, RB = 8;
    const bool breg = p.nblk <= (int64_t)BB * BS_THREADS;
    // keys of blocks b0 + tid + 1024 u (0 past the end) into key[0..U)
    auto load_blocks = [&](int64_t b0, auto &key) {
        constexpr int U = sizeof(key) / sizeof(key[0]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t b = b0 + tid + (int64_t)u * BS_THREADS;
            key[u] = bm[b < p.nblk ? b : p.nblk - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) asm volatile("" : "+v"(key[u]));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t b = b0 + tid + (int64_t)u * BS_THREADS;
            key[u] = b < p.nblk ? present_key(key[u]) : 0u;
        }
    };
    // keys of vectors vv[u] (0 past the end) into key[0..U)
    auto load_vectors = [&](const int64_t *vv, auto &key) {
        constexpr int U = sizeof(key) / sizeof(key[0]);
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = row[vv[u] < p.n ? vv[u] : p.n - 1];
#pragma unroll
        for (int u = 0; u < U; ++u) asm volatile("" : "+v"(key[u]));
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = vv[u] < p.n ? present_key(key[u]) : 0u;
    };
    uint32_t bk[BB];
    if (breg) load_blocks(0, bk);
    auto each_block = [&](auto fn) {
        if (breg) {
#pragma unroll
            for (int u = 0; u < BB; ++u) {
                const int64_t b = tid + (int64_t)u * BS_THREADS;
                if (b < p.nblk) fn(b, bk[u]);
            }
            return;
        }
        for (int64_t b0 = 0; b0 < p.nblk; b0 += (int64_t)RB * BS_THREADS) {
            uint32_t key[RB];
            load_blocks(b0, key);
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                const int64_t b = b0 + tid + (int64_t)u * BS_THREADS;
                if (b < p.nblk) fn(b, key[u]);
            }
        }
    };
    uint32_t lk[LB];
    bool lreg = false;
    int nu = 0;   // listed blocks of this wave (register keys)
    auto load_listed = [&](int nl) {
        lreg = nl <= LB * BS_WAVES;
        if (!lreg) return;
        nu = nl > wave ? (nl - wave + BS_WAVES - 1) / BS_WAVES : 0;
        int64_t vv[LB];
#pragma unroll
        for (int u = 0; u < LB; ++u)
            vv[u] = u < nu ? (int64_t)list[wave + u * BS_WAVES] * 64 + lane : p.n;
        load_vectors(vv, lk);
    };
    auto each_listed = [&](int nl, auto fn) {
        if (lreg) {
#pragma unroll
            for (int u = 0; u < LB; ++u) {
                if (u >= nu) break;
                const int64_t v = (int64_t)list[wave + u * BS_WAVES] * 64 + lane;
                if (v < p.n) fn(v, lk[u]);
            }
            return;
        }
        for (int j0 = 0; j0 < nl; j0 += RB * BS_WAVES) {
            uint32_t key[RB];
            int64_t vv[RB];
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                const int j = j0 + wave + u * BS_WAVES;
                vv[u] = j < nl ? (int64_t)list[j] * 64 + lane : p.n;
            }
            load_vectors(vv, key);
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                const int j = j0 + wave + u * BS_WAVES;
                const int64_t v = j < nl ? (int64_t)list[j] * 64 + lane : p.n;
                if (v < p.n) fn(v, key[u]);
            }
        }
    };
    // radix selection: the K-th largest key (1 <= K <= #keys) of a visitor;
    // returns it and the number of keys above it
    auto kth = [&](auto each, int K, int &above) -> uint32_t {
        clear_hist();
        __syncthreads();
        each([&](int64_t, uint32_t key) { atomicAdd(&hc[key >> 8], 1); });
        __syncthreads();
        if (wave == 0) find_digit(hist, K, sh);
        __syncthreads();
        const int hi = sh[0], a1 = sh[1];
        clear_hist();
        __syncthreads();
        each([&](int64_t, uint32_t key) {
            if ((int)(key >> 8) == hi) atomicAdd(&hc[key & 255u], 1);
        });
        __syncthreads();
        if (wave == 0) find_digit(hist, K - a1, sh);
        __syncthreads();
        above = a1 + sh[1];
        const uint32_t t = ((uint32_t)hi << 8) | (uint32_t)sh[0];
        __syncthreads();   // sh is read before it is written again
        return t;
    };
    auto finish = [&](float am, int st) {
        if (tid == 0) {
            p.amin[q] = am;
            p.state[q] = st;
        }
    };
    // theta_a: the R-th largest block key (0, every block that holds a
    // vector for the query, when there are fewer than R)
    uint32_t tha = 0;
    if (p.nblk > R) {
        int above;
        tha = kth(each_block, R, above);
    }
    const bool all_blocks = tha == 0u;
    if (tid == 0) {
        sh[2] = 0;
        sh[3] = 0;
        sh[4] = 0;
        sh[5] = 0;
    }
    __syncthreads();
    each_block([&](int64_t b, uint32_t key) {
        if (key != 0u && key >= tha) {
            const int pos = atomicAdd(&sh[2], 1);
            if (pos < kListMaxB) list[pos] = (int)b;
        }
    });
    __syncthreads();
    const int nl = sh[2];
    if (nl > kListMaxB) {
        // too many blocks tie at the threshold: no candidates
        for (int i = tid; i < KC; i += BS_THREADS) out_i[i] = INT_MAX;
        finish(INFINITY, kSelOverflow);
        return;
    }
    load_listed(nl);
    if (all_blocks) {
        // every vector for the query lies in a listed block: if at most KC,
        // all are candidates
        each_listed(nl, [&](int64_t v, uint32_t key) {
            if (key != 0u) {
                const int pos = atomicAdd(&sh[3], 1);
                if (pos < KC) put(pos, v, key);
            }
        });
        __syncthreads();
        const int c = sh[3];
        if (c <= KC) {
            for (int i = c + tid; i < KC; i += BS_THREADS) out_i[i] = INT_MAX;
            finish(-INFINITY, kSelAll);
            return;
        }
    }
    if (!all_blocks) {
        // the vectors that reach theta_a (at least R)
        each_listed(nl, [&](int64_t v, uint32_t key) {
            if (key >= tha) {
                const int pos = atomicAdd(&sh[3], 1);
                if (pos < KC) put(pos, v, key);
            }
        });
        __syncthreads();
        const int c = sh[3];
        if (c <= KC) {
            for (int i = c + tid; i < KC; i += BS_THREADS) out_i[i] = INT_MAX;
            finish(hkey_value(tha), kSelBound);
            return;
        }
    }
    // the KC best scores of the listed blocks
    int n_gt;
    const uint32_t thb = kth([&](auto fn) { each_listed(nl, fn); }, KC, n_gt);
    const int need_eq = KC - n_gt;   // keys equal to theta_b to take (>= 1)
    each_listed(nl, [&](int64_t v, uint32_t key) {
        if (key > thb) {
            put(atomicAdd(&sh[4], 1), v, key);
        } else if (key == thb) {
            const int e = atomicAdd(&sh[5], 1);
            if (e < need_eq) put(n_gt + e, v, key);
        }
    });
    finish(hkey_value(thb), kSelBound);
}

// ------------------------------------------------------- exact rescoring
struct RescoreParams {
    const uint4 *codes;
    const float *scales;
    const float *qrot;         // [nqt][d] float32 rotated queries
    const float *qconst;       // [nqt] TQ+ constant terms, or null
    const float *cents;
    const int *top_i;          // [nqt][KC] candidates (INT_MAX: none)
    const float *top_s;        // [nqt][KC] their stored (approximate) scores
    const float *amin;         // [nqt] bound on the approximate score of non-candidates
    const int *state;          // [nqt] kSel*
    const QInfo *info;
    int64_t *ids;              // [nqt][k]
    float *scores;
    int d, bits, chunks, lut_words, k;
    // queries whose top k is not proven, over all passes of the search:
    // their number, rows, rotated queries, allowlists and global bounds
    int *fb_count;
    int *fb_rows;
    float *fb_q;
    float *fb_const;
    uint64_t *fb_allow;
    int *fb_bound;
    const uint64_t *allow;     // [nqt][W] or null
    int W;
    int q0;                    // the pass's first row
    int nqt, tile_q;           // queries, and those of a tile or pass
    Gate gate;
};

// One workgroup per query, KC = 64 S candidate slots.
//  1. The query's integer table (as the single-query scan builds it).
//  0. The candidates that may be among the top k: with a the k-th largest
//     stored score and e(.) the error of a stored score (see 4), k vectors
//     score at least a - e(a), and a candidate whose b + e(b) is less is out.
//     At k = 10 about 15 of 128 remain, in R runs of 64 (R a power of two up
//     to S); each of a candidate's chunks is a line of memory, and reading
//     all of them took 44 us for 256 queries (25 now) and 26 for 32.
//  2. Lane = candidate: wave w takes the 64 candidates of run w % R and the
//     (w / R)-th of 16 / R slices of the chunks, so all lanes read the same
//     table rows (as in the scan); partial integer sums meet in LDS (exact,
//     order-free): bit-identical to the single-query scan's scores.  8-bit
//     codes are summed in float32 chunk by chunk: for one run after the
//     other, the waves compute the sums of every sixteenth chunk, which wave 0
//     then adds in the scan's order.  A run takes 12 us of LDS reads, so the
//     64 best come first, and their k-th exact score can end the loop.
//  3. Waves 0..R-1 sort their 64 exact scores; an entry's rank is its lane
//     plus, in every other sorted run, the number of entries ahead of it
//     (binary search); ranks below k are written.
//  4. Certificate: a vector outside the candidates has a stored score at
//     most amin, so its exact score is at most amin + 2^-11 |amin| +
//     2^-25 norm + err; if that is below the k-th exact score it cannot
//     enter the top k.
//  5. Without a certificate the workgroup appends the query's row, its
//     rotated coordinates and allowlist to the list that the single-query
//     scan takes.
// Appends the query of this workgroup to the list that the single-query scan
// answers; *slot_s is a word of LDS.
__device__ inline void hand_over(const RescoreParams &p, int q, int *slot_s) {
    const int tid = threadIdx.x;
    if (tid == 0) *slot_s = atomicAdd(p.fb_count, 1);
    __syncthreads();
    const int slot = *slot_s;
    for (int j = tid; j < p.d; j += kTableThreads)
        p.fb_q[(int64_t)slot * p.d + j] = p.qrot[(int64_t)q * p.d + j];
    if (p.qconst && tid == 0) p.fb_const[slot] = p.qconst[q];
    if (p.allow)
        for (int w = tid; w < p.W; w += kTableThreads)
            p.fb_allow[(int64_t)slot * p.W + w] = p.allow[(int64_t)q * p.W + w];
    if (tid == 0) {
        p.fb_rows[slot] = p.q0 + q;
        if (p.fb_bound) p.fb_bound[slot] = kBoundInit;
    }
}

template <int MODE, int S>
__global__ __launch_bounds__(kTableThreads) void rescore_kernel(RescoreParams p) {
    constexpr int KC = 64 * S;
    constexpr int CB = 12;                 // chunk loads of a lane in flight at once
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float *red = lds + p.lut_words;         // 16
    int *sums = reinterpret_cast<int *>(red + 16);   // [KC]: ranks, integer sums, then ranks
    float *run_s = reinterpret_cast<float *>(sums + KC);
    int *run_i = reinterpret_cast<int *>(run_s + KC);
    int *kept = run_i + KC;                 // [KC] candidates that may be in the top k
    // [0] sorted entries, [1] k-th exact score, [2] certified, [3] list slot,
    // [4] key of the k-th largest stored score, [5] kept, [6] candidates,
    // [7] 8 bits: key of the largest stored score after the first 64
    int *sh = kept + KC;
    const int q = blockIdx.x;
    if (scan_is_faster_for(p.gate, q, p.nqt, p.tile_q)) {
        hand_over(p, q, sh + 3);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const TableShape ts{p.d, p.bits, p.lut_words};
    // Loads in the order they are needed (completion is in order): the
    // candidates and the certificate inputs, the query's coordinates, then
    // the kept candidates' chunks, in flight while the table is built.
    // Every load is unconditional, from a clamped address.
    const int ce = tid % KC;
    const int cv = p.top_i[(int64_t)q * KC + ce];
    const float cs = p.top_s[(int64_t)q * KC + ce];
    const QInfo qi = p.info[q];
    const float amin_s = p.amin[q];
    const int st = p.state[q];
    QueryRegs<MODE> qv;
    const float *qr = p.qrot + (int64_t)q * p.d;
    if constexpr (MODE != BYTE) load_query<MODE>(ts, qr, qv);
    const float C = p.qconst ? p.qconst[q] : 0.f;
    const float own = cv == INT_MAX ? -INFINITY : cs;
    if (tid < KC) {
        run_s[ce] = own;
        sums[ce] = 0;
    }
    if (tid == 0) {
        sh[0] = 0;
        sh[1] = __float_as_int(-INFINITY);
        sh[4] = INT_MAX;
        sh[5] = 0;
        sh[6] = 0;
        sh[7] = fkey(-INFINITY);
    }
    __syncthreads();
    {
        constexpr int LEN = KC * KC / kTableThreads;   // entries that a thread compares its own with
        const int j0 = tid / KC * LEN;
        int ahead = 0;
#pragma unroll 4
        for (int j = 0; j < LEN; ++j) {   // ranks without ties: stored scores often agree
            const float o = run_s[j0 + j];
            ahead += o > own || (o == own && j0 + j < ce);
        }
        if (ahead) atomicAdd(&sums[ce], ahead);
    }
    __syncthreads();
    if (tid < KC) {
        const uint64_t there = __ballot(cv != INT_MAX);
        if (lane == 0 && there) atomicAdd(&sh[6], (int)__popcll(there));
        if (cv != INT_MAX && sums[ce] < p.k) atomicMin(&sh[4], fkey(own));
    }
    __syncthreads();
    // largest error of a stored score x / norm
    auto stored_err = [&](double x) {
        return ldexp(1.0, -11) * fabs(x) + ldexp(1.0, -25) * qi.norm + (double)qi.err;
    };
    bool rest = false;
    if (tid < KC) {
        bool keep = cv != INT_MAX;
        if (qi.err < INFINITY && sh[6] >= p.k) {
            // only a comparison that holds puts a candidate out: stored scores
            // past the float16 range (a TQ+ constant term far larger than the
            // rest) are infinite, and with one of those as kth nothing is known
            const double kth = (double)unfkey(sh[4]) * qi.norm, x = (double)own * qi.norm;
            keep = keep && !(x + stored_err(x) < kth - stored_err(kth));
        }
        auto take = [&](bool in) {
            const uint64_t m = __ballot(in);
            int at = 0;
            if (lane == 0 && m) at = atomicAdd(&sh[5], (int)__popcll(m));
            at = __shfl(at, 0) + (int)__popcll(m & ((1ull << lane) - 1));
            if (in) kept[at] = cv;
        };
        if constexpr (MODE == BYTE) {
            // the 64 best first; [7]: the largest of the others
            const bool first = keep && sums[ce] < 64;
            take(first);
            rest = keep && !first;
            if (rest) atomicMax(&sh[7], fkey(own));
        } else {
            take(keep);
        }
        sums[ce] = 0;
        run_s[ce] = -INFINITY;
        run_i[ce] = INT_MAX;
    }
    __syncthreads();
    if constexpr (MODE == BYTE) {
        if (tid < KC) {
            const uint64_t m = __ballot(rest);
            int at = 0;
            if (lane == 0 && m) at = atomicAdd(&sh[5], (int)__popcll(m));
            at = __shfl(at, 0) + (int)__popcll(m & ((1ull << lane) - 1));
            if (rest) kept[at] = cv;
        }
        __syncthreads();
    }
    const int nk = sh[5];
    int R = 1;                             // runs of 64 kept candidates
    while (R < S && 64 * R < nk) R *= 2;
    const int run = wave % R, slice = wave / R, SL = kTableWaves / R;
    const int c0 = MODE == BYTE ? wave : p.chunks * slice / SL;
    const int c1 = MODE == BYTE ? p.chunks : p.chunks * (slice + 1) / SL;
    constexpr int CS = MODE == BYTE ? kTableWaves : 1;   // step of a wave's chunks
    uint4 w[CB];
    const uint4 *src;
    auto take_run = [&](int r) {           // the lane's candidate of run r
        const int e = r * 64 + lane;
        const int v = e < nk ? kept[e] : INT_MAX;
        const int vc = v != INT_MAX ? v : 0;
        src = p.codes + ((int64_t)(vc >> 6) * p.chunks) * 64 + (vc & 63);
        return v;
    };
    auto load_chunks = [&](int cb) {
#pragma unroll
        for (int r = 0; r < CB; ++r) {
            const int c = cb + CS * r < c1 ? cb + CS * r : cb;
            w[r] = src[(int64_t)c * 64];
        }
    };
    const int v = take_run(MODE == BYTE ? 0 : run);
    const bool valid = v != INT_MAX;
    const float scl = p.scales[valid ? v : 0];
    const bool any = c0 < c1 && __ballot(valid) != 0;
    if (any) load_chunks(c0);
    int shx = 0;
    if constexpr (MODE == BYTE) {
        for (int e = tid; e < kByteRepWords; e += kTableThreads) lds[e] = p.cents[e >> 5];
        for (int e = tid; e < p.d; e += kTableThreads) lds[kByteRepWords + e] = qr[e];
    } else {
        query_abs_sum<MODE>(red, qv);
        __syncthreads();
        shx = build_int_table<MODE>(lds, red, p.cents, ts, qv, C);
    }
    __syncthreads();
    // waves 0..R-1 sort their runs of 64 exact scores
    auto sort_run = [&](int r, float s_, int i_) {
        wave_sort64(s_, i_, lane);
        run_s[r * 64 + lane] = s_;
        run_i[r * 64 + lane] = i_;
        const int c = __popcll(__ballot(i_ != INT_MAX));
        if (lane == 0 && c) atomicAdd(&sh[0], c);
    };
    if constexpr (MODE == BYTE) {
        float *part = lds + kByteRepWords + p.d;   // [chunk][64]
        for (int r = 0; r < R; ++r) {
            // the first run's k-th exact score may put all others out
            if (r == 1 && p.k <= 64 && qi.err < INFINITY) {
                const double x = (double)unfkey(sh[7]) * qi.norm;
                if (x + stored_err(x) < (double)run_s[p.k - 1]) break;
            }
            const int vr = r == 0 ? v : take_run(r);
            if (c0 < c1) {
                if (r > 0) load_chunks(c0);
                for (int cb = c0; cb < c1; cb += CS * CB) {
                    if (cb > c0) load_chunks(cb);
#pragma unroll
                    for (int u = 0; u < CB; ++u)
                        if (cb + CS * u < c1)
                            part[(cb + CS * u) * 64 + lane] = byte_chunk(lds, cb + CS * u, w[u]);
                }
            }
            __syncthreads();
            if (wave == 0) {
                float facc = C;
                for (int c = 0; c < p.chunks; c += 4) {   // whole rings of 4 chunks
                    float t[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) t[u] = part[(c + u) * 64 + lane];
#pragma unroll
                    for (int u = 0; u < 4; ++u) facc += t[u];
                }
                const bool in = vr != INT_MAX;
                sort_run(r, in ? facc * p.scales[vr] : -INFINITY, vr);
            }
            __syncthreads();   // the sums have been read
        }
    } else {
        const char *lut = reinterpret_cast<const char *>(lds);
        int acc = 0;
        if (any)
            for (int cb = c0; cb < c1; cb += CB) {
                if (cb > c0) load_chunks(cb);
#pragma unroll
                for (int r = 0; r < CB; ++r)
                    if (cb + r < c1) acc += int_chunk<MODE>(lut + (cb + r) * kChunkTableBytes<MODE>, w[r]);
            }
        if (valid) atomicAdd(&sums[run * 64 + lane], acc);
        __syncthreads();
        if (wave < R)   // slice 0: the run's own candidates
            sort_run(wave, valid ? ldexpf((float)sums[wave * 64 + lane] * scl, -shx) : -INFINITY, v);
    }
    __syncthreads();
    // rank of entry e = its place in its run + the entries ahead of it in
    // each other run (binary search); thread t searches for entry t % KC in
    // the runs (run(e) + 1 + t / KC + g * (1024 / KC)) % S
    for (int e = tid; e < KC; e += kTableThreads) sums[e] = e & 63;
    __syncthreads();
    {
        const int e = tid % KC, er = e >> 6;
        const float es = run_s[e];
        const int ei = run_i[e];
        int add = 0;
        if (ei != INT_MAX) {
            for (int o = 1 + tid / KC; o < S; o += kTableThreads / KC) {
                const int b = (er + o) % S;
                const float *rs = run_s + b * 64;
                const int *ri = run_i + b * 64;
                int pos = 0;
#pragma unroll
                for (int step = 64; step >= 1; step >>= 1)
                    if (pos + step <= 64 && better(rs[pos + step - 1], ri[pos + step - 1], es, ei))
                        pos += step;
                add += pos;
            }
        }
        if (add) atomicAdd(&sums[e], add);
    }
    __syncthreads();
    for (int e = tid; e < KC; e += kTableThreads) {
        const int ei = run_i[e];
        const int rank = sums[e];
        if (ei != INT_MAX && rank < p.k) {
            p.ids[(int64_t)q * p.k + rank] = (int64_t)ei;
            p.scores[(int64_t)q * p.k + rank] = run_s[e];
            if (rank == p.k - 1) sh[1] = __float_as_int(run_s[e]);
        }
    }
    __syncthreads();
    const int nv = sh[0];
    for (int r = nv + tid; r < p.k; r += kTableThreads) {
        p.ids[(int64_t)q * p.k + r] = -1;
        p.scores[(int64_t)q * p.k + r] = -INFINITY;
    }
    if (tid == 0) {
        const float ek = __int_as_float(sh[1]);
        const double amin = (double)amin_s * qi.norm;
        const double reach = amin + stored_err(amin);
        // an error bound that is not finite (scales or queries that are not)
        // proves nothing, nor does a list shorter than the candidates allow
        const bool cert = qi.err < INFINITY && nv >= (sh[6] < p.k ? sh[6] : p.k) &&
                          (st == kSelAll || (st == kSelBound && reach < (double)ek));
        sh[2] = cert;
    }
    __syncthreads();
    if (!sh[2]) hand_over(p, q, sh + 3);
}

// ============================================================ wide passes
// Passes of up to 256 queries (QP = 256 query slots) read the code store once
// per pass and keep no score matrix (taken where wide_pass says so):
//  1. prep_kernel, then frag_kernel: the float16 queries in the A operand
//     order of v_mfma_f32_32x32x16_f16.  Piece (c, f, l) (16 bytes) holds
//     coordinates 32c + 16(f & 1) + 8(l >> 5) .. +7 of query
//     32(f >> 1) + (l & 31), so the query part of a chunk is QP * 64
//     contiguous bytes, and lane l of a wave reads fragment f (query tile
//     f / 2, k-half f & 1) at offset (f * 64 + l) * 16.
//  2. wide_scores_kernel, pilot launch: tiles of NG blocks (every pstride-th
//     tile of the store, at most one per workgroup); every approximate score
//     of their vectors is written, [query][pilot vector].
//  3. pilot_select_kernel: per query, theta = about the KC-th largest allowed
//     pilot score (see pilot_rank; -inf when no more pilot vectors are
//     allowed), and the allowed pilot vectors that reach it as candidates.
//  4. wide_scores_kernel, main launch: every other tile; a vector whose
//     score reaches its query's theta (and that is live and whose tenant the
//     query allows) is appended to the workgroup's list for that query.
//  5. final_select_kernel: the KC best of the pilot's and the workgroups'
//     candidates, and amin = the KC-th one's score.  A vector that is not
//     taken scores below theta <= amin (never appended) or at most amin
//     (behind the KC-th), which is the bound the certificate needs.
//  6. rescore_kernel: exact scores, top k and certificate, as for tiles.
// Work items of the score kernel are steps (tile, chunk): for each, the
// workgroup stages one slab in LDS -- the chunk's query pieces and the
// chunk of each of its NG blocks -- and its eight waves multiply them: wave
// w takes block w % NG of the tile against query half w / NG (QW queries).
// Slabs go straight from global memory into a ring of NB LDS buffers
// (direct loads, NB - 2 steps ahead); one barrier per step publishes the
// next slab, whose codes are turned into MFMA operands while the current
// slab is multiplied.
constexpr int WD_THREADS = 512;
constexpr int WD_WAVES = WD_THREADS / 64;
constexpr int PS_THREADS = 1024;               // pilot_select_kernel, final_select_kernel
constexpr int kPilotMax = 65536;               // pilot vectors per query (16-bit keys in 128 KiB of LDS)
constexpr int kFinalMax = 16384;               // candidates a query's final selection gathers
constexpr int kWideMaxQ = 256;
constexpr int64_t kWideWork = 1000000;       // see wide_pass
constexpr int kWideMinChunks = 8;            // chunks per vector of a wide pass: more than its slabs ahead

// Order-preserving map of float32 onto uint32; 0 marks an absent entry
// (below every finite value and -inf).
__device__ inline uint32_t ukey(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float ukey_value(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

__global__ void frag_kernel(const _Float16 *__restrict__ q16, const QInfo *__restrict__ info,
                            int nqt, int QP, int d, uint4 *__restrict__ qfrag,
                            float *__restrict__ qf) {
    const int64_t per_chunk = (int64_t)QP * 4;
    const int64_t tot = (int64_t)(d / 32) * per_chunk;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(e / per_chunk);
        const int rem = (int)(e - c * per_chunk);
        const int f = rem >> 6, l = rem & 63;   // fragment (query tile f / 2, k-half f & 1)
        const int q = 32 * (f >> 1) + (l & 31);
        uint4 v = make_uint4(0, 0, 0, 0);
        if (q < nqt)
            v = *reinterpret_cast<const uint4 *>(q16 + (int64_t)q * d + 32 * c + 16 * (f & 1) +
                                                 8 * (l >> 5));
        qfrag[e] = v;
    }
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < QP;
         q += (int64_t)gridDim.x * blockDim.x) {
        qf[q] = q < nqt ? info[q].f : 0.f;
        qf[QP + q] = q < nqt ? info[q].c : 0.f;
    }
}

struct WideParams {
    const uint4 *codes;        // blocked store (b = 4)
    const float *scales;
    const uint4 *qfrag;        // [chunks][QP * 4] query pieces
    const float *qf;           // [QP] score factors (0 for unused slots), then [QP] constant terms
    const float *cents;        // 16 levels
    int64_t n, nblk, ntiles;   // tiles of NG blocks
    int chunks, pstride, npil; // pilot tiles: i * pstride, i < npil
    int pilot;                 // 1: pilot launch, 0: main launch (selects the kernel)
    float *pil;                // pilot: [QP][npil * 64 NG] scores
    const float *theta;        // main: [nqt] thresholds
    // main, filtered
    const uint16_t *tenants;
    const uint32_t *tmask;     // [tenant][QP / 32] queries that admit it (null: not filtered)
    const uint64_t *live;      // [nblk] or null
    Gate gate;
    int nqt;
    float *cand_s;             // main: [grid][QP][S] appended scores and ids
    int *cand_i;
    int *cand_n;               // main: [grid][QP] appended per workgroup and query
    int S;
};

constexpr int WD_NG = 4;                       // blocks per tile (wave w: block w % 4)
constexpr int WD_NH = WD_WAVES / WD_NG;        // query halves (wave w: half w / 4)

// Slab buffers in LDS per query-slot count.  A slab holds the chunk's QF
// query pieces (pieces 0..QF-1) and the chunk of each of the tile's 4 blocks
// (pieces QF..QF+3), 1 KiB each; piece i is loaded by wave i % 8 as its
// (i / 8)-th load and stored among the wave's pieces, which are contiguous
// (one LDS base per wave and slab).  NB buffers hold the slab being
// multiplied, the next one (whose codes are turned into operands meanwhile)
// and NB - 2 in flight; four of 20 KiB leave room for a table of 64 replicas,
// whose lookups take one vector instruction instead of two.
template <int QW>
struct WideShape {
    static constexpr int QP = QW * WD_NH;
    static constexpr int QF = QP / 16;                 // query pieces of a slab
    static constexpr int NI = QF + WD_NG;              // 1 KiB pieces of a slab
    static constexpr int DW = (NI + WD_WAVES - 1) / WD_WAVES;   // most loads of a wave per slab
    static constexpr int DH = NI - (DW - 1) * WD_WAVES;         // waves that make so many (the others one fewer)
    static constexpr int SU = NI * 64;                 // uint4 of a slab
    static constexpr int NB = 4;                       // slab buffers
    static constexpr int NR = 64;                      // table replicas
    static constexpr int PD = NB - 1;                  // slabs requested ahead
    static constexpr size_t lds = 256 * NR * 4 + (size_t)NB * SU * 16 + 2 * 1024 +
                                  4 * (size_t)QP * 4;
    // uint4 offset of piece i within a slab
    static constexpr __host__ __device__ int first(int wave) { return wave * (DW - 1) + (wave < DH ? wave : DH); }
    static constexpr __host__ __device__ int pos(int i) { return (first(i % WD_WAVES) + i / WD_WAVES) * 64; }
};

template <int QW, bool PILOT, bool FILT>
__global__ __launch_bounds__(WD_THREADS) void wide_scores_kernel(WideParams p) {
    using WS = WideShape<QW>;
    constexpr int QP = WS::QP, QF = WS::QF, NI = WS::NI, SU = WS::SU, NB = WS::NB, PD = WS::PD;
    static_assert(WS::DW * 1024 <= 4096, "a wave's loads of a slab within one instruction-offset span");
    constexpr int NG = WD_NG;
    constexpr int QT = QW / 32;                // 32-query tiles of a wave
    constexpr int QU = QF * 64;                // uint4 of a slab's query part
    // 1 KiB loads of a slab per wave: load i goes to wave i % 8
    constexpr int DHI = (NI + WD_WAVES - 1) / WD_WAVES, NHI = NI - (DHI - 1) * WD_WAVES;
    static_assert(PD >= 2, "the next slab must be present a step ahead");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int NR = WS::NR;
    uint32_t *T = reinterpret_cast<uint32_t *>(smem);                 // byte table x NR
    uint4 *slab = reinterpret_cast<uint4 *>(smem + 256 * NR * 4);     // [NB][SU]
    float *sclv = reinterpret_cast<float *>(slab + NB * SU);           // [2][256] tile scales
    float *fq = sclv + 512;                                            // [QP]
    float *th = fq + QP;                                               // [QP]
    int *cnt = reinterpret_cast<int *>(th + QP);                       // [QP]
    float *cq = reinterpret_cast<float *>(cnt + QP);                   // [QP]
    if (scan_is_faster(p.gate, 0, p.nqt)) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar branches
    const int g = wave % NG, h = wave / NG;
    const int G = gridDim.x, wg = blockIdx.x;
    const int CH = p.chunks;
    const int64_t nt_all = PILOT ? p.npil : p.ntiles - p.npil;
    const int64_t my_tiles = nt_all > wg ? (nt_all - wg + G - 1) / G : 0;
    // the i-th tile of this workgroup
    auto tile_of = [&](int64_t i) -> int64_t {
        const int64_t j = wg + i * G;
        if (PILOT) return j * p.pstride;
        const int64_t r = p.pstride - 1;   // >= 1 whenever there are main tiles
        return (j / r) * p.pstride + 1 + j % r;
    };

    for (int e = tid; e < 256 * NR; e += WD_THREADS) {
        const int v = e / NR;
        const uint32_t lo = __builtin_bit_cast(uint16_t, (_Float16)p.cents[v & 15]);
        const uint32_t hi = __builtin_bit_cast(uint16_t, (_Float16)p.cents[v >> 4]);
        T[e] = lo | (hi << 16);
    }
    for (int q = tid; q < QP; q += WD_THREADS) {
        fq[q] = p.qf[q];
        cq[q] = p.qf[QP + q];
        th[q] = (!PILOT && q < p.nqt) ? p.theta[q] : INFINITY;
        cnt[q] = 0;
    }
    if (my_tiles > 0) {
        const uint32_t lb = (uint32_t)(lane & (NR - 1)) * 4;
        const uint32_t lo16 = (uint32_t)lane * 16;
        const uint32_t slab_lds = (uint32_t)(uintptr_t)slab;
        const uint32_t scl_lds = (uint32_t)(uintptr_t)sclv;
        // this wave's loads of a slab: DHI of them for waves below NHI
        const bool hi_wave = wave < NHI;
        // next slab to request: tile ordinal, tile, chunk, buffer
        int64_t ld_i = 0, ld_tile = tile_of(0);
        int ld_c = 0, ld_b = 0;
        // the j-th load of this wave for the next slab to request (piece
        // i = 8j + wave, stored at this wave's base + j KiB); request_base
        // first, once per slab
        auto request_base = [&]() {
            set_lds_base(slab_lds + (uint32_t)ld_b * (SU * 16) + (uint32_t)WS::first(wave) * 1024);
        };
        auto request_part = [&](auto J) {
            constexpr int j = decltype(J)::value;
            const int i = j * WD_WAVES + wave;
            if (i < NI) {   // uniform
                if (i < QF) {
                    lds_dma16_s_at<j, false>(lo16, p.qfrag + (int64_t)ld_c * QU + i * 64);
                } else {
                    int64_t b = ld_tile * NG + (i - QF);
                    b = b < p.nblk ? b : p.nblk - 1;
                    lds_dma16_s_at<j, true>(lo16, p.codes + (b * CH + ld_c) * 64);
                }
            }
        };
        auto request_done = [&]() {
            if (ld_c == 0 && wave == WD_WAVES - 1) {
                // the tile's 256 scales (4 per lane, block clamped like the codes)
                int64_t v = ld_tile * 256 + 4 * lane;
                if (v >= p.nblk * 64) v -= (ld_tile * NG + lane / 16 - (p.nblk - 1)) * 64;
                lds_dma16(p.scales + v, scl_lds + (uint32_t)(ld_i & 1) * 1024);
            }
            ld_b = ld_b + 1 == NB ? 0 : ld_b + 1;
            // past the last step the last tile's slabs are requested again (unused)
            if (++ld_c == CH) {
                ld_c = 0;
                if (ld_i + 1 < my_tiles) ld_tile = tile_of(++ld_i);
            }
        };
        static_assert(DHI == 3 && 2 * QT >= 4, "a wave's loads of a slab follow product groups 1, 2 and 3");
        auto request = [&]() {
            request_base();
            request_part(std::integral_constant<int, 0>());
            request_part(std::integral_constant<int, 1>());
            request_part(std::integral_constant<int, 2>());
            request_done();
        };
        // until the oldest requested slab but `ahead` has landed
        auto wait_slabs = [&](auto ahead) {
            constexpr int A = decltype(ahead)::value;
            if (hi_wave) wait_vmem<A * DHI>();
            else wait_vmem<A * (DHI - 1)>();
        };
        // B operands of a chunk: b[2m + ks] for vectors 32m .. 32m + 31 of the
        // wave's block and coordinates 16ks .. 16ks + 15 of the chunk (lane l:
        // vector 32m + (l & 31), coordinates 16ks + 8(l >> 5) .. +7).  Lane v
        // holds words 0..3 of vector v; permlane32_swap(w0, w1) leaves word 0
        // of vectors 0..31 in lanes 0..31 and word 1 of the same vectors in
        // lanes 32..63 (first result), and words 0, 1 of vectors 32..63 the
        // same way (second); likewise (w2, w3) for the second k-half.
        half8 bop[2][4];   // of the current and the next step, in turn
        auto operands = [&](const uint4 *sb, half8 (&b)[4]) {
            const uint4 w = sb[WS::pos(QF + g) + lane];
            const auto k0 = __builtin_amdgcn_permlane32_swap(w.x, w.y, false, false);
            const auto k1 = __builtin_amdgcn_permlane32_swap(w.z, w.w, false, false);
            b[0] = dequant8<NR>(k0[0], lb);   // vectors 0..31, k-half 0
            b[1] = dequant8<NR>(k1[0], lb);   // vectors 0..31, k-half 1
            b[2] = dequant8<NR>(k0[1], lb);   // vectors 32..63, k-half 0
            b[3] = dequant8<NR>(k1[1], lb);   // vectors 32..63, k-half 1
        };
#pragma unroll 1
        for (int x = 0; x < PD; ++x) request();
        wait_slabs(std::integral_constant<int, PD - 1>());
        lds_barrier();
        operands(slab, bop[0]);
        // this wave's A operands of a slab: fragment 2t + ks of its query half
        half8 acur[2 * QT];
        auto a_operands = [&](const uint4 *sb) {
#pragma unroll
            for (int f = 0; f < 2 * QT; ++f)
                acur[f] = reinterpret_cast<const half8 *>(sb)[WS::pos(h * 2 * QT + f) + lane];
        };
        a_operands(slab);

        float16v acc[QT][2];
        auto clear_acc = [&]() {
#pragma unroll
            for (int t = 0; t < QT; ++t)
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[t][m][e] = 0.f;
        };
        clear_acc();
        int64_t ti = 0;       // tile ordinal of the current step
        int64_t tile = tile_of(0);
        int buf = 0;          // buffer of the current step's slab
        // lane holds vectors 32m + (lane & 31) of its block and, in element e
        // of tile t, query h QW + 32t + 8(e >> 2) + 4(lane >> 5) + (e & 3)
        auto epilogue = [&]() {
            // hq is made opaque so that the per-query offsets below are
            // formed here, once per tile, rather than hoisted out of the step
            // loop into registers held across it
            int hq = h * QW + 4 * (lane >> 5);
            asm volatile("" : "+v"(hq));
            const float *ts = sclv + (ti & 1) * 256 + g * 64 + (lane & 31);
            const float scl[2] = {ts[0], ts[32]};
            const int64_t vb = (tile * NG + g) * 64 + (lane & 31);
            const bool vin[2] = {vb < p.n, vb + 32 < p.n};
            if constexpr (PILOT) {
                const int64_t prow = (int64_t)p.npil * 64 * NG;
                const int64_t pcol = (wg + ti * G) * 64 * NG + g * 64 + (lane & 31);
#pragma unroll
                for (int t = 0; t < QT; ++t)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int q = hq + 32 * t + 8 * (e >> 2) + (e & 3);
                        const float f = fq[q], k = cq[q];
#pragma unroll
                        for (int m = 0; m < 2; ++m)
                            p.pil[q * prow + pcol + 32 * m] =
                                vin[m] ? fmaf(acc[t][m][e], f, k) * scl[m] : -INFINITY;
                    }
            } else {
                // which entries reach their query's threshold, without
                // branches (bit 2e + m of hit[t]) ...
                uint32_t hit[QT];
#pragma unroll
                for (int t = 0; t < QT; ++t) {
                    uint32_t hb = 0u;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        // four queries' factors and thresholds, read together
                        const float4 f4 = *reinterpret_cast<const float4 *>(fq + hq + 32 * t + 8 * i);
                        const float4 k4 = *reinterpret_cast<const float4 *>(cq + hq + 32 * t + 8 * i);
                        const float4 t4 = *reinterpret_cast<const float4 *>(th + hq + 32 * t + 8 * i);
                        const float fr[4] = {f4.x, f4.y, f4.z, f4.w}, tr[4] = {t4.x, t4.y, t4.z, t4.w};
                        const float kr[4] = {k4.x, k4.y, k4.z, k4.w};
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int e = 4 * i + j;
                            hb |= (vin[0] && fmaf(acc[t][0][e], fr[j], kr[j]) * scl[0] >= tr[j]) ? 1u << (2 * e) : 0u;
                            hb |= (vin[1] && fmaf(acc[t][1][e], fr[j], kr[j]) * scl[1] >= tr[j]) ? 2u << (2 * e) : 0u;
                        }
                    }
                    hit[t] = hb;
                }
                // ... restricted to the vectors that a query may return (bit
                // 8i + j of a mask word past the lane half's shift: entry
                // e = 4i + j)
                if constexpr (FILT) {
                    // loads without branches: an absent live mask reads the
                    // tenant masks instead, unused
                    const uint64_t *lp = p.live ? p.live : reinterpret_cast<const uint64_t *>(p.tmask);
                    const uint64_t all = p.live ? 0ull : ~0ull;
                    const int sh = 4 * (lane >> 5);
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        int v = vin[m] ? (int)vb + 32 * m : 0;
                        asm volatile("" : "+v"(v));   // formed here, not held across the steps
                        const uint64_t lv = lp[p.live ? v >> 6 : 0] | all;
                        const uint32_t may = (lv >> (v & 63)) & 1ull ? ~0u : 0u;
                        const uint32_t *tw = p.tmask + p.tenants[v] * (QP / 32) + h * QT;
#pragma unroll
                        for (int t = 0; t < QT; ++t) {
                            uint32_t x = (tw[t] >> sh) & may & 0x0F0F0F0Fu;
                            x = (x | (x << 2)) & 0x33333333u;
                            x = (x | (x << 1)) & 0x55555555u;
                            hit[t] &= (x << m) | (0xAAAAAAAAu >> m);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // ... then append those (rare): one entry per lane and round,
                // its value picked out of the accumulators by its bit index
                // (a fixed select chain: the accumulators stay in registers)
                uint32_t pend[QT];
#pragma unroll
                for (int t = 0; t < QT; ++t) pend[t] = hit[t];
                auto any_pending = [&]() {
                    uint32_t o = 0u;
#pragma unroll
                    for (int t = 0; t < QT; ++t) o |= pend[t];
                    return o != 0u;
                };
                while (__ballot(any_pending())) {
                    if (any_pending()) {
                        int bt = 0;   // lowest pending bit: tile bt, bit bb = 2e + m
#pragma unroll
                        for (int t = QT - 1; t >= 0; --t)
                            if (pend[t]) bt = t;
                        uint32_t word = pend[0];
#pragma unroll
                        for (int t = 1; t < QT; ++t) word = bt == t ? pend[t] : word;
                        const int bb = __builtin_ctz(word);
#pragma unroll
                        for (int t = 0; t < QT; ++t)
                            if (bt == t) pend[t] &= pend[t] - 1u;
                        float a = 0.f;
#pragma unroll
                        for (int t = 0; t < QT; ++t)
#pragma unroll
                            for (int e = 0; e < 16; ++e)
#pragma unroll
                                for (int m = 0; m < 2; ++m)
                                    a = (bt == t && bb == 2 * e + m) ? acc[t][m][e] : a;
                        const int e = bb >> 1, m = bb & 1;
                        const int q = hq + 32 * bt + 8 * (e >> 2) + (e & 3);
                        const float val = fmaf(a, fq[q], cq[q]) * scl[m];
                        const int slot = atomicAdd(&cnt[q], 1);
                        if (slot < p.S) {
                            const int64_t o = ((int64_t)wg * QP + q) * p.S + slot;
                            p.cand_s[o] = val;
                            p.cand_i[o] = (int)(vb + 32 * m);
                        }
                    }
                }
            }
            clear_acc();
        };
        // one step, with operands bcur; the next one's go to bnext
        auto step = [&](const half8 (&bcur)[4], half8 (&bnext)[4]) {
            {
                // the next step's slab has landed (own loads), then everyone's;
                // every wave is done with the buffer the new request overwrites
                wait_slabs(std::integral_constant<int, PD - 2>());
                lds_barrier();
                // the products of slab s (operands read a step ahead) in groups
                // of two; the code word of slab s + 1 turned into the next B
                // operands, and this step's loads, are issued between the
                // groups so that they overlap the matrix cores' work
                buf = buf + 1 == NB ? 0 : buf + 1;
                const uint4 wn = slab[buf * SU + WS::pos(QF + g) + lane];
                const half8 *an = reinterpret_cast<const half8 *>(slab + buf * SU) + lane;
                // k-half outer, so that the two products into one accumulator
                // are 2 QT products apart (a product waits for the previous
                // one into the same accumulator to finish)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int t = 0; t < QT; ++t) {
                        const half8 a = acur[2 * t + ks];
                        acc[t][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bcur[ks], acc[t][0], 0, 0, 0);
                        acc[t][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bcur[2 + ks], acc[t][1], 0, 0, 0);
                        const int grp = ks * QT + t;   // groups of two products
                        if (grp == 0) {
                            const auto k0 = __builtin_amdgcn_permlane32_swap(wn.x, wn.y, false, false);
                            const auto k1 = __builtin_amdgcn_permlane32_swap(wn.z, wn.w, false, false);
                            bnext[0] = dequant8<NR>(k0[0], lb);
                            bnext[1] = dequant8<NR>(k1[0], lb);
                            bnext[2] = dequant8<NR>(k0[1], lb);
                            bnext[3] = dequant8<NR>(k1[1], lb);
                        }
                        if (grp == 1) {
                            request_base();
                            request_part(std::integral_constant<int, 0>());
                        }
                        if (grp == 2) request_part(std::integral_constant<int, 1>());
                        if (grp == 3) request_part(std::integral_constant<int, 2>());
                        // the next slab's A operands, as soon as the tile's
                        // last product has been issued
                        if (ks == 1) {
                            acur[2 * t] = an[WS::pos(h * 2 * QT + 2 * t)];
                            acur[2 * t + 1] = an[WS::pos(h * 2 * QT + 2 * t + 1)];
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                request_done();
            }
        };
        for (;;) {
            for (int c = 0; c < CH; c += 2) {   // CH is even
                step(bop[0], bop[1]);
                step(bop[1], bop[0]);
            }
            epilogue();
            if (++ti == my_tiles) break;
            tile = tile_of(ti);
            // the next step's operands again (its slab stays in place until the
            // next request): not held in registers across the epilogue
            a_operands(slab + buf * SU);
            operands(slab + buf * SU, bop[0]);
        }
    }
    if (!PILOT) {
        __syncthreads();
        for (int q = tid; q < QP; q += WD_THREADS) p.cand_n[(int64_t)wg * QP + q] = cnt[q];
    }
}

// K-th largest of the BITS-bit keys visited by `each` (K >= 1, at most the
// number of non-zero keys; zero keys are absent): 8-bit radix passes with
// LDS histograms.  Returns the key and sets n_above to the number of
// keys above it.  Called by every thread of the workgroup.
template <int BITS, class Each>
__device__ uint32_t radix_kth(Each each, int K, int *hist, int *sh, int &n_above) {
    static_assert(BITS % 8 == 0, "8-bit digits");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int *hc = hist + (lane & 3) * kHistStride;
    uint32_t prefix = 0, pmask = 0;
    int above = 0;
    for (int pass = 0; pass < BITS / 8; ++pass) {
        const int shift = BITS - 8 - 8 * pass;
        for (int i = tid; i < kHistCopies * kHistStride; i += blockDim.x) hist[i] = 0;
        __syncthreads();
        // the lanes of a wave that share the first active lane's digit add
        // their count once (the high digits of one query's scores are mostly
        // equal, and their single-lane atomics would serialise); the others
        // add one each
        each([&](uint32_t k) {
            const bool act = k != 0u && (k & pmask) == prefix;
            const uint32_t dg = (k >> shift) & 255u;
            const uint64_t live = __ballot(act);
            if (live) {
                const int leader = __builtin_ctzll(live);
                const uint32_t dl = __builtin_amdgcn_readlane(dg, leader);
                const bool same = act && dg == dl;
                const uint64_t sm = __ballot(same);
                if (lane == leader) atomicAdd(&hc[dl], (int)__popcll(sm));
                else if (act && !same) atomicAdd(&hc[dg], 1);
            }
        });
        __syncthreads();
        if (wave == 0) find_digit(hist, K - above, sh);
        __syncthreads();
        prefix |= (uint32_t)sh[0] << shift;
        pmask |= 255u << shift;
        above += sh[1];
        __syncthreads();   // sh is read before it is written again
    }
    n_above = above;
    return prefix;
}

struct PilotParams {
    const float *pil;          // [QP][npv]
    int64_t npv;               // pilot vectors per query (npil * 64 WD_NG)
    int pstride;
    int64_t n;
    const uint16_t *tenants;
    const uint64_t *allow;     // [nqt][W] or null
    const uint64_t *live;      // [nblk] or null
    Gate gate;
    int nqt;
    int W, PCM;
    int rank;                  // see pilot_rank
    int groups;                // maxima per thread: 1, 2 or 4
    int most;                  // pilot candidates that need no exact threshold
    float *theta;              // [nqt]
    int *pc_n;                 // [nqt] pilot candidates (may exceed PCM: overflow)
    int *pc_i;                 // [nqt][PCM]
    float *pc_s;
};

// One workgroup per query.  The selection runs on 16-bit keys, the top half
// of the order-preserving key of each allowed pilot score, held in LDS: with
// kt a key that at least `rank` allowed pilot vectors reach, theta = the
// smallest float whose key starts with kt, and a pilot vector reaches theta
// exactly when its 16-bit key reaches kt.  kt is the rank-th largest of the
// largest keys of G = 1,024, 2,048 or 4,096 groups (G / rank at least 8), each
// of up to 65,536 / G vectors: where scores lie at random G ln(G / (G - rank))
// vectors reach it, at most 7% more than rank, and one pass over the keys
// replaces three.  (With one group per thread also at rank 512 it was 39%
// more, and a call of 256 queries at 1,500,000 vectors, d = 256, k = 100 took
// 14.6 ms for the queries that overflowed, 0.51 now.)  Where more than `most`
// reach it, or fewer than `rank` groups hold an allowed vector, kt is the
// rank-th largest key itself.
__global__ __launch_bounds__(PS_THREADS) void pilot_select_kernel(PilotParams p) {
    constexpr int TV = 64 * WD_NG;                 // vectors per pilot tile
    extern __shared__ __attribute__((aligned(16))) uint16_t k16[];   // [npv], 0: absent
    __shared__ int hist[kHistCopies * kHistStride];
    __shared__ int sh[8];
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    if (scan_is_faster(p.gate, 0, p.nqt)) return;
    const int npv = (int)p.npv;
    const float *row = p.pil + (int64_t)q * p.npv;
    const uint64_t *arow = p.allow ? p.allow + (int64_t)q * p.W : nullptr;
    auto vec_of = [&](int e) -> int64_t { return (int64_t)(e / TV) * p.pstride * TV + e % TV; };
    if (tid == 0) {
        sh[4] = 0;
        sh[5] = 0;
        sh[6] = 0;
    }
    __shared__ uint64_t allow_s[64];
    if (arow)
        for (int w = tid; w < p.W; w += PS_THREADS) allow_s[w] = arow[w];
    __syncthreads();
    int cnt = 0;
    uint32_t best[4] = {0u, 0u, 0u, 0u};   // the largest keys of this thread's groups
    // rounds of 16 loads per thread, all issued before any is used
    constexpr int R = 16;
    for (int e0 = 0; e0 < npv; e0 += R * PS_THREADS) {
        float val[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int e = e0 + tid + u * PS_THREADS;
            val[u] = row[e < npv ? e : 0];
        }
        int tn[R];
        if (arow) {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int e = e0 + tid + u * PS_THREADS;
                const int64_t v = vec_of(e < npv ? e : 0);
                tn[u] = p.tenants[v < p.n ? v : 0];
            }
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int e = e0 + tid + u * PS_THREADS;
            if (e < npv) {
                bool ok = val[u] > -INFINITY;
                if (arow)
                    ok = ok && (tn[u] >> 6) < p.W && ((allow_s[tn[u] >> 6] >> (tn[u] & 63)) & 1ull);
                if (p.live) {
                    const int64_t v = vec_of(e);
                    ok = ok && ((p.live[v < p.n ? v >> 6 : 0] >> (v & 63)) & 1ull);
                }
                const uint32_t key = ok ? ukey(val[u]) >> 16 : 0u;   // a finite key's top half is >= 0x80
                k16[e] = (uint16_t)key;
                best[u & 3] = key > best[u & 3] ? key : best[u & 3];
                cnt += ok;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if (p.groups < 4)
        for (int i = 0; i < 2; ++i) best[i] = best[i] > best[i + 2] ? best[i] : best[i + 2];
    if (p.groups < 2) best[0] = best[0] > best[1] ? best[0] : best[1];
    int some = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) some += __popcll(__ballot(i < p.groups && best[i] != 0u));
    __syncthreads();
    if (lane == 0) {
        atomicAdd(&sh[5], cnt);
        atomicAdd(&sh[6], some);
    }
    __syncthreads();
    const int allowed = sh[5];
    uint32_t thk = 1u;   // every present key
    auto take_from = [&](uint32_t key) {
        for (int e = tid; e < npv; e += PS_THREADS) {
            const uint32_t k = k16[e];
            if (k != 0u && k >= key) {
                const int pos = atomicAdd(&sh[4], 1);
                if (pos < p.PCM) {
                    p.pc_i[(int64_t)q * p.PCM + pos] = (int)vec_of(e);
                    p.pc_s[(int64_t)q * p.PCM + pos] = row[e];
                }
            }
        }
    };
    bool taken = false;
    int n_above;
    if (allowed > p.rank && sh[6] >= p.rank) {
        thk = radix_kth<16>([&](auto fn) {
            for (int i = 0; i < p.groups; ++i) fn(best[i]);
        }, p.rank, hist, sh, n_above);
        take_from(thk);
        __syncthreads();
        taken = sh[4] <= p.most;
        __syncthreads();
        if (!taken && tid == 0) sh[4] = 0;
    }
    if (!taken) {
        if (allowed > p.rank)
            thk = radix_kth<16>([&](auto fn) {
                for (int e = tid; e < npv; e += PS_THREADS) fn((uint32_t)k16[e]);
            }, p.rank, hist, sh, n_above);
        __syncthreads();
        take_from(thk);
    }
    if (tid == 0) p.theta[q] = allowed > p.rank ? ukey_value(thk << 16) : -INFINITY;
    __syncthreads();
    if (tid == 0) p.pc_n[q] = sh[4];
}

struct FinalParams {
    const float *theta;
    const int *pc_n;
    const int *pc_i;
    const float *pc_s;
    int PCM;
    const float *cand_s;       // [G][QP][S]
    const int *cand_i;
    const int *cand_n;         // [G][QP]
    int G, QP, S, KC;
    int nqt;
    Gate gate;
    int *top_i;                // [nqt][KC] (INT_MAX: none)
    float *top_s;
    float *amin;
    int *state;
};

// One workgroup per query: the query's candidates gathered in LDS, then the
// KC best.
__global__ __launch_bounds__(PS_THREADS) void final_select_kernel(FinalParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint32_t *ck = reinterpret_cast<uint32_t *>(smem);        // [kFinalMax] keys
    int *cv = reinterpret_cast<int *>(ck + kFinalMax);         // [kFinalMax] ids
    __shared__ int hist[kHistCopies * kHistStride];
    __shared__ int sh[8];
    const int q = blockIdx.x, tid = threadIdx.x;
    if (scan_is_faster(p.gate, 0, p.nqt)) return;
    int *out = p.top_i + (int64_t)q * p.KC;
    float *out_s = p.top_s + (int64_t)q * p.KC;
    __shared__ int goff[1025];                  // exclusive offsets of the workgroup lists
    __shared__ int wsum[PS_THREADS / 64];
    const int lane = tid & 63, wave = tid >> 6;
    const int n0 = p.pc_n[q];
    const int base = n0 < p.PCM ? n0 : p.PCM;
    if (tid == 0) {
        sh[3] = n0 > p.PCM;         // overflow
        sh[4] = 0;
        sh[5] = 0;
    }
    __syncthreads();
    // the G list lengths (G <= PS_THREADS), an exclusive scan over them
    int c = 0;
    if (tid < p.G) {
        c = p.cand_n[(int64_t)tid * p.QP + q];
        if (c > p.S) sh[3] = 1;
    }
    int incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    goff[tid] = base + before + incl - c;
    if (tid == PS_THREADS - 1) goff[PS_THREADS] = base + before + incl;
    __syncthreads();
    const int ng = p.G < PS_THREADS ? p.G : PS_THREADS;
    const int total_all = goff[ng];
    for (int e = tid; e < base && e < kFinalMax; e += PS_THREADS) {
        ck[e] = ukey(p.pc_s[(int64_t)q * p.PCM + e]);
        cv[e] = p.pc_i[(int64_t)q * p.PCM + e];
    }
    if (!sh[3] && total_all <= kFinalMax) {
        for (int e = base + tid; e < total_all; e += PS_THREADS) {
            int lo = 0, hi = ng - 1;   // last list whose offset is <= e
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (goff[mid] <= e) lo = mid;
                else hi = mid - 1;
            }
            const int64_t src = ((int64_t)lo * p.QP + q) * p.S + (e - goff[lo]);
            ck[e] = ukey(p.cand_s[src]);
            cv[e] = p.cand_i[src];
        }
    }
    if (tid == 0) sh[2] = total_all;
    __syncthreads();
    const int tot = sh[2];
    const float theta = p.theta[q];
    if (sh[3] || tot > kFinalMax) {
        for (int i = tid; i < p.KC; i += PS_THREADS) out[i] = INT_MAX;
        if (tid == 0) {
            p.amin[q] = INFINITY;
            p.state[q] = kSelOverflow;
        }
        return;
    }
    if (tot <= p.KC) {
        // every candidate kept: all allowed vectors when theta = -inf, else
        // every vector below theta is outside
        for (int i = tid; i < p.KC; i += PS_THREADS) {
            out[i] = i < tot ? cv[i] : INT_MAX;
            if (i < tot) out_s[i] = ukey_value(ck[i]);
        }
        if (tid == 0) {
            p.amin[q] = theta;
            p.state[q] = theta == -INFINITY ? kSelAll : kSelBound;
        }
        return;
    }
    int n_gt;
    const uint32_t thk = radix_kth<32>([&](auto fn) {
        for (int i = tid; i < tot; i += PS_THREADS) fn(ck[i]);
    }, p.KC, hist, sh, n_gt);
    const int need_eq = p.KC - n_gt;   // keys equal to thk to take (>= 1)
    for (int i = tid; i < tot; i += PS_THREADS) {
        const uint32_t k = ck[i];
        if (k > thk) {
            const int e = atomicAdd(&sh[4], 1);
            out[e] = cv[i];
            out_s[e] = ukey_value(k);
        } else if (k == thk) {
            const int e = n_gt + atomicAdd(&sh[5], 1);
            if (e < n_gt + need_eq) {
                out[e] = cv[i];
                out_s[e] = ukey_value(k);
            }
        }
    }
    if (tid == 0) {
        p.amin[q] = ukey_value(thk);
        p.state[q] = kSelBound;
    }
}

__global__ void scale_max_kernel(const float *__restrict__ s, int64_t n, int *smax_bits) {
    int m = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int b = __float_as_int(s[i]) & 0x7FFFFFFF;   // |s|: bit order is value order
        m = b > m ? b : m;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const int x = __shfl_xor(m, o, 64);
        m = x > m ? x : m;
    }
    if ((threadIdx.x & 63) == 0) atomicMax(smax_bits, m);
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Candidate slots for a given k: eight per result, 64 to 512 (the
// certificate needs the KC-th approximate score, plus the error bound, to
// fall below the k-th exact one; candidates are cheap next to a re-run).
int batch_candidates(int k) {
    int kc = kCandMin;
    while (kc < 8 * k && kc < kCandMax) kc *= 2;
    return kc;
}

// Calls fn with std::integral_constant<int, KC / 64>.
template <class Fn>
void with_slots(int KC, Fn fn) {
    switch (KC) {
    case 64: fn(std::integral_constant<int, 1>()); break;
    case 128: fn(std::integral_constant<int, 2>()); break;
    case 256: fn(std::integral_constant<int, 4>()); break;
    default: fn(std::integral_constant<int, 8>()); break;
    }
}

// Tiles of a group: as many as the queries need, at most kGroupTiles and
// 256 MiB of scores (a tile of 1,000,000 vectors has 64 MiB).
constexpr int kGroupTiles = 8;

struct BatchLayout {
    bool wide;   // whole passes of wide_pass take the wide kernels
    int tiles;   // of a group
    size_t q16, info, approx, bmax, top_i, top_s, amin, state, tickets, count, rows, qc, tmask, list,
        qconst_c, allow_c, qconst, lut, total;
    // wide passes
    size_t w_q16, w_info, w_qfrag, w_qf, w_pil, w_theta, w_pcn, w_pci, w_pcs, w_cs, w_ci, w_cn,
        w_top, w_tops, w_amin, w_state;
};

// Geometry of a wide pass with NG blocks per tile.
struct WideGeom {
    int NG, tilev, pstride, npil, S;
    int64_t ntiles, nmain;
};

WideGeom wide_geom(const ScanShape &s, int NG, int grid, int KC) {
    WideGeom w{};
    w.NG = NG;
    w.tilev = 64 * NG;
    w.ntiles = (s.nblk + NG - 1) / NG;
    // pilot tiles: at most one per workgroup, their scores within kPilotMax per query
    const int64_t cap = std::min<int64_t>(grid, kPilotMax / w.tilev);
    w.pstride = (int)((w.ntiles + cap - 1) / cap);
    w.npil = (int)((w.ntiles + w.pstride - 1) / w.pstride);
    w.nmain = w.ntiles - w.npil;
    // theta is about the (KC ntiles / npil)-th score of the store, so a
    // workgroup appends about KC nmain / (npil grid) vectors per query
    const double per = (double)KC * (double)w.nmain / ((double)w.npil * grid);
    int S = (int)std::ceil(2.0 * per + 16.0);
    S = (S + 7) / 8 * 8;
    w.S = std::min(std::max(S, 16), 512);
    return w;
}

// Pilot candidates of a query up to which its candidates in the whole store,
// `part` times the pilot's, fit the final selection but for chance: the store's
// share above a threshold that KC pilot vectors reach has a standard deviation
// of about 1 / sqrt(KC) of it, of which four and a half are left as room (one query in
// 300,000; a query that overflows costs the call a scan, 0.35 ms at 1,800,000
// vectors, d = 256, k = 100).
double pilot_most(double part, int KC) {
    return kFinalMax / (part * (1.0 + 4.5 / std::sqrt((double)KC)));
}
// The rank of the pilot score that is the threshold: KC, or fewer where that
// many (and 2% that share a 16-bit key) would be too many.  The store has
// `part` times as many vectors above it, far more than KC either way.
int pilot_rank(double part, int KC) { return std::min(KC, (int)(pilot_most(part, KC) / 1.02)); }

// Whether a pass over nq more queries takes the wide kernels: enough queries
// and vectors, and an index of which the pilot (at most 65,536 vectors) is
// large enough a part, so that the threshold's rank is still three quarters of KC
// (N up to 7.8M at k = 10, 2.2M at k = 100) and about 2 per + 16 candidates fit
// a workgroup's list.
bool wide_pass(const ScanShape &s, int64_t nq, int KC, int grid) {
    // Six tiles or more and 1,000,000 vectors at 6 tiles, 500,000 at 7, 333,333
    // at 8.  256 queries, tiles / wide, d = 1536: 188 / 231 us at 100,000
    // vectors, 368 / 405 at 300,000, 1,214 / 982 at 1,000,000; d = 256: 75 / 100
    // at 300,000, 330 / 255 at 1,000,000.  192 queries: 950 / 919 and 253 / 240
    // at 1,000,000; 128: 617 / 635 and 133 / 158.
    const int64_t tiles = (std::min<int64_t>(nq, kWideMaxQ) + kTile - 1) / kTile;
    if (s.bits != 4 || tiles < 6 || s.n * (tiles - 5) < kWideWork || s.chunks < kWideMinChunks || grid > PS_THREADS) return false;
    const WideGeom w = wide_geom(s, WD_NG, grid, KC);
    const double part = (double)w.ntiles / (double)w.npil;
    return 4 * pilot_rank(part, KC) >= 3 * KC && 2.0 * KC * part / grid + 16.0 <= 512.0;
}

// Row length of the approximate-score matrix: whole 512-vector select units.
int64_t approx_row(const ScanShape &s) { return (s.nblk * 64 + 511) / 512 * 512; }

// Tiles of the largest group that a search of nq queries is given.
int group_tiles(const ScanShape &s, int64_t nq, int k, int grid, bool wide) {
    // after whole wide passes the rest, if it is not another one, is left for tiles
    int64_t tile_q = nq;
    if (wide) {
        tile_q = nq % kWideMaxQ;
        if (tile_q == 0 || wide_pass(s, tile_q, batch_candidates(k), grid)) tile_q = 1;
    }
    const int64_t need = (tile_q + kTile - 1) / kTile, fit = ((int64_t)256 << 20) / (kTile * approx_row(s) * 2 + 1);
    return (int)std::max<int64_t>(1, std::min<int64_t>({need, fit, kGroupTiles, grid}));
}

BatchLayout batch_layout(const ScanShape &s, int64_t nq, int k, int grid, bool calibrated, bool wide, int tiles) {
    BatchLayout L{};
    size_t o = align256((size_t)nq * s.d * sizeof(float));   // rotated queries
    const int64_t npad = approx_row(s);
    L.wide = wide;
    L.tiles = tiles;
    const size_t gq = (size_t)L.tiles * kTile;   // queries of a group
    L.q16 = o;
    o += align256(gq * s.d * 2);
    L.info = o;
    o += align256(gq * sizeof(QInfo));
    L.approx = o;
    o += align256(gq * npad * 2);
    L.bmax = o;
    o += align256(gq * s.nblk * 2);
    L.top_i = o;
    o += align256(gq * kCandMax * 4);
    L.top_s = o;
    o += align256(gq * kCandMax * 4);
    L.amin = o;
    o += align256(gq * 4);
    L.state = o;
    o += align256(gq * 4);
    L.tickets = o;
    o += align256(((size_t)grid * kTicketStride + 2 * kGroupTiles) * 4);   // ... and the filter counts
    L.tmask = o;
    o += align256((size_t)s.W * 64 * (kWideMaxQ / 32) * 4);   // as many words for a group of 8 tiles
    L.list = o;
    o += align256((size_t)L.tiles * s.nblk * 4);
    L.count = o;
    o += align256(4);
    L.rows = o;
    o += align256((size_t)nq * 4);
    L.qc = o;
    o += align256((size_t)nq * s.d * sizeof(float));
    L.qconst_c = o;
    o += align256((size_t)nq * sizeof(float));
    L.allow_c = o;
    o += align256((size_t)nq * s.W * sizeof(uint64_t));
    L.qconst = o;
    o += calibrated ? align256((size_t)nq * sizeof(float)) : 0;
    L.lut = o;
    o += lut_search_workspace_bytes(s, nq, k, grid);
    if (wide) {
        const int KC = batch_candidates(k), PCM = 2 * KC;
        constexpr int QP = kWideMaxQ;
        const WideGeom w = wide_geom(s, WD_NG, grid, KC);
        auto take = [&](size_t bytes) {
            const size_t at = o;
            o += align256(bytes);
            return at;
        };
        L.w_q16 = take((size_t)QP * s.d * 2);
        L.w_info = take((size_t)QP * sizeof(QInfo));
        L.w_qfrag = take((size_t)QP * s.d * 2);
        L.w_qf = take((size_t)QP * 2 * 4);
        L.w_pil = take((size_t)QP * w.npil * w.tilev * 4);
        L.w_theta = take((size_t)QP * 4);
        L.w_pcn = take((size_t)QP * 4);
        L.w_pci = take((size_t)QP * PCM * 4);
        L.w_pcs = take((size_t)QP * PCM * 4);
        L.w_cs = take((size_t)grid * QP * w.S * 4);
        L.w_ci = take((size_t)grid * QP * w.S * 4);
        L.w_cn = take((size_t)grid * QP * 4);
        L.w_top = take((size_t)QP * KC * 4);
        L.w_tops = take((size_t)QP * KC * 4);
        L.w_amin = take((size_t)QP * 4);
        L.w_state = take((size_t)QP * 4);
    }
    L.total = o + 256;
    return L;
}

// Launches the score kernel of a tile.
template <int BITS, int NR, int RING, bool FILT>
hipError_t launch_scores_as(const ScoreParams &sp, int grid, size_t lds, hipStream_t stream) {
    static bool attr = false;
    if (!attr) {
        const hipError_t e =
            hipFuncSetAttribute((const void *)mfma_scores_kernel<BITS, NR, RING, FILT>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr = true;
    }
    hipLaunchKernelGGL((mfma_scores_kernel<BITS, NR, RING, FILT>), dim3(grid), dim3(MF_THREADS), lds, stream, sp);
    return hipGetLastError();
}
template <int BITS, int NR>
hipError_t launch_scores_ring(const ScoreParams &sp, int grid, hipStream_t stream) {
    const size_t lds = score_lds(BITS, sp.chunks, NR);
    if (sp.list)
        return sp.chunks % 8 == 0 ? launch_scores_as<BITS, NR, 8, true>(sp, grid, lds, stream)
                                  : launch_scores_as<BITS, NR, 4, true>(sp, grid, lds, stream);
    return sp.chunks % 8 == 0 ? launch_scores_as<BITS, NR, 8, false>(sp, grid, lds, stream)
                              : launch_scores_as<BITS, NR, 4, false>(sp, grid, lds, stream);
}
hipError_t launch_scores(int bits, const ScoreParams &sp, int grid, hipStream_t stream) {
    const bool r64 = score_replicas(bits, sp.chunks) == 64;
    switch (bits) {
    case 2: return launch_scores_ring<2, 64>(sp, grid, stream);
    case 3: return launch_scores_ring<3, 64>(sp, grid, stream);
    case 4:
        return r64 ? launch_scores_ring<4, 64>(sp, grid, stream) : launch_scores_ring<4, 32>(sp, grid, stream);
    default:
        return r64 ? launch_scores_ring<8, 64>(sp, grid, stream) : launch_scores_ring<8, 32>(sp, grid, stream);
    }
}

// LDS of the rescoring: the table (8 bits: and a run's chunk sums), 16
// floats, integer sums, sorted (score, id) runs and the list, eight words.
int rescore_lut_words(const ScanShape &s) {
    return s.bits == 8 ? kByteRepWords + s.d + 64 * s.chunks : s.bits == 3 ? s.chunks * 320 : s.chunks * 512;
}
size_t rescore_lds(const ScanShape &s, int KC) {
    return (size_t)rescore_lut_words(s) * 4 + 16 * 4 + (size_t)KC * 16 + 32;
}
template <int MODE, int S>
hipError_t launch_rescore_as(const RescoreParams &rp, int nqt, size_t lds, hipStream_t stream) {
    static bool attr = false;
    if (!attr) {
        const hipError_t e = hipFuncSetAttribute((const void *)rescore_kernel<MODE, S>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr = true;
    }
    hipLaunchKernelGGL((rescore_kernel<MODE, S>), dim3(nqt), dim3(kTableThreads), lds, stream, rp);
    return hipGetLastError();
}
hipError_t launch_rescore(const ScanShape &s, int KC, const RescoreParams &rp, int nqt, hipStream_t stream) {
    const size_t lds = rescore_lds(s, KC);
    hipError_t e = hipSuccess;
    with_slots(KC, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        e = s.bits == 8   ? launch_rescore_as<BYTE, S>(rp, nqt, lds, stream)
            : s.bits == 3 ? launch_rescore_as<TRIBIT, S>(rp, nqt, lds, stream)
                          : launch_rescore_as<NIBBLE, S>(rp, nqt, lds, stream);
    });
    return e;
}

// Launches wide_scores_kernel (kWideMaxQ / 2 queries per wave).
hipError_t launch_wide_scores(const WideParams &wp, int grid, hipStream_t stream) {
    hipError_t err = hipSuccess;
    auto go = [&](auto pilot, auto filt) {
        constexpr int QW = kWideMaxQ / WD_NH;
        constexpr bool P = decltype(pilot)::value, F = decltype(filt)::value;
        static bool attr = false;
        if (!attr) {
            err = hipFuncSetAttribute((const void *)wide_scores_kernel<QW, P, F>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)WideShape<QW>::lds);
            if (err != hipSuccess) return;
            attr = true;
        }
        hipLaunchKernelGGL((wide_scores_kernel<QW, P, F>), dim3(grid), dim3(WD_THREADS), WideShape<QW>::lds,
                           stream, wp);
        err = hipGetLastError();
    };
    if (wp.pilot) go(std::true_type(), std::false_type());
    else if (wp.tmask) go(std::false_type(), std::true_type());
    else go(std::false_type(), std::false_type());
    return err;
}

}  // namespace

// The batched path's kernels take 2-, 3-, 4- and 8-bit codes in whole rings
// of 4 chunks (d a multiple of 128, and of 256 at b = 2).
bool batch_search_supported(const ScanShape &s, int k) {
    return (s.bits == 2 || s.bits == 3 || s.bits == 4 || s.bits == 8) && s.chunks % 4 == 0 &&
           k <= kMaxBatchK && s.W <= 64 &&
           score_lds(s.bits, s.chunks, score_replicas(s.bits, s.chunks)) <= 160 * 1024 &&
           rescore_lds(s, batch_candidates(k)) <= 160 * 1024;
}

bool mfma_search_supported(const ScanShape &s, int k) {
    return s.bits == 4 && s.chunks % 8 == 0 && s.d <= 1792 && batch_search_supported(s, k);
}

// The score matrix of a tile of 32 queries within 1 GiB (N up to 16.7M).
bool batch_matrix_fits(const ScanShape &s) {
    return (size_t)kTile * approx_row(s) * 2 <= (size_t)1 << 30;
}

BatchPlan batch_plan(const ScanShape &s, int64_t nq, int k, int grid, bool calibrated, size_t room) {
    BatchPlan p;
    for (bool wide = wide_pass(s, nq, batch_candidates(k), grid);; wide = false) {
        for (int tiles = group_tiles(s, nq, k, grid, wide); tiles >= 1; --tiles) {
            const BatchLayout L = batch_layout(s, nq, k, grid, calibrated, wide, tiles);
            p.bytes = L.total;
            if (L.total > room) continue;
            p.fits = true;
            p.wide = wide;
            p.tiles = tiles;
            p.qconst = L.qconst;
            return p;
        }
        if (!wide) return p;
    }
}

hipError_t update_scale_max(const float *scales, int64_t n, float *smax, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    int64_t g = (n + 255) / 256;
    if (g > 2048) g = 2048;
    hipLaunchKernelGGL(scale_max_kernel, dim3((int)g), dim3(256), 0, stream, scales, n,
                       reinterpret_cast<int *>(smax));
    return hipGetLastError();
}

hipError_t mfma_search(const ScanShape &s, const uint8_t *blocked, const float *scales,
                       const float *smax, const uint16_t *tenants, const uint64_t *summaries,
                       const float *cents32, float cmax16, float dmax, const float *Qrot,
                       const float *qconst, int64_t nq, int k,
                       const SearchFilter &filter, int grid, const BatchPlan &plan, void *ws, int64_t *ids,
                       float *scores, int *n_fallback, hipStream_t stream) {
    const uint64_t *allow = filter.allow, *live = filter.live;
    const bool filtered = filter.any();
    const BatchLayout L = batch_layout(s, nq, k, grid, qconst != nullptr, plan.wide, plan.tiles);
    uint8_t *w8 = static_cast<uint8_t *>(ws);
    _Float16 *q16 = reinterpret_cast<_Float16 *>(w8 + L.q16);
    QInfo *info = reinterpret_cast<QInfo *>(w8 + L.info);
    _Float16 *approx = reinterpret_cast<_Float16 *>(w8 + L.approx);
    _Float16 *bmax = reinterpret_cast<_Float16 *>(w8 + L.bmax);
    int *top_i = reinterpret_cast<int *>(w8 + L.top_i);
    float *top_s = reinterpret_cast<float *>(w8 + L.top_s);
    float *amin = reinterpret_cast<float *>(w8 + L.amin);
    int *state = reinterpret_cast<int *>(w8 + L.state);
    int *tickets = reinterpret_cast<int *>(w8 + L.tickets);
    int *counts = tickets + (size_t)grid * kTicketStride;
    uint32_t *tmask = filtered ? reinterpret_cast<uint32_t *>(w8 + L.tmask) : nullptr;
    int *list = reinterpret_cast<int *>(w8 + L.list);
    int *count = reinterpret_cast<int *>(w8 + L.count);
    int *rows = reinterpret_cast<int *>(w8 + L.rows);
    float *qc = reinterpret_cast<float *>(w8 + L.qc);
    float *qconst_c = reinterpret_cast<float *>(w8 + L.qconst_c);
    uint64_t *allow_c = reinterpret_cast<uint64_t *>(w8 + L.allow_c);
    void *lut_ws = w8 + L.lut;
    int *lut_bounds = lut_search_bounds(s, nq, k, grid, lut_ws);
    const int64_t npad = approx_row(s);
    const int KC = batch_candidates(k);   // candidates per query
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)final_select_kernel,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(kFinalMax * 8));
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)pilot_select_kernel,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kPilotMax * 2);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    // The scan of a pass's queries against the pass (see Gate; the explicit
    // path always runs the pass).  Both read 5 MB a us, a tile the union's
    // blocks only.  Measured at 16,000 vectors, d = 1536, k = 10, in us:
    //  - the scan, a query: 12 (8 bits 31) where every workgroup has a block of
    //    it and builds its table, 2.5 and 5 of that reading; 6 (2.8) where few
    //    have one, one tenant of 16 neighbours.  9 and 30 lean to the pass,
    //    which costs the same whatever the allowlists;
    //  - the tiles of 32, 64 and 256 queries with one tenant each: 73, 80 and 90
    //    (8 bits 95, 101, 112), 15 of them for the rotation and the scan's own
    //    launches.  58 (83) shared by the tiles of the group and 8 a tile more
    //    are 4 a tile too many;
    //  - a wide pass: 930 and 255 a call of 256 queries at 1,000,000 vectors, d =
    //    1536 (768 MB) and 256 (128 MB): 150 and 1 a MB.
    const double block_bytes = s.chunks * 1024.0;
    auto gate_of = [&](int QP, int tiles) {
        Gate g{};
        if (!allow || n_fallback) return g;
        g.counts = counts;
        g.scan_us = s.bits == 8 ? 30.f : 9.f;
        g.block_us = (float)(block_bytes / 5.0e6);
        if (QP == kTile) {
            g.pass_us = (s.bits == 8 ? 83.f : 58.f) / tiles + (tiles > 1 ? 8.f : 0.f);
            g.read_us = g.block_us;
        } else {
            g.pass_us = (float)(150.0 + (double)s.nblk * block_bytes / 1.0e6);
        }
        return g;
    };
    auto apply_filter = [&](int64_t q0, int nqt, int QP) {
        FilterParams fp{};
        fp.allow = allow ? allow + q0 * s.W : nullptr;
        fp.live = live;
        fp.summaries = summaries;
        fp.nblk = s.nblk;
        fp.W = s.W;
        fp.nqt = nqt;
        fp.words = QP / 32;
        fp.tmask = tmask;
        fp.counts = counts;
        if (QP == kTile) {
            fp.list = list;
            fp.bmax = reinterpret_cast<uint16_t *>(bmax);
        }
        const int64_t mask_wgs = (64 * (int64_t)s.W * fp.words + FK_THREADS - 1) / FK_THREADS;
        const unsigned tiles = QP == kTile ? (nqt + kTile - 1) / kTile : 1;
        hipLaunchKernelGGL(filter_kernel,
                           dim3((unsigned)(mask_wgs + (s.nblk + FK_THREADS - 1) / FK_THREADS), tiles),
                           dim3(FK_THREADS), 0, stream, fp);
    };
    auto rescore = [&](int64_t q0, int nqt, const int *ti, const float *ts, const float *am, const int *st,
                       const QInfo *qi, const Gate &gate, int tile_q) {
        RescoreParams rp{};
        rp.codes = reinterpret_cast<const uint4 *>(blocked);
        rp.scales = scales;
        rp.qrot = Qrot + q0 * s.d;
        rp.qconst = qconst ? qconst + q0 : nullptr;
        rp.cents = cents32;
        rp.top_i = ti;
        rp.top_s = ts;
        rp.amin = am;
        rp.state = st;
        rp.info = qi;
        rp.ids = ids + q0 * k;
        rp.scores = scores + q0 * k;
        rp.fb_count = count;
        rp.fb_rows = rows;
        rp.fb_q = qc;
        rp.fb_const = qconst_c;
        rp.fb_allow = allow_c;
        rp.fb_bound = lut_bounds;
        rp.allow = allow ? allow + q0 * s.W : nullptr;
        rp.W = s.W;
        rp.q0 = (int)q0;
        rp.nqt = nqt;
        rp.tile_q = tile_q;
        rp.gate = gate;
        rp.d = s.d;
        rp.bits = s.bits;
        rp.chunks = s.chunks;
        rp.lut_words = rescore_lut_words(s);
        rp.k = k;
        return launch_rescore(s, KC, rp, nqt, stream);
    };
    for (int64_t q0 = 0; q0 < nq;) {
        if (L.wide && wide_pass(s, nq - q0, KC, grid)) {
            // a wide pass of up to kWideMaxQ queries
            const int nqt = (int)std::min<int64_t>(nq - q0, kWideMaxQ);
            constexpr int QP = kWideMaxQ;
            const int PCM = 2 * KC;
            const WideGeom w = wide_geom(s, WD_NG, grid, KC);
            _Float16 *wq16 = reinterpret_cast<_Float16 *>(w8 + L.w_q16);
            QInfo *winfo = reinterpret_cast<QInfo *>(w8 + L.w_info);
            uint4 *wqfrag = reinterpret_cast<uint4 *>(w8 + L.w_qfrag);
            float *wqf = reinterpret_cast<float *>(w8 + L.w_qf);
            float *wpil = reinterpret_cast<float *>(w8 + L.w_pil);
            float *wtheta = reinterpret_cast<float *>(w8 + L.w_theta);
            int *wpcn = reinterpret_cast<int *>(w8 + L.w_pcn);
            int *wpci = reinterpret_cast<int *>(w8 + L.w_pci);
            float *wpcs = reinterpret_cast<float *>(w8 + L.w_pcs);
            float *wcs = reinterpret_cast<float *>(w8 + L.w_cs);
            int *wci = reinterpret_cast<int *>(w8 + L.w_ci);
            int *wcn = reinterpret_cast<int *>(w8 + L.w_cn);
            int *wtop = reinterpret_cast<int *>(w8 + L.w_top);
            float *wtops = reinterpret_cast<float *>(w8 + L.w_tops);
            float *wamin = reinterpret_cast<float *>(w8 + L.w_amin);
            int *wstate = reinterpret_cast<int *>(w8 + L.w_state);
            const uint64_t *allow_p = allow ? allow + q0 * s.W : nullptr;
            const Gate gate = gate_of(QP, 1);
            hipLaunchKernelGGL(prep_kernel, dim3(nqt), dim3(SEL_THREADS), 0, stream,
                               Qrot + q0 * s.d, qconst ? qconst + q0 : nullptr, nqt, s.d, s.bits, smax,
                               cmax16, dmax, wq16, winfo,
                               counts, 2, q0 == 0 ? count : nullptr);
            if (filtered) apply_filter(q0, nqt, QP);
            const int64_t fr = (int64_t)(s.d / 32) * QP * 4;
            hipLaunchKernelGGL(frag_kernel, dim3((int)std::min<int64_t>((fr + 255) / 256, 1024)),
                               dim3(256), 0, stream, wq16, winfo, nqt, QP, s.d, wqfrag, wqf);
            WideParams wp{};
            wp.codes = reinterpret_cast<const uint4 *>(blocked);
            wp.scales = scales;
            wp.qfrag = wqfrag;
            wp.qf = wqf;
            wp.cents = cents32;
            wp.n = s.n;
            wp.nblk = s.nblk;
            wp.ntiles = w.ntiles;
            wp.chunks = s.chunks;
            wp.pstride = w.pstride;
            wp.npil = w.npil;
            wp.pil = wpil;
            wp.theta = wtheta;
            wp.tenants = tenants;
            wp.tmask = tmask;
            wp.live = live;
            wp.gate = gate;
            wp.nqt = nqt;
            wp.cand_s = wcs;
            wp.cand_i = wci;
            wp.cand_n = wcn;
            wp.S = w.S;
            wp.pilot = 1;
            hipError_t e = launch_wide_scores(wp, grid, stream);
            if (e != hipSuccess) return e;
            PilotParams pp{};
            pp.pil = wpil;
            pp.npv = (int64_t)w.npil * w.tilev;
            pp.pstride = w.pstride;
            pp.n = s.n;
            pp.tenants = tenants;
            pp.allow = allow_p;
            pp.live = live;
            pp.gate = gate;
            pp.nqt = nqt;
            pp.W = s.W;
            pp.PCM = PCM;
            const double part = (double)w.ntiles / (double)w.npil;
            pp.rank = pilot_rank(part, KC);
            pp.groups = KC <= 128 ? 1 : KC / 128;
            pp.most = (int)std::min(1.25 * pp.rank, pilot_most(part, KC));
            pp.theta = wtheta;
            pp.pc_n = wpcn;
            pp.pc_i = wpci;
            pp.pc_s = wpcs;
            hipLaunchKernelGGL(pilot_select_kernel, dim3(nqt), dim3(PS_THREADS), (size_t)pp.npv * 2, stream,
                               pp);
            wp.pilot = 0;
            e = launch_wide_scores(wp, grid, stream);
            if (e != hipSuccess) return e;
            FinalParams fp{};
            fp.theta = wtheta;
            fp.pc_n = wpcn;
            fp.pc_i = wpci;
            fp.pc_s = wpcs;
            fp.PCM = PCM;
            fp.cand_s = wcs;
            fp.cand_i = wci;
            fp.cand_n = wcn;
            fp.G = grid;
            fp.QP = QP;
            fp.S = w.S;
            fp.KC = KC;
            fp.nqt = nqt;
            fp.gate = gate;
            fp.top_i = wtop;
            fp.top_s = wtops;
            fp.amin = wamin;
            fp.state = wstate;
            hipLaunchKernelGGL(final_select_kernel, dim3(nqt), dim3(PS_THREADS),
                               (size_t)kFinalMax * 8, stream, fp);
            e = hipGetLastError();
            if (e == hipSuccess) e = rescore(q0, nqt, wtop, wtops, wamin, wstate, winfo, gate, QP);
            if (e != hipSuccess) return e;
            q0 += nqt;
            continue;
        }
        // a group of tiles
        const int nqt = (int)std::min<int64_t>(nq - q0, (int64_t)L.tiles * kTile);
        const int tiles = (nqt + kTile - 1) / kTile;
        // its workgroups, as many for each tile: the tiles read the codes at
        // the same time, one of them from HBM and the others from the caches
        int per_tile = grid / tiles;
        if (per_tile > 8) per_tile &= ~7;
        hipLaunchKernelGGL(prep_kernel, dim3(nqt), dim3(SEL_THREADS), 0, stream, Qrot + q0 * s.d,
                           qconst ? qconst + q0 : nullptr, nqt, s.d, s.bits, smax, cmax16, dmax, q16, info, tickets,
                           grid * kTicketStride + 2 * kGroupTiles, q0 == 0 ? count : nullptr);
        const Gate gate = gate_of(kTile, tiles);
        if (filtered) apply_filter(q0, nqt, kTile);
        ScoreParams sp{};
        sp.codes = reinterpret_cast<const uint4 *>(blocked);
        sp.scales = scales;
        sp.q16 = q16;
        sp.info = info;
        sp.cents = cents32;
        sp.out = approx;
        sp.bmax = bmax;
        sp.n = s.n;
        sp.nblk = s.nblk;
        sp.npad = npad;
        sp.d = s.d;
        sp.chunks = s.chunks;
        sp.nqt = nqt;
        sp.tickets = tickets;
        sp.tiles = tiles;
        sp.W = s.W;
        if (filtered) {
            sp.list = list;
            sp.counts = counts;
            sp.tmask = tmask;
            sp.tenants = tenants;
            sp.live = live;
            sp.gate = gate;
        }
        hipError_t e = launch_scores(s.bits, sp, per_tile * tiles, stream);
        if (e != hipSuccess) return e;
        BlockSelParams bp{};
        bp.approx = reinterpret_cast<const uint16_t *>(approx);
        bp.bmax = reinterpret_cast<const uint16_t *>(bmax);
        bp.top_i = top_i;
        bp.top_s = top_s;
        bp.amin = amin;
        bp.state = state;
        bp.n = s.n;
        bp.nblk = s.nblk;
        bp.npad = npad;
        bp.KC = KC;
        bp.nqt = nqt;
        bp.gate = gate;
        hipLaunchKernelGGL(block_select_kernel, dim3(nqt), dim3(BS_THREADS), 0, stream, bp);
        e = hipGetLastError();
        if (e == hipSuccess) e = rescore(q0, nqt, top_i, top_s, amin, state, info, gate, kTile);
        if (e != hipSuccess) return e;
        q0 += nqt;
    }
    // queries whose top k is not proven run on the single-query scan
    SearchFilter f;
    f.allow = allow ? allow_c : nullptr;
    f.live = live;
    QueryRows qr;
    qr.count = count;
    qr.rows = rows;
    hipError_t e = lut_search(s, blocked, scales, tenants, summaries, cents32, qc, nq, k, f, grid, lut_ws,
                              lut_search_workspace_bytes(s, nq, k, grid), ids, scores, stream,
                              qconst ? qconst_c : nullptr,
                              lut_bounds != nullptr, qr);
    if (e != hipSuccess || !n_fallback) return e;
    e = hipMemcpyAsync(n_fallback, count, sizeof(int), hipMemcpyDeviceToHost, stream);
    return e == hipSuccess ? hipStreamSynchronize(stream) : e;
}

}  // namespace tq
