// Assignment step for many clusters (k > 64) of fp32 and fp16 rows with up to 128 columns, at fp32 accuracy on the
// bf16 matrix cores.
//
// What it computes (EmbedPart paper, Alg. 3, step P <- KMeans(E, k)): labels[i] = argmin_j ||x_i - c_j||^2
// = argmax_j (x_i.c_j - ||c_j||^2 / 2), lowest j on ties.
//
//  1. blocks_prep_kernel writes one record per 32 centroids: the exact three-way bf16 split of their elements in the
//     lane order of the operand of v_mfma_f32_32x32x16_bf16 (columns past d and centroids past k as zeros) and the 32
//     values -||c||^2/2.  It also clears the packed winners.
//  2. blocks_assign_kernel: a wave keeps the exact terms (fp32: three, fp16: two) of 32 PT points in registers and
//     walks the records, which the 8 waves of a workgroup share through a 3-deep LDS ring (LDS-direct loads).  x.c is
//     six products of the terms (fp16: five).  Centroids are the rows of the product, so a lane holds 16 scores of one
//     point and folds them in ascending order without a lane exchange, while the next chain of products runs.
//     The (block of points, record) pairs are dealt to 256 workgroups in contiguous runs of equal length, so a last
//     wave of workgroups that fills a part of the chip does not exist and few rows still use all of it; a point's
//     winners from several runs meet in a 64-bit atomic maximum of (score, -index), whose result does not depend on
//     the order.
//  3. blocks_finish_kernel unpacks the winners and forms ||x - c||^2.
//
// What bounds it: the matrix pipe (6 bf16 products per fp32 product) at the clock that the chip's power allows.  The
// points' terms are formed once per run; walking the rows once per 64 centroids, as the k <= 64 kernel does, splits
// and reads every row k / 64 times and issues as many vector as matrix instructions.
// Measured at 400,000 x 128 fp32, k = 1,000: 498 us per assignment = 1.26 PFLOP/s of bf16 products; with one pass of the
// k <= 64 kernel per 64 centroids 1,060 us.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "small_common.h"

namespace ep {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int kTile = 32;      // centroids per record, points per operand tile
constexpr int kTerms = 3;      // terms of a centroid element
constexpr int kGridMax = 256;  // one workgroup of 8 waves per compute unit

constexpr int record_bytes(int ns) { return ns * kTerms * 1024 + kTile * 4; }
int k_steps(int32_t d) { return 2 * (int)ceil_div(d, 32); }   // K-steps of 16 columns, an even number

// ---- 1. records -----------------------------------------------------------------------------------
// One wave per (padded) centroid; a unit is the 8 columns that a lane of the product holds in one K-step.
// winner: cleared if it is given (n entries).
__global__ __launch_bounds__(256) void blocks_prep_kernel(int64_t n, int32_t d, int32_t k, int32_t ns,
                                                          const float *__restrict__ C, unsigned char *__restrict__ records,
                                                          unsigned long long *__restrict__ winner) {
    if (winner)
        for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) winner[i] = 0;
    const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // below the padded count by the grid's size
    const int lane = threadIdx.x & 63;
    const bool real = j < k;
    unsigned char *rec = records + (j / kTile) * record_bytes(ns);
    double acc = 0.0;
    if (lane < 2 * ns) {
        const int s = lane >> 1, half = lane & 1;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int col = 16 * s + 8 * half + e;
            v[e] = real && col < d ? C[j * d + col] : 0.f;
            acc += (double)v[e] * (double)v[e];
        }
        u32x4 h, m, l;
#pragma unroll
        for (int pr = 0; pr < 4; ++pr) {
            const Split3 t = split3_pair(v[2 * pr], v[2 * pr + 1]);
            h[pr] = t.h, m[pr] = t.m, l[pr] = t.l;
        }
        u32x4 *piece = reinterpret_cast<u32x4 *>(rec) + s * kTerms * 64 + 32 * half + j % kTile;
        piece[0] = h;
        piece[64] = m;
        piece[128] = l;
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    // a centroid past k never wins: no score is above minus infinity
    if (lane == 0) reinterpret_cast<float *>(rec + ns * kTerms * 1024)[j % kTile] = real ? (float)(-0.5 * acc) : -__builtin_inff();
}

// ---- 2. assignment ----------------------------------------------------------------------------------
// Scores order as the high word, lower indices win ties; 0 is below every score (and is not one).
__device__ __forceinline__ unsigned long long pack_winner(float score, uint32_t idx) {
    const uint32_t b = __float_as_uint(score + 0.f);   // one zero
    const uint32_t key = b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
    return ((unsigned long long)key << 32) | (0xFFFFFFFFu - idx);
}
__device__ __forceinline__ float winner_score(unsigned long long w) {
    const uint32_t key = (uint32_t)(w >> 32);
    return __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

// first_centroid: the index of the first record's first centroid.
// XN: also ||x||^2 of every row into norms (the labels' buffer: they are written by the last kernel).
template <typename XT, int NS, int PT, bool XN>
__global__ __launch_bounds__(kThreads, 2) void blocks_assign_kernel(int64_t n, int32_t d, int64_t ld, int32_t tiles,
                                                                    int64_t units, int32_t first_centroid, const XT *__restrict__ X,
                                                                    const unsigned char *__restrict__ records,
                                                                    unsigned long long *__restrict__ winner,
                                                                    float *__restrict__ norms) {
    constexpr bool kF32 = std::is_same<XT, float>::value;
    constexpr int TX = kF32 ? 3 : 2;
    constexpr int REC = record_bytes(NS), REC16 = REC / 16, STAGE = (REC16 + kThreads - 1) / kThreads;
    constexpr int kRows = kWaves * PT * kTile;   // rows of a block
    __shared__ __attribute__((aligned(16))) unsigned char ring[3][REC];
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    typedef __attribute__((address_space(3))) void *lds_ptr;
    auto stage = [&](int tile, int slot) {
        const uint4 *src = reinterpret_cast<const uint4 *>(records + (int64_t)tile * REC);
#pragma unroll
        for (int q = 0; q < STAGE; ++q) {
            const int wave_piece = q * kThreads + wave * 64;   // uniform
            if (wave_piece + lane < REC16)
                __builtin_amdgcn_global_load_lds(src + wave_piece + lane, (lds_ptr)(ring[slot] + wave_piece * 16), 16, 0, 0);
        }
    };
    auto load_bias = [&](const unsigned char *rec) {   // of the 16 centroids this lane's accumulators stand for
        f32x16 b;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 b4 = *reinterpret_cast<const f32x4 *>(rec + NS * kTerms * 1024 + (8 * q + 4 * half) * 4);
            b[4 * q + 0] = b4[0];
            b[4 * q + 1] = b4[1];
            b[4 * q + 2] = b4[2];
            b[4 * q + 3] = b4[3];
        }
        return b;
    };

    const int64_t lo = units * blockIdx.x / gridDim.x, hi = units * (blockIdx.x + 1) / gridDim.x;
    for (int64_t u = lo; u < hi;) {
        const int64_t pb = u / tiles;
        const int t0 = (int)(u % tiles), t1 = (int)min((int64_t)tiles, t0 + (hi - u));
        u += t1 - t0;
        __syncthreads();   // the previous run's readers are done with the ring
        stage(t0, 0);
        if (t0 + 1 < t1) stage(t0 + 1, 1);

        // The points' terms: lane (half, col) holds columns 16 s + 8 half .. + 7 of point col of an operand tile.  Rows
        // past the end are read as the last row and ignored; a 16-byte piece that starts past the last column is read
        // from column 0 (one that holds any column ends inside the row's stride) and columns past d become zeros.
        const int64_t row0 = pb * kRows + wave * (PT * kTile) + col;
        u32x4 xt[PT][NS][TX];
        float xn[PT];
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int64_t row = row0 + p * kTile;
            const XT *x = X + (row < n ? row : n - 1) * ld;
            xn[p] = 0.f;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int c0 = 16 * s + 8 * half;
                float v[8];
                if constexpr (kF32) {
                    const f32x4 a = *reinterpret_cast<const f32x4 *>(x + (c0 < d ? c0 : 0));
                    const f32x4 b = *reinterpret_cast<const f32x4 *>(x + (c0 + 4 < d ? c0 + 4 : 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = a[e], v[4 + e] = b[e];
                } else {
                    typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
                    const f16x8_t hv = *reinterpret_cast<const f16x8_t *>(x + (c0 < d ? c0 : 0));
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = (float)hv[e];
                }
                if (d < 16 * NS) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = c0 + e < d ? v[e] : 0.f;
                }
                if (XN) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) xn[p] = fmaf(v[e], v[e], xn[p]);
                }
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) {
                    const Split3 t = split3_pair(v[2 * pr], v[2 * pr + 1]);
                    xt[p][s][0][pr] = t.h;
                    xt[p][s][1][pr] = t.m;
                    if constexpr (TX > 2) xt[p][s][2][pr] = t.l;
                }
            }
        }
        if (XN && t0 == 0) {   // one run has the block's first record
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const float x2 = xn[p] + __shfl_xor(xn[p], 32, 64);
                const int64_t row = row0 + p * kTile;
                if (half == 0 && row < n) norms[row] = x2;
            }
        }
        float best[PT];
        int32_t code[PT];   // 16 tile + accumulator
#pragma unroll
        for (int p = 0; p < PT; ++p) best[p] = -__builtin_inff(), code[p] = 0;
        auto fold = [&](float s, int p, int at) {   // strict >: the lower index keeps a tie; a NaN never wins
            const bool better = s > best[p];
            best[p] = better ? s : best[p];
            code[p] = better ? at : code[p];
        };
        __syncthreads();   // records t0 and t0 + 1 are there

        // One chain of products per record and point tile; two accumulators in turn, the finished one is folded
        // between the products of the running one.
        f32x16 acc[2];
        int slot = 0;
        auto tile_step = [&](int t, auto parity, bool have_prev) {
            constexpr int P0 = decltype(parity)::value;   // accumulator of the first chain
            if (t + 2 < t1) stage(t + 2, slot >= 1 ? slot - 1 : 2);
            const unsigned char *rec = ring[slot];
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const int cur = (P0 + p) & 1;
                const int pp = p > 0 ? p - 1 : PT - 1, pt = p > 0 ? t : t - 1;
                acc[cur] = load_bias(rec);
                u32x4 a[2][kTerms];
#pragma unroll
                for (int ct = 0; ct < kTerms; ++ct) a[0][ct] = *reinterpret_cast<const u32x4 *>(rec + (ct * 64 + lane) * 16);
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (s + 1 < NS) {
#pragma unroll
                        for (int ct = 0; ct < kTerms; ++ct)
                            a[(s + 1) & 1][ct] = *reinterpret_cast<const u32x4 *>(rec + (((s + 1) * kTerms + ct) * 64 + lane) * 16);
                    }
                    // small products first: cl.xh; cm.xm, cm.xh; ch.xl, ch.xm, ch.xh
#pragma unroll
                    for (int ct = kTerms - 1; ct >= 0; --ct)
#pragma unroll
                        for (int tx = TX - 1; tx >= 0; --tx)
                            if (ct + tx < 3)
                                acc[cur] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                    __builtin_bit_cast(bf16x8_t, a[s & 1][ct]), __builtin_bit_cast(bf16x8_t, xt[p][s][tx]),
                                    acc[cur], 0, 0, 0);
                    if (p > 0 || have_prev) {
#pragma unroll
                        for (int v = 16 * s / NS; v < 16 * (s + 1) / NS; ++v) fold(acc[cur ^ 1][v], pp, 16 * pt + v);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            slot = slot == 2 ? 0 : slot + 1;
            __syncthreads();   // the next record is there, this one's slot is free
        };
        auto fold_last = [&](auto parity) {
#pragma unroll
            for (int v = 0; v < 16; ++v) fold(acc[decltype(parity)::value][v], PT - 1, 16 * (t1 - 1) + v);
        };
        using Even = std::integral_constant<int, 0>;
        using Odd = std::integral_constant<int, 1>;
        if constexpr (PT % 2 == 0) {
            tile_step(t0, Even(), false);
            for (int t = t0 + 1; t < t1; ++t) tile_step(t, Even(), true);
            fold_last(Odd());
        } else {
            tile_step(t0, Even(), false);
            int t = t0 + 1;
            for (; t + 1 < t1; t += 2) {
                tile_step(t, Odd(), true);
                tile_step(t + 1, Even(), true);
            }
            if (t < t1) {
                tile_step(t, Odd(), true);
                fold_last(Odd());
            } else {
                fold_last(Even());
            }
        }
        // accumulator v of a lane is row 8 (v / 4) + 4 half + v % 4 of the tile
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            float b = best[p];
            int32_t i = first_centroid + (code[p] >> 4) * kTile + 8 * ((code[p] & 15) >> 2) + 4 * half + (code[p] & 3);
            const float ob = __shfl_xor(b, 32, 64);
            const int32_t oi = __shfl_xor(i, 32, 64);
            if (ob > b || (ob == b && oi < i)) b = ob, i = oi;
            const int64_t row = row0 + p * kTile;
            if (half == 0 && row < n && b > -__builtin_inff()) atomicMax(&winner[row], pack_winner(b, (uint32_t)i));
        }
    }
}

// ---- 3. labels, distances, the rest of the objective ---------------------------------------------------
// A row without a winner has an infinity, a NaN or a value whose split overflows, or no centroid gives it a score.
template <typename XT>
__global__ __launch_bounds__(256) void blocks_finish_kernel(int64_t n, int32_t d, int64_t ld, int32_t k, bool want_d2,
                                                            const XT *__restrict__ X, const float *__restrict__ C,
                                                            const unsigned long long *__restrict__ winner,
                                                            int32_t *__restrict__ labels, float *__restrict__ min_d2,
                                                            double *__restrict__ obj_part) {
    __shared__ double red[4];
    double obj = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const unsigned long long w = winner[i];
        int32_t idx = (int32_t)(0xFFFFFFFFu - (uint32_t)w);
        float s = winner_score(w);
        const float xn = want_d2 ? __int_as_float(labels[i]) : 0.f;
        if (__builtin_expect(w == 0, 0)) {
            idx = 0;
            s = kNoScore;
            plain_scores(X + i * ld, d, C, k, s, idx, [&](int32_t j) {
                double c2 = 0.0;
                for (int m = 0; m < d; ++m) c2 += (double)C[(int64_t)j * d + m] * (double)C[(int64_t)j * d + m];
                return (float)(-0.5 * c2);
            });
        }
        labels[i] = idx;
        if (want_d2) {
            const float d2 = fmaxf(xn - 2.f * s, 0.f);
            obj += (double)d2;
            if (min_d2) min_d2[i] = d2;
        }
    }
    if (want_d2) {
        for (int off = 32; off > 0; off >>= 1) obj += __shfl_down(obj, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = obj;
        __syncthreads();
        if (threadIdx.x == 0) obj_part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
    }
}

__global__ __launch_bounds__(64) void blocks_objective_kernel(const double *__restrict__ part, int count,
                                                              double *__restrict__ out) {
    double o = 0.0;
    for (int q = threadIdx.x; q < count; q += 64) o += part[q];
    for (int off = 32; off > 0; off >>= 1) o += __shfl_down(o, off, 64);
    if (threadIdx.x == 0) *out = o;
}

template <typename XT>
int launch_blocks(const ep_problem &p, const XT *X, const float *C, const KmeansWs &w, int32_t *labels, float *min_d2,
                  double *objective, hipStream_t s) {
    constexpr bool kF32 = std::is_same<XT, float>::value;
    const int ns = k_steps(p.d), all_tiles = (int)ceil_div(p.k, kTile);
    const bool xn = min_d2 || objective;
    for (int first = 0; first < all_tiles; first += w.block_slice) {   // once, unless the workspace is the static array
        const int tiles = std::min(w.block_slice, all_tiles - first);
        blocks_prep_kernel<<<(unsigned)(tiles * (kTile / 4)), 256, 0, s>>>(p.n, p.d, p.k - first * kTile, ns,
                                                                           C + (int64_t)first * kTile * p.d, w.block_records,
                                                                           first == 0 ? w.winner : nullptr);
        EP_LAUNCH_CHECK();
        auto go = [&](auto ns_, auto pt_) {
            constexpr int NS = decltype(ns_)::value, PT = decltype(pt_)::value;
            const int64_t units = ceil_div(p.n, (int64_t)kWaves * PT * kTile) * tiles;
            const int wgs = (int)std::min<int64_t>(units, kGridMax);
            const bool norms = xn && first == 0;
            ProfScope prof(EP_PROF_LLOYD_MAIN, s);
            auto kern = norms ? blocks_assign_kernel<XT, NS, PT, true> : blocks_assign_kernel<XT, NS, PT, false>;
            kern<<<wgs, kThreads, 0, s>>>(p.n, p.d, p.ld, tiles, units, first * kTile, X, w.block_records, w.winner,
                                          reinterpret_cast<float *>(labels));
            EP_LAUNCH_CHECK();
            return (int)EP_OK;
        };
        // point tiles per wave: as many as leave the terms at most 128 of the 256 registers
#define EP_BLOCKS(NS_, PT_F32_, PT_F16_) go(std::integral_constant<int, NS_>(), std::integral_constant<int, kF32 ? PT_F32_ : PT_F16_>())
        const int rc = ns == 2 ? EP_BLOCKS(2, 4, 4) : ns == 4 ? EP_BLOCKS(4, 2, 2) : ns == 6 ? EP_BLOCKS(6, 1, 2) : EP_BLOCKS(8, 1, 2);
#undef EP_BLOCKS
        if (rc != EP_OK) return rc;
    }
    const int blocks = (int)std::min<int64_t>(512, ceil_div(p.n, 256));   // few partials: one wave adds them
    blocks_finish_kernel<XT><<<blocks, 256, 0, s>>>(p.n, p.d, p.ld, p.k, xn, X, C, w.winner, labels, min_d2,
                                                    w.obj_part);
    EP_LAUNCH_CHECK();
    if (objective) {
        blocks_objective_kernel<<<1, 64, 0, s>>>(w.obj_part, blocks, objective);
        EP_LAUNCH_CHECK();
    }
    return EP_OK;
}

}  // namespace

// 128 columns: the terms of 32 points of fp32 rows are 96 registers then.
bool blocks_path_supported(const ep_problem &p) {
    return (p.dtype == EP_F32 || p.dtype == EP_F16) && p.k > 64 && p.d <= 128;
}

size_t block_record_bytes(const ep_problem &p) { return (size_t)record_bytes(k_steps(p.d)); }

int launch_blocks_assign(const ep_problem &p, const void *X, const float *C, const KmeansWs &w, int32_t *labels,
                         float *min_d2, double *objective, hipStream_t s) {
    return p.dtype == EP_F32 ? launch_blocks(p, static_cast<const float *>(X), C, w, labels, min_d2, objective, s)
                             : launch_blocks(p, static_cast<const f16_t *>(X), C, w, labels, min_d2, objective, s);
}

}  // namespace ep
