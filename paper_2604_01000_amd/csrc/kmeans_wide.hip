// Assignment and update for the widths and cluster counts that the fused kernels (kmeans_small.hip) and the
// reordering-scale kernel (kmeans_large.hip) do not cover: any d up to 1,024 (odd ones included), any row
// stride, any k, fp32, bfloat16 and fp16 rows.
//
// What they compute (EmbedPart paper, Alg. 3, step P <- KMeans(E, k)): labels[i] = argmin_j ||x_i - c_j||^2
// = argmax_j (x_i.c_j - ||c_j||^2 / 2), lowest j on ties, and for k <= 64 the per-cluster sums and counts.
//
//  1. wide_prep_kernel writes the centroids as matrix-instruction operands ("records"): blocks of 16 KT
//     centroids, K-steps of 32 columns, columns past d and centroids past k as zeros.  fp32 and fp16 rows: the
//     exact three-way bf16 split of every centroid element; bfloat16 rows: the centroid rounded to bfloat16.
//  2. wide_assign_kernel: a wave owns 16 PT points and walks the columns 32 at a time with all centroids of a
//     block in its accumulators (centroids are the rows of the product, points the columns, so a lane ends
//     with 4 KT scores of one point and the arg-max needs two lane exchanges per point tile).  x.c of fp32
//     rows is six bf16 products of the exact splits, of fp16 rows five (two terms hold an fp16), of bfloat16
//     rows one: as accurate as fp32 fused multiply-adds at several times their rate.
//     The records pass through LDS in panels; with one centroid block that fits they are staged once for the
//     life of the workgroup.
//  3. wide_sums_kernel (k <= 64): sums[centroid][column] += onehot[centroid][point] x[point][column] on the
//     matrix cores, the rows again as exact bf16 terms (fp16 rows: one fp16 product), so that every product is
//     exact and only the fp32 accumulation rounds.  A lane reads whole 16-byte pieces of a row and its tile t is
//     column NC c + t of the slab, so the transposed operand needs no trip through LDS.  Unlike a table of sums
//     in LDS its cost does not depend on how the labels collide, and unlike sorting the rows it reads them in
//     order.
//  4. wide_finalize_kernel: fp64 sum of the partials in a fixed order, means.
//
// What bounds them: memory, twice over X per round (the sums need the labels of whole rows).  Measured per round at
// 500,003 x 256 fp32, k = 32: assignment 99 us = 5.2 TB/s, sums 86 us = 6.0 TB/s (104 and 91 us with one K-step in flight
// and parts of consecutive rows); on the vector unit (one point per lane, then a table of sums in LDS, then one thread
// adding 1,024 partials) 474 + 465 + 258 us, and a single thread adding the objective 117 us.  200,003 x 516 bf16,
// k = 20: 47 + 41 us (the sums 46 us with two waves more than are resident at once) against 353 us + 62 ms (one wave per
// cluster walked its rows).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "kernels.h"
#include "small_common.h"

namespace ep {

namespace {

constexpr int kStep = 32;              // columns per K-step
constexpr int kPanelBytes = 144 * 1024;   // LDS for records (one workgroup per compute unit)
constexpr int kAssignThreads = 512;

template <typename XT> constexpr int x_terms() { return std::is_same<XT, float>::value ? 3 : std::is_same<XT, f16_t>::value ? 2 : 1; }
constexpr int c_terms(int dtype) { return dtype == EP_BF16 ? 1 : 3; }

int cent_tiles(int32_t k) { return k >= 64 ? 4 : (int)ceil_div(k, 16); }          // KT
int64_t cent_blocks(int32_t k) { return ceil_div(k, 16 * (int64_t)cent_tiles(k)); }
int64_t k_steps(int32_t d) { return ceil_div(d, kStep); }
int step_bytes(const ep_problem &p) { return c_terms(p.dtype) * cent_tiles(p.k) * 1024; }

// ---- 1. records -----------------------------------------------------------------------------------
// One wave per (padded) centroid.  A unit is the 8 columns that lane (g, c) of the product holds in one K-step:
// fp32 rows 16 q + 4 g .. + 3 for q = 0, 1 (two 16-byte pieces of the row), 2-byte rows 8 g .. + 7 (one piece).
__global__ __launch_bounds__(256) void wide_prep_kernel(int32_t d, int32_t k, int32_t kt, int64_t ksteps, int dtype,
                                                        const float *__restrict__ C, unsigned char *__restrict__ records,
                                                        float *__restrict__ bias, int64_t padded_k) {
    const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= padded_k) return;
    const int lane = threadIdx.x & 63;
    const bool real = j < k;
    const int terms = c_terms(dtype);
    const int64_t block = j / (16 * kt);
    const int mt = (int)(j / 16 % kt), c = (int)(j % 16);
    double acc = 0.0;
    for (int64_t u = lane; u < 4 * ksteps; u += 64) {
        const int64_t ks = u >> 2;
        const int g = (int)(u & 3);
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t col = ks * kStep + (dtype == EP_F32 ? 16 * (e >> 2) + 4 * g + (e & 3) : 8 * g + e);
            v[e] = real && col < d ? C[j * d + col] : 0.f;
            if (dtype == EP_BF16) v[e] = bf16_to_f32(f32_to_bf16_rne(v[e]));
            acc += (double)v[e] * (double)v[e];
        }
        u32x4 h, m, l;
#pragma unroll
        for (int pr = 0; pr < 4; ++pr) {
            const Split3 t = split3_pair(v[2 * pr], v[2 * pr + 1]);
            h[pr] = t.h, m[pr] = t.m, l[pr] = t.l;
        }
        unsigned char *rec = records + ((block * ksteps + ks) * terms * kt + mt) * 1024 + (16 * g + c) * 16;
        *reinterpret_cast<u32x4 *>(rec) = h;
        if (terms == 3) {
            *reinterpret_cast<u32x4 *>(rec + kt * 1024) = m;
            *reinterpret_cast<u32x4 *>(rec + 2 * kt * 1024) = l;
        }
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if (lane == 0) bias[j] = real ? (float)(-0.5 * acc) : -3.0e38f;
}

// ---- 2. assignment ----------------------------------------------------------------------------------
// XN: also ||x||^2 (min_d2 or the objective is wanted).
template <typename XT, int KT, int PT, bool XN>
__global__ __launch_bounds__(kAssignThreads, 2) void wide_assign_kernel(
    int64_t n, int32_t d, int64_t ld, int32_t ksteps, int32_t panel_steps, int32_t blocks_of_centroids,
    const XT *__restrict__ X, const unsigned char *__restrict__ records, const float *__restrict__ bias,
    const float *__restrict__ C, int32_t k, int32_t *__restrict__ labels, float *__restrict__ min_d2,
    double *__restrict__ obj_part) {
    constexpr bool kF32 = std::is_same<XT, float>::value, kBf16 = std::is_same<XT, bf16_t>::value;
    constexpr int CT = kBf16 ? 1 : 3;            // terms of a centroid element
    constexpr int TX = x_terms<XT>();
    constexpr int NP = kF32 ? 2 : 1;             // 16-byte pieces per lane, point tile and K-step
    constexpr int PE = 16 / (int)sizeof(XT);     // elements of a piece
    constexpr int kRec = CT * KT * 1024;
    extern __shared__ __attribute__((aligned(16))) unsigned char panel[];
    __shared__ double red[kAssignThreads / 64];
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int64_t tile_rows = (int64_t)waves * PT * 16;
    const int64_t tiles = (n + tile_rows - 1) / tile_rows;
    const bool resident = blocks_of_centroids == 1 && panel_steps >= ksteps;
    const bool ragged = d % kStep != 0;
    bool staged = false;
    double obj = 0.0;

    // Row pointers of this lane's points in a tile; rows past the end are read as the last row and ignored.
    const XT *row[PT];
    auto point_at = [&](int64_t tile) {
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int64_t i = tile * tile_rows + (wave * PT + p) * 16 + c;
            row[p] = X + (i < n ? i : n - 1) * ld;
        }
    };
    // Raw pieces of a K-step.  A piece that starts past the last column is read from column 0 instead and masked
    // where it is used; one that holds any column ends inside the row (the stride is a multiple of a piece).
    int lks = 0, lcb = 0;   // the step that is loaded next, ahead of the one worked on, in the next tile if need be
    int64_t ltile = blockIdx.x;
    auto load_next = [&](u32x4(&dst)[PT][NP]) {
        if (lks == ksteps) {
            lks = 0;
            if (++lcb == blocks_of_centroids) {
                lcb = 0;
                ltile += gridDim.x;
                point_at(ltile);
            }
        }
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int col = lks * kStep + 4 * PE * q + PE * g;
            const int at = col < d ? col : 0;
#pragma unroll
            for (int p = 0; p < PT; ++p) dst[p][q] = *reinterpret_cast<const u32x4 *>(row[p] + at);
        }
        ++lks;
    };

    float best[PT], xn[PT];
    int32_t bidx[PT];
    f32x4 acc[PT][KT];
    int ks = 0, cb = 0;

    auto step = [&](u32x4(&x)[PT][NP], u32x4(&ahead)[PT][NP]) {
        if (ks % panel_steps == 0 && !staged) {   // uniform over the workgroup
            __syncthreads();
            const int steps = min(panel_steps, ksteps - ks);
            const uint4 *src = reinterpret_cast<const uint4 *>(records + ((int64_t)cb * ksteps + ks) * kRec);
            for (int i = threadIdx.x; i < steps * (kRec / 16); i += blockDim.x) reinterpret_cast<uint4 *>(panel)[i] = src[i];
            __syncthreads();
            staged = resident;
        }
        if (ks == 0) {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) {
                const f32x4 b = *reinterpret_cast<const f32x4 *>(bias + ((int64_t)cb * KT + mt) * 16 + 4 * g);
#pragma unroll
                for (int p = 0; p < PT; ++p) acc[p][mt] = b;
            }
        }
        const bool last_step = ks + 1 == ksteps;
        load_next(ahead);

        // this step's operand: the rows' terms (columns past d become zeros: they may hold anything in memory)
        u32x4 xt[TX][PT];
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            float v[8];
            if constexpr (kF32) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(x[p][e >> 2][e & 3]);
            } else if constexpr (kBf16) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[2 * e] = __uint_as_float(x[p][0][e] << 16);
                    v[2 * e + 1] = __uint_as_float(x[p][0][e] & 0xffff0000u);
                }
            } else {
                typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
                const f16x8_t hv = __builtin_bit_cast(f16x8_t, x[p][0]);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = (float)hv[e];
            }
            if (ragged && last_step) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int col = ks * kStep + (kF32 ? 16 * (e >> 2) + 4 * g + (e & 3) : 8 * g + e);
                    v[e] = col < d ? v[e] : 0.f;
                }
            }
            if (XN && cb == 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) xn[p] = fmaf(v[e], v[e], xn[p]);
            }
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                if constexpr (kBf16) {
                    xt[0][p][pr] = (__float_as_uint(v[2 * pr + 1]) & 0xffff0000u) | (__float_as_uint(v[2 * pr]) >> 16);
                } else {
                    const Split3 t = split3_pair(v[2 * pr], v[2 * pr + 1]);
                    xt[0][p][pr] = t.h;
                    if constexpr (TX > 1) xt[1][p][pr] = t.m;
                    if constexpr (TX > 2) xt[2][p][pr] = t.l;
                }
            }
        }
        // products, small centroid terms first: cl.xh; cm.xm, cm.xh; ch.xl, ch.xm, ch.xh
        const unsigned char *rec = panel + (ks % panel_steps) * kRec + lane * 16;
#pragma unroll
        for (int ct = CT - 1; ct >= 0; --ct)
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) {
                const u32x4 a = *reinterpret_cast<const u32x4 *>(rec + (ct * KT + mt) * 1024);
#pragma unroll
                for (int tx = TX - 1; tx >= 0; --tx)
                    if (tx + ct < (kBf16 ? 1 : 3)) {
#pragma unroll
                        for (int p = 0; p < PT; ++p) acc[p][mt] = mfma_bf16_k32(a, xt[tx][p], acc[p][mt]);
                    }
            }
        ++ks;
        if (last_step) {   // this block's scores are complete: fold them into the best so far, ascending index
#pragma unroll
            for (int p = 0; p < PT; ++p)
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float s = acc[p][mt][v];
                        const int idx = (cb * KT + mt) * 16 + v;   // + 4 g, added at the end
                        if (s > best[p]) { best[p] = s; bidx[p] = idx; }
                    }
            ks = 0;
            ++cb;
        }
    };

    // Winners of a finished tile: the four lanes g of a point merge theirs (larger score, then lower index), lane g
    // keeps point tile g.
    auto finish_tile = [&](int64_t tile) {
        float my_best = 0.f, my_xn = 0.f;
        int32_t my_idx = 0;
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            float b = best[p], x2 = xn[p];
            int32_t i = bidx[p] + 4 * g;
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) {
                const float ob = __shfl_xor(b, off, 64);
                const int32_t oi = __shfl_xor(i, off, 64);
                if (ob > b || (ob == b && oi < i)) { b = ob; i = oi; }
                if (XN) x2 += __shfl_xor(x2, off, 64);
            }
            if (g == p) my_best = b, my_idx = i, my_xn = x2;
        }
        const int64_t i = tile * tile_rows + (wave * PT + g) * 16 + c;
        if (__builtin_expect(__any(g < PT && i < n && my_best == kNoScore), 0))
            if (g < PT && i < n && my_best == kNoScore) plain_scores(X + i * ld, d, C, k, my_best, my_idx, [&](int32_t j) { return bias[j]; });
        if (g < PT && i < n) {
            labels[i] = my_idx;
            if (XN) {
                const float d2 = fmaxf(my_xn - 2.f * my_best, 0.f);
                if (min_d2) min_d2[i] = d2;
                obj += (double)d2;
            }
        }
    };
    auto begin_tile = [&]() {
#pragma unroll
        for (int p = 0; p < PT; ++p) best[p] = kNoScore, bidx[p] = 0, xn[p] = 0.f;
        cb = 0;
    };
    // One K-step is worked on while the next two are in flight (fp32 rows and four centroid tiles: the next one, there
    // are no registers for more).
    constexpr bool kTwoAhead = !(kF32 && KT == 4 && PT == 4);
    u32x4 xa[PT][NP], xb[PT][NP], xc[PT][NP];
    int64_t tile = blockIdx.x;
    bool more = tile < tiles;   // uniform over the workgroup
    if (more) {
        point_at(tile);
        load_next(xa);
        if (kTwoAhead) load_next(xb);
        begin_tile();
    }
    auto advance = [&]() {
        if (cb != blocks_of_centroids) return;
        finish_tile(tile);
        tile += gridDim.x;
        more = tile < tiles;
        begin_tile();
    };
    while (more) {
        step(xa, kTwoAhead ? xc : xb);
        advance();
        if (!more) break;
        step(xb, xa);
        advance();
        if (kTwoAhead) {
            if (!more) break;
            step(xc, xb);
            advance();
        }
    }
    if (XN && obj_part) {
        for (int off = 32; off > 0; off >>= 1) obj += __shfl_down(obj, off, 64);
        if (lane == 0) red[wave] = obj;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w = 0; w < waves; ++w) t += red[w];
            obj_part[blockIdx.x] = t;
        }
    }
}

// Objective from the workgroups' partials, in a fixed order.
__global__ __launch_bounds__(64) void wide_objective_kernel(const double *__restrict__ part, int count,
                                                            double *__restrict__ out) {
    double o = 0.0;
    for (int q = threadIdx.x; q < count; q += 64) o += part[q];
    for (int off = 32; off > 0; off >>= 1) o += __shfl_down(o, off, 64);
    if (threadIdx.x == 0) *out = o;
}

// ---- 3. sums for k <= 64 ------------------------------------------------------------------------------
// A wave owns a slab of 16 NC columns and every parts-th 32-row group ("part"); it leaves the sums of
// its rows in psum[part][k][dpad] (dpad = slabs * 16 NC) and, on slab 0, their counts in pcnt[part][k].
template <typename XT> constexpr int slab_cols() { return 16 * (16 / (int)sizeof(XT)); }
int slab_cols_of(int dtype) { return dtype == EP_F32 ? slab_cols<float>() : slab_cols<bf16_t>(); }
int64_t slabs_of(const ep_problem &p) { return ceil_div(p.d, slab_cols_of(p.dtype)); }

typedef int i32x4u __attribute__((ext_vector_type(4), aligned(4)));

template <typename XT, int KT>
__global__ __launch_bounds__(256, KT == 4 && sizeof(XT) == 2 ? 1 : 2) void wide_sums_kernel(int64_t n, int32_t d, int32_t k, int64_t ld, int32_t slabs,
                                                           int32_t parts, int64_t groups, const XT *__restrict__ X,
                                                           const int32_t *__restrict__ labels, float *__restrict__ psum,
                                                           int32_t *__restrict__ pcnt) {
    constexpr bool kF32 = std::is_same<XT, float>::value, kBf16 = std::is_same<XT, bf16_t>::value;
    constexpr int NC = 16 / (int)sizeof(XT);   // columns per lane = column tiles of a slab
    const int64_t unit = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (unit >= (int64_t)slabs * parts) return;
    const int slab = (int)(unit % slabs);
    const int64_t part = unit / slabs;
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    // the groups part, part + parts, ..., the last one first: the assignment has just read the end of X, and what the
    // memory-side cache still holds of it is read again before it is lost
    int64_t grp = part + (groups - 1 - part) / parts * parts;   // (part < parts <= groups)
    const int col = slab * 16 * NC + NC * c;
    const XT *Xc = X + (col < d ? col : 0);   // a lane without columns reads column 0; its sums are never used

    f32x4 acc[KT][NC];
    int32_t cnt[KT];
#pragma unroll
    for (int mt = 0; mt < KT; ++mt) {
        cnt[mt] = 0;
#pragma unroll
        for (int t = 0; t < NC; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // rows 8 g + j of a 32-row group; rows past the end are read as the last row, with label -1
    auto load_rows = [&](int64_t grp, u32x4(&x)[8], i32x4(&lab)[2]) {
        const int64_t r0 = grp * 32 + 8 * g;
        if (grp * 32 + 32 <= n) {   // uniform
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = *reinterpret_cast<const u32x4 *>(Xc + (r0 + j) * ld);
            lab[0] = *reinterpret_cast<const i32x4u *>(labels + r0);
            lab[1] = *reinterpret_cast<const i32x4u *>(labels + r0 + 4);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t r = r0 + j < n ? r0 + j : n - 1;
                x[j] = *reinterpret_cast<const u32x4 *>(Xc + r * ld);
                lab[j >> 2][j & 3] = r0 + j < n ? labels[r] : -1;
            }
        }
    };
    auto add = [&](const u32x4(&x)[8], const i32x4(&lab)[2]) {
        u32x4 hot[KT];   // one-hot operand: points 8 g .. + 7 against centroid 16 mt + c
        constexpr unsigned kOne = (kF32 || kBf16) ? 0x3F80u : 0x3C00u;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                const unsigned lo = lab[pr >> 1][2 * (pr & 1)] == 16 * mt + c ? kOne : 0u;
                const unsigned hi = lab[pr >> 1][2 * (pr & 1) + 1] == 16 * mt + c ? kOne << 16 : 0u;
                hot[mt][pr] = lo | hi;
            }
        if (slab == 0) {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) cnt[mt] += __popc(hot[mt][pr] & 0x10001u * (kOne & (0u - kOne)));
        }
#pragma unroll
        for (int t = 0; t < NC; ++t) {
            if constexpr (kF32) {
                u32x4 xh, xm, xl;
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) {
                    const Split3 s = split3_pair(__uint_as_float(x[2 * pr][t]), __uint_as_float(x[2 * pr + 1][t]));
                    xh[pr] = s.h, xm[pr] = s.m, xl[pr] = s.l;
                }
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) acc[mt][t] = mfma_bf16_k32(hot[mt], xl, acc[mt][t]);
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) acc[mt][t] = mfma_bf16_k32(hot[mt], xm, acc[mt][t]);
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) acc[mt][t] = mfma_bf16_k32(hot[mt], xh, acc[mt][t]);
            } else {
                u32x4 b;
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) {   // element t of rows 2 pr and 2 pr + 1
                    const unsigned r0 = x[2 * pr][t >> 1], r1 = x[2 * pr + 1][t >> 1];
                    b[pr] = t & 1 ? (r0 >> 16) | (r1 & 0xffff0000u) : (r0 & 0xffffu) | (r1 << 16);
                }
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) {
                    if constexpr (kBf16) {
                        acc[mt][t] = mfma_bf16_k32(hot[mt], b, acc[mt][t]);
                    } else {
                        typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
                        acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, hot[mt]),
                                                                            __builtin_bit_cast(f16x8_t, b), acc[mt][t], 0, 0, 0);
                    }
                }
            }
        }
    };
    u32x4 xa[8], xb[8];
    i32x4 la[2], lb[2];
    load_rows(grp, xa, la);
    while (grp >= 0) {
        load_rows(grp >= parts ? grp - parts : grp, xb, lb);
        __builtin_amdgcn_sched_barrier(0);
        add(xa, la);
        grp -= parts;
        if (grp < 0) break;
        load_rows(grp >= parts ? grp - parts : grp, xa, la);
        __builtin_amdgcn_sched_barrier(0);
        add(xb, lb);
        grp -= parts;
    }
    // An infinity or a NaN times the zeros of the one-hot operand is a NaN in every centroid's sum: then this part's
    // rows are added again one by one, each to its own centroid only.  (Columns past d may hold anything.)
    bool odd = false;
#pragma unroll
    for (int t = 0; t < NC; ++t)
        if (col + t < d) {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v) odd |= !(fabsf(acc[mt][t][v]) < __builtin_inff());
        }
    if (__builtin_expect(__any(odd), 0)) {
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int t = 0; t < NC; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int64_t q = 0; part * 32 + (q >> 5) * 32 * parts + (q & 31) < n; ++q) {
            const int64_t r = part * 32 + (q >> 5) * 32 * parts + (q & 31);
            const int32_t l = labels[r];
            const u32x4 x = *reinterpret_cast<const u32x4 *>(Xc + r * ld);
#pragma unroll
            for (int t = 0; t < NC; ++t) {
                float xv;
                if constexpr (kF32) xv = __uint_as_float(x[t]);
                else if constexpr (kBf16) xv = bf16_to_f32((bf16_t)(x[t >> 1] >> (16 * (t & 1))));
                else xv = (float)__builtin_bit_cast(_Float16, (unsigned short)(x[t >> 1] >> (16 * (t & 1))));
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (l == 16 * mt + 4 * g + v) acc[mt][t][v] += xv;
            }
        }
    }
    const int64_t dpad = (int64_t)slabs * 16 * NC;
#pragma unroll
    for (int mt = 0; mt < KT; ++mt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int cent = 16 * mt + 4 * g + v;
            if (cent < k) {
                float *dst = psum + (part * k + cent) * dpad + col;
#pragma unroll
                for (int q = 0; q < NC / 4; ++q)
                    *reinterpret_cast<f32x4 *>(dst + 4 * q) =
                        f32x4{acc[mt][4 * q][v], acc[mt][4 * q + 1][v], acc[mt][4 * q + 2][v], acc[mt][4 * q + 3][v]};
            }
        }
        if (slab == 0) {
            int32_t v = cnt[mt];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (g == 0 && 16 * mt + c < k) pcnt[part * k + 16 * mt + c] = v;
        }
    }
}

// ---- 4. second pass ------------------------------------------------------------------------------------
// Workgroup (j, slice) forms 32 columns of centroid j: thread (seg, m4) adds columns 4 m4 .. + 3 of the partials
// seg, seg + 32, ... in fp64 in ascending order, eight loads in flight; then the 32 segment sums in order.
constexpr int kFinThreads = 256, kFinCols = 32, kFinSegs = kFinThreads / (kFinCols / 4);
__global__ __launch_bounds__(kFinThreads) void wide_finalize_kernel(int32_t dpad, int32_t d, int32_t k, int parts,
                                                                    const float *__restrict__ psum,
                                                                    const int32_t *__restrict__ pcnt,
                                                                    const float *__restrict__ C_prev,
                                                                    float *__restrict__ C_out, int64_t *__restrict__ counts,
                                                                    UpdateAcc acc) {
    __shared__ double seg_sum[kFinSegs * kFinCols];
    __shared__ unsigned long long total_cnt;
    const int slices = dpad / kFinCols;
    const int j = blockIdx.x / slices, col0 = kFinCols * (blockIdx.x % slices), t = threadIdx.x;
    const int m4 = t % (kFinCols / 4), seg = t / (kFinCols / 4);
    int64_t c = 0;
    for (int b = t; b < parts; b += kFinThreads) c += pcnt[(int64_t)b * k + j];
    const float4 *col = reinterpret_cast<const float4 *>(psum + (int64_t)j * dpad + col0) + m4;
    const int64_t stride4 = (int64_t)k * dpad / 4;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    for (int b0 = 0; b0 < parts; b0 += 8 * kFinSegs) {
        float4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int b = b0 + q * kFinSegs + seg;
            v[q] = b < parts ? col[(int64_t)b * stride4] : float4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            s0 += (double)v[q].x;
            s1 += (double)v[q].y;
            s2 += (double)v[q].z;
            s3 += (double)v[q].w;
        }
    }
    if (t == 0) total_cnt = 0;
    __syncthreads();
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
    if ((t & 63) == 0 && c) atomicAdd(&total_cnt, (unsigned long long)c);   // integers: order-free
    seg_sum[seg * kFinCols + 4 * m4 + 0] = s0;
    seg_sum[seg * kFinCols + 4 * m4 + 1] = s1;
    seg_sum[seg * kFinCols + 4 * m4 + 2] = s2;
    seg_sum[seg * kFinCols + 4 * m4 + 3] = s3;
    __syncthreads();
    if (t < kFinCols && col0 + t < d) {
        double tot = seg_sum[t];
        for (int q = 1; q < kFinSegs; ++q) tot += seg_sum[q * kFinCols + t];
        finish_centroid_element(acc, (int64_t)j * d + col0 + t, j, t == 0 && col0 == 0, tot, (int64_t)total_cnt, C_prev, C_out,
                                counts);
    }
}

template <typename F>
int by_dtype(const ep_problem &p, F &&f) {
    if (p.dtype == EP_F32) return f(static_cast<const float *>(nullptr));
    if (p.dtype == EP_F16) return f(static_cast<const f16_t *>(nullptr));
    return f(static_cast<const bf16_t *>(nullptr));
}

template <int V> using Int = std::integral_constant<int, V>;
template <typename F>
int by_cent_tiles(int kt, F &&f) {
    switch (kt) {
        case 1: return f(Int<1>());
        case 2: return f(Int<2>());
        case 3: return f(Int<3>());
        default: return f(Int<4>());
    }
}

// Row parts of the sums: as many waves as are resident at once (8 per compute unit; two more than that took 46 instead
// of 41 us at 200,003 x 516 bf16), at least two 32-row groups each, and no more partials than the workspace holds.
int wide_parts(const ep_problem &p) {
    const int64_t groups = ceil_div(p.n, 32), slabs = slabs_of(p);
    const int64_t dpad = slabs * slab_cols_of(p.dtype);
    int64_t parts = std::min<int64_t>(256 * 8 / slabs, ceil_div(groups, 2));
    parts = std::min<int64_t>(parts, kWidePartialElems / (p.k * dpad));
    return (int)std::max<int64_t>(1, parts);
}

}  // namespace

size_t wide_record_bytes(const ep_problem &p) {
    return (size_t)cent_blocks(p.k) * (size_t)k_steps(p.d) * (size_t)step_bytes(p);
}
size_t wide_bias_elems(const ep_problem &p) { return (size_t)cent_blocks(p.k) * 16 * (size_t)cent_tiles(p.k); }
size_t wide_psum_elems(const ep_problem &p) {
    return (size_t)wide_parts(p) * (size_t)p.k * (size_t)(slabs_of(p) * slab_cols_of(p.dtype));
}
size_t wide_pcnt_elems(const ep_problem &p) { return (size_t)wide_parts(p) * (size_t)p.k; }

int launch_wide_assign(const ep_problem &p, const void *X, const float *C, const KmeansWs &w, int32_t *labels,
                       float *min_d2, double *objective, hipStream_t s) {
    const int kt = cent_tiles(p.k), ksteps = (int)k_steps(p.d), blocks = (int)cent_blocks(p.k);
    const int64_t padded_k = (int64_t)blocks * 16 * kt;
    wide_prep_kernel<<<(unsigned)ceil_div(padded_k, 4), 256, 0, s>>>(p.d, p.k, kt, ksteps, p.dtype, C, w.wide_records,
                                                                     w.wide_bias, padded_k);
    EP_LAUNCH_CHECK();
    // 64 points per wave amortise the operand reads of a K-step over four matrix instructions each; with fewer rows
    // than fill the chip that way, 16 points per wave and smaller workgroups spread them further.
    const bool big = p.n >= 64 * 2048;
    const int threads = p.n >= 16 * 2048 ? kAssignThreads : 256;
    const int64_t tile_rows = (int64_t)(threads / 64) * (big ? 64 : 16);
    const int grid = (int)std::min<int64_t>(ceil_div(p.n, tile_rows), big ? 256 : 1024);
    const int panel_steps = std::min(ksteps, kPanelBytes / step_bytes(p));
    const int lds = panel_steps * step_bytes(p);
    const bool xn = min_d2 || objective;
    int rc = by_dtype(p, [&](auto *tag) {
        using XT = std::remove_cv_t<std::remove_pointer_t<decltype(tag)>>;
        return by_cent_tiles(kt, [&](auto kt_) {
            constexpr int KT = decltype(kt_)::value;
            auto go = [&](auto kern) {
                static std::atomic<uint64_t> attr_set{0};   // the LDS limit is raised once per variant and device
                int dev = 0;
                EP_HIP_TRY(hipGetDevice(&dev));
                const uint64_t bit = 1ull << (dev & 63);
                if (!(attr_set.load(std::memory_order_acquire) & bit)) {
                    EP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern.value),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, kPanelBytes));
                    attr_set.fetch_or(bit, std::memory_order_release);
                }
                ProfScope prof(EP_PROF_LLOYD_MAIN, s);
                kern.value<<<grid, threads, lds, s>>>(p.n, p.d, p.ld, ksteps, panel_steps, blocks, static_cast<const XT *>(X),
                                                      w.wide_records, w.wide_bias, C, p.k, labels, min_d2,
                                                      objective ? w.obj_part : nullptr);
                EP_LAUNCH_CHECK();
                return (int)EP_OK;
            };
#define EP_WIDE(PT_, XN_) go(std::integral_constant<decltype(&wide_assign_kernel<XT, KT, PT_, XN_>), &wide_assign_kernel<XT, KT, PT_, XN_>>())
            if (big) return xn ? EP_WIDE(4, true) : EP_WIDE(4, false);
            return xn ? EP_WIDE(1, true) : EP_WIDE(1, false);
#undef EP_WIDE
        });
    });
    if (rc != EP_OK) return rc;
    if (objective) {
        wide_objective_kernel<<<1, 64, 0, s>>>(w.obj_part, grid, objective);
        EP_LAUNCH_CHECK();
    }
    return EP_OK;
}

int launch_wide_update(const ep_problem &p, const void *X, const int32_t *labels, const float *C_prev, float *C_out,
                       int64_t *counts, const KmeansWs &w, const UpdateAcc &acc, hipStream_t s) {
    const int slabs = (int)slabs_of(p), parts = wide_parts(p);
    const int dpad = slabs * slab_cols_of(p.dtype);
    const int64_t groups = ceil_div(p.n, 32);
    int rc = by_dtype(p, [&](auto *tag) {
        using XT = std::remove_cv_t<std::remove_pointer_t<decltype(tag)>>;
        return by_cent_tiles(cent_tiles(p.k), [&](auto kt_) {
            ProfScope prof(EP_PROF_UPDATE_SUMS, s);
            wide_sums_kernel<XT, decltype(kt_)::value><<<(unsigned)ceil_div((int64_t)slabs * parts, 4), 256, 0, s>>>(
                p.n, p.d, p.k, p.ld, slabs, parts, groups, static_cast<const XT *>(X), labels, w.psum,
                w.pcnt);
            EP_LAUNCH_CHECK();
            return (int)EP_OK;
        });
    });
    if (rc != EP_OK) return rc;
    wide_finalize_kernel<<<(unsigned)((int64_t)p.k * (dpad / kFinCols)), kFinThreads, 0, s>>>(
        dpad, p.d, p.k, parts, w.psum, w.pcnt, C_prev, C_out, counts, acc);
    EP_LAUNCH_CHECK();
    return EP_OK;
}

}  // namespace ep
