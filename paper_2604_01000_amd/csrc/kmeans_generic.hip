// K-Means kernels that every path shares: the initial rows, the sample, the label check, the layout of the
// workspace, and the centroid update by sorted rows for k > 64.
//
// What they compute (EmbedPart paper, Alg. 3, step P <- KMeans(E, k)): a centroid moves to the mean of the
// embeddings assigned to it; an empty cluster keeps its centroid.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace ep {

namespace {

constexpr int kBlock = 256;

// ---- init: C[j,:] = X[idx[j],:] ------------------------------------------------------------
template <typename XT>
__global__ void gather_rows_kernel(int32_t d, int32_t k, int64_t ld, const XT *__restrict__ X,
                                   const int64_t *__restrict__ idx, float *__restrict__ C) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)k * d) return;
    const int32_t j = (int32_t)(t / d), m = (int32_t)(t % d);
    C[t] = load_elem(X + idx[j] * ld + m);
}

// ---- sample: S[i,:] = X[rows[i],:] in the element type of X, row stride ld_s >= d -----------------
// (the columns d .. ld_s - 1 of S are zeroed; no kernel reads them)
template <typename XT>
__global__ void sample_rows_kernel(int32_t d, int64_t m, int64_t ld, int64_t ld_s, const XT *__restrict__ X,
                                   const int64_t *__restrict__ rows, XT *__restrict__ S) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m * ld_s) return;
    const int64_t i = t / ld_s, c = t % ld_s;
    S[t] = c < d ? X[rows[i] * ld + c] : XT(0);
}

}  // namespace

__global__ void accumulate_counts_kernel(int32_t k, UpdateAcc acc) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < k) acc.cnt[j] = ((acc.flags & EP_UPDATE_ACCUMULATE) ? acc.cnt[j] : 0) + acc.chunk_cnt[j];
}

// result[0] += labels outside [0, k) among this workgroup's, result[1] = min(result[1], first such index).
__global__ __launch_bounds__(kBlock) void validate_labels_kernel(int64_t n, int32_t k,
                                                                  const int32_t *__restrict__ labels,
                                                                  unsigned long long *__restrict__ result) {
    __shared__ unsigned long long bad_lds[kBlock / 64], first_lds[kBlock / 64];
    unsigned long long bad = 0, first = (unsigned long long)n;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        if ((uint32_t)labels[i] >= (uint32_t)k) {   // a negative label is a large unsigned one
            ++bad;
            first = min(first, (unsigned long long)i);
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        bad += __shfl_down(bad, off, 64);
        first = min(first, (unsigned long long)__shfl_down(first, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        bad_lds[threadIdx.x >> 6] = bad;
        first_lds[threadIdx.x >> 6] = first;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) {
            bad += bad_lds[w];
            first = min(first, first_lds[w]);
        }
        if (bad) {   // integers: the order of the atomics does not matter
            atomicAdd(&result[0], bad);
            atomicMin(&result[1], first);
        }
    }
}

__global__ void validate_labels_init_kernel(int64_t n, unsigned long long *__restrict__ result) {
    result[0] = 0;
    result[1] = (unsigned long long)n;
}

namespace {

// ---- update, large k: rows sorted by label, one wave per cluster --------------------------------
// seg[j] = first sorted position whose key is >= j, for j = 0 .. k.  The key is the one the sort used:
// the label, or k for a label outside [0, k); such rows sit behind seg[k] and belong to no cluster.
// The keys are monotone along `order`, so every seg entry is written exactly once.
__global__ void segment_offsets_kernel(int64_t n, int32_t k, const int32_t *__restrict__ labels,
                                       const int32_t *__restrict__ order, int64_t *__restrict__ seg) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    const int32_t prev = i == 0 ? -1 : (int32_t)min((uint32_t)labels[order[i - 1]], (uint32_t)k);
    const int32_t cur = i == n ? k : (int32_t)min((uint32_t)labels[order[i]], (uint32_t)k);
    for (int32_t j = prev + 1; j <= cur; ++j) seg[j] = i;
}

// kLanes lanes share a row's slab of 8 kLanes columns (8 consecutive columns each, one or two 16-byte loads; 64
// columns for d <= 64, else 128), so a wave reads 64 / kLanes rows per step; wider rows take several slabs, the waves
// of one cluster's slabs side by side.  Sums are fp64 from the start.  The row groups are added in a fixed order
// at the end.
// load8: 8 elements at p; `second` is where the upper four of a fp32 piece lie (a piece that ends past the last
// column repeats its lower half: those sums are not used).
template <typename XT>
__device__ __forceinline__ void load8(const XT *p, int second, float (&v)[8]);
template <>
__device__ __forceinline__ void load8<float>(const float *p, int second, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + second);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <>
__device__ __forceinline__ void load8<f16_t>(const f16_t *p, int, float (&v)[8]) {
    const float4 a = load4(p), b = load4(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <>
__device__ __forceinline__ void load8<bf16_t>(const bf16_t *p, int, float (&v)[8]) {
    const uint4 r = *reinterpret_cast<const uint4 *>(p);
    v[0] = __uint_as_float(r.x << 16); v[1] = __uint_as_float(r.x & 0xFFFF0000u);
    v[2] = __uint_as_float(r.y << 16); v[3] = __uint_as_float(r.y & 0xFFFF0000u);
    v[4] = __uint_as_float(r.z << 16); v[5] = __uint_as_float(r.z & 0xFFFF0000u);
    v[6] = __uint_as_float(r.w << 16); v[7] = __uint_as_float(r.w & 0xFFFF0000u);
}

// Sum of the rows order[b .. e) over one slab in fp64 by one wave: lane = (sub, chunk) adds the rows b + sub,
// b + sub + 64 / kLanes, ... in 8 columns, then the sub-lanes are added in a fixed butterfly.  Every lane ends with
// the totals of its 8 columns.
template <typename XT, int kLanes>
__device__ __forceinline__ void sum_sorted_rows(const XT *__restrict__ X, int64_t ld, int32_t d, int slab,
                                                const int32_t *__restrict__ order, int64_t b, int64_t e, int lane,
                                                double (&acc)[8]) {
    constexpr int kRows = 64 / kLanes;
    const int chunk = lane % kLanes, sub = lane / kLanes;
    const int col = slab * 8 * kLanes + 8 * chunk;
    const XT *Xc = X + (col < d ? col : 0);          // a lane without columns reads column 0
    const int second = col + 4 < d ? 4 : 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.0;
    // Four rows in flight per lane, and the row indices of the next four loaded (unconditionally, from positions
    // clamped into the segment) before these rows are waited for: one exposed latency per four rows instead of an
    // index latency and a row latency per two.  Every lane still adds its rows in ascending order.
    constexpr int kAhead = 4;
    int64_t t = b + sub;
    if (e > b) {
        auto index_at = [&](int64_t pos) { return (int64_t)order[pos < e ? pos : e - 1]; };
        int64_t a[kAhead];
#pragma unroll
        for (int r = 0; r < kAhead; ++r) a[r] = index_at(t + r * kRows);
        for (; t + (kAhead - 1) * kRows < e; t += kAhead * kRows) {
            int64_t nx[kAhead];
#pragma unroll
            for (int r = 0; r < kAhead; ++r) nx[r] = index_at(t + (kAhead + r) * kRows);
            float v[kAhead][8];
#pragma unroll
            for (int r = 0; r < kAhead; ++r) load8(Xc + a[r] * ld, second, v[r]);
#pragma unroll
            for (int r = 0; r < kAhead; ++r)
#pragma unroll
                for (int q = 0; q < 8; ++q) acc[q] += (double)v[r][q];
#pragma unroll
            for (int r = 0; r < kAhead; ++r) a[r] = nx[r];
        }
#pragma unroll
        for (int r = 0; r < kAhead - 1; ++r) {   // what is left of this lane's rows, one by one (their indices are loaded)
            if (t + r * kRows < e) {
                float v0[8];
                load8(Xc + a[r] * ld, second, v0);
#pragma unroll
                for (int q = 0; q < 8; ++q) acc[q] += (double)v0[q];
            }
        }
    }
#pragma unroll
    for (int off = kLanes; off < 64; off <<= 1)
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] += __shfl_xor(acc[q], off, 64);
}

// Few, long segments (k well below the number of waves the chip runs): every segment is cut into
// `pieces` contiguous parts, one wave each and slab; the parts' sums go to the workspace in fp64 and
// segment_combine_kernel adds them in order.  The cut depends on (n, k, d) only: reproducible.
template <typename XT, int kLanes>
__global__ __launch_bounds__(kBlock) void segment_partial_kernel(int32_t d, int32_t k, int32_t slabs, int32_t pieces,
                                                                  int64_t ld, const XT *__restrict__ X,
                                                                  const int32_t *__restrict__ order,
                                                                  const int64_t *__restrict__ seg,
                                                                  double *__restrict__ part) {
    const int64_t w = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (w >= (int64_t)k * pieces * slabs) return;
    const int slab = (int)(w % slabs), lane = threadIdx.x & 63;
    const int64_t wp = w / slabs;
    const int j = (int)(wp / pieces), piece = (int)(wp % pieces);
    const int64_t b = seg[j], cnt = seg[j + 1] - b;
    double acc[8];
    sum_sorted_rows<XT, kLanes>(X, ld, d, slab, order, b + cnt * piece / pieces, b + cnt * (piece + 1) / pieces, lane, acc);
    if (lane < kLanes) {
#pragma unroll
        for (int q = 0; q < 8; ++q) part[w * 8 * kLanes + 8 * lane + q] = acc[q];
    }
}

__global__ __launch_bounds__(kBlock) void segment_combine_kernel(int32_t d, int32_t k, int32_t dseg, int32_t pieces,
                                                                  const int64_t *__restrict__ seg,
                                                                  const double *__restrict__ part,
                                                                  const float *__restrict__ C_prev,
                                                                  float *__restrict__ C_out,
                                                                  int64_t *__restrict__ counts, UpdateAcc acc) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= (int64_t)k * d) return;
    const int j = (int)(t / d), col = (int)(t % d);
    const int64_t cnt = seg[j + 1] - seg[j];
    double tot = 0.0;
    for (int piece = 0; piece < pieces; ++piece) tot += part[((int64_t)j * pieces + piece) * dseg + col];
    finish_centroid_element(acc, t, j, col == 0, tot, cnt, C_prev, C_out, counts);
}

template <typename XT, int kLanes>
__global__ __launch_bounds__(kBlock) void segment_mean_kernel(int32_t d, int32_t k, int32_t slabs, int64_t ld,
                                                               const XT *__restrict__ X,
                                                               const int32_t *__restrict__ order,
                                                               const int64_t *__restrict__ seg,
                                                               const float *__restrict__ C_prev,
                                                               float *__restrict__ C_out,
                                                               int64_t *__restrict__ counts, UpdateAcc upd) {
    const int64_t w = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (w >= (int64_t)k * slabs) return;
    const int j = (int)(w / slabs), slab = (int)(w % slabs), lane = threadIdx.x & 63;
    const int64_t b = seg[j], e = seg[j + 1];
    const int64_t cnt = e - b;
    const int chunk = lane % kLanes, sub = lane / kLanes;
    double acc[8];
    sum_sorted_rows<XT, kLanes>(X, ld, d, slab, order, b, e, lane, acc);
    if (sub == 0) {
        const int col = slab * 8 * kLanes + 8 * chunk;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (col + q < d)
                finish_centroid_element(upd, (int64_t)j * d + col + q, j, col + q == 0, acc[q], cnt, C_prev, C_out, counts);
    }
}

template <typename F>
int by_dtype(const ep_problem &p, F &&f) {
    if (p.dtype == EP_F32) return f(static_cast<const float *>(nullptr));
    if (p.dtype == EP_F16) return f(static_cast<const f16_t *>(nullptr));
    return f(static_cast<const bf16_t *>(nullptr));
}

}  // namespace

namespace {
// Slabs of the sorted update, and the parts a segment is cut into: enough waves to fill the chip, at least a few
// rows each, and (at widths other than 64 and 128, where the rest of the workspace fits the static array of
// kmeans_run_noalloc) no more than that array has room for.
struct SegPlan {
    int lanes, slabs, pieces;
    size_t part_elems() const { return (size_t)slabs * 8 * lanes; }   // per cluster and piece
};
SegPlan seg_plan(const ep_problem &p, size_t other_bytes) {
    SegPlan s;
    s.lanes = p.d <= 64 ? 8 : 16;
    s.slabs = (int)ceil_div(p.d, 8 * s.lanes);
    int64_t pieces = std::min<int64_t>(kSegWavesTarget / ((int64_t)p.k * s.slabs), p.n / ((int64_t)p.k * kSegRowsMin));
    if (p.d != 64 && p.d != 128 && other_bytes < (size_t)EP_NOALLOC_SCRATCH_BYTES)
        pieces = std::min<int64_t>(pieces, ((size_t)EP_NOALLOC_SCRATCH_BYTES - other_bytes) / ((size_t)p.k * s.part_elems() * 8));
    s.pieces = (int)std::max<int64_t>(1, pieces);
    return s;
}
}  // namespace

KmeansWs carve_kmeans_ws(const ep_problem &p, void *ws, bool records_over_sums) {
    Carver c(ws);
    KmeansWs w{};
    const size_t kd = (size_t)p.k * p.d;
    const bool small = small_path_supported(p), large = large_path_supported(p);
    const bool blocks = !small && blocks_path_supported(p);
    const bool wide = !small && !large && !blocks;
    const size_t rec_bytes = wide ? wide_record_bytes(p) : 0;
    w.obj_part = c.take<double>(kObjBlocksMax);
    // the running sums of a chunked update come first: their place must not depend on n, because the
    // chunks of one update may differ in size
    w.acc_sum = reinterpret_cast<double *>(c.take<unsigned char>(std::max(kd * 8, records_over_sums ? rec_bytes : 0)));
    w.acc_cnt = c.take<int64_t>(p.k);
    w.chunk_cnt = c.take<int64_t>(p.k);
    w.idx = c.take<int64_t>(p.k);
    if (large) {
        w.cnorm = c.take<float>(p.k);
        w.cq16 = c.take<bf16_t>(kd);
        w.records = c.take<unsigned char>(large_record_bytes(p));
        w.best_tile = c.take<int32_t>((size_t)p.n);
    }
    if (wide && !update_by_sorted_rows(p)) w.wide_bias = c.take<float>(wide_bias_elems(p));
    if (small) {
        w.psum = c.take<float>((size_t)kUpdBlocksMax * (size_t)p.k * (size_t)small_padded_d(p));
        w.pcnt = c.take<int32_t>((size_t)kUpdBlocksMax * p.k);
    } else if (!update_by_sorted_rows(p)) {
        // the assignment is through with its records when the update writes its partial sums: one place for both
        unsigned char *both = c.take<unsigned char>(std::max(wide_psum_elems(p) * 4, records_over_sums ? 0 : rec_bytes));
        w.psum = reinterpret_cast<float *>(both);
        w.wide_records = both;
        w.pcnt = c.take<int32_t>(wide_pcnt_elems(p));
    } else if (blocks) {
        // the winners lie over the row order, the records over what else only the update uses; with records_over_sums
        // they take the larger of that and the running sums, as many at a time as fit there
        const size_t n4 = align_up((size_t)p.n * 4, 256);
        unsigned char *both = c.take<unsigned char>(2 * n4);
        w.order = reinterpret_cast<int32_t *>(both);
        w.order_tmp = reinterpret_cast<int32_t *>(both + n4);
        w.winner = reinterpret_cast<unsigned long long *>(both);
        const size_t start = align_up(c.used, 256), record = block_record_bytes(p);
        const int64_t records = ceil_div(p.k, 32);
        w.seg = c.take<int64_t>((size_t)p.k + 1);
        w.sort_hist = c.take<int32_t>(sort_hist_elems());
        const SegPlan sp = seg_plan(p, align_up(c.used, 256) + 256);
        w.seg_pieces = sp.pieces;
        if (sp.pieces > 1) w.seg_part = c.take<double>((size_t)p.k * sp.pieces * sp.part_elems());
        if (!records_over_sums) c.used = std::max(c.used, start + (size_t)records * record);
        size_t room = c.used - start;   // at least the radix sort's megabyte: dozens of records
        w.block_records = reinterpret_cast<unsigned char *>(c.base ? c.base + start : nullptr);
        if (records_over_sums && kd * 8 > room) {
            room = kd * 8;
            w.block_records = reinterpret_cast<unsigned char *>(w.acc_sum);
        }
        w.block_slice = (int)std::min<int64_t>(records, (int64_t)(room / record));
        w.bytes = align_up(c.used, 256);
        return w;
    } else {
        const size_t n4 = align_up((size_t)p.n * 4, 256);
        unsigned char *both = c.take<unsigned char>(std::max(2 * n4, records_over_sums ? 0 : rec_bytes));
        w.order = reinterpret_cast<int32_t *>(both);   // (the same for the row order)
        w.order_tmp = reinterpret_cast<int32_t *>(both + n4);
        w.wide_records = both;
        w.seg = c.take<int64_t>((size_t)p.k + 1);
        w.sort_hist = c.take<int32_t>(sort_hist_elems());
        if (wide) w.wide_bias = reinterpret_cast<float *>(w.sort_hist);   // (the assignment's)
        // (the parts must not depend on where the records lie: count them as lying over the sums)
        const size_t moved = records_over_sums ? 0 : align_up(std::max(kd * 8, rec_bytes), 256) - align_up(kd * 8, 256);
        const size_t shared = records_over_sums ? 0 : align_up(std::max(2 * n4, rec_bytes), 256) - 2 * n4;
        const SegPlan sp = seg_plan(p, align_up(c.used, 256) + moved - shared + 256);
        w.seg_pieces = sp.pieces;
        if (sp.pieces > 1) w.seg_part = c.take<double>((size_t)p.k * sp.pieces * sp.part_elems());
    }
    if (records_over_sums) w.wide_records = reinterpret_cast<unsigned char *>(w.acc_sum);
    w.bytes = align_up(c.used, 256);
    return w;
}

int launch_gather_rows(const ep_problem &p, const void *X, const int64_t *idx_dev, float *C, hipStream_t s) {
    const int64_t total = (int64_t)p.k * p.d;
    return by_dtype(p, [&](auto *tag) {
        using XT = std::remove_cv_t<std::remove_pointer_t<decltype(tag)>>;
        gather_rows_kernel<XT><<<(unsigned)ceil_div(total, kBlock), kBlock, 0, s>>>(
            p.d, p.k, p.ld, static_cast<const XT *>(X), idx_dev, C);
        EP_LAUNCH_CHECK();
        return EP_OK;
    });
}

int launch_sample_rows(const ep_problem &p, const void *X, int64_t m, int64_t ld_s, const int64_t *rows_dev, void *S,
                       hipStream_t s) {
    const int64_t total = m * ld_s;
    return by_dtype(p, [&](auto *tag) {
        using XT = std::remove_cv_t<std::remove_pointer_t<decltype(tag)>>;
        sample_rows_kernel<XT><<<(unsigned)ceil_div(total, kBlock), kBlock, 0, s>>>(
            p.d, m, p.ld, ld_s, static_cast<const XT *>(X), rows_dev, static_cast<XT *>(S));
        EP_LAUNCH_CHECK();
        return EP_OK;
    });
}

int launch_accumulate_counts(int32_t k, const UpdateAcc &acc, hipStream_t s) {
    accumulate_counts_kernel<<<(unsigned)ceil_div(k, kBlock), kBlock, 0, s>>>(k, acc);
    EP_LAUNCH_CHECK();
    return EP_OK;
}

int launch_validate_labels(int64_t n, int32_t k, const int32_t *labels, int64_t *result, hipStream_t s) {
    auto out = reinterpret_cast<unsigned long long *>(result);
    validate_labels_init_kernel<<<1, 1, 0, s>>>(n, out);
    EP_LAUNCH_CHECK();
    const unsigned grid = (unsigned)std::min<int64_t>(ceil_div(n, kBlock * 4), 2048);
    validate_labels_kernel<<<grid, kBlock, 0, s>>>(n, k, labels, out);
    EP_LAUNCH_CHECK();
    return EP_OK;
}

int launch_update_sorted(const ep_problem &p, const void *X, const int32_t *labels, const float *C_prev,
                         float *C_out, int64_t *counts, const KmeansWs &w, const UpdateAcc &acc, hipStream_t s) {
    int rc = launch_sort_by_label(p.n, p.k, labels, nullptr, w.order, w.order_tmp, w.sort_hist, s);
    if (rc != EP_OK) return rc;
    segment_offsets_kernel<<<(unsigned)ceil_div(p.n + 1, kBlock), kBlock, 0, s>>>(p.n, p.k, labels, w.order, w.seg);
    EP_LAUNCH_CHECK();
    return by_dtype(p, [&](auto *tag) {
        using XT = std::remove_cv_t<std::remove_pointer_t<decltype(tag)>>;
        ProfScope prof(EP_PROF_UPDATE_SUMS, s);
        const XT *Xt = static_cast<const XT *>(X);
        const int lanes = p.d <= 64 ? 8 : 16, slabs = (int)ceil_div(p.d, 8 * lanes), pieces = w.seg_pieces;
        const unsigned grid = (unsigned)ceil_div((int64_t)p.k * slabs * pieces, kBlock / 64);
        if (pieces > 1) {
            if (lanes == 16)
                segment_partial_kernel<XT, 16><<<grid, kBlock, 0, s>>>(p.d, p.k, slabs, pieces, p.ld, Xt, w.order, w.seg, w.seg_part);
            else
                segment_partial_kernel<XT, 8><<<grid, kBlock, 0, s>>>(p.d, p.k, slabs, pieces, p.ld, Xt, w.order, w.seg, w.seg_part);
            EP_LAUNCH_CHECK();
            segment_combine_kernel<<<(unsigned)ceil_div((int64_t)p.k * p.d, kBlock), kBlock, 0, s>>>(
                p.d, p.k, slabs * 8 * lanes, pieces, w.seg, w.seg_part, C_prev, C_out, counts, acc);
            EP_LAUNCH_CHECK();
            return EP_OK;
        }
        if (lanes == 16)
            segment_mean_kernel<XT, 16><<<grid, kBlock, 0, s>>>(p.d, p.k, slabs, p.ld, Xt, w.order, w.seg, C_prev, C_out, counts, acc);
        else
            segment_mean_kernel<XT, 8><<<grid, kBlock, 0, s>>>(p.d, p.k, slabs, p.ld, Xt, w.order, w.seg, C_prev, C_out, counts, acc);
        EP_LAUNCH_CHECK();
        return EP_OK;
    });
}

}  // namespace ep
