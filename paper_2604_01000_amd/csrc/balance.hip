// Balancing of a partition: one of the three while-loops of the EmbedPart paper's Alg. 3 with the
// migration policy of Alg. 4 (movers leave overloaded partitions smallest degree first and land in
// underloaded ones in proportion to free capacity), for one vertex class, entirely on the device
// and in integers.
//
// A migration round:
//   1. per partition, the number of class members of every degree 0 .. B-2 and of degree >= B-1 (LDS
//      histogram, integer atomics); the loads L_i are the row sums;
//   2. plan: capacity C = max(floor(beta |S| / k), ceil(|S| / k)), m_i = L_i - C on the overloaded
//      partitions, the running sum of the free capacities C - L_i of the underloaded ones, their total F;
//      and, from the degree counts, the degree t_i at which the m_i-th smallest member of partition i sits
//      and how many members of exactly that degree still have to go (need_i).  If t_i falls into the last
//      bin, the range that holds it is counted again with narrower bins until a bin is one degree wide (at
//      most a few passes up to degree 2^24 - 1, the value degrees are clamped to);
//   3. selection instead of a sort: the movers of partition i are its members of degree < t_i and,
//      among those of degree t_i, the need_i with the smallest ids: the count of such members before a
//      vertex range, plus the ordered count inside it;
//   4. the destination of a mover v is the partition whose interval of the running sum holds
//      (mix(seed, round, v) mod F).
// The draw is a function of (seed, round, v) only, so the result does not depend on the order in
// which threads get to the vertices.  All rounds of a call run in one launch, which ends at the first
// round that leaves nothing overloaded: the host never reads anything back.
#include <algorithm>
#include <atomic>

#include "kernels.h"

namespace ep {

namespace {

constexpr int kPartMax = 255;
constexpr int kBalBlock = 1024;
constexpr int kBalWaves = kBalBlock / 64;
constexpr int kPer = 8;                // vertices per thread and turn: their loads are in flight together
constexpr int kTurn = kPer * kBalBlock;
constexpr int kCounters = 8192;        // LDS counters of the degree histogram (32 KB)
constexpr int kBinsMax = 256;
constexpr int kDegreeLimit = 1 << 24;  // degrees are clamped to kDegreeLimit - 1
constexpr int64_t kSingleN = 32768;    // up to here one workgroup does the call
constexpr int64_t kBalRowsMin = 2048;  // beyond: vertices per workgroup, at least
constexpr int kGroups = 8;             // barrier groups: workgroups with the same index mod 8 share an XCD

// What the workgroups of a call share.  Within the launch it is only touched with device-scope atomics (a plain
// access would be served by the L2 of the accessing die).
struct BalShared {
    unsigned int arrive[kGroups * 32];      // barrier: arrivals per group, one 128-byte line each,
    unsigned int root[32];                  // and of whole groups
    unsigned long long moved;
    unsigned int arrived[3][256];           // movers that landed in a partition, three rounds in rotation
    unsigned int hist[3][kCounters];        // degree histograms, three counting passes in rotation
};

__device__ __forceinline__ uint64_t draw64(uint64_t seed, uint32_t round, int64_t v) {
    uint64_t z = seed + (((uint64_t)round << 32) + (uint64_t)v + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// x mod F without a 64-bit division per draw: with magic = floor((2^64 - 1) / F), q = high half of x * magic
// is the quotient or up to two less, so at most two subtractions finish the remainder (exact for every x).
__device__ __forceinline__ uint64_t magic_of(uint64_t F) { return F ? ~0ull / F : 0; }
__device__ __forceinline__ uint64_t mod_by(uint64_t x, uint64_t F, uint64_t magic) {
    uint64_t r = x - __umul64hi(x, magic) * F;
    if (r >= F) r -= F;
    if (r >= F) r -= F;
    return r;
}


template <typename T>
__device__ __forceinline__ T dev_load(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ void dev_store(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T dev_add(T *p, T v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ __forceinline__ void wave_lds_fence_() {   // orders a wave's own LDS accesses
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Barrier over the workgroups of a cooperative launch (all resident, so every wait ends).  Every wave first waits
// for its own atomics; nothing is flushed, because the workgroups exchange data with device-scope atomics only.
// Two levels of counters: 256 arrivals on one line cost 3.8 us, 32 cost 0.95 us.
__device__ __forceinline__ void grid_barrier(BalShared *sh, unsigned int &generation) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    ++generation;
    if (gridDim.x > 1 && threadIdx.x == 0) {
        const unsigned int group = blockIdx.x % kGroups;
        const unsigned int members = (gridDim.x - group + kGroups - 1) / kGroups;
        const unsigned int groups = min(gridDim.x, (unsigned int)kGroups);
        if (dev_add(&sh->arrive[group * 32], 1u) + 1 == generation * members) dev_add(&sh->root[0], 1u);
        while ((int)(dev_load(&sh->root[0]) - generation * groups) < 0) __builtin_amdgcn_s_sleep(1);
    }
    __syncthreads();
}

__global__ __launch_bounds__(kBalBlock) void bal_reset_kernel(BalShared *sh) {
    const int t = threadIdx.x;
    if (t < kGroups * 32) sh->arrive[t] = 0;
    if (t == 0) {
        sh->root[0] = 0;
        sh->moved = 0;
    }
    if (t < 256) sh->arrived[0][t] = 0;
    for (int i = t; i < kCounters; i += kBalBlock) sh->hist[0][i] = 0;
}

// LDS of bal_rounds_kernel.
struct BalLds {
    unsigned int mine[kCounters];            // this workgroup's histogram of the counting pass in hand
    unsigned int all[kCounters + 256];       // the whole graph's, rows padded by one counter (bank spread)
    int32_t wcnt[kBalWaves][256];            // degree-t members per wave and partition
    long long load_of[256], m_of[256], cumf[256], need[256], below[256], running[256];
    int32_t lo[256], hi[256], width[256], tdeg[256], refining[256];
    unsigned int tie_mine[256];              // this workgroup's degree-t members
    unsigned int arrived[256];
    long long cap, F;
    int32_t over, refine_any;
    unsigned int moved;
};

// Every workgroup owns one range of vertices in every pass, so the labels it rewrites are read again by itself
// alone.  What bounds the call: for large graphs two passes over class, label and offsets (13 bytes per vertex) per
// round, for small ones the cooperative launch (about 17 us more than an ordinary one) and three to four barriers.
// Measured, three calls for three classes: 2.45 M vertices 136 us, 20 M 740 us.  As a chain of launches (count, plan,
// refinement, tie count, scan, move) with max_rounds rounds enqueued whatever happens it took about 180 launches per
// call and 1,706 and 2,546 us; one workgroup for the whole call, as used up to 2^18 vertices, 870 us at 170,000
// vertices and k = 100 (now 180).  Up to kSingleN vertices one workgroup is still the faster (30,000 vertices:
// 136 against 150 us; 50,000: 183 against 133).
template <typename RowT>
__global__ __launch_bounds__(kBalBlock) void bal_rounds_kernel(int64_t n, int64_t rows_per_block, int32_t k,
                                                               const RowT *__restrict__ rowptr,
                                                               const uint8_t *__restrict__ vclass, int32_t class_id,
                                                               double beta, uint64_t seed, int32_t max_rounds,
                                                               int32_t *labels, int64_t *__restrict__ stats, BalShared *sh,
                                                               unsigned int *tie) {
    extern __shared__ __attribute__((aligned(16))) unsigned char bal_lds[];
    BalLds &s = *reinterpret_cast<BalLds *>(bal_lds);
    const int t = threadIdx.x, wave = t >> 6;
    const unsigned lane = t & 63;
    const int bins = min(kBinsMax, kCounters / k), cells = k * bins;
    const int64_t begin = min(n, (int64_t)blockIdx.x * rows_per_block), end = min(n, begin + rows_per_block);
    unsigned int generation = 0;   // barriers passed
    int pass = 0;                  // counting passes started
    if (t == 0) s.moved = 0;

    // Partition and clamped degree of the kPer vertices base + 512 wave + 64 q + lane; -1 for a vertex that is not a
    // member of the class (or past the end).  All loads are issued before anything is looked at.
    auto fetch = [&](int64_t base, int32_t(&l)[kPer], int32_t(&deg)[kPer]) {
        int32_t cls[kPer], lab[kPer];
        RowT r0[kPer], r1[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t v = base + wave * (64 * kPer) + 64 * q + lane;
            const int64_t vs = v < end ? v : 0;
            cls[q] = vclass ? (int32_t)vclass[vs] : class_id;
            lab[q] = labels[vs];
            r0[q] = rowptr[vs];
            r1[q] = rowptr[vs + 1];
            if (v >= end) cls[q] = class_id + 1;
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const bool member = cls[q] == class_id && lab[q] >= 0 && lab[q] < k;
            l[q] = member ? lab[q] : -1;
            const int64_t d = (int64_t)(r1[q] - r0[q]);
            deg[q] = (int32_t)min(max(d, (int64_t)0), (int64_t)kDegreeLimit - 1);
        }
    };
    // One counting pass over the graph: bin_of(l, deg) is the bin or -1.  Leaves this workgroup's counts in s.mine and
    // everybody's in s.all (row stride bins + 1).
    auto count_pass = [&](auto &&bin_of) {
        unsigned int *hist = sh->hist[pass % 3], *next = sh->hist[(pass + 1) % 3];
        ++pass;
        for (int i = t; i < cells; i += kBalBlock) s.mine[i] = 0;
        __syncthreads();
        for (int64_t base = begin; base < end; base += kTurn) {
            int32_t l[kPer], deg[kPer];
            fetch(base, l, deg);
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int b = l[q] >= 0 ? bin_of(l[q], deg[q]) : -1;
                if (b >= 0) atomicAdd(&s.mine[l[q] * bins + b], 1u);
            }
        }
        __syncthreads();
        if (gridDim.x == 1) {
            for (int i = t; i < cells; i += kBalBlock) s.all[i + i / bins] = s.mine[i];
            __syncthreads();
            return;
        }
        for (int i = t; i < cells; i += kBalBlock)
            if (s.mine[i]) dev_add(&hist[i], s.mine[i]);
        // the next pass's counters: last read two passes ago, cleared before this pass's barrier
        for (int i = blockIdx.x * kBalBlock + t; i < cells; i += gridDim.x * kBalBlock) dev_store(&next[i], 0u);
        grid_barrier(sh, generation);
        for (int i = t; i < cells; i += kBalBlock) s.all[i + i / bins] = dev_load(&hist[i]);
        __syncthreads();
    };

    for (int32_t round = 0;; ++round) {
        // ---- loads of the class per partition and the exact degree bins 0 .. bins - 2 (+ "bins - 1 or more") ----
        count_pass([&](int32_t, int32_t deg) { return min(deg, bins - 1); });
        if (t < 256) {
            long long L = 0;
            if (t < k)
                for (int b = 0; b < bins; ++b) L += s.all[t * (bins + 1) + b];
            s.load_of[t] = L;
        }
        __syncthreads();
        if (t == 0) {
            long long total = 0;
            for (int j = 0; j < k; ++j) total += s.load_of[j];
            long long cap = (long long)floor(beta * (double)total / (double)k);
            const long long reach = (total + k - 1) / k;
            if (cap < reach) cap = reach;
            long long F = 0;
            int32_t over = 0;
            for (int j = 0; j < k; ++j) {
                const long long Lj = s.load_of[j];
                if (Lj < cap) F += cap - Lj;
                s.cumf[j] = F;
                if (Lj > cap) ++over;
            }
            s.cap = cap;
            s.F = F;
            s.over = over;
            s.refine_any = 0;
        }
        __syncthreads();
        if (s.over == 0 || round >= max_rounds) {   // uniform over the grid: balanced, or the closing evaluation
            if (blockIdx.x == 0 && t == 0) {
                stats[0] = round;
                stats[1] = gridDim.x == 1 ? (int64_t)s.moved : (int64_t)dev_load(&sh->moved);
                stats[2] = s.over;
            }
            return;
        }

        // ---- threshold degree t_i of every overloaded partition: where its m_i-th smallest member sits ----
        if (t < 256) {
            const long long m = t < k && s.load_of[t] > s.cap ? s.load_of[t] - s.cap : 0;
            s.m_of[t] = m;
            s.tdeg[t] = -1;
            s.need[t] = 0;
            s.refining[t] = 0;
            s.tie_mine[t] = 0;
            s.arrived[t] = 0;
            if (m > 0) {
                long long seen = 0;
                int b = 0;
                for (; b < bins - 1; ++b) {
                    const long long c = s.all[t * (bins + 1) + b];
                    if (seen + c >= m) break;
                    seen += c;
                }
                if (b < bins - 1) {
                    s.tdeg[t] = b;
                    s.need[t] = m - seen;
                    s.tie_mine[t] = s.mine[t * bins + b];
                } else {   // beyond the exact bins: narrow the range [bins - 1, 2^24) down
                    s.below[t] = seen;
                    s.lo[t] = bins - 1;
                    s.hi[t] = kDegreeLimit;
                    s.width[t] = (kDegreeLimit - (bins - 1) + bins - 1) / bins;
                    s.refining[t] = 1;
                    s.refine_any = 1;
                }
            }
        }
        __syncthreads();
        while (s.refine_any) {   // uniform over the grid
            count_pass([&](int32_t l, int32_t deg) {
                return s.refining[l] && deg >= s.lo[l] && deg < s.hi[l] ? (deg - s.lo[l]) / s.width[l] : -1;
            });
            if (t == 0) s.refine_any = 0;
            __syncthreads();
            if (t < 256 && s.refining[t]) {
                long long seen = s.below[t];
                int b = 0;
                for (; b < bins - 1; ++b) {   // the m-th smallest lies in the range, so the last bin ends the search
                    const long long c = s.all[t * (bins + 1) + b];
                    if (seen + c >= s.m_of[t]) break;
                    seen += c;
                }
                s.below[t] = seen;
                s.lo[t] += b * s.width[t];
                s.hi[t] = min(s.hi[t], s.lo[t] + s.width[t]);
                if (s.width[t] == 1) {
                    s.tdeg[t] = s.lo[t];
                    s.need[t] = s.m_of[t] - seen;
                    s.tie_mine[t] = s.mine[t * bins + b];
                    s.refining[t] = 0;
                } else {
                    s.width[t] = (s.hi[t] - s.lo[t] + bins - 1) / bins;
                    s.refine_any = 1;
                }
            }
            __syncthreads();
        }

        // ---- members at the threshold in the ranges before this one ----
        if (t < 256) s.running[t] = 0;
        if (gridDim.x > 1) {
            if (t < k) dev_store(&tie[(int64_t)blockIdx.x * k + t], s.tie_mine[t]);
            if (blockIdx.x == 0 && t < 256) dev_store(&sh->arrived[(round + 1) % 3][t], 0u);   // last read two rounds ago
            grid_barrier(sh, generation);
            for (int64_t i = t; i < (int64_t)blockIdx.x * k; i += kBalBlock) {
                const int l = (int)(i % k);
                if (s.m_of[l] > 0) atomicAdd(reinterpret_cast<unsigned long long *>(&s.running[l]), (unsigned long long)dev_load(&tie[i]));
            }
        }

        // ---- the movers, in id order: below the threshold, or at it among the first need_i ----
        const uint64_t F = (uint64_t)s.F, magic = magic_of(F);
        unsigned int moved_here = 0;
        for (int64_t base = begin; base < end; base += kTurn) {   // uniform over the workgroup
            int32_t l[kPer], deg[kPer];
            fetch(base, l, deg);
            for (int i = t; i < kBalWaves * 256; i += kBalBlock) (&s.wcnt[0][0])[i] = 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kPer; ++q)
                if (l[q] >= 0 && deg[q] == s.tdeg[l[q]]) atomicAdd(&s.wcnt[wave][l[q]], 1);
            __syncthreads();
            if (t < 256) {   // exclusive scan over the waves, on top of what came before this turn
                int32_t run = 0;
                for (int w = 0; w < kBalWaves; ++w) {
                    const int32_t c = s.wcnt[w][t];
                    s.wcnt[w][t] = run;
                    run += c;
                }
                s.load_of[t] = run;   // (the loads are not needed any more this round)
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int64_t v = base + wave * (64 * kPer) + 64 * q + lane;
                const bool cand = l[q] >= 0 && s.m_of[l[q]] > 0;
                const bool at_threshold = cand && deg[q] == s.tdeg[l[q]];
                bool move = cand && deg[q] < s.tdeg[l[q]];
                if (__ballot(at_threshold)) {   // uniform in the wave
                    const int key = at_threshold ? l[q] : 0;
                    uint64_t peers = __ballot(at_threshold);   // lanes at the threshold of the same partition
                    for (int bit = 0; bit < 8; ++bit) {
                        const uint64_t mb = __ballot((key >> bit) & 1);
                        peers &= ((key >> bit) & 1) ? mb : ~mb;
                    }
                    const uint64_t lanes_before = lane == 0 ? 0ull : (~0ull >> (64 - lane));
                    const int rank_in_wave = __popcll(peers & lanes_before);
                    if (at_threshold) move = s.running[key] + s.wcnt[wave][key] + rank_in_wave < s.need[key];
                    wave_lds_fence_();
                    if (at_threshold && rank_in_wave == 0) s.wcnt[wave][key] += __popcll(peers);
                    wave_lds_fence_();
                }
                if (move) {
                    const uint64_t r = mod_by(draw64(seed, (uint32_t)round, v), F, magic);
                    int a = 0, b = k - 1;               // first partition whose running sum exceeds r
                    while (a < b) {
                        const int mid = (a + b) >> 1;
                        if ((uint64_t)s.cumf[mid] > r) b = mid; else a = mid + 1;
                    }
                    labels[v] = a;
                    atomicAdd(&s.arrived[a], 1u);   // integer: order does not matter
                }
                moved_here += (unsigned int)__popcll(__ballot(move));
            }
            __syncthreads();
            if (t < 256) s.running[t] += s.load_of[t];
        }
        if (lane == 0 && moved_here) atomicAdd(&s.moved, moved_here);
        __syncthreads();
        if (gridDim.x > 1) {
            if (t < k && s.arrived[t]) dev_add(&sh->arrived[round % 3][t], s.arrived[t]);
            if (t == 0 && s.moved) {
                dev_add(&sh->moved, (unsigned long long)s.moved);
                s.moved = 0;
            }
            grid_barrier(sh, generation);
            if (t < k) s.arrived[t] = dev_load(&sh->arrived[round % 3][t]);
        }
        // The loads after this round are known without counting again: every overloaded partition is down to the
        // capacity and the others got their arrivals; the capacity itself (a function of the class size) stays.
        // If nothing exceeds it, the next round's evaluation would find the same and end the call.
        if (t == 0) s.over = 0;
        __syncthreads();
        if (t < k && s.m_of[t] == 0) {
            const long long before = s.cap - (s.cumf[t] - (t > 0 ? s.cumf[t - 1] : 0));   // free capacity = cap - load, or 0 at load == cap
            if (before + (long long)s.arrived[t] > s.cap) s.over = 1;
        }
        __syncthreads();
        if (s.over == 0) {   // uniform over the grid
            if (blockIdx.x == 0 && t == 0) {
                stats[0] = round + 1;
                stats[1] = gridDim.x == 1 ? (int64_t)s.moved : (int64_t)dev_load(&sh->moved);
                stats[2] = 0;
            }
            return;
        }
        __syncthreads();
    }
}

constexpr int kBalBlocksMax = 256;     // workgroups: one per compute unit

// Compute units of the current device (asked once per device).
int compute_units(int *out) {
    static std::atomic<int> cached[64];
    int dev = 0;
    EP_HIP_TRY(hipGetDevice(&dev));
    int cus = cached[dev & 63].load(std::memory_order_relaxed);
    if (cus == 0) {
        EP_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        cached[dev & 63].store(cus, std::memory_order_relaxed);
    }
    *out = cus;
    return EP_OK;
}

template <typename RowT>
int launch_rounds(int64_t n, int32_t k, const RowT *rowptr, const uint8_t *vclass, int32_t class_id, double beta,
                  uint64_t seed, int32_t max_rounds, int32_t *labels, int64_t *stats, const BalanceWs &w, hipStream_t s) {
    static std::atomic<uint64_t> attr_set{0};   // the LDS limit is raised once per device
    int dev = 0, cus = 0;
    EP_HIP_TRY(hipGetDevice(&dev));
    const void *kern = reinterpret_cast<const void *>(&bal_rounds_kernel<RowT>);
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_set.load(std::memory_order_acquire) & bit)) {
        EP_HIP_TRY(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(BalLds)));
        attr_set.fetch_or(bit, std::memory_order_release);
    }
    int rc = compute_units(&cus);
    if (rc != EP_OK) return rc;
    const int64_t most = std::min(kBalBlocksMax, std::max(1, cus));
    const int64_t rows_per_block = n <= kSingleN ? n : ceil_div(std::max<int64_t>(ceil_div(n, most), kBalRowsMin), 64) * 64;
    const unsigned grid = (unsigned)ceil_div(n, rows_per_block);
    BalShared *sh = reinterpret_cast<BalShared *>(w.shared);
    if (grid == 1) {   // nobody to wait for: an ordinary launch
        bal_rounds_kernel<RowT><<<1, kBalBlock, sizeof(BalLds), s>>>(n, rows_per_block, k, rowptr, vclass, class_id, beta, seed,
                                                                     max_rounds, labels, stats, sh, w.tie);
        EP_LAUNCH_CHECK();
        return EP_OK;
    }
    bal_reset_kernel<<<1, kBalBlock, 0, s>>>(sh);
    EP_LAUNCH_CHECK();
    int64_t n_ = n, rows_ = rows_per_block;
    unsigned int *tie = w.tie;
    void *args[] = {&n_, &rows_, &k, &rowptr, &vclass, &class_id, &beta, &seed, &max_rounds, &labels, &stats, &sh, &tie};
    EP_HIP_TRY(hipLaunchCooperativeKernel(kern, dim3(grid), dim3(kBalBlock), args, (unsigned)sizeof(BalLds), s));
    return EP_OK;
}

}  // namespace

BalanceWs carve_balance_ws(int64_t n, void *ws) {
    (void)n;
    Carver c(ws);
    BalanceWs w{};
    w.shared = c.take<unsigned char>(sizeof(BalShared));
    w.tie = c.take<unsigned int>((size_t)kBalBlocksMax * 256);
    w.bytes = align_up(c.used, 256);
    return w;
}

int launch_balance(int64_t n, int32_t k, const void *rowptr, bool i64, const uint8_t *vclass, int32_t class_id,
                   double beta, uint64_t seed, int32_t max_rounds, int32_t *labels, int64_t *stats,
                   const BalanceWs &w, hipStream_t s) {
    if (k > kPartMax) return EP_EUNSUPPORTED;
    return i64 ? launch_rounds(n, k, static_cast<const int64_t *>(rowptr), vclass, class_id, beta, seed, max_rounds, labels,
                               stats, w, s)
               : launch_rounds(n, k, static_cast<const int32_t *>(rowptr), vclass, class_id, beta, seed, max_rounds, labels,
                               stats, w, s);
}

}  // namespace ep
