// Workload scheduling kernels: hash-set size classes, bucket grouping keys,
// class segments and statistics.
//
// Queries of a workload whose candidate sets overlap are processed back to
// back: the sort key is a min-hash of the candidate set (the minimum over the
// query's buckets of each bucket's minimum id_mix(id), kept in the probe
// table), equal for two queries with probability equal to the Jaccard
// similarity of their sets.  The shared ids and points are then fetched from
// HBM once and served from L2 / the Infinity Cache -- the GPU counterpart of
// keeping reused index files and data objects in the cache (Sections 4 and
// 5.1).
#include "qw_internal.h"
#include "qw_mlp.h"

namespace qw {

__device__ inline uint32_t mix32(uint64_t x)
{
    x ^= x >> 33;
    x *= 0xFF51AFD7ED558CCDull;
    x ^= x >> 33;
    x *= 0xC4CEB9FE1A85EC53ull;
    x ^= x >> 33;
    return (uint32_t)x;
}

// Size class of a query from its predicted number of unique candidates
// `need`: the smallest c >= cmin with 3/4 * 2^c >= need (hash-set load factor
// <= 3/4).  Classes 0 .. ncls-2 are LDS classes (c = cmin + class), class
// ncls-1 keeps its set in global memory.
// has_pred: pred = the model's log(1 + |C(q)|) prediction.
__device__ inline int class_of(uint64_t tsum, int64_t n, const int32_t *__restrict__ exact, int64_t q,
                               bool has_pred, float pred, float margin, int32_t force_max,
                               int32_t cmin, int32_t cfloor, int32_t cmax, int32_t ncls)
{
    // |C(q)| <= min(sum of the bucket sizes, n): the class of that bound
    // always holds the set; a predicted or exact count may pick a smaller
    // one, but never one below cfloor (no occupancy gained there)
    const uint64_t bound = min(tsum, (uint64_t)n);
    uint64_t need = bound;
    if (exact) {
        need = min(need, (uint64_t)exact[q]);
    } else if (has_pred) {
        const float p = expm1f(pred + margin) + 32.f;
        if (p == p && p < (float)need) need = p > 0.f ? (uint64_t)ceilf(p) : 0;
    }
    int cb = cmin;
    while (cb < 40 && (3ull << cb) < 4 * bound) ++cb;
    int c = cmin;
    while (c < 40 && (3ull << c) < 4 * need) ++c;
    c = max(c, min(cb, cfloor));
    if (force_max && c <= cmax) c = cmax;
    return c <= cmax ? c - cmin : ncls - 1;
}

// Groups of queries that share a workgroup need a key that all the queries of a
// region have in common.  The min-hash of C(q) alone is not: for about one
// query in forty (1M x 960, w = 12) it is a point from elsewhere that collided
// by chance in one layer.  The smallest minimum of at least two layers, t(q),
// is a point near the query, but misses the region's smallest where that one
// collided once.  So the queries vote: for each recurring minimum v of a query,
// label[v] = the smallest t over the queries that have v; a query's label is
// that of t(q), followed twice.  A workload beyond kLabelSample queries is
// sampled evenly.  (Simulated on clusters of 2,000 points: keyed by the
// min-hash, 95 % of a cluster's queries agree, by t 77 to 84 %, by the label all.)
// tag[slot] holds the v that owns the slot; a v whose slot is another's keeps
// its own value.
constexpr int64_t kLabelSample = 8192;
__device__ inline uint32_t label_slot(uint32_t v, uint32_t slots) { return mix32(v) & (slots - 1u); }

// One wave per query, lane l holding layer l's minimum v (0xFFFFFFFF: a miss, or
// no layer): whether two layers at least hold it, and the smallest such value
// in *t (0xFFFFFFFF: none).
__device__ inline bool recurs(uint32_t v, int32_t L, uint32_t *t)
{
    int same = 0;
    for (int32_t i = 0; i < L; ++i) same += (uint32_t)__builtin_amdgcn_readlane((int)v, i) == v ? 1 : 0;
    const bool r = same >= 2 && v != 0xFFFFFFFFu;
    uint32_t m = r ? v : 0xFFFFFFFFu;
    for (int o = 32; o > 0; o >>= 1) m = min(m, (uint32_t)__shfl_xor((int)m, o));
    *t = m;
    return r;
}

__global__ __launch_bounds__(kBlock) void label_kernel(int64_t Q, int32_t L, int32_t step,
                                                       const uint32_t *__restrict__ bmh, uint32_t slots,
                                                       uint32_t *__restrict__ tag, uint32_t *__restrict__ label)
{
    const int lane = threadIdx.x & 63;
    const int64_t q = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * step;
    if (q >= Q) return;
    const uint32_t v = lane < L ? bmh[q * L + lane] : 0xFFFFFFFFu;
    uint32_t t;
    if (!recurs(v, L, &t)) return;
    const uint32_t s = label_slot(v, slots);
    uint32_t o = tag[s];
    if (o == 0xFFFFFFFFu) {
        o = atomicCAS(&tag[s], 0xFFFFFFFFu, v);
        if (o == 0xFFFFFFFFu) o = v;
    }
    if (o == v && label[s] > t) atomicMin(&label[s], t);
}

// Class, and bin of its label and t, of every query.  A bin is a hash of the
// label with kSub finer ones by t's: queries of one label that agree on t too are
// neighbours in the order.  (Counted bins instead of a sort: any order of the
// bins will do.)  A wave finds kBinWave queries' t after each other, lane l on
// layer l; then a thread per query looks its label up, and a bin's queries of
// one workgroup take their places there with one atomic (a skewed workload has
// one label for a seventh of its queries).
constexpr uint32_t kSub = 4;
constexpr int kBinWave = 8, kBinBlock = kBinWave * (kBlock / 64);
__device__ inline uint32_t bin_count(uint32_t v) { return v + 1u; }  // they start at 0xFFFFFFFF, like the tables

__global__ __launch_bounds__(kBlock) void group_bin_kernel(GroupOrderArgs A, uint32_t slots, uint32_t bins,
                                                           const uint32_t *__restrict__ tag,
                                                           uint32_t *__restrict__ count)
{
    __shared__ uint32_t hist[32], s_t[kBinBlock], s_m[kBinBlock], s_bin[kBinBlock], s_at[kBinBlock], s_sum[kBinBlock];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, L = A.L;
    const int64_t q0 = (int64_t)blockIdx.x * kBinBlock;
    if (tid < 32) hist[tid] = 0;
    constexpr int R = kBinWave < 8 ? kBinWave : 8;
    for (int r0 = 0; r0 < kBinWave; r0 += R) {
        uint32_t v[R], z[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t q = q0 + wv * kBinWave + r0 + r;
            const bool in = lane < L && q < A.Q;
            v[r] = in ? A.bmh[q * L + lane] : 0xFFFFFFFFu;
            z[r] = in ? A.bsize[q * L + lane] : 0u;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t tsum = z[r];  // below 2^31: the layers hold n * L entries
            uint32_t m = v[r], t;
            for (int o = 32; o > 0; o >>= 1) {
                tsum += (uint32_t)__shfl_xor((int)tsum, o);
                m = min(m, (uint32_t)__shfl_xor((int)m, o));
            }
            (void)recurs(v[r], L, &t);
            if (lane == 0) {
                s_t[wv * kBinWave + r0 + r] = t;
                s_m[wv * kBinWave + r0 + r] = m;
                s_sum[wv * kBinWave + r0 + r] = tsum;
            }
        }
    }
    __syncthreads();
    const int64_t q = q0 + tid;
    uint32_t bin = 0xFFFFFFFFu;
    if (tid < kBinBlock) {
        if (q < A.Q) {
            uint32_t t = s_t[tid], lb = t;
            for (int i = 0; i < 2 && lb != 0xFFFFFFFFu; ++i) {
                const uint32_t s = label_slot(lb, slots);
                if (tag[s] == lb) lb = min(lb, tag[slots + s]);
            }
            if (t == 0xFFFFFFFFu) t = lb = s_m[tid];
            const int cls = class_of(s_sum[tid], A.n, A.exact, q, A.pred_log != nullptr, A.pred_log ? A.pred_log[q] : 0.f,
                                     A.margin, A.force_max, A.cmin, A.cfloor, A.cmax, A.ncls);
            atomicAdd(&hist[cls], 1u);
            bin = ((mix32(lb) & (bins - 1u)) + (cls > A.gmax ? bins : 0u)) * kSub + mix32(t) % kSub;
            A.cls[q] = cls;
        }
        s_bin[tid] = bin;
    }
    __syncthreads();
    uint32_t before = 0, all = 0;
    int lead = 0;
    if (bin != 0xFFFFFFFFu) {  // the first of the bin's queries here takes their places
        lead = kBinBlock;
        for (int i = 0; i < kBinBlock; ++i) {
            const bool same = s_bin[i] == bin;
            before += same && i < tid ? 1u : 0u;
            all += same ? 1u : 0u;
            lead = same && i < lead ? i : lead;
        }
        if (lead == tid) s_at[tid] = bin_count(atomicAdd(&count[bin], all));
    }
    __syncthreads();
    if (tid < kBinBlock && q < A.Q) A.bin[q] = uint2{bin, bin != 0xFFFFFFFFu ? s_at[lead] + before : 0u};
    if (tid < A.ncls && hist[tid]) atomicAdd(&A.class_count[tid], (unsigned long long)hist[tid]);
}

// A label with minrun queries at least gives groups of kGroupMax at most, of
// even sizes, at the front of gorder; the other labels' queries go to its back,
// and so do those of classes no group takes (the second half of the bins: they
// run query by query, but neighbours still share rows in L2 -- 100,000 skewed
// queries over 1M x 960 in one class took 160 ms in label order, 199 in none).
// count[] becomes the finer bins' places there (kBack: counted from the back).
// The class segments start empty.
constexpr uint32_t kBack = 0x80000000u;
__global__ __launch_bounds__(kBlock) void group_place_kernel(GroupOrderArgs A, uint32_t bins,
                                                             uint32_t *__restrict__ count)
{
    __shared__ uint32_t wsum[3][kBlock / 64], s_base[3];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t b = blockIdx.x * kBlock + tid;
    if (blockIdx.x == 0 && tid < 2 * A.ncls) A.seg[tid] = (unsigned long long)(tid / 2) * (unsigned long long)A.Q;
    uint4 *cw = reinterpret_cast<uint4 *>(count + (size_t)b * kSub);
    uint32_t c[kSub], sum = 0;
    static_assert(kSub == 4, "one load");
    const uint4 v = b < 2u * bins ? cw[0] : uint4{~0u, ~0u, ~0u, ~0u};
    c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
#pragma unroll
    for (uint32_t i = 0; i < kSub; ++i) sum += bin_count(c[i]);
    const bool take = b < bins && sum > 0u && sum >= A.minrun;
    const uint32_t ng = take ? (sum + kGroupMax - 1u) / kGroupMax : 0u;
    const uint32_t mine[3] = {ng, take ? sum : 0u, take ? 0u : sum};  // as gcount's words
    uint32_t x[3] = {mine[0], mine[1], mine[2]};
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t y = (uint32_t)__shfl_up((int)x[k], off);
            if (lane >= off) x[k] += y;
        }
    if (lane == 63)
#pragma unroll
        for (int k = 0; k < 3; ++k) wsum[k][wv] = x[k];
    __syncthreads();
    if (tid < 3) {
        uint32_t t = 0;
        for (int w = 0; w < kBlock / 64; ++w) t += wsum[tid][w];
        s_base[tid] = t ? atomicAdd(A.gcount + tid, t) : 0u;
    }
    __syncthreads();
    if (b >= 2u * bins) return;
    uint32_t at[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        at[k] = s_base[k] + x[k] - mine[k];
        for (int w = 0; w < wv; ++w) at[k] += wsum[k][w];
    }
    uint32_t first = at[1];
    for (uint32_t i = 0; i < ng; ++i) {
        const uint32_t size = sum / ng + (i < sum % ng ? 1u : 0u);
        A.groups[at[0] + i] = uint2{first, size};
        first += size;
    }
    uint32_t pos = take ? at[1] : kBack | at[2];
#pragma unroll
    for (uint32_t i = 0; i < kSub; ++i) {
        const uint32_t n = bin_count(c[i]);
        c[i] = pos;
        pos += n;
    }
    cw[0] = uint4{c[0], c[1], c[2], c[3]};
}

// This workgroup's queries (q < 0: none) to the ends of their classes' segments
// (class c's queries at order[c * Q ..)).  Whole workgroup.
__device__ inline void append_classes(const GroupOrderArgs &A, int64_t q)
{
    __shared__ uint32_t hist[32];
    __shared__ unsigned long long base[32];
    const int tid = threadIdx.x;
    if (tid < 32) hist[tid] = 0;
    __syncthreads();
    const int cls = q >= 0 ? A.cls[q] : 0;
    const uint32_t p = q >= 0 ? atomicAdd(&hist[cls], 1u) : 0u;
    __syncthreads();
    if (tid < A.ncls && hist[tid]) base[tid] = atomicAdd(&A.seg[2 * tid + 1], (unsigned long long)hist[tid]);
    __syncthreads();
    if (q >= 0) A.order[base[cls] + p] = (int32_t)q;
}

// Every query to its place in gorder.
__global__ __launch_bounds__(kBlock) void group_scatter_kernel(GroupOrderArgs A, const uint32_t *__restrict__ place)
{
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= A.Q) return;
    const uint2 b = A.bin[q];
    const uint32_t at = place[b.x] + b.y;
    A.gorder[at & kBack ? A.Q - 1 - (int64_t)(at & ~kBack) : (int64_t)at] = (int32_t)q;
}

// The queries at the back of gorder to their classes: queries of one label stay
// together.
__global__ __launch_bounds__(kBlock) void group_rest_kernel(GroupOrderArgs A)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x, n = A.gcount[2];
    if (i - threadIdx.x >= n) return;  // uniform
    append_classes(A, i < n ? A.gorder[A.Q - 1 - i] : -1);
}

// Enough for the labels (a query each at most) to seldom share a bin: two regions
// in one group overflow its set.
uint32_t group_bins(int64_t Q)
{
    uint32_t b = 1024;
    while (b < (1u << 17) && (int64_t)b < 16 * Q) b <<= 1;
    return b;
}
size_t group_table_bytes(int64_t Q)
{
    return sizeof(uint32_t) * (2 * (size_t)kLabelSlots + 2 * (size_t)group_bins(Q) * kSub);
}

// Order of a workload whose queries share workgroups.  tab: the slots' owners and
// labels (64 slots a query, kLabelSlots at most), then the bins, twice.  100,000 queries:
// 0.12 ms (sorting them by class, label and t took 0.3).
qw_status launch_group_order(const GroupOrderArgs &a, uint32_t *tab, hipStream_t s)
{
    if (a.Q <= 0) return QW_OK;
    if (a.L > 64 || a.ncls > 32) return QW_EINTERNAL;
    uint32_t slots = 1024;
    while (slots < kLabelSlots && (int64_t)slots < 64 * a.Q) slots <<= 1;
    const uint32_t bins = group_bins(a.Q);
    uint32_t *count = tab + 2 * (size_t)slots;
    QW_TRY(launch_fill_u32(tab, 0xFFFFFFFFu, 2 * (int64_t)slots + 2 * (int64_t)bins * kSub, s));
    constexpr int wpb = kBlock / 64;
    const int32_t step = (int32_t)std::max<int64_t>(1, a.Q / kLabelSample);
    label_kernel<<<(unsigned)ceil_div(ceil_div(a.Q, step), wpb), kBlock, 0, s>>>(a.Q, a.L, step, a.bmh, slots, tab, tab + slots);
    QW_HIP(hipGetLastError());
    group_bin_kernel<<<(unsigned)ceil_div(a.Q, kBinBlock), kBlock, 0, s>>>(a, slots, bins, tab, count);
    QW_HIP(hipGetLastError());
    group_place_kernel<<<(unsigned)ceil_div(2 * (int64_t)bins, kBlock), kBlock, 0, s>>>(a, bins, count);
    QW_HIP(hipGetLastError());
    group_scatter_kernel<<<(unsigned)ceil_div(a.Q, kBlock), kBlock, 0, s>>>(a, count);
    QW_HIP(hipGetLastError());
    group_rest_kernel<<<(unsigned)ceil_div(a.Q, kBlock), kBlock, 0, s>>>(a);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

// Key = class << 16 | 16-bit group of every query, for the radix sort.
__global__ __launch_bounds__(kBlock) void classify_kernel(
    int64_t Q, int32_t L, int64_t n,
    const uint32_t *__restrict__ bmh, const uint32_t *__restrict__ bsize,
    const int32_t *__restrict__ exact, const float *__restrict__ pred_log, float margin,
    int32_t force_max, int32_t cmin, int32_t cfloor, int32_t cmax, int32_t ncls,
    unsigned long long *__restrict__ keys, int32_t *__restrict__ vals,
    unsigned long long *class_count)
{
    __shared__ uint32_t hist[32];
    if (threadIdx.x < 32) hist[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < Q;
         q += (int64_t)gridDim.x * blockDim.x) {
        uint64_t tsum = 0;
        for (int32_t l = 0; l < L; ++l) tsum += bsize[q * L + l];
        const int cls = class_of(tsum, n, exact, q, pred_log != nullptr,
                                 pred_log ? pred_log[q] : 0.f, margin, force_max, cmin, cfloor,
                                 cmax, ncls);
        uint32_t m = 0xFFFFFFFFu;  // min-hash of C(q): misses carry 0xFFFFFFFF
        for (int32_t l = 0; l < L; ++l) m = min(m, bmh[q * L + l]);
        keys[q] = ((unsigned long long)cls << 16) | (mix32(m) & 0xFFFFu);
        vals[q] = (int32_t)q;
        atomicAdd(&hist[cls], 1u);
    }
    __syncthreads();
    if (threadIdx.x < ncls && hist[threadIdx.x])
        atomicAdd(&class_count[threadIdx.x], (unsigned long long)hist[threadIdx.x]);
}

// Without bucket grouping the order within a class is free, so one kernel
// bins the queries: class c's queries go to order[c * Q ..) (any order), a
// workgroup taking one range per class per round of kBlock queries with one
// atomic on the class count.  The last workgroup to finish (its done-counter
// increment sees every other one) writes seg[2c], seg[2c+1] = [c * Q,
// c * Q + count_c).
// mlp_lane (nullable): the count model.  A prediction can only move a query
// whose bound class lies above cfloor (below it the class is the bound's), so
// only those queries are gathered into LDS and run through the MFMA
// inference, 16 at a time.
__global__ __launch_bounds__(kBlock) void classify_bin_kernel(
    int64_t Q, int32_t L, int64_t n, const uint32_t *__restrict__ bsize,
    const int32_t *__restrict__ exact, const uint32_t *__restrict__ mlp_lane, float margin,
    int32_t force_max, int32_t cmin, int32_t cfloor, int32_t cmax, int32_t ncls,
    int32_t *__restrict__ order, unsigned long long *class_count, uint32_t *done,
    unsigned long long *__restrict__ seg)
{
    extern __shared__ __align__(16) uint16_t fsh[];  // mlp: features [kBlock][ld] (bf16)
    __shared__ float pred_sh[kBlock];
    __shared__ uint32_t hist[32];
    __shared__ unsigned long long base[32];
    __shared__ uint32_t last, nmodel;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ksteps = (L + 15) / 16, kp = 16 * ksteps, ld = kp + 4;
    MlpLane m;
    if (mlp_lane) mlp_lane_load_packed(mlp_lane, m);  // in flight with the first sizes
    for (int64_t q0 = (int64_t)blockIdx.x * kBlock; q0 < Q; q0 += (int64_t)gridDim.x * kBlock) {
        const int64_t q = q0 + tid;
        if (tid < 32) hist[tid] = 0;
        if (tid == 0) nmodel = 0;
        // the query's bucket sizes, all loads in flight together (L <= 64)
        uint32_t sz[kMaxL];
#pragma unroll
        for (int32_t l = 0; l < kMaxL; ++l) sz[l] = q < Q && l < L ? bsize[q * L + l] : 0u;
        uint64_t tsum = 0;
#pragma unroll
        for (int32_t l = 0; l < kMaxL; ++l) tsum += sz[l];
        __syncthreads();  // hist and nmodel cleared
        // a slot in the model's list when the bound class exceeds cfloor
        const uint64_t bound = min(tsum, (uint64_t)n);
        const bool use = mlp_lane && q < Q && !exact && (3ull << cfloor) < 4 * bound;
        int slot = -1;
        if (use) {
            slot = (int)atomicAdd(&nmodel, 1u);
            // f_l = log(1 + s_l) by the hardware logarithm (1 + s_l is exact
            // for s_l < 2^24; the feature is rounded to bfloat16 anyway)
#pragma unroll
            for (int32_t l = 0; l < kMaxL; ++l) {
                if (l < L) fsh[slot * ld + l] = bf16_bits(__logf(1.0f + (float)sz[l]));
                else if (l < kp) fsh[slot * ld + l] = 0;
            }
        }
        __syncthreads();
        const int nm = (int)nmodel;
        for (int r0 = wave * 16; r0 < nm; r0 += kBlock / 4) {  // 16 rows per wave step
            // rows past nm hold stale features; their predictions are unused
            const mlp_f4 y = mlp_predict16(fsh + r0 * ld, ld, ksteps, m);
            if ((lane & 15) == 0)
#pragma unroll
                for (int j = 0; j < 4; ++j) pred_sh[r0 + (lane >> 4) * 4 + j] = y[j];
        }
        __syncthreads();  // predictions written
        int cls = 0;
        uint32_t p = 0;
        if (q < Q) {
            cls = class_of(tsum, n, exact, q, use, use ? pred_sh[slot] : 0.f, margin, force_max,
                           cmin, cfloor, cmax, ncls);
            p = atomicAdd(&hist[cls], 1u);
        }
        __syncthreads();
        if (tid < ncls && hist[tid])
            base[tid] = atomicAdd(&class_count[tid], (unsigned long long)hist[tid]);
        __syncthreads();
        if (q < Q) order[(int64_t)cls * Q + (int64_t)(base[cls] + p)] = (int32_t)q;
        __syncthreads();  // hist is cleared for the next round
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) last = atomicAdd(done, 1u) == gridDim.x - 1 ? 1u : 0u;
    __syncthreads();
    if (last && tid < ncls) {
        __threadfence();
        const unsigned long long cnt = atomicAdd(&class_count[tid], 0ull);  // device-coherent read
        seg[2 * tid] = (unsigned long long)tid * (unsigned long long)Q;
        seg[2 * tid + 1] = (unsigned long long)tid * (unsigned long long)Q + cnt;
    }
}

qw_status launch_classify_bin(int64_t Q, int32_t L, int64_t n, const uint32_t *bsize,
                              const int32_t *exact, const uint32_t *mlp_lane, float margin,
                              int32_t force_max, int32_t cmin, int32_t cfloor, int32_t cmax,
                              int32_t ncls, int32_t *order, unsigned long long *class_count,
                              uint32_t *done, unsigned long long *seg, hipStream_t s)
{
    if (Q <= 0) return QW_OK;
    if (ncls > 32 || L > kMaxL) return QW_EINVAL;
    const int g = (int)std::min<int64_t>(1024, ceil_div(Q, kBlock));
    // features of up to kBlock rows (a wave's steps start at multiples of 16)
    const size_t lds = mlp_lane ? sizeof(uint16_t) * (size_t)kBlock * (16 * ((L + 15) / 16) + 4) : 0;
    classify_bin_kernel<<<g, kBlock, lds, s>>>(Q, L, n, bsize, exact, mlp_lane, margin, force_max,
                                               cmin, cfloor, cmax, ncls, order, class_count, done,
                                               seg);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

qw_status launch_classify(int64_t Q, int32_t L, int64_t n,
                          const uint32_t *bmh, const uint32_t *bsize, const int32_t *exact,
                          const float *pred_log, float margin, int32_t force_max, int32_t cmin,
                          int32_t cfloor, int32_t cmax, int32_t ncls, unsigned long long *keys, int32_t *vals,
                          unsigned long long *class_count, hipStream_t s)
{
    if (Q <= 0) return QW_OK;
    int g = (int)std::min<int64_t>(1024, ceil_div(Q, kBlock));
    classify_kernel<<<g, kBlock, 0, s>>>(Q, L, n, bmh, bsize, exact, pred_log, margin,
                                         force_max, cmin, cfloor, cmax, ncls, keys, vals,
                                         class_count);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

// seg[2c], seg[2c+1] = [begin, end) of class c in the class-sorted order.
__global__ void segments_kernel(const unsigned long long *class_count, int32_t ncls,
                                unsigned long long *seg)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    unsigned long long off = 0;
    for (int c = 0; c < ncls; ++c) {
        seg[2 * c] = off;
        off += class_count[c];
        seg[2 * c + 1] = off;
    }
}

qw_status launch_segments(const unsigned long long *class_count, int32_t ncls,
                          unsigned long long *seg, hipStream_t s)
{
    segments_kernel<<<1, 64, 0, s>>>(class_count, ncls, seg);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

__global__ void max_u32_kernel(const uint32_t *__restrict__ v, int64_t count, uint32_t *out)
{
    uint32_t m = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        m = max(m, v[i]);
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    if ((threadIdx.x & 63) == 0) atomicMax(out, m);
}

qw_status launch_max_u32(const uint32_t *v, int64_t count, uint32_t *out, hipStream_t s)
{
    if (count <= 0) return QW_OK;
    int g = (int)std::min<int64_t>(1024, ceil_div(count, kBlock));
    max_u32_kernel<<<g, kBlock, 0, s>>>(v, count, out);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

// max over queries of sum_l s_{q,l} (clamped to 2^32 - 1), one atomic per wave
__global__ __launch_bounds__(kBlock) void max_bucket_sum_kernel(const uint32_t *__restrict__ bsize,
                                                                int64_t Q, int32_t L, uint32_t *out)
{
    uint32_t m = 0;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < Q;
         q += (int64_t)gridDim.x * blockDim.x) {
        uint64_t t = 0;
        for (int32_t l = 0; l < L; ++l) t += bsize[q * L + l];
        m = max(m, (uint32_t)min(t, (uint64_t)0xFFFFFFFFu));
    }
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    if ((threadIdx.x & 63) == 0 && m) atomicMax(out, m);
}

qw_status launch_max_bucket_sum(const uint32_t *bsize, int64_t Q, int32_t L, uint32_t *out,
                                hipStream_t s)
{
    if (Q <= 0) return QW_OK;
    const int g = (int)std::min<int64_t>(64, ceil_div(Q, kBlock));
    max_bucket_sum_kernel<<<g, kBlock, 0, s>>>(bsize, Q, L, out);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

// probes that hit a bucket, and the total of the bucket sizes
// Count of non-zero entries and their sum (one atomic pair per workgroup).
__global__ __launch_bounds__(kBlock) void probe_stats_kernel(const uint32_t *__restrict__ v,
                                                             int64_t count,
                                                             unsigned long long *nonzero,
                                                             unsigned long long *total)
{
    __shared__ unsigned long long sh[kBlock / 64], st[kBlock / 64];
    unsigned long long h = 0, t = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t x = v[i];
        h += x ? 1 : 0;
        t += x;
    }
    for (int off = 32; off > 0; off >>= 1) {
        h += __shfl_xor(h, off);
        t += __shfl_xor(t, off);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6] = h;
        st[threadIdx.x >> 6] = t;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) {
            h += sh[w];
            t += st[w];
        }
        atomicAdd(nonzero, h);
        atomicAdd(total, t);
    }
}

qw_status launch_probe_stats(const uint32_t *v, int64_t count, unsigned long long *nonzero,
                             unsigned long long *total, hipStream_t s)
{
    if (count <= 0) return QW_OK;
    int g = (int)std::min<int64_t>(64, ceil_div(count, kBlock));
    probe_stats_kernel<<<g, kBlock, 0, s>>>(v, count, nonzero, total);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

// Training minibatch gather and labels.
__global__ void gather_batch_kernel(const float *__restrict__ feats, const float *__restrict__ labels,
                                    const int32_t *__restrict__ perm, int32_t L, int32_t B,
                                    float *__restrict__ fb, float *__restrict__ tb)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < B * L; i += gridDim.x * blockDim.x) {
        const int s = i / L, l = i - s * L;
        fb[i] = feats[(int64_t)perm[s] * L + l];
        if (l == 0) tb[s] = labels[perm[s]];
    }
}

qw_status launch_gather_batch(const float *feats, const float *labels, const int32_t *perm,
                              int32_t L, int32_t B, float *fb, float *tb, hipStream_t s)
{
    if (B <= 0) return QW_OK;
    gather_batch_kernel<<<(unsigned)ceil_div((int64_t)B * L, kBlock), kBlock, 0, s>>>(
        feats, labels, perm, L, B, fb, tb);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

__global__ void labels_kernel(const int32_t *__restrict__ counts, int64_t m, float *__restrict__ out)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = log1pf((float)counts[i]);
}

qw_status launch_labels(const int32_t *counts, int64_t m, float *out, hipStream_t s)
{
    if (m <= 0) return QW_OK;
    int g = (int)std::min<int64_t>(4096, ceil_div(m, kBlock));
    labels_kernel<<<g, kBlock, 0, s>>>(counts, m, out);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

}  // namespace qw
