// Index construction: L layers of k p-stable functions (Sections 1.1 and 3).
//
// All layers of a chunk together (a chunk holds as many layers as its
// temporaries allow): hash every point (the same exact hashing as the query
// path), pack the k-tuples into exact keys, partition each layer's points by
// the top bits of the mixed key, and let one workgroup group each partition's
// equal keys in LDS: it lays the buckets out as CSR id lists and writes its
// region of the layer's probe table, keyed by the packed keys.
//
// A partition's keys meet only inside its workgroup, so grouping needs no
// global atomics beyond the partitioning's (one per tile and partition), no
// table of a layer's size and no host round trip per layer; the host reads
// back twice per chunk (the value ranges that fix the key packing, the
// buckets that fix the table sizes).  Bound by the passes over memory: the
// hash values (4 k bytes per point and layer) written once and read twice,
// the keys and ids four times, the tables written once.
// Measured (1M x 128 uint8, L = 20, k = 10, w = 1200, everything after the
// hashing): 19.4 ms of kernels, 20 waits and 40 allocations a layer at a time
// through a global table; 1.1 ms, 8 waits and 6 allocations in 4 chunks here,
// the whole build with its first workload 32.7 ms before and 3.2 now.
// A dominant bucket is the work of one workgroup, whose atomics meet on it.  All
// points in one bucket of each of 20 layers (1M x 32): 38.8 ms (2,245 through the
// global table), half of them 17.3 (1,149); 10M points, 4 layers of one bucket 271
// (4,339).
#include <algorithm>
#include <cmath>
#include <memory>
#include <vector>

#include "qw_internal.h"
#include "qw_keys.h"

namespace qw {

// ---------------------------------------------------------------- kernels

// Per function, for the host's checks: sum |a_i| (inflated past its rounding),
// the largest |a_i| as FP32 bits (a NaN's exceed infinity's) and b.
struct FunInfo {
    double an;
    uint32_t amax;
    float b;
};

__host__ __device__ inline double gamma_n(double n, double u) { return n * u / (1.0 - n * u); }

// One wave per function of the nf_pad rows: the zero-padded parameters in FP32
// and, layer-major, in FP64 (a64l[l][e][j] = a[l * k + j][e]); their FP16 split
// (ahi null: none); the guard-band coefficients, coef * max|v| bounding
// |approximate projection - FP64 index-order projection|; FunInfo.  The sums
// run in another order than an index-order loop's; the inflation by 10^-6
// covers either's rounding.
__global__ __launch_bounds__(kBlock) void params_kernel(
    const float *__restrict__ a, const float *__restrict__ b, int32_t L, int32_t k, int32_t d, int32_t dp,
    int32_t nf_pad, float *__restrict__ a32, double *__restrict__ a64l, _Float16 *__restrict__ ahi,
    _Float16 *__restrict__ alo, float *__restrict__ b32, double *__restrict__ gb_plain,
    double *__restrict__ gb_fast, FunInfo *__restrict__ info)
{
    const int lane = threadIdx.x & 63, nf = L * k;
    const int f = (int)blockIdx.x * (kBlock / 64) + (int)(threadIdx.x >> 6);
    if (f >= nf_pad) return;  // whole waves
    const int l = f / k, j = f - l * k;
    double an = 0.0, ahn = 0.0, aln = 0.0, rep = 0.0;
    uint32_t amax = 0;
    for (int i = lane; i < dp; i += 64) {
        const float v = f < nf && i < d ? a[(int64_t)f * d + i] : 0.f;
        a32[(int64_t)f * dp + i] = v;
        if (f < nf) a64l[((int64_t)l * dp + i) * k + j] = (double)v;
        an += fabs((double)v);
        amax = max(amax, __float_as_uint(v) & 0x7FFFFFFFu);
        if (ahi) {
            const _Float16 h = (_Float16)v;
            const float r = v - (float)h;  // exact: h is v rounded to 11 bits
            _Float16 lo = (_Float16)r;
            if (fabsf((float)lo) < 6.103515625e-05f) lo = (_Float16)0.f;  // no FP16 subnormals
            ahi[(int64_t)f * dp + i] = h;
            alo[(int64_t)f * dp + i] = lo;
            ahn += fabs((double)(float)h);
            aln += fabs((double)(float)lo);
            rep += fabs((double)v - (double)(float)h - (double)(float)lo);
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        an += __shfl_xor(an, o);
        ahn += __shfl_xor(ahn, o);
        aln += __shfl_xor(aln, o);
        rep += __shfl_xor(rep, o);
        amax = max(amax, (uint32_t)__shfl_xor((int)amax, o));
    }
    if (lane != 0 || f >= nf) return;
    const double u32 = 0x1p-24, u64 = 0x1p-53, safety = 1.0 + 1e-6;
    const double g32 = gamma_n(d + 2, u32), g64 = gamma_n(d + 2, u64);
    an *= safety;
    gb_plain[f] = (g32 + g64) * an * safety;
    if (ahi) {
        gb_fast[f] = (rep * safety + 2.0 * g32 * (ahn + aln) * safety + g64 * an) * safety;
    } else {
        // FP32 matrix cores, float data: FP32 within each chunk of kHashChunkF32
        // elements (factor 2: unknown internal order), FP64 over the chunk sums
        const double g32c = gamma_n(kHashChunkF32 + 3, u32);
        const double g64c = gamma_n((dp + kHashChunkF32 - 1) / kHashChunkF32 + 1, u64);
        gb_fast[f] = (2.0 * g32c + g64c + g64) * an * safety;
    }
    b32[f] = b[f];
    info[f] = FunInfo{an, amax, b[f]};
}

// Largest |x| as FP32 bits, which order as the values do; a NaN's exceed
// infinity's (rejected later).  One atomic per workgroup: one per wave of a
// grid sized by the elements serialised on its address (1M x 960: 3.07 ms,
// 0.63 ms now).
__global__ __launch_bounds__(kBlock) void maxabs_f32_kernel(const float4 *__restrict__ x, int64_t count4,
                                                            uint32_t *out)
{
    __shared__ uint32_t part[kBlock / 64];
    uint32_t m = 0;
    auto bits = [](float v) { return __float_as_uint(v) & 0x7FFFFFFFu; };
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count4;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float4 v = x[i];
        m = max(max(m, max(bits(v.x), bits(v.y))), max(bits(v.z), bits(v.w)));
    }
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) m = max(m, part[w]);
        atomicMax(out, m);
    }
}

// Value range of every function: a thread keeps one function and walks the
// workgroup's rows, so a wave reads consecutive functions of a row.
__global__ __launch_bounds__(kBlock) void minmax_kernel(const int32_t *__restrict__ h, int64_t n,
                                                        int32_t ld, int32_t rows_per_block,
                                                        int32_t *hmin, int32_t *hmax)
{
    __shared__ int32_t smin[kBlock], smax[kBlock];
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r1 = min(n, r0 + rows_per_block);
    const int rp = ld >= kBlock ? 1 : kBlock / ld;  // rows side by side
    for (int f0 = 0; f0 < ld; f0 += kBlock) {       // one round unless ld > kBlock
        const int r = rp > 1 ? (int)threadIdx.x / ld : 0;
        const int f = rp > 1 ? (int)threadIdx.x - r * ld : f0 + (int)threadIdx.x;
        int32_t mn = INT32_MAX, mx = INT32_MIN;
        if (r < rp && f < ld) {
#pragma unroll 8
            for (int64_t i = r0 + r; i < r1; i += rp) {
                const int32_t v = h[i * ld + f];
                mn = min(mn, v);
                mx = max(mx, v);
            }
        }
        __syncthreads();
        smin[threadIdx.x] = mn;
        smax[threadIdx.x] = mx;
        __syncthreads();
        if (r == 0 && f < ld) {
            for (int i = 1; i < rp; ++i) {
                mn = min(mn, smin[i * ld + f]);
                mx = max(mx, smax[i * ld + f]);
            }
            // most workgroups find the range settled already
            if (mn < hmin[f]) atomicMin(&hmin[f], mn);
            if (mx > hmax[f]) atomicMax(&hmax[f], mx);
        }
    }
}

// Packed keys of the nl layers in [n][nl * k] hash values, layer-major:
// klo[l * n + p], khi likewise (nullable: every layer's keys fit 64 bits).
// Rows are staged through LDS (tr at a time, an odd stride), so the values are
// read in whole rows and the keys written in whole lines.
__global__ __launch_bounds__(kBlock) void pack_kernel(const int32_t *__restrict__ h, int64_t n,
                                                      int32_t nl, int32_t k, int32_t tr,
                                                      const int32_t *__restrict__ hmin,
                                                      const int32_t *__restrict__ shift,
                                                      uint64_t *__restrict__ klo,
                                                      uint64_t *__restrict__ khi)
{
    extern __shared__ int32_t sh[];
    const int nf = nl * k, ld = nf | 1;
    int32_t *smin = sh, *sshift = sh + nf, *rows = sh + 2 * nf;
    for (int f = threadIdx.x; f < nf; f += kBlock) {
        smin[f] = hmin[f];
        sshift[f] = shift[f];
    }
    for (int64_t t0 = (int64_t)blockIdx.x * tr; t0 < n; t0 += (int64_t)gridDim.x * tr) {
        const int m = (int)min((int64_t)tr, n - t0);
        __syncthreads();  // the previous rows have been read (and the constants written)
        if ((nf & 3) == 0) {  // whole 16-byte pieces of the tile
            const int4 *src = reinterpret_cast<const int4 *>(h + t0 * nf);
            const int np = m * (nf / 4);
#pragma unroll 4
            for (int e = threadIdx.x; e < np; e += kBlock) {
                const int4 v = src[e];
                const int r = e / (nf / 4);
                int32_t *dst = rows + r * ld + 4 * (e - r * (nf / 4));
                dst[0] = v.x;
                dst[1] = v.y;
                dst[2] = v.z;
                dst[3] = v.w;
            }
        } else {
#pragma unroll 4
            for (int e = threadIdx.x; e < m * nf; e += kBlock) {
                const int r = e / nf;
                rows[r * ld + (e - r * nf)] = h[t0 * nf + e];
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < tr * nl; i += kBlock) {
            const int r = i % tr, l = i / tr;  // tr: a power of two
            if (r >= m) continue;
            uint64_t lo = 0, hi = 0;
            const int32_t *v = rows + r * ld + l * k;
            for (int j = 0; j < k; ++j)
                key_put(lo, hi, (uint64_t)((int64_t)v[j] - (int64_t)smin[l * k + j]), sshift[l * k + j]);
            klo[(int64_t)l * n + t0 + r] = lo;
            if (khi) khi[(int64_t)l * n + t0 + r] = hi;
        }
    }
}

// ---------------------------------------------------------------- partitioning
// Points of layer blockIdx.y go to partition key_part(mix) of 2^pb.  A
// workgroup takes a tile of kTile points; with LDSH it counts them per
// partition in LDS and touches a partition's global counter once per tile,
// else (more partitions than LDS counters) once per point.
constexpr int kTile = 16384;
constexpr int kLdsPart = 13;  // log2 of the partitions LDS counters cover

template <bool LDSH>
__global__ __launch_bounds__(kBlock) void part_count_kernel(const uint64_t *__restrict__ klo,
                                                            const uint64_t *__restrict__ khi, int64_t n,
                                                            int32_t pb, uint32_t *__restrict__ total)
{
    extern __shared__ uint32_t cnt[];
    const int P = 1 << pb;
    const int64_t lo = (int64_t)blockIdx.y * n, t0 = (int64_t)blockIdx.x * kTile;
    const int64_t t1 = min(n, t0 + kTile);
    uint32_t *tot = total + ((int64_t)blockIdx.y << pb);
    if (LDSH) {
        for (int p = threadIdx.x; p < P; p += kBlock) cnt[p] = 0u;
        __syncthreads();
    }
#pragma unroll 4
    for (int64_t i = t0 + threadIdx.x; i < t1; i += kBlock) {
        const uint32_t p = key_part(key_mix(klo[lo + i], khi ? khi[lo + i] : 0ull), pb);
        if (LDSH) atomicAdd(&cnt[p], 1u);
        else atomicAdd(&tot[p], 1u);
    }
    if (LDSH) {
        __syncthreads();
        for (int p = threadIdx.x; p < P; p += kBlock)
            if (cnt[p]) atomicAdd(&tot[p], cnt[p]);
    }
}

// Per layer: first[p] = points in the partitions before p (first[P] = n), and
// total[p] becomes the cursor the scatter takes ranges from.
__global__ __launch_bounds__(kBlock) void part_scan_kernel(uint32_t *__restrict__ total, int32_t pb,
                                                           uint32_t *__restrict__ first)
{
    __shared__ uint32_t wsum[kBlock / 64];
    const int64_t P = int64_t(1) << pb;
    uint32_t *tot = total + (int64_t)blockIdx.x * P;
    uint32_t *f = first + (int64_t)blockIdx.x * (P + 1);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int64_t b = 0; b < P; b += kBlock) {
        const int64_t p = b + threadIdx.x;
        const uint32_t v = p < P ? tot[p] : 0u;
        uint32_t x = v;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, off);
            if (lane >= off) x += y;
        }
        __syncthreads();  // the previous round's sums have been read
        if (lane == 63) wsum[wv] = x;
        __syncthreads();
        uint32_t before = carry, all = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            before += w < wv ? wsum[w] : 0u;
            all += wsum[w];
        }
        if (p < P) {
            f[p] = before + x - v;
            tot[p] = before + x - v;
        }
        carry += all;
    }
    if (threadIdx.x == 0) f[P] = carry;
}

// A partitioned point: its key and id, in one record (a scattered record costs
// one memory transaction where separate arrays cost one each).
template <bool WIDE> struct PartRec;
template <> struct PartRec<false> {
    uint32_t w[3];
    __device__ uint64_t lo() const { return (uint64_t)w[1] << 32 | w[0]; }
    __device__ uint64_t hi() const { return 0ull; }
    __device__ uint32_t id() const { return w[2]; }
    __device__ void set(uint64_t l, uint64_t, uint32_t i)
    {
        w[0] = (uint32_t)l;
        w[1] = (uint32_t)(l >> 32);
        w[2] = i;
    }
};
template <> struct PartRec<true> {
    uint32_t w[5];
    __device__ uint64_t lo() const { return (uint64_t)w[1] << 32 | w[0]; }
    __device__ uint64_t hi() const { return (uint64_t)w[4] << 32 | w[3]; }
    __device__ uint32_t id() const { return w[2]; }
    __device__ void set(uint64_t l, uint64_t h, uint32_t i)
    {
        w[0] = (uint32_t)l;
        w[1] = (uint32_t)(l >> 32);
        w[2] = i;
        w[3] = (uint32_t)h;
        w[4] = (uint32_t)(h >> 32);
    }
};

// Scatter of a tile of `tile` points (at most 8 per thread): ranked per
// partition and reordered in LDS, so that a partition's points of the tile
// leave as one run (8192 points over 1024 partitions: runs of 96 bytes; point
// by point the same records took 0.79 ms for 20 layers of 1M, in runs
// 0.11).
constexpr int kScatBlock = 1024;
__host__ __device__ inline size_t scatter_lds_bytes(int tile, int pb, bool wide)
{
    return (size_t)tile * (wide ? 20 : 12) + (size_t(8) << pb);
}

template <bool WIDE>
__global__ __launch_bounds__(kScatBlock) void part_scatter_kernel(
    const uint64_t *__restrict__ klo, const uint64_t *__restrict__ khi, int64_t n, int32_t pb,
    int32_t tile, uint32_t *__restrict__ cursor, PartRec<WIDE> *__restrict__ out)
{
    using Rec = PartRec<WIDE>;
    extern __shared__ uint32_t sm[];
    __shared__ uint32_t wsum[kScatBlock / 64];
    const int P = 1 << pb, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t *cnt = sm, *delta = sm + P;  // counts, then local starts; global minus local start
    Rec *recs = reinterpret_cast<Rec *>(sm + 2 * P);
    const int64_t lo = (int64_t)blockIdx.y * n, t0 = (int64_t)blockIdx.x * tile;
    const int m = (int)min((int64_t)tile, n - t0);
    uint32_t *cur = cursor + ((int64_t)blockIdx.y << pb);
    for (int p = tid; p < P; p += kScatBlock) cnt[p] = 0u;
    uint64_t kl[8], kh[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int e = tid + i * kScatBlock;
        kl[i] = e < m ? klo[lo + t0 + e] : 0ull;
        kh[i] = WIDE && e < m ? khi[lo + t0 + e] : 0ull;
    }
    __syncthreads();
    uint32_t part[8], rank[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        part[i] = key_part(key_mix(kl[i], kh[i]), pb);
        rank[i] = tid + i * kScatBlock < m ? atomicAdd(&cnt[part[i]], 1u) : 0u;
    }
    __syncthreads();
    uint32_t carry = 0;
    for (int b = 0; b < P; b += kScatBlock) {
        const int p = b + tid;
        const uint32_t v = p < P ? cnt[p] : 0u;
        uint32_t x = v;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, off);
            if (lane >= off) x += y;
        }
        __syncthreads();  // the previous round's sums have been read
        if (lane == 63) wsum[wv] = x;
        __syncthreads();
        uint32_t before = carry, all = 0;
        for (int w = 0; w < kScatBlock / 64; ++w) {
            before += w < wv ? wsum[w] : 0u;
            all += wsum[w];
        }
        if (p < P) {
            const uint32_t start = before + x - v;
            cnt[p] = start;
            if (v) delta[p] = atomicAdd(&cur[p], v) - start;
        }
        carry += all;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int e = tid + i * kScatBlock;
        if (e < m) recs[cnt[part[i]] + rank[i]].set(kl[i], kh[i], (uint32_t)(t0 + e));
    }
    __syncthreads();
    for (int e = tid; e < m; e += kScatBlock) {
        const Rec r = recs[e];
        out[lo + (uint32_t)(delta[key_part(key_mix(r.lo(), r.hi()), pb)] + (uint32_t)e)] = r;
    }
}

// More partitions than LDS counters: every point takes its place by itself.
template <bool WIDE>
__global__ __launch_bounds__(kBlock) void part_scatter_direct_kernel(
    const uint64_t *__restrict__ klo, const uint64_t *__restrict__ khi, int64_t n, int32_t pb,
    uint32_t *__restrict__ cursor, PartRec<WIDE> *__restrict__ out)
{
    const int64_t lo = (int64_t)blockIdx.y * n;
    uint32_t *cur = cursor + ((int64_t)blockIdx.y << pb);
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        const uint64_t a = klo[lo + i], b = WIDE ? khi[lo + i] : 0ull;
        PartRec<WIDE> r;
        r.set(a, b, (uint32_t)i);
        out[lo + atomicAdd(&cur[key_part(key_mix(a, b), pb)], 1u)] = r;
    }
}

// ---------------------------------------------------------------- grouping
// One partition's points [p0, p0 + m): its distinct keys in an LDS table of
// tmask + 1 slots.  rep[s] = a point (partition-relative) holding the slot's
// key, cnt[s] = points with that key.
template <bool WIDE> struct Group {
    const PartRec<WIDE> *pt;
    uint32_t *rep, *cnt;
    uint32_t tmask;
    __device__ bool same(uint32_t a, uint64_t l, uint64_t h) const
    {
        return pt[a].lo() == l && (!WIDE || pt[a].hi() == h);
    }
    __device__ uint32_t home(uint64_t l, uint64_t h) const { return (uint32_t)(key_mix(l, h) >> 20) & tmask; }
    // the slot of a key that is in the table
    __device__ uint32_t find(uint64_t l, uint64_t h) const
    {
        uint32_t s = home(l, h);
        while (!same(rep[s], l, h)) s = (s + 1) & tmask;
        return s;
    }
};

// Whole workgroup: clears the table and inserts the m points.  Returns false
// (uniform) when they hold more than `limit` distinct keys, else their number
// in *distinct.
template <bool WIDE>
__device__ inline bool group_insert(const Group<WIDE> &g, uint32_t m, uint32_t limit, uint32_t *distinct)
{
    for (uint32_t s = threadIdx.x; s <= g.tmask; s += kBlock) {
        g.rep[s] = kEmpty;
        g.cnt[s] = 0u;
    }
    if (threadIdx.x == 0) *distinct = 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < m; i += kBlock) {
        const uint64_t l = g.pt[i].lo(), h = g.pt[i].hi();
        uint32_t s = g.home(l, h);
        // a table with no slot left for a new key ends the walk
        for (uint32_t it = 0; it <= g.tmask; ++it) {
            uint32_t r = g.rep[s];
            if (r == kEmpty) {
                r = atomicCAS(&g.rep[s], kEmpty, i);
                if (r == kEmpty) {
                    r = i;
                    atomicAdd(distinct, 1u);
                }
            }
            if (r == i || g.same(r, l, h)) {
                atomicAdd(&g.cnt[s], 1u);
                break;
            }
            if (*(volatile uint32_t *)distinct > limit) break;
            s = (s + 1) & g.tmask;
        }
    }
    __syncthreads();
    return *distinct <= limit;
}

struct GroupStats {  // of a partition, or of a layer
    unsigned long long buckets, sumsq;
    uint32_t max_bucket, max_distinct;  // max_distinct: per partition; kEmpty = beyond the table
};

// Buckets of each partition: number, sum of size^2 (with the layer's n points,
// sum s^2 / n is the mean size of the bucket a point, or a query near the
// data, falls in), largest.  One record per partition, summed by the next
// kernel: 20 K workgroups adding to their layer's counters took 1.2 ms.
constexpr int kCountTab = 12;
template <bool WIDE>
__global__ __launch_bounds__(kBlock) void group_count_kernel(const PartRec<WIDE> *__restrict__ recs,
                                                             int64_t n, int32_t pb,
                                                             const uint32_t *__restrict__ first,
                                                             GroupStats *__restrict__ pstats)
{
    __shared__ uint32_t rep[1 << kCountTab], cnt[1 << kCountTab];
    __shared__ uint32_t distinct;
    __shared__ unsigned long long wsq[kBlock / 64];
    __shared__ uint32_t wmx[kBlock / 64];
    const int64_t p = blockIdx.x;
    const uint32_t *f = first + (int64_t)blockIdx.y * ((int64_t(1) << pb) + 1);
    const uint32_t b = f[p], m = f[p + 1] - b;
    int tl = 6;
    while (tl < kCountTab && (3u << tl) < 4u * m) ++tl;
    const Group<WIDE> g{recs + (int64_t)blockIdx.y * n + b, rep, cnt, (1u << tl) - 1u};
    const bool fits = group_insert(g, m, 3u << (tl - 2), &distinct);
    unsigned long long sq = 0;
    uint32_t mx = 0;
    for (uint32_t s = threadIdx.x; s <= g.tmask; s += kBlock) {
        sq += (unsigned long long)cnt[s] * cnt[s];
        mx = max(mx, cnt[s]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        sq += __shfl_xor(sq, o);
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
    }
    if ((threadIdx.x & 63) == 0) {
        wsq[threadIdx.x >> 6] = sq;
        wmx[threadIdx.x >> 6] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) {
            sq += wsq[w];
            mx = max(mx, wmx[w]);
        }
        pstats[((int64_t)blockIdx.y << pb) + p] = GroupStats{distinct, sq, mx, fits ? distinct : kEmpty};
    }
}

// One workgroup per layer: its partitions' records to one.
__global__ __launch_bounds__(kBlock) void group_sum_kernel(const GroupStats *__restrict__ pstats, int32_t pb,
                                                           GroupStats *__restrict__ stats)
{
    __shared__ GroupStats part[kBlock / 64];
    GroupStats t = {0, 0, 0, 0};
    auto add = [&](const GroupStats &o) {
        t.buckets += o.buckets;
        t.sumsq += o.sumsq;
        t.max_bucket = max(t.max_bucket, o.max_bucket);
        t.max_distinct = max(t.max_distinct, o.max_distinct);
    };
    for (int64_t p = threadIdx.x; p < (int64_t(1) << pb); p += kBlock) add(pstats[((int64_t)blockIdx.x << pb) + p]);
    for (int o = 32; o > 0; o >>= 1)
        add(GroupStats{__shfl_xor(t.buckets, o), __shfl_xor(t.sumsq, o),
                       (uint32_t)__shfl_xor((int)t.max_bucket, o), (uint32_t)__shfl_xor((int)t.max_distinct, o)});
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) add(part[w]);
        stats[blockIdx.x] = t;
    }
}

__host__ __device__ inline size_t group_lds_bytes(int tl, uint32_t ents) { return (size_t(16) << tl) + size_t(4) * ents; }

// The CSR lists and the probe-table region of one partition: the layer's
// regions hold ents entries each; a key's entry is the first free one from
// key_slot on, round the region.
template <bool WIDE>
__global__ __launch_bounds__(kBlock) void group_write_kernel(
    const PartRec<WIDE> *__restrict__ recs, int64_t n, int32_t pb, const uint32_t *__restrict__ first,
    int32_t tl, TabEntry *const *__restrict__ tabs, const uint32_t *__restrict__ tab_ents,
    int32_t *__restrict__ ids)
{
    extern __shared__ uint32_t sm[];
    __shared__ uint32_t distinct, wsum[kBlock / 64];
    const uint32_t T = 1u << tl, ents = tab_ents[blockIdx.y];
    uint32_t *rep = sm, *cnt = sm + T, *cur = sm + 2 * T, *mh = sm + 3 * T, *rmap = sm + 4 * T;
    const int64_t p = blockIdx.x, at = (int64_t)blockIdx.y * n;
    const uint32_t *f = first + (int64_t)blockIdx.y * ((int64_t(1) << pb) + 1);
    const uint32_t b = f[p], m = f[p + 1] - b;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const Group<WIDE> g{recs + at + b, rep, cnt, T - 1u};
    for (uint32_t e = tid; e < ents; e += kBlock) rmap[e] = kEmpty;
    (void)group_insert(g, m, T, &distinct);  // the table holds every partition's keys
    // bucket starts: an exclusive prefix of the counts over the slots
    uint32_t carry = b;
    for (uint32_t s0 = 0; s0 < T; s0 += kBlock) {
        const uint32_t s = s0 + tid;
        const uint32_t v = s < T ? cnt[s] : 0u;
        uint32_t x = v;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, off);
            if (lane >= off) x += y;
        }
        __syncthreads();
        if (lane == 63) wsum[wv] = x;
        __syncthreads();
        uint32_t before = carry, all = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            before += w < wv ? wsum[w] : 0u;
            all += wsum[w];
        }
        if (s < T) {
            cur[s] = before + x - v;
            mh[s] = 0xFFFFFFFFu;
            if (v) {  // its entry of the region
                const PartRec<WIDE> r = g.pt[rep[s]];
                uint32_t e = key_slot(key_mix(r.lo(), r.hi()), ents);
                while (atomicCAS(&rmap[e], kEmpty, s) != kEmpty) e = e + 1 < ents ? e + 1 : 0u;
            }
        }
        carry += all;
    }
    __syncthreads();
    // the lists, and each bucket's min-hash
    for (uint32_t i = tid; i < m; i += kBlock) {
        const PartRec<WIDE> r = g.pt[i];
        const uint32_t s = g.find(r.lo(), r.hi());
        ids[at + atomicAdd(&cur[s], 1u)] = (int32_t)r.id();
        atomicMin(&mh[s], id_mix(r.id()));
    }
    __syncthreads();
    TabEntry *t = tabs[blockIdx.y] + p * (int64_t)ents;
    for (uint32_t e = tid; e < ents; e += kBlock) {
        TabEntry w = {0, 0, 0, 0, 0, 0};
        const uint32_t s = rmap[e];
        if (s != kEmpty) {
            const PartRec<WIDE> r = g.pt[rep[s]];
            w.klo = r.lo();
            w.khi = r.hi();
            w.size = cnt[s];
            w.start = cur[s] - cnt[s];
            w.mh = mh[s];
        }
        t[e] = w;
    }
}

// Partitions the packed keys of nl layers into `recs` and counts their
// buckets; the layers' records arrive in hst once `s` has been waited for.
template <bool WIDE>
static qw_status partition_layers(const uint64_t *klo, const uint64_t *khi, int64_t n, int32_t nl, int pb,
                                  uint32_t *cursor, uint32_t *first, PartRec<WIDE> *recs,
                                  GroupStats *pstats, GroupStats *st, size_t lds_max, hipStream_t s)
{
    QW_TRY(launch_fill_u32(cursor, 0u, (int64_t)nl << pb, s));
    const dim3 tg((unsigned)ceil_div(n, kTile), (unsigned)nl);
    const bool ldsh = pb <= kLdsPart;
    if (ldsh) part_count_kernel<true><<<tg, kBlock, sizeof(uint32_t) << pb, s>>>(klo, khi, n, pb, cursor);
    else part_count_kernel<false><<<tg, kBlock, 0, s>>>(klo, khi, n, pb, cursor);
    QW_HIP(hipGetLastError());
    part_scan_kernel<<<(unsigned)nl, kBlock, 0, s>>>(cursor, pb, first);
    QW_HIP(hipGetLastError());
    if (ldsh) {
        int tile = 8 * kScatBlock;
        while (tile > kScatBlock && scatter_lds_bytes(tile, pb, WIDE) + 1024 > lds_max) tile >>= 1;
        part_scatter_kernel<WIDE><<<dim3((unsigned)ceil_div(n, tile), (unsigned)nl), kScatBlock,
                                    scatter_lds_bytes(tile, pb, WIDE), s>>>(klo, khi, n, pb, tile, cursor, recs);
    } else {
        part_scatter_direct_kernel<WIDE><<<dim3((unsigned)std::min<int64_t>(4096, ceil_div(n, kBlock)),
                                                (unsigned)nl), kBlock, 0, s>>>(klo, khi, n, pb, cursor, recs);
    }
    QW_HIP(hipGetLastError());
    group_count_kernel<WIDE><<<dim3(1u << pb, (unsigned)nl), kBlock, 0, s>>>(recs, n, pb, first, pstats);
    QW_HIP(hipGetLastError());
    group_sum_kernel<<<(unsigned)nl, kBlock, 0, s>>>(pstats, pb, st);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

// ---------------------------------------------------------------- host side

qw_status build_index(const void *data, int64_t n, int32_t d, int32_t dtype, const float *a,
                      const float *b, float w, int32_t L, int32_t k, int32_t form,
                      hipStream_t s, qw_index **out)
{
    std::unique_ptr<qw_index> ix(new qw_index());
    QW_HIP(hipGetDevice(&ix->device));
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, ix->device) == hipSuccess && v > 0)
        ix->cus = v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, ix->device) == hipSuccess && v > 0)
        ix->lds_max = (size_t)v;
    QW_HIP(hipStreamCreateWithFlags(&ix->side, hipStreamNonBlocking));
    for (auto &e : ix->fork) QW_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    ix->n = n;
    ix->d = d;
    ix->dp = (int32_t)((d + 15) / 16 * 16);
    ix->dtype = dtype;
    ix->L = L;
    ix->nprobe = 1;
    ix->nl = L;
    ix->pmagic = 0;
    ix->k = k;
    ix->nf = L * k;
    // one extra 64-row tile: function tiles may start at any f0 during the build
    ix->nf_pad = (int32_t)((ix->nf + 63) / 64 * 64 + 64);
    ix->w = w;
    const int32_t nf = ix->nf, dp = ix->dp;

    // parameters in the forms the kernels read, guard-band coefficients, and
    // what the checks below need of them
    const size_t pad = (size_t)ix->nf_pad * dp;
    DevBuf dinfo;
    QW_TRY(ix->a32.ensure(sizeof(float) * pad));
    QW_TRY(ix->a64l.ensure(sizeof(double) * (size_t)nf * dp));
    QW_TRY(ix->b32.ensure(sizeof(float) * nf));
    QW_TRY(ix->gb_plain.ensure(sizeof(double) * nf));
    QW_TRY(ix->gb_fast.ensure(sizeof(double) * nf));
    if (dtype == QW_U8) {
        QW_TRY(ix->a_hi.ensure(sizeof(_Float16) * pad));
        QW_TRY(ix->a_lo.ensure(sizeof(_Float16) * pad));
    }
    QW_TRY(dinfo.ensure(sizeof(FunInfo) * nf + sizeof(uint32_t)));
    FunInfo *fi = dinfo.as<FunInfo>();
    uint32_t *dmax = reinterpret_cast<uint32_t *>(fi + nf);
    params_kernel<<<(unsigned)ceil_div(ix->nf_pad, kBlock / 64), kBlock, 0, s>>>(
        a, b, L, k, d, dp, ix->nf_pad, ix->a32.as<float>(), ix->a64l.as<double>(), ix->a_hi.as<_Float16>(),
        ix->a_lo.as<_Float16>(), ix->b32.as<float>(), ix->gb_plain.as<double>(), ix->gb_fast.as<double>(), fi);
    QW_HIP(hipGetLastError());

    // data copy with padded rows
    QW_TRY(ix->data.ensure(row_data_bytes(ix.get())));
    QW_TRY(launch_pad_rows(data, n, d, dp, dtype, ix->data.p, s));
    QW_TRY(launch_fill_u32(dmax, 0u, 1, s));
    if (dtype == QW_F32) {
        const int64_t n4 = n * (int64_t)dp / 4;
        maxabs_f32_kernel<<<(unsigned)std::min<int64_t>(2048, ceil_div(n4, kBlock)), kBlock, 0, s>>>(
            ix->data.as<float4>(), n4, dmax);
        QW_HIP(hipGetLastError());
    }
    std::vector<FunInfo> info(nf + 1);  // the last entry's first bytes: dmax
    QW_HIP(hipMemcpyAsync(info.data(), fi, sizeof(FunInfo) * nf + sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    QW_HIP(hipStreamSynchronize(s));
    auto as_float = [](uint32_t bits) {
        float v;
        std::memcpy(&v, &bits, 4);
        return v;
    };
    float amax = 0.f;
    for (int32_t f = 0; f < nf; ++f) {
        const float v = as_float(info[f].amax);
        if (!std::isfinite(v) || !std::isfinite(info[f].b)) return QW_EINVAL;
        amax = std::max(amax, v);
    }
    ix->fast_f16 = dtype == QW_U8 && amax < 32768.f;
    // |a.v + b| / w must stay far inside int32
    double vmax = 255.0;
    if (dtype == QW_F32) {
        uint32_t bits = 0;
        std::memcpy(&bits, &info[nf], 4);
        if (!std::isfinite(as_float(bits))) return QW_EINVAL;
        vmax = as_float(bits);
    }
    for (int32_t f = 0; f < nf; ++f)
        if ((info[f].an * vmax + std::fabs((double)info[f].b)) / (double)w + 2.0 >= std::ldexp(1.0, 30))
            return QW_EINVAL;

    // per-function key ranges and shifts
    QW_TRY(ix->hmin.ensure(sizeof(int32_t) * nf));
    QW_TRY(ix->hmax.ensure(sizeof(int32_t) * nf));
    QW_TRY(ix->shift.ensure(sizeof(int32_t) * nf));
    std::vector<int32_t> hmin(nf), hmax(nf), shift(nf, 0);
    ix->key_bits.assign(L, 0);
    QW_TRY(ix->ids.ensure(sizeof(int32_t) * (size_t)L * n));

    // Layers per chunk: 384 MB of temporaries (1M points, k = 10: six layers,
    // 60 of a hash tile's 64 functions), one layer at least.
    const int64_t layer_bytes = n * (std::max<int64_t>(4 * (int64_t)k, sizeof(PartRec<true>)) + 16);
    const int64_t chunk_layers = std::max<int64_t>(1, std::min<int64_t>(L, (int64_t)384000000 / layer_bytes));
    // partitions per layer: about 512 to 1024 points each, up to 2048 before
    // their number outgrows the LDS counters (10M points: scattering point by
    // point to 2^14 partitions took 2.4 ms for 2 layers, reordered tiles to
    // 2^13 take 0.43 ms)
    int pb = 0;
    while ((n >> pb) > (pb < kLdsPart ? 1024 : 2048)) ++pb;
    const size_t cn = (size_t)(n * chunk_layers);
    // the hash values are dead once packed: the partitioned records take their
    // place
    auto aligned = [](size_t v) { return (v + 255) & ~size_t(255); };
    const size_t kbytes = aligned(sizeof(uint64_t) * cn);
    const size_t hbytes = std::max(aligned(sizeof(int32_t) * cn * (size_t)k), aligned(sizeof(PartRec<true>) * cn));
    std::vector<GroupStats> hst((size_t)L);
    DevBuf stats, pbuf;
    int tries = 0;
    QW_TRY(stats.ensure(sizeof(GroupStats) * L));
    QW_TRY(ix->tab_ptr.ensure(sizeof(TabEntry *) * L));
    QW_TRY(ix->tab_ents.ensure(sizeof(uint32_t) * L));
    std::vector<TabEntry *> tptr(L);
    TabEntry *tab_next = nullptr;
    int64_t tab_left = 0;
    std::vector<uint32_t> ents(L);
    DevBuf arena;  // one allocation: freeing a large one costs 0.3 ms
    QW_TRY(arena.ensure(hbytes + 2 * kbytes));
    char *const mem = arena.as<char>();

    for (int32_t l0 = 0; l0 < L; l0 += (int32_t)chunk_layers) {
        const int32_t nl = (int32_t)std::min<int64_t>(chunk_layers, L - l0);
        const int32_t f0 = l0 * k, nfun = nl * k;
        int32_t *hbuf = reinterpret_cast<int32_t *>(mem);
        uint64_t *klo = reinterpret_cast<uint64_t *>(mem + hbytes);
        uint64_t *khi = reinterpret_cast<uint64_t *>(mem + hbytes + kbytes);
        QW_TRY(launch_hash(ix.get(), ix->data.p, n, f0, nfun, form, hbuf, nfun, nullptr, s));
        QW_TRY(launch_fill_u32(reinterpret_cast<uint32_t *>(ix->hmin.as<int32_t>() + f0),
                               (uint32_t)INT32_MAX, nfun, s));
        QW_TRY(launch_fill_u32(reinterpret_cast<uint32_t *>(ix->hmax.as<int32_t>() + f0),
                               (uint32_t)INT32_MIN, nfun, s));
        const int32_t rpb = (int32_t)std::max<int64_t>(64, ceil_div(n, 2048));
        minmax_kernel<<<(unsigned)ceil_div(n, rpb), kBlock, 0, s>>>(
            hbuf, n, nfun, rpb, ix->hmin.as<int32_t>() + f0, ix->hmax.as<int32_t>() + f0);
        QW_HIP(hipGetLastError());
        QW_HIP(hipMemcpyAsync(hmin.data() + f0, ix->hmin.as<int32_t>() + f0, sizeof(int32_t) * nfun,
                              hipMemcpyDeviceToHost, s));
        QW_HIP(hipMemcpyAsync(hmax.data() + f0, ix->hmax.as<int32_t>() + f0, sizeof(int32_t) * nfun,
                              hipMemcpyDeviceToHost, s));
        QW_HIP(hipStreamSynchronize(s));
        bool wide = false;  // some layer's keys exceed 64 bits
        for (int32_t l = l0; l < l0 + nl; ++l) {
            int32_t pos = 0;
            for (int32_t j = 0; j < k; ++j) {
                const int32_t f = l * k + j;
                const uint64_t range = (uint64_t)((int64_t)hmax[f] - (int64_t)hmin[f]) + 1;
                const int32_t bits = range <= 1 ? 0 : ceil_log2(range);
                if (pos < 64 && pos + bits > 64) pos = 64;
                shift[f] = pos;
                pos += bits;
            }
            if (pos > 128) return QW_EUNSUPPORTED;
            ix->key_bits[l] = pos;
            wide |= pos > 64;
        }
        QW_HIP(hipMemcpyAsync(ix->shift.as<int32_t>() + f0, shift.data() + f0,
                              sizeof(int32_t) * nfun, hipMemcpyHostToDevice, s));
        if (!wide) khi = nullptr;
        int tr = 64;  // rows staged at a time
        auto pack_lds = [&](int r) { return sizeof(int32_t) * (2 * (size_t)nfun + (size_t)r * (nfun | 1)); };
        while (tr > 1 && pack_lds(tr) > 40 * 1024) tr >>= 1;
        pack_kernel<<<(unsigned)std::min<int64_t>(4096, ceil_div(n, tr)), kBlock, pack_lds(tr), s>>>(
            hbuf, n, nl, k, tr, ix->hmin.as<int32_t>() + f0, ix->shift.as<int32_t>() + f0, klo, khi);
        QW_HIP(hipGetLastError());

        GroupStats *st = stats.as<GroupStats>() + l0;
        // cursors, partition starts, partition records
        const size_t cwords = ((size_t)chunk_layers << pb), fwords = (size_t)chunk_layers * ((size_t(1) << pb) + 1);
        const size_t pword = (cwords + fwords + 1) & ~size_t(1);
        QW_TRY(pbuf.ensure(sizeof(uint32_t) * pword + sizeof(GroupStats) * cwords));
        uint32_t *cursor = pbuf.as<uint32_t>(), *first = cursor + cwords;
        GroupStats *pstats = reinterpret_cast<GroupStats *>(cursor + pword);
        auto *rec3 = reinterpret_cast<PartRec<false> *>(mem);
        auto *rec5 = reinterpret_cast<PartRec<true> *>(mem);
        QW_TRY(wide ? partition_layers<true>(klo, khi, n, nl, pb, cursor, first, rec5, pstats, st, ix->lds_max, s)
                    : partition_layers<false>(klo, khi, n, nl, pb, cursor, first, rec3, pstats, st, ix->lds_max, s));
        QW_HIP(hipMemcpyAsync(hst.data() + l0, st, sizeof(GroupStats) * nl, hipMemcpyDeviceToHost, s));
        QW_HIP(hipStreamSynchronize(s));
        bool over = false;
        for (int32_t l = l0; l < l0 + nl; ++l) over |= hst[l].max_distinct == kEmpty;
        if (over) {
            // a partition with more distinct keys than the counting table holds
            // (the mix failed to spread them): all layers again, four times as
            // many partitions
            if (pb >= 22 || ++tries > 4) return QW_EINTERNAL;
            pb += 2;
            ix->tabs.clear();
            ix->buckets = ix->max_bucket = 0;
            l0 = -(int32_t)chunk_layers;
            continue;
        }
        // regions: 2/5 full on average, the fullest at most half: 10K queries of
        // 60 probes over 1M points take 31.8 us in the probe kernel; half full,
        // 36.3 (longer probe sequences); a quarter, 29.5 (for 1.6 times the memory)
        uint32_t max_distinct = 0, emax = 0;
        int64_t total = 0;
        for (int32_t l = l0; l < l0 + nl; ++l) {
            const uint64_t nb = hst[l].buckets, md = hst[l].max_distinct;
            if (nb == 0 || (int64_t)nb > n) return QW_EINTERNAL;
            ents[l] = (uint32_t)std::max<uint64_t>({4, ((5 * nb / 2) >> pb) + 1, 2 * md});
            total += (int64_t)ents[l] << pb;
            max_distinct = std::max(max_distinct, (uint32_t)md);
            emax = std::max(emax, ents[l]);
            ix->buckets += (int64_t)nb;
            ix->max_bucket = std::max<int64_t>(ix->max_bucket, hst[l].max_bucket);
        }
        int tl = 6;
        while ((3u << tl) < 4u * max_distinct) ++tl;
        const size_t glds = group_lds_bytes(tl, emax);
        if (glds + 1024 > ix->lds_max) return QW_EINTERNAL;
        // One allocation for every layer's table, sized from the first chunk's
        // with a quarter to spare (its layers are draws of the same family); a
        // chunk that outgrows it gets its own.  Probes of tables spread over
        // one allocation per chunk missed the address translation twice as
        // often (10M points, 24 layers: 141 us where one block takes 70).
        if (ix->tabs.empty() || total > tab_left) {
            int64_t want = total;
            if (ix->tabs.empty()) want += ((int64_t)emax << pb) * (L - l0 - nl) * 5 / 4;
            ix->tabs.emplace_back();
            QW_TRY(ix->tabs.back().ensure(sizeof(TabEntry) * (size_t)want));
            tab_next = ix->tabs.back().as<TabEntry>();
            tab_left = want;
        }
        TabEntry *t = tab_next;
        tab_next += total;
        tab_left -= total;
        for (int32_t l = l0; l < l0 + nl; ++l) {
            tptr[l] = t;
            t += (int64_t)ents[l] << pb;
        }
        QW_HIP(hipMemcpyAsync(ix->tab_ptr.as<TabEntry *>() + l0, tptr.data() + l0, sizeof(TabEntry *) * nl,
                              hipMemcpyHostToDevice, s));
        QW_HIP(hipMemcpyAsync(ix->tab_ents.as<uint32_t>() + l0, ents.data() + l0, sizeof(uint32_t) * nl,
                              hipMemcpyHostToDevice, s));
        const dim3 wg(1u << pb, (unsigned)nl);
        TabEntry *const *tp = ix->tab_ptr.as<TabEntry *>() + l0;
        const uint32_t *te = ix->tab_ents.as<uint32_t>() + l0;
        int32_t *ids = ix->ids.as<int32_t>() + (int64_t)l0 * n;
        if (wide)
            group_write_kernel<true><<<wg, kBlock, glds, s>>>(rec5, n, pb, first, tl, tp, te, ids);
        else
            group_write_kernel<false><<<wg, kBlock, glds, s>>>(rec3, n, pb, first, tl, tp, te, ids);
        QW_HIP(hipGetLastError());
    }
    ix->tab_pb = pb;
    QW_HIP(hipStreamSynchronize(s));  // the temporaries and the host arrays go
    arena.retire(ix->device);
    pbuf.retire(ix->device);
    double sb = 0.0;
    for (int32_t l = 0; l < L; ++l) sb += (double)hst[l].sumsq / (double)n;
    ix->mean_hit_bucket = sb / L;
    *out = ix.release();
    return QW_OK;
}

}  // namespace qw
