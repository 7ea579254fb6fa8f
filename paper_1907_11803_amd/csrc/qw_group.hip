// Candidate work for float rows, several queries per workgroup: queries whose
// candidate sets overlap (neighbours of the grouped order with the same
// min-hash) form their union together and verify every row of it once, on the
// matrix cores -- the bucket's points are staged once and reused by the
// queries that hit it (Sections 4 and 5.1).
//
// group_union_kernel, one workgroup per group of at most 32 queries: every
// query's listed ids go into one LDS set, each slot with a mask of the queries
// that list it; the set is compacted into (id, mask) rows and a key range is
// taken for every query's candidates.  A set beyond its capacity sends the
// group's queries to the per-query kernel, as does a small overlap with q0's
// candidates a single query.
//
// group_verify_kernel, one workgroup per group, or per piece of a group's rows
// where there are few groups: 16 x 16 blocks of rows x queries,
// v_mfma_f32_16x16x4f32 over x' = x - q0 and q' = q - q0 (q0: one query of the
// group), give F = |x'|^2 + |q'|^2 - 2 x'.q', and each (row, query) pair of the
// mask writes its (F, id) key for the select kernel.
//
// Error of F against the exact squared distance D (u = 2^-24, c = 2 (dp + 16) u,
// S = |x'| + |q'|): rounding x' and q' moves the distance by at most 2u S^2 + u^2 S^2,
// the FP32 sums of |x'|^2 and |q'|^2 by gamma_{dp/4+4} S^2, the matrix product
// (2 gamma_{dp+2} |x'||q'| for any internal order) by gamma_{dp+2} S^2, the last
// additions by 3u S^2: together at most c S^2.  With Q = |q'|, |x'| <= sqrt(D) + Q,
// so |F - D| <= c (sqrt(D) + 2Q)^2 <= 2c D + 8c Q^2.  The select kernel widens its
// bound by the relative part (group_eps) and the query's absolute part
// (abs_err), and re-ranks that band in FP64; the result does not change.
//
// The unions are bound by LDS latency (many waves, little else); the
// verification, where queries share their candidates, by the matrix cores' FP32
// rate (32 cycles per 1024 products), where they do not, by the rows' bytes.  A
// set's slots follow the ids' hash, so the rows of groups with the same
// candidates come in the same order, and the workgroups of an XCD, which take
// neighbouring groups, read them from its L2 at about the same time.
// Measured (1M x 960, w = 12): 100,000 clustered queries took 63 ms query by
// query; the unions now take 2.2 ms, the verification 7.7 (the matrix cores busy
// for half of it); 1,000 scattered ones 2.3 ms before, 0.10 and 1.02 now.
#include <algorithm>

#include "qw_dedup.h"
#include "qw_internal.h"

namespace qw {
namespace {

constexpr int kGB = 512;                                // threads per workgroup
constexpr int kGW = kGB / 64;                           // waves
constexpr int kVB = 768, kVW = kVB / 64;                // of the verification
constexpr int kGQ = 32;                                 // queries per group
constexpr int kGSetLog2 = 13;                           // set slots
constexpr uint32_t kGLimit = (1u << kGSetLog2) / 4 * 3;  // rows of a group at most (load <= 3/4)
constexpr int kGRound = 4;                              // listed ids per thread per round
constexpr int kGChunk = 64;                             // columns per chunk of a row

typedef float f4 __attribute__((ext_vector_type(4)));

__host__ __device__ inline size_t ga16(size_t v) { return (v + 15) & ~size_t(15); }

// set slots {id, mask} | list prefixes | list offsets
__host__ __device__ inline size_t union_lds(int nl)
{
    return (size_t(8) << kGSetLog2) + ga16(size_t(kGQ) * (nl + 1) * 4) + ga16(size_t(kGQ) * nl * 4);
}
// q' rows of dp + 4 floats (the padding spreads a column of rows over the banks) | q0
__host__ __device__ inline size_t verify_lds(int dp) { return size_t(kGQ) * (dp + 4) * 4 + size_t(dp) * 4; }

// Groups of the order's first seg[2 cls + 1] items: a group starts where the
// class or label changes (a run) and at every kGQ-th item of a run.  out[0] = their
// number, out[1 + g] = first item of group g, out[1 + number] = the items'
// number.  One workgroup; the keys are read once, in order.
constexpr int kRunBlock = 1024, kRunItems = 4;
template <class Key>
__device__ inline void find_groups(Key keys, int64_t N, uint32_t *__restrict__ out)
{
    __shared__ uint32_t wsum[kRunBlock / 64], wrun[kRunBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t carry = 0, crun = 0;  // groups so far, start of the run before this round (+ 1)
    for (int64_t b = 0; b < N; b += kRunBlock * kRunItems) {
        const int64_t i0 = b + (int64_t)tid * kRunItems;
        unsigned long long k[kRunItems], prev = i0 > 0 && i0 < N ? keys(i0 - 1) >> kGroupOrderBits : 0ull;
#pragma unroll
        for (int r = 0; r < kRunItems; ++r) k[r] = i0 + r < N ? keys(i0 + r) >> kGroupOrderBits : 0ull;
        // the last run start at or before each item: within the thread, then a
        // running maximum over the threads before it
        uint32_t start[kRunItems], last = 0;  // position + 1; 0: before this thread
#pragma unroll
        for (int r = 0; r < kRunItems; ++r) {
            if (i0 + r < N && (i0 + r == 0 || k[r] != prev)) last = (uint32_t)(i0 + r) + 1u;
            prev = k[r];
            start[r] = last;
        }
        uint32_t x = last;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, off);
            if (lane >= off) x = max(x, y);
        }
        uint32_t before = (uint32_t)__shfl_up((int)x, 1);
        if (lane == 0) before = 0u;
        __syncthreads();  // the previous round's values have been read
        if (lane == 63) wrun[wv] = x;
        __syncthreads();
        uint32_t all = crun;
        before = max(before, crun);
        for (int w = 0; w < kRunBlock / 64; ++w) {
            before = w < wv ? max(before, wrun[w]) : before;
            all = max(all, wrun[w]);
        }
        crun = all;
        uint32_t flags = 0;
#pragma unroll
        for (int r = 0; r < kRunItems; ++r) {
            const uint32_t st = (start[r] ? start[r] : before) - 1u;
            if (i0 + r < N && ((uint32_t)(i0 + r) - st) % kGQ == 0u) flags |= 1u << r;
        }
        const uint32_t c = (uint32_t)__popc(flags);
        x = c;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, off);
            if (lane >= off) x += y;
        }
        if (lane == 63) wsum[wv] = x;
        __syncthreads();
        uint32_t at = carry + x - c;
        for (int w = 0; w < kRunBlock / 64; ++w) {
            at += w < wv ? wsum[w] : 0u;
            carry += wsum[w];
        }
#pragma unroll
        for (int r = 0; r < kRunItems; ++r)
            if ((flags >> r) & 1u) out[1 + at++] = (uint32_t)(i0 + r);
    }
    if (tid == 0) {
        out[0] = carry;
        out[1 + carry] = (uint32_t)N;
    }
}

__global__ __launch_bounds__(kRunBlock) void group_runs_kernel(const unsigned long long *__restrict__ keys,
                                                               const unsigned long long *__restrict__ seg,
                                                               int32_t cls, uint32_t *__restrict__ out)
{
    find_groups([&](int64_t i) { return keys[i]; }, (int64_t)seg[2 * cls + 1], out);
}

// The whole order of a small workload in one workgroup: a bitonic sort of (key,
// query) words in LDS, the class segments, the groups.  (Radix passes are three
// launches each: five of them took 95 us for 1,000 queries, this 18.)
__global__ __launch_bounds__(kRunBlock) void small_order_kernel(
    unsigned long long *__restrict__ keys, int32_t *__restrict__ vals, int32_t Q,
    const unsigned long long *__restrict__ class_count, int32_t ncls, unsigned long long *__restrict__ seg,
    int32_t cls, uint32_t *__restrict__ groups)
{
    __shared__ unsigned long long w[kSmallOrder];
    __shared__ unsigned long long s_end;
    const int tid = threadIdx.x;
    int n2 = 2;
    while (n2 < Q) n2 <<= 1;
    // vals[i] = i: the key with the query below it sorts as the stable order
    for (int i = tid; i < n2; i += kRunBlock) w[i] = i < Q ? keys[i] << 12 | (unsigned)i : ~0ull;
    __syncthreads();
    for (int size = 2; size <= n2; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < n2 / 2; i += kRunBlock) {
                const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                const unsigned long long a = w[lo], b = w[hi];
                if ((b < a) == ((lo & size) == 0)) {
                    w[lo] = b;
                    w[hi] = a;
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < Q; i += kRunBlock) {
        keys[i] = w[i] >> 12;
        vals[i] = (int32_t)(w[i] & 4095u);
    }
    if (tid == 0) {
        unsigned long long off = 0;
        s_end = 0;
        for (int c = 0; c < ncls; ++c) {
            seg[2 * c] = off;
            off += class_count[c];
            seg[2 * c + 1] = off;
            if (c == cls) s_end = off;
        }
    }
    __syncthreads();
    if (groups) find_groups([&](int64_t i) { return w[i] >> 12; }, (int64_t)s_end, groups);
}

// Adds `bit` to the masks of the valid ids, inserting those not yet in the set;
// returns how many were new, sets `full` when one found no slot.  Most ids are
// there already (a candidate recurs across layers and queries), so a slot is
// read before anything is written.
__device__ inline uint32_t group_insert_ids(uint2 *tab, const uint32_t (&id)[kGRound], uint32_t valid,
                                            uint32_t bit, bool &full)
{
    constexpr uint32_t mask = (1u << kGSetLog2) - 1u;
    uint32_t slot[kGRound], nnew = 0, pend = valid;
#pragma unroll
    for (int r = 0; r < kGRound; ++r) slot[r] = hash_id(id[r], kGSetLog2);
    for (uint32_t np = 0; pend; ++np) {
        if (np >= kShortProbe) {
            full = true;
            break;
        }
        uint2 v[kGRound];
#pragma unroll
        for (int r = 0; r < kGRound; ++r) v[r] = tab[slot[r]];
#pragma unroll
        for (int r = 0; r < kGRound; ++r) {
            if (!((pend >> r) & 1u)) continue;
            uint32_t o = v[r].x;
            if (o == kEmpty) {
                o = atomicCAS(&tab[slot[r]].x, kEmpty, id[r]);
                if (o == kEmpty) {
                    ++nnew;
                    o = id[r];
                    v[r].y = 0u;
                }
            }
            if (o == id[r]) {
                if (!(v[r].y & bit)) atomicOr(&tab[slot[r]].y, bit);
                pend &= ~(1u << r);
            } else {
                slot[r] = (slot[r] + hash_step(id[r], kGSetLog2)) & mask;
            }
        }
    }
    return nnew;
}

// What the verification reads: rows in glist, and of group `group` the queries
// that the record answers (keep) and q0's place among them.  A group whose
// candidate sets fall apart gives one record per part; record g is group g's
// first, the others follow the groups.
struct GroupRec {
    unsigned long long rows;
    uint32_t U, keep;
    int32_t j0;
    uint32_t group;
};

__global__ __launch_bounds__(kGB, 4) void group_union_kernel(GroupedArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int32_t s_q[kGQ];
    __shared__ uint32_t s_T[kGQ], s_cnt[kGQ], s_over[kGQ], s_wc[kGW];
    __shared__ unsigned long long s_rows;
    __shared__ uint32_t s_next, s_u, s_full;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nl = A.nl;
    uint2 *tab = reinterpret_cast<uint2 *>(smem);
    uint32_t *lpref = reinterpret_cast<uint32_t *>(tab + (1u << kGSetLog2));  // [kGQ][nl + 1]
    uint32_t *lstart = reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(lpref) +
                                                    ga16(size_t(kGQ) * (nl + 1) * 4));
    GroupRec *recs = static_cast<GroupRec *>(A.recs);
    const uint32_t ng = A.groups[0];
    const int xcd = blockIdx.x % kXcd;
    auto item_of = [&](uint32_t k) -> uint32_t {  // the k-th group of this XCD
        const uint64_t it = ((uint64_t)(k / A.xchunk) * kXcd + xcd) * A.xchunk + k % A.xchunk;
        return it < ng ? (uint32_t)it : ng;
    };
    if (tid == 0) s_next = item_of(atomicAdd(A.xwork + xcd, 1u));
    __syncthreads();
    while (true) {
        const uint32_t g = s_next;
        if (g >= ng) return;  // uniform
        const uint32_t i0 = A.groups[1 + g], m = A.groups[2 + g] - i0;  // 1 <= m <= kGQ
        __syncthreads();
        if (tid == 0) s_next = item_of(atomicAdd(A.xwork + xcd, 1u));
        if (tid < kGQ) {
            s_q[tid] = tid < (int)m ? A.order[i0 + tid] : -1;
            s_cnt[tid] = 0u;
            s_over[tid] = 0u;
            s_T[tid] = 0u;
        }
        if (tid == 0) {
            s_u = 0u;
            s_full = 0u;
        }
        for (uint32_t i = 2 * tid; i < (1u << kGSetLog2); i += 2 * kGB)
            *reinterpret_cast<uint4 *>(tab + i) = uint4{kEmpty, 0u, kEmpty, 0u};
        __syncthreads();
        // each query's list prefix, one wave per query
        for (int j = wv; j < (int)m; j += kGW) {
            const int64_t q = s_q[j];
            const uint32_t st = lane < nl ? A.bstart[q * nl + lane] : 0u;
            const uint32_t sz = lane < nl ? A.bsize[q * nl + lane] : 0u;
            uint32_t v = sz;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t t = (uint32_t)__shfl_up((int)v, off);
                if (lane >= off) v += t;
            }
            if (lane < nl) {
                lpref[j * (nl + 1) + lane + 1] = v;
                lstart[j * nl + lane] = list_offset(lane, st, v - sz, A.n, A.pmagic);
            }
            if (lane == 0) lpref[j * (nl + 1)] = 0u;
            if (lane == 63) s_T[j] = v;
        }
        __syncthreads();
        // the union: rounds of kGRound * kGB positions of one query's lists,
        // the next round's ids loading while this one's are inserted
        {
            auto load = [&](int j, uint32_t base, uint32_t (&id)[kGRound]) -> uint32_t {
                const uint32_t T = s_T[j];
                const uint32_t *lp = lpref + j * (nl + 1), *ls = lstart + j * nl;
                uint32_t pos[kGRound], valid = 0;
                int lo[kGRound];
#pragma unroll
                for (int r = 0; r < kGRound; ++r) {
                    pos[r] = base + (uint32_t)(r * kGB + tid);
                    lo[r] = 0;
                }
#pragma unroll
                for (int step = 32; step > 0; step >>= 1)
                    if (step < nl)  // uniform
#pragma unroll
                        for (int r = 0; r < kGRound; ++r) {
                            const int c = lo[r] + step;
                            const uint32_t v = lp[c < nl ? c : nl];  // lp[nl] = T > pos ends the search
                            lo[r] = v <= pos[r] && c < nl ? c : lo[r];
                        }
#pragma unroll
                for (int r = 0; r < kGRound; ++r) {
                    id[r] = 0;
                    if (pos[r] < T) {
                        id[r] = (uint32_t)A.ids[ls[lo[r]] + pos[r]];
                        valid |= 1u << r;
                    }
                }
                return valid;
            };
            auto next = [&](int &j, uint32_t &base) {  // uniform: the next non-empty round
                base += kGRound * kGB;
                while (j < (int)m && base >= s_T[j]) {
                    ++j;
                    base = 0;
                }
            };
            int j = 0;
            uint32_t base = 0;
            while (j < (int)m && s_T[j] == 0u) ++j;
            uint32_t idn[kGRound], vn = 0;
            if (j < (int)m) vn = load(j, base, idn);
            uint32_t nnew = 0;
            bool full = false;
            while (j < (int)m) {
                uint32_t idc[kGRound];
#pragma unroll
                for (int r = 0; r < kGRound; ++r) idc[r] = idn[r];
                const uint32_t vc = vn, bit = 1u << j;
                next(j, base);
                if (j < (int)m) vn = load(j, base, idn);
                nnew += group_insert_ids(tab, idc, vc, bit, full);
            }
            for (int off = 32; off > 0; off >>= 1) nnew += (uint32_t)__shfl_xor((int)nnew, off);
            const bool anyfull = __ballot(full) != 0ull;
            if (lane == 0) {
                if (nnew) atomicAdd(&s_u, nnew);
                if (anyfull) s_full = 1u;
            }
        }
        __syncthreads();
        if (s_full || s_u > kGLimit) {  // uniform: beyond the set
            if (tid == 0) recs[g] = GroupRec{0ull, 0u, 0u, 0, g};
            if (tid < (int)m) A.ovf_list[atomicAdd(A.ovf_count, 1u)] = s_q[tid];
            __syncthreads();
            continue;
        }
        // |C(q_j)|: this wave's slots, by ballots
        constexpr int kPer = (1 << kGSetLog2) / kGB;  // rounds of 64 slots per wave
        uint2 v[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r) v[r] = tab[(wv * kPer + r) * 64 + lane];
        for (int j = 0; j < (int)m; ++j) {  // uniform
            uint32_t cj = 0;
#pragma unroll
            for (int r = 0; r < kPer; ++r) cj += (uint32_t)__popcll(__ballot((v[r].y >> j) & 1u));
            if (lane == 0 && cj) atomicAdd(&s_cnt[j], cj);
        }
        __syncthreads();
        uint32_t pend = (uint32_t)__ballot(lane < (int)m && s_cnt[lane < kGQ ? lane : 0] != 0u);
        if (tid < (int)m && s_cnt[tid] == 0u) {  // no candidates at all
            A.ucount[s_q[tid]] = 0u;
            A.coff[s_q[tid]] = 0ull;
        }
        bool first = true;
        while (pend) {  // uniform
            // q0: the first query left; those that share at least half of their
            // candidates with it are one record (a lesser overlap gains little,
            // and a query far from q0 has a wide error band)
            const int j0 = __ffs(pend) - 1;
            if (tid < kGQ) s_over[tid] = 0u;
            __syncthreads();
            for (int j = 0; j < (int)m; ++j) {  // uniform
                if (!((pend >> j) & 1u)) continue;
                uint32_t oj = 0;
                const uint32_t both = 1u << j | 1u << j0;
#pragma unroll
                for (int r = 0; r < kPer; ++r) oj += (uint32_t)__popcll(__ballot((v[r].y & both) == both));
                if (lane == 0 && oj) atomicAdd(&s_over[j], oj);
            }
            __syncthreads();
            const uint32_t l32 = lane < kGQ ? lane : 0;
            const bool in = lane < kGQ && ((pend >> l32) & 1u) && 2u * s_over[l32] >= s_cnt[l32];
            const uint32_t keep = (uint32_t)__ballot(in);  // the same in every wave; j0 is in it
            pend &= ~keep;
            uint32_t c = 0;
#pragma unroll
            for (int r = 0; r < kPer; ++r) c += (uint32_t)__popcll(__ballot((v[r].y & keep) != 0u));
            if (lane == 0) s_wc[wv] = c;
            __syncthreads();
            if (wv == 0) {  // rows for the record, a key range for every query; lanes are queries
                uint32_t U = 0;
                for (int w = 0; w < kGW; ++w) U += s_wc[w];
                const uint32_t cnt = in ? s_cnt[l32] : 0u;
                uint32_t x = cnt;
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t t = (uint32_t)__shfl_up((int)x, off);
                    if (lane >= off) x += t;
                }
                const uint32_t tot = (uint32_t)__shfl((int)x, 63);
                unsigned long long at = 0, off = 0;
                uint32_t slot = g;
                if (lane == 0) {
                    at = atomicAdd(A.galloc + xcd, (unsigned long long)U);
                    if (!first) slot = ng + atomicAdd(A.extra, 1u);
                }
                at = __shfl(at, 0);
                const bool room = at + U <= A.gregion;
                if (lane == 0 && room) off = atomicAdd(A.alloc + xcd, (unsigned long long)tot);
                off = __shfl(off, 0);
                const bool ok = room && off + tot <= A.region;
                if (room && !ok && lane == 0) atomicMax(A.fail + xcd, ~off);
                if (in) {
                    const int32_t q = s_q[l32];
                    if (!room) {  // beyond the list space
                        A.ovf_list[atomicAdd(A.ovf_count, 1u)] = q;
                    } else {
                        A.ucount[q] = ok ? cnt : 0u;
                        A.coff[q] = off + (unsigned long long)xcd * A.region + (x - cnt);
                        if (!ok) A.flag[q] = 1u;  // no key space: answered by the fallback
                    }
                }
                at += (unsigned long long)xcd * A.gregion;
                if (lane == 0) {
                    recs[slot] = GroupRec{at, ok ? U : 0u, keep, j0, g};
                    s_rows = ok ? at : ~0ull;
                }
            }
            __syncthreads();
            if (s_rows != ~0ull) {  // uniform
                unsigned long long at = s_rows;
                for (int w = 0; w < wv; ++w) at += s_wc[w];
                const unsigned long long lt = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
                for (int r = 0; r < kPer; ++r) {
                    const bool of = (v[r].y & keep) != 0u;
                    const unsigned long long b = __ballot(of);
                    if (of) A.glist[at + (unsigned long long)__popcll(b & lt)] = v[r];
                    at += (unsigned long long)__popcll(b);
                }
            }
            first = false;
            __syncthreads();
        }
        if (first && tid == 0) recs[g] = GroupRec{0ull, 0u, 0u, 0, g};
        __syncthreads();
    }
}

// CB: 16-query column blocks of the group (1: at most 16 queries kept within
// the first half).  Two blocks of 16 rows per wave step; the next 64 columns of
// them load while the current ones multiply.
template <int CB>
__device__ inline void verify_rows(const GroupedArgs &A, const uint2 *rows, uint32_t U, uint32_t keep,
                                   const float *qp, const float *q0s, const float *s_qn,
                                   const unsigned long long *s_base, uint32_t *s_pos)
{
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int dp = A.dp, ldq = dp + 4;
    const int nch = (dp + kGChunk - 1) / kGChunk;
    const int ntile = (int)((U + 31u) / 32u);
    const int row16 = lane & 15, kg = lane >> 4;
    if (wv >= ntile) return;
    auto entry = [&](int t, int h) -> uint2 {
        const uint32_t r = (uint32_t)(t * 32 + h * 16 + row16);
        const uint2 e = rows[r < U ? r : U - 1u];
        return uint2{e.x, r < U ? e.y & keep : 0u};  // rows past the end: nobody's
    };
    uint2 e0 = entry(wv, 0), e1 = entry(wv, 1), n0 = e0, n1 = e1;
    if (wv + kVW < ntile) {
        n0 = entry(wv + kVW, 0);
        n1 = entry(wv + kVW, 1);
    }
    const float *p0 = A.data + (int64_t)e0.x * dp + kg * 4;
    const float *p1 = A.data + (int64_t)e1.x * dp + kg * 4;
    f4 acc0[CB], acc1[CB];
    float xn0 = 0.f, xn1 = 0.f;
#pragma unroll
    for (int b = 0; b < CB; ++b) acc0[b] = acc1[b] = f4{0.f, 0.f, 0.f, 0.f};
    // the chunk at p0 / p1; columns past the row (the next row's, or the slack
    // after the last) are not used
    auto load = [&](f4 (&b)[8]) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            b[2 * s] = *reinterpret_cast<const f4 *>(p0 + s * 16);
            b[2 * s + 1] = *reinterpret_cast<const f4 *>(p1 + s * 16);
        }
        p0 += kGChunk;
        p1 += kGChunk;
    };
    auto compute = [&](const f4 (&x)[8], int c) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = c * kGChunk + s * 16;
            if (k >= dp) break;  // uniform
            f4 bq[CB];
#pragma unroll
            for (int b = 0; b < CB; ++b)
                bq[b] = *reinterpret_cast<const f4 *>(qp + (b * 16 + row16) * ldq + k + kg * 4);
            const f4 z = *reinterpret_cast<const f4 *>(q0s + k + kg * 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x0 = x[2 * s][i] - z[i], x1 = x[2 * s + 1][i] - z[i];
                xn0 = fmaf(x0, x0, xn0);
                xn1 = fmaf(x1, x1, xn1);
#pragma unroll
                for (int b = 0; b < CB; ++b) {
                    acc0[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x0, bq[b][i], acc0[b], 0, 0, 0);
                    acc1[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x1, bq[b][i], acc1[b], 0, 0, 0);
                }
            }
        }
    };
    auto finish = [&](const uint2 e, const f4 (&acc)[CB], float xn) {
        xn += __shfl_xor(xn, 16);
        xn += __shfl_xor(xn, 32);
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // row 4 kg + i, query 16 b + row16
            const int src = 4 * kg + i;
            const uint32_t id = (uint32_t)__shfl((int)e.x, src);
            const uint32_t mk = (uint32_t)__shfl((int)e.y, src);
            const float xr = __shfl(xn, src);
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const int j = b * 16 + row16;
                float F = (xr + s_qn[j]) - 2.f * acc[b][i];
                F = F < 0.f ? 0.f : F;
                if (!(F < INFINITY) || !(xr < INFINITY)) F = INFINITY;  // not a number: beyond every bound
                if ((mk >> j) & 1u) {
                    const uint32_t p = atomicAdd(&s_pos[j], 1u);
                    A.keys[s_base[j] + p] = ((unsigned long long)__float_as_uint(F) << 32) | id;
                }
            }
        }
    };
    int t = wv, c = 0;    // being computed
    int lt = wv, lc = 0;  // being loaded
    auto load_next = [&](f4 (&b)[8]) {
        if (++lc == nch) {
            lc = 0;
            lt += kVW;
            if (lt >= ntile) return;  // uniform
            p0 = A.data + (int64_t)n0.x * dp + kg * 4;
            p1 = A.data + (int64_t)n1.x * dp + kg * 4;
        }
        if (lt < ntile) load(b);
    };
    auto step = [&](f4 (&cur)[8], f4 (&nxt)[8]) {
        load_next(nxt);
        __builtin_amdgcn_sched_barrier(0);
        compute(cur, c);
        if (++c == nch) {
            finish(e0, acc0, xn0);
            finish(e1, acc1, xn1);
#pragma unroll
            for (int b = 0; b < CB; ++b) acc0[b] = acc1[b] = f4{0.f, 0.f, 0.f, 0.f};
            xn0 = xn1 = 0.f;
            c = 0;
            t += kVW;
            e0 = n0;
            e1 = n1;
            if (t + kVW < ntile) {
                n0 = entry(t + kVW, 0);
                n1 = entry(t + kVW, 1);
            }
        }
    };
    f4 ba[8], bb[8];
    load(ba);
    while (true) {
        step(ba, bb);
        if (t >= ntile) break;
        step(bb, ba);
        if (t >= ntile) break;
    }
}

__global__ __launch_bounds__(kVB, kVB / 256) void group_verify_kernel(GroupedArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int32_t s_q[kGQ];
    __shared__ uint32_t s_pos[kGQ], s_next;
    __shared__ unsigned long long s_base[kGQ];
    __shared__ float s_qn[kGQ];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dp = A.dp, ldq = dp + 4;
    float *qp = reinterpret_cast<float *>(smem);  // q' [kGQ][dp + 4]
    float *q0s = qp + (size_t)kGQ * ldq;
    const GroupRec *recs = static_cast<const GroupRec *>(A.recs);
    const uint32_t nrec = A.groups[0] + *A.extra;
    if (nrec == 0) return;
    // few records: pieces of their rows, four per workgroup of the launch
    const uint32_t np = nrec >= 4u * gridDim.x ? 1u : min(16u, (4u * gridDim.x + nrec - 1u) / nrec);
    // records are dealt to the XCDs in blocks of neighbours, which share rows
    const uint32_t blk = nrec >= gridDim.x ? gridDim.x / kXcd : 1u;
    const int xcd = blockIdx.x % kXcd;
    const uint32_t nblk = (nrec + blk - 1u) / blk;
    const uint32_t mine = nblk > (uint32_t)xcd ? (nblk - xcd + kXcd - 1u) / kXcd : 0u;  // blocks of this XCD
    const uint32_t nit = mine * blk * np;
    if (tid == 0) s_next = atomicAdd(A.xwork2 + xcd, 1u);
    __syncthreads();
    while (true) {
        const uint32_t it = s_next;
        if (it >= nit) return;  // uniform
        const uint32_t rk = it / np, pc = it - rk * np;
        const uint32_t ri = (rk / blk * kXcd + xcd) * blk + rk % blk;
        GroupRec rec = {0ull, 0u, 0u, 0, 0u};
        if (ri < nrec) rec = recs[ri];
        const uint32_t i0 = A.groups[1 + rec.group], m = A.groups[2 + rec.group] - i0;
        __syncthreads();
        if (tid == 0) s_next = atomicAdd(A.xwork2 + xcd, 1u);
        // this piece's rows, whole tiles of 32
        const uint32_t tiles = (rec.U + 31u) / 32u;
        const uint32_t r0 = min(rec.U, tiles * pc / np * 32u), r1 = min(rec.U, tiles * (pc + 1u) / np * 32u);
        const uint2 *rows = A.glist + rec.rows + r0;
        const uint32_t U = r1 - r0, keep = rec.keep;
        if (U == 0u || keep == 0u) {  // uniform
            __syncthreads();
            continue;
        }
        if (tid < kGQ) {
            s_q[tid] = tid < (int)m ? A.order[i0 + tid] : -1;
            s_pos[tid] = 0u;
        }
        __syncthreads();
        const float *q0 = A.queries + (int64_t)s_q[rec.j0] * dp;
        for (int i = tid; i < dp; i += kVB) q0s[i] = q0[i];
        const int cols = (keep >> 16) ? 32 : 16;
        for (int j = wv; j < cols; j += kVW) {
            const bool in = (keep >> j) & 1u;  // uniform
            float acc = 0.f;
            const float *qr = A.queries + (int64_t)(in ? s_q[j] : s_q[rec.j0]) * dp;
            for (int i = lane; i < dp; i += 64) {
                const float t = in ? qr[i] - q0[i] : 0.f;
                qp[j * ldq + i] = t;
                acc = fmaf(t, t, acc);
            }
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
            if (lane == 0) {
                s_qn[j] = acc;
                if (in && pc == 0u) {
                    // 8c Q^2, inflated past the rounding of |q'|^2; a query
                    // beyond FP32's range (or not a number) is left to the fallback
                    A.abs_err[s_q[j]] = acc * (16.f * (float)(dp + 16) * 0x1p-24f * 1.01f);
                    if (!(acc < 1e30f)) A.flag[s_q[j]] = 1u;
                }
            }
            if (np == 1u) {
                if (lane == 0 && in) s_base[j] = A.coff[s_q[j]];
            } else {  // this piece's share of the query's key range
                uint32_t cnt = 0;
                for (uint32_t r = lane; r < U; r += 64) cnt += (rows[r].y >> j) & 1u;
                for (int off = 32; off > 0; off >>= 1) cnt += (uint32_t)__shfl_xor((int)cnt, off);
                if (lane == 0 && in) s_base[j] = A.coff[s_q[j]] + atomicAdd(&A.kpos[s_q[j]], cnt);
            }
        }
        __syncthreads();
        if (cols == 32) verify_rows<2>(A, rows, U, keep, qp, q0s, s_qn, s_base, s_pos);
        else verify_rows<1>(A, rows, U, keep, qp, q0s, s_qn, s_base, s_pos);
        __syncthreads();  // q' is read before the next group's
    }
}

int blocks_per_cu(const void *fn, int threads, size_t lds)
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, threads, lds) != hipSuccess) {
        (void)hipGetLastError();
        nb = 1;
    }
    return std::max(nb, 1);
}

}  // namespace

float group_eps(int dp) { return 4.f * (float)(dp + 16) * 0x1p-24f * 1.01f; }

// Workspace for Q queries: a record per group, and candidate rows (kGRows per
// query; a group beyond the space goes to the per-query kernel).
constexpr int64_t kGRows = 2048;
size_t group_rec_bytes(int64_t Q) { return sizeof(GroupRec) * (size_t)Q; }
size_t group_list_bytes(int64_t Q) { return sizeof(uint2) * (size_t)std::max<int64_t>(Q * kGRows, 8 * 65536); }

// Float rows whose group of queries fits LDS; at most 64 lists per query.
bool group_applies(int dtype, int dp, int nl, size_t lds_max)
{
    return dtype == QW_F32 && nl >= 1 && nl <= 64 && verify_lds(dp) + 2048 <= lds_max &&
           union_lds(nl) + 2048 <= lds_max / 2;
}

qw_status launch_group_runs(const unsigned long long *keys, const unsigned long long *seg, int cls,
                            uint32_t *groups, hipStream_t s)
{
    group_runs_kernel<<<1, kRunBlock, 0, s>>>(keys, seg, cls, groups);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

qw_status launch_small_order(unsigned long long *keys, int32_t *vals, int64_t Q,
                             const unsigned long long *class_count, int32_t ncls, unsigned long long *seg,
                             int cls, uint32_t *groups, hipStream_t s)
{
    if (Q < 1 || Q > kSmallOrder) return QW_EINTERNAL;
    small_order_kernel<<<1, kRunBlock, 0, s>>>(keys, vals, (int32_t)Q, class_count, ncls, seg, cls, groups);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

qw_status launch_grouped(GroupedArgs a, int cus, size_t lds_max, hipStream_t s)
{
    if (!group_applies(QW_F32, a.dp, a.nl, lds_max) || a.dp % 16 != 0) return QW_EINTERNAL;
    a.xchunk = std::max(1u, a.xchunk / kGQ);  // in groups
    const size_t ul = union_lds(a.nl), vl = verify_lds(a.dp);
    group_union_kernel<<<blocks_per_cu((const void *)group_union_kernel, kGB, ul) * cus, kGB, ul, s>>>(a);
    QW_HIP(hipGetLastError());
    group_verify_kernel<<<blocks_per_cu((const void *)group_verify_kernel, kVB, vl) * cus, kVB, vl, s>>>(a);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

}  // namespace qw
