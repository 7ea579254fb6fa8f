// Candidate work of several queries per workgroup: queries whose candidate sets
// overlap (neighbours of the grouped order with the same label) form their
// union together and verify every row of it once, on the matrix cores -- the
// bucket's points are staged once and reused by the queries that hit it
// (Sections 4 and 5.1).
//
// group_gain_kernel (uint8 rows) keeps the groups whose queries list the same
// buckets often enough.
//
// group_union_kernel, one workgroup per group of at most 32 queries: the queries'
// buckets, each once with a mask of the queries that list it, then their ids into
// one LDS set whose slots hold the mask of the queries that list the id; the set
// is compacted into (id, mask) rows and a key range is taken for every query's
// candidates.  A set beyond its capacity sends the group's queries to the
// per-query kernel; queries that share little with the group's others are split
// off.
//
// group_verify_kernel, one workgroup per group, or per piece of a group's rows
// where there are few groups, 16 x 16 blocks of rows x queries: distances by
// v_mfma_i32_16x16x64_i8 (uint8 rows: exact, x - 128 and q - 128 are signed
// bytes), or v_mfma_f32_16x16x4f32 over x' = x - q0 and q' = q - q0 (q0: one
// query of the group), F = |x'|^2 + |q'|^2 - 2 x'.q'.  Each (row, query) pair of
// the mask that may be among the query's K nearest writes its (F, id) key for the
// select kernel.
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
// verification by the rows' bytes, read once per group: 100,000 clustered
// queries of 960 columns read 35 GB at 4.7 TB/s while the matrix cores are busy
// for half of the time (groups of more queries do not fit LDS; the same region's
// groups run on one XCD, but seldom close enough in time to share its 4 MB L2:
// 17 % of their requests hit).
// Measured (1M x 960, w = 12): 100,000 clustered queries took 63 ms query by
// query; the unions now take 0.75 ms (2.25 when every query inserted its ids by
// itself), the verification 7.4, the select kernel 1.7 (2.3 when all candidates
// wrote keys); 1,000 scattered queries 2.3 ms before, 0.08, 0.75 and 0.03 now.
// uint8 (10M x 96, 100,000 skewed queries): 2.9 ms query by query, now the unions
// 0.34, the verification 0.37 (bound by the work on its outputs), the select
// kernel 0.24 and the queries given back 0.34.
#include <algorithm>
#include <type_traits>

#include "qw_dedup.h"
#include "qw_internal.h"
#include "qw_band.h"

namespace qw {
namespace {

constexpr int kGB = 512;                                // threads per workgroup
constexpr int kGW = kGB / 64;                           // waves
// of the verification (float rows: the queries fill LDS, one workgroup per CU;
// uint8: 256 threads took 0.67 ms where 512 take 0.46 and 1024 0.48)
template <int DT> constexpr int kVB = DT == QW_F32 ? 768 : 512;
template <int DT> constexpr int kVW = kVB<DT> / 64;
// minima per query: wave, quarter of its lanes, 16-row block
template <int DT> constexpr int kVCells = kVW<DT> * 8;
template <int DT> constexpr int kGFilterK = kVCells<DT> / 2;  // K up to which they bound the K-th key
constexpr int kGQ = kGroupMax;                          // queries per group
constexpr int kGSetLog2 = 13;                           // set slots
constexpr uint32_t kGLimit = (1u << kGSetLog2) / 4 * 3;  // rows of a group at most (load <= 3/4)
constexpr int kGRound = 4;                              // listed ids per thread per round

typedef float f4 __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));

// 16 bytes of a uint8 row less 128 each: distances stay, the products are those
// of signed bytes
__device__ inline v4i signed_part(v4i v)
{
    constexpr int flip = (int)0x80808080u;
    return v4i{v.x ^ flip, v.y ^ flip, v.z ^ flip, v.w ^ flip};
}

__device__ inline int norm_part(v4i v)
{
    int s = __builtin_amdgcn_sdot4(v.x, v.x, 0, false);
    s = __builtin_amdgcn_sdot4(v.y, v.y, s, false);
    s = __builtin_amdgcn_sdot4(v.z, v.z, s, false);
    return __builtin_amdgcn_sdot4(v.w, v.w, s, false);
}

__host__ __device__ inline size_t ga16(size_t v) { return (v + 15) & ~size_t(15); }

constexpr int kGMapLog2 = 12;                           // slots of the bucket map
constexpr uint32_t kGPart = 512;                        // ids of a bucket part at most
constexpr uint32_t kGParts = 1536;                      // bucket parts of a group at most

// set slots {id, mask} (before it is filled: the bucket map) | parts {offset, mask} | their sizes
constexpr size_t kUnionLds = (size_t(8) << kGSetLog2) + size_t(kGParts) * 10;
static_assert((size_t(12) << kGMapLog2) <= (size_t(8) << kGSetLog2), "the bucket map lies in the set");
static_assert(64 * kGQ <= 1 << (kGMapLog2 - 1), "the bucket map never fills");
// Adds bits[r] to the masks of the valid ids, inserting those not yet in the
// set; returns how many were new, sets `full` when one found no slot.  Most ids
// are there already (a candidate recurs across layers), so a slot is read
// before anything is written.
__device__ inline uint32_t group_insert_ids(uint2 *tab, const uint32_t (&id)[kGRound], uint32_t valid,
                                            const uint32_t (&bits)[kGRound], bool &full)
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
                if ((v[r].y & bits[r]) != bits[r]) atomicOr(&tab[slot[r]].y, bits[r]);
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

// Whole wave, a query per lane (q < 0: none): these queries are answered one by
// one, from a queue or their classes' segments.  Queries of one class go there
// together, so they stay neighbours.
__device__ inline void group_give_back(const GroupedArgs &A, int32_t q)
{
    const int lane = threadIdx.x & 63;
    if (q >= 0 && A.ovf_flag) A.flag[q] = A.ovf_flag;
    const int c = q < 0 ? -1 : A.seg ? A.cls[q] : 0;
    for (unsigned long long left = __ballot(c >= 0); left;) {
        const int k = __shfl(c, __ffsll((long long)left) - 1);
        const unsigned long long same = __ballot(c == k);
        const int lead = __ffsll((long long)same) - 1;
        unsigned long long at = 0;
        if (lane == lead)
            at = A.seg ? atomicAdd(&A.seg[2 * k + 1], (unsigned long long)__popcll(same))
                       : atomicAdd(A.ovf_count, (uint32_t)__popcll(same));
        at = __shfl(at, lead);
        if (c == k) A.ovf_list[at + (unsigned long long)__popcll(same & (lane ? ~0ull >> (64 - lane) : 0ull))] = q;
        left &= ~same;
    }
}

// Which groups share a workgroup: over kGainLists of the lists, the ids that the
// queries list (enough per query, too) against the ids of the distinct buckets.
// One wave per group, two lists of its queries at a time.  Marks the group and
// counts its queries.
constexpr int kGainLists = 8, kGainBlock = 1024, kGainGroups = kGainBlock / 64;
constexpr uint32_t kGainMark = 0x80000000u;
__global__ __launch_bounds__(kGainBlock) void group_gain_kernel(GroupedArgs A)
{
    __shared__ uint32_t s_queries;
    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, half = lane & 32;
    const uint32_t ng = A.gcount[0], g = blockIdx.x * kGainGroups + (tid >> 6);
    if (blockIdx.x * kGainGroups >= ng) return;  // uniform
    if (tid == 0) s_queries = 0u;
    __syncthreads();
    const uint2 gr = g < ng ? A.groups[g] : uint2{0u, 0u};
    const int32_t q = (uint32_t)j < gr.y ? A.order[gr.x + j] : -1;
    uint32_t st[kGainLists / 2], sz[kGainLists / 2];
#pragma unroll
    for (int i = 0; i < kGainLists / 2; ++i) {
        const int r = 2 * i + (half ? 1 : 0);
        const int l = A.nl <= kGainLists ? r : r * A.nl / kGainLists;
        const bool in = q >= 0 && l < A.nl;
        st[i] = in ? A.bstart[(int64_t)q * A.nl + l] : 0u;
        sz[i] = in ? min(A.bsize[(int64_t)q * A.nl + l], 1u << 16) : 0u;
        if (sz[i] == 0u) st[i] = 0xFFFFFFFFu;  // no bucket starts there
    }
    uint32_t listed = 0, once = 0;
#pragma unroll
    for (int i = 0; i < kGainLists / 2; ++i) {
        bool first = true;
#pragma unroll
        for (int k = 0; k < 31; ++k) {
            const uint32_t os = (uint32_t)__shfl((int)st[i], half | k);
            first = first && !(k < j && os == st[i]);
        }
        listed += sz[i];
        once += first ? sz[i] : 0u;
    }
    for (int off = 32; off > 0; off >>= 1) {
        listed += (uint32_t)__shfl_xor((int)listed, off);
        once += (uint32_t)__shfl_xor((int)once, off);
    }
    // uniform in the wave; listed <= 2^24
    const uint64_t all = (uint64_t)listed * (uint32_t)A.nl / (uint32_t)min(A.nl, kGainLists);
    if (g < ng && listed >= A.gain * once && all >= (uint64_t)A.gain_listed * gr.y && lane == 0) {
        A.groups[g].y = gr.y | kGainMark;
        atomicAdd(&s_queries, gr.y);
    }
    __syncthreads();
    if (tid == 0 && s_queries) atomicAdd(A.gcount + kGroupCounts + 2, s_queries);
}

// The marked groups become groups2, their queries qlist2 -- unless they are few:
// the two kernels take about 60 us for any number of them.  The other groups'
// queries are given back.  What a workgroup's groups take of a counter they take
// together: thousands of atomics on one address take 20 ns each (50,000 queries,
// 1,600 groups given back: 65 us group by group, 10 so).
__global__ __launch_bounds__(kGainBlock) void group_split_kernel(GroupedArgs A)
{
    __shared__ uint32_t s_cls[32], s_groups, s_queries;
    __shared__ unsigned long long s_base[32];
    constexpr int per = kGainBlock / 32;
    const int tid = threadIdx.x, j = tid & 31;
    const uint32_t ng = A.gcount[0], g = blockIdx.x * per + (tid >> 5);
    if (blockIdx.x * per >= ng) return;  // uniform
    if (tid < 32) s_cls[tid] = 0u;
    if (tid == 0) s_groups = s_queries = 0u;
    __syncthreads();
    uint2 gr = g < ng ? A.groups[g] : uint2{0u, 0u};
    const bool share = (gr.y & kGainMark) && (uint64_t)A.gcount[kGroupCounts + 2] * 16u >= (uint64_t)A.Q * A.gain_part;
    gr.y &= ~kGainMark;
    const int32_t q = (uint32_t)j < gr.y ? A.order[gr.x + j] : -1;
    const int c = q >= 0 ? A.cls[q] : 0;
    const bool rest = !share && q >= 0;
    uint32_t at = 0, qat = 0;
    if (rest) {
        at = atomicAdd(&s_cls[c], 1u);
        if (A.ovf_flag) A.flag[q] = A.ovf_flag;
    } else if (share && j == 0) {
        at = atomicAdd(&s_groups, 1u);
        qat = atomicAdd(&s_queries, gr.y);
    }
    __syncthreads();
    if (tid < 32 && s_cls[tid]) s_base[tid] = atomicAdd(&A.seg[2 * tid + 1], (unsigned long long)s_cls[tid]);
    if (tid == 32 && s_groups) s_groups = atomicAdd(A.gcount + kGroupCounts, s_groups);
    if (tid == 33 && s_queries) s_queries = atomicAdd(A.gcount + kGroupCounts + 1, s_queries);
    __syncthreads();
    if (rest) A.ovf_list[s_base[c] + at] = q;
    qat = (uint32_t)__shfl((int)qat, tid & 32);
    if (share) {
        if (j == 0) A.groups2[s_groups + at] = gr;
        if (q >= 0) A.qlist2[s_queries + qat + j] = q;
    }
}

__global__ __launch_bounds__(kGB, 4) void group_union_kernel(GroupedArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int32_t s_q[kGQ];
    __shared__ uint32_t s_cnt[kGQ], s_over[kGQ], s_wc[kGW];
    __shared__ unsigned long long s_rows;
    __shared__ uint32_t s_next, s_u, s_full, s_nb, s_grab;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nl = A.nl;
    uint2 *tab = reinterpret_cast<uint2 *>(smem);
    uint2 *part = tab + (1u << kGSetLog2);
    uint16_t *psize = reinterpret_cast<uint16_t *>(part + kGParts);
    constexpr uint32_t nmap = 1u << kGMapLog2;
    uint32_t *mkey = reinterpret_cast<uint32_t *>(smem), *mmask = mkey + nmap, *msize = mmask + nmap;
    GroupRec *recs = static_cast<GroupRec *>(A.recs);
    const uint32_t ng = *A.gcount;
    if (ng == 0) return;
    const int xcd = blockIdx.x % kXcd;
    auto overflow = [&](int32_t q) { group_give_back(A, q); };  // wave 0
    auto item_of = [&](uint32_t k) -> uint32_t {  // the k-th group of this XCD
        const uint64_t it = ((uint64_t)(k / A.xchunk) * kXcd + xcd) * A.xchunk + k % A.xchunk;
        return it < ng ? (uint32_t)it : ng;
    };
    if (tid == 0) s_next = item_of(atomicAdd(A.xwork + xcd, 1u));
    __syncthreads();
    while (true) {
        const uint32_t g = s_next;
        if (g >= ng) return;  // uniform
        const uint32_t i0 = A.groups[g].x, m = A.groups[g].y;  // 1 <= m <= kGQ
        __syncthreads();
        if (tid == 0) s_next = item_of(atomicAdd(A.xwork + xcd, 1u));
        if (tid < kGQ) {
            s_q[tid] = tid < (int)m ? A.order[i0 + tid] : -1;
            s_cnt[tid] = 0u;
        }
        if (tid == 0) {
            s_u = 0u;
            s_full = 0u;
            s_nb = 0u;
            s_grab = 0u;
        }
        for (uint32_t i = tid; i < nmap; i += kGB) {
            mkey[i] = kEmpty;
            mmask[i] = 0u;
        }
        __syncthreads();
        // the queries' buckets, each once, with a mask of the queries that list
        // it (neighbours share most of them)
        for (int i = tid; i < (int)m * nl; i += kGB) {
            const int j = i / nl, l = i - j * nl;
            const int64_t e = (int64_t)s_q[j] * nl + l;
            const uint32_t sz = A.bsize[e];
            if (sz == 0u) continue;
            const uint32_t off = list_offset(l, A.bstart[e], 0u, A.n, A.pmagic);
            uint32_t sl = hash_id(off, kGMapLog2);
            while (true) {  // ends: at most half of the slots are ever taken
                uint32_t o = mkey[sl];
                if (o == kEmpty) o = atomicCAS(&mkey[sl], kEmpty, off);
                if (o == kEmpty || o == off) break;
                sl = (sl + 1u) & (nmap - 1u);
            }
            msize[sl] = sz;  // every writer stores the bucket's size
            atomicOr(&mmask[sl], 1u << j);
        }
        __syncthreads();
        // their list, the larger ones in parts
        for (uint32_t i = tid; i < nmap; i += kGB) {
            const uint32_t off = mkey[i];
            if (off == kEmpty) continue;
            const uint32_t sz = msize[i], mk = mmask[i];
            if (sz > kGLimit) {
                s_full = 1u;
                continue;
            }
            const uint32_t np = (sz + kGPart - 1u) / kGPart;
            const uint32_t at = atomicAdd(&s_nb, np);
            for (uint32_t p = 0; p < np && at + p < kGParts; ++p) {
                part[at + p] = uint2{off + p * kGPart, mk};
                psize[at + p] = (uint16_t)min(kGPart, sz - p * kGPart);
            }
        }
        __syncthreads();
        const uint32_t nb = s_nb;
        const bool many = nb > kGParts || s_full;  // uniform
        if (many) {
            if (tid == 0) recs[g] = GroupRec{0ull, 0u, 0u, 0, g};
            if (wv == 0) overflow(lane < (int)m ? s_q[lane] : -1);
            __syncthreads();
            continue;
        }
        for (uint32_t i = 2 * tid; i < (1u << kGSetLog2); i += 2 * kGB)
            *reinterpret_cast<uint4 *>(tab + i) = uint4{kEmpty, 0u, kEmpty, 0u};
        __syncthreads();
        // the union: each half of a wave takes part after part, 32 ids at a
        // time, the next round's ids loading while this one's are inserted
        {
            const uint32_t hl = lane & 31;
            uint32_t off = 0, mk = 0, rem = 0;  // the half's part: its next id, mask, ids left
            bool more = true;
            auto load = [&](uint32_t (&id)[kGRound], uint32_t (&bits)[kGRound]) -> uint32_t {
                uint32_t valid = 0;
#pragma unroll
                for (int r = 0; r < kGRound; ++r) {
                    if (rem == 0u && more) {  // uniform in the half
                        uint32_t e = 0;
                        if (hl == 0) e = atomicAdd(&s_grab, 1u);
                        e = (uint32_t)__shfl((int)e, lane & 32);
                        more = e < nb;
                        if (more) {
                            const uint2 b = part[e];
                            off = b.x;
                            mk = b.y;
                            rem = psize[e];
                        }
                    }
                    id[r] = 0;
                    bits[r] = mk;
                    if (hl < rem) {
                        id[r] = (uint32_t)A.ids[off + hl];
                        valid |= 1u << r;
                    }
                    off += 32u;
                    rem -= min(rem, 32u);
                }
                return valid;
            };
            uint32_t idn[kGRound], bn[kGRound];
            uint32_t vn = load(idn, bn);
            uint32_t nnew = 0;
            bool full = false;
            while (__ballot(vn != 0u)) {  // a half without ids stays so
                uint32_t idc[kGRound], bc[kGRound];
#pragma unroll
                for (int r = 0; r < kGRound; ++r) {
                    idc[r] = idn[r];
                    bc[r] = bn[r];
                }
                const uint32_t vc = vn;
                vn = load(idn, bn);
                nnew += group_insert_ids(tab, idc, vc, bc, full);
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
            if (wv == 0) overflow(lane < (int)m ? s_q[lane] : -1);
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
                const uint32_t cnt = in ? min(s_cnt[l32], A.keep) : 0u;
                uint32_t x = cnt;
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t t = (uint32_t)__shfl_up((int)x, off);
                    if (lane >= off) x += t;
                }
                const uint32_t tot = (uint32_t)__shfl((int)x, 63);
                unsigned long long at = 0, off = 0;
                if (lane == 0) at = atomicAdd(A.galloc + xcd, (unsigned long long)U);
                at = __shfl(at, 0);
                const bool room = at + U <= A.gregion;
                if (lane == 0 && room) off = atomicAdd(A.alloc + xcd, (unsigned long long)tot);
                off = __shfl(off, 0);
                const bool ok = room && off + tot <= A.region;
                if (room && !ok && lane == 0) atomicMax(A.fail + xcd, ~off);
                if (in) {
                    const int32_t q = s_q[l32];
                    if (room) {
                        A.ucount[q] = ok ? s_cnt[l32] : 0u;
                        A.kroom[q] = cnt;
                        A.coff[q] = off + (unsigned long long)xcd * A.region + (x - cnt);
                        if (!ok) A.flag[q] = 1u;  // no key space: answered by the fallback
                    }
                }
                if (!room) overflow(in ? s_q[l32] : -1);  // beyond the list space
                at += (unsigned long long)xcd * A.gregion;
                if (lane == 0) {
                    recs[first ? g : ng + atomicAdd(A.extra, 1u)] = GroupRec{at, ok ? U : 0u, keep, j0, g};
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
            __syncthreads();
            first = false;
        }
        if (first && tid == 0) recs[g] = GroupRec{0ull, 0u, 0u, 0, g};
        __syncthreads();
    }
}

// A key's distance as the bits of a float, or of an integer (uint8 rows): both
// order as unsigned words.
constexpr uint32_t kNoKey = 0xFFFFFFFFu;

// What a workgroup of the verification holds of its record.
struct VerifyGroup {
    const uint2 *rows;
    uint32_t U, keep;
    const unsigned char *qp;   // q' [kGQ][ldq bytes]
    const float *q0s;          // q0 (float rows)
    const uint32_t *qn;        // |q'|^2 per query
    uint32_t *minima;          // [kGQ][kVCells<DT>]
    uint32_t *thr;             // per query: keys beyond it are not needed
    const float *err;          // absolute part of the keys' error (float rows)
    const unsigned long long *base;
    const uint32_t *room;
    uint32_t *pos;             // keys written by this workgroup
    const int32_t *q;
    bool pieces;
    int64_t row0, stride;      // brute force: the rows' ids instead of `rows`
    int64_t at0;               // brute force without a bound: row r's key goes to place at0 + r (else -1)
};
// Bytes of a row per step (a 16-byte part per quarter of the lanes), and steps
// whose loads are in flight together.
constexpr int kStepBytes = 64;
template <int DT> constexpr int verify_steps() { return DT == QW_F32 ? 4 : 2; }
template <int DT> __host__ __device__ inline int verify_ldq(int dp)
{
    // the 16 bytes more spread a column of rows over the banks
    return (dp * (DT == QW_F32 ? 4 : 1) + kStepBytes - 1) / kStepBytes * kStepBytes + 16;
}

// CB: 16-query column blocks of the group (1: at most 16 queries kept within
// the first half).  Two blocks of 16 rows per wave step; the next NS steps'
// bytes of them load while the current ones multiply.
//
// Few of a query's rows are among its K nearest, so few keys are written: after
// the waves' first tiles (32 rows each, in the order of the ids' hash) the K-th
// smallest of a query's minima over disjoint parts of them bounds its K-th
// key; rows beyond that bound (float rows: beyond its error band) give no key.
// DENSE (brute force): row r is point row0 + r * stride, everybody's, and the bound
// is given.
template <int DT, int CB, bool DENSE>
__device__ inline void verify_rows(const GroupedArgs &A, const VerifyGroup &G)
{
    constexpr int NS = verify_steps<DT>();
    using acc_t = typename std::conditional<DT == QW_F32, f4, v4i>::type;
    using sum_t = typename std::conditional<DT == QW_F32, float, int>::type;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int dp = A.dp, ldq = verify_ldq<DT>(dp);
    const int64_t rb = (int64_t)dp * (DT == QW_F32 ? 4 : 1);
    const int nst = ((int)rb + kStepBytes - 1) / kStepBytes;
    const int nch = (nst + NS - 1) / NS;
    const uint32_t U = G.U;
    const int ntile = (int)((U + 31u) / 32u);
    const int row16 = lane & 15, kg = lane >> 4;
    const unsigned char *data = static_cast<const unsigned char *>(A.data);
    // the K-th smallest of each query's minima: its bits from the top, each
    // kept where fewer than K minima lie below
    auto bounds = [&]() {
        __syncthreads();
        for (int j = wv; j < 16 * CB; j += kVW<DT>) {  // uniform
            const uint32_t *c = G.minima + j * kVCells<DT>;
            const uint32_t v0 = lane < kVCells<DT> ? c[lane] : kNoKey, v1 = lane + 64 < kVCells<DT> ? c[lane + 64] : kNoKey;
            uint32_t t = 0;
            for (int b = 31; b >= 0; --b) {
                const uint32_t x = t | 1u << b;
                const int below = __popcll(__ballot(v0 < x)) + __popcll(__ballot(v1 < x));
                if (below < A.K) t = x;
            }
            if (DT == QW_F32 && t != kNoKey)
                t = __float_as_uint(band_threshold(__uint_as_float(t), A.eps, G.err[j]));
            if (lane == 0) G.thr[j] = t;
        }
        __syncthreads();
    };
    static_assert(kVCells<DT> <= 128, "two minima per lane");
    if (wv >= ntile) {  // no tile: its minima are empty
        if (!DENSE && A.K <= kGFilterK<DT>) {
            for (int i = lane; i < 16 * CB * 8; i += 64) G.minima[(i >> 3) * kVCells<DT> + wv * 8 + (i & 7)] = kNoKey;
            bounds();
        }
        return;
    }
    auto entry = [&](int t, int h) -> uint2 {
        const uint32_t r = (uint32_t)(t * 32 + h * 16 + row16);
        // rows past the end: nobody's
        if (DENSE) return uint2{(uint32_t)(G.row0 + (int64_t)(r < U ? r : U - 1u) * G.stride), r < U ? G.keep : 0u};
        const uint2 e = G.rows[r < U ? r : U - 1u];
        return uint2{e.x, r < U ? e.y & G.keep : 0u};
    };
    uint2 e0 = entry(wv, 0), e1 = entry(wv, 1), n0 = e0, n1 = e1;
    if (wv + kVW<DT> < ntile) {
        n0 = entry(wv + kVW<DT>, 0);
        n1 = entry(wv + kVW<DT>, 1);
    }
    const unsigned char *p0 = data + (int64_t)e0.x * rb + kg * 16;
    const unsigned char *p1 = data + (int64_t)e1.x * rb + kg * 16;
    acc_t acc0[CB], acc1[CB];
    sum_t xn0 = 0, xn1 = 0;
#pragma unroll
    for (int b = 0; b < CB; ++b) acc0[b] = acc1[b] = acc_t{0, 0, 0, 0};
    // the chunk at p0 / p1; bytes past the row (the next row's, or the slack
    // after the last) are not used
    auto load = [&](acc_t (&b)[2 * NS]) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            b[2 * s] = *reinterpret_cast<const acc_t *>(p0 + s * kStepBytes);
            b[2 * s + 1] = *reinterpret_cast<const acc_t *>(p1 + s * kStepBytes);
        }
        p0 += NS * kStepBytes;
        p1 += NS * kStepBytes;
    };
    auto compute = [&](const acc_t (&x)[2 * NS], int c) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int st = c * NS + s;
            if (st >= nst) break;  // uniform
            acc_t bq[CB];
#pragma unroll
            for (int b = 0; b < CB; ++b)
                bq[b] = *reinterpret_cast<const acc_t *>(G.qp + (b * 16 + row16) * ldq + st * kStepBytes + kg * 16);
            if constexpr (DT == QW_F32) {
                const f4 z = *reinterpret_cast<const f4 *>(G.q0s + st * 16 + kg * 4);
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
            } else {
                const bool in = st * kStepBytes + kg * 16 < (int)rb;  // else q' is zero there
                const v4i x0 = signed_part(x[2 * s]), x1 = signed_part(x[2 * s + 1]);
                xn0 += in ? norm_part(x0) : 0;
                xn1 += in ? norm_part(x1) : 0;
#pragma unroll
                for (int b = 0; b < CB; ++b) {
                    acc0[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, bq[b], acc0[b], 0, 0, 0);
                    acc1[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, bq[b], acc1[b], 0, 0, 0);
                }
            }
        }
    };
    // the keys of a tile's pairs, kNoKey where the query does not list the row
    // (row 4 kg + i of block h, query 16 b + row16)
    uint32_t key[2][CB][4];
    auto tile_keys = [&](const uint2 e, const acc_t (&acc)[CB], sum_t xn, uint32_t (&k)[CB][4]) {
        xn += __shfl_xor(xn, 16);
        xn += __shfl_xor(xn, 32);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int src = 4 * kg + i;
            const uint32_t mk = (uint32_t)__shfl((int)e.y, src);
            const sum_t xr = __shfl(xn, src);
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const int j = b * 16 + row16;
                uint32_t w;
                if constexpr (DT == QW_F32) {
                    float F = (xr + __uint_as_float(G.qn[j])) - 2.f * acc[b][i];
                    F = F < 0.f ? 0.f : F;
                    if (!(F < INFINITY) || !(xr < INFINITY)) F = INFINITY;  // not a number: beyond every bound
                    w = __float_as_uint(F);
                } else {
                    w = (uint32_t)(xr + (int)G.qn[j] - 2 * acc[b][i]);
                }
                k[b][i] = (mk >> j) & 1u ? w : kNoKey;
            }
        }
    };
    // each query's keys of tile t within its bound: lanes of one row16 share
    // a query, one of them takes the room for all
    auto emit = [&](int t) {
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            const int j = b * 16 + row16;
            if (DENSE && G.at0 >= 0) {  // uniform: every key, by its row
                unsigned long long *out = A.keys + G.base[j] + G.at0;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t id = (uint32_t)__shfl((int)(h ? e1.x : e0.x), 4 * kg + i);
                        if (key[h][b][i] != kNoKey)
                            out[t * 32 + h * 16 + 4 * kg + i] = ((unsigned long long)key[h][b][i] << 32) | id;
                    }
                continue;
            }
            const uint32_t thr = G.thr[j];
            uint32_t c = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) c += key[h][b][i] <= thr && key[h][b][i] != kNoKey ? 1u : 0u;
            if (!__ballot(c != 0u)) continue;  // uniform
            const uint32_t c1 = (uint32_t)__shfl_xor((int)c, 16);
            const uint32_t s1 = c + c1, s2 = (uint32_t)__shfl_xor((int)s1, 32);
            uint32_t at = 0;
            if (kg == 0 && s1 + s2) at = G.pieces ? atomicAdd(&A.kpos[G.q[j]], s1 + s2) : atomicAdd(&G.pos[j], s1 + s2);
            at = (uint32_t)__shfl((int)at, row16) + (kg & 1 ? c1 : 0u) + (kg & 2 ? s2 : 0u);
            const uint32_t room = G.room[j];
            unsigned long long *out = A.keys + G.base[j];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t id = (uint32_t)__shfl((int)(h ? e1.x : e0.x), 4 * kg + i);
                    const uint32_t k = key[h][b][i];
                    if (k <= thr && k != kNoKey) {
                        if (at < room) out[at] = ((unsigned long long)k << 32) | id;
                        ++at;
                    }
                }
        }
    };
    int t = wv, c = 0;    // being computed
    int lt = wv, lc = 0;  // being loaded
    auto load_next = [&](acc_t (&b)[2 * NS]) {
        if (++lc == nch) {
            lc = 0;
            lt += kVW<DT>;
            if (lt >= ntile) return;  // uniform
            p0 = data + (int64_t)n0.x * rb + kg * 16;
            p1 = data + (int64_t)n1.x * rb + kg * 16;
        }
        if (lt < ntile) load(b);
    };
    auto step = [&](acc_t (&cur)[2 * NS], acc_t (&nxt)[2 * NS]) {
        load_next(nxt);
        __builtin_amdgcn_sched_barrier(0);
        compute(cur, c);
        if (++c == nch) {
            tile_keys(e0, acc0, xn0, key[0]);
            tile_keys(e1, acc1, xn1, key[1]);
            if (!DENSE && t == wv && A.K <= kGFilterK<DT>) {  // uniform in the workgroup: every wave's first tile
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        G.minima[(b * 16 + row16) * kVCells<DT> + wv * 8 + kg * 2 + h] =
                            min(min(key[h][b][0], key[h][b][1]), min(key[h][b][2], key[h][b][3]));
                bounds();
            }
            emit(t);
#pragma unroll
            for (int b = 0; b < CB; ++b) acc0[b] = acc1[b] = acc_t{0, 0, 0, 0};
            xn0 = xn1 = 0;
            c = 0;
            t += kVW<DT>;
            e0 = n0;
            e1 = n1;
            if (t + kVW<DT> < ntile) {
                n0 = entry(t + kVW<DT>, 0);
                n1 = entry(t + kVW<DT>, 1);
            }
        }
    };
    acc_t ba[2 * NS], bb[2 * NS];
    load(ba);
    while (true) {
        step(ba, bb);
        if (t >= ntile) break;
        step(bb, ba);
        if (t >= ntile) break;
    }
}

// q' of the group's queries (zeros in the columns of others) and |q'|^2; float
// rows: q0 and the keys' error, once (`first`) for the select kernel too.
// DENSE: the flag has no other writer.
template <int DT, bool DENSE>
__device__ inline void stage_queries(const GroupedArgs &A, const int32_t *s_q, uint32_t keep, int j0, bool first,
                                     unsigned char *qp, float *q0s, uint32_t *s_qn, float *s_err)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dp = A.dp, ldq = verify_ldq<DT>(dp), cols = (keep >> 16) ? 32 : 16;
    const unsigned char *queries = static_cast<const unsigned char *>(A.queries);
    const int64_t rb = (int64_t)dp * (DT == QW_F32 ? 4 : 1);
    const float *q0 = reinterpret_cast<const float *>(queries + (int64_t)s_q[j0] * rb);
    if constexpr (DT == QW_F32)
        for (int i = tid; i < dp; i += kVB<DT>) q0s[i] = q0[i];
    for (int j = wv; j < cols; j += kVW<DT>) {
        const bool in = (keep >> j) & 1u;  // uniform
        const int32_t q = in ? s_q[j] : s_q[j0];
        if constexpr (DT == QW_F32) {
            const float *qr = reinterpret_cast<const float *>(queries + (int64_t)q * rb);
            float *qo = reinterpret_cast<float *>(qp + (size_t)j * ldq);
            float acc = 0.f;
            for (int i = lane; i < dp; i += 64) {
                const float t = in ? qr[i] - q0[i] : 0.f;
                qo[i] = t;
                acc = fmaf(t, t, acc);
            }
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
            // 8c Q^2, inflated past the rounding of |q'|^2; a query beyond
            // FP32's range (or not a number) is left to the fallback
            const float err = acc * (16.f * (float)(dp + 16) * 0x1p-24f * 1.01f);
            if (lane == 0) {
                s_qn[j] = __float_as_uint(acc);
                s_err[j] = err;
                if (in && first) {
                    A.abs_err[q] = err;
                    if (DENSE) A.flag[q] = acc < 1e30f ? 0u : 1u;
                    else if (!(acc < 1e30f)) A.flag[q] = 1u;
                }
            }
        } else {
            const v4i *qr = reinterpret_cast<const v4i *>(queries + (int64_t)q * rb);
            v4i *qo = reinterpret_cast<v4i *>(qp + (size_t)j * ldq);
            int acc = 0;
            for (int i = lane; i < (ldq - 16) / 16; i += 64) {
                const v4i t = in && i < dp / 16 ? signed_part(qr[i]) : v4i{0, 0, 0, 0};
                qo[i] = t;
                acc += norm_part(t);
            }
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
            if (lane == 0) s_qn[j] = (uint32_t)acc;
        }
    }
}

template <int DT>
__global__ __launch_bounds__(kVB<DT>, DT == QW_F32 ? 3 : 4) void group_verify_kernel(GroupedArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int32_t s_q[kGQ];
    __shared__ uint32_t s_pos[kGQ], s_room[kGQ], s_thr[kGQ], s_qn[kGQ], s_next;
    __shared__ unsigned long long s_base[kGQ];
    __shared__ float s_err[kGQ];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dp = A.dp, ldq = verify_ldq<DT>(dp);
    uint32_t *minima = reinterpret_cast<uint32_t *>(smem);
    unsigned char *qp = smem + sizeof(uint32_t) * kGQ * kVCells<DT>;  // q' [kGQ][ldq]
    float *q0s = reinterpret_cast<float *>(qp + (size_t)kGQ * ldq);
    const GroupRec *recs = static_cast<const GroupRec *>(A.recs);
    const uint32_t nrec = *A.gcount + *A.extra;
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
        const uint32_t i0 = A.groups[rec.group].x, m = A.groups[rec.group].y;
        __syncthreads();
        if (tid == 0) s_next = atomicAdd(A.xwork2 + xcd, 1u);
        // this piece's rows, whole tiles of 32
        const uint32_t tiles = (rec.U + 31u) / 32u;
        const uint32_t r0 = min(rec.U, tiles * pc / np * 32u), r1 = min(rec.U, tiles * (pc + 1u) / np * 32u);
        const uint32_t keep = rec.keep;
        if (r1 == r0 || keep == 0u) {  // uniform
            __syncthreads();
            continue;
        }
        if (tid < kGQ) {
            s_q[tid] = tid < (int)m ? A.order[i0 + tid] : -1;
            s_pos[tid] = 0u;
            s_thr[tid] = kNoKey;
        }
        __syncthreads();
        const int cols = (keep >> 16) ? 32 : 16;
        // (the piece of the first rows: pieces before it are empty where there are
        // fewer tiles than pieces)
        stage_queries<DT, false>(A, s_q, keep, rec.j0, r0 == 0u, qp, q0s, s_qn, s_err);
        for (int j = tid; j < cols; j += kVB<DT>) {
            const int32_t q = s_q[j];
            if ((keep >> j) & 1u) {
                s_base[j] = A.coff[q];
                s_room[j] = A.kroom[q];
            }
        }
        __syncthreads();
        VerifyGroup G = {A.glist + rec.rows + r0, r1 - r0, keep, qp, q0s, s_qn, minima, s_thr, s_err,
                         s_base, s_room, s_pos, s_q, np > 1u, 0, 0, -1};
        if (cols == 32) verify_rows<DT, 2, false>(A, G);
        else verify_rows<DT, 1, false>(A, G);
        __syncthreads();  // every key is counted; q' is read before the next group's
        if (np == 1u && tid < cols && ((keep >> tid) & 1u)) A.kpos[s_q[tid]] = s_pos[tid];
        __syncthreads();  // the group's queries and counts are read before the next one's
    }
}

// Brute force over float rows: 32 consecutive queries and a piece of the rows per
// item, items of the same piece on one XCD (its L2 holds the rows while the
// queries pass).  Without a bound (the sample, or few rows) every row's key has its
// place in a query's list, and the item of the first rows sets up the lists and the
// fallback queue (ovf_count: its two words).  Bound by the matrix cores' FP32 rate from 32 queries on, by the
// rows' bytes below; rows beyond about 1,100 columns (LDS) stay with the
// per-query kernel, one workgroup per query.
// Measured (whole calls): 25 queries over 186,000 x 512: 44 ms with a workgroup
// per query, 0.30 here (the rows once: 0.08 ms at 4.9 TB/s); 120 over 200,000 x
// 280: 42 and 0.33; one over 64,000 x 418: 14 and 0.10.
__global__ __launch_bounds__(kVB<QW_F32>, 3) void dense_verify_kernel(GroupedArgs A, DenseArgs D)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int32_t s_q[kGQ];
    __shared__ uint32_t s_room[kGQ], s_thr[kGQ], s_qn[kGQ];
    __shared__ unsigned long long s_base[kGQ];
    __shared__ float s_err[kGQ];
    const int tid = threadIdx.x;
    unsigned char *qp = smem;  // q' [kGQ][ldq]
    float *q0s = reinterpret_cast<float *>(qp + (size_t)kGQ * verify_ldq<QW_F32>(A.dp));
    const uint32_t ng = (uint32_t)((A.Q + kGQ - 1) / kGQ), items = ng * D.pieces;
    const uint32_t per = (items + kXcd - 1u) / kXcd;
    const int64_t tiles = (D.rows + 31) / 32;
    for (uint32_t i = blockIdx.x; i < per * kXcd; i += gridDim.x) {
        const uint32_t it = i % kXcd * per + i / kXcd;
        if (it >= items) continue;  // uniform
        const uint32_t pc = it / ng, g = it - pc * ng;
        const int64_t r0 = min(D.rows, tiles * pc / D.pieces * 32), r1 = min(D.rows, tiles * (pc + 1) / D.pieces * 32);
        const int32_t m = (int32_t)min((int64_t)kGQ, A.Q - (int64_t)g * kGQ);
        const uint32_t keep = m == 32 ? ~0u : (1u << m) - 1u;
        if (r1 == r0) continue;  // uniform
        if (tid < kGQ) {
            const int32_t q = (int32_t)(g * kGQ) + tid;
            s_q[tid] = tid < m ? q : -1;
            s_thr[tid] = tid < m && D.bound ? D.bound[q] : kNoKey;
            s_room[tid] = D.cap;
            s_base[tid] = (unsigned long long)q * D.cap;
            if (!D.bound && r0 == 0) {
                if (q < 2) A.ovf_count[q] = 0u;
                if (tid < m) {
                    A.kpos[q] = (uint32_t)D.rows;
                    A.kroom[q] = D.cap;
                    A.coff[q] = (unsigned long long)q * D.cap;
                }
            }
        }
        __syncthreads();
        stage_queries<QW_F32, true>(A, s_q, keep, 0, !D.bound && r0 == 0, qp, q0s, s_qn, s_err);
        __syncthreads();
        VerifyGroup G = {nullptr, (uint32_t)(r1 - r0), keep, qp, q0s, s_qn, nullptr, s_thr, s_err,
                         s_base, s_room, nullptr, s_q, true, r0 * D.stride, D.stride, D.bound ? -1 : r0};
        if (m > 16) verify_rows<QW_F32, 2, true>(A, G);
        else verify_rows<QW_F32, 1, true>(A, G);
        __syncthreads();  // q' is read before the next item's
    }
}

// One workgroup per query: the K-th smallest key of a sample of the rows, widened
// by the keys' error, bounds the query's K-th key; its key list is empty again.
// Radix select over the keys' high words in LDS, a byte at a time.
__global__ __launch_bounds__(kBlock) void dense_bound_kernel(GroupedArgs A, DenseArgs D)
{
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *v = reinterpret_cast<uint32_t *>(smem);  // [D.rows]
    __shared__ uint32_t hist[256], s_pick, s_left;
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t q = blockIdx.x;
    const uint32_t n = (uint32_t)D.rows;
    const unsigned long long *keys = A.keys + q * D.cap;
    for (uint32_t i = tid; i < n; i += kBlock) v[i] = (uint32_t)(keys[i] >> 32);
    uint32_t t = 0, left = (uint32_t)A.K;  // the K-th smallest's bits so far; its rank among their equals
    if (n >= left)                         // uniform
        for (int sh = 24; sh >= 0; sh -= 8) {
            hist[tid] = 0;
            __syncthreads();
            for (uint32_t i = tid; i < n; i += kBlock)
                if (sh == 24 || v[i] >> (sh + 8) == t >> (sh + 8)) atomicAdd(&hist[v[i] >> sh & 255u], 1u);
            __syncthreads();
            if (tid < 64) {  // four bins per lane
                uint32_t h[4], sum = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) sum += h[i] = hist[4 * lane + i];
                uint32_t x = sum;
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t y = (uint32_t)__shfl_up((int)x, off);
                    if (lane >= off) x += y;
                }
                uint32_t before = x - sum;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (before < left && left <= before + h[i]) {
                        s_pick = (uint32_t)(4 * lane + i);
                        s_left = left - before;
                    }
                    before += h[i];
                }
            }
            __syncthreads();
            t |= s_pick << sh;
            left = s_left;
            __syncthreads();
        }
    if (tid == 0) {
        D.bound[q] = n >= (uint32_t)A.K ? __float_as_uint(band_threshold(__uint_as_float(t), A.eps, A.abs_err[q])) : kNoKey;
        A.kpos[q] = 0u;
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

// minima | q' rows | q0 (float rows)
static size_t verify_lds(int dtype, int dp)
{
    const size_t m = sizeof(uint32_t) * kGQ;
    return dtype == QW_F32 ? m * kVCells<QW_F32> + size_t(kGQ) * verify_ldq<QW_F32>(dp) + ga16(size_t(dp) * 4)
                           : m * kVCells<QW_U8> + size_t(kGQ) * verify_ldq<QW_U8>(dp);
}

float group_eps(int dp) { return 4.f * (float)(dp + 16) * 0x1p-24f * 1.01f; }

// Workspace for Q queries: a record per group, and candidate rows (a group
// beyond the space goes to the per-query kernel).
size_t group_rec_bytes(int64_t Q) { return (sizeof(GroupRec) * (size_t)Q + 255) & ~size_t(255); }
int group_filter_topk(int dtype) { return dtype == QW_F32 ? kGFilterK<QW_F32> : kGFilterK<QW_U8>; }
size_t group_list_bytes(int dtype, int64_t Q)
{
    const int64_t rows = dtype == QW_U8 ? 1024 : 2048;  // uint8: groups of several queries only
    return sizeof(uint2) * (size_t)std::max<int64_t>(Q * rows, 8 * 65536);
}

// Rows whose group of queries fits LDS (uint8 distances fit 31 bits); at most 64
// lists per query.
bool group_applies(int dtype, int dp, int nl, size_t lds_max)
{
    return nl >= 1 && nl <= 64 && dp <= 4096 && verify_lds(dtype, dp) + 2048 <= lds_max &&
           kUnionLds + 1024 <= lds_max / 2;
}

qw_status launch_grouped(GroupedArgs a, int cus, size_t lds_max, hipStream_t s)
{
    if (!group_applies(a.dtype, a.dp, a.nl, lds_max) || a.dp % 16 != 0) return QW_EINTERNAL;
    a.xchunk = std::max(1u, a.xchunk / kGQ);  // in groups
    if (a.gain > 0) {
        // groups have a.minrun / 2 queries at least (a label's are of even sizes)
        const int64_t most = 2 * a.Q / std::max<int64_t>(1, a.minrun) + 1;
        group_gain_kernel<<<(unsigned)ceil_div(most, kGainGroups), kGainBlock, 0, s>>>(a);
        QW_HIP(hipGetLastError());
        group_split_kernel<<<(unsigned)ceil_div(most, kGainBlock / 32), kGainBlock, 0, s>>>(a);
        QW_HIP(hipGetLastError());
        a.groups = a.groups2;
        a.gcount += kGroupCounts;
    }
    const size_t vl = verify_lds(a.dtype, a.dp);
    group_union_kernel<<<blocks_per_cu((const void *)group_union_kernel, kGB, kUnionLds) * cus, kGB, kUnionLds, s>>>(a);
    QW_HIP(hipGetLastError());
    const void *fn = a.dtype == QW_F32 ? (const void *)group_verify_kernel<QW_F32> : (const void *)group_verify_kernel<QW_U8>;
    const int grid = blocks_per_cu(fn, a.dtype == QW_F32 ? kVB<QW_F32> : kVB<QW_U8>, vl) * cus;
    if (a.dtype == QW_F32) group_verify_kernel<QW_F32><<<grid, kVB<QW_F32>, vl, s>>>(a);
    else group_verify_kernel<QW_U8><<<grid, kVB<QW_U8>, vl, s>>>(a);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

// Brute force: the sample holds `sample` rows, every list cap keys.  With s rows
// sampled about K n / s keys pass their bound; s near sqrt(K n) makes both small.
bool dense_plan(int64_t n, int32_t dtype, int32_t dp, int64_t Q, int32_t K, size_t lds_max, DensePlan *p)
{
    if (dtype != QW_F32 || n < 2048 || Q < 1 || dp % 16 != 0 || verify_lds(QW_F32, dp) + 2048 > lds_max) return false;
    int64_t s = 2048;
    while (s < kDenseSample && s * s < (int64_t)K * n) s += s / 2 / 32 * 32;
    s = std::min(s, kDenseSample);
    p->sample = n <= 2 * s ? n : s;  // few rows: their keys all, without a bound
    p->cap = (uint32_t)std::max<int64_t>(p->sample, 4 * K * n / s + 1024);
    if (p->sample == n) p->cap = (uint32_t)n;
    // queries per round: their lists stay within 256 MiB, whole groups
    p->chunk = std::min<int64_t>(Q, std::max<int64_t>(kGQ, ((int64_t)256 << 20) / (8 * (int64_t)p->cap) / kGQ * kGQ));
    return true;
}

// a.Q <= p.chunk queries.
qw_status launch_dense(const DensePlan &p, GroupedArgs a, int64_t n, uint32_t *bound, int cus, hipStream_t s)
{
    if (a.Q < 1 || a.Q > p.chunk || a.dp % 16 != 0 || p.sample > n || p.sample < 1) return QW_EINTERNAL;
    const size_t lds = verify_lds(QW_F32, a.dp);
    const int64_t ng = ceil_div(a.Q, kGQ);
    auto pass = [&](int64_t rows, int64_t stride, uint32_t *b) -> qw_status {
        DenseArgs d;
        d.rows = rows;
        d.stride = stride;
        d.bound = b;
        d.cap = p.cap;
        // about two pieces per CU in all, a tile for every wave of each
        const int64_t most = std::max<int64_t>(1, rows / (32 * kVW<QW_F32>));
        d.pieces = (uint32_t)std::min<int64_t>(most, std::max<int64_t>(1, 2 * cus / ng));
        const int64_t items = ng * d.pieces;
        const int grid = (int)std::min<int64_t>(ceil_div(items, kXcd) * kXcd, ceil_div(cus, kXcd) * kXcd);
        dense_verify_kernel<<<grid, kVB<QW_F32>, lds, s>>>(a, d);
        QW_HIP(hipGetLastError());
        return QW_OK;
    };
    const DenseArgs d = {p.sample, 0, bound, p.cap, 0};
    if (p.sample == n) return pass(n, 1, nullptr);
    QW_TRY(pass(p.sample, n / p.sample, nullptr));
    dense_bound_kernel<<<(unsigned)a.Q, kBlock, sizeof(uint32_t) * (size_t)p.sample, s>>>(a, d);
    QW_HIP(hipGetLastError());
    return pass(n, 1, bound);
}

}  // namespace qw
