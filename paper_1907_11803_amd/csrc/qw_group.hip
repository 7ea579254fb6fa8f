// Candidate work for float rows, several queries per workgroup: queries whose
// candidate sets overlap (neighbours of the grouped order with the same
// min-hash) form their union together and verify every row of it once, on the
// matrix cores -- the bucket's points are staged once and reused by the
// queries that hit it (Sections 4 and 5.1).
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
// where there are few groups: 16 x 16 blocks of rows x queries,
// v_mfma_f32_16x16x4f32 over x' = x - q0 and q' = q - q0 (q0: one query of the
// group), give F = |x'|^2 + |q'|^2 - 2 x'.q', and each (row, query) pair of the
// mask that may be among the query's K nearest writes its (F, id) key for the
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
// wrote keys); 1,000 scattered queries 2.3 ms before, 0.08, 0.99 and 0.03 now.
#include <algorithm>
#include <type_traits>

#include "qw_dedup.h"
#include "qw_internal.h"
#include "qw_band.h"

namespace qw {
namespace {

constexpr int kGB = 512;                                // threads per workgroup
constexpr int kGW = kGB / 64;                           // waves
constexpr int kVB = 768, kVW = kVB / 64;                // of the verification
constexpr int kGQ = 32;                                 // queries per group
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
        for (uint32_t i = 2 * tid; i < (1u << kGSetLog2); i += 2 * kGB)
            *reinterpret_cast<uint4 *>(tab + i) = uint4{kEmpty, 0u, kEmpty, 0u};
        __syncthreads();
        // the union: each half of a wave takes part after part, 32 ids at a
        // time, the next round's ids loading while this one's are inserted
        if (!many) {
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
        if (many || s_full || s_u > kGLimit) {  // uniform: beyond the set
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
                const uint32_t cnt = in ? min(s_cnt[l32], A.keep) : 0u;
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
                        A.ucount[q] = ok ? s_cnt[l32] : 0u;
                        A.kroom[q] = cnt;
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
    uint32_t *minima;          // [kGQ][kVCells]
    uint32_t *thr;             // per query: keys beyond it are not needed
    const float *err;          // absolute part of the keys' error (float rows)
    const unsigned long long *base;
    const uint32_t *room;
    uint32_t *pos;             // keys written by this workgroup
    const int32_t *q;
    bool pieces;
};
constexpr int kVCells = kVW * 8;  // minima per query: wave, quarter of its lanes, 16-row block
constexpr int kGFilterK = kVCells / 2;  // K up to which the minima bound the K-th key

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
// the waves' first tiles (384 rows, in the order of the ids' hash) the K-th
// smallest of a query's 96 minima over disjoint parts of them bounds its K-th
// key; rows beyond that bound (float rows: beyond its error band) give no key.
template <int DT, int CB>
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
        for (int j = wv; j < 16 * CB; j += kVW) {  // uniform
            const uint32_t *c = G.minima + j * kVCells;
            const uint32_t v0 = c[lane], v1 = lane + 64 < kVCells ? c[lane + 64] : kNoKey;
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
    static_assert(kVCells <= 128, "two minima per lane");
    if (wv >= ntile) {  // no tile: its minima are empty
        if (A.K <= kGFilterK) {
            for (int i = lane; i < 16 * CB * 8; i += 64) G.minima[(i >> 3) * kVCells + wv * 8 + (i & 7)] = kNoKey;
            bounds();
        }
        return;
    }
    auto entry = [&](int t, int h) -> uint2 {
        const uint32_t r = (uint32_t)(t * 32 + h * 16 + row16);
        const uint2 e = G.rows[r < U ? r : U - 1u];
        return uint2{e.x, r < U ? e.y & G.keep : 0u};  // rows past the end: nobody's
    };
    uint2 e0 = entry(wv, 0), e1 = entry(wv, 1), n0 = e0, n1 = e1;
    if (wv + kVW < ntile) {
        n0 = entry(wv + kVW, 0);
        n1 = entry(wv + kVW, 1);
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
    // each query's keys of the tile within its bound: lanes of one row16 share
    // a query, one of them takes the room for all
    auto emit = [&]() {
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            const int j = b * 16 + row16;
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
            lt += kVW;
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
            if (t == wv && A.K <= kGFilterK) {  // uniform in the workgroup: every wave's first tile
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        G.minima[(b * 16 + row16) * kVCells + wv * 8 + kg * 2 + h] =
                            min(min(key[h][b][0], key[h][b][1]), min(key[h][b][2], key[h][b][3]));
                bounds();
            }
            emit();
#pragma unroll
            for (int b = 0; b < CB; ++b) acc0[b] = acc1[b] = acc_t{0, 0, 0, 0};
            xn0 = xn1 = 0;
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
    acc_t ba[2 * NS], bb[2 * NS];
    load(ba);
    while (true) {
        step(ba, bb);
        if (t >= ntile) break;
        step(bb, ba);
        if (t >= ntile) break;
    }
}

template <int DT>
__global__ __launch_bounds__(kVB, kVB / 256) void group_verify_kernel(GroupedArgs A)
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
    unsigned char *qp = smem + sizeof(uint32_t) * kGQ * kVCells;  // q' [kGQ][ldq]
    float *q0s = reinterpret_cast<float *>(qp + (size_t)kGQ * ldq);
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
        const unsigned char *queries = static_cast<const unsigned char *>(A.queries);
        const int64_t rb = (int64_t)dp * (DT == QW_F32 ? 4 : 1);
        const float *q0 = reinterpret_cast<const float *>(queries + (int64_t)s_q[rec.j0] * rb);
        if constexpr (DT == QW_F32)
            for (int i = tid; i < dp; i += kVB) q0s[i] = q0[i];
        const int cols = (keep >> 16) ? 32 : 16;
        for (int j = wv; j < cols; j += kVW) {
            const bool in = (keep >> j) & 1u;  // uniform
            const int32_t q = in ? s_q[j] : s_q[rec.j0];
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
                    if (in && pc == 0u) {
                        A.abs_err[q] = err;
                        if (!(acc < 1e30f)) A.flag[q] = 1u;
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
            if (lane == 0 && in) {
                s_base[j] = A.coff[q];
                s_room[j] = A.kroom[q];
            }
        }
        __syncthreads();
        VerifyGroup G = {A.glist + rec.rows + r0, r1 - r0, keep, qp, q0s, s_qn, minima, s_thr, s_err,
                         s_base, s_room, s_pos, s_q, np > 1u};
        if (cols == 32) verify_rows<DT, 2>(A, G);
        else verify_rows<DT, 1>(A, G);
        __syncthreads();  // every key is counted; q' is read before the next group's
        if (np == 1u && tid < cols && ((keep >> tid) & 1u)) A.kpos[s_q[tid]] = s_pos[tid];
        __syncthreads();  // the group's queries and counts are read before the next one's
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
    const size_t m = sizeof(uint32_t) * kGQ * kVCells;
    return dtype == QW_F32 ? m + size_t(kGQ) * verify_ldq<QW_F32>(dp) + ga16(size_t(dp) * 4)
                           : m + size_t(kGQ) * verify_ldq<QW_U8>(dp);
}

float group_eps(int dp) { return 4.f * (float)(dp + 16) * 0x1p-24f * 1.01f; }

// Workspace for Q queries: a record per group, and candidate rows (kGRows per
// query; a group beyond the space goes to the per-query kernel).
constexpr int64_t kGRows = 2048;
size_t group_rec_bytes(int64_t Q) { return sizeof(GroupRec) * (size_t)Q; }
int group_filter_topk() { return kGFilterK; }
size_t group_list_bytes(int64_t Q) { return sizeof(uint2) * (size_t)std::max<int64_t>(Q * kGRows, 8 * 65536); }

// Float rows whose group of queries fits LDS; at most 64 lists per query.
bool group_applies(int dtype, int dp, int nl, size_t lds_max)
{
    return dtype == QW_F32 && nl >= 1 && nl <= 64 && verify_lds(dtype, dp) + 2048 <= lds_max &&
           kUnionLds + 1024 <= lds_max / 2;
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
    const size_t ul = kUnionLds, vl = verify_lds(QW_F32, a.dp);
    group_union_kernel<<<blocks_per_cu((const void *)group_union_kernel, kGB, ul) * cus, kGB, ul, s>>>(a);
    QW_HIP(hipGetLastError());
    group_verify_kernel<QW_F32><<<blocks_per_cu((const void *)group_verify_kernel<QW_F32>, kVB, vl) * cus, kVB, vl, s>>>(a);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

}  // namespace qw
