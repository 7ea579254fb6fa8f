// Exact k nearest neighbours of a batch of queries over every point (the
// ground truth that recall is measured against), uint8 rows of at most 1024
// bytes, on the matrix cores.
//
// |x - q|^2 = |x'|^2 + |q'|^2 - 2 x'.q' with x' = x - 128 (a flipped top bit):
// the products are those of signed bytes, v_mfma_i32_16x16x64_i8 forms them
// exactly (|sum| <= 1024 * 2^14), so every distance is the exact integer.
//
// Two passes of the same product, and no distance matrix in memory:
//   sample   every r-th row; each lane keeps the smallest distance of its own
//            stream of points per query.  A stream's minimum is the distance
//            of some point and streams are disjoint, so the K-th smallest
//            minimum of a query bounds its K-th distance from above.
//   collect  every row; a point within its query's bound (or one beyond it)
//            is appended to the query's key list (about K r entries), from
//            which the select kernel takes the K smallest by (distance, id).
// A list that overflows (many equal distances, or rows whose order the sample
// missed) sends its query to the per-query kernel, so the bound's quality
// never changes a result.
//
// Bound by the matrix cores' issue and the LDS reads that feed them: a wave
// holds its queries' operands in registers for its whole run of points and
// reads 1 KB of point operands from LDS per NC MFMAs (of 16 cycles each).
// Accumulators start at -(|x'|^2 >> 1), so the test of an output is one
// integer compare against a per-lane constant, and four outputs share it
// through two max3.
// Measured (1M x 128, 2000 queries, K = 10): 27.4 ms with one workgroup per
// query re-reading every row through v_dot4, 0.41 ms here (collect 0.33,
// sample 0.04, bounds 0.02): the matrix cores issue a third of the time, the
// compares of the outputs as long.
#include <algorithm>

#include "qw_internal.h"

namespace qw {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

// LDS hit buffer of a workgroup.  A tile of 128 points and 512 queries has about
// 65,536 K r / n hits of its own (K r keys per query of n rows; half a buffer may
// be left from tiles before it): what the buffer does not hold goes to the lists
// directly, up to kHitMax (beyond it many rows are equal, and such queries
// overflow their lists anyway: they take no more).  500 queries, K = 1000, over 200,000 x 128: 2.75
// ms with a workgroup per query, 3.43 when a hit beyond the buffer sent its query
// there after this kernel, 0.75 now.
constexpr int kHitBuf = 1024, kHitMax = 2 * kHitBuf;
constexpr int32_t kNoPoint = 0x7FFFFFFE;  // |x'|^2 of a row past the end: never within a bound

// 16 bytes of a row as signed bytes; zeros past the row's parts (both
// operands hold them, and zeros add nothing to a product or a norm)
__device__ inline v4i signed_part(uint4 v, bool in)
{
    return in ? v4i{(int)(v.x ^ 0x80808080u), (int)(v.y ^ 0x80808080u), (int)(v.z ^ 0x80808080u),
                    (int)(v.w ^ 0x80808080u)}
              : v4i{0, 0, 0, 0};
}

__device__ inline int norm_part(v4i v)
{
    int s = __builtin_amdgcn_sdot4(v.x, v.x, 0, false);
    s = __builtin_amdgcn_sdot4(v.y, v.y, s, false);
    s = __builtin_amdgcn_sdot4(v.z, v.z, s, false);
    return __builtin_amdgcn_sdot4(v.w, v.w, s, false);
}

// Sum over aligned groups of RP lanes (4 .. 64), in every lane of the group:
// DPP exchanges inside 16 lanes (quads, then mirrored halves of 8 and 16,
// whose lanes already agree within each half), shuffles above.
template <int RP> __device__ inline int row_sum(int v)
{
    v += __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);                  // quad_perm [1,0,3,2]
    v += __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);                  // quad_perm [2,3,0,1]
    if constexpr (RP >= 8) v += __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    if constexpr (RP >= 16) v += __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false);  // row_mirror
    if constexpr (RP >= 32) v += __shfl_xor(v, 16);
    if constexpr (RP >= 64) v += __shfl_xor(v, 32);
    return v;
}

// KS: 64-byte steps of a row (a power of two, rows of at most 64 KS bytes).
// A wave multiplies NC blocks of 16 queries: NC KS <= 16 keeps their operands
// in 64 registers.
// 1M x 128, 2000 queries, both passes: NC = 8 0.41 ms, NC = 4 0.46 (it reads
// LDS twice as often per product); rows of 64 bytes: 0.14 and 0.12 (there the
// outputs' compares bound, and NC = 4 leaves more waves to overlap them).
constexpr int brute_blocks(int ks) { return ks == 2 ? 8 : ks < 4 ? 4 : 16 / ks; }

template <int KS> struct BruteTile {
    static constexpr int NC = brute_blocks(KS);
    static constexpr int PT = KS <= 4 ? 128 : 512 / KS;  // points staged at a time
    static constexpr int RP = KS * 4;                    // 16-byte parts per staged row
    static constexpr int NL = PT * RP / kBlock;          // parts staged per thread
    static constexpr int RS = KS * 64 + 16;              // staged row stride, bytes
};

// Workgroup b: run `slab` of the point tiles against query tile `qt`; the
// query tiles of one run are dealt to the same XCD back to back, so its points
// are read into that L2 once.  Of the four waves, qw take different query
// blocks and 4 / qw different points of each tile (few queries).
template <int KS, bool COLLECT>
__global__ __launch_bounds__(kBlock, 2) void brute_kernel(BruteArgs A)
{
    using T = BruteTile<KS>;
    constexpr int NC = T::NC, PT = T::PT, RP = T::RP, NL = T::NL, RS = T::RS;
    __shared__ __align__(16) unsigned char xs[PT * RS];
    __shared__ __align__(16) int32_t ninit[PT];  // -(|x'|^2 >> 1): the accumulators' start
    __shared__ int32_t nodd[COLLECT ? PT : 1];   // |x'|^2 & 1
    __shared__ unsigned long long hkey[COLLECT ? kHitBuf : 1];
    __shared__ int32_t hq[COLLECT ? kHitBuf : 1];
    __shared__ uint32_t hcnt;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kg = lane >> 4;
    const int32_t b = (int32_t)blockIdx.x, nqt = A.nqt;
    const int32_t slab = (b / (kXcd * nqt)) * kXcd + b % kXcd;
    const int32_t qt = (b / kXcd) % nqt;
    const int qw = A.qw, pw = 4 / qw;  // waves over queries, over points
    const int wq = wv % qw, wp = wv / qw;
    const int32_t q0 = qt * (16 * NC * qw) + wq * (16 * NC);
    const int parts = A.dp / 16;
    const uint4 *queries = reinterpret_cast<const uint4 *>(A.queries);
    const uint4 *data = reinterpret_cast<const uint4 *>(A.data);

    // query operands: lane (col, kg) holds bytes 64 st + 16 kg .. + 15 of
    // query q0 + 16 c + col
    v4i bq[NC][KS];
    int32_t qq[NC], best[NC];
    bool live[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int32_t q = q0 + 16 * c + col;
        live[c] = q < A.Q;
        const int64_t row = (int64_t)(live[c] ? q : A.Q - 1) * parts;
        int s = 0;
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const int p = st * 4 + kg;
            bq[c][st] = signed_part(queries[row + (p < parts ? p : parts - 1)], p < parts);
            s += norm_part(bq[c][st]);
        }
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        qq[c] = s;
        // COLLECT: |x - q|^2 <= bound needs acc >= (|q'|^2 - bound) / 2, rounded
        // up; a column past the last query takes nothing
        best[c] = COLLECT ? (live[c] ? (int32_t)(((int64_t)s - (int64_t)A.bound[q] + 1) >> 1) : INT32_MAX)
                          : INT32_MIN;
    }
    if (tid == 0) hcnt = 0;

    const int32_t ntile = (int32_t)((A.rows + PT - 1) / PT);
    const int32_t t0 = (int32_t)((int64_t)ntile * slab / A.slabs);
    const int32_t t1 = (int32_t)((int64_t)ntile * (slab + 1) / A.slabs);
    uint4 xr[NL];
    auto load_tile = [&](int32_t t) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int e = tid + i * kBlock, r = e / RP, p = e % RP;
            int64_t row = ((int64_t)t * PT + r) * A.stride;
            row = row < A.n ? row : A.n - 1;
            xr[i] = data[row * parts + (p < parts ? p : parts - 1)];
        }
    };
    auto append = [&](int32_t q, unsigned long long key) {
        const uint32_t pos = atomicAdd(&A.count[q], 1u);
        if (pos < A.cap) A.keys[(int64_t)q * A.cap + pos] = key;
        else A.flag[q] = 1u;
    };
    if (t0 < t1) load_tile(t0);
    for (int32_t t = t0; t < t1; ++t) {
        __syncthreads();  // the previous tile has been read
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int e = tid + i * kBlock, r = e / RP, p = e % RP;
            const v4i v = signed_part(xr[i], p < parts);
            *reinterpret_cast<v4i *>(xs + r * RS + p * 16) = v;
            const int s = row_sum<RP>(norm_part(v));  // over the RP consecutive lanes of the row
            if (p == 0) {
                const int32_t xx = (int64_t)t * PT + r < A.rows ? s : kNoPoint;
                ninit[r] = -(xx >> 1);
                if (COLLECT) nodd[r] = xx & 1;
            }
        }
        __syncthreads();
        if (t + 1 < t1) load_tile(t + 1);
        // the next 16 points' operands are read while the current ones multiply
        v4i an[KS], in;
        auto read_sub = [&](int sub) {
            in = *reinterpret_cast<const v4i *>(ninit + sub * 16 + kg * 4);
#pragma unroll
            for (int st = 0; st < KS; ++st)
                an[st] = *reinterpret_cast<const v4i *>(xs + (sub * 16 + col) * RS + st * 64 + kg * 16);
        };
        read_sub(wp);
#pragma unroll 2
        for (int sub = wp; sub < PT / 16; sub += pw) {
            v4i acc[NC], a[KS];
            const v4i init = in;
#pragma unroll
            for (int st = 0; st < KS; ++st) a[st] = an[st];
            read_sub(sub + pw < PT / 16 ? sub + pw : sub);
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[c] = init;
#pragma unroll
            for (int st = 0; st < KS; ++st)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[st], bq[c][st], acc[c], 0, 0, 0);
            // a result is read only after all products are issued: read one by
            // one, each would stall the wave for a product's latency
            __builtin_amdgcn_sched_barrier(0);
            // acc[c][i]: point sub * 16 + 4 kg + i, query q0 + 16 c + col
            int32_t m[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) m[c] = max(max(acc[c][0], acc[c][1]), max(acc[c][2], acc[c][3]));
            if (!COLLECT) {
#pragma unroll
                for (int c = 0; c < NC; ++c) best[c] = max(best[c], m[c]);
            } else {
                bool any = false;
#pragma unroll
                for (int c = 0; c < NC; ++c) any |= m[c] >= best[c];
                if (__ballot(any) != 0ull) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        if (m[c] < best[c]) continue;
                        const int32_t q = q0 + 16 * c + col;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int pt = sub * 16 + kg * 4 + i;
                            const int64_t row = (int64_t)t * PT + pt;
                            const int32_t dist = qq[c] - 2 * acc[c][i] + nodd[pt];
                            if (acc[c][i] < best[c] || row >= A.rows) continue;
                            const uint32_t e = atomicAdd(&hcnt, 1u);
                            if (e < (uint32_t)kHitBuf) {
                                hkey[e] = ((unsigned long long)(uint32_t)dist << 32) | (uint32_t)row;
                                hq[e] = q;
                            } else if (e < (uint32_t)kHitMax) {  // to the query's list at once
                                append(q, ((unsigned long long)(uint32_t)dist << 32) | (uint32_t)row);
                            } else {  // equal rows: no more of this query here
                                A.flag[q] = 1u;
                                best[c] = INT32_MAX;
                            }
                        }
                    }
                }
            }
        }
        if (COLLECT) {
            __syncthreads();
            const uint32_t nh = hcnt < (uint32_t)kHitBuf ? hcnt : (uint32_t)kHitBuf;
            const bool over = hcnt > (uint32_t)kHitMax;  // some queries are flagged
            if (nh > (uint32_t)kHitBuf / 2 || (t + 1 == t1 && nh)) {  // uniform
                for (uint32_t e = tid; e < nh; e += kBlock)
                    if (!over || A.flag[hq[e]] == 0u) append(hq[e], hkey[e]);
                __syncthreads();
                if (tid == 0) hcnt = 0;
            }
        }
    }
    if (!COLLECT) {
        // stream (slab, wp, kg) of each query: an upper bound on its smallest
        // distance (the low bit of |x'|^2 is not in the accumulator)
        const int32_t stream = (slab * pw + wp) * 4 + kg;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (live[c]) {
                const int64_t v = (int64_t)qq[c] - 2 * (int64_t)best[c] + 1;
                A.minima[(int64_t)(q0 + 16 * c + col) * A.streams + stream] =
                    (int32_t)(v < ((int64_t)2 << A.top_bit) - 1 ? v : ((int64_t)2 << A.top_bit) - 1);
            }
    }
}

// One workgroup per query: the K-th smallest of its `streams` minima (at most
// 32 per thread), by a radix search from the top bit, and the query's list
// state cleared, with the round's fallback queue.
constexpr int kMinPerThread = 32;
__global__ __launch_bounds__(kBlock) void brute_bound_kernel(BruteArgs A)
{
    __shared__ uint32_t wc[2][kBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t q = blockIdx.x;
    const int nper = (A.streams + kBlock - 1) / kBlock;  // uniform
    uint32_t v[kMinPerThread];
#pragma unroll
    for (int i = 0; i < kMinPerThread; ++i) {
        const int e = tid + i * kBlock;
        v[i] = i < nper && e < A.streams ? (uint32_t)A.minima[q * A.streams + e] : 0xFFFFFFFFu;
    }
    uint32_t prefix = 0, k = (uint32_t)A.K;
    for (int bit = A.top_bit; bit >= 0; --bit) {  // minima are below 2^(top_bit + 1)
        const uint32_t above = ~0u << (bit + 1);
        uint32_t cnt = 0;  // of this wave, by ballots: no shuffle tree
#pragma unroll
        for (int i = 0; i < kMinPerThread; ++i)
            if (i < nper)
                cnt += (uint32_t)__popcll(__ballot(((v[i] ^ prefix) & above) == 0u && ((v[i] >> bit) & 1u) == 0u));
        uint32_t *w = wc[bit & 1];
        if (lane == 0) w[wv] = cnt;
        __syncthreads();  // the other buffer's readers have passed the previous one
        uint32_t tot = 0;
        for (int i = 0; i < kBlock / 64; ++i) tot += w[i];
        if (tot < k) {
            prefix |= 1u << bit;
            k -= tot;
        }
    }
    if (tid == 0) {
        A.bound[q] = (int32_t)prefix;
        A.count[q] = 0u;
        A.flag[q] = 0u;
        A.coff[q] = (unsigned long long)q * A.cap;
        if (q == 0) A.fb_count[0] = A.fb_count[1] = 0u;
    }
}

int brute_steps(int dp)
{
    int ks = 1;
    while (ks * 64 < dp) ks <<= 1;
    return ks;
}

template <bool COLLECT>
void launch_pass(int ks, unsigned grid, const BruteArgs &a, hipStream_t s)
{
    switch (ks) {
    case 1: brute_kernel<1, COLLECT><<<grid, kBlock, 0, s>>>(a); break;
    case 2: brute_kernel<2, COLLECT><<<grid, kBlock, 0, s>>>(a); break;
    case 4: brute_kernel<4, COLLECT><<<grid, kBlock, 0, s>>>(a); break;
    case 8: brute_kernel<8, COLLECT><<<grid, kBlock, 0, s>>>(a); break;
    default: brute_kernel<16, COLLECT><<<grid, kBlock, 0, s>>>(a); break;
    }
}

int round_up_pow2(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

}  // namespace

// Sample rate, list capacity, query and point tiling for Q queries over n
// rows of dp bytes.  The list of a query holds about K r points: r = 8 costs
// an eighth of a pass; larger K sample more, so that lists stay a few K long,
// and every query has room for four times what is expected.  At least 8 K
// streams (where the tiles allow) keep two of the K nearest out of one stream,
// and 2 K are needed for a bound at all.
bool brute_plan(int64_t n, int32_t dtype, int32_t dp, int64_t Q, int32_t K, BrutePlan *p)
{
    if (dtype != QW_U8 || dp > 1024 || n < 4096 || Q < 1) return false;
    p->ks = brute_steps(dp);
    const int nc = brute_blocks(p->ks), pt = p->ks <= 4 ? 128 : 512 / p->ks;
    p->r = K <= 64 ? 8 : K <= 256 ? 4 : 2;
    while (p->r > 1 && n / p->r < std::max<int64_t>(16384, 64 * (int64_t)K)) p->r >>= 1;
    p->cap = round_up_pow2(std::max(1024, 4 * K * p->r));
    // queries per round: their lists stay within 128 MiB
    p->chunk = std::min<int64_t>(Q, std::max<int64_t>(256, ((int64_t)128 << 20) / (8 * (int64_t)p->cap)));
    const int64_t qblk = (p->chunk + 16 * nc - 1) / (16 * nc);
    p->qw = qblk >= 3 ? 4 : (int)qblk;
    if (p->qw * (pt / 16) < 4) p->qw = 64 / pt;  // every wave has points of each tile
    p->nqt = (int)((qblk + p->qw - 1) / p->qw);
    const int pw = 4 / p->qw;
    // about four workgroups per CU; whole groups of XCDs
    const int64_t want = std::max<int64_t>(8, ((1024 + p->nqt - 1) / p->nqt + 7) / 8 * 8);
    const int64_t rows_s = (n + p->r - 1) / p->r;
    auto slabs = [&](int64_t rows, int64_t w) {
        const int64_t tiles = (rows + pt - 1) / pt;
        return (int)std::max<int64_t>(8, std::min<int64_t>(w, (tiles + 7) / 8 * 8));
    };
    const int64_t need = ((8 * (int64_t)K + 4 * pw - 1) / (4 * pw) + 7) / 8 * 8;
    p->slabs_s = slabs(rows_s, std::min<int64_t>(std::max(want, need), 8192 / (4 * pw)));
    p->streams = p->slabs_s * pw * 4;
    p->slabs_c = slabs(n, want);
    // streams that hold points at all: one per tile and lane group
    const int64_t full = std::min<int64_t>(p->streams, (rows_s + pt - 1) / pt * pw * 4);
    return full >= 2 * (int64_t)K;
}

// Q <= p.chunk queries.
qw_status launch_brute(const BrutePlan &p, BruteArgs a, hipStream_t s)
{
    if (a.Q < 1 || a.Q > p.chunk || a.n < 1 || a.dp % 16 != 0 || a.dp > 64 * p.ks) return QW_EINTERNAL;
    a.nqt = p.nqt;
    a.qw = p.qw;
    a.cap = (uint32_t)p.cap;
    a.streams = p.streams;
    // every distance and stream minimum is at most dp * 255^2 + 1
    a.top_bit = 0;
    while (((int64_t)2 << a.top_bit) - 1 < (int64_t)a.dp * 65025 + 1) ++a.top_bit;
    a.slabs = p.slabs_s;
    a.stride = p.r;
    a.rows = (a.n + p.r - 1) / p.r;
    launch_pass<false>(p.ks, (unsigned)(a.slabs * a.nqt), a, s);
    QW_HIP(hipGetLastError());
    brute_bound_kernel<<<(unsigned)a.Q, kBlock, 0, s>>>(a);
    QW_HIP(hipGetLastError());
    a.slabs = p.slabs_c;
    a.stride = 1;
    a.rows = a.n;
    launch_pass<true>(p.ks, (unsigned)(a.slabs * a.nqt), a, s);
    QW_HIP(hipGetLastError());
    return QW_OK;
}

}  // namespace qw
