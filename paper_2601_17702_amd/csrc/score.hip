// Generation-time co-activation scoring (Sec. 3.5 scoring equation; App. D.2 / App. E weights;
// Sec. 3.5 "Adaptive Granularity" read as box pooling + fixed-length spans with NMS).
//
//   1. query weights   qw[h][f] = IDF_h(f) * sum of the query activations that name f (summed per head in LDS)
//   2. postings gather S[t] += qw[h][f] for every t in I_h[f], all heads into one S: a workgroup keeps the scores
//      of one block of positions in LDS and reads, of every list, only the postings of its block (the index's
//      block table); no atomic ever reaches global memory, at any context length
//   3. span pooling    W[s] = S[s] + ... + S[s + len - 1], with the best window of every tile
//   4. Top-B           greedy best window, optional suppression of overlapping windows
//
// Every sum is carried in 64-bit fixed point (power-of-two scales derived on the device from a head's
// largest query activation / the largest weight), so additions commute exactly: the result does not
// depend on the order in which wavefronts reach a position, run-to-run output is bit-identical,
// and a window's score is exactly the sum of its members.  Values are rounded to fp32 once, on
// output.
#include "greedy.h"
#include "s3_common.h"

#include <math.h>

#include <type_traits>

namespace {

// A posting list with a non-zero query weight.
struct alignas(16) ActiveList {
    double w;
    int32_t f;
    int32_t pad;
};

struct ScoreArgs {
    const int32_t* qids;
    const float* qvals;
    const int32_t* offsets;
    const int32_t* positions;
    int64_t off_stride, pos_stride;
    const int32_t* btab;             // block table of the index (null: none or not usable)
    int nblk;                        // blocks the table covers
    // compact index (all null / 0 for the plain one): 16-bit block-relative postings in block-major order
    const uint16_t* delta;           // [n_heads] x delta_stride
    const int32_t* cstart;           // [n_heads] x cstart_stride: start of segment (block b, feature f) at b * n_feat + f
    const int32_t* cfreq;            // [n_heads][n_feat] list lengths (0: dropped)
    int64_t delta_stride, cstart_stride;
    int n_heads, n_feat, k, nq;
    int nr;                          // feature ranges per head (sc_prep_kernel)
    int64_t L, nW;
    int len, top_b, nms, hb;
    int32_t max_freq;
    unsigned long long* wmax;        // [n_heads * nr] bits (as double) of each range's largest weight; [n_heads * nr]: of all; behind it the
                                     // number of partial arrays that were written (post)
    ActiveList* act;                 // [n_heads * n_feat] lists with a non-zero weight, packed per (head, range)
    int* nact;                       // [n_heads * nr] their number
    int* post;                       // [n_heads * nr] their postings / 64, for kernels that decide how many parts there are (else null)
    unsigned long long* sfix;        // [L]
    unsigned long long* part;        // [ngroup][L] partial sums of the gather's groups (ngroup > 1)
    int nsum;                        // arrays that the pooling sums at most: part's, or 1 if sfix holds the scores
    int pb, npb, heads_per, parts, ngroup, sorted;   // the gather: position blocks, heads of a group, parts of these, groups in all
    int mixed;                       // lists of several heads and ranges may be looked at together
    long long* wfix;                 // [nW]
    unsigned long long* tmaxv;       // [nsub] best window of every 2^sublog starts: its sum + 1, 0 for none
    int* tmaxi;                      // [nsub] its start
    int sublog;                      // 6 where the search brings blocks into LDS, else kSubLog2
    int need, room;                  // blocks that it brings there at least, entries of its list of choices
    int ntile, nsub, topshift;       // tiles of tile starts; sc_topb_long_kernel works on tiles of kSubW << topshift
    int tile;                        // windows per workgroup of the pooling kernel
    float* scores_out;
    int32_t* span_start;
    float* span_score;
    int32_t* n_found;
};

constexpr int kRange = 16384;        // features whose sums one workgroup of sc_prep_kernel holds in LDS
constexpr int kPrepThreads = 1024;
constexpr int kRun = 32;             // consecutive windows per thread (sliding sum, exact in integers)
constexpr int kTileW = 64 * kRun;    // windows per tile = per wavefront of the pooling kernel
constexpr int kSubLog2 = 8;
constexpr int kSubW = 1 << kSubLog2; // windows per entry of the tile maxima (sc_topb_kernel, sc_topb_long_kernel)
// For so few spans, or so few that reach into so many blocks, bringing blocks into LDS is not worth its beginning, nor where a span's
// blocks take longer to look through than to read again: us for a look-up with the maxima in registers / blocks in LDS, 4 spans of 64 as
// long; 5 of 64 in 1000 to 1000000 positions 27 to 49 / 26 to 48, without a match 22 to 44 / 25 to 49; 8 26 to 44 / 22 to 38; 5 of 512 29 to
// 51 / 33 to 53, 8 35 to 58 / 33 to 55 (with few matches 28 to 52 / 30 to 65), 12 35 to 52 / 29 to 46; 16 of 1024 in 16384 positions 37 / 45.
constexpr int kTopFew = 4;
inline bool top_many(int64_t found, int64_t reach) { return found > kTopFew && found > reach / 50 && reach < 900; }
constexpr int kTopSlots = 256;       // blocks of 64 windows that the search holds in LDS at most (135 KB, and 12 of choices in rounds)
static_assert(s3greedy::lds_bytes<unsigned long long>(kTopSlots) + s3greedy::kListMax * 12 + s3greedy::lds_static(kTopSlots) <= s3greedy::kLdsMost);
constexpr int kTopRegs = 4;          // registers per lane for the maxima of a short context
constexpr int kTopThreads = 1024;    // long contexts: all of them load the tile maxima, one wavefront searches
constexpr int kTopTiles = 4096;      // tiles of the Top-B search: 64 groups of 64, one group per lane

__device__ __forceinline__ int exp_s(unsigned long long wmax_bits, int hb) {   // weights are scaled by 2^exp_s: sums < 2^62
    double w = __longlong_as_double((long long)wmax_bits);
    if (!(w > 0.0)) return 0;
    int e;
    frexp(w, &e);
    return 62 - hb - e;
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        unsigned int lo = (unsigned int)__shfl_xor((int)(unsigned int)v, o);
        unsigned int hi = (unsigned int)__shfl_xor((int)(unsigned int)(v >> 32), o);
        unsigned long long other = ((unsigned long long)hi << 32) | lo;
        v = other > v ? other : v;
    }
    return v;
}

// Query weights of one (head, range of kRange features): the head's query pairs are summed per feature in LDS
// (64-bit fixed point, scaled by the head's largest activation, so the sum does not depend on the order), turned
// into weights qw[f] = IDF(f) * sum (App. D.2; natural log; lists longer than max_freq skipped, App. E), and the
// lists with a non-zero weight are packed for the gather.  One workgroup writes its own slice of every output:
// nothing has to be zeroed beforehand and no atomic leaves the workgroup.
__global__ __launch_bounds__(kPrepThreads) void sc_prep_kernel(ScoreArgs a) {
    extern __shared__ unsigned long long tbl[];
    __shared__ unsigned int amax[kPrepThreads / 64];
    __shared__ unsigned long long wmx[kPrepThreads / 64];
    __shared__ int wsum[kPrepThreads / 64], psum[kPrepThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = blockIdx.y, r = blockIdx.x;
    const int f0 = r * kRange, nf = min(kRange, a.n_feat - f0);
    for (int i = tid; i < nf; i += kPrepThreads) tbl[i] = 0ull;
    const size_t per_head = (size_t)a.nq * a.k;
    const float* qv = a.qvals + (size_t)h * per_head;
    const int32_t* qi = a.qids + (size_t)h * per_head;
    unsigned int m = 0;
    constexpr int kU = 8;            // loads in flight per thread (32768 pairs a head, 32 heads: 40 us with one)
    for (size_t i0 = tid; i0 < per_head; i0 += kU * kPrepThreads) {
        float v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = qv[min(i0 + u * kPrepThreads, per_head - 1)];
#pragma unroll
        for (int u = 0; u < kU; ++u) m = max(m, __float_as_uint(fmaxf(v[u], 0.f)));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, (unsigned int)__shfl_xor((int)m, o));
    if (lane == 0) amax[wave] = m;
    __syncthreads();
    m = 0;
#pragma unroll
    for (int q = 0; q < kPrepThreads / 64; ++q) m = max(m, amax[q]);
    int eq = 0;                      // activations are scaled by 2^eq: each below 2^40, a sum of 2^20 of them below 2^60
    if (m) {
        int e;
        frexpf(__uint_as_float(m), &e);
        eq = 40 - e;
    }
    const double scale = ldexp(1.0, eq), inv = ldexp(1.0, -eq);
    for (size_t i0 = tid; i0 < per_head; i0 += kU * kPrepThreads) {
        float v[kU];
        int f[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const size_t i = min(i0 + u * kPrepThreads, per_head - 1);
            v[u] = i0 + u * kPrepThreads < per_head ? qv[i] : 0.f;
            f[u] = qi[i];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (v[u] > 0.f && (unsigned)(f[u] - f0) < (unsigned)nf) atomicAdd(&tbl[f[u] - f0], (unsigned long long)llrint((double)v[u] * scale));
    }
    __syncthreads();
    constexpr int kPer = kRange / kPrepThreads;
    const int32_t* off = a.cfreq ? nullptr : a.offsets + (size_t)h * a.off_stride + f0;
    double w[kPer];
    int c = 0, postings = 0;
    double mx = 0.0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = j * kPrepThreads + tid;
        w[j] = 0.0;
        if (i < nf) {
            const unsigned long long sacc = tbl[i];
            if (sacc) {
                const int freq = a.cfreq ? a.cfreq[(size_t)h * a.n_feat + f0 + i] : off[i + 1] - off[i];
                if (freq > 0 && !(a.max_freq > 0 && freq > a.max_freq)) {
                    w[j] = (double)sacc * inv / ((double)logf(1.0f + (float)freq) + 1.0);
                    postings += freq;
                }
            }
        }
        c += w[j] > 0.0 ? 1 : 0;
        mx = fmax(mx, w[j]);
    }
    int tot;
    int slot = s3_block_excl_scan<kPrepThreads>(c, wsum, tot);
    ActiveList* out = a.act + (size_t)h * a.n_feat + f0;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (w[j] > 0.0) out[slot++] = ActiveList{w[j], f0 + j * kPrepThreads + tid, 0};
    const unsigned long long mb = wave_max_u64((unsigned long long)__double_as_longlong(mx));
    const int wp = s3_wave_incl_scan(postings);
    if (lane == 63) { wmx[wave] = mb; psum[wave] = wp; }
    __syncthreads();
    if (tid == 0) {
        unsigned long long best = 0;
        int sum = 0;
        for (int q = 0; q < kPrepThreads / 64; ++q) { best = wmx[q] > best ? wmx[q] : best; sum += psum[q]; }
        a.wmax[h * a.nr + r] = best;
        a.nact[h * a.nr + r] = tot;
        if (a.post) a.post[h * a.nr + r] = sum >> 6;
    }
}

// The same for queries of few pairs (at most kPrepThreads a head): a thread has a pair, a table of 2048 places in LDS finds those that
// name the same feature, and the thread that came first to a feature's place carries its list on, whose length it asked
// for beside the look for the largest activation.  All lists of a head go to its first range.  A table of all features
// took 12.4 us for 128 pairs in each of 256 heads (clearing it and looking through it, and one latency after the other), this 5.
constexpr int kHash = 2 * kPrepThreads;
__global__ __launch_bounds__(kPrepThreads) void sc_prep_few_kernel(ScoreArgs a) {
    __shared__ int name[kHash];
    __shared__ unsigned long long sum[kHash];
    __shared__ unsigned int amax[kPrepThreads / 64];
    __shared__ unsigned long long wmx[kPrepThreads / 64];
    __shared__ int wsum[kPrepThreads / 64], psum[kPrepThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = blockIdx.x;
    const int per_head = a.nq * a.k;
    float v = 0.f;
    int f = 0;
    if (tid < per_head) {
        v = fmaxf(a.qvals[(size_t)h * per_head + tid], 0.f);
        f = a.qids[(size_t)h * per_head + tid];
    }
    for (int i = tid; i < kHash; i += kPrepThreads) { name[i] = -1; sum[i] = 0ull; }
    const bool mine = v > 0.f && (unsigned)f < (unsigned)a.n_feat;
    int freq = 0;
    if (mine) {
        if (a.cfreq) {
            freq = a.cfreq[(size_t)h * a.n_feat + f];
        } else {
            const int32_t* off = a.offsets + (size_t)h * a.off_stride + f;
            freq = off[1] - off[0];
        }
    }
    const unsigned most = s3_wave_max_u32(__float_as_uint(v));
    if (lane == 0) amax[wave] = most;
    __syncthreads();
    const unsigned m = s3_wave_max_u32(amax[lane & (kPrepThreads / 64 - 1)]);
    int eq = 0;                      // activations are scaled by 2^eq: each below 2^40, a sum of 2^20 of them below 2^60
    if (m) {
        int e;
        frexpf(__uint_as_float(m), &e);
        eq = 40 - e;
    }
    int place = -1;                  // of the feature, in the thread that came first
    if (mine) {
        int i = (int)(((unsigned)f * 2654435761u) >> 21);                 // 0 .. kHash - 1
        for (;;) {                   // at most half of the places are taken
            const int was = atomicCAS(&name[i], -1, f);
            if (was == -1) place = i;
            if (was == -1 || was == f) break;
            i = (i + 1) & (kHash - 1);
        }
        atomicAdd(&sum[i], (unsigned long long)llrint((double)v * ldexp(1.0, eq)));
    }
    __syncthreads();
    double w = 0.0;
    if (place >= 0) {
        const unsigned long long sacc = sum[place];
        if (sacc && freq > 0 && !(a.max_freq > 0 && freq > a.max_freq))
            w = (double)sacc * ldexp(1.0, -eq) / ((double)logf(1.0f + (float)freq) + 1.0);
    }
    int tot;
    const int slot = s3_block_excl_scan<kPrepThreads>(w > 0.0 ? 1 : 0, wsum, tot);
    if (w > 0.0) a.act[(size_t)h * a.n_feat + slot] = ActiveList{w, f, 0};
    const unsigned long long mb = wave_max_u64((unsigned long long)__double_as_longlong(w));
    const int wp = s3_wave_incl_scan(w > 0.0 ? freq : 0);
    if (lane == 63) { wmx[wave] = mb; psum[wave] = wp; }
    __syncthreads();
    for (int r = tid; r < a.nr; r += kPrepThreads) {
        unsigned long long best = 0;
        int sum = 0;
        for (int q = 0; q < kPrepThreads / 64; ++q) { best = wmx[q] > best ? wmx[q] : best; sum += psum[q]; }
        a.wmax[h * a.nr + r] = r ? 0ull : best;
        a.nact[h * a.nr + r] = r ? 0 : tot;
        if (a.post) a.post[h * a.nr + r] = r ? 0 : sum >> 6;
    }
}

// Parts of a group's lists that are worth it, for a group with so many postings in a position block: one more saves gathering, about
// 0.27 ns a posting, and is one more array to write and to sum, 5 ps a position of all groups (as many as 4096, for the
// latency of few); a part has 1024 postings or more.
// The host knows how many lists there can be, not how long they are: it reckons as many as the square root of their share of the features
// would have of all postings, since queries name the features that many tokens have too (1 to 65 times the average list in 120 calls whose
// queries are encoded like their context), and with 64 lists a part or more.  The kernels know the lists, which may be few or none (queries
// without a match, max_freq), and leave workgroups idle that four times their postings are not worth.  That is 0.7 us in the way of the sums, so
// it is asked where the arrays have more than kArraysMost positions (179 queries of k 32 without a match, 13 heads of 28741
// positions: 33 us in one part, 60 with one for every 64 lists, 34 so).
// More time than with the best number of parts for each call: 120 calls whose queries are encoded like their context, a part for every 64
// lists 3.5 %, postings of average lists alone 4.4 % (up to a sixth), this 3.0 %; 432 whose queries name features at random 6.3, 2.4 and 3.6 %.
// us for a look-up, a part for every 64 lists / this: 16 queries of k 16 in 64 heads of 16384 positions 48 / 34, 100 in 16 heads 55 / 42; 300 of
// k 32 in one head 48 / 41; 2 in 1000 positions the gather 7.0 in six parts / 6.1 in one.
constexpr int kPartLists = 64;
constexpr int64_t kArraysMost = 1 << 20;
inline __host__ __device__ int parts_worth(float postings, int groups, int64_t L) {
    const int parts = (int)fminf(sqrtf(64.f * postings / ((float)groups * (float)(L > 4096 ? L : 4096))) + 0.5f, postings * (1.f / 1024.f));
    return parts > 1 ? parts : 1;
}

// Postings gather with the scores of one block of positions held in LDS.
// Workgroup (b, g) owns positions [b * pb, (b + 1) * pb) and the lists of group g: of some heads, or, where there are fewer heads than
// the chip wants workgroups, a part of the lists of one head.  (All heads' lists dealt to all groups: the workgroups meet more
// pages, 156 us instead of 116 for 64 heads of 65536 positions, compact.)  The workgroup adds the postings of its lists that fall into
// its block with LDS atomics (64-bit fixed point, so the order of the additions does not matter), then stores the block: into S
// when there is one group, else into that group's partial array, which the pooling kernel sums.  (Additions to one array per XCD, in
// its L2, instead: the pooling kernel has 8 arrays to sum instead of 128, 12 -> 5 us, but a workgroup's 16384 additions take 6 to 8 us.)
// 1024 lists at a time, a thread fetches weight and feature of a list and the part of the list that lies in the block (its
// segment) -- from the index's block table when there is one; else, for lists sorted by position, by a search; else the whole
// list, every posting filtered.  Postings are read as aligned vectors of four; the vectors of all the segments are numbered through,
// the wavefronts take 64 kFlight of them in turn, and lane l of load u has vector 64 u + l, whichever segment it belongs to: what
// is in flight bounds the rate, and this way every load is full and every wavefront has as much to do whatever the lengths are.
// us for the kernel, one segment a wavefront or some lanes at a time, heads alone as groups / batches of 64 lists
// a wavefront / now: 256 queries of k 128 in 32 heads of 14001 positions 426 / 80 / 65, 896 of k 64 in 112 of 16384 355 / 117 / 121, 256 of
// k 32 in 64 of 16384, skewed, 116 / 67 / 44, in 64 of 65536, compact, skewed, 116 / 113 / 87; 4 in 256 heads of 32768 39.5 / 40 / 32; a
// whole look-up of 5 queries in 64 heads of 97420 positions, skewed, 216 / 295 / 135.
constexpr int kScatterThreads = 1024;
constexpr int kFlight = 4;           // vector loads per lane in flight
constexpr int kPairs = 512;          // (head, range) pairs looked at together
constexpr int kNarrowMin = 128;      // sorted lists longer than this are narrowed to the position block by search
constexpr int kMaxPB = 1 << kS3PosBlockLog2;

// First index in [b, e) whose position is >= key (e if none); pos[b .. e) ascending.  Eight-way search: the seven
// pivots of a step are independent loads, so a list of n postings costs about log8(n) memory latencies.
__device__ __forceinline__ int lower_bound_pos(const int32_t* pos, int b, int e, int64_t key) {
    while (e - b > 8) {
        const int step = (e - b) >> 3;
        int32_t v[7];
#pragma unroll
        for (int u = 0; u < 7; ++u) v[u] = pos[b + (u + 1) * step];
        int c = 0;
#pragma unroll
        for (int u = 0; u < 7; ++u) c += (int64_t)v[u] < key ? 1 : 0;
        const int nb = c ? b + c * step + 1 : b;          // everything up to the last pivot below the key is below it
        if (c < 7) e = b + (c + 1) * step;                // the first pivot at or above the key bounds the answer
        b = nb;
    }
    int32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = b + u < e ? pos[b + u] : 0;
    int c = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) c += (b + u < e && (int64_t)v[u] < key) ? 1 : 0;
    return b + c;
}

// element j of a vector of four postings (int32: a 16-byte vector; uint16: an 8-byte one), as an unsigned position value
__device__ __forceinline__ unsigned vec_posting(const uint4& v, int j) {
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
    return w[j];
}
__device__ __forceinline__ unsigned vec_posting(const uint2& v, int j) {
    const unsigned w[2] = {v.x, v.y};
    return (w[j >> 1] >> ((j & 1) * 16)) & 0xFFFFu;
}

// A segment: vector v (of those numbered through) lies at base + v vectors, and element 4 v + j of it is the segment's if
// first <= 4 v + j < end.
struct Segment {
    uint64_t base;
    unsigned first, end;
};

// Where position p of the block lies in LDS: lanes that add four positions apart (vectors of a dense list) meet all banks.
__device__ __forceinline__ unsigned spread(unsigned p) { return p ^ ((p >> 5) & 3u); }

template <bool CMP>
__global__ __launch_bounds__(kScatterThreads) void sc_gather_kernel(ScoreArgs a) {
    using Posting = typename std::conditional<CMP, uint16_t, int32_t>::type;
    using Vec = typename std::conditional<CMP, uint2, uint4>::type;        // four postings
    constexpr int kW = kScatterThreads / 64;
    extern __shared__ __align__(16) unsigned long long sblk[];
    __shared__ unsigned long long wmx[kW];
    __shared__ Segment seg[kScatterThreads];
    __shared__ unsigned long long weight[kScatterThreads];
    __shared__ int start[kScatterThreads];                                 // the segments' first vectors
    __shared__ __align__(16) unsigned starts_all[kW][2 * kFlight];
    __shared__ int upto[kPairs];                                           // lists of the (head, range) pairs up to this one
    __shared__ int wsum[kW], wcnt[kW];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned* const starts = starts_all[wave];
    int unit, blk;                                                // the position blocks of a group share an XCD
    s3_block_to_tile(blockIdx.x, a.ngroup, a.npb, unit, blk);
    const int group = unit / a.parts, part = unit - group * a.parts;
    const int64_t p0 = (int64_t)blk * a.pb;
    const int64_t p1 = p0 + a.pb < a.L ? p0 + a.pb : a.L;
    const unsigned span = (unsigned)(p1 - p0);
    const unsigned pbase = CMP ? 0u : (unsigned)p0;               // what a stored posting is relative to
    const bool cmp_empty = CMP && blk >= a.nblk;                  // the compact index holds nothing beyond its blocks
    for (int i = tid; i < a.pb / 2; i += kScatterThreads) ((uint4*)sblk)[i] = make_uint4(0, 0, 0, 0);      // pb is a multiple of 64
    // the largest weight over all heads fixes the fixed-point scale (every workgroup derives the same one)
    unsigned long long mb = 0;
    int postings = 0;
    for (int i = tid; i < a.n_heads * a.nr; i += kScatterThreads) {
        const unsigned long long w = a.wmax[i];
        if (a.post) postings += a.post[i];
        mb = w > mb ? w : mb;
    }
    mb = wave_max_u64(mb);
    postings = s3_wave_incl_scan(postings);
    if (lane == 63) { wmx[wave] = mb; wcnt[wave] = postings; }
    const int nbk = a.nblk - 1;
    const int pair1 = min(a.n_heads, (group + 1) * a.heads_per) * a.nr;
    __syncthreads();
    mb = wmx[lane & (kW - 1)];
    mb = wave_max_u64(mb);
    if (blockIdx.x == 0 && tid == 0) a.wmax[a.n_heads * a.nr] = mb;      // for the kernels that follow
    int parts = a.parts;                                          // the same in every workgroup
    if (a.post) {
        const int groups = a.ngroup / a.parts;
        postings = __builtin_amdgcn_readlane(s3_row_incl_scan(wcnt[lane & (kW - 1)]), kW - 1);
        parts = min(a.parts, parts_worth(256.f * (float)postings / ((float)groups * (float)a.npb), groups, a.L));
        if (blockIdx.x == 0 && tid == 0) a.wmax[a.n_heads * a.nr + 1] = (unsigned long long)(groups * parts);
        if (part >= parts) return;
    }
    const double scale = ldexp(1.0, exp_s(mb, a.hb));

    // Adds w at the vector's postings that belong to the segment (`whole`: all do, in all lanes) and lie in the block.  Compact
    // postings are handled two in a register; what does not belong goes to a place of the lane's own behind the block.
    const unsigned pb = (unsigned)a.pb, nowhere = pb + lane;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned long long*)sblk;
    const auto add = [&](const Vec& v, bool whole, unsigned e0, unsigned first, unsigned end, unsigned long long w) {
        if constexpr (CMP) {                                      // two postings in a register: 16-bit operations on both
            typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
            unsigned q[2] = {v.x, v.y};
            if (!whole) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const unsigned e = e0 + 2 * j;
                    const unsigned keep = (e >= first && e < end ? 0xFFFFu : 0u) | (e + 1 >= first && e + 1 < end ? 0xFFFF0000u : 0u);
                    q[j] = (q[j] & keep) | (nowhere * 0x10001u & ~keep);
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const u16x2 most = {(unsigned short)(pb + 63), (unsigned short)(pb + 63)};
                const unsigned p = __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(u16x2, q[j]), most));
                const unsigned at = p ^ (p >> 5 & 0x00030003u);   // spread() of both
                unsigned a0, a1;                                  // 8 times either half and the block's place in LDS
                asm("v_mad_u32_u16 %0, %1, 8, %2 op_sel:[0,0,0,0]" : "=v"(a0) : "v"(at), "v"(lds0));
                asm("v_mad_u32_u16 %0, %1, 8, %2 op_sel:[1,0,0,0]" : "=v"(a1) : "v"(at), "v"(lds0));
                typedef __attribute__((address_space(3))) unsigned long long lds_u64;
                __hip_atomic_fetch_add((lds_u64*)(uintptr_t)a0, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add((lds_u64*)(uintptr_t)a1, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned rr = vec_posting(v, j) - pbase;
                if ((whole || (e0 + j >= first && e0 + j < end)) && rr < span) atomicAdd(&sblk[spread(rr)], w);
            }
        }
    };
    for (int pair0 = group * a.heads_per * a.nr; pair0 < pair1; pair0 += kPairs) {
        const int n_pairs = min(kPairs, pair1 - pair0), n_mine = tid < n_pairs ? a.nact[pair0 + tid] : 0;
        int lists;
        const int ahead = s3_block_excl_scan<kScatterThreads>(n_mine, wsum, lists);
        if (tid < kPairs) upto[tid] = ahead + n_mine;
        __syncthreads();
        const int list1 = (int)((int64_t)lists * (part + 1) / parts);      // this part's: [list0, list1)
        int list0 = (int)((int64_t)lists * part / parts);
        const auto pair_of = [&](int i) {                         // the pair that list i belongs to
            int q = 0;
            for (int s = kPairs / 2; s > 0; s >>= 1)
                if (q + s < n_pairs && upto[q + s - 1] <= i) q += s;
            return q;
        };
        int pair = 0;
        uint4 raw = make_uint4(0, 0, 0, 0);
        const auto ask = [&]() {                                  // a list's weight and feature
            const int i = list0 + tid;
            if (i >= list1) return;
            pair = n_pairs > 1 ? pair_of(i) : 0;
            const int hr = pair0 + pair, h = hr / a.nr;
            const int at = i - (pair ? upto[pair - 1] : 0);
            raw = *reinterpret_cast<const uint4*>(a.act + (size_t)h * a.n_feat + (size_t)(hr - h * a.nr) * kRange + at);
        };
        ask();
        while (list0 < list1) {
            // without a bound on the segments' lengths, the lists of one pair at a time: their vectors fit 32 bits
            const int here = a.mixed ? list1 : min(list1, upto[pair_of(list0)]), next = min(here, list0 + kScatterThreads);
            unsigned long long wf = 0;
            int b = 0, e = 0;
            uint64_t pos = 0;
            if (list0 + tid < next) {
                const int h = (pair0 + pair) / a.nr;
                const int32_t* off = CMP ? a.cstart + (size_t)h * a.cstart_stride + (size_t)blk * a.n_feat
                                         : a.offsets + (size_t)h * a.off_stride;
                const int32_t* tab = !CMP && a.btab ? a.btab + (size_t)h * a.n_feat * nbk : nullptr;
                pos = CMP ? (uint64_t)(uintptr_t)(a.delta + (size_t)h * a.delta_stride) : (uint64_t)(uintptr_t)(a.positions + (size_t)h * a.pos_stride);
                const double lw = __longlong_as_double((long long)(((unsigned long long)raw.y << 32) | raw.x));
                wf = (unsigned long long)llrint(lw * scale);
                if (wf) {
                    const int f = (int)raw.z;
                    if (CMP) {
                        if (!cmp_empty) {
                            b = off[f];
                            e = off[f + 1];
                        }
                    } else if (a.npb == 1) {
                        b = off[f];
                        e = off[f + 1];
                    } else if (tab) {         // blocks at or beyond the table's end hold nothing
                        const int lb = off[f], le = off[f + 1];
                        b = blk == 0 ? lb : (blk <= nbk ? tab[(size_t)f * nbk + blk - 1] : le);
                        e = blk < nbk ? tab[(size_t)f * nbk + blk] : le;
                        b = max(b, lb);       // whatever the table holds, nothing outside the list is read
                        e = min(e, le);
                    } else {
                        b = off[f];
                        e = off[f + 1];
                        if (a.sorted && e - b > kNarrowMin) {      // the first and the last block need one search
                            const int32_t* pl = a.positions + (size_t)h * a.pos_stride;
                            if (blk > 0) b = lower_bound_pos(pl, b, e, p0);
                            if (blk < a.npb - 1) e = lower_bound_pos(pl, b, e, p1);
                        }
                    }
                }
            }
            list0 = next;
            const unsigned n = wf ? (unsigned)max(e - b, 0) : 0u;
            const uint64_t at = pos + (uint64_t)(unsigned)b * sizeof(Posting);
            const unsigned skip = (unsigned)(at & (sizeof(Vec) - 1)) / (unsigned)sizeof(Posting);
            const int nv = n ? (int)((skip + n + 3) >> 2) : 0;
            const int vincl = s3_wave_incl_scan(nv);
            const unsigned long long some = __ballot(nv > 0);
            if (lane == 63) { wsum[wave] = vincl; wcnt[wave] = (int)__popcll(some); }
            __syncthreads();
            const int vs = s3_row_incl_scan(wsum[lane & (kW - 1)]), cs = s3_row_incl_scan(wcnt[lane & (kW - 1)]);
            const int total = __builtin_amdgcn_readlane(vs, kW - 1), n_seg = __builtin_amdgcn_readlane(cs, kW - 1);
            if (nv > 0) {
                const int v_at = (wave ? __builtin_amdgcn_readlane(vs, max(wave - 1, 0)) : 0) + vincl - nv;
                const int s = (wave ? __builtin_amdgcn_readlane(cs, max(wave - 1, 0)) : 0) +
                              (int)__builtin_amdgcn_mbcnt_hi((unsigned)(some >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)some, 0u));
                seg[s] = Segment{at - skip * sizeof(Posting) - (uint64_t)(unsigned)v_at * sizeof(Vec), 4u * (unsigned)v_at + skip, 4u * (unsigned)v_at + skip + n};
                weight[s] = wf;
                start[s] = v_at;
            }
            __syncthreads();
            ask();                                                // the next lists' are on their way beside the postings
            for (int v0 = wave * 64 * kFlight; v0 < total; v0 += kScatterThreads * kFlight) {
                // the segment that vector v0 belongs to: the last that starts at or before it
                const int x = lane * 16 + 15 < n_seg ? start[lane * 16 + 15] : 0x7FFFFFFF, j16 = (int)__popcll(__ballot(x <= v0)) * 16;
                const int y = j16 + (lane & 15) < n_seg ? start[j16 + (lane & 15)] : 0x7FFFFFFF;
                int before = j16 + (int)__popcll(__ballot(y <= v0) & 0xFFFFull) - 1;
                const int v1 = v0 + 64 * kFlight;
                if (v1 < total && !(before + 1 < n_seg && start[before + 1] <= v1)) {
                    // all of one segment that goes on behind: whole vectors, but perhaps the first
                    const Segment one = seg[before];
                    const unsigned long long w1 = weight[before];
                    Vec v[kFlight];
#pragma unroll
                    for (int u = 0; u < kFlight; ++u) v[u] = ((const Vec*)one.base)[v0 + u * 64 + lane];
                    add(v[0], 4u * (unsigned)v0 >= one.first, 4u * (unsigned)(v0 + lane), one.first, one.end, w1);
#pragma unroll
                    for (int u = 1; u < kFlight; ++u) add(v[u], true, 0u, 0u, 0u, w1);
                    continue;
                }
                // a bit for every vector of these at which a further segment starts; a vector's segment: starts at or before it
                s3_wave_fence();
                if (lane < 2 * kFlight) starts[lane] = 0;
                s3_wave_fence();
                for (int s = before + 1;; s += 64) {
                    const int at_v = s + lane < n_seg ? start[s + lane] : 0x7FFFFFFF;
                    if (at_v < v1) atomicOr(&starts[(at_v - v0) >> 5], 1u << ((at_v - v0) & 31));
                    if (__ballot(at_v < v1) != ~0ull) break;
                }
                s3_wave_fence();
                Segment sg[kFlight];
                Vec raw4[kFlight];
                unsigned long long w[kFlight];
#pragma unroll
                for (int u = 0; u < kFlight; ++u) {
                    const unsigned lo = starts[2 * u], hi = starts[2 * u + 1];
                    // starts at lanes 1 .. lane of this load, and at its lane 0
                    const int own = before + (int)(lo & 1u) + (int)__builtin_amdgcn_mbcnt_hi(hi >> 1, __builtin_amdgcn_mbcnt_lo((lo >> 1) | (hi << 31), 0u));
                    before += (int)__popc(lo) + (int)__popc(hi);
                    sg[u] = seg[own];
                    w[u] = weight[own];
                }
#pragma unroll
                for (int u = 0; u < kFlight; ++u) {
                    const int v = v0 + u * 64 + lane;
                    raw4[u] = ((const Vec*)sg[u].base)[v < total ? v : (int)(sg[u].first >> 2)];
                    if (v >= total) sg[u].end = 0;
                }
#pragma unroll
                for (int u = 0; u < kFlight; ++u) add(raw4[u], false, 4u * (unsigned)(v0 + u * 64 + lane), sg[u].first, sg[u].end, w[u]);
            }
            __syncthreads();                                      // the segments are read
        }
    }
    __syncthreads();
    unsigned long long* const dst = (a.ngroup > 1 ? a.part + ((size_t)group * parts + part) * a.L : a.sfix) + p0;
    for (unsigned i = tid; i < span; i += kScatterThreads) dst[i] = sblk[spread(i)];
}

// The wavefront's best window, in every lane: largest key (sum + 1; 0: none), ties -> smallest start.
__device__ __forceinline__ void wave_best(unsigned long long& key, int& start) {
    const unsigned hi = s3_wave_max_u32((unsigned)(key >> 32));
    const unsigned lo = s3_wave_max_u32((unsigned)(key >> 32) == hi ? (unsigned)key : 0u);
    const unsigned long long best = ((unsigned long long)hi << 32) | lo;
    start = (int)~s3_wave_max_u32(key == best ? ~(unsigned)start : 0u);
    key = best;
}

// Partial arrays that the gather wrote.
__device__ __forceinline__ int arrays_of(const ScoreArgs& a) {
    return a.post ? __builtin_amdgcn_readfirstlane((int)a.wmax[a.n_heads * a.nr + 1]) : a.ngroup;
}

// S = sum of the groups' partial arrays, where the pooling kernel does not sum them itself (score_run).  64 positions per workgroup,
// whose wavefronts (four, or sixteen for many arrays) take the arrays in turn, eight loads in flight per thread: with few positions
// it is the chain of a wavefront's loads that takes the time (256 arrays of 5115 positions 11.3 us with four wavefronts and two loads, 5.2 now).
constexpr int kReduceFew = 32;
__global__ __launch_bounds__(1024) void sc_reduce_kernel(ScoreArgs a) {
    __shared__ unsigned long long partial[16][64];
    constexpr int U = 8;
    const int p = threadIdx.x & 63, q = threadIdx.x >> 6, nw = blockDim.x >> 6, n = arrays_of(a);
    const int64_t t = (int64_t)blockIdx.x * 64 + p, at = t < a.L ? t : a.L - 1;
    unsigned long long sum = 0;
    for (int g = q; g < n; g += U * nw) {
        unsigned long long v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = a.part[(size_t)min(g + u * nw, n - 1) * a.L + at];
#pragma unroll
        for (int u = 0; u < U; ++u) sum += g + u * nw < n ? v[u] : 0ull;
    }
    partial[q][p] = sum;
    __syncthreads();
    if (q == 0 && t < a.L) {
        for (int w = 1; w < nw; ++w) sum += partial[w][p];
        a.sfix[t] = sum;
    }
}

// Inclusive prefix sum of one 64-bit value per thread over the block (wrap-around arithmetic: exact differences).
template <int NT>
__device__ __forceinline__ unsigned long long block_incl_scan_u64(unsigned long long v, unsigned long long* wsum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int lo = (unsigned int)__shfl_up((int)(unsigned int)v, o);
        const unsigned int hi = (unsigned int)__shfl_up((int)(unsigned int)(v >> 32), o);
        if (lane >= o) v += ((unsigned long long)hi << 32) | lo;
    }
    if (lane == 63) wsum[wave] = v;
    __syncthreads();
    unsigned long long base = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) base += w < wave ? wsum[w] : 0ull;
    __syncthreads();
    return v + base;
}

// Sum of the groups, span pooling, the fp32 scores, and the best window of every 2^sublog windows (one workgroup per a.tile
// windows).  The tile's positions are summed over the groups' arrays into LDS and turned into prefix sums there, so a window costs two
// LDS reads whatever its length: W[s] = P[s + len - 1] - P[s - 1], exact in 64-bit integers.  Larger value wins, ties ->
// smaller start.  What bounds it is a chain of memory, LDS and barrier latencies, so tiles are short where they are few: down to
// kTilesMost of them or 256 windows, but no shorter than a window.  Longer ones for 1000000 positions: look-up of 2 queries in one
// head 88 -> 39 us (tiles of 256), 300000: 33 -> 30.5 (at most 256 tiles instead of 128).
// The positions of a tile's last windows lie beyond it and are summed twice.  So where the groups' arrays are many and windows long
// (together more than kSumMost positions a tile), sc_reduce_kernel sums them first.  us for a look-up, sums here / by it: 256 arrays,
// windows of 64 44 / 45, 256 50 / 46, 1024 92 / 46, 4096 206 / 46; 16 arrays, 256 29.4 / 30.1, 1024 32.1 / 30.4; 4 arrays, 1024 25.2 / 25.7.
constexpr int kPoolThreads = 1024;
constexpr int kPoolMaxLen = 4096;      // longer windows take sc_pool_wide_kernel
constexpr int kTilesMost = 128;
constexpr int64_t kSumMost = 16384;

__global__ __launch_bounds__(kPoolThreads) void sc_pool_kernel(ScoreArgs a) {
    extern __shared__ unsigned long long pre[];          // [tile + len - 1] prefix sums
    __shared__ unsigned long long wsum[kPoolThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kW = kPoolThreads / 64;
    const double inv = ldexp(1.0, -exp_s(a.wmax[a.n_heads * a.nr], a.hb));
    const int64_t s0 = (int64_t)blockIdx.x * a.tile;
    const int64_t tend = (int)blockIdx.x == a.ntile - 1 ? a.L : s0 + a.tile;      // positions whose fp32 score this tile writes
    const int n_in = (int)(min(a.L, s0 + a.tile + a.len - 1) - s0);               // positions the tile's windows read
    const int nsum = a.nsum == 1 ? 1 : arrays_of(a);
    if (nsum == 1) {
        const unsigned long long* const src = a.nsum == 1 ? a.sfix : a.part;
        constexpr int kBatch = 4;                        // coalesced loads in flight per thread
        for (int i0 = tid; i0 < n_in; i0 += kBatch * kPoolThreads) {
            unsigned long long v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) v[u] = i0 + u * kPoolThreads < n_in ? src[s0 + i0 + u * kPoolThreads] : 0ull;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int i = i0 + u * kPoolThreads;
                if (i >= n_in) continue;
                pre[i] = v[u];
                if (a.scores_out && s0 + i < tend) a.scores_out[s0 + i] = (float)((double)v[u] * inv);
            }
        }
    } else {
        // a wavefront sums a share of the groups for 64 positions, sixteen loads in flight per lane
        constexpr int kSum = 16;
        const int chunks = (n_in + 63) >> 6, shares = max(1, min(kW / chunks, (nsum + kSum - 1) / kSum));
        if (shares > 1) {
            for (int i = tid; i < n_in; i += kPoolThreads) pre[i] = 0;
            __syncthreads();
        }
        for (int c = wave; c < chunks * shares; c += kW) {
            const int i = (c % chunks) * 64 + lane, g0 = nsum * (c / chunks) / shares, g1 = nsum * (c / chunks + 1) / shares;
            if (i >= n_in) continue;
            unsigned long long sum = 0;
            const auto take = [&](int g, auto n) {
                unsigned long long v[n];
#pragma unroll
                for (int u = 0; u < n; ++u) v[u] = a.part[(size_t)min(g + u, g1 - 1) * a.L + s0 + i];
#pragma unroll
                for (int u = 0; u < n; ++u) sum += g + u < g1 ? v[u] : 0ull;
            };
            int g = g0;
            for (; g + kSum / 2 < g1; g += kSum) take(g, std::integral_constant<int, kSum>());
            for (; g < g1; g += kSum / 4) take(g, std::integral_constant<int, kSum / 4>());
            if (shares > 1) atomicAdd(&pre[i], sum);
            else pre[i] = sum;
        }
    }
    __syncthreads();
    // each thread sums its own run, the block scans the run totals, the thread writes its run's prefixes
    const int per = (n_in + kPoolThreads - 1) / kPoolThreads;                     // consecutive positions per thread
    unsigned long long run = 0;
    for (int j = 0; j < per; ++j) {
        const int i = tid * per + j;
        if (i < n_in) {
            run += pre[i];
            if (nsum > 1 && a.scores_out && s0 + i < tend) a.scores_out[s0 + i] = (float)((double)pre[i] * inv);
        }
    }
    unsigned long long sum = block_incl_scan_u64<kPoolThreads>(run, wsum) - run;
    for (int j = 0; j < per; ++j) {
        const int i = tid * per + j;
        if (i < n_in) {
            sum += pre[i];
            pre[i] = sum;
        }
    }
    __syncthreads();
    for (int b = wave; a.sublog == 6 && b < a.tile / 64; b += kW) {
        const int i = b * 64 + lane;
        if (s0 + b * 64 >= a.nW) return;
        unsigned long long w = 0;
        if (s0 + i < a.nW) {
            const unsigned long long v = pre[i + a.len - 1] - (i ? pre[i - 1] : 0ull);
            a.wfix[s0 + i] = (long long)v;
            w = v + 1;
        }
        const unsigned top = s3_wave_max_u32((unsigned)(w >> 32));
        unsigned long long m = __ballot((unsigned)(w >> 32) == top);
        s3greedy::settle(w, top, m);                                              // ties -> the first lane, the smaller start
        const int e = (int)blockIdx.x * (a.tile / 64) + b, lead = (int)__builtin_ctzll(m);
        if (lane == lead) { a.tmaxv[e] = w; a.tmaxi[e] = (int)(s0 + i); }
    }
    if (a.sublog == 6) return;
    for (int q = wave; q < a.tile / kSubW; q += kW) {
        const int sub = (int)blockIdx.x * (a.tile / kSubW) + q;
        if (s0 + q * kSubW >= a.nW) break;
        unsigned long long key = 0;
        int start = 0x7FFFFFFF;
#pragma unroll
        for (int u = 0; u < kSubW / 64; ++u) {                                    // ascending starts per lane
            const int i = q * kSubW + u * 64 + lane;
            if (s0 + i < a.nW) {
                const unsigned long long w = pre[i + a.len - 1] - (i ? pre[i - 1] : 0ull);
                a.wfix[s0 + i] = (long long)w;
                if (w + 1 > key) { key = w + 1; start = (int)(s0 + i); }
            }
        }
        wave_best(key, start);
        if (lane == 0) { a.tmaxv[sub] = key; a.tmaxi[sub] = start; }
    }
}

// The same for windows longer than kPoolMaxLen: sliding sums from global memory, one wavefront per tile.
__global__ __launch_bounds__(256) void sc_pool_wide_kernel(ScoreArgs a) {
    const double inv = ldexp(1.0, -exp_s(a.wmax[a.n_heads * a.nr], a.hb));
    if (a.scores_out)
        for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < a.L; t += (int64_t)gridDim.x * 256)
            a.scores_out[t] = (float)((double)a.sfix[t] * inv);
    const int lane = threadIdx.x & 63;
    const int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (tile >= a.ntile) return;
    const int64_t s0 = tile * kTileW + (int64_t)lane * kRun;
    unsigned long long key = 0;
    int start = 0x7FFFFFFF;
    if (s0 < a.nW) {
        unsigned long long acc = 0;
        for (int t = 0; t < a.len; ++t) acc += a.sfix[s0 + t];
        a.wfix[s0] = (long long)acc;
        key = acc + 1;
        start = (int)s0;
        for (int j = 1; j < kRun && s0 + j < a.nW; ++j) {
            acc += a.sfix[s0 + j + a.len - 1] - a.sfix[s0 + j - 1];
            a.wfix[s0 + j] = (long long)acc;
            if (acc + 1 > key) { key = acc + 1; start = (int)(s0 + j); }
        }
    }
    const int share = (1 << a.sublog) / kRun;             // lanes that share one entry of the tile maxima
    for (int o = share / 2; o > 0; o >>= 1) {
        const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)key, o), hi = (unsigned)__shfl_xor((int)(unsigned)(key >> 32), o);
        const unsigned long long other = ((unsigned long long)hi << 32) | lo;
        const int os = __shfl_xor(start, o);
        if (other > key || (other == key && os < start)) { key = other; start = os; }
    }
    const int64_t sub = tile * (64 / share) + lane / share;
    if (lane % share == 0 && sub < a.nsub) { a.tmaxv[sub] = key; a.tmaxi[sub] = start; }
}

// Greedy Top-B with optional suppression of overlapping windows.  The rounds depend on each other, so what bounds it is
// the latency of a round.
//
// sc_topb_rounds_kernel, sc_topb_slots_kernel: the blocks of 64 windows that the choices can lie in are brought into LDS (greedy.h),
// for up to kTopSlots such blocks.  The first takes all choices that do not depend on each other at once, the second (few
// windows suppressed by each, or none) one a round, by one wavefront.
// The others, for more: one wavefront walks the rounds without a barrier, with maxima of blocks of 256 windows in its registers.
// A round takes the best, clears the tiles that the suppression covers whole and searches the two blocks of kSubW windows at its
// ends again, loads of both in flight together.  A window that is gone is marked -1 in memory; window s belongs to lane s % 64 in
// every round, so a lane only ever reads back its own marks.  A tile without live windows stays so (its windows need not be marked).
//
// sc_topb_kernel: the registers hold the maxima of up to kTopRegs * 64 tiles of one block.
// sc_topb_long_kernel: tile maxima in LDS, those of groups of 64 tiles in registers, so that a round costs the same at any
// length; the groups at both ends are reduced again in the next round, beside its search and not behind this one's.  Beyond
// kTopTiles blocks a tile has several; their maxima come from memory beside the windows, block e belongs to the same lane in
// every round, too.
//
// us for a whole look-up of 8 queries in two indexes, with these two / with blocks in LDS: 16 spans of 64, 8000 positions 48 / 27,
// 300000 59 / 37, 1000000 73 / 49; 64 spans of 64, 8000 positions 128 / 31, 300000 160 / 44; in 32768 positions 16 spans of 8 45 / 28, of
// 256 51 / 36, of 64 that may overlap 42 / 32.
// The line between these two, 16 spans: 65536 positions take 51 us in 4 registers, 57 in groups; with 8 registers 131072
// take 55.5 instead of 56.5, but 32768 take 56 instead of 51.
struct TopBest {
    unsigned long long key;                               // window sum + 1; 0: none
    int start;
};
constexpr int kTopNone = 0x7FFFFFFF;
__device__ __forceinline__ void top_take(TopBest& b, const TopBest& o) {
    if (o.key > b.key || (o.key == b.key && o.start < b.start)) b = o;
}

// The best live windows of the blocks of kSubW windows that hold windows lo and hi, after [lo, hi] is marked.
__device__ __forceinline__ void top_search_ends(const ScoreArgs& a, int64_t lo, int64_t hi, int lane, TopBest& l, TopBest& h) {
    constexpr int U = kSubW / 64;
    const int64_t b0 = (lo >> kSubLog2 << kSubLog2) + lane, b1 = (hi >> kSubLog2 << kSubLog2) + lane;
    long long w0[U], w1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        w0[u] = b0 + u * 64 < a.nW ? a.wfix[b0 + u * 64] : -1;
        w1[u] = b1 + u * 64 < a.nW ? a.wfix[b1 + u * 64] : -1;
    }
    l = h = TopBest{0, kTopNone};
#pragma unroll
    for (int u = 0; u < U; ++u) {                         // one store per window and round where the blocks are one: the same mark
        const int64_t p0 = b0 + u * 64, p1 = b1 + u * 64;
        if (p0 >= lo && p0 <= hi) { w0[u] = -1; a.wfix[p0] = -1; }
        if (p1 >= lo && p1 <= hi) { w1[u] = -1; a.wfix[p1] = -1; }
        const unsigned long long k0 = (unsigned long long)(w0[u] + 1), k1 = (unsigned long long)(w1[u] + 1);
        if (k0 > l.key) { l.key = k0; l.start = (int)p0; }
        if (k1 > h.key) { h.key = k1; h.start = (int)p1; }
    }
    wave_best(l.key, l.start);
    wave_best(h.key, h.start);
}

__device__ __forceinline__ void top_finish(const ScoreArgs& a, int found, int lane) {
    for (int r = found + lane; r < a.top_b; r += 64) { a.span_start[r] = -1; a.span_score[r] = 0.f; }
    if (lane == 0) a.n_found[0] = found;
}

__global__ __launch_bounds__(64) void sc_topb_kernel(ScoreArgs a) {
    const int lane = threadIdx.x;
    TopBest t[kTopRegs];
#pragma unroll
    for (int q = 0; q < kTopRegs; ++q) {
        t[q] = TopBest{0, kTopNone};
        if (q * 64 + lane < a.nsub) t[q] = TopBest{a.tmaxv[q * 64 + lane], a.tmaxi[q * 64 + lane]};
    }
    const double inv = ldexp(1.0, -exp_s(a.wmax[a.n_heads * a.nr], a.hb));
    const int reach = a.nms ? a.len - 1 : 0;              // windows within `reach` of a chosen start are gone
    int found = 0;
    while (found < a.top_b) {
        TopBest best = t[0];
#pragma unroll
        for (int q = 1; q < kTopRegs; ++q) top_take(best, t[q]);
        wave_best(best.key, best.start);
        if (best.key == 0) break;
        if (lane == 0) {
            a.span_start[found] = best.start;
            a.span_score[found] = (float)((double)(long long)(best.key - 1) * inv);
        }
        ++found;
        const int64_t lo = max((int64_t)0, (int64_t)best.start - reach), hi = min(a.nW - 1, (int64_t)best.start + reach);
        const int tl = (int)(lo >> kSubLog2), th = (int)(hi >> kSubLog2);
        TopBest l, h;
        top_search_ends(a, lo, hi, lane, l, h);
#pragma unroll
        for (int q = 0; q < kTopRegs; ++q) {
            const int i = q * 64 + lane;
            if (i > tl && i < th) t[q].key = 0;
            if (i == tl && t[q].key) t[q] = l;
            if (i == th && t[q].key) t[q] = h;            // the same where tl == th
        }
    }
    top_finish(a, found, lane);
}

__global__ __launch_bounds__(kTopThreads) void sc_topb_long_kernel(ScoreArgs a) {
    __shared__ unsigned long long cv[kTopTiles], gv[64];
    __shared__ int ci[kTopTiles], gi[64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = 1 << a.topshift, nt = (a.nsub + per - 1) >> a.topshift, ng = (nt + 63) >> 6;
    for (int g = wave; g < ng; g += kTopThreads / 64) {
        const int t = g * 64 + lane;
        TopBest b{0, kTopNone};
        if (t < nt) {
            const int64_t e0 = (int64_t)t << a.topshift, e1 = min((int64_t)a.nsub, e0 + per);
            int64_t at = e0;
            for (int64_t e = e0; e < e1; ++e) {           // ascending starts
                const unsigned long long v = a.tmaxv[e];
                if (v > b.key) { b.key = v; at = e; }
            }
            if (b.key) b.start = a.tmaxi[at];
            cv[t] = b.key;
            ci[t] = b.start;
        }
        wave_best(b.key, b.start);
        if (lane == 0) { gv[g] = b.key; gi[g] = b.start; }
    }
    __syncthreads();
    if (tid >= 64) return;
    const double inv = ldexp(1.0, -exp_s(a.wmax[a.n_heads * a.nr], a.hb));
    const int tlog = kSubLog2 + a.topshift;
    const int reach = a.nms ? a.len - 1 : 0;              // windows within `reach` of a chosen start are gone
    TopBest top{lane < ng ? gv[lane] : 0ull, lane < ng ? gi[lane] : kTopNone};      // this lane's group; none while its tiles are in va / vb
    TopBest va{0, kTopNone}, vb{0, kTopNone};                   // tiles of the groups ga, gb, which changed last
    int ga = -1, gb = -1, found = 0;
    while (found < a.top_b) {
        TopBest best = top, ma = va, mb = vb;
        top_take(best, va);
        top_take(best, vb);
        wave_best(best.key, best.start);
        wave_best(ma.key, ma.start);                      // beside the reduction above, not behind it
        wave_best(mb.key, mb.start);
        if (lane == ga) top = ma;
        if (lane == gb) top = mb;
        if (best.key == 0) break;
        if (lane == 0) {
            a.span_start[found] = best.start;
            a.span_score[found] = (float)((double)(long long)(best.key - 1) * inv);
        }
        ++found;
        const int64_t lo = max((int64_t)0, (int64_t)best.start - reach), hi = min(a.nW - 1, (int64_t)best.start + reach);
        const int tl = (int)(lo >> tlog), th = (int)(hi >> tlog);
        const int64_t el = lo >> kSubLog2, eh = hi >> kSubLog2;
        for (int t = tl + 1 + lane; t < th; t += 64) cv[t] = 0;
        s3_wave_fence();                                  // the cleared tiles are read by other lanes
        ga = tl >> 6;
        gb = th >> 6;
        if (lane >= ga && lane <= gb) top = TopBest{0, kTopNone};
        va = vb = TopBest{0, kTopNone};
        const int la = ga * 64 + lane, lb = gb * 64 + lane;
        if (la < nt) va = TopBest{cv[la], ci[la]};
        if (lb < nt) vb = TopBest{cv[lb], ci[lb]};
        TopBest l, h;
        top_search_ends(a, lo, hi, lane, l, h);
        if (a.topshift) {                                 // from the two blocks to their tiles
            TopBest nl{0, kTopNone}, nh{0, kTopNone};
            for (int s = lane; s < per; s += 64) {
                const int64_t e0 = ((int64_t)tl << a.topshift) + s, e1 = ((int64_t)th << a.topshift) + s;
                unsigned long long v0 = e0 < a.nsub ? a.tmaxv[e0] : 0ull, v1 = e1 < a.nsub ? a.tmaxv[e1] : 0ull;
                int i0 = e0 < a.nsub ? a.tmaxi[e0] : kTopNone, i1 = e1 < a.nsub ? a.tmaxi[e1] : kTopNone;
                if (v0 && e0 >= el && e0 <= eh) {         // a block without live windows stays so
                    v0 = e0 == el ? l.key : (e0 == eh ? h.key : 0ull);
                    i0 = e0 == el ? l.start : h.start;
                    a.tmaxv[e0] = v0;
                    a.tmaxi[e0] = i0;
                }
                if (v1 && e1 >= el && e1 <= eh) {         // where tl == th: the same block, the same values
                    v1 = e1 == eh ? h.key : (e1 == el ? l.key : 0ull);
                    i1 = e1 == eh ? h.start : l.start;
                    a.tmaxv[e1] = v1;
                    a.tmaxi[e1] = i1;
                }
                top_take(nl, TopBest{v0, i0});
                top_take(nh, TopBest{v1, i1});
            }
            wave_best(nl.key, nl.start);
            wave_best(nh.key, nh.start);
            l = nl;
            h = nh;
        }
        // a tile without live windows stays so
        const unsigned long long tv = cv[tl], uv = cv[th];
        if (!tv) l = TopBest{0, kTopNone};
        if (!uv) h = TopBest{0, kTopNone};
        s3_wave_fence();                                  // va, vb, tv and uv are read
        if (lane == 0) {                                  // the same values where tl == th
            cv[tl] = l.key;
            ci[tl] = l.start;
            cv[th] = h.key;
            ci[th] = h.start;
        }
        s3_wave_fence();
        if (la == tl) va = l;
        if (la == th) va = h;
        if (lb == tl) vb = l;
        if (lb == th) vb = h;
    }
    top_finish(a, found, lane);
}

// The blocks' maxima and their windows, P a thread, and with them the slots.
template <int P>
__device__ __forceinline__ void top_fill(const ScoreArgs& a, const s3greedy::Slots<unsigned long long>& slots) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per = P == 1 ? 1 : s3greedy::per_thread(a.nsub);
    unsigned long long key[P];
    int at[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const int b = q < per ? (wave * per + q) * 64 + lane : a.nsub;
        key[q] = b < a.nsub ? a.tmaxv[b] : 0ull;
        at[q] = b < a.nsub ? a.tmaxi[b] : 0;
    }
    s3greedy::fill<unsigned long long, P>(slots, key, at, a.need, a.nW, [&](int64_t w) { return a.wfix[w]; },
                                          [](long long w) { return (unsigned long long)(w + 1); });
}

template <int P, int C>                                // maxima per thread, slots
__global__ __launch_bounds__(s3greedy::kThreads) void sc_topb_rounds_kernel(ScoreArgs a) {
    extern __shared__ __align__(16) unsigned long long top_lds[];
    const auto slots = s3greedy::slots_of<unsigned long long>(top_lds, C);
    unsigned long long* const list_key = (unsigned long long*)((char*)top_lds + s3greedy::lds_bytes<unsigned long long>(C));
    const double inv = ldexp(1.0, -exp_s(a.wmax[a.n_heads * a.nr], a.hb));
    top_fill<P>(a, slots);
    const int found = s3greedy::rounds<C, unsigned long long>(slots, list_key, (int*)(list_key + a.room), (unsigned)a.nW, (unsigned)(a.len - 1), a.top_b,
                                                              [&](int r, unsigned long long k, int w) {
        a.span_start[r] = w;
        a.span_score[r] = (float)((double)(long long)(k - 1) * inv);
    });
    if (threadIdx.x < 64) top_finish(a, found, threadIdx.x);
}

template <int P, int R>                                // maxima per thread, slots per lane
__global__ __launch_bounds__(s3greedy::kThreads) void sc_topb_slots_kernel(ScoreArgs a) {
    extern __shared__ __align__(16) unsigned long long top_lds[];
    const int lane = threadIdx.x & 63;
    const auto slots = s3greedy::slots_of<unsigned long long>(top_lds, 64 * R);
    const double inv = ldexp(1.0, -exp_s(a.wmax[a.n_heads * a.nr], a.hb));
    top_fill<P>(a, slots);
    if (threadIdx.x >= 64) return;
    unsigned long long left;
    int left_at;
    const int found = s3greedy::walk<R, unsigned long long>(slots, (unsigned)a.nW, a.nms ? (unsigned)(a.len - 1) : 0u, a.top_b, left, left_at,
                                                            [&](int r, unsigned long long k, int w) {
        if (lane == 0) {
            a.span_start[r] = w;
            a.span_score[r] = (float)((double)(long long)(k - 1) * inv);
        }
    }, [](int, unsigned long long, int) { return false; });
    top_finish(a, found, lane);
}

// Scratch of a call.  `full`: what the entry points ask for, room for kGroups workgroups' partial sums of a position block and for the
// maxima of blocks of 64 windows; it does not shrink for longer contexts, more heads or more features.  Else the least that a call
// takes, as much as one did before a head's lists were shared by several workgroups: heads in groups, maxima of 256 windows.
struct Layout {
    size_t wmax, nact, post, sfix, wfix, tmaxv, tmaxi, part, act, total;
    int nr, pb, npb, heads_per, parts, ngroup;   // feature ranges per head; position blocks, heads of a group, parts and groups at most of the gather
    bool full;
};
constexpr int kGroups = 256;

Layout layout(int n_heads, int n_feat, int64_t L, bool full) {
    Layout l;
    l.full = full;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += s3_align(bytes); return at; };
    const int64_t nW_max = L;
    const size_t nsub = full ? (size_t)(nW_max + 63) / 64 : (size_t)(nW_max + kSubW - 1) / kSubW;
    l.nr = (n_feat + kRange - 1) / kRange;
    l.wmax = take(((size_t)n_heads * l.nr + (full ? 2 : 1)) * 8);
    l.nact = take((size_t)n_heads * l.nr * 4);
    l.post = full ? take((size_t)n_heads * l.nr * 4) : 0;
    l.sfix = take((size_t)L * 8);
    l.wfix = take((size_t)L * 8);
    l.tmaxv = take(nsub * 8);
    l.tmaxi = take(nsub * 4);
    // position blocks of at most kMaxPB scores (128 KB of LDS); enough groups for about one workgroup per compute unit
    l.pb = (int)(L < kMaxPB ? (L + 63) / 64 * 64 : kMaxPB);
    l.npb = (int)((L + l.pb - 1) / l.pb);
    const int want = kGroups / l.npb < 1 ? 1 : kGroups / l.npb, groups = n_heads < want ? n_heads : want;
    l.heads_per = (n_heads + groups - 1) / groups;
    l.parts = full ? want / groups : 1;
    l.ngroup = (n_heads + l.heads_per - 1) / l.heads_per * l.parts;
    l.part = o;
    if (full) l.part = take((size_t)kGroups * (L < kMaxPB ? L : kMaxPB) * 8);      // ngroup <= kGroups / npb arrays of L
    else if (l.ngroup > 1) l.part = take((size_t)l.ngroup * L * 8);
    l.act = take((size_t)n_heads * n_feat * sizeof(ActiveList));
    l.total = o;
    return l;
}

// What a scoring call reads from: the plain index (CSR + block table) or the compact one.
struct ScoreSource {
    int n_heads, n_feat, k;
    int64_t tokens;
    bool sorted;
    const int32_t* offsets = nullptr; const int32_t* positions = nullptr; int64_t off_stride = 0, pos_stride = 0;
    const int32_t* btab = nullptr; int nblk = 1;
    const uint16_t* delta = nullptr; const int32_t* cstart = nullptr; const int32_t* cfreq = nullptr;
    int64_t delta_stride = 0, cstart_stride = 0;
};

static int score_run(const char* who, const ScoreSource& v, const int32_t* qids, const float* qvals, int nq,
                     int64_t n_positions, int span_len, int top_b, int32_t max_freq, int nms, float* scores_out,
                     int32_t* span_start, float* span_score, int32_t* n_found, void* ws, size_t ws_bytes, void* stream) {
    if (!span_start || !span_score || !n_found || !ws) return s3_fail(S3_EINVAL, "%s: null pointer", who);
    if (nq < 0 || (nq > 0 && (!qids || !qvals))) return s3_fail(S3_EINVAL, "%s: bad query arrays", who);
    if (span_len < 1 || top_b < 1 || top_b > 1024)
        return s3_fail(S3_EINVAL, "%s: span_len %d (>= 1) / top_b %d (1..1024) out of range", who, span_len, top_b);
    if (n_positions < 1 || n_positions >= (1LL << 31))
        return s3_fail(S3_EINVAL, "%s: n_positions %lld out of range", who, (long long)n_positions);
    ScoreArgs a;
    a.n_heads = v.n_heads; a.n_feat = v.n_feat; a.k = v.k;
    a.offsets = v.offsets; a.off_stride = v.off_stride; a.positions = v.positions; a.pos_stride = v.pos_stride;
    a.btab = v.btab; a.nblk = v.nblk;
    a.delta = v.delta; a.cstart = v.cstart; a.cfreq = v.cfreq; a.delta_stride = v.delta_stride; a.cstart_stride = v.cstart_stride;
    if ((int64_t)nq * a.k > (1 << 20)) return s3_fail(S3_EINVAL, "%s: nq * k %lld > 2^20", who, (long long)nq * a.k);
    Layout l = layout(a.n_heads, a.n_feat, n_positions, true);
    if (ws_bytes < l.total) l = layout(a.n_heads, a.n_feat, n_positions, false);
    if (ws_bytes < l.total) return s3_fail(S3_ECAPACITY, "%s: workspace %zu < %zu bytes", who, ws_bytes, l.total);
    if ((uintptr_t)ws & 255) return s3_fail(S3_EINVAL, "%s: workspace must be 256-byte aligned", who);

    char* base = (char*)ws;
    a.qids = qids; a.qvals = qvals; a.nq = nq;
    a.L = n_positions;
    a.len = (int)(span_len < n_positions ? span_len : n_positions);
    a.nW = n_positions - a.len + 1;
    a.top_b = top_b; a.nms = nms ? 1 : 0; a.max_freq = max_freq;
    // Headroom of the 64-bit fixed point: a position sums at most n_heads * k weights, a window at most span_len
    // positions; four more bits are spare.  Weights keep 62 - hb significant bits below the largest one.
    a.hb = s3_ceil_log2((unsigned)(a.n_heads * a.k)) + s3_ceil_log2((unsigned)a.len) + 4;
    if (a.hb > 40)
        return s3_fail(S3_EINVAL, "%s: n_heads * k * span_len too large for the 64-bit fixed-point sums "
                                  "(log2 of it, rounded up per factor, must be <= 36)", who);
    a.nr = l.nr;
    a.wmax = (unsigned long long*)(base + l.wmax);
    a.nact = (int*)(base + l.nact);
    a.sfix = (unsigned long long*)(base + l.sfix);
    a.act = (ActiveList*)(base + l.act);
    a.wfix = (long long*)(base + l.wfix);
    a.tmaxv = (unsigned long long*)(base + l.tmaxv);
    a.tmaxi = (int*)(base + l.tmaxi);
    a.part = (unsigned long long*)(base + l.part);
    a.pb = l.pb; a.npb = l.npb; a.sorted = v.sorted ? 1 : 0;
    const int groups = l.ngroup / l.parts;
    const int64_t pairs = (int64_t)nq * a.k, named = pairs < a.n_feat ? pairs : (int64_t)a.n_feat, most = l.heads_per * named / kPartLists;
    const double postings = l.heads_per * (double)v.tokens * a.k * sqrt((double)named / a.n_feat) / l.npb;
    int parts = parts_worth((float)postings, groups, a.L);
    if (parts > most) parts = most > 1 ? (int)most : 1;
    a.heads_per = l.heads_per;
    a.parts = parts < l.parts ? parts : l.parts;
    a.ngroup = groups * a.parts;
    a.post = a.parts > 1 && (int64_t)a.ngroup * a.L > kArraysMost ? (int*)(base + l.post) : nullptr;
    // The elements of 1024 segments are numbered in 32 bits.  A segment is at most a block of the compact index or of the block table,
    // else a whole list, which an id that stands in a row more than once makes longer than there are tokens.
    a.mixed = v.delta || (v.btab && l.npb > 1) || (v.tokens < (1 << 20) && (int64_t)l.heads_per * v.tokens * a.k < (1LL << 31)) ? 1 : 0;
    // sc_pool_kernel: its tiles, and whether the groups' arrays are summed before it
    a.tile = kTileW;
    while (a.tile > 256 && a.tile >= 2 * a.len && (a.nW + a.tile - 1) / a.tile < kTilesMost) a.tile >>= 1;
    const bool apart = a.ngroup > 1 && (a.len > kPoolMaxLen || (int64_t)a.ngroup * a.len > kSumMost);
    a.nsum = apart ? 1 : a.ngroup;
    a.ntile = (int)((a.nW + a.tile - 1) / a.tile);
    const int64_t reach = a.nms ? a.len - 1 : 0, most_found = s3greedy::choices(a.nW, reach, top_b), need = s3greedy::slots_needed(a.nW, reach, most_found);
    const bool slots = l.full && top_many(most_found, reach) && need <= kTopSlots && (a.nW + 63) / 64 <= 16 * s3greedy::kThreads;
    const s3greedy::Way sw = s3greedy::way_of(need, reach);
    a.need = (int)(slots ? need : 0);
    a.room = sw.room;
    a.sublog = slots ? 6 : kSubLog2;
    a.nsub = (int)((a.nW + (1 << a.sublog) - 1) >> a.sublog);
    // the smallest tiles of which the search's lanes hold all groups: beyond 1M windows a tile has several blocks
    a.topshift = 0;
    while (((a.nsub - 1) >> a.topshift) + 1 > kTopTiles) ++a.topshift;
    a.scores_out = scores_out; a.span_start = span_start; a.span_score = span_score; a.n_found = n_found;

    hipStream_t st = (hipStream_t)stream;
    static S3LdsOnce once_prep, once_gather[2];
    const int prep_lds = (a.n_feat < kRange ? a.n_feat : kRange) * 8;
    if (int rc = s3_allow_lds(once_prep, (const void*)sc_prep_kernel, kRange * 8)) return rc;
    const bool cmp = v.delta != nullptr;
    auto gather = cmp ? sc_gather_kernel<true> : sc_gather_kernel<false>;
    if (int rc = s3_allow_lds(once_gather[cmp], (const void*)gather, (kMaxPB + 64) * 8)) return rc;
    // four or five launches: query weights, gather, perhaps the sum of the groups, pooling (with that sum) and tile maxima, Top-B
    if ((int64_t)nq * a.k <= kPrepThreads) hipLaunchKernelGGL(sc_prep_few_kernel, dim3((unsigned)a.n_heads), dim3(kPrepThreads), 0, st, a);
    else hipLaunchKernelGGL(sc_prep_kernel, dim3((unsigned)a.nr, (unsigned)a.n_heads), dim3(kPrepThreads), (size_t)prep_lds, st, a);
    hipLaunchKernelGGL(gather, dim3((unsigned)(a.npb * a.ngroup)), dim3(kScatterThreads), (size_t)(a.pb + 64) * 8, st, a);
    if (apart) hipLaunchKernelGGL(sc_reduce_kernel, dim3((unsigned)((a.L + 63) / 64)), dim3(a.ngroup <= kReduceFew ? 256 : 1024), 0, st, a);
    if (a.len <= kPoolMaxLen) {
        static S3LdsOnce once_pool;
        if (int rc = s3_allow_lds(once_pool, (const void*)sc_pool_kernel, (kTileW + kPoolMaxLen) * 8)) return rc;
        hipLaunchKernelGGL(sc_pool_kernel, dim3((unsigned)a.ntile), dim3(kPoolThreads), (size_t)(a.tile + a.len) * 8, st, a);
    } else {
        hipLaunchKernelGGL(sc_pool_wide_kernel, dim3((unsigned)((a.ntile + 3) / 4)), dim3(256), 0, st, a);
    }
    if (slots) {
        static void (*const ways[18])(ScoreArgs) = {
            sc_topb_rounds_kernel<1, 64>, sc_topb_rounds_kernel<1, 128>, sc_topb_rounds_kernel<1, 256>,
            sc_topb_rounds_kernel<4, 64>, sc_topb_rounds_kernel<4, 128>, sc_topb_rounds_kernel<4, 256>,
            sc_topb_rounds_kernel<16, 64>, sc_topb_rounds_kernel<16, 128>, sc_topb_rounds_kernel<16, 256>,
            sc_topb_slots_kernel<1, 1>, sc_topb_slots_kernel<1, 2>, sc_topb_slots_kernel<1, 4>,
            sc_topb_slots_kernel<4, 1>, sc_topb_slots_kernel<4, 2>, sc_topb_slots_kernel<4, 4>,
            sc_topb_slots_kernel<16, 1>, sc_topb_slots_kernel<16, 2>, sc_topb_slots_kernel<16, 4>};
        const int way = (sw.rounds ? 0 : 9) + (a.nsub <= s3greedy::kThreads ? 0 : (a.nsub <= 4 * s3greedy::kThreads ? 3 : 6)) + sw.up;
        const int fixed = s3greedy::lds_bytes<unsigned long long>(sw.cap);
        static S3LdsOnce once_top[18];
        if (int rc = s3_allow_lds(once_top[way], (const void*)ways[way], fixed + (sw.rounds ? s3greedy::kListMax * 12 : 0))) return rc;
        hipLaunchKernelGGL(ways[way], dim3(1), dim3(s3greedy::kThreads), (size_t)(fixed + (sw.rounds ? sw.room * 12 : 0)), st, a);
    } else if (a.nsub <= kTopRegs * 64) hipLaunchKernelGGL(sc_topb_kernel, dim3(1), dim3(64), 0, st, a);
    else hipLaunchKernelGGL(sc_topb_long_kernel, dim3(1), dim3(kTopThreads), 0, st, a);
    S3_HIP(hipGetLastError());
    return S3_OK;
}

}  // namespace

extern "C" size_t s3_coactivate_score_workspace(const s3_index* idx, int64_t n_positions) {
    if (!idx || n_positions < 1) return 0;
    S3IndexView v;
    s3_index_view(idx, &v);
    return layout(v.n_heads, v.n_feat, n_positions, true).total;
}

extern "C" int s3_coactivate_score(const s3_index* idx, const int32_t* qids, const float* qvals, int nq,
                                   int64_t n_positions, int span_len, int top_b, int32_t max_freq, int nms,
                                   float* scores_out, int32_t* span_start, float* span_score, int32_t* n_found,
                                   void* ws, size_t ws_bytes, void* stream) {
    if (!idx) return s3_fail(S3_EINVAL, "s3_coactivate_score: null pointer");
    S3IndexView v;
    s3_index_view(idx, &v);
    if (!v.finalized) return s3_fail(S3_ESTATE, "s3_coactivate_score: index not finalized");
    ScoreSource src;
    src.n_heads = v.n_heads; src.n_feat = v.n_feat; src.k = v.k; src.tokens = v.tokens; src.sorted = v.sorted;
    src.offsets = v.offsets; src.off_stride = v.off_stride; src.positions = v.positions; src.pos_stride = v.pos_stride;
    src.btab = v.btab_valid ? v.btab : nullptr;
    src.nblk = v.btab_valid ? v.nblk : 1;
    return score_run("s3_coactivate_score", src, qids, qvals, nq, n_positions, span_len, top_b, max_freq, nms, scores_out,
                     span_start, span_score, n_found, ws, ws_bytes, stream);
}

extern "C" size_t s3_coactivate_score_compact_workspace(const s3_cindex* cidx, int64_t n_positions) {
    if (!cidx || n_positions < 1) return 0;
    S3CompactView c;
    s3_cindex_view(cidx, &c);
    return layout(c.n_heads, c.n_feat, n_positions, true).total;
}

extern "C" int s3_coactivate_score_compact(const s3_cindex* cidx, const int32_t* qids, const float* qvals, int nq,
                                           int64_t n_positions, int span_len, int top_b, int32_t max_freq, int nms,
                                           float* scores_out, int32_t* span_start, float* span_score, int32_t* n_found,
                                           void* ws, size_t ws_bytes, void* stream) {
    if (!cidx) return s3_fail(S3_EINVAL, "s3_coactivate_score_compact: null pointer");
    S3CompactView c;
    s3_cindex_view(cidx, &c);
    ScoreSource src;
    src.n_heads = c.n_heads; src.n_feat = c.n_feat; src.k = c.k; src.tokens = c.tokens; src.sorted = true;
    src.nblk = c.nblk;
    src.delta = c.delta; src.cstart = c.cstart; src.cfreq = c.cfreq; src.delta_stride = c.delta_stride;
    src.cstart_stride = c.cstart_stride;
    return score_run("s3_coactivate_score_compact", src, qids, qvals, nq, n_positions, span_len, top_b, max_freq, nms,
                     scores_out, span_start, span_score, n_found, ws, ws_bytes, stream);
}
