// The rest of Phase 2 and the set operations of Phase 3 (Sec. 3.5 "Adaptive Granularity", Sec. 3.6, Alg. 1):
//
//   s3_select_spans : S' = Conv1D(S) (the semantic density curve), density peaks by greedy non-maximum suppression
//                     (N centres), and a variable-length span around every peak: the positions where the density
//                     stays at or above a fraction of the peak's, up to a largest half length
//   s3_fuse_indices : Idx_final = spans U an index list supplied by the caller (the lexical retriever's) U the first
//                     and last positions (Lead/Tail), as a 0/1 mask and as the ascending list of selected positions
//
// The density is accumulated in fp64 in tap order from the fp32 scores and weights (each product of two fp32 values
// is exact in fp64, so the sum does not depend on whether the compiler fuses the multiply-add) and rounded to fp32
// once; every decision -- which position is a peak, where a span ends -- is taken on those fp32 values, with the
// threshold product formed in fp64.  A CPU reference that follows the same steps reaches the same integers.
#include "greedy.h"
#include "s3_common.h"

#include <math.h>

namespace {

constexpr int kMaxTaps = 4096;
constexpr int kConvPer = 4;                 // consecutive positions per thread of the convolution
constexpr int kConvSmall = 64, kConvLarge = 256;      // its workgroup sizes: below / from kConvLargeFrom positions
constexpr int64_t kConvLargeFrom = 1 << 18; // 64 threads fill the chip up to 2^18 positions; beyond, the halo is shared by more
constexpr int kTile = 64;                   // positions per block: one bit or one lane each
constexpr int kConvKeyShift = 4;            // blocks per workgroup of the large convolution: 2^4
constexpr int kNmsThreads = s3greedy::kThreads;
// Which searches bring blocks into LDS (the others take 1.1 us a centre, and begin sooner): those for more than so many centres, the
// more the more blocks a choice may reach into, which are all looked through in every round.  us for a whole selection without /
// with it, curves of noise, smoothed or not: 8 centres of 1000 to 300000 positions 15 to 20 / 14 to 20; 40 of 8000 48 / 19; 12 at a
// radius of 300 20 to 24 / 17 to 25; 9 at 500 19 to 22 / 19 to 27, 16 25 to 35 / 21 to 36, 20 31 / 26; at 1000 16 of 70000 positions
// 25 / 36, 20 of 20000 25 / 30, 33 of 32768 39 / 30.  And where more than 512 blocks of many are asked for, which are taken one choice
// a round (0.9 us) behind a threshold between 512 and 576 counts, for more than kNmsManyTight: 32 at 500 of 70000 47 / 57.
constexpr int kNmsFew = 8, kNmsManyTight = 64;
inline bool nms_many(int64_t found, int64_t radius) { return found > kNmsFew && found > (radius + 16) / 32; }
constexpr int kNmsSlots = 576;              // blocks that the peak search holds in LDS at most (157.5 KB; in rounds 512, 140 KB and 8 of choices)
static_assert(s3greedy::lds_bytes<unsigned>(kNmsSlots) + s3greedy::lds_static(0) <= s3greedy::kLdsMost &&
              s3greedy::lds_bytes<unsigned>(512) + s3greedy::kListMax * 8 + s3greedy::lds_static(512) <= s3greedy::kLdsMost);
constexpr int kNmsTiles = 16384;            // tile maxima that the peak search keeps in LDS at most (128 KB): four groups of 64 per lane
constexpr int kNmsTilesMin = 8192;          // as many fit beside the most centres
static_assert(kConvLarge * kConvPer == kTile << kConvKeyShift && kConvLargeFrom <= (int64_t)kNmsTilesMin * kTile);
constexpr int kNmsLds = 152 << 10;          // its LDS: tile maxima, centres, group maxima

struct SelArgs {
    const float* scores;
    const float* kernel;
    int64_t L;
    int K, n_centers, radius, max_half;
    float rel;
    float* dens;                 // [L]
    unsigned long long* tkey;    // [nblk] best position of every block of kTile positions (peak_key)
    unsigned long long* ckey;    // [nckey] best position of every kTile << kshift positions (kshift > 0 only)
    unsigned long long* dead;    // [nblk] positions of every block that are gone, a bit each (sel_nms_long_kernel)
    int nblk, nckey;
    int need, room;              // blocks that the peak search brings into LDS at least, and entries of its list of choices
    int shift, kshift;           // the peak search works on tiles of kTile << shift positions, shift >= kshift
    int32_t* center;
    float* center_density;
    int32_t* span_lo;
    int32_t* span_hi;
    int32_t* n_found;
};

// Orders positions by (density, smaller position first); 0 for a position that cannot be a centre (density not positive).
__device__ __forceinline__ unsigned long long peak_key(float d, int64_t t) {
    return d > 0.f ? ((unsigned long long)__float_as_uint(d) << 32) | (unsigned)~(unsigned)t : 0ull;
}

// Largest key of the wavefront, in every lane: the high words first, then the low words of the lanes that hold it.
__device__ __forceinline__ unsigned long long wave_max_key(unsigned long long v) {
    const unsigned hi = s3_wave_max_u32((unsigned)(v >> 32));
    const unsigned lo = s3_wave_max_u32((unsigned)(v >> 32) == hi ? (unsigned)v : 0u);
    return ((unsigned long long)hi << 32) | lo;
}

// D[t] = sum_j g[j] * S[t + j - floor(K / 2)] with zeros outside the context, and the best position of every block and of
// every kTile << kshift positions.
// Inputs and weights are staged in LDS; a thread has four consecutive positions, so four taps cost two 16-byte reads
// for 16 multiply-adds (one 4-byte read per operand before).
template <int NT>
__global__ __launch_bounds__(NT) void sel_conv_kernel(SelArgs a) {
    extern __shared__ __align__(16) float lds[];
    const int kp = (a.K + 3) & ~3;
    float* g = lds;                          // [kp]
    float* s = lds + kp;                     // [NT * kConvPer + kp + 4]
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * (NT * kConvPer);
    const int c = a.K / 2;
    for (int j = tid; j < a.K; j += NT) g[j] = a.kernel[j];
    for (int i = tid; i < NT * kConvPer + a.K - 1; i += NT) {
        const int64_t u = t0 + i - c;
        s[i] = (u >= 0 && u < a.L) ? a.scores[u] : 0.f;
    }
    __syncthreads();
    double acc[kConvPer] = {0.0, 0.0, 0.0, 0.0};
    const float4* sv = (const float4*)(s + tid * kConvPer);
    float4 lo = sv[0];
    int j = 0;
    for (; j + 4 <= a.K; j += 4) {
        const float4 hi = sv[j / 4 + 1];
        const float4 gv = *(const float4*)(g + j);
        const float w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        const float gg[4] = {gv.x, gv.y, gv.z, gv.w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < kConvPer; ++q) acc[q] += (double)gg[u] * (double)w[u + q];
        lo = hi;
    }
    for (; j < a.K; ++j)
#pragma unroll
        for (int q = 0; q < kConvPer; ++q) acc[q] += (double)g[j] * (double)s[tid * kConvPer + q + j];
    unsigned long long best = 0;
#pragma unroll
    for (int q = 0; q < kConvPer; ++q) {
        const int64_t t = t0 + tid * kConvPer + q;
        if (t < a.L) {
            const float dv = (float)acc[q];
            a.dens[t] = dv;
            const unsigned long long k = peak_key(dv, t);
            best = k > best ? k : best;
        }
    }
    // the 16 lanes of a row hold one block
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        const unsigned hi = (unsigned)__shfl_xor((int)(unsigned)(best >> 32), o), lw = (unsigned)__shfl_xor((int)(unsigned)best, o);
        const unsigned long long other = ((unsigned long long)hi << 32) | lw;
        best = other > best ? other : best;
    }
    const int64_t blk = t0 / kTile + tid / 16;
    if ((tid & 15) == 0 && blk < a.nblk) {
        a.tkey[blk] = best;
        if (a.dead) a.dead[blk] = 0;
    }
    if (NT == kConvSmall || a.kshift == 0) return;
    __shared__ unsigned long long bk[NT / 16];
    if ((tid & 15) == 0) bk[tid / 16] = best;
    __syncthreads();
    const int64_t at = (t0 / kTile >> a.kshift) + tid;
    if (tid < (NT / 16 >> a.kshift) && at < a.nckey) {
        best = 0;
        for (int j = tid << a.kshift; j < (tid + 1) << a.kshift; ++j) best = bk[j] > best ? bk[j] : best;
        a.ckey[at] = best;
    }
}

// Greedy peak selection, then the span of every peak.  One workgroup: the rounds depend on each other, so what bounds it is
// the latency of a round.
//
// sel_peaks_kernel, sel_nms_kernel: the blocks that the choices can lie in are brought into LDS (greedy.h), for up to 512 or 576
// such blocks (all of them below 32769 or 36865 positions, else three a centre at a radius of 64).  The first takes all choices that do not
// depend on each other at once, the second (small radii, where there may be many) one a round, by one wavefront.
// sel_nms_long_kernel, for few centres (nms_many()) and for more than that: one wavefront walks the rounds without a barrier over all tiles: maxima of groups of 64
// tiles are in its registers, the tile maxima in LDS.  A round takes the best group, clears the tiles that the suppression
// covers whole and searches the two blocks of 64 positions at its ends again; the groups at both ends are reduced in the
// next round, beside its search and not behind this one's.  The curve is read from memory beside a bit per position that says
// which ones are gone (word e belongs to lane e % 64 in every round, so a lane only ever reads back its own marks).  A tile or
// block without live positions stays so (its bits need not be set).  Beyond kNmsTilesMin blocks a tile may have several; from
// four on their keys come from memory, too, and the convolution leaves the first maxima of up to 1024 positions, so that one
// workgroup has fewer to load.
//
// us for a whole selection, K 48, half lengths of 64, by one choice a round over all tiles (below 36000 positions with the curve in
// LDS) / with blocks in LDS: 40 centres, radius 64: 8000 positions 48 / 19, 36000 51 / 19, 300000 59 / 27, 1000000 70 / 29; radius 0
// 46 / 32, 49 / 33, 56 / 34, 67 / 38; 128 centres, radius 64, 36000 positions 141 / 40.
struct NmsLds {
    unsigned long long* key;                                          // [nt] tile maxima
    unsigned long long* gkey;                                         // [ng] maxima of groups of 64 tiles
    int* cen;                                                         // [n_centers]
    float* cden;                                                      // [n_centers]
    int nt, ng;
};
__device__ __forceinline__ NmsLds nms_lds_of(const SelArgs& a, unsigned long long* lds) {
    NmsLds l;
    l.nt = (a.nblk + (1 << a.shift) - 1) >> a.shift;
    l.ng = (l.nt + 63) >> 6;
    l.key = lds;
    l.gkey = l.key + l.nt;
    l.cen = (int*)(l.gkey + l.ng);
    l.cden = (float*)(l.cen + a.n_centers);
    return l;
}

// Tile and group maxima from `per` keys a tile, of which there are n.
__device__ __forceinline__ void nms_load_keys(const NmsLds& l, const unsigned long long* keys, int n, int per, int wave, int lane) {
    for (int g = wave; g < l.ng; g += kNmsThreads / 64) {
        const int t = g * 64 + lane;
        unsigned long long best = 0;
        if (t < l.nt) {
            const int64_t e0 = (int64_t)t * per, e1 = min((int64_t)n, e0 + per);
            for (int64_t e = e0; e < e1; ++e) {
                const unsigned long long v = keys[e];
                best = v > best ? v : best;
            }
            l.key[t] = best;
        }
        best = wave_max_key(best);
        if (lane == 0) l.gkey[g] = best;
    }
}

// The state of the walk: maxima of the lane's groups (0 while their tiles are in va / vb), and the tiles (ga * 64 + lane,
// gb * 64 + lane) that changed last.
template <int G>                                                      // groups per lane
struct NmsTop {
    unsigned long long top[G], va, vb;
    int ga, gb;
};
template <int G>
__device__ __forceinline__ void nms_start(NmsTop<G>& w, const NmsLds& l, int lane) {
#pragma unroll
    for (int q = 0; q < G; ++q) w.top[q] = q * 64 + lane < l.ng ? l.gkey[q * 64 + lane] : 0ull;
    w.va = w.vb = 0;
    w.ga = w.gb = -1;
}
// The best live position; the groups that changed last go back to their lanes' registers.
template <int G>
__device__ __forceinline__ unsigned long long nms_best(NmsTop<G>& w, int lane) {
    unsigned long long best = w.va > w.vb ? w.va : w.vb;
#pragma unroll
    for (int q = 0; q < G; ++q) best = w.top[q] > best ? w.top[q] : best;
    best = wave_max_key(best);
    const unsigned long long ma = wave_max_key(w.va), mb = wave_max_key(w.vb);      // beside the reduction above, not behind it
#pragma unroll
    for (int q = 0; q < G; ++q) {
        if (q * 64 + lane == w.ga) w.top[q] = ma;
        if (q * 64 + lane == w.gb) w.top[q] = mb;
    }
    return best;
}
// Reads the tiles of the groups at both ends, behind a fence.
template <int G>
__device__ __forceinline__ void nms_open(NmsTop<G>& w, const NmsLds& l, int tl, int th, int lane) {
    w.ga = tl >> 6;
    w.gb = th >> 6;
#pragma unroll
    for (int q = 0; q < G; ++q)
        if (q * 64 + lane >= w.ga && q * 64 + lane <= w.gb) w.top[q] = 0;
    w.va = w.ga * 64 + lane < l.nt ? l.key[w.ga * 64 + lane] : 0ull;
    w.vb = w.gb * 64 + lane < l.nt ? l.key[w.gb * 64 + lane] : 0ull;
}
// Stores the new maxima of the tiles at both ends.
template <int G>
__device__ __forceinline__ void nms_close(NmsTop<G>& w, const NmsLds& l, int tl, int th, unsigned long long kl, unsigned long long kh, int lane) {
    s3_wave_fence();                                                  // va and vb are read
    if (lane == 0) { l.key[tl] = kl; l.key[th] = kh; }                // the same value where tl == th
    s3_wave_fence();
    if (w.ga * 64 + lane == tl) w.va = kl;
    if (w.ga * 64 + lane == th) w.va = kh;
    if (w.gb * 64 + lane == tl) w.vb = kl;
    if (w.gb * 64 + lane == th) w.vb = kh;
}

__device__ __forceinline__ void nms_spans(const SelArgs& a, const int* cen, const float* cden, int found, int tid, int lane, int wave) {
    // spans: a wavefront per centre walks outwards 64 positions at a time, both sides at once; a side ends before the
    // first position whose density is below rel * D[centre] or that is farther than max_half from the centre.  The first 64
    // positions of four centres are asked for together (40 centres, half lengths of 64: 2.9 -> 2.3 us).
    constexpr int kW = kNmsThreads / 64, U = 4;
    for (int r0 = wave; r0 < found; r0 += U * kW) {
        float ahead[U][2];
        int c[U];
        double thr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = min(r0 + u * kW, found - 1);
            c[u] = cen[r];
            thr[u] = (double)a.rel * (double)cden[r];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int64_t t = side == 0 ? (int64_t)c[u] - 1 - lane : (int64_t)c[u] + 1 + lane;
                ahead[u][side] = t >= 0 && t < a.L ? a.dens[t] : -1.f;
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * kW;
            if (r >= found) break;
            const int limit[2] = {(int)min((int64_t)a.max_half, (int64_t)c[u]), (int)min((int64_t)a.max_half, a.L - 1 - c[u])};
            int n[2] = {0, 0};
            bool open[2] = {limit[0] > 0, limit[1] > 0};
            float d[2] = {ahead[u][0], ahead[u][1]};
            while (open[0] || open[1]) {
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    if (!open[side]) continue;
                    const bool ok = (int64_t)n[side] + 1 + lane <= limit[side] && (double)d[side] >= thr[u];
                    const unsigned long long m = __ballot(ok);
                    const int run = m == ~0ull ? 64 : (int)__builtin_ctzll(~m);      // leading positions that pass
                    n[side] += run;
                    open[side] = run == 64 && n[side] < limit[side];
                }
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    const int64_t off = (int64_t)n[side] + 1 + lane;      // distance from the centre
                    if (open[side] && off <= limit[side]) d[side] = a.dens[side == 0 ? c[u] - off : c[u] + off];
                }
            }
            if (lane == 0) {
                if (cen != a.center) { a.center[r] = c[u]; a.center_density[r] = cden[r]; }
                a.span_lo[r] = c[u] - n[0];
                a.span_hi[r] = c[u] + n[1];
            }
        }
    }
    for (int r = found + tid; r < a.n_centers; r += kNmsThreads) {
        a.center[r] = -1; a.center_density[r] = 0.f; a.span_lo[r] = -1; a.span_hi[r] = -1;
    }
    if (tid == 0) a.n_found[0] = found;
}

// The blocks' maxima and their places, P a thread, and with them the slots.
template <int P>
__device__ __forceinline__ void nms_fill(const SelArgs& a, const s3greedy::Slots<unsigned>& slots) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per = P == 1 ? 1 : s3greedy::per_thread(a.nblk);
    unsigned key[P];
    int at[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const int b = q < per ? (wave * per + q) * 64 + lane : a.nblk;
        const unsigned long long v = b < a.nblk ? a.tkey[b] : 0ull;
        key[q] = (unsigned)(v >> 32);
        at[q] = (int)~(unsigned)v;
    }
    s3greedy::fill<unsigned, P>(slots, key, at, a.need, a.L, [&](int64_t t) { return a.dens[t]; },
                                [](float d) { return d > 0.f ? __float_as_uint(d) : 0u; });
}

template <int P, int C>                       // maxima per thread, slots
__global__ __launch_bounds__(s3greedy::kThreads) void sel_peaks_kernel(SelArgs a) {
    extern __shared__ __align__(16) unsigned long long nms_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const auto slots = s3greedy::slots_of<unsigned>(nms_lds, C);
    unsigned* const list_key = (unsigned*)((char*)nms_lds + s3greedy::lds_bytes<unsigned>(C));
    nms_fill<P>(a, slots);
    const int found = s3greedy::rounds<C, unsigned>(slots, list_key, (int*)(list_key + a.room), (unsigned)a.L, (unsigned)a.radius, a.n_centers,
                                                    [&](int r, unsigned k, int t) { a.center[r] = t; a.center_density[r] = __uint_as_float(k); });
    __syncthreads();                          // the centres were written by this workgroup
    nms_spans(a, a.center, a.center_density, found, tid, lane, wave);
}

template <int P, int R>                       // maxima per thread, slots per lane
__global__ __launch_bounds__(s3greedy::kThreads) void sel_nms_kernel(SelArgs a) {
    extern __shared__ __align__(16) unsigned long long nms_lds[];
    __shared__ int found_s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const auto slots = s3greedy::slots_of<unsigned>(nms_lds, 64 * R);
    nms_fill<P>(a, slots);
    if (wave == 0) {
        unsigned left;
        int left_at;
        const int found = s3greedy::walk<R, unsigned>(slots, (unsigned)a.L, (unsigned)a.radius, a.n_centers, left, left_at, [&](int r, unsigned k, int t) {
            if (lane == 0) { a.center[r] = t; a.center_density[r] = __uint_as_float(k); }
        }, [](int, unsigned, int) { return false; });
        if (lane == 0) found_s = found;
    }
    __syncthreads();                          // the centres were written by this workgroup
    nms_spans(a, a.center, a.center_density, found_s, tid, lane, wave);
}

__device__ __forceinline__ unsigned long long lane_value(unsigned long long v, int src) {
    return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(v >> 32), src) << 32) |
           (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, src);
}

// The word of block e with the positions of [lo, hi] marked.
__device__ __forceinline__ unsigned long long nms_mark(unsigned long long m, int e, int64_t lo, int64_t hi) {
    const int64_t p = (int64_t)e << 6;
    const int from = (int)max((int64_t)0, lo - p), upto = (int)min((int64_t)63, hi - p);
    return from <= upto ? m | (~0ull << from & ~0ull >> (63 - upto)) : m;
}

// U > 0: tiles of U blocks, searched whole.  U == 0: tiles of more blocks, searched by their keys.
template <int U, int G>
__global__ __launch_bounds__(kNmsThreads) void sel_nms_long_kernel(SelArgs a) {
    extern __shared__ __align__(16) unsigned long long nms_lds[];
    __shared__ int found_s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const NmsLds l = nms_lds_of(a, nms_lds);
    if (U == 1) nms_load_keys(l, a.tkey, a.nblk, 1, wave, lane);
    else nms_load_keys(l, a.ckey, a.nckey, 1 << (a.shift - a.kshift), wave, lane);
    __syncthreads();
    if (wave == 0) {
        const int tlog = 6 + a.shift, per = 1 << a.shift;             // blocks per tile
        NmsTop<G> w;
        nms_start(w, l, lane);
        int found = 0;
        while (found < a.n_centers) {
            const unsigned long long best = nms_best(w, lane);
            if (best == 0) break;                                     // only positive density makes a centre
            const int64_t c = (int64_t)(unsigned)~(unsigned)best;
            if (lane == 0) { l.cen[found] = (int)c; l.cden[found] = __uint_as_float((unsigned)(best >> 32)); }
            ++found;
            const int64_t lo = max((int64_t)0, c - a.radius), hi = min(a.L - 1, c + a.radius);
            const int tl = (int)(lo >> tlog), th = (int)(hi >> tlog);
            const int b0 = tl << a.shift, b1 = th << a.shift;         // first blocks of both tiles
            const int g0 = (b0 & ~63) + lane, g1 = (b1 & ~63) + lane; // blocks of this lane (the first of them, if a tile has more than 64)
            const bool in0 = g0 >= b0 && g0 < b0 + per && g0 < a.nblk, in1 = g1 >= b1 && g1 < b1 + per && g1 < a.nblk;
            const bool live_l = l.key[tl] != 0, live_h = l.key[th] != 0;
            unsigned long long kl = 0, kh = 0;                        // best live position of the tile at either end
            if constexpr (U > 0) {
                float d0[U], d1[U];
                unsigned long long m0 = 0, m1 = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t p0 = ((int64_t)(b0 + u) << 6) + lane, p1 = ((int64_t)(b1 + u) << 6) + lane;
                    d0[u] = d1[u] = 0.f;
                    if (p0 < a.L) d0[u] = a.dens[p0];
                    if (p1 < a.L) d1[u] = a.dens[p1];
                }
                if (in0) m0 = a.dead[g0];
                if (in1) m1 = a.dead[g1];
                for (int t = tl + 1 + lane; t < th; t += 64) l.key[t] = 0;
                s3_wave_fence();                                      // the cleared tiles are read by other lanes
                nms_open(w, l, tl, th, lane);
                unsigned long long s0 = m0, s1 = m1;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i0 = (b0 & 63) + u, i1 = (b1 & 63) + u; // lanes that own the blocks; the words are scalars
                    const unsigned long long w0 = nms_mark(lane_value(m0, i0), b0 + u, lo, hi);
                    const unsigned long long w1 = nms_mark(lane_value(m1, i1), b1 + u, lo, hi);
                    if (lane == i0) s0 = w0;
                    if (lane == i1) s1 = w1;
                    const int64_t p0 = ((int64_t)(b0 + u) << 6) + lane, p1 = ((int64_t)(b1 + u) << 6) + lane;
                    if (!(w0 >> lane & 1)) kl = max(kl, peak_key(d0[u], p0));
                    if (!(w1 >> lane & 1)) kh = max(kh, peak_key(d1[u], p1));
                }
                if (in0) a.dead[g0] = s0;
                if (in1) a.dead[g1] = s1;                             // the same words and values where tl == th
                kl = wave_max_key(kl);
                kh = wave_max_key(kh);
            } else {
                const int el = (int)(lo >> 6), eh = (int)(hi >> 6);
                const int64_t p0 = ((int64_t)el << 6) + lane, p1 = ((int64_t)eh << 6) + lane;
                const bool own0 = lane == (el & 63), own1 = lane == (eh & 63);
                float d0 = 0.f, d1 = 0.f;
                unsigned long long m0 = 0, m1 = 0, t0 = 0, t1 = 0, v0 = 0, v1 = 0;
                if (p0 < a.L) d0 = a.dens[p0];
                if (p1 < a.L) d1 = a.dens[p1];
                if (own0) { m0 = a.dead[el]; t0 = a.tkey[el]; }
                if (own1) { m1 = a.dead[eh]; t1 = a.tkey[eh]; }
                if (in0) v0 = a.tkey[g0];
                if (in1) v1 = a.tkey[g1];
                for (int t = tl + 1 + lane; t < th; t += 64) l.key[t] = 0;
                s3_wave_fence();                                      // the cleared tiles are read by other lanes
                nms_open(w, l, tl, th, lane);
                m0 = nms_mark(lane_value(m0, el & 63), el, lo, hi);
                m1 = nms_mark(lane_value(m1, eh & 63), eh, lo, hi);
                if (own0) a.dead[el] = m0;
                if (own1) a.dead[eh] = m1;                            // the same where el == eh
                unsigned long long k0 = 0, k1 = 0;                    // (a block without live positions stays so)
                if (!(m0 >> lane & 1) && lane_value(t0, el & 63)) k0 = peak_key(d0, p0);
                if (!(m1 >> lane & 1) && lane_value(t1, eh & 63)) k1 = peak_key(d1, p1);
                // both tiles: the positions of the blocks at the ends, the keys of the blocks outside the interval
                unsigned long long n0 = tl == th ? max(k0, k1) : k0, n1 = tl == th ? max(k0, k1) : k1;
                auto outside = [&](int e, unsigned long long v, unsigned long long& n) {
                    if (e < el || e > eh) n = max(n, v);
                    if (v && e > el && e < eh) a.tkey[e] = 0;
                };
                outside(g0, v0, n0);
                outside(g1, v1, n1);
                for (int s = 64; s < per; s += 64) {
                    if (g0 + s < a.nblk) outside(g0 + s, a.tkey[g0 + s], n0);
                    if (g1 + s < a.nblk) outside(g1 + s, a.tkey[g1 + s], n1);
                }
                kl = wave_max_key(n0);
                kh = wave_max_key(n1);
                const unsigned long long e0 = wave_max_key(k0), e1 = wave_max_key(k1);
                if (own0) a.tkey[el] = e0;
                if (own1) a.tkey[eh] = e1;                            // the same where el == eh
            }
            nms_close(w, l, tl, th, live_l ? kl : 0ull, live_h ? kh : 0ull, lane);      // a tile without live positions stays so
        }
        if (lane == 0) found_s = found;
    }
    __syncthreads();
    nms_spans(a, l.cen, l.cden, found_s, tid, lane, wave);
}

// ---- Phase 3 set operations ----
// What bounds them at the lengths of a context is the number of launches.  Two are enough: fuse_block_kernel builds the
// mask of a block of positions in LDS (every block looks through all spans and the whole index list) and counts it,
// fuse_compact_kernel adds up the counts of the blocks before its own.  A block's look through a long list takes longer than
// two more launches, and the looks of all blocks are quadratic in the context's length, so beyond kFuseListMax list entries
// or kFuseLookMax entries looked at in all (64 MB through L2) the mask is marked in memory first.  Device time in us, looked
// through / marked, of 1000 and of 131072 positions: 300 entries 4.8 / 7.3 and 5.7 / 8.2, 32768 entries 12.2 / 7.4 and
// 13.0 / 8.5, 262144 entries 68 / 8.0 and 69 / 9.4; on the host four launches take 22, two 17, so the line lies where the
// look still hides behind those (about 14 us, as long as the five launches that these replaced).  A span costs about four
// entries (two loads, two adds in LDS): 4096 of them 6.8 / 7.8 and 7.6 / 9.1.  (A wavefront that marked one span after the
// other took 118 us for 4096 spans in 1000 positions.)  Beyond kFuseSelfMax blocks the counts are scanned by a launch of
// their own.
constexpr int kFuseThreads = 256;
constexpr int kFusePer = 4;                             // consecutive positions per thread
constexpr int kFuseBlock = kFuseThreads * kFusePer;     // positions per workgroup
constexpr int64_t kFuseListMax = 9 << 12;
constexpr int64_t kFuseLookMax = 1 << 24;
constexpr int kFuseSelfMax = 4096;

// number of selected positions among a thread's four (bytes are 0 or 1), and the mask bytes themselves
__device__ __forceinline__ uint32_t fuse_load4(const unsigned char* mask, int64_t t, int64_t L, bool aligned) {
    if (aligned && t + kFusePer <= L) return *(const uint32_t*)(mask + t);
    uint32_t v = 0;
#pragma unroll
    for (int j = 0; j < kFusePer; ++j)
        if (t + j < L) v |= (uint32_t)mask[t + j] << (8 * j);
    return v;
}

__global__ __launch_bounds__(kFuseThreads) void fuse_block_kernel(unsigned char* mask, int64_t L, const int32_t* lo, const int32_t* hi,
                                                                  const int32_t* n_spans, int max_spans, const int32_t* extra,
                                                                  int64_t n_extra, int lead, int tail, int* bsum) {
    __shared__ uint32_t m4[kFuseThreads];
    __shared__ __align__(16) int step[kFuseBlock + 4];          // spans that start here less spans that ended before
    __shared__ int wsum[kFuseThreads / 64];
    __shared__ int met;                                         // whether any span meets the block
    unsigned char* const m = (unsigned char*)m4;
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * kFuseBlock, t1 = min(L, t0 + kFuseBlock) - 1;      // first and last position
    uint32_t v = 0;
#pragma unroll
    for (int j = 0; j < kFusePer; ++j) {
        const int64_t t = t0 + tid * kFusePer + j;
        if (t < L && (t < lead || t >= L - tail)) v |= 1u << (8 * j);
    }
    m4[tid] = v;
    *(int4*)(step + tid * kFusePer) = make_int4(0, 0, 0, 0);
    if (tid == 0) met = 0;
    __syncthreads();
    const int ns = n_spans ? min(*n_spans, max_spans) : max_spans;
    for (int i = tid; i < ns; i += kFuseThreads) {
        const int64_t a = max((int64_t)lo[i], t0), b = min((int64_t)hi[i], t1);
        if (a > b) continue;
        met = 1;
        atomicAdd(step + (int)(a - t0), 1);
        atomicAdd(step + (int)(b - t0) + 1, -1);                // the place behind the block is read by nobody
    }
    for (int64_t i0 = tid; i0 < n_extra; i0 += 8 * kFuseThreads) {
        int32_t p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = i0 + u * kFuseThreads < n_extra ? extra[i0 + u * kFuseThreads] : -1;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if ((int64_t)p[u] >= t0 && (int64_t)p[u] <= t1) m[(int)(p[u] - t0)] = 1;
    }
    __syncthreads();
    v = m4[tid];
    const int64_t t = t0 + tid * kFusePer;
    if (met) {
        const int4 d = *(const int4*)(step + tid * kFusePer);
        int all;
        int open = s3_block_excl_scan<kFuseThreads>(d.x + d.y + d.z + d.w, wsum, all);      // spans that reach this thread's positions
        const int dj[kFusePer] = {d.x, d.y, d.z, d.w};
#pragma unroll
        for (int j = 0; j < kFusePer; ++j) {
            open += dj[j];
            if (open > 0) v |= 1u << (8 * j);
        }
    }
    if (((uintptr_t)mask & 3) == 0 && t + kFusePer <= L) {
        *(uint32_t*)(mask + t) = v;
    } else {
#pragma unroll
        for (int j = 0; j < kFusePer; ++j)
            if (t + j < L) mask[t + j] = (unsigned char)(v >> (8 * j));
    }
    int tot;
    s3_block_excl_scan<kFuseThreads>(__popc(v), wsum, tot);
    if (tid == 0) bsum[blockIdx.x] = tot;
}

__global__ void fuse_init_kernel(unsigned char* mask, int64_t L, int lead, int tail) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < L; t += (int64_t)gridDim.x * blockDim.x)
        mask[t] = (t < lead || t >= L - tail) ? 1 : 0;
}

// block x < max_spans: span x (if it exists); the other blocks: the caller's index list
__global__ void fuse_mark_kernel(unsigned char* mask, int64_t L, const int32_t* lo, const int32_t* hi, const int32_t* n_spans,
                                 int max_spans, const int32_t* extra, int64_t n_extra) {
    if ((int)blockIdx.x < max_spans) {
        const int ns = n_spans ? min(*n_spans, max_spans) : max_spans;
        if ((int)blockIdx.x >= ns) return;
        const int64_t a = max((int64_t)lo[blockIdx.x], (int64_t)0), b = min((int64_t)hi[blockIdx.x], L - 1);
        for (int64_t t = a + threadIdx.x; t <= b; t += blockDim.x) mask[t] = 1;
    } else {
        const int64_t i = ((int64_t)blockIdx.x - max_spans) * blockDim.x + threadIdx.x;
        if (i < n_extra) {
            const int32_t p = extra[i];
            if (p >= 0 && p < L) mask[p] = 1;
        }
    }
}

__global__ __launch_bounds__(kFuseThreads) void fuse_count_kernel(const unsigned char* mask, int64_t L, int* bsum) {
    __shared__ int wsum[kFuseThreads / 64];
    const int64_t t = (int64_t)blockIdx.x * kFuseBlock + threadIdx.x * kFusePer;
    const uint32_t v = fuse_load4(mask, t, L, ((uintptr_t)mask & 3) == 0);
    int tot;
    s3_block_excl_scan<kFuseThreads>(__popc(v), wsum, tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// exclusive prefix of the block counts (one workgroup, in place); the total is the number of selected positions
__global__ __launch_bounds__(kFuseThreads) void fuse_scan_kernel(int* bsum, int nblocks, int32_t* n_out) {
    __shared__ int wsum[kFuseThreads / 64];
    int carry = 0;
    for (int b0 = 0; b0 < nblocks; b0 += kFuseThreads) {
        const int b = b0 + threadIdx.x;
        const int v = b < nblocks ? bsum[b] : 0;
        int tot;
        const int ex = s3_block_excl_scan<kFuseThreads>(v, wsum, tot);
        if (b < nblocks) bsum[b] = carry + ex;
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) n_out[0] = carry;
}

// Thread i of a workgroup owns four consecutive positions, so that the output order is the position order.  `scanned`:
// bsum holds the exclusive prefix; else the block counts, and the last workgroup also writes the total.
__global__ __launch_bounds__(kFuseThreads) void fuse_compact_kernel(const unsigned char* mask, int64_t L, const int* bsum, int scanned,
                                                                     int32_t* idx, int32_t* n_out) {
    __shared__ int wsum[kFuseThreads / 64];
    const int64_t t = (int64_t)blockIdx.x * kFuseBlock + threadIdx.x * kFusePer;
    const uint32_t v = fuse_load4(mask, t, L, ((uintptr_t)mask & 3) == 0);
    int before = 0;
    if (scanned) {
        before = bsum[blockIdx.x];
    } else {
        int part = 0;
        for (int b = threadIdx.x; b < (int)blockIdx.x; b += kFuseThreads) part += bsum[b];
        s3_block_excl_scan<kFuseThreads>(part, wsum, before);
    }
    int tot;
    int o = before + s3_block_excl_scan<kFuseThreads>(__popc(v), wsum, tot);
#pragma unroll
    for (int j = 0; j < kFusePer; ++j)
        if ((v >> (8 * j)) & 1u) idx[o++] = (int32_t)(t + j);
    if (!scanned && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) n_out[0] = before + tot;
}

struct SelLayout {
    size_t dens, tkey, ckey, dead, total;
    int nblk;
};
SelLayout sel_layout(int64_t L) {
    SelLayout l;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += s3_align(bytes); return at; };
    l.nblk = (int)((L + kTile - 1) / kTile);
    l.dens = take((size_t)L * 4);
    l.tkey = take((size_t)l.nblk * 8);
    l.ckey = take(l.nblk > kNmsTilesMin ? (size_t)(l.nblk + 1) / 2 * 8 : 0);      // kshift is at least 1 where there are any
    l.dead = take((size_t)l.nblk * 8);
    l.total = o;
    return l;
}

}  // namespace

extern "C" int s3_smoothing_kernel(int kind, int K, float* weights) {
    if (!weights) return s3_fail(S3_EINVAL, "s3_smoothing_kernel: null pointer");
    if (K < 1 || K > kMaxTaps || kind < S3_KERNEL_BOX || kind > S3_KERNEL_GAUSSIAN)
        return s3_fail(S3_EINVAL, "s3_smoothing_kernel: kind %d / K %d (1..%d) out of range", kind, K, kMaxTaps);
    auto shape = [&](int j) {
        if (kind == S3_KERNEL_TRIANGULAR) return (double)(j + 1 < K - j ? j + 1 : K - j);
        if (kind == S3_KERNEL_GAUSSIAN) {
            const double u = ((double)j - 0.5 * (K - 1)) / ((double)K / 6.0);
            return exp(-0.5 * u * u);
        }
        return 1.0;
    };
    double sum = 0.0;
    for (int j = 0; j < K; ++j) sum += shape(j);
    for (int j = 0; j < K; ++j) weights[j] = (float)(shape(j) / sum);
    return S3_OK;
}

extern "C" size_t s3_select_spans_workspace(int64_t n_positions) {
    if (n_positions < 1 || n_positions >= (1LL << 31)) return 0;
    return sel_layout(n_positions).total;
}

extern "C" int s3_select_spans(const float* scores, int64_t n_positions, const float* kernel, int K, int n_centers,
                               int nms_radius, float rel_threshold, int max_half_len, float* density_out,
                               int32_t* center, float* center_density, int32_t* span_lo, int32_t* span_hi,
                               int32_t* n_found, void* ws, size_t ws_bytes, void* stream) {
    if (!scores || !kernel || !center || !center_density || !span_lo || !span_hi || !n_found || !ws)
        return s3_fail(S3_EINVAL, "s3_select_spans: null pointer");
    if (n_positions < 1 || n_positions >= (1LL << 31))
        return s3_fail(S3_EINVAL, "s3_select_spans: n_positions %lld out of range", (long long)n_positions);
    if (K < 1 || K > kMaxTaps) return s3_fail(S3_EINVAL, "s3_select_spans: K %d not in [1, %d]", K, kMaxTaps);
    if (n_centers < 1 || n_centers > 4096 || nms_radius < 0 || max_half_len < 0)
        return s3_fail(S3_EINVAL, "s3_select_spans: n_centers %d (1..4096) / nms_radius %d / max_half_len %d out of range",
                       n_centers, nms_radius, max_half_len);
    if (!(rel_threshold >= 0.f && rel_threshold <= 1.f))
        return s3_fail(S3_EINVAL, "s3_select_spans: rel_threshold %g not in [0, 1]", (double)rel_threshold);
    const SelLayout l = sel_layout(n_positions);
    if (ws_bytes < l.total) return s3_fail(S3_ECAPACITY, "s3_select_spans: workspace %zu < %zu bytes", ws_bytes, l.total);
    if ((uintptr_t)ws & 255) return s3_fail(S3_EINVAL, "s3_select_spans: workspace must be 256-byte aligned");
    char* base = (char*)ws;
    SelArgs a;
    a.scores = scores; a.kernel = kernel; a.L = n_positions; a.K = K; a.n_centers = n_centers; a.radius = nms_radius;
    a.max_half = max_half_len; a.rel = rel_threshold;
    a.dens = density_out ? density_out : (float*)(base + l.dens);
    a.tkey = (unsigned long long*)(base + l.tkey);
    a.ckey = (unsigned long long*)(base + l.ckey);
    a.nblk = l.nblk;
    const int64_t most_found = s3greedy::choices(n_positions, nms_radius, n_centers), need = s3greedy::slots_needed(n_positions, nms_radius, most_found);
    const s3greedy::Way sw = s3greedy::way_of(need, nms_radius);
    const bool slots = nms_many(most_found, nms_radius) && need <= kNmsSlots &&
                       (need <= 512 || l.nblk <= kNmsSlots || most_found > kNmsManyTight) && l.nblk <= 16 * kNmsThreads;
    a.need = (int)(slots ? need : 0);
    a.room = sw.room;
    // sel_nms_long_kernel: tiles of one block as long as their maxima fit the search's LDS beside the centres; from there on no
    // more tiles than it takes, since loading them costs more than searching longer ones (2^21 positions, one centre: 24 us with
    // 16384 tiles, 20 with 8192)
    size_t nt, fixed;
    for (a.shift = 0;; ++a.shift) {
        nt = (size_t)((l.nblk + (1 << a.shift) - 1) >> a.shift);
        fixed = (nt + (nt + 63) / 64) * 8 + (size_t)n_centers * 8;
        if (nt <= kNmsTilesMin || (a.shift == 0 && nt <= kNmsTiles && fixed <= kNmsLds)) break;
    }
    // the convolution leaves one key per tile of the search, as far as a workgroup's positions reach
    a.kshift = slots ? 0 : (a.shift < kConvKeyShift ? a.shift : kConvKeyShift);
    a.nckey = a.kshift ? (l.nblk + (1 << a.kshift) - 1) >> a.kshift : 0;
    a.dead = slots ? nullptr : (unsigned long long*)(base + l.dead);
    a.center = center; a.center_density = center_density; a.span_lo = span_lo; a.span_hi = span_hi; a.n_found = n_found;
    hipStream_t st = (hipStream_t)stream;
    const bool large = n_positions >= kConvLargeFrom;
    const int per_wg = (large ? kConvLarge : kConvSmall) * kConvPer;
    const size_t lds = (size_t)(per_wg + 2 * ((K + 3) & ~3) + 4) * 4;      // at most 36 KB: within the default limit
    const dim3 grid((unsigned)((n_positions + per_wg - 1) / per_wg));
    if (large) hipLaunchKernelGGL(sel_conv_kernel<kConvLarge>, grid, dim3(kConvLarge), lds, st, a);
    else hipLaunchKernelGGL(sel_conv_kernel<kConvSmall>, grid, dim3(kConvSmall), lds, st, a);
    void (*nms)(SelArgs);
    int way, bytes, most;
    if (slots) {
        static void (*const ways[16])(SelArgs) = {
            sel_peaks_kernel<1, 64>, sel_peaks_kernel<1, 128>, sel_peaks_kernel<1, 256>, sel_peaks_kernel<1, 512>,
            sel_peaks_kernel<16, 64>, sel_peaks_kernel<16, 128>, sel_peaks_kernel<16, 256>, sel_peaks_kernel<16, 512>,
            sel_nms_kernel<1, 1>, sel_nms_kernel<1, 2>, sel_nms_kernel<1, 4>, sel_nms_kernel<1, 9>,
            sel_nms_kernel<16, 1>, sel_nms_kernel<16, 2>, sel_nms_kernel<16, 4>, sel_nms_kernel<16, 9>};
        way = (sw.rounds ? 0 : 8) + (l.nblk <= kNmsThreads ? 0 : 4) + sw.up;
        nms = ways[way];
        bytes = s3greedy::lds_bytes<unsigned>(sw.cap) + (sw.rounds ? sw.room * 8 : 0);
        most = s3greedy::lds_bytes<unsigned>(sw.cap) + (sw.rounds ? s3greedy::kListMax * 8 : 0);
    } else {
        // us a round, radius 48: 1.2 in tiles of one block (two or four groups per lane), 1.5 of two blocks, 2.0 of four
        // searched whole and 1.7 to 1.8 by their keys
        static void (*const ways[4])(SelArgs) = {sel_nms_long_kernel<1, 2>, sel_nms_long_kernel<1, 4>, sel_nms_long_kernel<2, 2>, sel_nms_long_kernel<0, 2>};
        const int w = a.shift == 0 ? (nt <= kNmsTilesMin ? 0 : 1) : (a.shift == 1 ? 2 : 3);
        way = 16 + w;
        nms = ways[w];
        most = kNmsLds;
        bytes = (int)fixed;
    }
    static S3LdsOnce once[20];
    if (int rc = s3_allow_lds(once[way], (const void*)nms, most)) return rc;
    hipLaunchKernelGGL(nms, dim3(1), dim3(kNmsThreads), (size_t)bytes, st, a);
    S3_HIP(hipGetLastError());
    return S3_OK;
}

extern "C" size_t s3_fuse_indices_workspace(int64_t n_positions) {
    if (n_positions < 1 || n_positions >= (1LL << 31)) return 0;
    return s3_align((size_t)((n_positions + kFuseBlock - 1) / kFuseBlock) * 4);
}

extern "C" int s3_fuse_indices(int64_t n_positions, const int32_t* span_lo, const int32_t* span_hi, const int32_t* n_spans,
                               int max_spans, const int32_t* extra, int64_t n_extra, int lead, int tail,
                               unsigned char* mask, int32_t* idx_out, int32_t* n_out, void* ws, size_t ws_bytes,
                               void* stream) {
    if (!mask || !idx_out || !n_out || !ws) return s3_fail(S3_EINVAL, "s3_fuse_indices: null pointer");
    if (n_positions < 1 || n_positions >= (1LL << 31))
        return s3_fail(S3_EINVAL, "s3_fuse_indices: n_positions %lld out of range", (long long)n_positions);
    if (max_spans < 0 || max_spans > 65535 || (max_spans > 0 && (!span_lo || !span_hi)))
        return s3_fail(S3_EINVAL, "s3_fuse_indices: bad span arrays (max_spans %d)", max_spans);
    if (n_extra < 0 || n_extra >= (1LL << 31) || (n_extra > 0 && !extra))
        return s3_fail(S3_EINVAL, "s3_fuse_indices: bad index list (n_extra %lld)", (long long)n_extra);
    if (lead < 0 || tail < 0) return s3_fail(S3_EINVAL, "s3_fuse_indices: lead %d / tail %d negative", lead, tail);
    const size_t need = s3_fuse_indices_workspace(n_positions);
    if (ws_bytes < need) return s3_fail(S3_ECAPACITY, "s3_fuse_indices: workspace %zu < %zu bytes", ws_bytes, need);
    if ((uintptr_t)ws & 255) return s3_fail(S3_EINVAL, "s3_fuse_indices: workspace must be 256-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    int* bsum = (int*)ws;
    const int nblocks = (int)((n_positions + kFuseBlock - 1) / kFuseBlock);
    if (n_extra + 4 * (int64_t)max_spans <= kFuseListMax && (int64_t)nblocks * (n_extra + max_spans) <= kFuseLookMax) {
        hipLaunchKernelGGL(fuse_block_kernel, dim3((unsigned)nblocks), dim3(kFuseThreads), 0, st, mask, n_positions, span_lo,
                           span_hi, n_spans, max_spans, extra, n_extra, lead, tail, bsum);
    } else {
        const unsigned gi = (unsigned)((n_positions + 255) / 256 > 4096 ? 4096 : (n_positions + 255) / 256);
        hipLaunchKernelGGL(fuse_init_kernel, dim3(gi), dim3(256), 0, st, mask, n_positions, lead, tail);
        const unsigned gm = (unsigned)max_spans + (unsigned)((n_extra + 255) / 256);
        hipLaunchKernelGGL(fuse_mark_kernel, dim3(gm), dim3(256), 0, st, mask, n_positions, span_lo, span_hi, n_spans,
                           max_spans, extra, n_extra);
        hipLaunchKernelGGL(fuse_count_kernel, dim3((unsigned)nblocks), dim3(kFuseThreads), 0, st, mask, n_positions, bsum);
    }
    const int scanned = nblocks > kFuseSelfMax;
    if (scanned) hipLaunchKernelGGL(fuse_scan_kernel, dim3(1), dim3(kFuseThreads), 0, st, bsum, nblocks, n_out);
    hipLaunchKernelGGL(fuse_compact_kernel, dim3((unsigned)nblocks), dim3(kFuseThreads), 0, st, mask, n_positions, bsum, scanned,
                       idx_out, n_out);
    S3_HIP(hipGetLastError());
    return S3_OK;
}
