// Scan encoder: the fused SAE encoder + Top-k (Sec. 3.3) of bf16, d_head 128, n_feat a multiple of 128, k <= 128, for calls that
// have scratch and enough features and tokens (s3_encode_scan_pays).
//
// What bounds it: for k <= 64 the clock and the vector instructions beside the MFMAs.  At 2048 tokens x 256 heads x 16384 features
// (k 32, a later chunk of a stream) the chip runs at 1.8 to 1.9 GHz, as it does in a large plain matrix product (1366 TFLOP/s, MFMAs
// 72 % of the cycles); MFMAs are busy 46 % of them here, vector issue 44 %.  Every vector instruction that goes, every LDS
// read and every waiting cycle counts; 2756 -> 2365 us there against the kernel with lists in LDS, 3337 -> 2146 us for 112 heads x
// 32768 features and k 64.  For k <= 128 latency: 2.3 GHz and more, 45 % of the wavefronts' cycles waiting; 1387 -> 617 us for 32
// heads (198 -> 446 TFLOP/s), one wavefront per SIMD.
//
//   - Features lie on the M axis of the 32x32x16 MFMA, tokens on N.  A wavefront has 64 tokens (two sets of 32 in registers), so that a
//     fragment of W that is read from LDS serves two MFMAs; a workgroup is four wavefronts, two workgroups share a compute unit.
//   - Every token has a threshold from the start: from the bound that a stream carries, or from a sample of the features
//     (enc_start_kernel).  What exceeds it is a candidate.  Candidates go to lists in scratch (each of the two lanes that hold
//     a token's accumulators has its own, so nothing is shared), 76 a token for k 32 and 216 for k 128 where thresholds are
//     carried.  LDS holds W alone, which is what allows two wavefronts per SIMD at every k.
//   - The accumulators of one set are looked through between the MFMAs of the next one: four quad maxima, the first quad with
//     a hit by selects under scalar masks, the first element inside it, one store: 43 to 48 vector instructions a set with the
//     ring's addresses.  (A queue of hit groups in LDS, worked off 64 at a time, cost as much again in LDS writes: 2655 us.)
//   - W comes through registers into a ring of eight 32-feature stages, a barrier every four: a wavefront that is delayed by a
//     second hit or a cut does not hold the other three up at once (2505 us with a barrier a stage).
//   - A tile ends with its selection: a lane or a few sort a token's candidates as doubles (value and id in one number),
//     merging 32 a lane at a time.  A token with fewer than k candidates started too high: its tile is walked again from -inf.
//     So the result is the exact Top-k whatever the thresholds were.
//   - Calls with few tokens split the features over workgroups; enc_join_kernel selects from all ranges' lists.
#include "s3_common.h"
#include "topk_wave.h"

#include <float.h>
#include <math.h>

namespace {

using s3topk::key_of;
using s3topk::value_of;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef f32x4 f32x4u __attribute__((aligned(4)));      // the biases may lie at any float

constexpr int DH = 128;
constexpr int RB = DH * 2;              // bytes of a row of W or x
constexpr int NS = DH / 16;             // MFMA K steps
constexpr int kFT = 32;                 // features per stage (MFMA M)
constexpr int kTokWave = 64;            // tokens per wavefront: two sets of 32 (MFMA N)
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kTokWG = kWaves * kTokWave;
constexpr int kRow = RB + 16;           // bytes of an LDS row: 16 lanes' 16-byte reads of 16 rows meet 64 banks
constexpr int kStageB = kFT * kRow;
constexpr int kPeriod = 4;              // stages between barriers
constexpr int kRing = 2 * kPeriod;      // stages in the ring: one that is read is at most kPeriod behind one that is written
constexpr int kSlots = 512;             // workgroups that run at once

constexpr int kOffBias = kRing * kStageB;
constexpr int kOffWave = kOffBias + kRing * kFT * 4;
constexpr int kWNorm = kTokWave * 4;                 // inside a wavefront's part: a value per token (threshold, later k-th value), |x|,
constexpr int kWCnt = kWNorm + kTokWave * 4;         // counts of the tokens' two lists
constexpr int kWaveB = kWCnt + 2 * kTokWave * 4;
constexpr int kLds = kOffWave + kWaves * kWaveB;
constexpr int kLanes = 2 * kTokWave;                 // lists of a wavefront: a token has one per lane that holds its accumulators
constexpr int kFront = NS - 3;          // MFMAs of a chain that run before the appends' branches
// Entries of one lane's list at which the lists are cut, and that there is room for: all of the about k survivors may be one lane's.
__host__ __device__ constexpr int cap_of(int k) { return k <= 32 ? 112 : (k <= 64 ? 168 : 208); }
constexpr int trim_regs(int G) { return G == 1 ? 64 : (G == 2 ? 96 : 144); }
constexpr int cut_regs(int G) { return (2 * cap_of(32 * G) + 63) / 64; }           // a token's two lists over 64 lanes
constexpr int kRoom = 16;                            // a lane can take this many candidates of a stage

constexpr float kHintMargin = 0.04f;    // a stream's tokens start this far below the carried bound
constexpr float kRedoMargin = 0.05f;    // bounds of a head where a token started too high are lowered by this much more

struct ScanArgs {
    const char* x;
    const char* w;
    const float* b;
    int32_t* ids;
    float* vals;
    int T, n_feat, k, n_heads;
    int tiles_per_head, n_tiles;     // 256-token tiles
    int parts, per;                  // feature ranges, stages per range
    int cap;                         // entries of a list
    int sample;                      // stages of the sample
    int vec;                         // outputs can be written 16 bytes at a time
    uint2* list;                     // [slot][wave][cap][128]
    int* count;                      // [tile][part][wave][128] (parts > 1)
    int* few;                        // [tile] whether a token has too few candidates (parts > 1)
    float* norm;                     // [n_heads * T] (parts > 1, streamed)
    float* tau0;                     // [n_heads * T]
    const float* hint;               // [n_heads][2] or null
    float* hint_next;
    unsigned* hint_out;              // [n_heads][2] ordered keys of the minima
    float* hint_sum;                 // [n_heads][3]
    int* n_fail;                     // [n_heads]
};

__device__ __forceinline__ float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float max16(const f32x16& a) {
    const float m0 = vmax(vmax(a[0], a[1]), a[2]), m1 = vmax(vmax(a[3], a[4]), a[5]), m2 = vmax(vmax(a[6], a[7]), a[8]);
    const float m3 = vmax(vmax(a[9], a[10]), a[11]), m4 = vmax(vmax(a[12], a[13]), a[14]);
    return vmax(vmax(vmax(vmax(m0, m1), a[15]), m2), vmax(m3, m4));
}
__device__ __forceinline__ float pair_fsum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ bool no_bound(const float* hint, int head) {
    return hint[2 * head] == -INFINITY && hint[2 * head + 1] == -INFINITY;
}

// The tokens of a wavefront as MFMA B operands, and |x|.
struct Tokens {
    bf16x8 a[NS], b[NS];
};
__device__ __forceinline__ void load_set(bf16x8 (&f)[NS], const char* x, int head, int T, int tok, int half) {
    const bool ok = tok < T;
    const char* row = x + ((size_t)head * T + (ok ? tok : 0)) * RB;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const uint4 u = ok ? *(const uint4*)(row + (16 * s + 8 * half) * 2) : make_uint4(0, 0, 0, 0);
        f[s] = __builtin_bit_cast(bf16x8, u);
    }
}
__device__ __forceinline__ float norm_of(const bf16x8 (&f)[NS]) {
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const u32x4 u = __builtin_bit_cast(u32x4, f[s]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float lo = __uint_as_float(u[j] << 16), hi = __uint_as_float(u[j] & 0xFFFF0000u);
            ss += lo * lo + hi * hi;
        }
    }
    return sqrtf(pair_fsum(ss));
}

// A token's list of candidates in scratch: entry i of lane list l (0 .. 127 of the wavefront) at list[128 i + l].  Token t has
// the lists of the two lanes that hold its accumulators.
__device__ __forceinline__ int list_of(int t, int half) { return (t >> 5) * 64 + half * 32 + (t & 31); }

// The lane's side of one set of 32 tokens.
struct Lane {
    float tau;
    unsigned off;            // byte offset of the end of its list
};

// Cuts the lists of the set's tokens in `which` to about k elements, one token after the other, and raises their thresholds to
// the smallest value kept: k or more elements reach it, all with lower ids than what is still to come, so an element that only
// equals it has lost.  A token's two lists (at most 64 N entries) are read once, by the whole wavefront, and searched by
// counts of ballots; what is kept is dealt to both lists in turn.  For lists that are full inside the walk, for ties and for
// few long lists.  A call takes 7000 to 10000 cycles.  When every lane searched its own list in the walk, and read it again in each
// pass because the walk leaves few registers, it took 100000 to 137000, and 1.45 million among ties: later chunks of 64 heads x 2048
// tokens x 16384 skewed features, k 32, 845 -> 735 us, of 32768 1628 -> 1537; with a row of zeros and no biases (all
// pre-activations equal), 256 x 2048 x 16384, 6647 -> 4197, k 128, 32 x 2048, 1915 -> 965.
template <int N>
__device__ __attribute__((noinline)) Lane cut_tokens(char* list, Lane l, unsigned which, int k) {
    constexpr unsigned per = kLanes * sizeof(uint2);
    const int lane = threadIdx.x & 63, loose = k + (k >> 3) + 2;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    for (; which; which &= which - 1) {
        const int t = __builtin_ctz(which);
        const unsigned o0 = (unsigned)__builtin_amdgcn_readlane((int)l.off, t), o1 = (unsigned)__builtin_amdgcn_readlane((int)l.off, t + 32);
        const float tau = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(l.tau), t));
        const int c0 = (int)(o0 / per), total = c0 + (int)(o1 / per);
        char* const p = list + o0 % per;                                       // the other list begins 32 entries of a row further
        uint2 u[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int e = i * 64 + lane;
            u[i] = *(const uint2*)(p + (e < c0 ? e * per : (e < total ? (e - c0) * per + 32 * (unsigned)sizeof(uint2) : 0u)));
        }
        unsigned key[N], id[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            key[i] = i * 64 + lane < total ? key_of(__uint_as_float(u[i].x)) : 0u;
            id[i] = u[i].y;
        }
        unsigned lo = tau > -INFINITY ? key_of(tau) : 1u;
        const unsigned idcut = s3topk::raise(key, k, loose, lo, total) > loose ? s3topk::tie_cut(key, id, k, lo) : 0xFFFFu;
        int n = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const bool keep = key[i] > lo || (key[i] == lo && id[i] <= idcut);
            const unsigned long long m = __ballot(keep);
            const unsigned at = (unsigned)(n + s3topk::below(m));
            if (keep) *(uint2*)(p + (at >> 1) * per + (at & 1) * 32 * (unsigned)sizeof(uint2)) = u[i];
            n += (int)__popcll(m);
        }
        if ((lane & 31) == t) {
            l.off = l.off % per + (unsigned)(lane < 32 ? (n + 1) >> 1 : n >> 1) * per;
            l.tau = value_of(lo);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    return l;
}
__device__ __forceinline__ unsigned tokens_of(bool lane) {           // the set's tokens of which one lane or both say so
    const unsigned long long m = __ballot(lane);
    return (unsigned)m | (unsigned)(m >> 32);
}

// Cuts the lists of 32 tokens (the set of this lane) that hold more than about k elements, all at once: every lane searches
// its own list, the two lanes of a token count theirs together.  The search for the k-th value alternates interpolation on the
// logarithm of the counts (the upper tail is close to exponential) with halving of the keys; the first NR values of a lane are
// held in registers, further ones are read again in every pass.  Few tokens are cut one by one: with skewed features most have less
// than k elements after an eighth of them, some hundreds (limits of 3 / 6 / 10 tokens, later chunks, k 32: 256 heads x 2048 tokens 2899 ->
// 2867 / 2842 / 2869 us, 64 x 4096 1396 -> 1389 / 1356 / 1373).
constexpr int kFewCuts = 6;
template <int NR, int N>
__device__ __forceinline__ Lane trim(char* list, Lane l, int k) {
    constexpr unsigned per = kLanes * sizeof(uint2);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    const int cnt = (int)(l.off / per);
    char* const p = list + l.off % per;
    const auto both = [](int x) {
        auto r = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
        return (int)(r[0] + r[1]);
    };
    const int total = both(cnt), loose = k + (k >> 3) + 2;
    bool open = total > loose;
    const unsigned few = tokens_of(open);
    if (__builtin_popcount(few) <= kFewCuts) return few ? cut_tokens<N>(list, l, few, k) : l;
    const int n = (int)s3_wave_max_u32(open ? (unsigned)cnt : 0u);
    float held[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) held[i] = *(const float*)(p + (unsigned)(i < cnt ? i : 0) * per);
#pragma unroll
    for (int i = 0; i < NR; ++i) held[i] = i < cnt ? held[i] : -INFINITY;
    const auto pass = [&](auto f) {                   // f(value) of every entry
#pragma unroll
        for (int i = 0; i < NR; ++i) f(held[i]);
        for (int i0 = NR; i0 < n; i0 += 24) {
            float v[24];
#pragma unroll
            for (int i = 0; i < 24; ++i) v[i] = *(const float*)(p + (unsigned)(i0 + i < cnt ? i0 + i : 0) * per);
#pragma unroll
            for (int i = 0; i < 24; ++i) f(i0 + i < cnt ? v[i] : -INFINITY);
        }
    };
    unsigned kmx = 0;
    pass([&](float v) { kmx = max(kmx, key_of(v)); });
    auto r = __builtin_amdgcn_permlane32_swap(kmx, kmx, false, false);
    unsigned klo = l.tau > -INFINITY ? key_of(l.tau) : key_of(-FLT_MAX), khi = max((unsigned)r[0], (unsigned)r[1]) + 1u;
    int clo = total, chi = 0;                         // entries at or above klo, khi
    bool busy = open;
    const float want = __log2f(0.5f * (float)(k + loose));
    for (bool interp = true; __any(busy); interp = !interp) {
        unsigned mid = klo + (khi - klo) / 2;
        if (interp) {
            const float llo = __log2f((float)clo), lhi = __log2f((float)max(chi, 1));
            const float t = fminf(fmaxf((llo - want) * __builtin_amdgcn_rcpf(llo - lhi), 0.0625f), 0.9375f);
            const float flo = value_of(klo), fhi = value_of(khi);
            const unsigned m = key_of(flo + (fhi - flo) * t);
            if (m > klo && m < khi) mid = m;
        }
        const float fm = value_of(mid);
        int c = 0;
        pass([&](float v) { c += v >= fm ? 1 : 0; });
        c = both(c);
        if (busy) {
            if (c >= k) { klo = mid; clo = c; } else { khi = mid; chi = c; }
            busy = clo > loose && khi - klo > 1u;
        }
    }
    const unsigned tied = tokens_of(open && clo > loose);       // more elements equal the threshold than there is room for
    open = open && clo <= loose;
    const float lo = value_of(klo);
    int m = 0;
    for (int i0 = 0; i0 < n; i0 += 16) {              // every list keeps its order; entries are read before their places are written
        uint2 u[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) u[i] = *(const uint2*)(p + (unsigned)(i0 + i < cnt ? i0 + i : 0) * per);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (open && i0 + i < cnt && __uint_as_float(u[i].x) >= lo) *(uint2*)(p + m++ * per) = u[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    if (open) {
        l.off = l.off % per + m * per;
        l.tau = lo;
    }
    if (__builtin_expect(tied != 0, 0)) l = cut_tokens<N>(list, l, tied, k);
    return l;
}

__device__ __forceinline__ void store_one(char* list, unsigned& off, float z, unsigned id) {
    *(uint2*)(list + off) = make_uint2(__float_as_uint(z), id);
    off += kLanes * sizeof(uint2);
}

// Appends what the lane's 16 accumulators hold above its token's threshold.  A stage brings a lane seldom more than one: the
// first quad that has one is picked under scalar masks, then the first element inside it.  Lanes with more take the rest one
// by one.  The masks are combined by the scalar unit.
template <int SET, int N, class Mfma>
__device__ __forceinline__ void append(const f32x16& z, Lane& l, char* list, unsigned f0, unsigned lim, int k, Mfma mfma) {
    typedef unsigned long long mask;
#pragma unroll
    for (int i = 0; i < kFront; ++i) mfma(i);
    const f32x4 q0 = __builtin_shufflevector(z, z, 0, 1, 2, 3), q1 = __builtin_shufflevector(z, z, 4, 5, 6, 7);
    const f32x4 q2 = __builtin_shufflevector(z, z, 8, 9, 10, 11), q3 = __builtin_shufflevector(z, z, 12, 13, 14, 15);
    const float tau = l.tau;
    const bool b0 = !(vmax(vmax(vmax(q0[0], q0[1]), q0[2]), q0[3]) <= tau), b1 = !(vmax(vmax(vmax(q1[0], q1[1]), q1[2]), q1[3]) <= tau);
    const bool b2 = !(vmax(vmax(vmax(q2[0], q2[1]), q2[2]), q2[3]) <= tau), b3 = !(vmax(vmax(vmax(q3[0], q3[1]), q3[2]), q3[3]) <= tau);
    f32x4 c = b2 ? q2 : q3;
    c = b1 ? q1 : c;
    c = b0 ? q0 : c;
    const bool e0 = c[0] > tau, e1 = c[1] > tau, e2 = c[2] > tau, e3 = c[3] > tau;
    float v = e2 ? c[2] : c[3];
    v = e1 ? c[1] : v;
    v = e0 ? c[0] : v;
    unsigned qb = b2 ? 16u : 24u;
    qb = b1 ? 8u : qb;
    qb = b0 ? 0u : qb;
    unsigned eb = e2 ? 2u : 3u;
    eb = e1 ? 1u : eb;
    eb = e0 ? 0u : eb;
    const mask B0 = __ballot(b0), B1 = __ballot(b1), B2 = __ballot(b2), B3 = __ballot(b3);
    const mask E0 = __ballot(e0), E1 = __ballot(e1), E2 = __ballot(e2), E3 = __ballot(e3);
    const mask R1 = E0 & E1, R2 = (E0 | E1) & E2, R3 = (E0 | E1 | E2) & E3;        // further ones in the quad
    const mask M1 = B0 & B1, M2 = (B0 | B1) & B2, M3 = (B0 | B1 | B2) & B3;        // and in other quads
    // between the chain's MFMAs
#pragma unroll
    for (int i = 0; i < kFront; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 40 / kFront, 0);
        if (SET == 0) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    mfma(kFront);
    if (__builtin_amdgcn_inverse_ballot_w64(E0 | E1 | E2 | E3)) store_one(list, l.off, v, f0 + qb + eb);
    mfma(kFront + 1);
    if (__builtin_expect((R1 | R2 | R3 | M1 | M2 | M3) != 0, 0)) {
        if ((R1 | R2 | R3) != 0) {
            if (__builtin_amdgcn_inverse_ballot_w64(R1)) store_one(list, l.off, c[1], f0 + qb + 1);
            if (__builtin_amdgcn_inverse_ballot_w64(R2)) store_one(list, l.off, c[2], f0 + qb + 2);
            if (__builtin_amdgcn_inverse_ballot_w64(R3)) store_one(list, l.off, c[3], f0 + qb + 3);
        }
        auto rest = [&](mask M, const f32x4& q, unsigned fq) {
            if (M == 0) return;
            const bool g0 = q[0] > tau, g1 = q[1] > tau, g2 = q[2] > tau;
            const mask G0 = __ballot(g0) & M, G1 = __ballot(g1) & M, G2 = __ballot(g2) & M, G3 = __ballot(q[3] > tau) & M;
            float w = g2 ? q[2] : q[3];
            w = g1 ? q[1] : w;
            w = g0 ? q[0] : w;
            unsigned e = g2 ? 2u : 3u;
            e = g1 ? 1u : e;
            e = g0 ? 0u : e;
            if (__builtin_amdgcn_inverse_ballot_w64(G0 | G1 | G2 | G3)) store_one(list, l.off, w, fq + e);
            const mask S1 = G0 & G1, S2 = (G0 | G1) & G2, S3 = (G0 | G1 | G2) & G3;
            if (__builtin_expect((S1 | S2 | S3) != 0, 0)) {
                if (__builtin_amdgcn_inverse_ballot_w64(S1)) store_one(list, l.off, q[1], fq + 1);
                if (__builtin_amdgcn_inverse_ballot_w64(S2)) store_one(list, l.off, q[2], fq + 2);
                if (__builtin_amdgcn_inverse_ballot_w64(S3)) store_one(list, l.off, q[3], fq + 3);
            }
        };
        rest(M1, q1, f0 + 8);
        rest(M2, q2, f0 + 16);
        rest(M3, q3, f0 + 24);
    }
    mfma(kFront + 2);
    if (__builtin_expect(__any(l.off > lim), 0)) {
        l = cut_tokens<N>(list, l, tokens_of(l.off > lim), k);
        __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt(0): registers restored behind the call would be waited for in every stage, and W with them
    }
}

// Walks stages [s0, s0 + ns) (ns even) of the head's features for the wavefront's tokens.  64 N: a token's entries at most.
template <int N>
__device__ __forceinline__ void scan_stages(char* smem, const ScanArgs& a, int head, int tok0, Lane& la, Lane& lb, char* list, int cap, int k,
                                            const char* wsrc, const float* bsrc, int s0, int ns, bool active) {
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, half = lane >> 5;
    const char* const wp = wsrc + (size_t)s0 * kFT * RB;
    const float* const bp = bsrc + s0 * kFT;
    const int last = ns - 1;
    const unsigned goff = (unsigned)(tid * 16);                       // 256 threads x 16 bytes: half a stage
    char* const wdst = smem + (tid >> 4) * kRow + (tid & 15) * 16;
    const char* const fsrc = smem + n * kRow + half * 16;
    const char* const csrc = smem + kOffBias + half * 16;

    u32x4 r0[2], r1[2];
    float b0, b1;
    auto gload = [&](u32x4 (&r)[2], float& bb, int s) {
        const int sc = min(s, last);
        const char* p = wp + (size_t)sc * (kFT * RB);
        r[0] = *(const u32x4*)(p + goff);
        r[1] = *(const u32x4*)(p + goff + kThreads * 16);
        bb = bp[sc * kFT + (tid & 31)];
    };
    auto put = [&](const u32x4 (&r)[2], float bb, int slot) {
        *(u32x4*)(wdst + slot * kStageB) = r[0];
        *(u32x4*)(wdst + slot * kStageB + 16 * kRow) = r[1];
        if (tid < 32) *(float*)(smem + kOffBias + slot * (kFT * 4) + tid * 4) = bb;
    };
    Tokens tk;                             // loaded first: what is waited for below arrives later
    load_set(tk.a, a.x, head, a.T, tok0 + n, half);
    load_set(tk.b, a.x, head, a.T, tok0 + 32 + n, half);
    gload(r0, b0, 0);
    gload(r1, b1, 1);
    __syncthreads();                       // the ring may still be read by the walk before
#pragma unroll
    for (int s = 0; s < kPeriod; s += 2) {
        put(r0, b0, s);
        put(r1, b1, s + 1);
        gload(r0, b0, s + 2);
        gload(r1, b1, s + 3);
    }
    lds_barrier();

    // Stage s writes stage s + kPeriod and reads the fragments of stage s + 1 behind a barrier in every kPeriod-th stage.
    if (!active) {
        for (int s = 0; s < ns; s += 2) {
            put(r0, b0, (s + kPeriod) % kRing);
            gload(r0, b0, s + kPeriod + 2);
            if (s % kPeriod == 0) lds_barrier();
            put(r1, b1, (s + 1 + kPeriod) % kRing);
            gload(r1, b1, s + kPeriod + 3);
        }
        return;
    }

    bf16x8 f[NS];
    f32x16 c, accA, accB;
    auto fread = [&](int s, int slot) { return *(const bf16x8*)(fsrc + slot * kStageB + s * 32); };
    auto cread = [&](int slot, int q) {
        const f32x4 u = *(const f32x4*)(csrc + slot * (kFT * 4) + q * 32);
        c[4 * q] = u[0]; c[4 * q + 1] = u[1]; c[4 * q + 2] = u[2]; c[4 * q + 3] = u[3];
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) f[s] = fread(s, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) cread(0, q);
#pragma unroll
    for (int i = 0; i < 16; ++i) accB[i] = -INFINITY;      // set B of the stage before the first: above no threshold
    const unsigned lim = (unsigned)((cap - kRoom) * kLanes * sizeof(uint2));      // an end at or above leaves no room for a stage
    const unsigned fh = (unsigned)half * 4;

    auto stage = [&](u32x4 (&r)[2], float& bb, int s, bool sync) {
        const int nxt = (s + 1) % kRing;
        put(r, bb, (s + kPeriod) % kRing);
        gload(r, bb, s + kPeriod + 2);
        append<1, N>(accB, lb, list, (unsigned)(s0 + s - 1) * kFT + fh, lim, k, [&](int i) {
            accA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], tk.a[i], i ? accA : c, 0, 0, 0);
        });
        if (sync) lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
        append<0, N>(accA, la, list, (unsigned)(s0 + s) * kFT + fh, lim, k, [&](int i) {
            accB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], tk.b[i], i ? accB : c, 0, 0, 0);
            f[i] = fread(i, nxt);
            if (i < 4) cread(nxt, i);
        });
    };
    for (int s = 0; s < ns; s += 2) {
        if ((s & 31) == 0) {               // the older workgroup of a compute unit would win every conflict: they take turns (1-2 %)
            if (((s >> 5) ^ (blockIdx.x >> 8)) & 1) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
        stage(r0, b0, s, s % kPeriod == 0);
        stage(r1, b1, s + 1, false);
    }
    append<1, N>(accB, lb, list, (unsigned)(s0 + ns - 1) * kFT + fh, lim, k, [](int) {});
}

// ------------------------------------------------------------------------------------------------ selection
// A candidate as one number: (value descending, id ascending) is the descending order of these doubles.  48 bits (the
// value's ordered key, the complement of the id) in the mantissa of [1, 2); 0 is no candidate.  Compare-exchange is one
// v_max_f64 and one v_min_f64.
__device__ __forceinline__ double pack(float z, unsigned id) {
    const unsigned u = __float_as_uint(z + 0.f);
    const unsigned key = u ^ ((unsigned)((int)u >> 31) | 0x80000000u);
    return __hiloint2double((int)(0x3FF00000u | (key >> 12)), (int)((key << 20) | ((id ^ 0xFFFFu) << 4)));
}
__device__ __forceinline__ unsigned pack_id(double d) { return (((unsigned)__double2loint(d) >> 4) & 0xFFFFu) ^ 0xFFFFu; }
__device__ __forceinline__ float pack_value(double d) {
    return value_of(((unsigned)__double2hiint(d) << 12) | ((unsigned)__double2loint(d) >> 20));
}

constexpr int E = 32;                   // candidates per lane
__device__ __forceinline__ void exch(double& a, double& b) {       // a >= b afterwards
    const double x = fmax(a, b), y = fmin(a, b);
    a = x;
    b = y;
}
template <int D>
__device__ __forceinline__ void clean(double (&v)[E]) {            // bitonic sequences of 2 D -> descending
#pragma unroll
    for (int i = 0; i < E; ++i)
        if ((i & D) == 0) exch(v[i], v[i + D]);
    if constexpr (D > 1) clean<D / 2>(v);
}
template <int S>
__device__ __forceinline__ void sort_to(double (&v)[E]) {          // runs of S descending
    if constexpr (S > 1) {
        sort_to<S / 2>(v);
#pragma unroll
        for (int i = 0; i < E; ++i)
            if ((i & (S / 2)) == 0 && (i & (S - 1)) < S / 2) exch(v[i], v[(i & ~(S - 1)) + S - 1 - (i & (S - 1))]);
        if constexpr (S > 2) clean<S / 4>(v);
    }
}
template <int X>
__device__ __forceinline__ double lane_xor(double d) {             // the value of lane ^ X, X = 1 .. 7
    if constexpr (X > 3) {                                         // lanes of eight mirrored, then inside four
        d = __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(d), 0x141, 0xf, 0xf, true),
                             __builtin_amdgcn_update_dpp(0, __double2loint(d), 0x141, 0xf, 0xf, true));
        if constexpr (X == 7) return d;
        else return lane_xor<X ^ 7>(d);
    } else {
    constexpr int ctrl = X == 1 ? 0xB1 : (X == 2 ? 0x4E : 0x1B);
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(d), ctrl, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(d), ctrl, 0xf, 0xf, true));
    }
}
template <int X>
__device__ __forceinline__ void lane_clean(double (&v)[E], int q) {
    const bool up = (q & X) == 0;
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const double o = lane_xor<X>(v[i]);
        const double x = fmax(v[i], o), y = fmin(v[i], o);
        v[i] = up ? x : y;
    }
}
template <int X>
__device__ __forceinline__ void lane_fold(double (&v)[E], int q) { // lanes q, q ^ X (X = 1, 3) each descending -> the larger half below
    const bool up = (q & ((X + 1) / 2)) == 0;
#pragma unroll
    for (int i = 0; i < E / 2; ++i) {
        const double o = lane_xor<X>(v[E - 1 - i]), p = lane_xor<X>(v[i]);
        const double x0 = fmax(v[i], o), y0 = fmin(v[i], o), x1 = fmax(v[E - 1 - i], p), y1 = fmin(v[E - 1 - i], p);
        v[i] = up ? x0 : y0;
        v[E - 1 - i] = up ? x1 : y1;
    }
}
// G lanes of E candidates each -> descending over lane, then register
template <int G>
__device__ __forceinline__ void sort_lanes(double (&v)[E], int q) {
    sort_to<E>(v);
    if constexpr (G >= 2) {
        lane_fold<1>(v, q);
        clean<E / 2>(v);
    }
    if constexpr (G >= 4) {
        lane_fold<3>(v, q);
        lane_clean<1>(v, q);
        clean<E / 2>(v);
    }
}
// top <- the G E largest of top and v (both sorted)
template <int G>
__device__ __forceinline__ void merge_top(double (&top)[E], const double (&v)[E], int q) {
#pragma unroll
    for (int i = 0; i < E; ++i) {
        double o = v[E - 1 - i];
        if constexpr (G == 2) o = lane_xor<1>(o);
        if constexpr (G == 4) o = lane_xor<3>(o);
        top[i] = fmax(top[i], o);
    }
    if constexpr (G >= 4) lane_clean<2>(top, q);
    if constexpr (G >= 2) lane_clean<1>(top, q);
    clean<E / 2>(top);
}

// The sorted candidates of a lane (ranks q E .. of token t) -> the token's row; kth[t] (LDS): its k-th value.
template <int G>
__device__ __forceinline__ void write_rows(const ScanArgs& a, const double (&top)[E], int head, int tok0, int t, int q, bool ok, float* kth) {
    const int k = a.k, e0 = q * E;
    const size_t row = ((size_t)head * a.T + tok0 + t) * k;
    float last = -INFINITY;
#pragma unroll
    for (int j = 0; j < E; j += 4) {
        int id[4];
        float z[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            id[i] = (int)pack_id(top[j + i]);
            const float zz = pack_value(top[j + i]);
            if (e0 + j + i == k - 1 && top[j + i] >= 1.0) last = zz;
            z[i] = fmaxf(zz, 0.f);
        }
        if (ok && a.vec && e0 + j < k) {
            *(int4*)(a.ids + row + e0 + j) = make_int4(id[0], id[1], id[2], id[3]);
            *(float4*)(a.vals + row + e0 + j) = make_float4(z[0], z[1], z[2], z[3]);
        } else if (ok) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (e0 + j + i < k) {
                    a.ids[row + e0 + j + i] = id[i];
                    a.vals[row + e0 + j + i] = z[i];
                }
        }
    }
    if (ok && (k - 1) / E == q) kth[t] = last;
}

// Selects, orders and writes the k best of the wavefront's tokens in `which`, 64 / G at a time: the two lists are taken G E
// entries at a time, each sorted and merged into the best so far.  cnt (LDS): the wavefront's 128 counts.
template <int G>
__device__ __forceinline__ void select_list(const ScanArgs& a, int head, int tok0, const uint2* list, const int* cnt,
                                            unsigned long long which, float* kth) {
    const int lane = threadIdx.x & 63, q = lane % G;
    for (int tb = 0; tb < kTokWave; tb += 64 / G) {
        const int t = tb + lane / G, ts = t;
        const bool ok = ((which >> t) & 1) && tok0 + t < a.T;
        if (!__any(ok)) continue;
        const int n0 = ok ? cnt[list_of(ts, 0)] : 0, n = ok ? n0 + cnt[list_of(ts, 1)] : 0;
        const int nmax = (int)s3_wave_max_u32((unsigned)n);
        const uint2* const lp = list + list_of(ts, 0);
        double top[E];
        for (int e0 = 0; e0 == 0 || e0 < nmax; e0 += E * G) {
            uint2 u[E];
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const int e = e0 + j * G + q;
                u[j] = lp[(unsigned)(e < n0 ? e * kLanes : (e < n ? (e - n0) * kLanes + 32 : 0))];
            }
            double v[E];
#pragma unroll
            for (int j = 0; j < E; ++j) v[j] = e0 + j * G + q < n ? pack(__uint_as_float(u[j].x), u[j].y) : 0.0;
            sort_lanes<G>(v, q);
            if (e0 == 0) {
#pragma unroll
                for (int j = 0; j < E; ++j) top[j] = v[j];
            } else {
                merge_top<G>(top, v, q);
            }
        }
        write_rows<G>(a, top, head, tok0, t, q, ok, kth);
    }
}

// Rows with fewer than k elements above -inf: the lowest other ids, value 0.
__device__ __attribute__((noinline)) void fill_row(const uint2* list, int t, int n0, int n1, int k, int32_t* ids, float* vals) {
    s3topk::fill_short(k, n0 + n1, [&](int s) {
        return s < n0 ? list[(size_t)s * kLanes + list_of(t, 0)].y : list[(size_t)(s - n0) * kLanes + list_of(t, 1)].y;
    }, ids, vals);
}

// ------------------------------------------------------------------------------------------------ kernels
// Walks the features for 256 tokens per workgroup.  Whole tiles (parts == 1): a workgroup takes one tile after the other and
// selects at the end of each.  Ranges (parts > 1): lists and counts stay in scratch for enc_join_kernel (REDO), which selects
// from all ranges' lists.  Tokens whose first threshold was too high are walked again, from -inf, by either.
template <int G, bool REDO>
__global__ __launch_bounds__(kThreads, 2) void enc_scan_kernel(ScanArgs a) {
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, half = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t wstride = (size_t)a.cap * kLanes;
    const int nst = a.n_feat / kFT;
    char* const mem = smem + kOffWave + wv * kWaveB;
    float* const kth = (float*)mem;            // per token: the first threshold, then the k-th value
    float* const norm = (float*)(mem + kWNorm);
    int* const cnt = (int*)(mem + kWCnt);
    const int parts = REDO ? 1 : a.parts;      // ranges that are workgroups of their own here

    for (int unit = blockIdx.x; unit < a.n_tiles * parts; unit += gridDim.x) {
        int group, tt;
        s3_block_to_tile((unsigned)unit, a.n_heads * parts, a.tiles_per_head, group, tt);
        // Where a turn takes whole heads, a workgroup would take the same tile of a head every time: it moves on by one.  Rows that are
        // walked twice often stand at one place in all heads (padding, a first token).  One row of zeros a head and no biases,
        // 256 heads x 2048 tokens, k 32: 4077 -> 3150 us.
        if (__builtin_expect(!REDO && unit >= (int)gridDim.x, 0) && (gridDim.x >> 3) % (unsigned)a.tiles_per_head == 0)
            tt = (tt + unit / (int)gridDim.x) % a.tiles_per_head;
        const int head = group / parts, part = group - head * parts;
        const int tok0 = tt * kTokWG + wv * kTokWave;
        const bool active = tok0 < a.T, mine = tok0 + lane < a.T;     // lane t answers for token t of the wavefront
        const int tile = head * a.tiles_per_head + tt;
        if (REDO && a.few[tile] == 0) continue;
        const size_t slot = a.parts > 1 ? (size_t)tile * a.parts + part : blockIdx.x;
        uint2* const list = a.list + (slot * kWaves + wv) * wstride;
        int* const count = a.count + (size_t)tile * a.parts * (kWaves * kLanes) + wv * kLanes;
        const char* const wh = a.w + (size_t)head * a.n_feat * RB;
        const float* const bh = a.b + (size_t)head * a.n_feat;
        float start = -INFINITY;
        if (!REDO && active) {
            float xn;
            {
                bf16x8 xa[NS], xb[NS];
                load_set(xa, a.x, head, a.T, tok0 + n, half);
                load_set(xb, a.x, head, a.T, tok0 + 32 + n, half);
                const float na = norm_of(xa), nb = norm_of(xb);
                xn = half ? nb : na;
            }
            if (a.hint && !no_bound(a.hint, head)) {
                // carried bounds, lowered by a margin (one of the two is -inf; a bound that is still too high costs a second walk)
                const float hr = a.hint[2 * head], ha = a.hint[2 * head + 1];
                const float t0 = fmaxf(hr > -INFINITY ? hr * xn : -INFINITY, ha);
                const float t1 = t0 - kHintMargin * fabsf(t0);         // a NaN where the bound is infinite
                start = t1 > -INFINITY ? t1 : -INFINITY;
            } else if (mine) {
                start = a.tau0[(size_t)head * a.T + tok0 + lane];
            }
            s3_wave_fence();
            norm[lane] = xn;
            kth[lane] = mine ? start : INFINITY;
            if (a.norm && part == 0 && mine) a.norm[(size_t)head * a.T + tok0 + lane] = xn;
            s3_wave_fence();
        }
        Lane la, lb;
        const unsigned offA = (unsigned)lane * sizeof(uint2), offB = offA + 64 * sizeof(uint2);
        if (!REDO) {
            la = Lane{kth[n], offA};
            lb = Lane{kth[32 + n], offB};
        }
        bool bad = false;
        unsigned long long again = 0;
        bool walk = !REDO, go = active, second = false, rough = false;      // walk, second, rough: the same for the whole workgroup
        int s0 = part * a.per, ns = min(a.per, nst - s0);
        for (;;) {
            if (walk) {
                // An eighth, a quarter and half way, what k or more elements reach by then raises thresholds that were low; where
                // an eighth brings few lanes a quarter of k and none half of it, the thresholds are good and the rest is walked in one go.
                int from = s0, to = min(s0 + ns, nst);
                const int end = to;
                if (parts == 1 && ns >= 64) to = s0 + (ns >> 4) * 2;
                for (;;) {
                    scan_stages<cut_regs(G)>(smem, a, head, tok0, la, lb, (char*)list, a.cap, a.k, wh, bh, from, to - from, go);
                    if (to >= end) break;
                    constexpr unsigned per = kLanes * sizeof(uint2);
                    const unsigned many = (unsigned)(a.k - (a.k >> 2)) * per;
                    if (from == s0) {
                        const unsigned most = max(la.off, lb.off);
                        const bool some = go && most > (unsigned)(a.k >> 2) * per, dense = go && most > (unsigned)max(a.k >> 1, 16) * per;
                        rough = __syncthreads_count(some) + kThreads * (dense ? 1 : 0) > kThreads / 4;
                        rough = __syncthreads_or(rough);
                    }
                    if (go && __any(la.off > many)) la = trim<trim_regs(G), cut_regs(G)>((char*)list, la, a.k);
                    if (go && __any(lb.off > many)) lb = trim<trim_regs(G), cut_regs(G)>((char*)list, lb, a.k);
                    from = to;
                    to = rough ? min(s0 + 2 * (to - s0), end) : end;
                }
                s3_wave_fence();
                if (go && (second ? (again >> n) & 1 : true)) cnt[lane] = la.off / (kLanes * sizeof(uint2));
                if (go && (second ? (again >> (32 + n)) & 1 : true)) cnt[64 + lane] = lb.off / (kLanes * sizeof(uint2));
                s3_wave_fence();
            }
            if ((!REDO && a.parts > 1) || second) break;
            if (active && mine) {
                int total = 0;
                if (REDO)
#pragma unroll 8
                    for (int p = 0; p < 2 * a.parts; ++p) total += count[(p >> 1) * (kWaves * kLanes) + list_of(lane, p & 1)];
                else
                    total = cnt[list_of(lane, 0)] + cnt[list_of(lane, 1)];
                bad = total < a.k && (REDO || start > -INFINITY);
            }
            again = __ballot(bad);
            if (__builtin_expect(!__syncthreads_or(again != 0), 1)) break;
            // Tokens that started too high are walked again, from -inf.
            la = Lane{(again >> n) & 1 ? -INFINITY : INFINITY, offA};
            lb = Lane{(again >> (32 + n)) & 1 ? -INFINITY : INFINITY, offB};
            walk = second = true;
            go = again != 0;
            s0 = 0;
            ns = nst;
        }
        if (!REDO && a.parts > 1) {
            if (active) {
                count[part * (kWaves * kLanes) + lane] = cnt[lane];
                count[part * (kWaves * kLanes) + 64 + lane] = cnt[64 + lane];
            }
            continue;
        }
        if (!active) continue;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        if (REDO) {
            if (again == 0) continue;
            if (a.norm && mine) norm[lane] = a.norm[(size_t)head * a.T + tok0 + lane];
            if (!bad) kth[lane] = -INFINITY;           // answered for already
            s3_wave_fence();
        }
        select_list<G>(a, head, tok0, list, cnt, REDO ? again : ~0ull, kth);
        s3_wave_fence();
        for (unsigned long long few = __ballot(mine && (!REDO || bad) && cnt[list_of(lane, 0)] + cnt[list_of(lane, 1)] < a.k); few; few &= few - 1) {
            const int t = __builtin_ctzll(few);
            const size_t row = ((size_t)head * a.T + tok0 + t) * a.k;
            fill_row(list, t, cnt[list_of(t, 0)], cnt[list_of(t, 1)], a.k, a.ids + row, a.vals + row);
        }
        if (a.hint) {
            // the minima over the call (of tau / |x| and of tau) are the bounds that are carried on; the sums tell which of
            // the two was the tighter one
            const float z = mine ? kth[lane] : -INFINITY, xn = mine ? norm[lane] : 0.f;
            const bool use = z > -INFINITY;
            float r = use && xn > 0.f ? z / xn : INFINITY, m = use ? z : INFINITY;
            float s_tau = use ? z : 0.f, s_x = use ? xn : 0.f, s_n = use ? 1.f : 0.f;
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) {
                r = fminf(r, __shfl_xor(r, d));
                m = fminf(m, __shfl_xor(m, d));
                s_tau += __shfl_xor(s_tau, d);
                s_x += __shfl_xor(s_x, d);
                s_n += __shfl_xor(s_n, d);
            }
            if (lane == 0) {
                if (r < INFINITY) atomicMin(&a.hint_out[2 * head], key_of(r));
                if (m < INFINITY) atomicMin(&a.hint_out[2 * head + 1], key_of(m));
                if (s_n > 0.f) {
                    atomicAdd(&a.hint_sum[3 * head], s_tau);
                    atomicAdd(&a.hint_sum[3 * head + 1], s_x);
                    atomicAdd(&a.hint_sum[3 * head + 2], s_n);
                }
                if (again) atomicAdd(&a.n_fail[head], (int)__popcll(again));
            }
        }
    }
}

// Selects from the lists that the ranges of the features left, a wavefront per token.  Tokens
// that have too few candidates (a first threshold that was too high) are left to the walk behind this.
//
// TOK: tokens per workgroup.  Sixteen where they carry bounds, which then go to the head's in one go (additions to a head's few
// values from 128 workgroups were half of the time: 4096 tokens of 8 heads, k 32, 33 -> 18 us); else four, which leave their
// compute unit earlier (16384 tokens, k 32: 48 / 31).
// LR 4 (k > 64): the list is sorted whole; ranks by a comparison of every survivor with every other one, after a cut to about k of
// them, are two and a half times the instructions (4096 tokens, k 128: 33 -> 23 us).
template <int X>
__device__ __forceinline__ double wave_xor(double d) {     // the value of lane ^ X
    if constexpr (X <= 7) return lane_xor<X>(d);
    else if constexpr (X == 8 || X == 15) {
        constexpr int ctrl = X == 8 ? 0x128 : 0x140;       // rows of 16 turned by eight, mirrored
        return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(d), ctrl, 0xf, 0xf, true),
                                __builtin_amdgcn_update_dpp(0, __double2loint(d), ctrl, 0xf, 0xf, true));
    } else return __hiloint2double(__shfl_xor(__double2hiint(d), X), __shfl_xor(__double2loint(d), X));
}
template <int X>
__device__ __forceinline__ void wave_step(double (&v)[4], int lane, bool mirrored) {       // the larger ones to the lower lane of each pair
    constexpr int top = X <= 1 ? 1 : (X <= 3 ? 2 : (X <= 7 ? 4 : (X <= 15 ? 8 : (X <= 31 ? 16 : 32))));
    const bool up = (lane & top) == 0;
    double o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = wave_xor<X>(v[mirrored ? 3 - i : i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double x = fmax(v[i], o[i]), y = fmin(v[i], o[i]);
        v[i] = up ? x : y;
    }
}
template <int N>
__device__ __forceinline__ void wave_clean(double (&v)[4], int lane) {      // bitonic over N lanes -> descending
    if constexpr (N >= 2) {
        wave_step<N / 2>(v, lane, false);
        wave_clean<N / 2>(v, lane);
    } else {
        exch(v[0], v[2]); exch(v[1], v[3]);
        exch(v[0], v[1]); exch(v[2], v[3]);
    }
}
template <int N>
__device__ __forceinline__ void wave_sort(double (&v)[4], int lane) {       // place 4 lane + i, descending inside N lanes
    if constexpr (N == 1) {
        exch(v[0], v[1]); exch(v[2], v[3]);
        exch(v[0], v[3]); exch(v[1], v[2]);
        exch(v[0], v[1]); exch(v[2], v[3]);
    } else {
        wave_sort<N / 2>(v, lane);
        wave_step<N - 1>(v, lane, true);
        wave_clean<N / 2>(v, lane);
    }
}
template <int LR, int TOK>
__global__ __launch_bounds__(64 * TOK) void enc_join_kernel(ScanArgs a) {
    __shared__ float lval[TOK][64 * LR];
    __shared__ uint16_t lid[TOK][64 * LR];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __shared__ float seen[TOK][2];             // k-th value and |x| of the block's tokens
    constexpr int kPerBlock = TOK, kU = TOK > 4 ? 8 : 4;        // kU: loads in flight per lane
    const int tile = blockIdx.x / (kTokWG / kPerBlock), t = (blockIdx.x % (kTokWG / kPerBlock)) * kPerBlock + wv;
    const int head = tile / a.tiles_per_head, tok0 = (tile - head * a.tiles_per_head) * kTokWG;
    const int lists = 2 * a.parts, log2n = 32 - __builtin_clz((unsigned)(lists - 1)), p = lane & ((1 << log2n) - 1);
    const int slot = lane >> log2n, step = 64 >> log2n;
    const size_t wstride = (size_t)a.cap * kLanes;
    float z = -INFINITY, xn = 0.f;
    if (tok0 + t < a.T) {
        const int w = t >> 6, l = list_of(t & 63, p & 1);
        const size_t part = (size_t)tile * a.parts + (p >> 1);
        const int c = p < lists ? a.count[part * (kWaves * kLanes) + w * kLanes + l] : 0;
        const int incl = s3_wave_incl_scan(lane < lists ? c : 0);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        if (total < a.k && lane == 0) a.few[tile] = 1;
        if (total >= a.k) {
            const uint2* const src = a.list + (part * kWaves + w) * wstride + l;
            const int most = (int)s3_wave_max_u32((unsigned)c);
            s3_wave_fence();
            int n = 0;
            float tau = -INFINITY;
            for (int i0 = 0; i0 < most; i0 += kU * step) {
                uint2 u[kU];
#pragma unroll
                for (int j = 0; j < kU; ++j) {
                    const int i = i0 + j * step + slot;
                    u[j] = i < c ? src[(size_t)i * kLanes] : make_uint2(__float_as_uint(-INFINITY), 0u);
                }
                float v[kU];
#pragma unroll
                for (int j = 0; j < kU; ++j) v[j] = __uint_as_float(u[j].x);
                const float before = tau;
                s3topk::take<kU, LR>(v, [&](int j) { return u[j].y; }, a.k, a.k + (a.k >> 3) + 2, lval[wv], lid[wv], n, tau);
                // the elements come in no order of ids: one that equals the threshold may still belong to the k best
                if (tau != before) {
                    const unsigned key = key_of(tau);
                    tau = value_of(key == 0x80000000u ? key - 2 : key - 1);        // below 0 comes the first negative, not -0
                }
            }
            const size_t row = ((size_t)head * a.T + tok0 + t) * a.k;
            if constexpr (LR == 4) {
                double v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = i * 64 + lane < n ? pack(lval[wv][i * 64 + lane], lid[wv][i * 64 + lane]) : 0.0;
                wave_sort<64>(v, lane);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * lane + i < a.k) {
                        const float zi = pack_value(v[i]);
                        a.ids[row + 4 * lane + i] = (int32_t)pack_id(v[i]);
                        a.vals[row + 4 * lane + i] = fmaxf(zi, 0.f);
                        if (4 * lane + i == a.k - 1) z = zi;
                    }
            } else {
                unsigned key[LR], id[LR];
                int rank[LR];
                s3topk::finish<LR>(a.k, lval[wv], lid[wv], n, key, id, rank);
#pragma unroll
                for (int i = 0; i < LR; ++i)
                    if (rank[i] >= 0) {
                        a.ids[row + rank[i]] = (int32_t)id[i];
                        a.vals[row + rank[i]] = fmaxf(value_of(key[i]), 0.f);
                        if (rank[i] == a.k - 1) z = value_of(key[i]);
                    }
            }
            if (a.hint) {
                z = value_of(s3_wave_max_u32(key_of(z)));
                xn = a.norm[(size_t)head * a.T + tok0 + t];
            }
        }
    }
    if (!a.hint) return;
    if (lane == 0) {
        seen[wv][0] = z;
        seen[wv][1] = xn;
    }
    __syncthreads();
    if (threadIdx.x >= TOK) return;
    const float zq = seen[threadIdx.x][0], xq = seen[threadIdx.x][1];
    const bool use = zq > -INFINITY;
    float r = use && xq > 0.f ? zq / xq : INFINITY, m = use ? zq : INFINITY, s_tau = use ? zq : 0.f, s_x = use ? xq : 0.f, s_n = use ? 1.f : 0.f;
#pragma unroll
    for (int d = TOK / 2; d > 0; d >>= 1) {
        r = fminf(r, __shfl_xor(r, d));
        m = fminf(m, __shfl_xor(m, d));
        s_tau += __shfl_xor(s_tau, d);
        s_x += __shfl_xor(s_x, d);
        s_n += __shfl_xor(s_n, d);
    }
    if (threadIdx.x == 0 && s_n > 0.f) {
        if (r < INFINITY) atomicMin(&a.hint_out[2 * head], key_of(r));
        atomicMin(&a.hint_out[2 * head + 1], key_of(m));
        atomicAdd(&a.hint_sum[3 * head], s_tau);
        atomicAdd(&a.hint_sum[3 * head + 1], s_x);
        atomicAdd(&a.hint_sum[3 * head + 2], s_n);
    }
}

// First thresholds of tokens whose head carries no bound: the R-th largest maximum of 16 features over every eighth stage, the
// smaller one of the token's two lanes.  R is 3 standard deviations above the number that the sample is expected to hold of the k best, so
// about one token in 10^6 starts too high; the others have about 16 R candidates (128 for k 32).
// WS == 1: a wavefront has 64 tokens, and the workgroup's four share the stages through LDS, two a barrier, two more on their way.  Each
// read its fragments from L2 before: 16 bytes of 32 rows a load, which the address unit of a compute unit took as long for as three
// times the MFMAs (256 heads x 2048 tokens, k 32: 654 -> 290 us).  WS > 1: that many wavefronts share 64 tokens' stages, W straight from
// L2 (a stage is read by one of them only).
template <int R, int WS>
__global__ __launch_bounds__(kThreads) void enc_start_kernel(ScanArgs a) {
    __shared__ float part[WS > 1 ? WS : 1][2][WS > 1 ? R : 1][64];
    __shared__ __align__(16) char ring[WS > 1 ? 16 : 4 * kStageB];      // two pairs of stages: one is read, the other written
    __shared__ __align__(16) float ring_b[4][kFT];
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, half = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (a.hint && blockIdx.x == 0) {           // streamed calls: the call's minima and sums start empty
        for (int i = tid; i < a.n_heads; i += kThreads) a.n_fail[i] = 0;
        for (int i = tid; i < 2 * a.n_heads; i += kThreads) a.hint_out[i] = 0xFFFFFFFFu;
        for (int i = tid; i < 3 * a.n_heads; i += kThreads) a.hint_sum[i] = 0.f;
    }
    if (a.parts > 1 && blockIdx.x == 0)
        for (int i = tid; i < a.n_tiles; i += kThreads) a.few[i] = 0;
    constexpr int kTok = WS > 1 ? kTokWave : kTokWG;
    const int per_head = (a.T + kTok - 1) / kTok;
    for (int unit = blockIdx.x; unit < a.n_heads * per_head; unit += gridDim.x) {
        int head, tt;
        s3_block_to_tile((unsigned)unit, a.n_heads, per_head, head, tt);
        if (a.hint && !no_bound(a.hint, head)) continue;
        const int tok0 = tt * kTok + (WS > 1 ? 0 : wv * kTokWave);
        Tokens tk;
        load_set(tk.a, a.x, head, a.T, tok0 + n, half);
        load_set(tk.b, a.x, head, a.T, tok0 + 32 + n, half);
        const int nst = a.n_feat / kFT;
        float la[R], lb[R];
#pragma unroll
        for (int i = 0; i < R; ++i) la[i] = lb[i] = -INFINITY;
        auto insert = [](float (&l)[R], float m) {
#pragma unroll
            for (int i = R - 1; i > 0; --i) l[i] = __builtin_amdgcn_fmed3f(l[i - 1], l[i], m);
            l[0] = fmaxf(l[0], m);
        };
        auto stage_of = [&](int j) { return (int)((long long)min(j, a.sample - 1) * nst / a.sample); };
        auto product = [&](bf16x8 (&f)[NS], const f32x16& c, auto between) {
            f32x16 accA = c, accB = c;
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                accA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], tk.a[i], accA, 0, 0, 0);
                accB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i], tk.b[i], accB, 0, 0, 0);
            }
            between();                             // the fragments are used up
            insert(la, max16(accA));
            insert(lb, max16(accB));
        };
        if constexpr (WS == 1) {
            u32x4 r[4];
            float bb;
            auto gload = [&](int j) {
                const char* const w0 = a.w + ((size_t)head * a.n_feat + (size_t)stage_of(j) * kFT) * RB + tid * 16;
                const char* const w1 = a.w + ((size_t)head * a.n_feat + (size_t)stage_of(j + 1) * kFT) * RB + tid * 16;
                r[0] = *(const u32x4*)w0;
                r[1] = *(const u32x4*)(w0 + kThreads * 16);
                r[2] = *(const u32x4*)w1;
                r[3] = *(const u32x4*)(w1 + kThreads * 16);
                bb = a.b[(size_t)head * a.n_feat + stage_of(j + (lane >> 5)) * kFT + n];
            };
            auto put = [&](int pair) {
                char* const dst = ring + pair * (2 * kStageB) + (tid >> 4) * kRow + (tid & 15) * 16;
#pragma unroll
                for (int i = 0; i < 4; ++i) *(u32x4*)(dst + i * (16 * kRow)) = r[i];
                if (tid < 64) ring_b[2 * pair + half][n] = bb;
            };
            auto take = [&](int slot) {
                bf16x8 f[NS];
                f32x16 c;
                const char* const src = ring + slot * kStageB + n * kRow + half * 16;
#pragma unroll
                for (int i = 0; i < NS; ++i) f[i] = *(const bf16x8*)(src + i * 32);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 u = *(const f32x4*)&ring_b[slot][half * 4 + q * 8];
                    c[4 * q] = u[0]; c[4 * q + 1] = u[1]; c[4 * q + 2] = u[2]; c[4 * q + 3] = u[3];
                }
                product(f, c, [] {});
            };
            gload(0);
            put(0);
            gload(2);
            lds_barrier();
            for (int j = 0; j < a.sample; j += 2) {
                const int pair = (j >> 1) & 1;
                put(pair ^ 1);                     // read in the turn before, behind the barrier at its end
                gload(j + 4);
                take(2 * pair);
                if (j + 1 < a.sample) take(2 * pair + 1);
                lds_barrier();
            }
        } else {
            const char* const wp = a.w + (size_t)head * a.n_feat * RB + n * RB + half * 16;
            const float* const bp = a.b + (size_t)head * a.n_feat + half * 4;
            bf16x8 f[NS];
            f32x16 c;
            auto load = [&](int j) {
                const int s = stage_of(j);
#pragma unroll
                for (int i = 0; i < NS; ++i) f[i] = *(const bf16x8*)(wp + (size_t)s * kFT * RB + i * 32);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 u = *(const f32x4u*)(bp + s * kFT + q * 8);
                    c[4 * q] = u[0]; c[4 * q + 1] = u[1]; c[4 * q + 2] = u[2]; c[4 * q + 3] = u[3];
                }
            };
            load(wv);
            for (int j = wv; j < a.sample; j += WS) product(f, c, [&] { load(j + WS); });
        }
        if constexpr (WS > 1) {
#pragma unroll
            for (int i = 0; i < R; ++i) { part[wv][0][i][lane] = la[i]; part[wv][1][i][lane] = lb[i]; }
            __syncthreads();
            const int set = wv & 1;                // two wavefronts do the same
#pragma unroll
            for (int i = 0; i < R; ++i) la[i] = part[0][set][i][lane];
            for (int p = 1; p < WS; ++p)
#pragma unroll
                for (int i = 0; i < R; ++i) insert(la, part[p][set][i][lane]);
            auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(la[R - 1]), __float_as_uint(la[R - 1]), false, false);
            const float t = fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
            const int tok = tok0 + set * 32 + n;
            if (wv < 2 && half == 0 && tok < a.T) a.tau0[(size_t)head * a.T + tok] = t > -INFINITY ? t : -INFINITY;
            __syncthreads();
        } else {
            auto ra = __builtin_amdgcn_permlane32_swap(__float_as_uint(la[R - 1]), __float_as_uint(la[R - 1]), false, false);
            auto rb = __builtin_amdgcn_permlane32_swap(__float_as_uint(lb[R - 1]), __float_as_uint(lb[R - 1]), false, false);
            const float ta = fminf(__uint_as_float(ra[0]), __uint_as_float(ra[1]));
            const float tb = fminf(__uint_as_float(rb[0]), __uint_as_float(rb[1]));
            const float t = half ? tb : ta;
            if (tok0 + lane < a.T) a.tau0[(size_t)head * a.T + tok0 + lane] = t > -INFINITY ? t : -INFINITY;
        }
    }
}

// The call's minima become the bounds that are carried on.
__global__ void enc_carry_kernel(ScanArgs a) {
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= a.n_heads) return;
    const float extra = a.n_fail[h] > 0 ? kRedoMargin : 0.f;
    const float r = a.hint_out[2 * h] == 0xFFFFFFFFu ? -INFINITY : value_of(a.hint_out[2 * h]);
    const float m = a.hint_out[2 * h + 1] == 0xFFFFFFFFu ? -INFINITY : value_of(a.hint_out[2 * h + 1]);
    const float s_tau = a.hint_sum[3 * h], s_x = a.hint_sum[3 * h + 1], s_n = a.hint_sum[3 * h + 2];
    const float waste_r = r > -INFINITY ? s_tau - r * s_x : INFINITY;
    const float waste_m = m > -INFINITY ? s_tau - m * s_n : INFINITY;
    const bool use_r = waste_r <= waste_m;
    a.hint_next[2 * h] = use_r ? s3_carried(r, extra) : -INFINITY;
    a.hint_next[2 * h + 1] = use_r ? -INFINITY : s3_carried(m, extra);
}

// How a call is laid out.
struct Plan {
    int tiles_per_head, n_tiles, parts, per, cap, sample, units;
    size_t fail, hout, hsum, few, tau0, norm, count, list, total;
};
constexpr int kMaxParts = 16;
constexpr int kFewTiles = 128;          // so many tiles or fewer are split: 256 tiles in two ranges each waited longer for their join (k 128: 916 / 617 us)
// One lane's half of a sample of an eighth holds mu = k / 16 of the k best; mu + 3 sqrt(mu) + 1 is at most 7.3, 11 and 17.5.
int sample_rank(int k) { return k <= 32 ? 8 : (k <= 64 ? 12 : 18); }

// For calls that s3_encode_scan_pays takes: 8192 features, 256 stages, and more.
Plan plan(int n_heads, int T, int n_feat, int k) {
    Plan p;
    const int nst = n_feat / kFT;
    p.tiles_per_head = (T + kTokWG - 1) / kTokWG;
    p.n_tiles = n_heads * p.tiles_per_head;
    int parts = p.n_tiles <= kFewTiles ? kSlots / p.n_tiles : 1;
    parts = parts > kMaxParts ? kMaxParts : parts;
    p.per = ((nst + parts - 1) / parts + 1) & ~1;
    p.parts = (nst + p.per - 1) / p.per;
    p.cap = cap_of(k);
    p.units = p.parts > 1 ? p.n_tiles * p.parts : (p.n_tiles < kSlots ? p.n_tiles : kSlots);
    p.sample = nst / 8;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += s3_align(bytes); return at; };
    p.fail = take((size_t)n_heads * 4);
    p.hout = take((size_t)n_heads * 8);
    p.hsum = take((size_t)n_heads * 12);
    p.few = take(p.parts > 1 ? (size_t)kFewTiles * 4 : 0);
    p.tau0 = take((size_t)n_heads * T * 4);
    p.norm = take(p.parts > 1 ? (size_t)n_heads * T * 4 : 0);
    p.count = take((size_t)p.units * kWaves * kLanes * 4);
    p.list = take((size_t)p.units * kWaves * kLanes * p.cap * sizeof(uint2));
    p.total = o;
    return p;
}

template <int G, int LR>
int launch_scan(const ScanArgs& a, const Plan& p, hipStream_t st) {
    auto scan = enc_scan_kernel<G, false>;
    auto redo = enc_scan_kernel<G, true>;
    static S3LdsOnce once[2];
    if (int rc = s3_allow_lds(once[0], (const void*)scan, kLds)) return rc;
    hipLaunchKernelGGL(scan, dim3((unsigned)p.units), dim3(kThreads), kLds, st, a);
    if (p.parts > 1) {
        if (int rc = s3_allow_lds(once[1], (const void*)redo, kLds)) return rc;
        if (a.hint) hipLaunchKernelGGL((enc_join_kernel<LR, 16>), dim3((unsigned)p.n_tiles * (kTokWG / 16)), dim3(64 * 16), 0, st, a);
        else hipLaunchKernelGGL((enc_join_kernel<LR, 4>), dim3((unsigned)p.n_tiles * (kTokWG / 4)), dim3(64 * 4), 0, st, a);
        hipLaunchKernelGGL(redo, dim3((unsigned)p.n_tiles), dim3(kThreads), kLds, st, a);
    }
    return S3_OK;
}
template <int R>
void launch_start(const ScanArgs& a, hipStream_t st) {
    const long long groups = (long long)a.n_heads * ((a.T + kTokWave - 1) / kTokWave);
    // Up to 640 groups of 64 tokens both take as long; beyond, the stages of 256 tokens are better shared (first chunk of a stream, 16384
    // features, WS kWaves / 1: 40 heads x 2048, k 64, 867 / 823 us; 64, k 64, 1144 / 1050; 32, k 128, 1232 / 1196), below, a chip is not full.
    if (groups <= 512) hipLaunchKernelGGL((enc_start_kernel<R, kWaves>), dim3((unsigned)groups), dim3(kThreads), 0, st, a);
    else hipLaunchKernelGGL((enc_start_kernel<R, 1>), dim3((unsigned)(a.n_tiles < 4096 ? a.n_tiles : 4096)), dim3(kThreads), 0, st, a);
}

}  // namespace

// Whether a call is better off here than in the fast or the tiled kernel (us, those / this one, 16384 features unless stated).
//   - Up to 64 tiles the fast kernel leaves most of the chip idle (streamed, 8 heads x 512 tokens, k 32: 318 / 81, of 300 tokens
//     and k 128: 383 / 109; plain, one head x 4096 tokens, k 32 / 128: 128 / 91, 216 / 122).  Tiles that are mostly empty
//     waste this kernel's 256 tokens: 256 heads x 64 tokens, streamed: 266 / 361.
//   - k <= 32 from 65 to 256 tiles: less than two workgroups per compute unit, or a join of many tokens (16 heads x 2048: 334 /
//     380); beyond, 48 x 2048: 653 / 527, 256 x 2048: 2756 / 2365.
//   - Skewed features (Zipf) bring a token more candidates in narrow dictionaries: 128 x 2048, k 32: of 8192 features 1009 /
//     1167 (evenly used ones 64 x 2048, k 16: 810 / 666), of 16384 1525 / 1526, of 32768, 64 x 2048, 1322 / 1483 (first chunks 1992 / 1411,
//     even ones 1342 / 1090); k 64: of 8192 941 / 1028, of 32768 3491 / 2674; k 128: of 16384 2936 / 1929, of 8192 (even) 288 / 227.
//   - First chunks pay for the sample: k 32, 256 x 2048 3330 / 3468, later ones 2793 / 2381; x 1025 (a fifth tile with one token) 1842 /
//     2077 and 1638 / 1453.
//   - Plain calls have no carried thresholds and pay for the sample: k 32, 64 x 256: 449 / 168, 128 x 512: 496 / 560, 256 x 512:
//     942 / 914.
bool s3_encode_scan_pays(int n_heads, int T, int n_feat, int k, bool streamed) {
    const long long tiles = (long long)n_heads * ((T + kTokWG - 1) / kTokWG);
    if (n_feat < 8192 || T < kTokWG) return false;
    if (!streamed && (long long)n_heads * T < 4096) return false;
    if (tiles <= kFewTiles / 2) return true;
    if (k > 32) return n_feat >= (k <= 64 ? 12288 : 8192);
    return n_feat >= 16384 && (streamed ? tiles > kSlots / 2 : tiles <= kFewTiles || tiles >= kSlots);
}

size_t s3_encode_scan_workspace(int n_heads, int T, int n_feat, int k) { return T < 1 ? 0 : plan(n_heads, T, n_feat, k).total; }

// The most that a call of this many tokens or fewer takes, whatever n_feat and k are.
size_t s3_encode_scan_workspace_max(int n_heads, int T) {
    if (T < kTokWG) return 0;                          // s3_encode_scan_pays refuses them
    const long long tiles = (long long)n_heads * ((T + kTokWG - 1) / kTokWG);
    const long long split = tiles > kFewTiles ? kSlots : (tiles * kMaxParts < kSlots ? tiles * kMaxParts : kSlots), whole = tiles < kSlots ? tiles : kSlots;
    const long long units = split > whole ? split : whole;
    const size_t tokens = (size_t)n_heads * T, norms = tokens < (size_t)kFewTiles * kTokWG ? tokens : (size_t)kFewTiles * kTokWG;
    return s3_align((size_t)n_heads * 4) + s3_align((size_t)n_heads * 8) + s3_align((size_t)n_heads * 12) + s3_align(kFewTiles * 4) + s3_align(tokens * 4) +
           s3_align(norms * 4) + s3_align((size_t)units * kWaves * kLanes * 4) + s3_align((size_t)units * kWaves * kLanes * cap_of(S3_MAX_K) * sizeof(uint2));
}

int s3_encode_scan(const EncParams& e, float* hint, void* ws, hipStream_t st) {
    const Plan p = plan(e.n_heads, e.T, e.n_feat, e.k);
    char* base = (char*)ws;
    ScanArgs a;
    a.x = e.x; a.w = e.w; a.b = e.b; a.ids = e.ids; a.vals = e.vals;
    a.T = e.T; a.n_feat = e.n_feat; a.k = e.k; a.n_heads = e.n_heads;
    a.tiles_per_head = p.tiles_per_head; a.n_tiles = p.n_tiles;
    a.parts = p.parts; a.per = p.per; a.cap = p.cap; a.sample = p.sample;
    a.vec = e.k % 4 == 0 && (((uintptr_t)e.ids | (uintptr_t)e.vals) & 15) == 0;
    a.list = (uint2*)(base + p.list);
    a.count = (int*)(base + p.count);
    a.norm = hint && p.parts > 1 ? (float*)(base + p.norm) : nullptr;
    a.tau0 = (float*)(base + p.tau0);
    a.hint = hint; a.hint_next = hint;
    a.hint_out = (unsigned*)(base + p.hout);
    a.hint_sum = (float*)(base + p.hsum);
    a.n_fail = (int*)(base + p.fail);
    a.few = (int*)(base + p.few);
    switch (sample_rank(e.k)) {
        case 8: launch_start<8>(a, st); break;
        case 12: launch_start<12>(a, st); break;
        default: launch_start<18>(a, st);
    }
    int rc = e.k <= 32 ? launch_scan<1, 2>(a, p, st) : (e.k <= 64 ? launch_scan<2, 2>(a, p, st) : launch_scan<4, 4>(a, p, st));
    if (rc) return rc;
    if (hint) hipLaunchKernelGGL(enc_carry_kernel, dim3((unsigned)((e.n_heads + 255) / 256)), dim3(256), 0, st, a);
    S3_HIP(hipGetLastError());
    return S3_OK;
}
