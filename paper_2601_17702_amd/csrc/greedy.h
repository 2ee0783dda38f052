// Greedy choice of the best positions, each of which removes what lies within `reach` of it: the search behind the Top-B spans
// and the density peaks.  One workgroup; the rounds depend on each other, so what bounds it is the latency of a round.
//
// Positions are looked at in blocks of 64.  A choice touches at most c = (2 reach - 1) / 64 + 2 blocks (one if reach is 0), so when
// `want` positions are chosen, each lies in one of the c (want - 1) + 1 blocks with the best maxima: among so many at least one is
// untouched by the choices before, and what is chosen is no worse than its maximum (of equal maxima the first).  Only these blocks are brought into LDS (as
// "slots", in ascending order; fill()), and a round touches nothing else.  rounds() takes all choices that do not depend on each
// other at once; walk() takes one a round, for choices that remove few positions.
//
// Kernel times: 16 spans of 64 in 32768 positions 30.0 -> 8 us (one choice a round, the blocks at both ends read from memory:
// 1.6 us a round), 40 peaks of 32768 positions 44.6 -> 15 (the same with the curve in LDS and the maxima of all blocks in groups:
// 1.1 us a round).  Of the 15: maxima and threshold 3, values of the slots 2, rounds 4.5, order of the choices 2, spans 2.5.
#pragma once
#include "s3_common.h"

namespace s3greedy {

constexpr int kThreads = 1024, kWaves = kThreads / 64;
constexpr int kListMax = 1024;                        // choices of rounds()
constexpr int kNone = -0x7FFFFFFF - 1;                // the place of a slot that holds nothing

// The most choices there can be.
inline int64_t choices(int64_t n, int64_t reach, int64_t want) { return want < (n - 1) / (reach + 1) + 1 ? want : (n - 1) / (reach + 1) + 1; }
// Blocks that the choices before the last may touch, and one more.
inline int64_t slots_needed(int64_t n, int64_t reach, int64_t want) {
    const int64_t blocks = (n + 63) / 64, touched = reach > 0 ? (2 * reach - 1) / 64 + 2 : 1;
    return want - 1 >= blocks || touched >= blocks || touched * (want - 1) + 1 >= blocks ? blocks : touched * (want - 1) + 1;
}

__device__ __forceinline__ unsigned top_word(unsigned v) { return v; }
__device__ __forceinline__ unsigned top_word(unsigned long long v) { return (unsigned)(v >> 32); }
__device__ __forceinline__ unsigned of_lane(unsigned v, int src) { return (unsigned)__builtin_amdgcn_readlane((int)v, src); }
__device__ __forceinline__ unsigned long long of_lane(unsigned long long v, int src) {
    return ((unsigned long long)of_lane((unsigned)(v >> 32), src) << 32) | of_lane((unsigned)v, src);
}
// m: the lanes whose upper word is the largest, `top`.  Leaves those whose whole value is.
__device__ __forceinline__ void settle(unsigned, unsigned, unsigned long long&) {}
__device__ __forceinline__ void settle(unsigned long long v, unsigned top, unsigned long long& m) {
    if ((m & (m - 1)) == 0) return;
    const unsigned low = s3_wave_max_u32((unsigned)(v >> 32) == top ? (unsigned)v : 0u);
    m = __ballot((unsigned)(v >> 32) == top && (unsigned)v == low);
}

// LDS of a search with `cap` slots: values (64 a slot and 16 bytes more, so that lanes that read a row each meet different
// banks), then the slots' best values and their places.
template <class Key>
constexpr int kRow = 64 + 16 / (int)sizeof(Key);
template <class Key>
constexpr int lds_bytes(int cap) { return cap * ((kRow<Key> + 1) * (int)sizeof(Key) + 4); }
constexpr int kLdsMost = 160 << 10;
constexpr int lds_static(int slots) { return 512 + 16 * slots; }      // the kernels' own variables, rounded up; in rounds four words a slot at most

template <class Key>
struct Slots {
    Key* val;
    Key* key;
    int* at;
    int cap;
};
template <class Key>
__device__ __forceinline__ Slots<Key> slots_of(void* lds, int cap) {
    Slots<Key> s;
    s.val = (Key*)lds;
    s.key = s.val + (size_t)cap * kRow<Key>;
    s.at = (int*)(s.key + cap);
    s.cap = cap;
    return s;
}

// Sum over the workgroup of a value that is the same in a wavefront's lanes, in every thread; `before`: of the wavefronts
// before this one.  The two buffers take turns, so that a sum needs one barrier.
struct Sums {
    int (*buf)[kWaves];
    int turn;
};
__device__ __forceinline__ int block_sum(Sums& s, int v, int& before) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int* const b = s.buf[s.turn];
    s.turn ^= 1;
    if (lane == 0) b[wave] = v;
    __syncthreads();
    const int x = s3_row_incl_scan(b[lane & (kWaves - 1)]);
    before = wave ? __builtin_amdgcn_readlane(x, wave - 1) : 0;
    return __builtin_amdgcn_readlane(x, kWaves - 1);
}
template <class Key, int P>
__device__ __forceinline__ int block_count(Sums& s, const Key (&key)[P], Key at_least) {
    int c = 0, before;
#pragma unroll
    for (int q = 0; q < P; ++q) c += (int)__popcll(__ballot(key[q] >= at_least));
    return block_sum(s, c, before);
}

// Where to count next between lo (clo keys at or above it) and hi (chi): by interpolation on the logarithm of the counts where
// `interp` says so, else half way.
template <class Key>
__device__ __forceinline__ Key between(Key lo, Key hi, int clo, int chi, float want, bool interp) {
    if (interp) {
        const float llo = __log2f((float)clo), lhi = __log2f((float)max(chi, 1));
        const float t = fminf(fmaxf((llo - want) * __builtin_amdgcn_rcpf(llo - lhi), 0.03125f), 0.96875f);
        const Key mid = lo + of_lane((Key)((float)(hi - lo) * t), 0);
        if (mid > lo && mid < hi) return mid;
    }
    return lo + (hi - lo) / 2;
}
// Raises lo as long as more than `most` keys reach it and `need` still do.  count(t): keys at or above t; snap(lo, hi): moves both
// to the smallest and behind the largest key in [lo, hi).  Interpolates as long as that halves what is left; keys that are
// equal would take it one step per bit, so every fourth step snaps.
template <class Key, class Count, class Snap>
__device__ __forceinline__ void raise(Key& lo, Key hi, int& clo, int need, int most, Count count, Snap snap) {
    const float want = __log2f(0.5f * (float)(need + most));
    bool interp = true;
    int chi = 0;
    for (int step = 1; clo > most && hi - lo > 1; ++step) {
        if ((step & 3) == 0) {
            snap(lo, hi);
            if (hi - lo <= 1) break;
        }
        const Key was = hi - lo, mid = between(lo, hi, clo, chi, want, interp);
        const int c = count(mid);
        if (c >= need) { lo = mid; clo = c; } else { hi = mid; chi = c; }
        interp = hi - lo <= was / 2;
    }
}
__device__ __forceinline__ int shift_of(unsigned v) { return 0; }
__device__ __forceinline__ int shift_of(unsigned long long v) { return max(0, 32 - (int)__builtin_clzll(v | 1)); }

// A threshold that `need` to `most` of the workgroup's kThreads keys reach, as far as ties in 32 bits allow (never less
// than `need`; 1 if no more than `most` are live), by one wavefront, which has them all in its registers: a count is a compare
// and a bit count per register.  best: the largest key.
template <class Key>
__device__ __forceinline__ Key threshold(const Key* keys, int need, int most, Key& best) {
    constexpr int N = kThreads / 64;
    const int lane = threadIdx.x & 63;
    Key full[N], mx = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) { full[i] = keys[i * 64 + lane]; mx = full[i] > mx ? full[i] : mx; }
    const unsigned top = s3_wave_max_u32(top_word(mx));
    unsigned long long m = __ballot(top_word(mx) == top);
    settle(mx, top, m);
    best = of_lane(mx, (int)__builtin_ctzll(m));
    const int sh = shift_of(best);
    unsigned k[N], least = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < N; ++i) { k[i] = (unsigned)(full[i] >> sh); least = min(least, k[i] - 1); }      // not live: largest of all
    const auto count = [&](unsigned t) {
        int c = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) c += (int)__popcll(__ballot(k[i] >= t));
        return c;
    };
    unsigned lo = 0xFFFFFFFFu - s3_wave_max_u32(0xFFFFFFFFu - least) + 1;
    int clo = count(max(lo, 1u));
    if (clo <= most) return Key(1);
    raise(lo, (unsigned)(best >> sh) + 1, clo, need, most, count, [&](unsigned& l, unsigned& h) {
        unsigned above = 0, under = 0;                // the larger, the nearer to the end in question
#pragma unroll
        for (int i = 0; i < N; ++i) {
            above = max(above, k[i] >= l ? 0xFFFFFFFFu - k[i] : 0u);
            under = max(under, k[i] < h ? k[i] : 0u);
        }
        l = 0xFFFFFFFFu - s3_wave_max_u32(above);
        h = s3_wave_max_u32(under) + 1;
    });
    return (Key)lo << sh;
}

// Blocks whose maxima a thread has.  No more than it takes: all wavefronts share them, since the threshold is first looked for among
// the threads' largest.  (A fixed sixteen left 1094 blocks to two wavefronts: peaks of radius 500 in 70000 positions 19 -> 30 us.)
__device__ __forceinline__ int per_thread(int blocks) { return (blocks + kThreads - 1) / kThreads; }

// Fills the slots with the blocks that have the best maxima: at least `need` of them (fewer if fewer have a live position), at
// most s.cap, in ascending order.  Thread t has the maxima of blocks (wavefront per_thread() + q) 64 + lane, q < per_thread() <= P (0:
// nothing live, and for every other q), and their places.  read(i): what position i < n holds; key_of() of it: its value.
template <class Key, int P, class Read, class KeyOf>
__device__ __forceinline__ void fill(const Slots<Key>& s, const Key (&key)[P], const int (&at)[P], int need, int64_t n, Read read, KeyOf key_of) {
    __shared__ int buf[2][kWaves];
    __shared__ Key first[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Sums sums{buf, 0};
    Key* const most = s.val;                          // the slots' values come later
    for (int i = tid; i < s.cap; i += kThreads) { s.key[i] = 0; s.at[i] = kNone; }
    Key mx = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) mx = key[q] > mx ? key[q] : mx;
    most[tid] = mx;
    __syncthreads();
    // The threads' largest first (the blocks' own where a thread has one): no fewer blocks than threads reach what those reach.
    if (wave == 0) {
        Key best;
        const Key t = threshold(most, min(need, kThreads), s.cap, best);
        if (lane == 0) { first[0] = t; first[1] = best; }
    }
    __syncthreads();
    Key lo = first[0];                                // admitted: at or above lo
    const Key best = first[1];
    int quota = 0x7FFFFFFF;                           // of those that equal lo, so many
    int clo = block_count(sums, key, lo);
    if (clo < need) {                                 // P > 1: more blocks are asked for than there are threads
        lo = 1;
        clo = block_count(sums, key, lo);
    }
    if (clo > s.cap) {                                // P > 1, or ties
        if (lo != best && best - lo < Key(1) << shift_of(best)) {      // the best to 32 bits, perhaps all of them
            const int c = block_count(sums, key, best);
            if (c >= need) { lo = best; clo = c; }
        }
        if (lo != best) raise(lo, (Key)(best + 1), clo, need, s.cap, [&](Key t) { return block_count(sums, key, t); }, [&](Key& l, Key& h) {
            Key least = ~Key(0), largest = 0;
#pragma unroll
            for (int q = 0; q < P; ++q) {
                if (key[q] >= l && key[q] < least) least = key[q];
                if (key[q] < h && key[q] > largest) largest = key[q];
            }
            __syncthreads();
            if (tid == 0) { first[0] = ~Key(0); first[1] = 0; }
            __syncthreads();
            if (least != ~Key(0)) atomicMin(&first[0], least);
            atomicMax(&first[1], largest);
            __syncthreads();
            l = first[0];
            h = first[1] + 1;
        });
        if (clo > s.cap) quota = s.cap - block_count(sums, key, (Key)(lo + 1));      // more equal maxima than slots: the first ones
    }
    int ties = 0, before;
    if (quota != 0x7FFFFFFF) {
        int c = 0;
#pragma unroll
        for (int q = 0; q < P; ++q) c += (int)__popcll(__ballot(key[q] == lo));
        block_sum(sums, c, ties);
    }
    unsigned long long in[P];
    int mine = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const unsigned long long eq = __ballot(key[q] == lo);
        const int rank = ties + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(eq >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)eq, 0u));
        in[q] = __ballot(key[q] > lo || (key[q] == lo && rank < quota));
        ties += (int)__popcll(eq);
        mine += (int)__popcll(in[q]);
    }
    block_sum(sums, mine, before);
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const int o = before + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(in[q] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in[q], 0u));
        if (in[q] >> lane & 1) { s.key[o] = key[q]; s.at[o] = at[q]; }
        before += (int)__popcll(in[q]);
    }
    __syncthreads();
    constexpr int U = 8;                              // loads in flight per lane
    for (int i0 = wave; i0 < s.cap; i0 += U * kWaves) {
        int p[U];
        decltype(read(0)) v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) p[u] = i0 + u * kWaves < s.cap ? s.at[i0 + u * kWaves] : kNone;
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = read(p[u] != kNone ? min((int64_t)(p[u] >> 6) * 64 + lane, n - 1) : 0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kWaves < s.cap)
                s.val[(i0 + u * kWaves) * kRow<Key> + lane] = p[u] != kNone && (int64_t)(p[u] >> 6) * 64 + lane < n ? key_of(v[u]) : Key(0);
    }
    __syncthreads();
}

template <int R, class Key, class Put, class Enough>   // below
__device__ int walk(const Slots<Key>& s, unsigned n, unsigned reach, int want, Key& next, int& next_at, Put put, Enough enough);

template <int X>
__device__ __forceinline__ unsigned quad_xor(unsigned v) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, X == 1 ? 0xB1 : (X == 2 ? 0x4E : 0x141), 0xf, 0xf, true);      // 4: the other four, mirrored
}
template <int X>
__device__ __forceinline__ unsigned long long quad_xor(unsigned long long v) {
    return ((unsigned long long)quad_xor<X>((unsigned)(v >> 32)) << 32) | quad_xor<X>((unsigned)v);
}
// The choices in few rounds, by the whole workgroup, over C slots.  A position that is the best within its reach is chosen
// whatever happens elsewhere, so a round takes all slots' best positions that beat everything in the blocks they may reach into
// (the best of all always does), removes what they reach and searches the blocks concerned again.  That goes on until `want`
// choices come before everything left (larger value first, ties -> smaller position); one to four rounds are usual.
// Among equal values a position beats the ones behind it only, and a round may take as little as one choice, no faster than walk()
// takes two to four.  So where a round takes fewer than `few`, or two in a row settle fewer each, walk() goes on, until it and the
// rounds have `want` together.  us for a look-up, in rounds until every slot was used up / now: 64 windows of 16 among equal ones
// 890 / 54; 40 peaks of radius 8 on a level curve 1310 / 49.
// T threads have a slot, so that 512 threads do all this, two wavefronts a SIMD (a round takes 1.5 to 2 us; with all sixteen 2.8,
// with four 2.1).
// list_key, list_at (LDS): the choices; a slot has at most 64 / (reach + 1) of them, rounded up, kListMax all together.
// Then put(r, key, at) for the r-th best one, r < want, by some thread each.  Returns how many there are, in every thread.
template <int C, class Key, class Put>
__device__ __forceinline__ int rounds(const Slots<Key>& s, Key* list_key, int* list_at, unsigned n, unsigned reach, int want, Put put) {
    constexpr int T = 512 / C, few = 4;
    constexpr int V = 16 / (int)sizeof(Key), U = 64 / V / T;          // values a read, reads a thread
    static_assert(T == 1 || T == 2 || T == 4 || T == 8);
    __shared__ int buf[2][kWaves], blk[C], won[C], n_list, left_at[3];
    __shared__ Key shown[C], left[3];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool active = wave < C * T / 64;
    const int j = tid % T, me = active ? tid / T : 0;
    Sums sums{buf, 0};
    Key k = active ? s.key[me] : Key(0);
    int p = k ? s.at[me] : kNone;
    const int b = k ? p >> 6 : 0xFFFFFF;              // beyond every block
    const int first = b * 64;
    unsigned long long live = ~0ull;
    if (active && j == 0) { blk[me] = b; shown[me] = k; }
    if (tid == 0) n_list = 0;
    if (tid < 3) { left[tid] = 0; left_at[tid] = 0x7FFFFFFF; }
    __syncthreads();
    Key rest = 0;                                     // the best of what is left
    int rest_at = 0;
    const auto before_rest = [&](int i) { return list_key[i] > rest || (list_key[i] == rest && list_at[i] < rest_at); };
    int was = 0, was_done = 0, slow = 0;              // slow: rounds one after the other that brought few choices
    reach = min(reach, n);
    int t0 = me, t1 = me;                             // the slots that a choice in this one may reach into, and the other way round
    if (k) {
        const int far = (int)((reach + 63) >> 6);
        while (t0 > 0 && blk[t0 - 1] >= b - far) --t0;
        while (t1 < C - 1 && blk[t1 + 1] - b <= far) ++t1;
    }
    for (int turn = 0;; turn = turn == 2 ? 0 : turn + 1) {
        if (active) {
            bool wins = k != 0;
            if (k) {
                for (int t = t0; t <= t1; t += 4) {
                    Key o[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[i] = shown[min(t + i, t1)];
#pragma unroll
                    for (int i = 0; i < 4; ++i) wins = wins & ((o[i] < k) | ((o[i] == k) & (min(t + i, t1) >= me)));
                }
            }
            if (j == 0) {
                won[me] = wins ? p : kNone;
                if (wins) {
                    const int at = atomicAdd(&n_list, 1);
                    list_key[at] = k;
                    list_at[at] = p;
                }
            }
        }
        __syncthreads();                              // the choices
        const int chosen = n_list;
        if (active) {
            bool again = false;
            if (k) {
                for (int t = t0; t <= t1; t += 4) {   // what they remove from this slot's block
                    int w[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[i] = won[min(t + i, t1)];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int from = max(w[i] - (int)reach - first, 0), upto = min(w[i] + (int)reach - first, 63);
                        if (w[i] != kNone && from <= upto) live &= ~(~0ull << from & ~0ull >> (63 - upto));
                    }
                }
                again = !(live >> (p & 63) & 1);
            }
            if (__any(again)) {
                Key x[U * V], best = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    typedef __attribute__((ext_vector_type(V))) Key Vec;
                    const Vec v = *(const Vec*)(s.val + me * kRow<Key> + (u * T + j) * V);
                    const unsigned bits = (unsigned)(live >> ((u * T + j) * V));
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        x[u * V + i] = bits >> i & 1 ? v[i] : Key(0);
                        best = x[u * V + i] > best ? x[u * V + i] : best;
                    }
                }
                if constexpr (T >= 2) { const Key o = quad_xor<1>(best); best = o > best ? o : best; }
                if constexpr (T >= 4) { const Key o = quad_xor<2>(best); best = o > best ? o : best; }
                if constexpr (T >= 8) { const Key o = quad_xor<4>(best); best = o > best ? o : best; }
                unsigned at = 64;
#pragma unroll
                for (int u = U - 1; u >= 0; --u)
#pragma unroll
                    for (int i = V - 1; i >= 0; --i)
                        if (x[u * V + i] == best) at = (unsigned)((u * T + j) * V + i);      // the first one
                if constexpr (T >= 2) at = min(at, quad_xor<1>(at));
                if constexpr (T >= 4) at = min(at, quad_xor<2>(at));
                if constexpr (T >= 8) at = min(at, quad_xor<4>(at));
                if (again) { k = best; p = first + (int)at; }
            }
            if (j == 0) shown[me] = k;
            const unsigned top = s3_wave_max_u32(top_word(k));
            unsigned long long m = __ballot(top_word(k) == top);
            settle(k, top, m);
            const Key most = of_lane(k, (int)__builtin_ctzll(m));
            if (lane == 0) atomicMax(&left[turn], most);
            if (tid == 0) { left[turn == 2 ? 0 : turn + 1] = 0; left_at[turn == 2 ? 0 : turn + 1] = 0x7FFFFFFF; }
        }
        __syncthreads();                              // what is left
        rest = left[turn];
        if (rest == 0) break;
        if (chosen >= want || chosen - was < few) {
            const auto count = [&]() {
                int c = 0, before;
                for (int i = tid; i < chosen; i += kThreads) c += (int)__popcll(__ballot(before_rest(i)));
                return block_sum(sums, __builtin_amdgcn_readlane(c, 0), before);
            };
            rest_at = 0;                              // the larger ones alone
            int done = count();
            if (done >= want) break;
            slow = done - was_done < few ? slow + 1 : 0;
            if (slow) {
                if (active && j == 0 && k == rest) atomicMin(&left_at[turn], p);
                __syncthreads();
                rest_at = left_at[turn];
                done = count();
                if (done >= want) break;
            }
            if (slow == 2 || (slow && chosen - was < few)) {
                if (active) {                         // walk() goes on from the values and the slots' best ones in LDS
                    for (int i = j; ~live && i < 64; i += T)
                        if (!(live >> i & 1)) s.val[me * kRow<Key> + i] = 0;
                    if (j == 0) { s.key[me] = k; s.at[me] = p; }
                }
                __syncthreads();
                if (wave == 0) {
                    const int more = walk<C / 64, Key>(s, n, reach, want - done, rest, rest_at, [&](int r, Key x, int at) {
                        if (lane == 0) { list_key[chosen + r] = x; list_at[chosen + r] = at; }
                    }, [&](int found, Key x, int at) {    // those of the rounds that its choices have caught up with
                        if (chosen == done) return false;
                        int c = found;
                        for (int i0 = 0; i0 < chosen; i0 += 64) {
                            const int i = min(i0 + lane, chosen - 1);
                            c += (int)__popcll(__ballot(i0 + lane < chosen && (list_key[i] > x || (list_key[i] == x && list_at[i] < at))));
                        }
                        return c >= want;
                    });
                    if (lane == 0) { n_list = chosen + more; left[0] = rest; left_at[0] = rest_at; }
                }
                __syncthreads();
                rest = left[0];
                rest_at = left_at[0];
                break;
            }
            was_done = done;
        }
        was = chosen;
    }
    // Those that come before what is left, in their order: 64 of them a wavefront, against a part of all.
    Key* const key = s.val;
    int* const at = (int*)(key + kListMax);
    int* const rank = at + kListMax;
    const int total = n_list;
    if (tid == 0) won[0] = 0;
    __syncthreads();
    for (int i = tid; i < total; i += kThreads)
        if (before_rest(i)) {
            const int o = atomicAdd(&won[0], 1);
            key[o] = list_key[i];
            at[o] = list_at[i];
            rank[o] = 0;
        }
    __syncthreads();
    const int valid = won[0], groups = (valid + 63) >> 6, parts = max(1, kWaves / max(groups, 1));
    for (int g = wave / parts; g < groups; g += kWaves / parts) {
        const int i = min(g * 64 + lane, valid - 1), o0 = valid * (wave % parts) / parts, o1 = valid * (wave % parts + 1) / parts;
        const Key x = key[i];
        const int xa = at[i];
        int r = 0;
        for (int o = o0; o < o1; o += 64) {
            const Key y = key[min(o + lane, valid - 1)];
            const int ya = at[min(o + lane, valid - 1)];
            for (int q = 0; q < min(64, o1 - o); ++q) {
                const Key yq = of_lane(y, q);
                r += yq > x || (yq == x && __builtin_amdgcn_readlane(ya, q) < xa) ? 1 : 0;
            }
        }
        if (g * 64 + lane < valid) atomicAdd(&rank[i], r);
    }
    __syncthreads();
    for (int i = tid; i < valid; i += kThreads)
        if (rank[i] < want) put(rank[i], key[i], at[i]);
    return min(valid, want);
}

// How a search with at least `need` slots runs: in rounds, with 64, 128, 256 or 512 slots (up = 0 .. 3), where the list of choices
// has at most kListMax entries; else one choice after the other, with 64, 128, 256 or 576 slots.
struct Way {
    bool rounds;
    int up, cap, room;                                // room: entries of the list
};
inline Way way_of(int64_t need, int64_t reach) {
    Way w;
    w.up = need <= 64 ? 0 : (need <= 128 ? 1 : (need <= 256 ? 2 : 3));
    w.cap = 64 << w.up;
    w.room = w.cap * (int)(63 / (reach + 1) + 1);
    w.rounds = need <= w.cap && w.room <= kListMax;
    if (!w.rounds && w.up == 3) w.cap = 576;
    return w;
}

// The choices one after the other, by one wavefront, over 64 R slots and n positions: the slots' maxima are in its registers, a
// round wipes what it removes in the blocks at both ends and searches those again, beside the reduction over the other slots and
// not behind it (0.5 to 0.55 us a round).  No lane reads an LDS value of another one: value i of a slot is lane i's.  Then put(r, key, at)
// for the r-th choice.  Returns how many there were (fewer than `want` if nothing live was left); next, next_at: what would come
// then (next 0: nothing).  enough(found, next, next_at), asked after every fourth choice: whether to stop.  Larger value first, ties -> smaller position.
template <int R, class Key, class Put, class Enough>
__device__ __forceinline__ int walk(const Slots<Key>& s, unsigned n, unsigned reach, int want, Key& next, int& next_at, Put put, Enough enough) {
    const int lane = threadIdx.x & 63;
    Key k[R], lk = 0;
    int p[R], lp = 0;                                 // slot lane R + q
#pragma unroll
    for (int q = 0; q < R; ++q) {
        k[q] = s.key[lane * R + q];
        p[q] = k[q] ? s.at[lane * R + q] : kNone;
        if (k[q] > lk) { lk = k[q]; lp = p[q]; }
    }
    unsigned top = s3_wave_max_u32(top_word(lk));
    unsigned long long m = __ballot(top_word(lk) == top);
    settle(lk, top, m);
    Key best = of_lane(lk, (int)__builtin_ctzll(m));
    int at = (int)of_lane((unsigned)lp, (int)__builtin_ctzll(m));
    int found = 0;
    while (found < want && best && !(found > 0 && (found & 3) == 0 && enough(found, best, at))) {
        put(found++, best, at);
        const unsigned lo = (unsigned)at > reach ? (unsigned)at - reach : 0u, hi = min((unsigned)at + reach, n - 1);
        const int tl = (int)(lo >> 6), span = (int)(hi >> 6) - tl;
        int fl = -1, fh = -1;                         // the lane's slot of the block at either end
        lk = 0;
        lp = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int t = (p[q] >> 6) - tl;
            if (t == 0) fl = q;
            if (t == span) fh = q;
            const bool gone = (unsigned)t <= (unsigned)span;          // the ends come back below
            k[q] = gone ? Key(0) : k[q];
            p[q] = gone ? kNone : p[q];
            if (k[q] > lk) { lk = k[q]; lp = p[q]; }
        }
        const unsigned long long ml = __ballot(fl >= 0), mh = span ? __ballot(fh >= 0) : 0ull;
        Key vl = 0, vh = 0;
        s3_wave_fence();                              // what is wiped below is read, and what was wiped stays so
        if (ml) {
            const int src = (int)__builtin_ctzll(ml);
            Key* const v = s.val + (src * R + __builtin_amdgcn_readlane(fl, src)) * kRow<Key> + lane;
            const unsigned i = (unsigned)tl * 64 + lane;
            vl = *v;
            if (i >= lo && i <= hi) { vl = 0; *v = 0; }
        }
        s3_wave_fence();
        if (mh) {
            const int src = (int)__builtin_ctzll(mh);
            Key* const v = s.val + (src * R + __builtin_amdgcn_readlane(fh, src)) * kRow<Key> + lane;
            vh = *v;
            if ((unsigned)(tl + span) * 64 + lane <= hi) { vh = 0; *v = 0; }
        }
        s3_wave_fence();
        const unsigned tr = s3_wave_max_u32(top_word(lk)), t0 = s3_wave_max_u32(top_word(vl)), t1 = s3_wave_max_u32(top_word(vh));
        unsigned long long mr = __ballot(top_word(lk) == tr), m0 = __ballot(top_word(vl) == t0), m1 = __ballot(top_word(vh) == t1);
        settle(lk, tr, mr);
        settle(vl, t0, m0);
        settle(vh, t1, m1);
        const int sr = (int)__builtin_ctzll(mr), s0 = (int)__builtin_ctzll(m0), s1 = (int)__builtin_ctzll(m1);
        const Key kr = of_lane(lk, sr), k0 = of_lane(vl, s0), k1 = of_lane(vh, s1);
        const int pr = (int)of_lane((unsigned)lp, sr), p0 = tl * 64 + s0, p1 = (tl + span) * 64 + s1;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if (fl == q && k0) { k[q] = k0; p[q] = p0; }
            if (fh == q && k1) { k[q] = k1; p[q] = p1; }
        }
        best = kr;
        at = pr;
        if (k0 > best || (k0 == best && p0 < at)) { best = k0; at = p0; }
        if (k1 > best || (k1 == best && p1 < at)) { best = k1; at = p1; }
    }
    next = best;
    next_at = at;
    return found;
}

}  // namespace s3greedy
