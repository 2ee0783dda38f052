// Exact Top-k of one token by one wavefront: a list of candidates in LDS that new elements are filtered into, cut to
// (about) the k largest whenever it would overflow.  Shared by the tiled encoder and the merge of its feature ranges.
//
// Searches work on ordered keys (unsigned order = float order; 0 = no element).  -0 and +0 are one value, as in a float
// compare.  Inputs are finite; -inf marks the places that hold no element (nor does a NaN).  Elements arrive with ascending ids
// among equal values, so an element that only equals the threshold of a list that holds k at or above it loses to all of
// those.
//
// Everything that steers the search (counts, thresholds) is uniform: a count is one compare per register whose mask is
// counted by the scalar unit, so a bisection step over a 256-element list is 4 compares, 4 bit counts and 4 adds.
#pragma once
#include "s3_common.h"

namespace s3topk {

__device__ __forceinline__ unsigned key_of(float v) {
    const unsigned u = __float_as_uint(v + 0.f);                   // -0 -> +0
    const unsigned key = u ^ ((unsigned)((int)u >> 31) | 0x80000000u);
    return v == v ? key : 1u;
}
__device__ __forceinline__ float value_of(unsigned key) {
    return __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}
__device__ __forceinline__ int below(unsigned long long m) {       // set bits of m in lanes below this one
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

template <int N>
__device__ __forceinline__ int count_ge(const unsigned (&key)[N], unsigned m) {
    int c = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) c += (int)__popcll(__ballot(key[i] >= m));
    return c;
}

// The largest threshold found with k <= count(key >= threshold) <= loose, starting from lo (count clo >= k).  Returns the
// count; it exceeds `loose` only if more than loose - k elements equal the threshold.  Every other step interpolates on
// the logarithm of the counts (the upper tail of the values is close to exponential), the steps between halve the keys:
// about 6 steps instead of 20 for 256 fresh values.
template <int N>
__device__ __forceinline__ int raise(const unsigned (&key)[N], int k, int loose, unsigned& lo, int clo) {
    if (clo <= loose) return clo;
    unsigned mx = 0, mn = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        mx = max(mx, key[i]);
        mn = min(mn, key[i] - 1);                                  // no element: largest of all
    }
    unsigned hi = s3_wave_max_u32(mx) + 1;                              // keys stay below 0xFF800001
    lo = max(lo, 0xFFFFFFFFu - s3_wave_max_u32(0xFFFFFFFFu - mn) + 1);  // nothing lies below the smallest element
    int chi = 0;
    const float lwant = __log2f(0.5f * (float)(k + loose));
    bool interp = true;
    while (clo > loose && hi - lo > 1) {
        unsigned mid = lo + (hi - lo) / 2;
        if (interp) {
            const float llo = __log2f((float)clo), lhi = __log2f((float)max(chi, 1));
            const float t = fminf(fmaxf((llo - lwant) * __builtin_amdgcn_rcpf(llo - lhi), 0.0625f), 0.9375f);
            const float flo = value_of(lo), fhi = value_of(hi);
            const unsigned m = (unsigned)__builtin_amdgcn_readfirstlane((int)key_of(flo + (fhi - flo) * t));
            if (m > lo && m < hi) mid = m;
        }
        interp = !interp;
        const int c = count_ge(key, mid);
        if (c >= k) { lo = mid; clo = c; } else { hi = mid; chi = c; }
    }
    return clo;
}

// Of more than k elements at or above lo with fewer than k above it: the largest id up to which those that equal lo belong to
// the k best.
template <int N>
__device__ __forceinline__ unsigned tie_cut(const unsigned (&key)[N], const unsigned (&id)[N], int k, unsigned lo) {
    const int need = k - count_ge(key, lo + 1);
    int ilo = -1, ihi = 0xFFFF;           // count(tied, id <= ilo) < need <= count(tied, id <= ihi)
    while (ihi - ilo > 1) {
        const int mid = (ilo + ihi) >> 1;
        int c = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) c += (int)__popcll(__ballot(key[i] == lo && (int)id[i] <= mid));
        if (c >= need) ihi = mid; else ilo = mid;
    }
    return (unsigned)ihi;
}

// Cuts the N registers' elements to between k and `loose` (exactly k when loose == k) and stores them at lv / li[0 ..).
// `lo`: in, a threshold with at least k elements at or above it (at least 1); out, the new one.  Returns the number kept.
template <int N>
__device__ __forceinline__ int cut_and_store(const unsigned (&key)[N], const unsigned (&id)[N], int k, int loose, unsigned& lo,
                                             int clo, float* lv, uint16_t* li) {
    clo = raise(key, k, loose, lo, clo);
    const unsigned idcut = clo > loose ? tie_cut(key, id, k, lo) : 0xFFFFu;     // ties at the threshold: k elements in all
    int n = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const bool keep = key[i] > lo || (key[i] == lo && id[i] <= idcut);
        const unsigned long long m = __ballot(keep);
        if (keep) {
            const int at = n + below(m);
            lv[at] = value_of(key[i]);
            li[at] = (uint16_t)id[i];
        }
        n += (int)__popcll(m);
    }
    s3_wave_fence();
    return n;
}

// Takes the NC registers' elements above the list's threshold `tau` into a list of `cnt` with room for 64 * LR.  Element i of
// the lane has id id_of(i).  An append is kept short (most chunks bring a token one or two elements): four compares, and per
// register with a hit the position from the mask and two LDS writes.
template <int NC, int LR, class IdOf>
__device__ __forceinline__ void take(const float (&v)[NC], IdOf id_of, int k, int loose, float* lv, uint16_t* li, int& cnt,
                                     float& tau) {
    unsigned long long m[NC];
    int add = 0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        m[i] = __ballot(v[i] > tau);
        add += (int)__popcll(m[i]);
    }
    if (__builtin_expect(cnt + add <= 64 * LR, 1)) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            if (!m[i]) continue;
            if (v[i] > tau) {
                const int at = cnt + below(m[i]);
                lv[at] = v[i];
                li[at] = (uint16_t)id_of(i);
            }
            cnt += (int)__popcll(m[i]);
        }
        s3_wave_fence();
        return;
    }
    const int lane = threadIdx.x & 63;
    unsigned key[NC + LR], id[NC + LR];
#pragma unroll
    for (int i = 0; i < LR; ++i) {
        const int e = i * 64 + lane;
        key[i] = e < cnt ? key_of(lv[e]) : 0u;
        id[i] = e < cnt ? (unsigned)li[e] : 0u;
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) { key[LR + i] = v[i] > tau ? key_of(v[i]) : 0u; id[LR + i] = (unsigned)id_of(i); }
    // Every element is at or above tau, and there are more than 64 * LR >= k of them.
    unsigned lo = key_of(tau);
    cnt = cut_and_store<NC + LR>(key, id, k, loose, lo, cnt + add, lv, li);
    tau = value_of(lo);
}

// The list's k best (fewer if it holds fewer) in registers with their ranks (value descending, id ascending): element i of
// lane l has rank rank[i], or -1.
template <int LR>
__device__ __forceinline__ void finish(int k, float* lv, uint16_t* li, int cnt, unsigned (&key)[LR], unsigned (&id)[LR],
                                       int (&rank)[LR]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < LR; ++i) {
        const int e = i * 64 + lane;
        key[i] = e < cnt ? key_of(lv[e]) : 0u;
        id[i] = e < cnt ? (unsigned)li[e] : 0u;
    }
    const int loose = k + (k >> 3) + 2;            // the ranks below tell the k best of a few more than k
    if (cnt > loose) {
        unsigned lo = 1u;
        s3_wave_fence();
        cnt = cut_and_store<LR>(key, id, k, loose, lo, cnt, lv, li);
#pragma unroll
        for (int i = 0; i < LR; ++i) {
            const int e = i * 64 + lane;
            key[i] = e < cnt ? key_of(lv[e]) : 0u;
            id[i] = e < cnt ? (unsigned)li[e] : 0u;
        }
    }
    unsigned long long mine[LR];
#pragma unroll
    for (int i = 0; i < LR; ++i) {
        mine[i] = ((unsigned long long)key[i] << 32) | (0xFFFFFFFFu - id[i]);
        rank[i] = 0;
    }
#pragma unroll
    for (int r = 0; r < LR; ++r) {
        const int n = min(cnt - 64 * r, 64);
        for (int s = 0; s < n; ++s) {
            const unsigned ok = (unsigned)__builtin_amdgcn_readlane((int)key[r], s);
            const unsigned oi = (unsigned)__builtin_amdgcn_readlane((int)id[r], s);
            const unsigned long long other = ((unsigned long long)ok << 32) | (0xFFFFFFFFu - oi);
#pragma unroll
            for (int i = 0; i < LR; ++i) rank[i] += other > mine[i] ? 1 : 0;
        }
    }
#pragma unroll
    for (int i = 0; i < LR; ++i) if (!key[i] || rank[i] >= k) rank[i] = -1;
}

// The places [cnt, k) of a row with fewer than k elements above -inf (a bias of -inf, an overflow, a NaN): the lowest ids that
// are not in its list, id_at(0 .. cnt - 1) (k <= n_feat, so the first k ids are enough).  A row always holds k different ids
// below n_feat, in the order in which elements that equal -inf sort; with the ReLU their value is 0.
template <class IdAt>
__device__ __forceinline__ void fill_short(int k, int cnt, IdAt id_at, int32_t* ids, float* vals) {
    const int lane = threadIdx.x & 63;
    int at = cnt;
    for (int f0 = 0; f0 < k; f0 += 64) {
        const int f = f0 + lane;
        bool open = f < k;
        for (int s = 0; s < cnt; ++s) open = open && (int)id_at(s) != f;
        const unsigned long long m = __ballot(open);
        const int o = at + below(m);
        if (open && o < k) {
            ids[o] = f;
            vals[o] = 0.f;
        }
        at += (int)__popcll(m);
    }
}

}  // namespace s3topk
