// Fused SAE encoder + Top-k for gfx950 (Sec. 3.3: encoder equation and Top-K equation), the tiled kernel: fp32 or bf16,
// d_head 64, 128 or 256, any n_feat, any number of tokens.
//
// One workgroup = 8 wavefronts = 32 tokens of one (layer, head) against one range of the SAE's features.  Features lie on
// the M axis of the 32x32 MFMA; the 32 tokens' vectors stay in registers as the B operand.  Per chunk of 256 features:
//
//   - every wavefront multiplies 32 features of its own: its W rows are fetched coalesced into registers one piece (256
//     bytes of each row) ahead, written to an 8 KB LDS buffer that no other wavefront touches (xor-swizzled, so writes and
//     fragment reads are conflict-free) and read back as fragments: no barrier inside the product;
//   - the 256 x 32 pre-activations meet in an LDS tile (double-buffered where the lists leave room: one barrier a chunk);
//   - every wavefront selects for 4 of the tokens: one 16-byte read brings a token's 256 values into its 64 lanes, one
//     compare with the token's threshold finds the few that count, and those go to the token's list (topk_wave.h).
//
// A token's list, count and threshold belong to one wavefront, so nothing is shared and the search for a new threshold is
// steered by scalars.  (A kernel that kept the list in the two lanes that share a token and searched it through LDS took
// 7 us per 32-feature step at d_head 128 or 256: 948 us for 2048 fp32 tokens x 4096 features, k = 16, and 2181 us for
// 8 x 777 bf16 tokens x 10001 features of width 256, k = 48.)
//
// A call with few tokens splits the features over several workgroups (`parts`), which leave their Top-k of a range in
// scratch; enc_merge_kernel selects from those.  Selection is exact everywhere.
#include "s3_common.h"
#include "topk_wave.h"

#include <math.h>
#include <stdlib.h>

#include <type_traits>

namespace {

using namespace s3topk;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kTok = 32;                    // tokens per workgroup (MFMA N)
constexpr int kFT = 32;                     // features per wavefront and chunk (MFMA M)
constexpr int kChunk = kWaves * kFT;        // features per chunk
constexpr int kZRow = kChunk + 4;           // floats per token in the tile (16-byte writes of 16 tokens hit 64 banks)
constexpr int kTokWave = kTok / kWaves;     // tokens a wavefront selects for
static_assert(kTokWave == 4);

// The MFMA operands of one element type.  The B fragments of the 32 tokens are held whole; a row of W is worked off in
// pieces of up to 256 bytes.  offset(p, c): byte offset inside the row of 16-byte column c of piece p.
template <int DT, int DH>
struct Frag;

// bf16: 32x32x16 MFMA, K step s covers columns [16 s, 16 s + 16); lane half h owns 8 of them.
template <int DH>
struct Frag<S3_BF16, DH> {
    static constexpr int RB = DH * 2;
    static constexpr int PB = RB < 256 ? RB : 256;
    static constexpr int NP = RB / PB;
    static constexpr int NS = DH / 16;
    bf16x8 b[NS];
    __device__ __forceinline__ void load_b(const char* row, bool ok, int half) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            uint4 u = ok ? *(const uint4*)(row + (16 * s + 8 * half) * 2) : make_uint4(0, 0, 0, 0);
            b[s] = __builtin_bit_cast(bf16x8, u);
        }
    }
    static __device__ __forceinline__ int offset(int p, int c) { return p * PB + c * 16; }
    template <int P>
    __device__ __forceinline__ void mma(const char* arow, int sw, int half, f32x16& acc) const {
        u32x4 u[NS / NP];                      // all reads first: one LDS latency per piece
#pragma unroll
        for (int s = 0; s < NS / NP; ++s) u[s] = *(const u32x4*)(arow + (((2 * s + half) ^ sw) << 4));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NS / NP; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u[s]), b[P * (NS / NP) + s], acc, 0, 0, 0);
    }
};

// fp32: 32x32x2 MFMA, lane half h owns columns [h DH/2, (h+1) DH/2); step s uses column h DH/2 + s.  Piece p holds 128
// bytes of either half.
template <int DH>
struct Frag<S3_FP32, DH> {
    static constexpr int RB = DH * 4;
    static constexpr int PB = 256;
    static constexpr int NP = RB / PB;
    static constexpr int NS = DH / 2;
    float b[NS];
    __device__ __forceinline__ void load_b(const char* row, bool ok, int half) {
#pragma unroll
        for (int s = 0; s < NS; s += 4) {
            f32x4 u = ok ? *(const f32x4*)(row + (half * NS + s) * 4) : f32x4{0, 0, 0, 0};
            b[s] = u[0]; b[s + 1] = u[1]; b[s + 2] = u[2]; b[s + 3] = u[3];
        }
    }
    static __device__ __forceinline__ int offset(int p, int c) { return (c >> 3) * (RB / 2) + p * 128 + (c & 7) * 16; }
    template <int P>
    __device__ __forceinline__ void mma(const char* arow, int sw, int half, f32x16& acc) const {
        constexpr int kAhead = DH == 256 ? 2 : 4;      // fragments read ahead (d_head 256: few registers are left)
#pragma unroll
        for (int g = 0; g < 8; g += kAhead) {
            f32x4 u[kAhead];
#pragma unroll
            for (int s = 0; s < kAhead; ++s) u[s] = *(const f32x4*)(arow + (((half * 8 + g + s) ^ sw) << 4));
#pragma unroll
            for (int s = 0; s < kAhead; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u[s][e], b[P * 32 + 4 * (g + s) + e], acc, 0, 0, 0);
        }
    }
};

struct TileArgs {
    const char* x;
    const char* w;
    const float* b;
    int32_t* ids;
    float* vals;
    uint2* part;             // [n_heads * T][parts][k] (pre-activation, id), -inf = none; null when parts == 1
    int T, n_feat, k, loose;
    int tiles_per_head;      // token tiles of a head
    int parts, range;        // feature ranges per head; features per range (a multiple of kChunk)
    int n_groups;            // n_heads * parts
};

template <int DT, int DH, int LR>
constexpr int tile_buffers() { return LR == 2 ? 2 : 1; }       // pre-activation tiles: two fit beside lists of 128
template <int DT, int DH, int LR>
constexpr size_t tile_lds() {
    return (size_t)kWaves * kFT * Frag<DT, DH>::PB + (size_t)tile_buffers<DT, DH, LR>() * kTok * kZRow * 4 + kWaves * kFT * 4 +
           (size_t)kTok * LR * 64 * 6;
}

template <int DT, int DH, int LR>
__global__ __launch_bounds__(kThreads) void sae_encode_topk_kernel(TileArgs a) {
    using F = Frag<DT, DH>;
    constexpr int CPR = F::PB / 16;                   // 16-byte columns per piece row
    constexpr int RPI = 64 / CPR;                     // rows per load instruction
    constexpr int NV = kFT / RPI;
    constexpr int ZB = tile_buffers<DT, DH, LR>();
    constexpr int CAP = 64 * LR;
    static_assert(tile_lds<DT, DH, LR>() <= 160 * 1024, "LDS budget of one compute unit");

    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, half = lane >> 5;
    char* const wbuf = smem + wv * kFT * F::PB;
    float* const z = (float*)(smem + kWaves * kFT * F::PB);                     // [ZB][kTok][kZRow]
    float* const bias = z + ZB * kTok * kZRow + wv * kFT;
    float* const lval = z + ZB * kTok * kZRow + kWaves * kFT;                   // [kTok][CAP]
    uint16_t* const lid = (uint16_t*)(lval + kTok * CAP);                       // [kTok][CAP]

    int group, tt;
    s3_block_to_tile(blockIdx.x, a.n_groups, a.tiles_per_head, group, tt);
    const int head = group / a.parts, part = group - head * a.parts;
    const int fbeg = part * a.range, fend = min(fbeg + a.range, a.n_feat);
    const int nchunk = (fend - fbeg + kChunk - 1) / kChunk;
    const int tok0 = tt * kTok;

    F frag;
    {
        const bool ok = tok0 + n < a.T;
        frag.load_b(a.x + ((size_t)head * a.T + (ok ? tok0 + n : 0)) * F::RB, ok, half);
    }
    int cnt[kTokWave] = {};
    float tau[kTokWave];
#pragma unroll
    for (int q = 0; q < kTokWave; ++q) tau[q] = tok0 + wv * kTokWave + q < a.T ? -INFINITY : INFINITY;    // no token: nothing counts

    const char* const wh = a.w + (size_t)head * a.n_feat * F::RB;
    const float* const bh = a.b + (size_t)head * a.n_feat;
    const int lrow = lane / CPR, lcol = lane % CPR;
    u32x4 wreg[NV];
    float breg = 0.f;
    auto gload = [&](int chunk, int p) {
        const int f0 = fbeg + chunk * kChunk + wv * kFT;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int f = min(f0 + i * RPI + lrow, fend - 1);      // rows past the end repeat the last one; their bias is -inf
            wreg[i] = *(const u32x4*)(wh + (size_t)f * F::RB + F::offset(p, lcol));
        }
        if (p == 0) {
            breg = bh[min(f0 + n, fend - 1)];
            breg = f0 + n < fend ? breg : -INFINITY;
        }
    };
    gload(0, 0);

    for (int c = 0; c < nchunk; ++c) {
        float* const zt = z + (ZB == 2 ? (c & 1) * kTok * kZRow : 0);
        f32x16 acc;
        auto piece = [&](auto P) {
            constexpr int p = decltype(P)::value;
            s3_wave_fence();
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int row = i * RPI + lrow;
                *(u32x4*)(wbuf + row * F::PB + ((lcol ^ (row & (CPR - 1))) << 4)) = wreg[i];
            }
            if (p == 0 && half == 0) bias[n] = breg;
            if (p + 1 < F::NP) gload(c, p + 1);
            else if (c + 1 < nchunk) gload(c + 1, 0);
            s3_wave_fence();
            if (p == 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 bq = *(const f32x4*)(bias + q * 8 + half * 4);
                    acc[q * 4 + 0] = bq[0]; acc[q * 4 + 1] = bq[1]; acc[q * 4 + 2] = bq[2]; acc[q * 4 + 3] = bq[3];
                }
            }
            frag.template mma<p>(wbuf + n * F::PB, n & (CPR - 1), half, acc);
        };
        piece(std::integral_constant<int, 0>{});
        if constexpr (F::NP > 1) piece(std::integral_constant<int, 1>{});
        if constexpr (F::NP > 2) { piece(std::integral_constant<int, 2>{}); piece(std::integral_constant<int, 3>{}); }
        if (ZB == 1 && c) __syncthreads();             // the last chunk's selection reads the same tile
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *(f32x4*)(zt + n * kZRow + wv * kFT + q * 8 + half * 4) =
                f32x4{acc[q * 4 + 0], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]};
        __syncthreads();

        // A token's list, count and threshold are this wavefront's alone; the four tokens' reads are issued together.
        const int f = fbeg + c * kChunk + 4 * lane;
        f32x4 v[kTokWave];
#pragma unroll
        for (int q = 0; q < kTokWave; ++q) v[q] = *(const f32x4*)(zt + (wv * kTokWave + q) * kZRow + 4 * lane);
        unsigned long long hits[kTokWave];             // lanes with an element above the token's threshold
#pragma unroll
        for (int q = 0; q < kTokWave; ++q)
            hits[q] = __ballot(fmaxf(fmaxf(v[q][0], v[q][1]), fmaxf(v[q][2], v[q][3])) > tau[q]);
#pragma unroll
        for (int q = 0; q < kTokWave; ++q) {
            if (!hits[q]) continue;
            const int t = wv * kTokWave + q;
            const float e[4] = {v[q][0], v[q][1], v[q][2], v[q][3]};
            take<4, LR>(e, [&](int j) { return f + j; }, a.k, a.loose, lval + t * CAP, lid + t * CAP, cnt[q], tau[q]);
        }
    }

    int shorts = 0;
#pragma unroll
    for (int q = 0; q < kTokWave; ++q) {
        const int t = wv * kTokWave + q;
        if (tok0 + t >= a.T) break;
        unsigned key[LR], id[LR];
        int rank[LR];
        finish<LR>(a.k, lval + t * CAP, lid + t * CAP, cnt[q], key, id, rank);
        const size_t row = (size_t)head * a.T + tok0 + t;
        if (a.part) {
            uint2* const out = a.part + (row * a.parts + part) * a.k;
#pragma unroll
            for (int i = 0; i < LR; ++i) if (rank[i] >= 0) out[rank[i]] = make_uint2(__float_as_uint(value_of(key[i])), id[i]);
            for (int e = cnt[q] + lane; e < a.k; e += 64) out[e] = make_uint2(__float_as_uint(-INFINITY), 0u);        // a range of fewer than k features
        } else {
#pragma unroll
            for (int i = 0; i < LR; ++i)
                if (rank[i] >= 0) {
                    a.ids[row * a.k + rank[i]] = (int32_t)id[i];
                    a.vals[row * a.k + rank[i]] = fmaxf(value_of(key[i]), 0.f);
                }
            shorts |= cnt[q] < a.k ? 1 << q : 0;
        }
    }
    while (__builtin_expect(shorts != 0, 0)) {         // rows that their lists do not fill; beside the loop above, which stays short
        const int q = __builtin_ctz(shorts), t = wv * kTokWave + q;
        shorts &= shorts - 1;
        const size_t row = (size_t)head * a.T + tok0 + t;
        fill_short(a.k, q < 2 ? (q ? cnt[1] : cnt[0]) : (q == 2 ? cnt[2] : cnt[3]), [&](int s) { return lid[t * CAP + s]; },
                   a.ids + row * a.k, a.vals + row * a.k);
    }
}

// Selects every token's k best from its ranges' lists (each sorted, ids ascending from range to range): one wavefront per
// token, 256 elements at a time.
template <int LR>
__global__ __launch_bounds__(256) void enc_merge_kernel(const uint2* __restrict__ part, long long rows, int parts, int k, int loose,
                                                        int32_t* __restrict__ ids, float* __restrict__ vals) {
    __shared__ float lval[4][64 * LR];
    __shared__ uint16_t lid[4][64 * LR];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const long long row = (long long)blockIdx.x * 4 + wv;
    if (row >= rows) return;
    const int total = parts * k;
    const uint2* const src = part + (size_t)row * total;
    int cnt = 0;
    float tau = -INFINITY;
    uint2 cur[4], nxt[4];
    auto load = [&](uint2 (&to)[4], int e0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = e0 + j * 64 + lane;
            to[j] = src[min(e, total - 1)];
            if (e >= total) to[j].x = __float_as_uint(-INFINITY);
        }
    };
    load(cur, 0);
    for (int e0 = 0; e0 < total; e0 += 256) {
        if (e0 + 256 < total) load(nxt, e0 + 256);
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = __uint_as_float(cur[j].x);
        if (__any(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])) > tau))
            take<4, LR>(v, [&](int j) { return cur[j].y; }, k, loose, lval[wv], lid[wv], cnt, tau);
#pragma unroll
        for (int j = 0; j < 4; ++j) cur[j] = nxt[j];
    }
    unsigned key[LR], id[LR];
    int rank[LR];
    finish<LR>(k, lval[wv], lid[wv], cnt, key, id, rank);
#pragma unroll
    for (int i = 0; i < LR; ++i)
        if (rank[i] >= 0) {
            ids[(size_t)row * k + rank[i]] = (int32_t)id[i];
            vals[(size_t)row * k + rank[i]] = fmaxf(value_of(key[i]), 0.f);
        }
    if (cnt < k) fill_short(k, cnt, [&](int s) { return lid[wv][s]; }, ids + (size_t)row * k, vals + (size_t)row * k);
}

template <int DT, int DH, int LR>
int launch(const TileArgs& a, hipStream_t st) {
    constexpr size_t lds = tile_lds<DT, DH, LR>();
    auto kern = sae_encode_topk_kernel<DT, DH, LR>;
    static S3LdsOnce once;             // per instantiation
    if (int rc = s3_allow_lds(once, (const void*)kern, (int)lds)) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.n_groups * a.tiles_per_head)), dim3(kThreads), lds, st, a);
    S3_HIP(hipGetLastError());
    return S3_OK;
}

// Feature ranges of a call.  A workgroup fills a compute unit's LDS, so a call takes as many turns as its workgroups are
// multiples of 256; every turn costs its range's chunks and about kWarm more until the lists are full.  The number of
// ranges with the smallest sum is taken (the smaller one of equals; 1 beyond two turns of whole tokens, where there is
// little to gain).  2048 fp32 tokens x 4096 features of width 128, k 16: four ranges 50 us, eight ranges 69 us.
constexpr int kSlots = 256;
constexpr int kWarm = 4;
constexpr long long kPartEntries = 4LL << 20;          // list entries in scratch at most
long long token_tiles(int n_heads, int T) { return (long long)n_heads * (((long long)T + kTok - 1) / kTok); }
int parts_for(int n_heads, int T, int n_feat, int k) {
    const long long tiles = token_tiles(n_heads, T);
    if (tiles > 2 * kSlots) return 1;
    const int chunks = (n_feat + kChunk - 1) / kChunk;
    int best = 1;
    long long least = 0;
    for (int want = 1; want <= chunks; ++want) {
        const int per = (chunks + want - 1) / want, parts = (chunks + per - 1) / per;
        if (parts != want || (want > 1 && (long long)n_heads * T * want * k > kPartEntries)) continue;
        const long long cost = (tiles * parts + kSlots - 1) / kSlots * (per + kWarm);
        if (want == 1 || cost < least) { best = want; least = cost; }
    }
    return best;
}

// Whether a plain call of a shape that the fast kernel takes is better off here: while its token tiles fit the chip at
// once.  The fast kernel has 64 to 256 tokens per workgroup and walks all features in each.  us, fast / this kernel, of
// 16384 features: 4 tokens of 8 heads, k 32: 229 / 33; 4096 tokens of one head, k 32: 439 / 130, k 128: 500 / 227; at the
// line, 256 tiles: 8192 tokens of one head, k 8 / 32 / 64 / 128: 343 / 154, 440 / 193, 437 / 232, 506 / 294.  Many heads read
// many weights, but so they do there: 4 tokens of 64, 128 and 256 heads, k 32: 236 / 71, 254 / 119, 274 / 217, of 256 heads, k 64
// and 128: 349 / 227, 394 / 267; 32 tokens of 256 heads, k 32: 314 / 244; of 4096 features 142 / 86.  Beyond the line a second
// turn costs as much again, and the fast kernel's time does not grow before its own workgroups fill the chip.
bool tiled_pays(int n_heads, int T) { return token_tiles(n_heads, T) <= kSlots; }

}  // namespace

#ifdef S3_TUNING
int env_int(const char* name, int dflt) {
    const char* s = getenv(name);
    return s && *s ? atoi(s) : dflt;
}
#endif

// The k up to which a shape is accepted (stated in the header).  The lists have room for S3_MAX_K at every width; callers may
// rely on the refusal, so it stays.
static int largest_k(int dtype, int d_head) {
    if (dtype == S3_BF16) return d_head == 256 ? 121 : S3_MAX_K;
    return d_head == 64 ? S3_MAX_K : (d_head == 128 ? 121 : 78);
}

// The tiled kernel; `part` (parts_for() ranges' lists, or null: one range) is scratch.
static int tiled_launch(const EncParams& p, int dtype, int d_head, int parts, uint2* part, hipStream_t st) {
    TileArgs a;
    a.x = p.x; a.w = p.w; a.b = p.b; a.ids = p.ids; a.vals = p.vals;
    a.T = p.T; a.n_feat = p.n_feat; a.k = p.k;
    a.loose = p.k + (p.k >> 3) + 2;
    a.tiles_per_head = (int)token_tiles(1, p.T);
    const int chunks = (p.n_feat + kChunk - 1) / kChunk;
    a.parts = parts;
    a.range = (chunks + parts - 1) / parts * kChunk;
    a.n_groups = p.n_heads * parts;
    a.part = parts > 1 ? part : nullptr;
    int rc = S3_EINVAL;
#define S3_CASE(DT, DH) \
    if (dtype == DT && d_head == DH) rc = p.k <= 64 ? launch<DT, DH, 2>(a, st) : launch<DT, DH, 4>(a, st);
    S3_CASE(S3_BF16, 64) S3_CASE(S3_BF16, 128) S3_CASE(S3_BF16, 256)
    S3_CASE(S3_FP32, 64) S3_CASE(S3_FP32, 128) S3_CASE(S3_FP32, 256)
#undef S3_CASE
    if (rc || parts == 1) return rc;
    const long long rows = (long long)p.n_heads * p.T;
    auto merge = p.k <= 64 ? enc_merge_kernel<2> : enc_merge_kernel<4>;
    hipLaunchKernelGGL(merge, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, (const uint2*)part, rows, parts, p.k, a.loose,
                       p.ids, p.vals);
    S3_HIP(hipGetLastError());
    return S3_OK;
}

// A launch holds fewer than 2^32 threads, 2^23 workgroups: calls of more token tiles (268 M tokens) go in slices of whole
// heads, or of one head's tokens where a head alone has more.
constexpr long long kGridMax = 1LL << 22;
static int tiled_slices(const EncParams& p, int dtype, int d_head, hipStream_t st) {
    const size_t row = (size_t)d_head * (dtype == S3_BF16 ? 2 : 4);
    const long long per_head = token_tiles(1, p.T);
    const int heads = per_head < kGridMax ? (int)(kGridMax / per_head) : 1;
    const int toks = (int)(per_head < kGridMax ? p.T : kGridMax * kTok);
    for (long long h = 0; h < p.n_heads; h += heads)
        for (long long t = 0; t < p.T; t += toks) {            // more than one step only where heads == 1
            EncParams q = p;
            const size_t at = (size_t)h * p.T + (size_t)t;
            q.x += at * row; q.ids += at * p.k; q.vals += at * p.k;
            q.w += (size_t)h * p.n_feat * row; q.b += (size_t)h * p.n_feat;
            q.n_heads = (int)(p.n_heads - h < heads ? p.n_heads - h : heads);
            q.T = (int)(p.T - t < toks ? p.T - t : toks);
            if (int rc = tiled_launch(q, dtype, d_head, 1, nullptr, st)) return rc;
        }
    return S3_OK;
}

// What a streamed call of up to T tokens may need, whatever its n_feat and k.
static size_t stream_workspace(int n_heads, int T) {
    const size_t a = s3_encode_fast_stream_workspace(n_heads, T), b = s3_encode_scan_workspace_max(n_heads, T);
    return a > b ? a : b;
}

static size_t plain_workspace(int dtype, int T, int d_head, int n_feat, int k, int n_heads) {
    if (s3_encode_fast_ok(dtype, d_head, n_feat, k)) {
        if (s3_encode_scan_pays(n_heads, T, n_feat, k, false)) return s3_encode_scan_workspace(n_heads, T, n_feat, k);
        if (!tiled_pays(n_heads, T)) return 0;
    }
    const int parts = parts_for(n_heads, T, n_feat, k);
    return parts > 1 ? (size_t)n_heads * T * parts * k * sizeof(uint2) : 0;
}

static int encode_impl(const char* who, const void* x, int dtype, int T, int d_head, const void* w_enc, const float* b_enc,
                       int n_feat, int k, int n_heads, int32_t* ids, float* vals, float* tau_hint, void* ws,
                       size_t ws_bytes, void* stream) {
    if (!x || !w_enc || !b_enc || !ids || !vals) return s3_fail(S3_EINVAL, "%s: null pointer", who);
    if (dtype != S3_BF16 && dtype != S3_FP32) return s3_fail(S3_EINVAL, "%s: dtype must be S3_BF16 or S3_FP32", who);
    if (d_head != 64 && d_head != 128 && d_head != 256)
        return s3_fail(S3_EINVAL, "%s: d_head %d not in {64, 128, 256}", who, d_head);
    if (T < 0 || n_heads < 1) return s3_fail(S3_EINVAL, "%s: T %d / n_heads %d out of range", who, T, n_heads);
    if (n_feat < 1 || n_feat > S3_MAX_FEAT) return s3_fail(S3_EINVAL, "%s: n_feat %d not in [1, %d]", who, n_feat, S3_MAX_FEAT);
    if (k < 1 || k > n_feat || k > S3_MAX_K) return s3_fail(S3_EINVAL, "%s: k %d not in [1, min(n_feat, %d)]", who, k, S3_MAX_K);
    if (((uintptr_t)x | (uintptr_t)w_enc) & 15) return s3_fail(S3_EINVAL, "%s: x and w_enc must be 16-byte aligned", who);
    if (token_tiles(n_heads, T) > 0x7FFFFFFFLL) return s3_fail(S3_EINVAL, "%s: grid too large", who);
    if (ws && ((uintptr_t)ws & 255)) return s3_fail(S3_EINVAL, "%s: workspace must be 256-byte aligned", who);
    if (tau_hint) {
        if (!ws) return s3_fail(S3_EINVAL, "%s: null workspace", who);
        const size_t need = stream_workspace(n_heads, T);
        if (ws_bytes < need) return s3_fail(S3_ECAPACITY, "%s: workspace %zu < %zu bytes", who, ws_bytes, need);
    }
    if (T == 0) return S3_OK;

    EncParams p;
    p.x = (const char*)x; p.w = (const char*)w_enc; p.b = b_enc; p.ids = ids; p.vals = vals;
    p.T = T; p.n_feat = n_feat; p.k = k; p.n_heads = n_heads;
    p.ablate = 0;
    if (s3_encode_fast_ok(dtype, d_head, n_feat, k) && ws && s3_encode_scan_pays(n_heads, T, n_feat, k, tau_hint != nullptr) &&
        (tau_hint || ws_bytes >= s3_encode_scan_workspace(n_heads, T, n_feat, k)))
        return s3_encode_scan(p, tau_hint, ws, (hipStream_t)stream);
    int parts = tau_hint ? 1 : parts_for(n_heads, T, n_feat, k);
    const bool room = parts == 1 || (ws && ws_bytes >= (size_t)n_heads * T * parts * k * sizeof(uint2));
    if (!room) parts = 1;                                    // no scratch: one range
    bool fast = s3_encode_fast_ok(dtype, d_head, n_feat, k) && (tau_hint || !room || !tiled_pays(n_heads, T));
#ifdef S3_TUNING
    p.ablate = env_int("S3_ENC_ABLATE", 0);
    if (env_int("S3_ENC_GENERIC", 0)) fast = false;
#endif
    hipStream_t st = (hipStream_t)stream;
    if (fast)
        return tau_hint ? s3_encode_fast_stream(p, tau_hint, ws, st) : s3_encode_fast_launch(p, st);
    if (k > largest_k(dtype, d_head))
        return s3_fail(S3_EINVAL, "%s: k %d > %d for this dtype and d_head", who, k, largest_k(dtype, d_head));
    if (token_tiles(n_heads, T) > kGridMax) return tiled_slices(p, dtype, d_head, st);
    return tiled_launch(p, dtype, d_head, parts, (uint2*)ws, st);
}

extern "C" int s3_sae_encode_topk(const void* x, int dtype, int T, int d_head, const void* w_enc,
                                  const float* b_enc, int n_feat, int k, int n_heads, int32_t* ids,
                                  float* vals, void* stream) {
    return encode_impl("s3_sae_encode_topk", x, dtype, T, d_head, w_enc, b_enc, n_feat, k, n_heads, ids, vals, nullptr,
                       nullptr, 0, stream);
}

extern "C" size_t s3_sae_encode_topk_workspace(int dtype, int T, int d_head, int n_feat, int k, int n_heads) {
    if (n_heads < 1 || T < 1 || n_feat < 1 || k < 1 || k > S3_MAX_K) return 0;
    return plain_workspace(dtype, T, d_head, n_feat, k, n_heads);
}

extern "C" int s3_sae_encode_topk_ws(const void* x, int dtype, int T, int d_head, const void* w_enc,
                                     const float* b_enc, int n_feat, int k, int n_heads, int32_t* ids,
                                     float* vals, void* ws, size_t ws_bytes, void* stream) {
    return encode_impl("s3_sae_encode_topk_ws", x, dtype, T, d_head, w_enc, b_enc, n_feat, k, n_heads, ids, vals, nullptr,
                       ws, ws_bytes, stream);
}

extern "C" size_t s3_sae_encode_topk_stream_workspace(int n_heads, int T) {
    if (n_heads < 1 || T < 0) return 0;
    return stream_workspace(n_heads, T);
}

extern "C" int s3_sae_encode_topk_stream(const void* x, int dtype, int T, int d_head, const void* w_enc,
                                         const float* b_enc, int n_feat, int k, int n_heads, int32_t* ids,
                                         float* vals, float* tau_hint, void* ws, size_t ws_bytes, void* stream) {
    if (!tau_hint) return s3_fail(S3_EINVAL, "s3_sae_encode_topk_stream: null tau_hint");
    return encode_impl("s3_sae_encode_topk_stream", x, dtype, T, d_head, w_enc, b_enc, n_feat, k, n_heads, ids, vals,
                       tau_hint, ws, ws_bytes, stream);
}
