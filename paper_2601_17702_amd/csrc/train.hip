// One optimisation step of the Top-K SAE (Sec. 3.3: encoder, Top-K and decoder equations; App. B.3: Adam, batches of
// 4096 tokens, k = 128) on the mean squared reconstruction error, entirely on the GPU:
//
//   1. u = bf16(x - b_dec), bf16(W_enc)                       the encoder's operands in the inference path's format
//   2. (ids, zhat) = TopK(W_enc u + b_enc)                    the fused encoder of this library (s3_sae_encode_topk)
//   3. per token: xhat = zhat W_dec + b_dec, g = 2 (xhat - x) / (B d), dz = (g . W_dec[id]) [zhat > 0],
//      du = sum_i dz_i W_enc[id_i], and the token's part of the loss
//   4. inverted index of the batch: feature -> the (token, slot) pairs that selected it (s3_index_build on the
//      flattened ids, one posting per pair) -- the same structure the retrieval path builds, used here to turn the
//      scatter of the weight gradients into one ordered sum per feature
//   5. per feature: dW_dec[f] = sum zhat g_t, dW_enc[f] = sum dz u_t, db_enc[f] = sum dz over its postings, in
//      posting order (no atomics: the sums are the same from run to run)
//   6. db_dec = sum_t (g_t - du_t), loss = sum of the parts / (B d), both in a fixed order
//   7. Adam on all four parameter arrays
//
// The backward pass holds the selection fixed and treats the bf16 rounding of the encoder's operands as the identity.
#include "s3_common.h"

#include <math.h>

namespace {

constexpr int DH = 128;              // d_head of the fast encoder
constexpr int kTokThreads = 256;     // four tokens / four features per workgroup, one wavefront each
constexpr int kChunk = 32;           // tokens per partial column sum

__device__ __forceinline__ uint16_t bf16_rne(float v) {      // finite inputs
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Sum over the 64 lanes in a fixed order (lane shifts inside rows of 16, then across rows), returned to every lane.
#define S3_DPP_ADD(X, CTRL, ROWS) X += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(X), CTRL, ROWS, 0xf, false))
__device__ __forceinline__ float wave_sum(float x) {
    S3_DPP_ADD(x, 0x111, 0xf);
    S3_DPP_ADD(x, 0x112, 0xf);
    S3_DPP_ADD(x, 0x114, 0xf);
    S3_DPP_ADD(x, 0x118, 0xf);
    S3_DPP_ADD(x, 0x142, 0xa);
    S3_DPP_ADD(x, 0x143, 0xc);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
#undef S3_DPP_ADD

__global__ void tr_prep_kernel(const float* x, const float* b_dec, const float* w_enc, uint16_t* u_bf, uint16_t* w_bf,
                               int64_t n_x, int64_t n_w) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_x) u_bf[i] = bf16_rne(x[i] - b_dec[i & (DH - 1)]);
    if (i < n_w) w_bf[i] = bf16_rne(w_enc[i]);
}

struct TokArgs {
    const float* x;
    const float* w_dec;
    const float* b_dec;
    const uint16_t* w_bf;
    const int32_t* ids;
    const float* vals;
    float* g;
    float* dz;
    float* du;
    double* lossp;
    int B, k;
    float scale;          // 2 / (B d)
};

// Step 3: one wavefront per token; lane l holds columns 2 l and 2 l + 1.  The token's ids and values are read once
// (entry i in lane i % 64, register i / 64; k <= 128) and handed out by readlane, and the decoder rows are fetched
// kRows at a time, so that no load waits for the previous row's arithmetic; the sums keep the order of the entries.
// Latency bounds it: 4096 x 128 tokens, 16384 latents, k 128: 55 us with four rows in flight, 52 with eight.
constexpr int kRows = 8;
__global__ __launch_bounds__(kTokThreads) void tr_token_kernel(TokArgs a) {
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * (kTokThreads / 64) + (threadIdx.x >> 6);
    if (t >= a.B) return;
    const int32_t* __restrict__ ids = a.ids + (size_t)t * a.k;
    const float* __restrict__ vals = a.vals + (size_t)t * a.k;
    const float* __restrict__ w_dec = a.w_dec;
    const uint16_t* __restrict__ w_bf = a.w_bf;
    int my_id[2];
    float my_v[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int i = lane + 64 * r;
        my_id[r] = i < a.k ? ids[i] : 0;
        my_v[r] = i < a.k ? vals[i] : 0.f;
    }
    const float2 xv = *(const float2*)(a.x + (size_t)t * DH + 2 * lane);
    float2 acc = *(const float2*)(a.b_dec + 2 * lane);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int kk = min(a.k - 64 * r, 64);
        for (int i0 = 0; i0 < kk; i0 += kRows) {
            float2 row[kRows];
            float v[kRows];
#pragma unroll
            for (int q = 0; q < kRows; ++q) {        // entries past the end repeat the group's first one with value 0
                const int i = i0 + q < kk ? i0 + q : i0;
                const int f = __builtin_amdgcn_readlane(my_id[r], i);
                v[q] = i0 + q < kk ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_v[r]), i)) : 0.f;
                row[q] = *(const float2*)(w_dec + (size_t)f * DH + 2 * lane);
            }
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                acc.x += v[q] * row[q].x;
                acc.y += v[q] * row[q].y;
            }
        }
    }
    const float rx = acc.x - xv.x, ry = acc.y - xv.y;
    const float part = wave_sum(rx * rx + ry * ry);
    if (lane == 0) a.lossp[t] = (double)part;
    const float gx = rx * a.scale, gy = ry * a.scale;
    *(float2*)(a.g + (size_t)t * DH + 2 * lane) = make_float2(gx, gy);
    float dux = 0.f, duy = 0.f;
    float* __restrict__ dz_out = a.dz + (size_t)t * a.k;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int kk = min(a.k - 64 * r, 64);
        for (int i0 = 0; i0 < kk; i0 += kRows) {
            float2 row[kRows];
            uint32_t we[kRows];
            float v[kRows], dz[kRows];
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                const int i = i0 + q < kk ? i0 + q : i0;
                const int f = __builtin_amdgcn_readlane(my_id[r], i);
                v[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_v[r]), i));
                row[q] = *(const float2*)(w_dec + (size_t)f * DH + 2 * lane);
                we[q] = *(const uint32_t*)(w_bf + (size_t)f * DH + 2 * lane);
            }
#pragma unroll
            for (int q = 0; q < kRows; ++q) {        // independent reductions: their lane shifts interleave
                const float dot = wave_sum(gx * row[q].x + gy * row[q].y);
                dz[q] = (i0 + q < kk && v[q] > 0.f) ? dot : 0.f;
            }
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                if (lane == 0 && i0 + q < kk) dz_out[64 * r + i0 + q] = dz[q];
                dux += dz[q] * __uint_as_float(we[q] << 16);
                duy += dz[q] * __uint_as_float(we[q] & 0xFFFF0000u);
            }
        }
    }
    *(float2*)(a.du + (size_t)t * DH + 2 * lane) = make_float2(dux, duy);
}

// Adam (step 7) on one value.
struct AdamArgs {
    float lr, b1, b2, eps, c1, c2;      // c1 = 1 - b1^t, c2 = 1 - b2^t
};
__device__ __forceinline__ void adam(const AdamArgs& a, float g, float& p, float& m, float& v) {
    m = a.b1 * m + (1.f - a.b1) * g;
    v = a.b2 * v + (1.f - a.b2) * g * g;
    p -= a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

struct FeatArgs {
    const int32_t* offsets;
    const int32_t* slots;
    const float* vals;
    const float* dz;
    const float* g;
    const uint16_t* u_bf;
    float* grads;         // W_enc | b_enc | W_dec | b_dec, or null
    float* w_enc;
    float* b_enc;
    float* w_dec;
    float* m;             // both moments in the gradients' order
    float* v;
    AdamArgs adam;
    int n_feat, k;
    uint32_t kinv;        // ceil(2^32 / k): slot / k for slot < 2^24
    int n_long, per;      // workgroups that look for long lists, features each of them looks at
    int long_list;        // longer than this
};

// Step 5, and step 7 for W_enc, b_enc and W_dec: one wavefront per feature; its postings (flat slot = token * k + slot in the
// row, ascending) are taken 64 at a time -- each lane fetches one posting's scalars, then the wavefront walks them in order.  A
// posting is 8 bytes a lane from two rows (latency: 0.125 us each with four in flight, eight now), so one list of all 4096 tokens
// took 511 us: lists of more than long_list are shared by the wavefronts of a workgroup, whose sums are added in list order
// (4096 x 128 tokens, a few features in every token's selection).  The first workgroups of the launch look for these, kLongPer
// features each, so that they run beside the short lists (a launch of their own behind those: 64 + 26 to 40 us after hundreds of
// steps on one batch, now 71).  Below kFewFeat features lists are long: a workgroup of sixteen wavefronts each (a step of 4096
// tokens, k 128, 128 latents: 417 us with eight and four features a workgroup, 200 before, now 187), and from kLongListFew postings on,
// unless the batch is small and features are met seldom (200 tokens, k 4, 3968 latents 55 / 61 us with workgroups that find no list;
// 256 tokens, k 128, 128 latents, lists of 256: 154 / 109).
// Adam on the feature's two rows and its bias follows at once: the gradients need not be written and read again, and one
// wavefront's parameters and moments come while others walk lists (4096 x 128 tokens, 16384 latents, k 128: 64 us and 20 for Adam on
// all parameters -> 67; in workgroups of sixteen features, which all wait for their longest, 97).
constexpr int kLongList = 256, kLongListFew = 128;
constexpr int kLongPer = 4;
constexpr int kFewFeat = 4096;

struct FeatSums {
    float ex, ey, dx, dy, sb;
};
__device__ __forceinline__ FeatSums feature_sums(const FeatArgs& a, int beg, int end, int lane) {
    FeatSums r = {0.f, 0.f, 0.f, 0.f, 0.f};
    for (int j0 = beg; j0 < end; j0 += 64) {
        const int n = min(64, end - j0);
        int my_t = 0;
        float my_v = 0.f, my_dz = 0.f;
        if (lane < n) {
            const int s = a.slots[j0 + lane];
            my_t = a.k == 1 ? s : (int)(((uint64_t)(uint32_t)s * a.kinv) >> 32);
            my_v = a.vals[s];
            my_dz = a.dz[s];
        }
        for (int q0 = 0; q0 < n; q0 += kRows) {  // kRows postings' rows in flight; the sums keep the posting order
            float2 gv[kRows];
            uint32_t uu[kRows];
            float v[kRows], dz[kRows];
#pragma unroll
            for (int j = 0; j < kRows; ++j) {        // postings past the end repeat the last one with weights 0
                const int q = min(q0 + j, n - 1);
                const int t = __builtin_amdgcn_readlane(my_t, q);
                v[j] = q0 + j < n ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_v), q)) : 0.f;
                dz[j] = q0 + j < n ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_dz), q)) : 0.f;
                gv[j] = *(const float2*)(a.g + (size_t)t * DH + 2 * lane);
                uu[j] = *(const uint32_t*)(a.u_bf + (size_t)t * DH + 2 * lane);
            }
#pragma unroll
            for (int j = 0; j < kRows; ++j) {
                r.dx += v[j] * gv[j].x;
                r.dy += v[j] * gv[j].y;
                r.ex += dz[j] * __uint_as_float(uu[j] << 16);
                r.ey += dz[j] * __uint_as_float(uu[j] & 0xFFFF0000u);
                r.sb += dz[j];
            }
        }
    }
    return r;
}
// A feature's parameters and moments: two columns of both rows per lane, the bias in all lanes.  The arrays may lie at any float.
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef f32x2 f32x2u __attribute__((aligned(4)));
struct FeatState {
    f32x2 pe, me, ve, pd, md, vd;
    float pb, mb, vb;
};
__device__ __forceinline__ FeatState feature_load(const FeatArgs& a, int f, int lane) {
    const size_t e = (size_t)f * DH + 2 * lane, nw = (size_t)a.n_feat * DH, b = nw + f, d = nw + a.n_feat + e;
    FeatState s;
    s.pe = *(const f32x2u*)(a.w_enc + e);
    s.me = *(const f32x2u*)(a.m + e);
    s.ve = *(const f32x2u*)(a.v + e);
    s.pd = *(const f32x2u*)(a.w_dec + e);
    s.md = *(const f32x2u*)(a.m + d);
    s.vd = *(const f32x2u*)(a.v + d);
    s.pb = a.b_enc[f];
    s.mb = a.m[b];
    s.vb = a.v[b];
    return s;
}
__device__ __forceinline__ void adam2(const AdamArgs& a, float gx, float gy, f32x2& p, f32x2& m, f32x2& v) {
    float px = p[0], mx = m[0], vx = v[0], py = p[1], my = m[1], vy = v[1];
    adam(a, gx, px, mx, vx);
    adam(a, gy, py, my, vy);
    p = f32x2{px, py};
    m = f32x2{mx, my};
    v = f32x2{vx, vy};
}
__device__ __forceinline__ void feature_store(const FeatArgs& a, int f, int lane, const FeatSums& r) {
    FeatState s = feature_load(a, f, lane);
    const size_t e = (size_t)f * DH + 2 * lane, nw = (size_t)a.n_feat * DH, b = nw + f, d = nw + a.n_feat + e;
    if (a.grads) {
        *(f32x2u*)(a.grads + e) = f32x2{r.ex, r.ey};
        *(f32x2u*)(a.grads + d) = f32x2{r.dx, r.dy};
        if (lane == 0) a.grads[b] = r.sb;
    }
    adam2(a.adam, r.ex, r.ey, s.pe, s.me, s.ve);
    adam2(a.adam, r.dx, r.dy, s.pd, s.md, s.vd);
    adam(a.adam, r.sb, s.pb, s.mb, s.vb);
    *(f32x2u*)(a.w_enc + e) = s.pe;
    *(f32x2u*)(a.m + e) = s.me;
    *(f32x2u*)(a.v + e) = s.ve;
    *(f32x2u*)(a.w_dec + e) = s.pd;
    *(f32x2u*)(a.m + d) = s.md;
    *(f32x2u*)(a.v + d) = s.vd;
    if (lane == 0) { a.b_enc[f] = s.pb; a.m[b] = s.mb; a.v[b] = s.vb; }
}
template <int W>                             // wavefronts per workgroup
__global__ __launch_bounds__(W * 64) void tr_feature_kernel(FeatArgs a) {
    __shared__ float4 part[W][64];
    __shared__ float part_b[W];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((int)blockIdx.x >= a.n_long) {
        const int f = ((int)blockIdx.x - a.n_long) * W + wv;
        if (f >= a.n_feat) return;
        const int beg = a.offsets[f], end = a.offsets[f + 1];
        if (end - beg <= a.long_list) feature_store(a, f, lane, feature_sums(a, beg, end, lane));
        return;
    }
    const int f0 = blockIdx.x * a.per, fn = min(a.per, a.n_feat - f0);
    const int at = f0 + min(lane, fn - 1);
    const int my_beg = a.offsets[at], my_end = a.offsets[at + 1];
    for (unsigned long long todo = __ballot(lane < fn && my_end - my_beg > a.long_list); todo; todo &= todo - 1) {
        const int i = (int)__builtin_ctzll(todo);          // the same in every wavefront
        const int beg = __builtin_amdgcn_readlane(my_beg, i), end = __builtin_amdgcn_readlane(my_end, i);
        const int per = ((end - beg + W - 1) / W + kRows - 1) & ~(kRows - 1);
        const FeatSums r = feature_sums(a, min(beg + wv * per, end), min(beg + (wv + 1) * per, end), lane);
        part[wv][lane] = make_float4(r.ex, r.ey, r.dx, r.dy);
        if (lane == 0) part_b[wv] = r.sb;
        __syncthreads();
        if (wv == 0) {
            FeatSums t = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const float4 p = part[w][lane];
                t.ex += p.x;
                t.ey += p.y;
                t.dx += p.z;
                t.dy += p.w;
                t.sb += part_b[w];
            }
            feature_store(a, f0 + i, lane, t);
        }
        __syncthreads();
    }
}

// Step 6, first half: column sums of g - du and the loss parts of one chunk of tokens, rows in order.
constexpr int kColRows = 16;
__global__ __launch_bounds__(DH) void tr_colpart_kernel(const float* g, const float* du, const double* lossp, int B,
                                                        float* colpart, double* losspart) {
    const int c = threadIdx.x, t0 = blockIdx.x * kChunk, t1 = min(B, t0 + kChunk);
    float s = 0.f;
    double l = 0.0;
    for (int ta = t0; ta < t1; ta += kColRows) {          // 11 us with one row in flight, 4.7 with sixteen
        float gv[kColRows], dv[kColRows];
        double lv[kColRows];
#pragma unroll
        for (int j = 0; j < kColRows; ++j) {
            const size_t t = min(ta + j, t1 - 1);
            gv[j] = g[t * DH + c];
            dv[j] = du[t * DH + c];
            lv[j] = lossp[t];
        }
#pragma unroll
        for (int j = 0; j < kColRows; ++j) {
            s += ta + j < t1 ? gv[j] - dv[j] : 0.f;
            l += ta + j < t1 ? lv[j] : 0.0;
        }
    }
    colpart[(size_t)blockIdx.x * DH + c] = s;
    if (c == 0) losspart[blockIdx.x] = l;
}
// second half: the chunks in order (32 loads in flight; the loss parts are summed by a wavefront of their own), and Adam on b_dec
constexpr int kFinRows = 32;
__global__ __launch_bounds__(2 * DH) void tr_colfin_kernel(const float* __restrict__ colpart, const double* __restrict__ losspart,
                                                           int nchunk, double inv_n, float* g_b_dec, float* b_dec, float* m, float* v,
                                                           AdamArgs ad, float* loss_out) {
    const int c = threadIdx.x;
    if (c < DH) {
        float s = 0.f, pc = b_dec[c], mc = m[c], vc = v[c];
        for (int q0 = 0; q0 < nchunk; q0 += kFinRows) {
            float x[kFinRows];
#pragma unroll
            for (int j = 0; j < kFinRows; ++j) x[j] = colpart[(size_t)min(q0 + j, nchunk - 1) * DH + c];
#pragma unroll
            for (int j = 0; j < kFinRows; ++j) s += q0 + j < nchunk ? x[j] : 0.f;
        }
        if (g_b_dec) g_b_dec[c] = s;
        adam(ad, s, pc, mc, vc);
        b_dec[c] = pc;
        m[c] = mc;
        v[c] = vc;
    } else if (c == DH) {
        double l = 0.0;
        for (int q0 = 0; q0 < nchunk; q0 += kFinRows) {
            double x[kFinRows];
#pragma unroll
            for (int j = 0; j < kFinRows; ++j) x[j] = losspart[min(q0 + j, nchunk - 1)];
#pragma unroll
            for (int j = 0; j < kFinRows; ++j) l += q0 + j < nchunk ? x[j] : 0.0;
        }
        loss_out[0] = (float)(l * inv_n);
    }
}

struct Layout {
    size_t u_bf, w_bf, ids, vals, ews, g, dz, du, lossp, offsets, slots, colpart, losspart, iws, total, iws_bytes, ews_bytes;
};

Layout layout(int B, int n_feat, int k) {
    Layout L;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += s3_align(bytes); return at; };
    const int nchunk = (B + kChunk - 1) / kChunk;
    L.u_bf = take((size_t)B * DH * 2);
    L.w_bf = take((size_t)n_feat * DH * 2);
    L.ids = take((size_t)B * k * 4);
    L.vals = take((size_t)B * k * 4);
    L.ews_bytes = s3_sae_encode_topk_workspace(S3_BF16, B, DH, n_feat, k, 1);
    L.ews = take(L.ews_bytes);
    L.g = take((size_t)B * DH * 4);
    L.dz = take((size_t)B * k * 4);
    L.du = take((size_t)B * DH * 4);
    L.lossp = take((size_t)B * 8);
    L.offsets = take((size_t)(n_feat + 1) * 4);
    L.slots = take((size_t)B * k * 4);
    L.colpart = take((size_t)nchunk * DH * 4);
    L.losspart = take((size_t)nchunk * 8);
    L.iws_bytes = s3_index_build_workspace(B * k, 1, n_feat);
    L.iws = take(L.iws_bytes);
    L.total = o;
    return L;
}

bool shape_ok(int B, int d_head, int n_feat, int k) {
    return d_head == DH && B >= 1 && k >= 1 && k <= n_feat && (int64_t)B * k <= (1 << 24) &&
           s3_encode_fast_ok(S3_BF16, d_head, n_feat, k) && n_feat <= S3_MAX_FEAT;
}

}  // namespace

extern "C" {

size_t s3_sae_train_workspace(int B, int d_head, int n_feat, int k) {
    if (!shape_ok(B, d_head, n_feat, k)) return 0;
    return layout(B, n_feat, k).total;
}

int s3_sae_train_step(const float* x, int B, int d_head, int n_feat, int k, float* w_enc, float* b_enc, float* w_dec,
                      float* b_dec, float* adam_m, float* adam_v, float lr, float beta1, float beta2, float eps,
                      int step, float* loss_out, int32_t* ids_out, float* grads_out, void* ws, size_t ws_bytes,
                      void* stream) {
    if (!shape_ok(B, d_head, n_feat, k))
        return s3_fail(S3_EINVAL, "s3_sae_train_step: B %d, d_head %d, n_feat %d, k %d not supported (d_head 128, "
                       "n_feat a multiple of 128, k <= 128, B * k <= 2^24)", B, d_head, n_feat, k);
    if (!x || !w_enc || !b_enc || !w_dec || !b_dec || !adam_m || !adam_v || !loss_out || !ws)
        return s3_fail(S3_EINVAL, "s3_sae_train_step: null pointer");
    if (step < 1 || !(lr >= 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return s3_fail(S3_EINVAL, "s3_sae_train_step: step %d, lr %g, beta1 %g, beta2 %g, eps %g out of range", step,
                       (double)lr, (double)beta1, (double)beta2, (double)eps);
    const Layout L = layout(B, n_feat, k);
    if (ws_bytes < L.total) return s3_fail(S3_ECAPACITY, "s3_sae_train_step: workspace %zu < %zu bytes", ws_bytes, L.total);
    if ((uintptr_t)ws & 255) return s3_fail(S3_EINVAL, "s3_sae_train_step: workspace must be 256-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    char* base = (char*)ws;
    uint16_t* u_bf = (uint16_t*)(base + L.u_bf);
    uint16_t* w_bf = (uint16_t*)(base + L.w_bf);
    int32_t* ids = ids_out ? ids_out : (int32_t*)(base + L.ids);
    float* vals = (float*)(base + L.vals);
    float* g = (float*)(base + L.g);
    float* dz = (float*)(base + L.dz);
    float* du = (float*)(base + L.du);
    double* lossp = (double*)(base + L.lossp);
    int32_t* offsets = (int32_t*)(base + L.offsets);
    int32_t* slots = (int32_t*)(base + L.slots);
    float* colpart = (float*)(base + L.colpart);
    double* losspart = (double*)(base + L.losspart);
    const int64_t n_x = (int64_t)B * DH, n_w = (int64_t)n_feat * DH;
    const int64_t n_max = n_x > n_w ? n_x : n_w;

    hipLaunchKernelGGL(tr_prep_kernel, dim3((unsigned)((n_max + 255) / 256)), dim3(256), 0, st, x, (const float*)b_dec,
                       (const float*)w_enc, u_bf, w_bf, n_x, n_w);
    // one head and a few thousand tokens are too few token tiles for the chip: the encoder splits the features in that scratch
    int rc = s3_sae_encode_topk_ws(u_bf, S3_BF16, B, DH, w_bf, b_enc, n_feat, k, 1, ids, vals, base + L.ews, L.ews_bytes, stream);
    if (rc) return rc;
    TokArgs ta{x, w_dec, b_dec, w_bf, ids, vals, g, dz, du, lossp, B, k, 2.0f / ((float)B * (float)DH)};
    hipLaunchKernelGGL(tr_token_kernel, dim3((unsigned)((B + 3) / 4)), dim3(kTokThreads), 0, st, ta);
    rc = s3_index_build(ids, nullptr, B * k, 1, n_feat, offsets, slots, base + L.iws, L.iws_bytes, stream);
    if (rc) return rc;
    const AdamArgs ad{lr, beta1, beta2, eps, (float)(1.0 - pow((double)beta1, (double)step)), (float)(1.0 - pow((double)beta2, (double)step))};
    const bool few = n_feat < kFewFeat;
    const int per = few ? 1 : kLongPer;
    const int line = few && (B > kLongList || (int64_t)B * k >= 16 * (int64_t)n_feat) ? kLongListFew : kLongList;
    FeatArgs fa{offsets, slots, vals, dz, g, u_bf, grads_out, w_enc, b_enc, w_dec, adam_m, adam_v, ad, n_feat, k,
                k > 1 ? (uint32_t)(((1ull << 32) + (uint32_t)k - 1) / (uint32_t)k) : 0u,
                B > line ? (n_feat + per - 1) / per : 0, per, line};
    const int waves = few ? 16 : 8;
    hipLaunchKernelGGL(few ? tr_feature_kernel<16> : tr_feature_kernel<8>, dim3((unsigned)(fa.n_long + (n_feat + waves - 1) / waves)), dim3(waves * 64), 0, st, fa);
    const int nchunk = (B + kChunk - 1) / kChunk;
    hipLaunchKernelGGL(tr_colpart_kernel, dim3((unsigned)nchunk), dim3(DH), 0, st, (const float*)g, (const float*)du,
                       (const double*)lossp, B, colpart, losspart);
    const int64_t at_b = 2 * n_w + n_feat;               // of b_dec among all parameters
    hipLaunchKernelGGL(tr_colfin_kernel, dim3(1), dim3(2 * DH), 0, st, (const float*)colpart, (const double*)losspart, nchunk,
                       1.0 / ((double)B * DH), grads_out ? grads_out + at_b : nullptr, b_dec, adam_m + at_b, adam_v + at_b, ad, loss_out);
    S3_HIP(hipGetLastError());
    return S3_OK;
}

}  // extern "C"
