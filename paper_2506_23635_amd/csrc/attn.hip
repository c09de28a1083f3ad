// attn.hip -- kernels of the self-attention block of include/attn.h for a few
// new tokens (T <= 16: decode), in launch order:
//
//   norm_kernel     layer norm for more than 4 tokens, one workgroup per
//                   token (one pass, fp64 sums, fixed reduction order),
//                   h = bf16((x - mean) rstd gamma); up to 4 tokens the
//                   projection forms h itself
//   qkv_kernel      q|k|v = h Wqkv, and in its epilogue the rotary encoding
//                   of the query and key heads (angles reduced in fp64,
//                   rotation in fp32): bf16 q to the workspace, bf16 k and v
//                   appended to the cache
//   score_kernel    up to 16 query rows per key/value head and 1024 positions:
//                   attention of every query head of one key/value head over
//                   one chunk of 64 positions (4 waves): scores on the matrix
//                   cores, the chunk's softmax maximum and sum, and the
//                   unnormalised weighted sum of v
//   combine_kernel  merges the chunks of each (token, head) into bf16 a
//   flash_kernel    otherwise: attention on the matrix cores, the rows of a
//                   key/value head's whole group together, over one or
//                   several position ranges
//   merge_kernel    merges the ranges into bf16 a
//   gemv_kernel     o = a Wo (fp32) and y = bf16(x + o)
//
// Above 16 new tokens (prefill) the block is: norm_kernel -> q|k|v on the
// grouped GEMM of moe_prefill.hip, rotation and cache append in its end
// -> flash_kernel (and merge_kernel or merge_few_kernel) -> o = a Wo on the
// grouped GEMM, the residual in its end.  Where those reductions are split,
// rope_kernel and residual_kernel add the parts and do the ends' work.
//
// The GEMVs stream the fragment-tiled weights (the layout of moe_common.h)
// through v_mfma_f32_16x16x32_bf16 with the tokens as the B operand, as the
// MoE decode GEMVs do: one workgroup per 16 output features (or 32, see
// two_tiles), its 8 waves splitting K (wave w takes K tiles w, w + 8, ...), wave 0 adding the
// partial fragments in wave order.
#include <algorithm>
#include <cmath>

#include "moe_common.h"

namespace attn {

using moe::f32x4_t;
using moe::u32x4_t;
using moe::kTileK;
using moe::kTileBytes;
using moe::kTileRows;

constexpr int kSplit = 8;          // waves per GEMV workgroup (K split)
constexpr int kUnroll = 8;         // K tiles per wave and batch, tokens from LDS
// K tiles per wave and batch, tokens from memory: their fragments are loaded
// a batch ahead too, and with eight tiles both buffers would not leave two
// workgroups per CU their registers
constexpr int kUnrollX = 4;
constexpr int kChunk = 64;         // positions per score_kernel workgroup
constexpr int kPartPad = 4;        // m, l and padding after the hd sums of a partial

__device__ inline u32x4_t ld16_nt(const void* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
}

__device__ inline u32x4_t ld16(const void* p) { return *reinterpret_cast<const u32x4_t*>(p); }

// A projection's reduction with the tokens in memory: kUnrollX K tiles per
// wave and batch, weights and token fragments in two buffers in turn, the next
// batch's loads issued before this batch's MFMAs,
// so that both stay in flight while it is multiplied.  (With the token
// fragments loaded in their own batch every batch waited one cache latency
// for them: with this and the epilogues' loads and rotations ahead of the
// stream, the DBRX block at one token after 2047 positions 43.7 -> 42.2 us, at
// 16 tokens after 100 66.8 -> 64.8; three tiles per batch 41.9 and 64.0, but
// 24.6 against 23.8 at d 2048; six 42.3 and 66.8.)  The loads have no branches (an unused column reads token
// 0's row and feeds zeros), so a wait for them is not a wait for everything.
// The remainder is a shorter batch (tile after tile, every one waited for its
// loads, and a reduction shorter than a batch formed its rotations before any
// load: 32 heads of 128 without groups, 5 tokens, d 768 26.8 -> 25.2 us, d 1536
// 28.7 -> 26.4).
// kS row tiles, `slab` bytes apart, share each token fragment.
// `meanwhile` runs once while the first loads are in flight.
template <int kS, class F>
__device__ __forceinline__ void stream_batches(const uint8_t* pw, int64_t slab, const uint16_t* px, int KT,
                                               int w, bool has_tok, f32x4_t (&acc)[kS], F&& meanwhile)
{
    constexpr int kStep = kSplit * kUnrollX;
    const int nb = KT / kStep;
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    auto load = [&](int b, u32x4_t* wt, u32x4_t* xv) {
#pragma unroll
        for (int u = 0; u < kUnrollX; ++u) xv[u] = ld16(px + (b * kStep + w + kSplit * u) * kTileK);
#pragma unroll
        for (int u = 0; u < kUnrollX; ++u)
#pragma unroll
            for (int c = 0; c < kS; ++c)
                wt[u * kS + c] = ld16_nt(pw + c * slab + (int64_t)(b * kStep + w + kSplit * u) * kTileBytes);
    };
    auto mfmas = [&](const u32x4_t* wt, const u32x4_t* xv) {
#pragma unroll
        for (int u = 0; u < kUnrollX; ++u)
#pragma unroll
            for (int c = 0; c < kS; ++c)
                acc[c] = moe::mfma16x16x32(wt[u * kS + c], has_tok ? xv[u] : zero, acc[c]);
    };
    // the K tiles past the last full batch (K is a multiple of 256, so every
    // wave has as many)
    const int n_rest = (KT - nb * kStep) / kSplit;
    auto rest = [&](u32x4_t* wt, u32x4_t* xv) {
#pragma unroll
        for (int u = 0; u + 1 < kUnrollX; ++u)
            if (u < n_rest) {
                xv[u] = ld16(px + (nb * kStep + w + kSplit * u) * kTileK);
#pragma unroll
                for (int c = 0; c < kS; ++c)
                    wt[u * kS + c] = ld16_nt(pw + c * slab + (int64_t)(nb * kStep + w + kSplit * u) * kTileBytes);
            }
    };
    auto rest_mfmas = [&](const u32x4_t* wt, const u32x4_t* xv) {
#pragma unroll
        for (int u = 0; u + 1 < kUnrollX; ++u)
            if (u < n_rest) {
#pragma unroll
                for (int c = 0; c < kS; ++c)
                    acc[c] = moe::mfma16x16x32(wt[u * kS + c], has_tok ? xv[u] : zero, acc[c]);
            }
    };
    u32x4_t wa[kUnrollX * kS], wb[kUnrollX * kS], xa[kUnrollX], xb[kUnrollX];
    if (nb == 0) {
        rest(wa, xa);
        meanwhile();
        rest_mfmas(wa, xa);
        return;
    }
    load(0, wa, xa);
    meanwhile();
    int b = 0;
    for (; b + 2 < nb; b += 2) {
        load(b + 1, wb, xb);
        mfmas(wa, xa);
        load(b + 2, wa, xa);
        mfmas(wb, xb);
    }
    if (b + 1 < nb) {
        load(b + 1, wb, xb);
        mfmas(wa, xa);
        rest(wa, xa);
        mfmas(wb, xb);
        rest_mfmas(wa, xa);
    } else {
        rest(wb, xb);
        mfmas(wa, xa);
        rest_mfmas(wb, xb);
    }
}

// The output projection, o = a Wo (fp32) and y = bf16(x + o), one
// workgroup per kS tiles of 16 output features (two_tiles).
struct GemvArgs {
    const uint8_t* w;      // packed weights: N/16 row tiles of K/32 tiles
    const uint16_t* x;     // [T][K] bf16
    float* y32;            // [T][N] fp32
    const uint16_t* res;   // residual [T][N] bf16
    uint16_t* y16;         // bf16(res + y) [T][N]
    int K, N, T;
};

template <int kS>
__global__ __launch_bounds__(64 * kSplit) void gemv_kernel(GemvArgs a)
{
    __shared__ f32x4_t s_red[kS][kSplit * 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int q = blockIdx.x * kS;             // row tiles q .. q + kS - 1
    const int j = lane & 15, g = lane >> 4;    // token column, K group of 8
    const int KT = a.K / kTileK;
    const int64_t slab = (int64_t)KT * kTileBytes;
    const uint8_t* pw = a.w + moe::tile_offset(q, 0, KT) + lane * 16;
    const bool has_tok = j < a.T;
    const uint16_t* px = a.x + (has_tok ? (int64_t)j * a.K : 0) + g * 8;
    f32x4_t acc[kS] = {};
    // wave c < kS ends row tile q + c.  The residual of its lanes' outputs,
    // loaded ahead of the weights (output features 16 (q + c) + 4g .. +3 of
    // token j; other lanes read token 0's)
    const int c = min(w, kS - 1);
    const int64_t o = (int64_t)(has_tok ? j : 0) * a.N + (q + c) * kTileRows + g * 4;
    const uint2 r = *reinterpret_cast<const uint2*>(a.res + o);
    stream_batches<kS>(pw, slab, px, KT, w, has_tok, acc, [] {});
#pragma unroll
    for (int i = 0; i < kS; ++i) s_red[i][w * 64 + lane] = acc[i];
    __syncthreads();
    if (w >= kS) return;
    f32x4_t sum = s_red[c][lane];
    for (int i = 1; i < kSplit; ++i) sum += s_red[c][i * 64 + lane];
    if (!has_tok) return;
    *reinterpret_cast<float4*>(a.y32 + o) = make_float4(sum[0], sum[1], sum[2], sum[3]);
    const float r0 = __uint_as_float(r.x << 16), r1 = __uint_as_float(r.x & 0xFFFF0000u);
    const float r2 = __uint_as_float(r.y << 16), r3 = __uint_as_float(r.y & 0xFFFF0000u);
    const uint32_t lo = (uint32_t)moe::f32_to_bf16(r0 + sum[0]) |
                        ((uint32_t)moe::f32_to_bf16(r1 + sum[1]) << 16);
    const uint32_t hi = (uint32_t)moe::f32_to_bf16(r2 + sum[2]) |
                        ((uint32_t)moe::f32_to_bf16(r3 + sum[3]) << 16);
    *reinterpret_cast<uint2*>(a.y16 + o) = make_uint2(lo, hi);
}

// cos and sin of pos * inv_freq: the angle is formed and reduced modulo 2 pi
// in fp64 (2 pi split in two parts, Cody and Waite), so sincosf only sees an
// argument within [-pi, pi]
__device__ inline void rope_cs(int pos, double inv_freq, float& c, float& s)
{
    constexpr double kTwoPiHi = 6.28318530717958623200e+00;   // 2 pi rounded to fp64
    constexpr double kTwoPiLo = 2.44929359829470635445e-16;   // 2 pi - kTwoPiHi
    constexpr double kInvTwoPi = 1.59154943091895335769e-01;
    const double ang = (double)pos * inv_freq;
    const double k = rint(ang * kInvTwoPi);
    const double r = fma(-k, kTwoPiLo, fma(-k, kTwoPiHi, ang));
    sincosf((float)r, &s, &c);
}

// Layer norm, one workgroup of 256 threads per token: the thread's 8-element
// groups of x are loaded once into registers, x and x^2 summed in fp64 (so
// E[x^2] - mean^2 loses nothing), a butterfly per wave and the 4 wave sums in
// wave order, then h = bf16((x - mean) rstd gamma) from the registers.
constexpr int kNormThreads = 256;
constexpr int kNormGroups = 4;     // 8-element groups per thread (d <= 8192)

__global__ __launch_bounds__(kNormThreads) void norm_kernel(const uint16_t* __restrict__ x,
                                                            const float* __restrict__ gamma,
                                                            int d, float eps,
                                                            uint16_t* __restrict__ h,
                                                            const double* __restrict__ inv_freq,
                                                            float* __restrict__ cos_sin, int hd,
                                                            int pos0)
{
    __shared__ double red[2][kNormThreads / 64];
    const int t = blockIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint16_t* xr = x + (int64_t)t * d;
    u32x4_t v[kNormGroups];
    double sx = 0.0, sq = 0.0;
#pragma unroll
    for (int k = 0; k < kNormGroups; ++k) {
        const int e = threadIdx.x + k * kNormThreads;
        const u32x4_t zero = {0u, 0u, 0u, 0u};
        v[k] = e < d / 8 ? ld16(xr + e * 8) : zero;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double lo = __uint_as_float(v[k][i] << 16);
            const double hi = __uint_as_float(v[k][i] & 0xFFFF0000u);
            sx += lo + hi;
            sq = fma(lo, lo, fma(hi, hi, sq));
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        sx += __shfl_xor(sx, off, 64);
        sq += __shfl_xor(sq, off, 64);
    }
    if (lane == 0) { red[0][w] = sx; red[1][w] = sq; }
    __syncthreads();
    const double m1 = ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
    const double m2 = ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];
    const double mean = m1 / d;
    const float rstd = (float)(1.0 / sqrt(fmax(m2 / d - mean * mean, 0.0) + (double)eps));
    const float mu = (float)mean;
#pragma unroll
    for (int k = 0; k < kNormGroups; ++k) {
        const int e = threadIdx.x + k * kNormThreads;
        if (e >= d / 8) break;
        const float4 g0 = *reinterpret_cast<const float4*>(gamma + e * 8);
        const float4 g1 = *reinterpret_cast<const float4*>(gamma + e * 8 + 4);
        const float gm[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        u32x4_t out;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float lo = (__uint_as_float(v[k][i] << 16) - mu) * rstd * gm[2 * i];
            const float hi = (__uint_as_float(v[k][i] & 0xFFFF0000u) - mu) * rstd * gm[2 * i + 1];
            out[i] = (uint32_t)moe::f32_to_bf16(lo) | ((uint32_t)moe::f32_to_bf16(hi) << 16);
        }
        *reinterpret_cast<u32x4_t*>(h + (int64_t)t * d + e * 8) = out;
    }
    // prefill: the token's rotation, cos and sin of its position times every
    // frequency (formed once here instead of once per head)
    if (cos_sin && (int)threadIdx.x < hd / 2) {
        float c, s;
        rope_cs(pos0 + t, inv_freq[threadIdx.x], c, s);
        *reinterpret_cast<float2*>(cos_sin + ((int64_t)t * (hd / 2) + threadIdx.x) * 2) = make_float2(c, s);
    }
}

// The fused projection q|k|v = h Wqkv, one workgroup per 16 packed rows (8
// waves splitting K, as gemv_kernel).  The query and key heads are packed
// with rope_row, so in the epilogue lane (token j, group g), which holds
// rows 4g..4g+3 of the tile, and lane l ^ 32 hold the two members of four
// rotation pairs: the rotation (angle formed and reduced in fp64 from the
// layer's frequency table, sincosf, product in fp32) and the bf16 rounding
// happen there, q goes to the workspace and k, v to the cache at position
// pos0 + j; the unrotated fp32 values are kept for inspection.
struct QkvArgs {
    const uint8_t* w;      // packed Wqkv, query and key heads permuted by rope_row
    const uint16_t* h;     // [T][d] bf16, the normalised input (written here when the
                           // kernel normalises x itself)
    const uint16_t* x;     // [T][d] bf16 block input (normalising kernel only)
    const float* gamma;    // [d]
    float eps;
    const double* inv_freq;  // [hd/2]: theta^(-2f/hd)
    float* qkv;            // [T][nqkv] fp32, natural order, before rotation
    uint16_t* q;           // [T][H][hd]
    uint16_t* kc;          // this layer's K cache [G][max_seq][hd]
    uint16_t* vc;          // this layer's V cache
    int d, T, H, G, hd, max_seq, pos0;
};

// barrier for LDS traffic only: waits for this wave's LDS operations, not
// for its outstanding global loads (the weight batch in flight)
__device__ __forceinline__ void lds_barrier()
{
    constexpr int kWaitLgkm = 0xC07F;   // lgkmcnt 0; vmcnt and expcnt at their maxima
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitLgkm);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int kLnMaxT = 4;     // tokens up to which the projection normalises x itself
constexpr int kLnGroups = 2;   // 8-element groups per thread and token (d <= 8192)
constexpr int kHPad = 8;       // bf16 padding of a token row of h in LDS

// kNorm (T <= kLnMaxT): every workgroup forms the layer norm of the T tokens
// itself, into LDS, while its first weight batch is in flight -- x and gamma
// loaded first (thread i: 8-element groups i and i + 512), then the weights,
// then x and x^2 summed in fp64 (butterfly per wave, the 8 waves in order),
// h = bf16((x - mean) rstd gamma) to LDS (workgroup 0 also writes it out);
// the main loop then reads its B fragments from LDS.  Otherwise h comes from
// norm_kernel through global memory, and each fragment serves kS row tiles.
template <bool kNorm, int kS>
__global__ __launch_bounds__(64 * kSplit) void qkv_kernel(QkvArgs a)
{
    static_assert(kS == 1 || (kS == 2 && !kNorm && kSplit == 8));
    __shared__ f32x4_t s_red[kS][kSplit * 64];
    extern __shared__ __attribute__((aligned(16))) uint16_t hs[];   // kNorm: [T][d + kHPad]
    const int q = blockIdx.x * kS;             // row tiles q .. q + kS - 1
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = lane & 15, g = lane >> 4;
    const int KT = a.d / kTileK;
    const int hstride = a.d + kHPad;
    const int64_t slab = (int64_t)KT * kTileBytes;
    const uint8_t* pw = a.w + moe::tile_offset(q, 0, KT) + lane * 16;
    const bool has_tok = j < a.T;
    const uint16_t* px = a.h + (has_tok ? (int64_t)j * a.d : 0) + g * 8;
    const uint16_t* hx = hs + (has_tok ? j * hstride : 0) + g * 8;
    f32x4_t acc[kS] = {};
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    u32x4_t wv[kUnroll], xb[kUnroll];
    // wave c < kS ends row tile q + c.  The rotations that it applies are
    // formed while the first weights are in flight (in the epilogue they were
    // a chain of their own behind the stream): wave 4 c + e forms those of
    // the lanes' e-th pairs
    __shared__ float2 s_cs[kS][4][64];
    const int nqk_rows = (a.H + a.G) * a.hd;
    const int rc = min(w / 4, kS - 1), rrow = (q + rc) * kTileRows;
    const bool turn = rrow < nqk_rows && w < 4 * kS;
    const int fr = 8 * ((rrow % a.hd) / kTileRows) + 4 * (g & 1) + (w & 3);   // frequency of wave w's pair
    const double inv_fr = a.inv_freq[turn ? fr : 0];
    auto rotations = [&] {
        if (turn) {
            float c, sf;
            rope_cs(a.pos0 + j, inv_fr, c, sf);
            s_cs[rc][w & 3][lane] = make_float2(c, sf);
        }
    };
    if constexpr (kNorm) {
        __shared__ double red[2][kLnMaxT][kSplit];
        const int tid = threadIdx.x, ng = a.d / 8;
        u32x4_t xv[kLnMaxT][kLnGroups];
        float4 gv[kLnGroups][2];
        // unconditional loads (indices clamped, values masked after): no
        // branch between them and the weight batch, so the first use of x
        // waits for x alone
#pragma unroll
        for (int t = 0; t < kLnMaxT; ++t)
#pragma unroll
            for (int k = 0; k < kLnGroups; ++k) {
                const int e = tid + k * 64 * kSplit;
                const u32x4_t v = ld16(a.x + (int64_t)min(t, a.T - 1) * a.d + min(e, ng - 1) * 8);
                xv[t][k] = t < a.T && e < ng ? v : zero;
            }
#pragma unroll
        for (int k = 0; k < kLnGroups; ++k) {
            const int e = min(tid + k * 64 * kSplit, ng - 1);
            gv[k][0] = *reinterpret_cast<const float4*>(a.gamma + e * 8);
            gv[k][1] = *reinterpret_cast<const float4*>(a.gamma + e * 8 + 4);
        }
        // the first batch (tile indices clamped, so that the loads need no
        // branch; below 64 K tiles the values go unused)
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            wv[u] = ld16_nt(pw + (int64_t)min(w + kSplit * u, KT - 1) * kTileBytes);
        rotations();
#pragma unroll
        for (int t = 0; t < kLnMaxT; ++t) {
            if (t >= a.T) break;
            double sx = 0.0, sq = 0.0;
#pragma unroll
            for (int k = 0; k < kLnGroups; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const double lo = __uint_as_float(xv[t][k][i] << 16);
                    const double hi = __uint_as_float(xv[t][k][i] & 0xFFFF0000u);
                    sx += lo + hi;
                    sq = fma(lo, lo, fma(hi, hi, sq));
                }
            for (int off = 32; off >= 1; off >>= 1) {
                sx += __shfl_xor(sx, off, 64);
                sq += __shfl_xor(sq, off, 64);
            }
            if (lane == 0) { red[0][t][w] = sx; red[1][t][w] = sq; }
        }
        lds_barrier();
#pragma unroll
        for (int t = 0; t < kLnMaxT; ++t) {
            if (t >= a.T) break;
            double m1 = 0.0, m2 = 0.0;
#pragma unroll
            for (int i = 0; i < kSplit; ++i) { m1 += red[0][t][i]; m2 += red[1][t][i]; }
            const double mean = m1 / a.d;
            const float rstd = (float)(1.0 / sqrt(fmax(m2 / a.d - mean * mean, 0.0) + (double)a.eps));
            const float mu = (float)mean;
#pragma unroll
            for (int k = 0; k < kLnGroups; ++k) {
                const int e = tid + k * 64 * kSplit;
                if (e >= ng) break;
                const float gm[8] = {gv[k][0].x, gv[k][0].y, gv[k][0].z, gv[k][0].w,
                                     gv[k][1].x, gv[k][1].y, gv[k][1].z, gv[k][1].w};
                u32x4_t out;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float lo = (__uint_as_float(xv[t][k][i] << 16) - mu) * rstd * gm[2 * i];
                    const float hi = (__uint_as_float(xv[t][k][i] & 0xFFFF0000u) - mu) * rstd * gm[2 * i + 1];
                    out[i] = (uint32_t)moe::f32_to_bf16(lo) | ((uint32_t)moe::f32_to_bf16(hi) << 16);
                }
                *reinterpret_cast<u32x4_t*>(hs + t * hstride + e * 8) = out;
                if (q == 0) *reinterpret_cast<u32x4_t*>(const_cast<uint16_t*>(a.h) + (int64_t)t * a.d + e * 8) = out;
            }
        }
        lds_barrier();
    }
    if constexpr (!kNorm) {
        stream_batches<kS>(pw, slab, px, KT, w, has_tok, acc, rotations);
    } else {
        // two weight buffers in turn (the first batch was issued above, into
        // wv), tokens from LDS
        constexpr int kStep = kSplit * kUnroll;
        const int nb = KT / kStep;
        auto xload = [&](int k0, u32x4_t* xv) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int ko = (k0 + w + kSplit * u) * kTileK;
                xv[u] = has_tok ? *reinterpret_cast<const u32x4_t*>(hx + ko) : zero;
            }
        };
        auto wload = [&](int k0, u32x4_t* wt) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                wt[u] = ld16_nt(pw + (int64_t)(k0 + w + kSplit * u) * kTileBytes);
        };
        auto mfmas = [&](const u32x4_t* wt, const u32x4_t* xv) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) acc[0] = moe::mfma16x16x32(wt[u], xv[u], acc[0]);
        };
        if (nb > 0) {
            u32x4_t wb[kUnroll];
            int b = 0;
            for (; b + 2 < nb; b += 2) {
                xload(b * kStep, xb);
                wload((b + 1) * kStep, wb);
                mfmas(wv, xb);
                xload((b + 1) * kStep, xb);
                wload((b + 2) * kStep, wv);
                mfmas(wb, xb);
            }
            xload(b * kStep, xb);
            if (b + 1 < nb) {
                wload((b + 1) * kStep, wb);
                mfmas(wv, xb);
                xload((b + 1) * kStep, xb);
                mfmas(wb, xb);
            } else {
                mfmas(wv, xb);
            }
        }
        for (int kt = nb * kStep + w; kt < KT; kt += kSplit) {
            const u32x4_t xt = has_tok ? *reinterpret_cast<const u32x4_t*>(hx + kt * kTileK) : zero;
            acc[0] = moe::mfma16x16x32(ld16_nt(pw + (int64_t)kt * kTileBytes), xt, acc[0]);
        }
    }
#pragma unroll
    for (int i = 0; i < kS; ++i) s_red[i][w * 64 + lane] = acc[i];
    __syncthreads();
    if (w >= kS) return;
    f32x4_t sum = s_red[w][lane];
    for (int i = 1; i < kSplit; ++i) sum += s_red[w][i * 64 + lane];
    if (!has_tok) return;
    const int row0 = (q + w) * kTileRows;
    const int hd = a.hd, half = hd / 2;
    const int nqk = (a.H + a.G) * hd, nqkv = nqk + a.G * hd;
    const int pos = a.pos0 + j;
    float* qrow = a.qkv + (int64_t)j * nqkv;
    uint16_t* dst;
    float r[4];
    if (row0 < nqk) {
        const int head = row0 / hd, m = (row0 % hd) / kTileRows;
        const bool second = g >= 2;
        const int f0 = 8 * m + 4 * (g & 1);           // frequency index of sum[0]
        const int i0 = (second ? half : 0) + f0;       // feature index in the head
        *reinterpret_cast<float4*>(qrow + head * hd + i0) = make_float4(sum[0], sum[1], sum[2], sum[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float partner = __shfl_xor(sum[e], 32, 64);
            const float2 cs = s_cs[w][e][lane];
            r[e] = second ? sum[e] * cs.x + partner * cs.y : sum[e] * cs.x - partner * cs.y;
        }
        dst = head < a.H ? a.q + ((int64_t)j * a.H + head) * hd + i0
                         : a.kc + ((int64_t)(head - a.H) * a.max_seq + pos) * hd + i0;
    } else {
        const int n = row0 + 4 * g;                    // value features: natural order
        *reinterpret_cast<float4*>(qrow + n) = make_float4(sum[0], sum[1], sum[2], sum[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = sum[e];
        dst = a.vc + ((int64_t)((n - nqk) / hd) * a.max_seq + pos) * hd + (n - nqk) % hd;
    }
    const uint32_t lo = (uint32_t)moe::f32_to_bf16(r[0]) | ((uint32_t)moe::f32_to_bf16(r[1]) << 16);
    const uint32_t hi = (uint32_t)moe::f32_to_bf16(r[2]) | ((uint32_t)moe::f32_to_bf16(r[3]) << 16);
    *reinterpret_cast<uint2*>(dst) = make_uint2(lo, hi);
}

struct ScoreArgs {
    const uint16_t* q;     // [T][H][hd] bf16
    const uint16_t* kc;    // [G][max_seq][hd]
    const uint16_t* vc;
    float* part;           // [T][H][n_chunks][hd + kPartPad]: sum of p v, then m, l
    int T, H, G, max_seq, pos0, n_chunks;
    float scale;           // 1 / sqrt(hd)
};

// The attention of up to 16 query rows per key/value head over at most 1024
// positions (attn_short).  One workgroup of 4 waves per (key/value head g,
// chunk c of 64 positions); wave w owns positions 16 w .. 16 w + 15 of the
// chunk.  The query rows are every (token t, query head j of g), r = t * group
// + jj < 16; row r sees positions up to pos0 + t (causal).
//
// Scores on the matrix cores: v_mfma_f32_16x16x32_bf16 with the wave's 16
// positions x 32 dims of K as the A operand (lane l: position l%16, dims
// 8(l/16)..+7) and the q rows as B, so lane l ends with the scores of
// query row l%16 at positions 16 w + 4(l/16) + i (i = 0..3).  The chunk's
// maximum per row is the maximum of the four waves' (two butterfly steps in
// the wave, then LDS), exp(s - max) goes to LDS and the chunk's sum adds the
// waves' sums in wave order.  Then wave w sums P v over all 64 positions for
// dims w hd/4 .. (w+1) hd/4 - 1: lane l takes dims D(l%16)..+D-1 of that
// quarter at positions 4k + l/16 (V staged in LDS, rows padded so the four
// position groups hit distinct banks), two butterfly steps adding the four
// position groups in a fixed order.
template <int HD>
__global__ __launch_bounds__(256) void score_kernel(ScoreArgs a)
{
    constexpr int kPos = 64;           // positions per workgroup
    constexpr int kWaves = 4;          // 16 positions per wave
    constexpr int KS = HD / 32;        // MFMA K steps over the head
    constexpr int DQ = HD / kWaves;    // dims per wave in P v
    constexpr int D = DQ / 16;         // dims per lane in P v
    constexpr int VROW = HD + 32;      // padded V row (bf16)
    __shared__ __attribute__((aligned(16))) uint16_t vs[kPos * VROW];
    __shared__ float ps[16][kPos + 4];
    __shared__ float mx[kWaves][16], lx[kWaves][16];
    const int g = blockIdx.x, c = blockIdx.y;
    const int group = a.H / a.G;
    const int R = a.T * group;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p0 = c * kPos;
    const int n_pos = a.pos0 + a.T;
    const int last = min(kPos, n_pos - p0);          // live positions of the chunk
    const uint16_t* kbase = a.kc + (int64_t)g * a.max_seq * HD;
    const uint16_t* vbase = a.vc + (int64_t)g * a.max_seq * HD;
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    // K fragments of the wave's 16 positions (A operands), loaded once
    u32x4_t kf[KS];
    {
        const int p = w * 16 + (lane & 15);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            kf[ks] = p < last ? ld16(kbase + (int64_t)(p0 + p) * HD + ks * 32 + (lane >> 4) * 8)
                              : zero;
    }
    // V of the wave's 16 positions into LDS (16-byte pieces, coalesced)
    for (int e = lane; e < 16 * (HD / 8); e += 64) {
        const int p = w * 16 + e / (HD / 8), k8 = e % (HD / 8);
        *reinterpret_cast<u32x4_t*>(&vs[p * VROW + k8 * 8]) =
            p < last ? ld16(vbase + (int64_t)(p0 + p) * HD + k8 * 8) : zero;
    }
    const int dg = lane & 15, pq = lane >> 4;
    const bool row_ok = dg < R;                         // this lane's query row
    const int t_row = row_ok ? dg / group : 0;
    const int j_row = g * group + (row_ok ? dg % group : 0);
    const uint16_t* qrow = a.q + ((int64_t)t_row * a.H + j_row) * HD + pq * 8;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const u32x4_t qb = row_ok ? ld16(qrow + ks * 32) : zero;
        acc = moe::mfma16x16x32(kf[ks], qb, acc);
    }
    // scale, causal mask, the chunk's maximum per row
    const int lim = a.pos0 + t_row;
    float sv[4];
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int pos = p0 + w * 16 + pq * 4 + i;
        sv[i] = (row_ok && pos <= lim) ? acc[i] * a.scale : -INFINITY;
        m = fmaxf(m, sv[i]);
    }
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    if (lane < 16) mx[w][lane] = m;
    __syncthreads();
    m = fmaxf(fmaxf(mx[0][dg], mx[1][dg]), fmaxf(mx[2][dg], mx[3][dg]));
    float l = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float p = sv[i] == -INFINITY ? 0.f : expf(sv[i] - m);
        l += p;
        ps[dg][w * 16 + pq * 4 + i] = p;
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (lane < 16) lx[w][lane] = l;
    __syncthreads();
    // row statistics of the chunk: wave 0, lanes of the first position group
    if (w == 0 && pq == 0 && row_ok) {
        float* out = a.part + (((int64_t)t_row * a.H + j_row) * a.n_chunks + c) * (HD + kPartPad);
        out[HD] = m;
        out[HD + 1] = ((lx[0][dg] + lx[1][dg]) + lx[2][dg]) + lx[3][dg];
    }
    // P v for this wave's quarter of the dims, 8 rows at a time
    for (int r0 = 0; r0 < R; r0 += 8) {
        float o[8][D];
#pragma unroll
        for (int rr = 0; rr < 8; ++rr)
#pragma unroll
            for (int e = 0; e < D; ++e) o[rr][e] = 0.f;
#pragma unroll 4
        for (int k = 0; k < kPos / 4; ++k) {
            const int p = 4 * k + pq;
            const uint16_t* vr = &vs[p * VROW + w * DQ + dg * D];
            float vv[D];
            if constexpr (D == 2) {
                const uint32_t w2 = *reinterpret_cast<const uint32_t*>(vr);
                vv[0] = __uint_as_float(w2 << 16);
                vv[1] = __uint_as_float(w2 & 0xFFFF0000u);
            } else {
                vv[0] = __uint_as_float((uint32_t)vr[0] << 16);
            }
#pragma unroll
            for (int rr = 0; rr < 8; ++rr) {
                const float pw = ps[r0 + rr][p];
#pragma unroll
                for (int e = 0; e < D; ++e) o[rr][e] = fmaf(pw, vv[e], o[rr][e]);
            }
        }
#pragma unroll
        for (int rr = 0; rr < 8; ++rr)
#pragma unroll
            for (int e = 0; e < D; ++e) {
                float v = o[rr][e];
                v += __shfl_xor(v, 16, 64);
                v += __shfl_xor(v, 32, 64);
                o[rr][e] = v;
            }
        if (pq == 0) {
#pragma unroll
            for (int rr = 0; rr < 8; ++rr) {
                const int r = r0 + rr;
                if (r < R) {
                    const int t = r / group, j = g * group + r % group;
                    float* out = a.part + (((int64_t)t * a.H + j) * a.n_chunks + c) * (HD + kPartPad);
#pragma unroll
                    for (int e = 0; e < D; ++e) out[w * DQ + dg * D + e] = o[rr][e];
                }
            }
        }
    }
}

struct CombineArgs {
    const float* part;
    uint16_t* out;         // [T][H * hd] bf16
    int H, hd, pos0, n_chunks;
};

// (token t, head j) per workgroup, one thread per dimension: the chunks that
// hold positions of t, merged by their maxima in chunk order
__global__ __launch_bounds__(128) void combine_kernel(CombineArgs a)
{
    const int th = blockIdx.x, t = th / a.H;
    const int i = threadIdx.x;
    if (i >= a.hd) return;
    const int used = (a.pos0 + t) / kChunk + 1;
    const int stride = a.hd + kPartPad;
    const float* base = a.part + (int64_t)th * a.n_chunks * stride;
    float M = -INFINITY;
#pragma unroll 8
    for (int c = 0; c < used; ++c) M = fmaxf(M, base[(int64_t)c * stride + a.hd]);
    float L = 0.f, acc = 0.f;
#pragma unroll 8
    for (int c = 0; c < used; ++c) {
        const float* pc = base + (int64_t)c * stride;
        const float f = expf(pc[a.hd] - M);
        L = fmaf(pc[a.hd + 1], f, L);
        acc = fmaf(pc[i], f, acc);
    }
    a.out[(int64_t)th * a.hd + i] = moe::f32_to_bf16(acc / L);
}

// ---------------------------------------------------------------- prefill
// More than 16 new tokens: the projections run on the grouped GEMM of
// moe_prefill.hip (one "expert", its rows the tokens), then these kernels.

// rope_kernel, where the projection's reduction was split (otherwise its
// epilogue does this): the partial sums, [n_split][T][nqkv] fp32 in packed
// row order (query and key features placed by rope_row), added in order; the
// natural-order fp32 q|k|v (kept for inspection), q rotated to bf16 in the
// workspace, k rotated and v to the cache at position pos0 + t.  A thread
// takes four rotation pairs, or eight value features; a workgroup one token's
// share of blockDim.x such pieces.
struct RopeArgs {
    const float* qkvp;
    const float* cos_sin;  // [T][hd/2][2]
    float* qkv;            // [T][nqkv] fp32, natural order
    uint16_t* q;           // [T][H][hd]
    uint16_t* kc;
    uint16_t* vc;
    int T, H, G, hd, max_seq, pos0, n_split;
};

__device__ inline uint2 pack_bf16x4(float4 v)
{
    return make_uint2((uint32_t)moe::f32_to_bf16(v.x) | ((uint32_t)moe::f32_to_bf16(v.y) << 16),
                      (uint32_t)moe::f32_to_bf16(v.z) | ((uint32_t)moe::f32_to_bf16(v.w) << 16));
}

__global__ __launch_bounds__(256) void rope_kernel(RopeArgs a)
{
    const int t = blockIdx.x, hd = a.hd, half = hd / 2;
    const int nqk = (a.H + a.G) * hd, nqkv = nqk + a.G * hd;
    const int e = blockIdx.y * 256 + threadIdx.x;       // 8 consecutive packed features
    if (e >= nqkv / 8) return;
    const int64_t part = (int64_t)a.T * nqkv;
    const int64_t pos = a.pos0 + t;
    // packed features of a 16-row tile: 4 u .. + 3 and 8 + 4 u .. + 3 (u = e % 2)
    const float* src = a.qkvp + (int64_t)t * nqkv + e / 2 * 16 + e % 2 * 4;
    float4 x0 = *reinterpret_cast<const float4*>(src), x1 = *reinterpret_cast<const float4*>(src + 8);
    for (int k = 1; k < a.n_split; ++k) {
        const float4 p0 = *reinterpret_cast<const float4*>(src + k * part);
        const float4 p1 = *reinterpret_cast<const float4*>(src + k * part + 8);
        x0.x += p0.x; x0.y += p0.y; x0.z += p0.z; x0.w += p0.w;
        x1.x += p1.x; x1.y += p1.y; x1.z += p1.z; x1.w += p1.w;
    }
    float* nat = a.qkv + (int64_t)t * nqkv;
    const int n0 = e / 2 * 16;
    if (n0 < nqk) {
        const int head = n0 / hd, f0 = n0 % hd / 2 + e % 2 * 4;
        const float* cs = a.cos_sin + ((int64_t)t * half + f0) * 2;
        const float4 c01 = *reinterpret_cast<const float4*>(cs), c23 = *reinterpret_cast<const float4*>(cs + 4);
        const float4 r0 = make_float4(x0.x * c01.x - x1.x * c01.y, x0.y * c01.z - x1.y * c01.w,
                                      x0.z * c23.x - x1.z * c23.y, x0.w * c23.z - x1.w * c23.w);
        const float4 r1 = make_float4(x1.x * c01.x + x0.x * c01.y, x1.y * c01.z + x0.y * c01.w,
                                      x1.z * c23.x + x0.z * c23.y, x1.w * c23.z + x0.w * c23.w);
        *reinterpret_cast<float4*>(nat + head * hd + f0) = x0;
        *reinterpret_cast<float4*>(nat + head * hd + f0 + half) = x1;
        uint16_t* dst = (head < a.H ? a.q + ((int64_t)t * a.H + head) * hd
                                    : a.kc + ((int64_t)(head - a.H) * a.max_seq + pos) * hd) + f0;
        *reinterpret_cast<uint2*>(dst) = pack_bf16x4(r0);
        *reinterpret_cast<uint2*>(dst + half) = pack_bf16x4(r1);
    } else {
        const int n = n0 + e % 2 * 4;
        *reinterpret_cast<float4*>(nat + n) = x0;
        *reinterpret_cast<float4*>(nat + n + 8) = x1;
        uint16_t* dst = a.vc + ((int64_t)((n0 - nqk) / hd) * a.max_seq + pos) * hd + (n - nqk) % hd;
        *reinterpret_cast<uint2*>(dst) = pack_bf16x4(x0);
        *reinterpret_cast<uint2*>(dst + 8) = pack_bf16x4(x1);
    }
}

// flash_kernel: causal attention of T new tokens.  The query rows of one
// key/value head are the (token, query head of its group) pairs, r = t *
// group + jj; a workgroup of 4 waves takes a block of 128 or 64 of them
// (kPG = 1 or 2 position groups: the 4 / kPG waves of a group own 32 rows
// each) and one of n_split ranges of the positions they need.  Packing the group's
// heads into the rows reads K and V once for all of them and keeps a block's
// tokens, so the positions its causal mask wastes, few.
//
// Per step of kP positions K rows and V transposed (dims major) go to LDS,
// and each position group takes kP / kPG of them.  The scores are computed
// transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16 (A = 32 positions x
// 16 dims of K from LDS, B = the wave's query rows), so lane l ends with the
// scores of row l % 32 at positions 8 g + 4 (l / 32) + r of each 32-position
// block (register 4 g + r); the running maximum and sum per row (one
// exchange between the lane pair) rescale the output, and O^T += V^T P^T
// takes the P values straight from those registers as the B operand: the
// 16-position K step s of a block takes registers g = 2 s, 2 s + 1, i.e.
// positions 16 s + {4 h .. 4 h + 3, 8 + 4 h .. 8 + 4 h + 3} for h = l / 32,
// and the V^T operand is read from LDS in the same order.  P enters the
// matrix cores as kTerms bf16 terms (each the rounding of what the earlier
// ones left, which the subtraction gives exactly): three keep all 24 bits
// (few tokens), two keep 16 (prefill); V is bf16 and every product is exact
// in the fp32 accumulation.
//
// The position groups' sums are merged through LDS in group order.  With one
// range the result is written as bf16; with several, each writes its
// unnormalised sums, maximum (base 2) and sum of weights for merge_kernel: a
// few rows over a long context are split until about two workgroups per CU
// run (attn_split).
struct FlashArgs {
    const uint16_t* q;     // [T][H][HD] bf16, rotated
    const uint16_t* kc;    // this layer's K cache [G][max_seq][HD]
    const uint16_t* vc;
    uint16_t* out;         // a [T][H * HD] bf16
    float* part;           // n_split > 1: [T][H][n_split][HD + kPartPad]: sum of p v, then m, l
    int T, H, G, max_seq, pos0;
    int nrb;               // row blocks per key/value head
    int n_split;           // position ranges
    float scale2;          // 1/sqrt(head_dim) * log2(e): scores in base 2
};

constexpr int kXcds = 8;

__device__ inline uint32_t pack_bf16x2(float lo, float hi)
{
    return (uint32_t)moe::f32_to_bf16(lo) | ((uint32_t)moe::f32_to_bf16(hi) << 16);
}

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

__device__ inline f32x16_t mfma32x32x16(const u32x4_t a, const u32x4_t b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(moe::bf16x8_t, a),
                                                   __builtin_bit_cast(moe::bf16x8_t, b), c, 0, 0, 0);
}

// A maximum in base 2, with the product's one rounding everywhere: p, the
// rescaling and the merges then refer to the same value, and its rounding
// cancels (contracted into a difference it would not).
__device__ inline float base2(float m, float scale2)
{
#pragma clang fp contract(off)
    return m * scale2;
}

constexpr int flash_rows(int pg) { return 128 / pg; }        // query rows per workgroup
constexpr int kFlashP = 64;                                  // positions per step

// Two workgroups per CU: at most 256 registers per lane (the output block of
// 32 rows x 128 dims alone takes 64) and 70 KB of LDS, 2 waves per SIMD.  What
// bounds it is the alternation of MFMAs and vector work with two waves to
// overlap them; consecutive MFMAs on different accumulators and the scale
// folded into the exponent's multiply-add: 2048 tokens after 4000 positions
// 860 -> 825 us.
template <int HD, int kPG, int kTerms>
__global__ __launch_bounds__(256, 2) void flash_kernel(FlashArgs a)
{
    constexpr int KQ = HD / 16;              // 16-dim K steps of the score MFMAs
    constexpr int DB = HD / 32;              // 32-dim blocks of the output
    constexpr int kP = kFlashP;
    constexpr int NB = kP / 32 / kPG;        // 32-position blocks per wave and step
    constexpr int kRowWaves = 4 / kPG;       // waves on different rows
    constexpr int KROW = HD + 8;             // padded K row in LDS (bf16)
    // padded V^T row (positions, bf16): 34 words, so the 8-byte reads of
    // consecutive dims fall in distinct bank pairs (LDS bank conflicts 19.5 M
    // -> 6.5 M cycles per launch against 36 words)
    constexpr int VROW = kP + 4;
    constexpr int kQBytes = flash_rows(kPG) * KROW * 2;
    constexpr int kStageBytes = kP * KROW * 2 + HD * VROW * 2 + kQBytes;
    // merge of the position groups: per wave past the first group DB * 16
    // sums, the maximum and the weights' sum per lane
    constexpr int kMergeBytes = (4 - kRowWaves) * (DB * 16 + 2) * 64 * 4;
    __shared__ __attribute__((aligned(16))) uint8_t lds[kStageBytes > kMergeBytes ? kStageBytes : kMergeBytes];
    uint16_t* ks = reinterpret_cast<uint16_t*>(lds);
    uint32_t* vt32 = reinterpret_cast<uint32_t*>(lds + kP * KROW * 2);
    uint16_t* qs = reinterpret_cast<uint16_t*>(lds + kP * KROW * 2 + HD * VROW * 2);
    // XCD-aware numbering: hardware hands block b to XCD b % 8, and each XCD
    // takes a contiguous run of the logical order (key/value head, row block
    // from the last, position range), so the workgroups of one key/value
    // head share its K and V in one L2 (DBRX: one head per XCD) and on every
    // XCD the longest row blocks (the most positions) start first.  Logical
    // slots past the last block exit at once.
    const int group = a.H / a.G;
    const int per_xcd = gridDim.x / kXcds;
    const int logical = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    const int per_head = a.nrb * a.n_split;
    if (logical >= a.G * per_head) return;
    const int kvh = logical / per_head, rem = logical % per_head;
    const int rb = a.nrb - 1 - rem / a.n_split, split = rem % a.n_split;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 31, h = lane >> 5;
    const int pg = w / kRowWaves;                        // the wave's position group
    const int R = a.T * group;
    const int row_w0 = rb * flash_rows(kPG) + w % kRowWaves * 32;   // the wave's first row
    const int row = row_w0 + c;                          // this lane's row
    const bool wave_ok = row_w0 < R, row_ok = row < R;
    const int t = (row_ok ? row : 0) / group;            // its token and query head
    const int j = kvh * group + (row_ok ? row : 0) % group;
    const int lim = a.pos0 + t;                          // its last position
    const int lim_w0 = a.pos0 + row_w0 / group;          // the last position of the wave's first row
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    // the block's query rows in LDS, read again each step: in registers they
    // would leave none for the next step's K and V
    const uint16_t* qw = qs + (w % kRowWaves * 32 + c) * KROW + h * 8;
    if (pg == 0) {
        const uint16_t* qrow = a.q + ((int64_t)t * a.H + j) * HD + h * 8;
#pragma unroll
        for (int k = 0; k < KQ; ++k) {
            const u32x4_t v = ld16(qrow + k * 16);
            *reinterpret_cast<u32x4_t*>(const_cast<uint16_t*>(qw) + k * 16) = row_ok ? v : zero;
        }
    }
    f32x16_t o[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) o[b] = f32x16_t{};
    float m = -INFINITY, l = 0.f;
    const int t_last = (min((rb + 1) * flash_rows(kPG), R) - 1) / group;
    const int n_pos = a.pos0 + t_last + 1;               // positions the block needs
    const int n_steps = (n_pos + kP - 1) / kP;
    const int s_end = (int)((int64_t)n_steps * (split + 1) / a.n_split);
    const uint16_t* kbase = a.kc + (int64_t)kvh * a.max_seq * HD;
    const uint16_t* vbase = a.vc + (int64_t)kvh * a.max_seq * HD;
    // per step a thread stages KL 16-byte pieces of K rows and VL position
    // pairs of V; the next step's are loaded into registers while this one is
    // computed (barriers that wait for LDS only leave them in flight): DBRX
    // block, 2048 tokens after 4000 positions 757 -> 704 us, 512 after 8000 324
    // -> 322
    constexpr int KL = kP * (HD / 8) / 256;
    constexpr int VL = (kP / 2) * (HD / 8) / 256;
    static_assert(KL * 256 == kP * (HD / 8) && VL * 256 == (kP / 2) * (HD / 8),
                  "the staging pieces divide evenly over the 256 threads");
    u32x4_t kv[KL], va[VL], vb[VL];
    auto fetch = [&](int st) {
        const int p0 = st * kP, live = min(kP, n_pos - p0);
#pragma unroll
        for (int i = 0; i < KL; ++i) {
            const int e = threadIdx.x + i * 256;
            const int p = e / (HD / 8), k8 = e % (HD / 8);
            kv[i] = ld16(kbase + (int64_t)(p0 + min(p, live - 1)) * HD + k8 * 8);
        }
#pragma unroll
        for (int i = 0; i < VL; ++i) {
            const int e = threadIdx.x + i * 256;
            const int pp = e % (kP / 2), k8 = e / (kP / 2);
            va[i] = ld16(vbase + (int64_t)(p0 + min(2 * pp, live - 1)) * HD + k8 * 8);
            vb[i] = ld16(vbase + (int64_t)(p0 + min(2 * pp + 1, live - 1)) * HD + k8 * 8);
        }
    };
    int st = (int)((int64_t)n_steps * split / a.n_split);
    if (st < s_end) fetch(st);
    for (; st < s_end; ++st) {
        const int p0 = st * kP;
        lds_barrier();                                   // the last step's LDS reads are done
        // K rows: 16-byte pieces, coalesced.  Rows past `live` repeat the
        // last live row (the loads are clamped): every row's causal mask
        // removes those positions, so their scores never count and their
        // probabilities are exactly 0 against finite V rows.
#pragma unroll
        for (int i = 0; i < KL; ++i) {
            const int e = threadIdx.x + i * 256;
            const int p = e / (HD / 8), k8 = e % (HD / 8);
            *reinterpret_cast<u32x4_t*>(&ks[p * KROW + k8 * 8]) = kv[i];
        }
        // V transposed: a thread takes positions 2 pp, 2 pp + 1 at 8 dims and
        // writes 8 words of (position pair) per dim, each one byte permute
        // (low halves of the two words, then the high halves)
#pragma unroll
        for (int i = 0; i < VL; ++i) {
            const int e = threadIdx.x + i * 256;
            const int pp = e % (kP / 2), k8 = e / (kP / 2);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                vt32[((k8 * 8 + 2 * r) * VROW) / 2 + pp] = __builtin_amdgcn_perm(vb[i][r], va[i][r], 0x05040100u);
                vt32[((k8 * 8 + 2 * r + 1) * VROW) / 2 + pp] = __builtin_amdgcn_perm(vb[i][r], va[i][r], 0x07060302u);
            }
        }
        if (st + 1 < s_end) fetch(st + 1);
        lds_barrier();
        if (!wave_ok) continue;
        // S^T = K Q^T for the wave's 32-position blocks: lane (c, h) ends with
        // row c's scores at positions 32 pb + 8 g + 4 h + r (register 4 g + r)
        f32x16_t sc[NB];
#pragma unroll
        for (int pb = 0; pb < NB; ++pb) sc[pb] = f32x16_t{};
#pragma unroll
        for (int k = 0; k < KQ; ++k) {
            const u32x4_t qf = *reinterpret_cast<const u32x4_t*>(qw + k * 16);
#pragma unroll
            for (int pb = 0; pb < NB; ++pb) {
                const u32x4_t kf = *reinterpret_cast<const u32x4_t*>(
                    &ks[((pg * NB + pb) * 32 + c) * KROW + k * 16 + h * 8]);
                sc[pb] = mfma32x32x16(kf, qf, sc[pb]);
            }
        }
        // p = 2^((s - m) scale log2 e), one fused multiply-add and one exp per
        // score; the causal mask and the rows past R only on the steps that
        // need them
        // (wave-uniform: a step past the last position of the wave's first
        // row, or a wave with rows past R)
        const int pw0 = p0 + pg * NB * 32;               // the wave's first position
        float sv[NB * 16];
        float mx = -INFINITY;
        if (pw0 + NB * 32 - 1 > lim_w0 || row_w0 + 31 >= R) {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int pos = pw0 + pb * 32 + 8 * (i / 4) + 4 * h + (i % 4);
                    const float v = (row_ok && pos <= lim) ? sc[pb][i] : -INFINITY;
                    sv[pb * 16 + i] = v;
                    mx = fmaxf(mx, v);
                }
        } else {
#pragma unroll
            for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    sv[pb * 16 + i] = sc[pb][i];
                    mx = fmaxf(mx, sv[pb * 16 + i]);
                }
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mn = fmaxf(m, mx);
        // a row with every position masked so far keeps mn = -inf: subtract
        // 0 instead, so its p are 0, not NaN
        const float ms = base2(mn, a.scale2), msub = mn == -INFINITY ? 0.f : -ms;
        float ps = 0.f;
        float pv[NB * 16];
#pragma unroll
        for (int e = 0; e < NB * 16; ++e) {
            pv[e] = __builtin_amdgcn_exp2f(fmaf(sv[e], a.scale2, msub));
            ps += pv[e];
        }
        ps += __shfl_xor(ps, 32, 64);
        // rescale the running sums only where a maximum moved (m == mn gives
        // the factor 1 exactly, so skipping it changes no bit)
        if (__ballot(mn != m)) {
            const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(base2(m, a.scale2) - ms);
            l *= alpha;
#pragma unroll
            for (int b = 0; b < DB; ++b) o[b] *= alpha;
        }
        l += ps;
        m = mn;
        // O^T += V^T P^T, two 16-position K steps per block: step (pb, s)
        // takes the lane's registers 4 g + r for g = 2 s, 2 s + 1 of block
        // pb, i.e. positions 32 pb + 16 s + {4 h .. 4 h + 3, 8 + 4 h .. 8 + 4 h + 3},
        // and the V^T operand is read in the same order
#pragma unroll
        for (int pb = 0; pb < NB; ++pb)
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                float* pp = &pv[pb * 16 + sx * 8];
                u32x4_t bt[kTerms];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int q = 0; q < kTerms; ++q) {
                        const uint32_t hw = moe::cvt_pk_bf16(pp[2 * i], pp[2 * i + 1]);
                        bt[q][i] = hw;
                        pp[2 * i] -= __uint_as_float(hw << 16);
                        pp[2 * i + 1] -= __uint_as_float(hw & 0xFFFF0000u);
                    }
                // the terms outermost: consecutive MFMAs then add into different
                // output blocks instead of waiting for one another
                u32x4_t av[DB];
#pragma unroll
                for (int b = 0; b < DB; ++b) {
                    const uint32_t* vr = vt32 + ((b * 32 + c) * VROW + (pg * NB + pb) * 32 + sx * 16 + 4 * h) / 2;
                    const uint2 v0 = *reinterpret_cast<const uint2*>(vr);
                    const uint2 v1 = *reinterpret_cast<const uint2*>(vr + 4);
                    av[b] = u32x4_t{v0.x, v0.y, v1.x, v1.y};
                }
#pragma unroll
                for (int q = 0; q < kTerms; ++q)
#pragma unroll
                    for (int b = 0; b < DB; ++b) o[b] = mfma32x32x16(av[b], bt[q], o[b]);
            }
    }
    if constexpr (kPG > 1) {
        // the other position groups' sums, merged in group order by group 0
        float* mg = reinterpret_cast<float*>(lds);
        __syncthreads();
        if (pg > 0) {
            float* dst = mg + (w - kRowWaves) * (DB * 16 + 2) * 64 + lane;
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) dst[(b * 16 + i) * 64] = o[b][i];
            dst[DB * 16 * 64] = m;
            dst[(DB * 16 + 1) * 64] = l;
        }
        __syncthreads();
        if (pg > 0) return;
#pragma unroll
        for (int k = 1; k < kPG; ++k) {
            const float* src = mg + ((k - 1) * kRowWaves + w) * (DB * 16 + 2) * 64 + lane;
            const float m2 = src[DB * 16 * 64], l2 = src[(DB * 16 + 1) * 64];
            const float mn = fmaxf(m, m2);
            const float ms = base2(mn, a.scale2);
            const float f1 = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(base2(m, a.scale2) - ms);
            const float f2 = m2 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(base2(m2, a.scale2) - ms);
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    o[b][i] = fmaf(src[(b * 16 + i) * 64], f2, o[b][i] * f1);
            l = fmaf(l2, f2, l * f1);
            m = mn;
        }
    }
    if (!row_ok) return;
    // lane: dims 32 b + 8 g + 4 h + r of its row (register 4 g + r)
    if (a.n_split > 1) {
        float* dst = a.part + (((int64_t)t * a.H + j) * a.n_split + split) * (HD + kPartPad);
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4*>(dst + b * 32 + 8 * g + 4 * h) =
                    make_float4(o[b][4 * g], o[b][4 * g + 1], o[b][4 * g + 2], o[b][4 * g + 3]);
        if (h == 0) {
            dst[HD] = base2(m, a.scale2);
            dst[HD + 1] = l;
        }
        return;
    }
    // few tokens divide, as merge_kernel does.  (The bits still depend on the
    // number of ranges: each takes its own maximum, and their sums are added
    // in range order.)
    const float inv = 1.0f / l;
    auto norm = [&](float v) { return kTerms == 3 ? v / l : v * inv; };
    uint16_t* dst = a.out + ((int64_t)t * a.H + j) * HD + 4 * h;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<uint2*>(dst + b * 32 + 8 * g) =
                make_uint2(pack_bf16x2(norm(o[b][4 * g]), norm(o[b][4 * g + 1])),
                           pack_bf16x2(norm(o[b][4 * g + 2]), norm(o[b][4 * g + 3])));
}

// merge_kernel, one workgroup of 4 waves per (token, query head): the
// position ranges' sums merged by their maxima.  Thread s takes range s's
// maximum and weight (n_split <= 256); wave w adds the weighted sums of
// ranges w, w + 4, ... (two dims per lane at head_dim 128, one at 64), the
// four waves' sums are added in wave order.
struct MergeArgs {
    const float* part;
    uint16_t* out;         // [T][H * hd] bf16
    int n_split;
};

template <int HD>
__global__ __launch_bounds__(256) void merge_kernel(MergeArgs a)
{
    constexpr int D = HD / 64;
    __shared__ float fs[256], red[2][4], sums[4][HD];
    const int th = blockIdx.x, S = a.n_split;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const float* base = a.part + (int64_t)th * S * (HD + kPartPad);
    const float ms = tid < S ? base[(int64_t)tid * (HD + kPartPad) + HD] : -INFINITY;
    const float ls = tid < S ? base[(int64_t)tid * (HD + kPartPad) + HD + 1] : 0.f;
    float M = ms;
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
    if (lane == 0) red[0][w] = M;
    __syncthreads();
    M = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
    const float f = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - M);
    fs[tid] = f;
    float L = ls * f;
    for (int off = 32; off >= 1; off >>= 1) L += __shfl_xor(L, off, 64);
    if (lane == 0) red[1][w] = L;
    __syncthreads();
    L = ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];
    float acc[D];
#pragma unroll
    for (int e = 0; e < D; ++e) acc[e] = 0.f;
#pragma unroll 8
    for (int k = w; k < S; k += 4) {
        const float* pc = base + (int64_t)k * (HD + kPartPad) + lane * D;
        const float fk = fs[k];
        if constexpr (D == 2) {
            const float2 v = *reinterpret_cast<const float2*>(pc);
            acc[0] = fmaf(v.x, fk, acc[0]);
            acc[1] = fmaf(v.y, fk, acc[1]);
        } else {
            acc[0] = fmaf(pc[0], fk, acc[0]);
        }
    }
#pragma unroll
    for (int e = 0; e < D; ++e) sums[w][lane * D + e] = acc[e];
    __syncthreads();
    if (tid < HD) {
        const float v = ((sums[0][tid] + sums[1][tid]) + sums[2][tid]) + sums[3][tid];
        a.out[(int64_t)th * HD + tid] = moe::f32_to_bf16(v / L);
    }
}

// merge_few_kernel: the same for few ranges (n_split <= 64) and many rows,
// one wave per (token, query head): lane s takes range s's maximum and weight,
// then every lane adds its dims of the ranges in order.
template <int HD>
__global__ __launch_bounds__(256) void merge_few_kernel(MergeArgs a, int n)
{
    constexpr int D = HD / 64;
    const int th = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, S = a.n_split;
    if (th >= n) return;
    const float* base = a.part + (int64_t)th * S * (HD + kPartPad);
    const float ms = lane < S ? base[(int64_t)lane * (HD + kPartPad) + HD] : -INFINITY;
    const float ls = lane < S ? base[(int64_t)lane * (HD + kPartPad) + HD + 1] : 0.f;
    float M = ms;
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
    const float f = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - M);
    float L = ls * f;
    for (int off = 32; off >= 1; off >>= 1) L += __shfl_xor(L, off, 64);
    float acc[D];
#pragma unroll
    for (int e = 0; e < D; ++e) acc[e] = 0.f;
    for (int k = 0; k < S; ++k) {
        const float* pc = base + (int64_t)k * (HD + kPartPad) + lane * D;
        const float fk = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), k));
#pragma unroll
        for (int e = 0; e < D; ++e) acc[e] = fmaf(pc[e], fk, acc[e]);
    }
    uint16_t* dst = a.out + (int64_t)th * HD + lane * D;
    if constexpr (D == 2)
        *reinterpret_cast<uint32_t*>(dst) = pack_bf16x2(acc[0] / L, acc[1] / L);
    else
        dst[0] = moe::f32_to_bf16(acc[0] / L);
}

// Where the output projection's reduction was split: o = the partial sums
// [n_split][n] in order, and y = bf16(x + o); 8 elements per thread.
__global__ __launch_bounds__(256) void residual_kernel(const uint16_t* __restrict__ x,
                                                       const float* __restrict__ op, int n_split,
                                                       float* __restrict__ o, uint16_t* y, int64_t n8)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n8) return;
    const u32x4_t xv = ld16(x + i * 8);
    float4 o0 = *reinterpret_cast<const float4*>(op + i * 8);
    float4 o1 = *reinterpret_cast<const float4*>(op + i * 8 + 4);
    for (int k = 1; k < n_split; ++k) {
        const float* pk = op + (k * n8 + i) * 8;
        const float4 p0 = *reinterpret_cast<const float4*>(pk);
        const float4 p1 = *reinterpret_cast<const float4*>(pk + 4);
        o0.x += p0.x; o0.y += p0.y; o0.z += p0.z; o0.w += p0.w;
        o1.x += p1.x; o1.y += p1.y; o1.z += p1.z; o1.w += p1.w;
    }
    *reinterpret_cast<float4*>(o + i * 8) = o0;
    *reinterpret_cast<float4*>(o + i * 8 + 4) = o1;
    const float ov[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
    u32x4_t out;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        out[k] = pack_bf16x2(__uint_as_float(xv[k] << 16) + ov[2 * k],
                             __uint_as_float(xv[k] & 0xFFFF0000u) + ov[2 * k + 1]);
    *reinterpret_cast<u32x4_t*>(y + i * 8) = out;
}

}  // namespace attn

extern "C" {

hipError_t attn_launch_norm(const uint16_t* x, const float* gamma, int T, int d, float eps,
                            uint16_t* h, const double* inv_freq, float* cos_sin, int hd, int pos0,
                            hipStream_t s)
{
    hipLaunchKernelGGL(attn::norm_kernel, dim3(T), dim3(attn::kNormThreads), 0, s, x, gamma, d,
                       eps, h, inv_freq, cos_sin, hd, pos0);
    return hipGetLastError();
}

int attn_norm_in_projection(int T) { return T <= attn::kLnMaxT; }

// Two row tiles per workgroup in the decode projections: each token fragment,
// as many bytes as a weight tile's and read by every workgroup, then serves
// two tiles.  It pays
//  - where the halved grid covers three quarters of the CUs once, or all at
//    least twice (16 tokens of the DBRX block: 512 + 384 tiles 63.9 -> 55.3 us;
//    q|k|v of 1024 tiles at d 3072 54.2 -> 50.4; 256 of the output 39.1 -> 41.7,
//    192 of q|k|v 23.8 -> 25.0; in between, eight tokens, 640 tiles at d 3072
//    41.1 -> 43.0, 768 33.9 -> 35.4);
//  - from two batches of K on, or one where more than 8 tokens' fragments count
//    for more: shorter, it only takes loads out of flight (8 tokens, 512 tiles,
//    d 768 27.2 -> 28.6; d 1024, 1024 tiles, 8 tokens 32.9 -> 32.4, 16 tokens
//    37.7 -> 35.8);
//  - not at K 4096, where the row tiles lie 128 KiB apart (their loads seem to
//    meet in the same memory channels; 8 tokens, 512 tiles at d 4096 37.8 ->
//    40.0, 1024 53.1 -> 58.2), but with few tiles and more than 8 tokens' fragments
//    (384 tiles, 5 tokens 25.7 -> 26.7, 16 tokens 33.5 -> 31.4; 512 of
//    q|k|v, 12 tokens 41.9 -> 43.2; 512 of the output at d 8192, 9 tokens 68.5 -> 71.2).
// One token, whose q|k|v reads its fragments from LDS: the output projection
// alone 41.3 -> 40.5.
static bool two_tiles(int tiles, int K, int T)
{
    if (K < (T > 8 ? 1024 : 2048) || tiles < 384 || tiles % 2 != 0) return false;
    if (K == 4096) return tiles < 512 && T > 8;
    return tiles <= 512 || tiles >= 1024;
}

hipError_t attn_launch_qkv(const void* w, uint16_t* h, const uint16_t* x, const float* gamma,
                           float eps, const double* inv_freq, float* qkv, uint16_t* q,
                           uint16_t* kc, uint16_t* vc, int T, int d, int H, int G, int hd,
                           int max_seq, int pos0, hipStream_t s)
{
    attn::QkvArgs a{static_cast<const uint8_t*>(w), h, x, gamma, eps, inv_freq, qkv, q, kc, vc,
                    d, T, H, G, hd, max_seq, pos0};
    const int rows = (H + 2 * G) * hd;
    const dim3 grid(rows / moe::kTileRows), block(64 * attn::kSplit);
    if (attn_norm_in_projection(T)) {
        const size_t lds = (size_t)T * (d + attn::kHPad) * 2;
        hipLaunchKernelGGL((attn::qkv_kernel<true, 1>), grid, block, lds, s, a);
    } else {
        // (H + 2 G) hd is a multiple of 64: the row tiles are even in number
        if (two_tiles(grid.x, d, T)) hipLaunchKernelGGL((attn::qkv_kernel<false, 2>), dim3(grid.x / 2), block, 0, s, a);
        else hipLaunchKernelGGL((attn::qkv_kernel<false, 1>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

hipError_t attn_launch_out(const void* w, const uint16_t* x, int T, int K, int N, float* y32,
                           const uint16_t* res, uint16_t* y16, hipStream_t s)
{
    attn::GemvArgs a{static_cast<const uint8_t*>(w), x, y32, res, y16, K, N, T};
    const int tiles = N / moe::kTileRows;
    const dim3 block(64 * attn::kSplit);
    if (two_tiles(tiles, K, T)) hipLaunchKernelGGL(attn::gemv_kernel<2>, dim3(tiles / 2), block, 0, s, a);
    else hipLaunchKernelGGL(attn::gemv_kernel<1>, dim3(tiles), block, 0, s, a);
    return hipGetLastError();
}

hipError_t attn_launch_rope(const float* qkvp, const float* cos_sin, float* qkv, uint16_t* q,
                            uint16_t* kc, uint16_t* vc, int T, int H, int G, int hd, int max_seq,
                            int pos0, int n_split, hipStream_t s)
{
    attn::RopeArgs a{qkvp, cos_sin, qkv, q, kc, vc, T, H, G, hd, max_seq, pos0, n_split};
    const int pieces = (H + 2 * G) * hd / 8;
    hipLaunchKernelGGL(attn::rope_kernel, dim3(T, (pieces + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

int attn_part_stride(int hd) { return hd + attn::kPartPad; }

// Whether score_kernel and combine_kernel take the call: up to 16 query rows
// per key/value head and 1024 positions, where one step's fixed latency
// decides (one token, DBRX block, against flash_kernel: after 100 positions
// 42.0 us per block against 45.6, 500 42.1 against 44.1, 1000 43.5 against
// 43.4, 2047 45.4 against 43.7).  At most kShortChunks chunks.
constexpr int kShortPos = 1024;
constexpr int kShortChunks = kShortPos / attn::kChunk;
static_assert(attn::kChunk == attn::kFlashP, "attn_split_max counts both in the same steps");

int attn_short(int T, int H, int G, int n_pos) { return T * (H / G) <= 16 && n_pos <= kShortPos; }

// Position groups of flash_kernel's workgroups: 64 or 128 query rows (for up
// to 32 rows, four groups of 32-row workgroups measured slower: one token
// after 2047 positions 46.3 us per block against 43.7, after 16000 56.7
// against 54.8).
static int flash_pg(int T, int H, int G)
{
    const int R = T * (H / G);
    return R <= 64 ? 2 : 1;
}

// The most position ranges (or chunks of score_kernel) for T new tokens,
// whatever their positions: at most 1024 workgroups, 2^17 rows of partial sums
// (69 MB at head_dim 128), 128 ranges and the steps of max_seq positions.
static int attn_split_max(int T, int H, int G, int max_seq)
{
    const int pg = flash_pg(T, H, G), rows = attn::flash_rows(pg);
    const int64_t blocks = (int64_t)G * (((int64_t)T * (H / G) + rows - 1) / rows);
    const int64_t most = std::max<int64_t>(attn_short(T, H, G, 1) ? kShortChunks : 1,
                                           std::min<int64_t>({1024 / blocks, (1 << 17) / ((int64_t)T * H), 128}));
    return (int)std::min<int64_t>(most, ((int64_t)max_seq + attn::kFlashP - 1) / attn::kFlashP);
}

// The most ranges or chunks whose partial sums a call of T new tokens stores:
// score_kernel stores them with one chunk too, flash_kernel from two ranges on.
int attn_part_max(int T, int H, int G, int max_seq)
{
    const int most = attn_split_max(T, H, G, max_seq);
    return most > 1 || attn_short(T, H, G, 1) ? most : 0;
}

// Position ranges for T new tokens at pos0: the count with the least
// estimated time, in steps of one workgroup (about 2.8 us with two per CU).
// A workgroup costs its steps and about two more; 512 run at a time, in
// rounds that are cut short as far as the row blocks differ in length; the
// partial sums are written and read at about 5 TB/s.  Measured (DBRX block,
// whole call, by the number of ranges): 16 tokens after 16000 positions 219 us
// (1), 89 (32), 88 (64), 103 (128), it takes 63; 64 after 8000 426 (1), 134
// (16), 123 (32), 141 (64), it takes 18, which is too few; 300 after 1000 189
// (1), 168 (2), 161 (4), 169 (8), it takes 3; 512 after 8000 528 (1), 385 (2),
// 367 (5), it takes 5; 1024 from empty 306 (1), 339 (2), it takes 1.
int attn_split(int T, int H, int G, int pos0, int max_seq)
{
    const int pg = flash_pg(T, H, G), rows = attn::flash_rows(pg), step = attn::kFlashP;
    const int64_t nrb = ((int64_t)T * (H / G) + rows - 1) / rows;
    const double longest = (double)((pos0 + T + step - 1) / step), shortest = (double)(pos0 / step + 1);
    const int64_t most = std::min<int64_t>(attn_split_max(T, H, G, max_seq), (int64_t)longest);
    int best = 1;
    double best_cost = 0.0;
    for (int S = 1; S <= most; ++S) {
        const double n = (double)G * nrb * S, full = n / 512.0;
        const double longest_s = std::ceil(longest / S) + 2.0, shortest_s = std::ceil(shortest / S) + 2.0;
        double cost = std::max(longest_s, full * 0.5 * (longest_s + shortest_s) +
                                              (std::ceil(full) - full) * shortest_s);
        if (S > 1) cost += (double)T * H * S * 8e-5 + 1.5;
        if (S == 1 || cost < 0.98 * best_cost) { best = S; best_cost = cost; }
    }
    return best;
}

hipError_t attn_launch_flash(const uint16_t* q, const uint16_t* kc, const uint16_t* vc, float* part,
                             uint16_t* out, int T, int H, int G, int hd, int max_seq, int pos0,
                             int few, int n_split, hipStream_t s)
{
    const int pg = flash_pg(T, H, G), rows = attn::flash_rows(pg);
    const int nrb = (T * (H / G) + rows - 1) / rows;
    attn::FlashArgs a{q, kc, vc, out, part, T, H, G, max_seq, pos0, nrb, n_split,
                      (float)(1.4426950408889634 / sqrt((double)hd))};
    const dim3 grid((G * nrb * n_split + attn::kXcds - 1) / attn::kXcds * attn::kXcds), block(256);
#define ATTN_FLASH(HD, PG) \
    hipLaunchKernelGGL((few ? attn::flash_kernel<HD, PG, 3> : attn::flash_kernel<HD, PG, 2>), grid, block, 0, s, a)
    if (hd == 128) {
        if (pg == 2) ATTN_FLASH(128, 2);
        else ATTN_FLASH(128, 1);
    } else {
        if (pg == 2) ATTN_FLASH(64, 2);
        else ATTN_FLASH(64, 1);
    }
#undef ATTN_FLASH
    return hipGetLastError();
}

hipError_t attn_launch_short(const uint16_t* q, const uint16_t* kc, const uint16_t* vc, float* part,
                             int T, int H, int G, int hd, int max_seq, int pos0, hipStream_t s)
{
    const int n_chunks = (pos0 + T + attn::kChunk - 1) / attn::kChunk;
    attn::ScoreArgs a{q, kc, vc, part, T, H, G, max_seq, pos0, n_chunks,
                      (float)(1.0 / sqrt((double)hd))};
    if (hd == 128)
        hipLaunchKernelGGL(attn::score_kernel<128>, dim3(G, n_chunks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(attn::score_kernel<64>, dim3(G, n_chunks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t attn_launch_short_merge(const float* part, uint16_t* out, int T, int H, int hd, int pos0,
                                   hipStream_t s)
{
    attn::CombineArgs c{part, out, H, hd, pos0, (pos0 + T + attn::kChunk - 1) / attn::kChunk};
    hipLaunchKernelGGL(attn::combine_kernel, dim3(T * H), dim3(128), 0, s, c);
    return hipGetLastError();
}

hipError_t attn_launch_merge(const float* part, uint16_t* out, int T, int H, int hd, int n_split,
                             hipStream_t s)
{
    attn::MergeArgs a{part, out, n_split};
    const int n = T * H;
    // many rows of few ranges: a wave each (300 tokens of 48 heads, 4 ranges:
    // 15.9 -> 9 us); few rows: a workgroup each (48 rows of 8 ranges: 3.5 us
    // against 5.0)
    if (n >= 2048 && n_split <= 16) {
        if (hd == 128)
            hipLaunchKernelGGL(attn::merge_few_kernel<128>, dim3((n + 3) / 4), dim3(256), 0, s, a, n);
        else
            hipLaunchKernelGGL(attn::merge_few_kernel<64>, dim3((n + 3) / 4), dim3(256), 0, s, a, n);
    } else if (hd == 128) {
        hipLaunchKernelGGL(attn::merge_kernel<128>, dim3(n), dim3(256), 0, s, a);
    } else {
        hipLaunchKernelGGL(attn::merge_kernel<64>, dim3(n), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t attn_launch_residual(const uint16_t* x, const float* op, int n_split, float* o, uint16_t* y,
                                int64_t n, hipStream_t s)
{
    const int64_t n8 = n / 8;
    hipLaunchKernelGGL(attn::residual_kernel, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, s,
                       x, op, n_split, o, y, n8);
    return hipGetLastError();
}

}  // extern "C"
