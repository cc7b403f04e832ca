// The hierarchical non-linear codec of Alg. 1 (Sec. 4.1) for gfx950:
// encode (page normalization, chunk isolation, alpha-law transform, split
// into a signed 4-bit anchor and a signed 4-bit correction) and the
// deserializer's dequantization of the anchor alone or of the merged codes
// into BF16 pages (Sec. 4.2 Anchor and Residual phases).
//
// Per channel of a kv head (K and V alike), pages of 256 tokens, chunks of
// 32 (Sec. 6.1):
//   1. gmin = min x, gscale = max x - gmin over the page; X = (x - gmin) *
//      (1 / gscale);
//   2. mu = the chunk's mean of X (fp32 sum in token order / count),
//      Xc = X - mu, sigma = max |Xc|, Xf = Xc * (1 / sigma);
//   3. I = Round(M ln(1 + a|Xf|) / ln(1 + a)): the number of decision
//      thresholds theta_k <= |Xf|, found from the transform evaluated in
//      fp32 (within one of the count) and one exact step against the two
//      thresholds around it; S = sign(Xc); M = 127, or 7 for the 4-bit code;
//   4. by variant, with the sign-aware anchor Q_anc = V, or -V - 1 for S < 0:
//      biased:  V = min((I + 7) >> 4, 7), Q_res = clamp(16 V - I, -8, 7);
//      centred: V = I >> 4, Q_res = I - 16 V - 8 (every code kept);
//      4-bit:   V = I, no correction.
// A range whose reciprocal is not finite and positive normalizes to 0.  Every
// fp32 product that an add follows is rounded on its own (no contraction), so
// no fused multiply-add changes a result.
#include "lynx_internal.h"

#include <float.h>
#include <math.h>

namespace lynx {
namespace {

constexpr int kPage = 256;
constexpr int kChunk = 32;
constexpr int kHThreads = 256;

typedef uint32_t u32v2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16v2 __attribute__((ext_vector_type(2)));
typedef int16_t i16v2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16v2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float range_recip(float r) {
    const float v = 1.0f / r;  // IEEE division (correctly rounded)
    return (r > 0.0f && v <= FLT_MAX) ? v : 0.0f;
}

// The code byte of one channel in 16-bit fields, two tokens at a time: with
// J = min(I + bias, top), W = J ^ (low nibbles flipped by `flip`) ^ (the
// anchor's nibble of a negative value flipped).
//   biased:  J = min(I + 7, 127); V = J >> 4 and 16 V - I = 7 - (J & 15)
//            (an I above 120 keeps V = 7 and the lowest correction, -8),
//            whose nibble is (J & 15) ^ 7; -V - 1 = ~V;
//   centred: J = I; V = I >> 4, I - 16 V - 8 is the nibble (I & 15) ^ 8;
//   4-bit:   J = I, the whole code in the low nibble, ~V for a negative.
struct SplitRule {
    int bias;           // J - I
    uint32_t sign;      // nibbles a negative value flips, in both fields
    uint32_t flip;      // flips of the low nibbles, four to a 16-bit row piece
};
__device__ __forceinline__ SplitRule split_rule(int variant) {
    if (variant == kHBiased) return {7, 0x00F000F0u, 0x77777777u};
    if (variant == kHCentred) return {0, 0x00F000F0u, 0x88888888u};
    return {0, 0x000F000Fu, 0u};
}
constexpr uint32_t kTop = 0x007F007Fu;

// Decision thresholds in LDS, theta_k at entry k + kPad: entry kPad - 1 is
// below every value, the entries past the last threshold above.
constexpr int kPad = 8;
constexpr int kThetas = 128 + kPad;
// 2^23 + kPad: a float plus this rounds to an integer held in its low bits.
constexpr float kMagic = 8388608.0f + kPad;

// The low (high) 16 bits of two dwords, a in the low field.
__device__ __forceinline__ uint32_t low16s(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ __forceinline__ uint32_t high16s(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

// The low 16 bits of a, shifted left as 16 bits: one instruction, which also
// clears the high half.
__device__ __forceinline__ uint32_t shl16(uint32_t a, int n) {
    uint32_t r;
    asm("v_lshlrev_b16 %0, %1, %2" : "=v"(r) : "i"(n), "v"(a));
    return r;
}

// Workgroup (kv head, page, K or V): half wavefront c = tid / 32 owns chunk c
// of the page, lane cl = tid % 32 its channels 4 cl .. 4 cl + 3.  A half
// wavefront reads a whole 256-byte token row in one 8-byte load per lane and
// writes whole 64-byte plane rows, two bytes a lane; a channel's sum runs in
// token order inside one thread.  64 registers hold the tokens and 32 one
// channel's X, so four workgroups share a CU and a layer of 1024 pages x
// heads x 2 runs in one round.
//
// What bounds it is the vector ALU, which one instruction per element of a
// 16K layer (33.5M elements) occupies for 0.85 us.  So a code takes one
// threshold, not two (the transform less a half, rounded, leaves a single
// candidate boundary; the half is folded into the logarithm's argument and
// the rounding into the addition that makes the table index), a sigma comes
// from the chunk's extremes (rounding is monotone: the largest |X - mu| is at
// the smallest or largest x), the clamp rides on the product, and the split
// is done on 16-bit pairs.  Encode and anchor dequantization of a 16K layer
// together: 81.7 -> 51.1 us, against 39.4 for their bytes at a copy's rate.
// LAYOUT 0: one block per sequence; 1: paged.
// LINEAR: the transform is replaced by xf itself (alpha below 1e-3).
template <int LAYOUT, bool LINEAR>
__global__ __launch_bounds__(kHThreads, 4) void hencode_kernel(
    Geometry geo, int b, int T, const int32_t *__restrict__ block_table,
    const uint16_t *__restrict__ k, const uint16_t *__restrict__ v, uint8_t *__restrict__ k_anc,
    uint8_t *__restrict__ v_anc, uint8_t *__restrict__ k_res, uint8_t *__restrict__ v_res,
    HMetaPtrs meta, HTables tab, int variant) {
    // every product that an add follows is rounded on its own
#pragma clang fp contract(off)
    const int h = blockIdx.x;
    const int p = blockIdx.y;
    const int which = blockIdx.z;
    const int tid = threadIdx.x;
    const int c = tid >> 5;
    const int cl = tid & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Hkv = geo.Hkv;
    const int t0 = p * kPage;
    const int n = min(kPage, T - t0);
    const SplitRule sr = split_rule(variant);
    const bool has_res = variant != kHInt4;
    const uint16_t *src = which == 0 ? k : v;
    uint8_t *anc = which == 0 ? k_anc : v_anc;
    uint8_t *res = which == 0 ? k_res : v_res;
    float *gmin_a = which == 0 ? meta.k_gmin : meta.v_gmin;
    float *gsc_a = which == 0 ? meta.k_gscale : meta.v_gscale;
    float *mu_a = which == 0 ? meta.k_mu : meta.v_mu;
    float *sig_a = which == 0 ? meta.k_sigma : meta.v_sigma;

    __shared__ float s_theta[kThetas];
    __shared__ float s_lo[8][kHeadDim], s_hi[8][kHeadDim];

    // the thread's 32 tokens x 4 channels (BF16 pairs)
    u32v2 raw[kChunk];
    if (n == kPage && Hkv < 65536) {  // 32-bit offsets within a wavefront's rows
        const uint8_t *base = reinterpret_cast<const uint8_t *>(src + ((size_t)(t0 + 64 * wave) * Hkv + h) * kHeadDim);
        const uint32_t row = (uint32_t)Hkv * (2 * kHeadDim);
        const uint32_t off = (tid & 32) * row + 8 * cl;
#pragma unroll
        for (int i = 0; i < kChunk; ++i)
            raw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32v2 *>(base + (size_t)i * row + off));
    } else {
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
            const int tl = min(kChunk * c + i, n - 1);  // rows past the page re-read its last token
            raw[i] = *reinterpret_cast<const u32v2 *>(src + ((size_t)(t0 + tl) * Hkv + h) * kHeadDim + 4 * cl);
        }
    }
    if (tid < kThetas) s_theta[tid] = tid < kPad ? -INFINITY : tab.theta[tid - kPad];
    const int cnt = max(0, min(kChunk, n - kChunk * c));  // tokens of the thread

    auto value = [&](int i, int j) {
        const uint32_t w = raw[i][j >> 1];
        return __uint_as_float((j & 1) ? w & 0xffff0000u : w << 16);
    };

    // ---- stage 1: min / max per channel over the chunk, then the page (rows
    // past the page repeat its last token, which leaves both unchanged) ----
    float cmin[4], cmax[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        cmin[j] = INFINITY;
        cmax[j] = -INFINITY;
#pragma unroll
        for (int i = 0; i < kChunk; i += 2) {
            cmin[j] = fminf(fminf(cmin[j], value(i, j)), value(i + 1, j));
            cmax[j] = fmaxf(fmaxf(cmax[j], value(i, j)), value(i + 1, j));
        }
    }
    *reinterpret_cast<float4 *>(&s_lo[c][4 * cl]) = make_float4(cmin[0], cmin[1], cmin[2], cmin[3]);
    *reinterpret_cast<float4 *>(&s_hi[c][4 * cl]) = make_float4(cmax[0], cmax[1], cmax[2], cmax[3]);
    __syncthreads();
    float lo[4], hi[4], gsc[4], ig[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        lo[j] = s_lo[0][4 * cl + j];
        hi[j] = s_hi[0][4 * cl + j];
    }
#pragma unroll
    for (int q = 1; q < 8; ++q) {
        const float4 a = *reinterpret_cast<const float4 *>(&s_lo[q][4 * cl]);
        const float4 z = *reinterpret_cast<const float4 *>(&s_hi[q][4 * cl]);
        const float av[4] = {a.x, a.y, a.z, a.w}, zv[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lo[j] = fminf(lo[j], av[j]);
            hi[j] = fmaxf(hi[j], zv[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (lo[j] == 0.0f) lo[j] = 0.0f;  // -0 -> +0
        if (hi[j] == 0.0f) hi[j] = 0.0f;
        gsc[j] = hi[j] - lo[j];
        ig[j] = range_recip(gsc[j]);
    }
    if (c == 0) {
        const size_t pm = (((size_t)b * Hkv + h) * geo.n_pages + p) * kHeadDim + 4 * cl;
        *reinterpret_cast<float4 *>(gmin_a + pm) = make_float4(lo[0], lo[1], lo[2], lo[3]);
        *reinterpret_cast<float4 *>(gsc_a + pm) = make_float4(gsc[0], gsc[1], gsc[2], gsc[3]);
    }
    if (cnt == 0) return;  // no barrier follows

    if (n != kPage) {
        // rows past the page become the page's minimum, an X of +0: the sum
        // of X over the chunk's tokens passes them by
        const uint32_t l01 = (__float_as_uint(lo[0]) >> 16) | (__float_as_uint(lo[1]) & 0xffff0000u);
        const uint32_t l23 = (__float_as_uint(lo[2]) >> 16) | (__float_as_uint(lo[3]) & 0xffff0000u);
#pragma unroll
        for (int i = 1; i < kChunk; ++i)
            if (i >= cnt) raw[i] = u32v2{l01, l23};
    }

    // ---- stages 2-4, one channel at a time; codes of a channel pair as
    // bytes in 16-bit fields (two tokens), then both pairs' bytes together:
    // dword i2 of a plane is the two bytes of token 2 i2 and of token
    // 2 i2 + 1 ----
    uint32_t o_anc[kChunk / 2], o_res[kChunk / 2];
    float mu[4], sig[4];
#pragma unroll
    for (int jp = 0; jp < 2; ++jp) {
        uint32_t W[2][kChunk / 2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = 2 * jp + u;
            // unpacked anew, and not before the channel's turn: the unpacked
            // values would not fit beside the packed ones
#pragma unroll
            for (int i = 0; i < kChunk; ++i) asm volatile("" : "+v"(raw[i][jp]));
            __builtin_amdgcn_sched_barrier(0);
            // x - (-0) is +0 where x is -0: no X is -0, and the sign bit of
            // X - mu is its sign
            const float l = lo[j] == 0.0f ? -0.0f : lo[j];
            float X[kChunk];
#pragma unroll
            for (int i = 0; i < kChunk; ++i) X[i] = (value(i, j) - l) * ig[j];
            // the sum in token order over the chunk's tokens; X >= +0 or NaN
            float sum = X[0];
#pragma unroll
            for (int i = 1; i < kChunk; ++i) sum = sum + X[i];
            // a whole chunk divides by a power of two: the product is the quotient
            mu[j] = n == kPage ? sum * (1.0f / kChunk) : sum / (float)cnt;
            const float e0 = fabsf((cmin[j] - l) * ig[j] - mu[j]);
            const float e1 = fabsf((cmax[j] - l) * ig[j] - mu[j]);
            sig[j] = fmaxf(fmaxf(0.0f, e0), e1);  // 0 where the chunk holds a NaN
            const float is = range_recip(sig[j]);
            const uint32_t neg = mu[j] == mu[j] ? sr.sign : 0u;  // a NaN has no sign
#pragma unroll
            for (int i2 = 0; i2 < kChunk / 2; ++i2) {
                uint32_t J[2], xs[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float xc = X[2 * i2 + e] - mu[j];
                    const float xf = __builtin_amdgcn_fmed3f(fabsf(xc) * is, 0.0f, 1.0f);  // a NaN: 0
                    // The transform less a half of a code, rounded to the
                    // integer kk: within half a code of the exact value, the
                    // count is kk or kk + 1, and theta_kk decides.
                    const float ye = LINEAR ? xf - tab.yhalf
                                            : __builtin_amdgcn_logf(__builtin_fmaf(xf, tab.alpha_h, tab.one_h));
                    const uint32_t kk = __float_as_uint(__builtin_fmaf(ye, tab.yscale, kMagic));
                    const uint32_t at = shl16(kk, 2);
                    const float th = *reinterpret_cast<const float *>(reinterpret_cast<const uint8_t *>(s_theta) + at);
                    J[e] = kk + (uint32_t)(sr.bias - kPad) + (th <= xf ? 1u : 0u);
                    xs[e] = __float_as_uint(xc);
                }
                const u16v2 jm = __builtin_elementwise_min(__builtin_bit_cast(u16v2, low16s(J[0], J[1])),
                                                           __builtin_bit_cast(u16v2, kTop));
                const i16v2 sg = __builtin_bit_cast(i16v2, high16s(xs[0], xs[1])) >> (int16_t)15;
                W[u][i2] = __builtin_bit_cast(uint32_t, jm) ^ (__builtin_bit_cast(uint32_t, sg) & neg);
                asm volatile("" : "+v"(W[u][i2]));
            }
        }
#pragma unroll
        for (int i2 = 0; i2 < kChunk / 2; ++i2) {
            const uint32_t w0 = W[0][i2], w1 = W[1][i2];
            const uint32_t a = ((w0 >> 4) & 0x000F000Fu) | (w1 & 0x00F000F0u);
            const uint32_t r = (w0 & 0x000F000Fu) | ((w1 << 4) & 0x00F000F0u);
            // bytes 0, 2 of the first pair, then of the second
            o_anc[i2] = jp == 0 ? a : __builtin_amdgcn_perm(a, o_anc[i2], 0x06020400u);
            o_res[i2] = jp == 0 ? r : __builtin_amdgcn_perm(r, o_res[i2], 0x06020400u) ^ sr.flip;
        }
    }
    const size_t cm = (((size_t)b * Hkv + h) * geo.n_chunks + (size_t)t0 / kChunk + c) * kHeadDim + 4 * cl;
    *reinterpret_cast<float4 *>(mu_a + cm) = make_float4(mu[0], mu[1], mu[2], mu[3]);
    *reinterpret_cast<float4 *>(sig_a + cm) = make_float4(sig[0], sig[1], sig[2], sig[3]);

    // ---- the plane rows; the 4-bit code is the low nibble's ----
    const int32_t *bt_row = block_table + (size_t)b * geo.max_blocks;
    const int tc = t0 + kChunk * c;
    if (!has_res) {
#pragma unroll
        for (int i2 = 0; i2 < kChunk / 2; ++i2) o_anc[i2] = o_res[i2];
    }
    if (LAYOUT == 0 || geo.bt % kChunk == 0) {  // the chunk's rows follow each other
        const int bi = LAYOUT == 0 ? 0 : tc / geo.bt;
        const int blk = bt_row[bi];
        if (blk < 0 || blk >= geo.num_blocks) return;
        const size_t off = (((size_t)blk * Hkv + h) * geo.bt + (tc - (size_t)bi * geo.bt)) * kNibbleRow + 2 * cl;
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
            if (i < cnt) {
                const uint32_t sh = 16 * (i & 1);
                *reinterpret_cast<uint16_t *>(anc + off + i * kNibbleRow) = (uint16_t)(o_anc[i >> 1] >> sh);
                if (has_res) *reinterpret_cast<uint16_t *>(res + off + i * kNibbleRow) = (uint16_t)(o_res[i >> 1] >> sh);
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < kChunk; ++i) {
        if (i < cnt) {
            const int bi = (tc + i) / geo.bt;
            const int blk = bt_row[bi];
            if (blk >= 0 && blk < geo.num_blocks) {
                const size_t off = (((size_t)blk * Hkv + h) * geo.bt + (tc + i - bi * geo.bt)) * kNibbleRow + 2 * cl;
                const uint32_t sh = 16 * (i & 1);
                *reinterpret_cast<uint16_t *>(anc + off) = (uint16_t)(o_anc[i >> 1] >> sh);
                if (has_res) *reinterpret_cast<uint16_t *>(res + off) = (uint16_t)(o_res[i >> 1] >> sh);
            }
        }
    }
}

// Two floats rounded to BF16 to nearest even, a in the low half (a NaN stays
// one, quieted).
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    bf16v2 r;
    r.x = (__bf16)a;
    r.y = (__bf16)b;
    return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ int sext4(uint32_t nib) { return (int)nib >= 8 ? (int)nib - 16 : (int)nib; }

// The signed level of one code: the anchor nibble qa alone (the anchor
// planes), or with the correction nibble qr.  Biased: code 16 V, or 16 V -
// Q_res; centred: the bucket centre 16 V + 7.5, or 16 V + 8 + Q_res; 4-bit: V.
template <int FULL>
__device__ __forceinline__ float signed_level(const HTables &tab, int variant, uint32_t qa, uint32_t qr) {
    const int a = sext4(qa), r = sext4(qr);
    const int V = a >= 0 ? a : -a - 1;
    float lv;
    if (variant == kHBiased) lv = tab.level[min(max(16 * V - (FULL ? r : 0), 0), 127)];
    else if (variant == kHCentred) lv = FULL ? tab.level[16 * V + 8 + r] : tab.alevel[V];
    else lv = tab.level[V];
    return a >= 0 ? lv : -lv;
}

// Dequantization to BF16 [T][Hkv][128]: thread (kOct tokens, 8 dims), x =
// ((+-level * sigma) + mu) * gscale + gmin in fp32, rounded to BF16 to
// nearest even.  FULL 0: anchor nibble planes; 1: code planes.
// The output bounds it (67 of 84 MB of a 16K layer's anchors).  The vector ALU
// did before (25.9 us: a dozen instructions per element to find a level and
// round it), so the signed levels stand in LDS by plane byte -- of the one
// code, or of an anchor byte's two -- and a pair is rounded in one
// instruction.
constexpr int kOct = 16;  // tokens of a thread; a chunk is a multiple
template <int FULL, int LAYOUT>
__global__ __launch_bounds__(kHThreads) void hdequant_kernel(
    Geometry geo, int b, int T, int bt_shift, const int32_t *__restrict__ block_table,
    const uint8_t *__restrict__ k_plane, const uint8_t *__restrict__ v_plane, HMetaPtrs meta,
    HTables tab, int variant, uint16_t *__restrict__ k_out, uint16_t *__restrict__ v_out) {
    // every product that an add follows is rounded on its own
#pragma clang fp contract(off)
    __shared__ float s_level[FULL ? 256 : 512];
    if (FULL) {
        s_level[threadIdx.x] = signed_level<FULL>(tab, variant, threadIdx.x >> 4, threadIdx.x & 15);
    } else {
        s_level[2 * threadIdx.x] = signed_level<FULL>(tab, variant, threadIdx.x & 15, 0);
        s_level[2 * threadIdx.x + 1] = signed_level<FULL>(tab, variant, threadIdx.x >> 4, 0);
    }
    __syncthreads();
    const int Hkv = geo.Hkv;
    // item (tensor, token run, head, 8-dim piece), the piece fastest: a
    // thread loads the page and chunk scalars of its 8 dims once (a run never
    // straddles a chunk)
    const int n_oct = (T + kOct - 1) / kOct;
    const size_t per = (size_t)n_oct * Hkv * 16;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const int32_t *bt_row = block_table + (size_t)b * geo.max_blocks;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < 2 * per; e += stride) {
        const int which = e >= per ? 1 : 0;
        const size_t r = e - (size_t)which * per;
        const int d8 = (int)(r & 15);
        const size_t oh = r >> 4;  // run * Hkv + h
        const int h = (int)(oh % Hkv);
        const int t0 = kOct * (int)(oh / Hkv);
        const size_t pm = (((size_t)b * Hkv + h) * geo.n_pages + t0 / kPage) * kHeadDim + 8 * d8;
        const size_t cm = (((size_t)b * Hkv + h) * geo.n_chunks + t0 / kChunk) * kHeadDim + 8 * d8;
        const float *gmin_a = which == 0 ? meta.k_gmin : meta.v_gmin;
        const float *gsc_a = which == 0 ? meta.k_gscale : meta.v_gscale;
        const float *mu_a = which == 0 ? meta.k_mu : meta.v_mu;
        const float *sig_a = which == 0 ? meta.k_sigma : meta.v_sigma;
        float gm[8], gs[8], mu[8], sg[8];
#pragma unroll
        for (int k4 = 0; k4 < 2; ++k4) {
            const float4 a = *reinterpret_cast<const float4 *>(gmin_a + pm + 4 * k4);
            const float4 s = *reinterpret_cast<const float4 *>(gsc_a + pm + 4 * k4);
            const float4 m = *reinterpret_cast<const float4 *>(mu_a + cm + 4 * k4);
            const float4 g = *reinterpret_cast<const float4 *>(sig_a + cm + 4 * k4);
            gm[4 * k4] = a.x; gm[4 * k4 + 1] = a.y; gm[4 * k4 + 2] = a.z; gm[4 * k4 + 3] = a.w;
            gs[4 * k4] = s.x; gs[4 * k4 + 1] = s.y; gs[4 * k4 + 2] = s.z; gs[4 * k4 + 3] = s.w;
            mu[4 * k4] = m.x; mu[4 * k4 + 1] = m.y; mu[4 * k4 + 2] = m.z; mu[4 * k4 + 3] = m.w;
            sg[4 * k4] = g.x; sg[4 * k4 + 1] = g.y; sg[4 * k4 + 2] = g.z; sg[4 * k4 + 3] = g.w;
        }
        const uint8_t *plane = which == 0 ? k_plane : v_plane;
        uint16_t *out = which == 0 ? k_out : v_out;
        constexpr int kRow = FULL ? kCodeRow : kNibbleRow;
        const int nt = min(kOct, T - t0);
        auto row_of = [&](int t, bool &ok) -> size_t {
            int blk, tb;
            if (LAYOUT == 0) {
                blk = bt_row[0];
                tb = t;
            } else {
                const int bi = bt_shift >= 0 ? (t >> bt_shift) : t / geo.bt;
                blk = bt_row[bi];
                tb = t - bi * geo.bt;
            }
            ok = blk >= 0 && blk < geo.num_blocks;
            return ((size_t)blk * Hkv + h) * geo.bt + tb;
        };
        auto emit = [&](int t, uint2 cw) {
            float lv[8];
#pragma unroll
            for (int j = 0; j < 8; j += FULL ? 1 : 2) {
                const int by = FULL ? j : j / 2;  // the plane byte
                const uint32_t c = ((by < 4 ? cw.x : cw.y) >> (8 * (by & 3))) & 0xffu;
                if (FULL) {
                    lv[j] = s_level[c];
                } else {
                    const float2 two = *reinterpret_cast<const float2 *>(&s_level[2 * c]);
                    lv[j] = two.x;
                    lv[j + 1] = two.y;
                }
            }
            uint32_t o[4];
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                const float x0 = ((lv[j] * sg[j]) + mu[j]) * gs[j] + gm[j];
                const float x1 = ((lv[j + 1] * sg[j + 1]) + mu[j + 1]) * gs[j + 1] + gm[j + 1];
                o[j / 2] = bf16_pair(x0, x1);
            }
            *reinterpret_cast<uint4 *>(out + ((size_t)t * Hkv + h) * kHeadDim + 8 * d8) =
                make_uint4(o[0], o[1], o[2], o[3]);
        };
        auto piece = [&](size_t row) -> uint2 {
            if (FULL) return *reinterpret_cast<const uint2 *>(plane + row * kRow + 8 * d8);
            return make_uint2(*reinterpret_cast<const uint32_t *>(plane + row * kRow + 4 * d8), 0u);
        };
        // a run inside one block (every run of a contiguous cache, of blocks
        // of a multiple of the run): rows follow each other, and all of a
        // run's loads are in flight before its first store
        if (nt == kOct && (LAYOUT == 0 || geo.bt % kOct == 0)) {
            bool ok;
            const size_t row = row_of(t0, ok);
            if (!ok) continue;
            uint2 cw[kOct];
#pragma unroll
            for (int k = 0; k < kOct; ++k) cw[k] = piece(row + k);
#pragma unroll
            for (int k = 0; k < kOct; ++k) emit(t0 + k, cw[k]);
            continue;
        }
        for (int k = 0; k < nt; ++k) {
            bool ok;
            const size_t row = row_of(t0 + k, ok);
            if (ok) emit(t0 + k, piece(row));
        }
    }
}

int shift_of(int bt) {
    for (int sh = 0; sh < 31; ++sh)
        if ((1 << sh) == bt) return sh;
    return -1;
}

}  // namespace

void make_htables(float alpha, int variant, HTables *t) {
    const double la = log1p((double)alpha);
    const int M = variant == kHInt4 ? 7 : 127;
    for (int k = 0; k < 128; ++k)
        t->theta[k] = k < M ? (float)(expm1(((k + 0.5) / M) * la) / (double)alpha) : INFINITY;
    for (int i = 0; i < 128; ++i)
        t->level[i] = (float)(expm1(((double)(i < M ? i : M) / M) * la) / (double)alpha);
    for (int v = 0; v < 8; ++v) t->alevel[v] = (float)(expm1(((16 * v + 7.5) / 127.0) * la) / (double)alpha);
    t->linear = alpha < 1e-3f ? 1 : 0;
    const double ys = t->linear ? (double)M : M / log2(1.0 + (double)alpha);
    const double half = exp2(-0.5 / ys);  // log2(half * y) * ys = log2(y) * ys - 0.5
    t->yscale = (float)ys;
    t->yhalf = (float)(0.5 / ys);
    t->one_h = (float)half;
    t->alpha_h = (float)(half * (double)alpha);
}

hipError_t launch_hencode(const Geometry &g, int b, int T, const int32_t *block_table,
                          const uint16_t *k, const uint16_t *v, uint8_t *k_anc, uint8_t *v_anc,
                          uint8_t *k_res, uint8_t *v_res, HMetaPtrs meta, const HTables &tab,
                          int variant, hipStream_t stream) {
    if (T <= 0) return hipSuccess;
    dim3 grid(g.Hkv, (T + kPage - 1) / kPage, 2);
#define LYNX_HENCODE(LAYOUT, LINEAR)                                                              \
    hipLaunchKernelGGL((hencode_kernel<LAYOUT, LINEAR>), grid, dim3(kHThreads), 0, stream, g, b, T, \
                       block_table, k, v, k_anc, v_anc, k_res, v_res, meta, tab, variant)
    if (g.max_blocks == 1) {
        if (tab.linear) LYNX_HENCODE(0, true);
        else LYNX_HENCODE(0, false);
    } else {
        if (tab.linear) LYNX_HENCODE(1, true);
        else LYNX_HENCODE(1, false);
    }
#undef LYNX_HENCODE
    return hipGetLastError();
}

hipError_t launch_hdequant(bool full, const Geometry &g, int b, int T, const int32_t *block_table,
                           const uint8_t *k_plane, const uint8_t *v_plane, HMetaPtrs meta,
                           const HTables &tab, int variant, uint16_t *k_out, uint16_t *v_out,
                           hipStream_t stream) {
    if (T <= 0) return hipSuccess;
    size_t blocks = ((size_t)2 * ((T + kOct - 1) / kOct) * g.Hkv * 16 + kHThreads - 1) / kHThreads;
    if (blocks > 256 * 32) blocks = 256 * 32;
    const dim3 grid((unsigned)blocks);
    const int sh = shift_of(g.bt);
    if (full) {
        if (g.max_blocks == 1)
            hipLaunchKernelGGL((hdequant_kernel<1, 0>), grid, dim3(kHThreads), 0, stream, g, b, T, sh,
                               block_table, k_plane, v_plane, meta, tab, variant, k_out, v_out);
        else
            hipLaunchKernelGGL((hdequant_kernel<1, 1>), grid, dim3(kHThreads), 0, stream, g, b, T, sh,
                               block_table, k_plane, v_plane, meta, tab, variant, k_out, v_out);
    } else {
        if (g.max_blocks == 1)
            hipLaunchKernelGGL((hdequant_kernel<0, 0>), grid, dim3(kHThreads), 0, stream, g, b, T, sh,
                               block_table, k_plane, v_plane, meta, tab, variant, k_out, v_out);
        else
            hipLaunchKernelGGL((hdequant_kernel<0, 1>), grid, dim3(kHThreads), 0, stream, g, b, T, sh,
                               block_table, k_plane, v_plane, meta, tab, variant, k_out, v_out);
    }
    return hipGetLastError();
}

}  // namespace lynx
