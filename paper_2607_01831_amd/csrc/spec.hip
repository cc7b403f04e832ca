// Greedy acceptance of speculative tokens (Sec. 4.3): the verification pass
// gives the target model's scores at the k draft positions and the one after
// them; the drafts are kept up to the first position where the target's own
// choice (its highest score, the lowest vocabulary index among equal scores)
// differs, and that choice corrects the divergence (or, when all k drafts are
// kept, is the bonus token).
//
// Two passes, the first bound by the (k + 1) x V scores of a sequence, the
// second by its launch:
//  1. argmax_chunk_kernel -- grid (vocabulary chunk, position, sequence): the
//     best (score, index) of 4096 vocabulary entries, a thread's 16 scores
//     loaded together (16-byte loads when the rows allow it), the maximum
//     first and then the lowest index that has it, on the permute paths;
//  2. accept_kernel -- one workgroup per sequence, its wavefronts taking the
//     positions in turn, so that no position waits for the one before it; the
//     first disagreement is one ballot.  (A wavefront that walked the
//     positions in order waited for memory once for each kept draft.)
// 16 sequences, 8 drafts, 128256 entries (74 MB): 25.4 -> 18.5 us.
//
// Acceptance of sampled drafts (the speculative-sampling form of the same
// rule): draft i, token x, is kept when u_i q_i(x) <= p_i(x) (kept with
// probability min(1, p/q)); at the first draft not kept, n, the next token is
// drawn from max(p_n - q_n, 0), and when all are kept the bonus from p_k.
// The draw is an exact inverse-CDF draw: weights w_v = floor(r_v 2^40) with
// r_v clamped to [0, 1] (NaN 0), S = sum w, U = floor(u_k 2^32),
// t = floor(S U / 2^32), the token the first whose inclusive prefix of w
// exceeds t; a zero residual falls back to p_n, and an all-zero p_n gives
// -1.
// Two passes.  The tests read one entry of p and q per draft, so every
// workgroup of sample_chunk_kernel makes them for itself (two dependent
// loads) and then sums the integer weights of its chunk of row n alone: one
// row of each model is read instead of all 2 k + 1.  sample_pick_kernel
// locates t through the chunk sums and then one chunk, whose entries each
// thread holds in registers between the scan and the walk.
// 16 sequences, 8 drafts, 128256 entries: 36.5 -> 11.0 us (139 MB
// read before, 16 MB now).
#include "lane_ops.h"
#include "lynx_internal.h"

#include <limits.h>
#include <math.h>

namespace lynx {
namespace {

constexpr int kThreads = 256;
constexpr int kChunk = 4096;  // vocabulary entries per workgroup of pass 1

// (v, i) beats (bv, bi): a higher score, or the same score at a lower index.
// A NaN score never wins.
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
    return v > bv || (v == bv && i < bi);
}

// The best (score, index) over the wavefront, in every lane: the maximum, then
// the lowest index that holds it.
__device__ __forceinline__ void wave_best(float &bv, int &bi) {
    const float m = max_kg(row16_max(bv));
    int i = bv == m ? bi : INT_MAX;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) i = min(i, __shfl_xor(i, off));
    bv = m;
    bi = i;
}

constexpr int kPer = kChunk / kThreads;  // 16 entries per thread

__global__ __launch_bounds__(kThreads) void argmax_chunk_kernel(const float *__restrict__ logits,
                                                                int V, int n_chunks, int vec4,
                                                                float *part_v, int *part_i) {
    const int chunk = blockIdx.x;
    const int pos = blockIdx.y;
    const int b = blockIdx.z;
    const int tid = threadIdx.x;
    const float *row = logits + ((size_t)b * gridDim.y + pos) * (size_t)V;
    const int lo = chunk * kChunk;
    const int hi = min(V, lo + kChunk);
    // entry j of the thread: lo + 1024 (j / 4) + 4 tid + j % 4, or
    // lo + 256 j + tid; past the chunk a NaN, which never wins
    float x[kPer];
    if (vec4) {
        // V % 4 == 0 and 16-byte rows: every float4 lies inside [lo, hi)
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j) {
            const int e = lo + 4 * kThreads * j + 4 * tid;
            const float4 u = *reinterpret_cast<const float4 *>(row + min(e, hi - 4));
            const bool in = e < hi;
            x[4 * j] = in ? u.x : NAN;
            x[4 * j + 1] = in ? u.y : NAN;
            x[4 * j + 2] = in ? u.z : NAN;
            x[4 * j + 3] = in ? u.w : NAN;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int e = lo + kThreads * j + tid;
            const float u = row[min(e, hi - 1)];
            x[j] = e < hi ? u : NAN;
        }
    }
    float bv = -INFINITY;
#pragma unroll
    for (int j = 0; j < kPer; ++j) bv = fmaxf(bv, x[j]);  // passes over NaN
    int bi = INT_MAX;
#pragma unroll
    for (int j = kPer - 1; j >= 0; --j) {
        const int e = vec4 ? lo + 4 * kThreads * (j / 4) + 4 * tid + j % 4 : lo + kThreads * j + tid;
        bi = x[j] == bv ? e : bi;
    }
    wave_best(bv, bi);
    __shared__ float s_v[kThreads / 64];
    __shared__ int s_i[kThreads / 64];
    if ((tid & 63) == 0) {
        s_v[tid >> 6] = bv;
        s_i[tid >> 6] = bi;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kThreads / 64; ++w)
            if (better(s_v[w], s_i[w], bv, bi)) {
                bv = s_v[w];
                bi = s_i[w];
            }
        const size_t p = ((size_t)b * gridDim.y + pos) * n_chunks + chunk;
        part_v[p] = bv;
        part_i[p] = bi;
    }
}

constexpr int kMaxDrafts = 64;

__global__ __launch_bounds__(kThreads) void accept_kernel(const float *__restrict__ part_v,
                                                          const int *__restrict__ part_i, int k,
                                                          int n_chunks, const int32_t *__restrict__ drafts,
                                                          int32_t *accepted, int32_t *next_token) {
    const int b = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    __shared__ int s_choice[kMaxDrafts + 1];
    const int draft = lane < k ? drafts[(size_t)b * k + lane] : 0;
    for (int pos = w; pos <= k; pos += kThreads / 64) {
        const size_t p0 = ((size_t)b * (k + 1) + pos) * n_chunks;
        float bv = -INFINITY;
        int bi = INT_MAX;
        for (int c = lane; c < n_chunks; c += 64)
            if (better(part_v[p0 + c], part_i[p0 + c], bv, bi)) {
                bv = part_v[p0 + c];
                bi = part_i[p0 + c];
            }
        wave_best(bv, bi);  // every lane holds the position's choice
        if (lane == 0) s_choice[pos] = bi;
    }
    __syncthreads();
    if (w == 0) {
        const uint64_t stop = __ballot(lane < k && s_choice[min(lane, k)] != draft);
        const int n = stop ? __ffsll((long long)stop) - 1 : k;
        if (lane == 0) {
            accepted[b] = n;
            next_token[b] = s_choice[n];
        }
    }
}

__device__ __forceinline__ uint64_t sample_weight(float r) {
    r = r > 0.0f ? r : 0.0f;  // NaN and negatives count 0
    r = r < 1.0f ? r : 1.0f;
    return (uint64_t)(r * 1099511627776.0f);  // 2^40: exact scaling, then truncation
}

__device__ __forceinline__ uint32_t sample_uniform(float u) {
    const float s = u * 4294967296.0f;  // 2^32
    if (!(s > 0.0f)) return 0u;
    if (s >= 4294967296.0f) return 0xFFFFFFFFu;
    return (uint32_t)s;
}

// Exclusive prefix of x over the workgroup's threads in thread order, and the
// total.
__device__ __forceinline__ uint64_t block_scan_u64(uint64_t x, uint64_t *s_wave, uint64_t &total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t incl = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    __syncthreads();
    if (lane == 63) s_wave[w] = incl;
    __syncthreads();
    uint64_t pre = incl - x;
    total = 0;
    for (int j = 0; j < kThreads / 64; ++j) {
        if (j < w) pre += s_wave[j];
        total += s_wave[j];
    }
    return pre;
}

// The number of leading drafts kept: lane i tests draft i (k <= 64); the same
// in every lane.
__device__ __forceinline__ int kept_drafts(const float *pb, const float *qb, const int32_t *drafts,
                                           const float *u, int k, int V) {
    const int i = threadIdx.x & 63;
    bool stop = false;
    if (i < k) {
        const int x = drafts[i];
        stop = x < 0 || x >= V || !(u[i] * qb[(size_t)i * V + x] <= pb[(size_t)i * V + x]);
    }
    const uint64_t m = __ballot(stop);
    return m ? __ffsll((long long)m) - 1 : k;
}

// Pass 1 of the sampled acceptance: per (chunk of 4096 entries, sequence) the
// sums of the integer weights of the residual p_n - q_n (p_k at the last
// position) and of p_n alone (the fall-back draw), n the number of drafts
// kept, which chunk 0 writes down too.  Sums are integers, so the order of
// the additions does not matter.  sums: [B][n_chunks][2].
__global__ __launch_bounds__(kThreads) void sample_chunk_kernel(const float *__restrict__ p,
                                                                const float *__restrict__ q,
                                                                const int32_t *__restrict__ drafts,
                                                                const float *__restrict__ u, int k,
                                                                int V, int n_chunks, int vec4,
                                                                uint64_t *sums, int *kept) {
    const int chunk = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x;
    const float *pb = p + (size_t)b * (k + 1) * V;
    const float *qb = q + (size_t)b * k * V;
    const int n = kept_drafts(pb, qb, drafts + (size_t)b * k, u + (size_t)b * (k + 1), k, V);
    const float *prow = pb + (size_t)n * V;
    const float *qrow = n < k ? qb + (size_t)n * V : nullptr;
    const int lo = chunk * kChunk, hi = min(V, lo + kChunk);
    uint64_t sr = 0, sp = 0;
    if (vec4) {
        float4 a[kPer / 4], c[kPer / 4];
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j) {
            const int e = min(lo + 4 * kThreads * j + 4 * tid, hi - 4);
            a[j] = *reinterpret_cast<const float4 *>(prow + e);
            c[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (qrow) c[j] = *reinterpret_cast<const float4 *>(qrow + e);
        }
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j) {
            if (lo + 4 * kThreads * j + 4 * tid >= hi) break;
            sp += sample_weight(a[j].x) + sample_weight(a[j].y) + sample_weight(a[j].z) + sample_weight(a[j].w);
            sr += sample_weight(a[j].x - c[j].x) + sample_weight(a[j].y - c[j].y) +
                  sample_weight(a[j].z - c[j].z) + sample_weight(a[j].w - c[j].w);
        }
    } else {
        for (int e = lo + tid; e < hi; e += kThreads) {
            const float a = prow[e];
            sp += sample_weight(a);
            sr += sample_weight(qrow ? a - qrow[e] : a);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        sp += __shfl_xor(sp, off);
        sr += __shfl_xor(sr, off);
    }
    __shared__ uint64_t s_sum[2][kThreads / 64];
    if ((tid & 63) == 0) {
        s_sum[0][tid >> 6] = sr;
        s_sum[1][tid >> 6] = sp;
    }
    __syncthreads();
    if (tid < 2) {
        uint64_t t = 0;
        for (int j = 0; j < kThreads / 64; ++j) t += s_sum[tid][j];
        sums[((size_t)b * n_chunks + chunk) * 2 + tid] = t;
    }
    if (chunk == 0 && tid == 0) kept[b] = n;
}

// Pass 2: one workgroup per sequence.  S is the residual's sum, or p_n's when
// that is 0; a scan over the chunk sums finds the chunk that holds t, and a
// scan over that chunk's 16-entry thread slices the slice; its thread walks
// it.
__global__ __launch_bounds__(kThreads) void sample_pick_kernel(
    const float *__restrict__ p, const float *__restrict__ q, const float *__restrict__ u, int k, int V,
    int n_chunks, int vec4, const uint64_t *__restrict__ sums, const int *__restrict__ kept,
    int32_t *accepted, int32_t *next_token) {
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    __shared__ int s_tok, s_chunk;
    __shared__ uint64_t s_t;
    __shared__ uint64_t s_wave[kThreads / 64];
    if (tid == 0) {
        s_tok = -1;
        s_chunk = -1;
    }
    // thread slices of the chunk sums: ceil(n_chunks / 256) chunks each
    const uint64_t *cs = sums + (size_t)b * n_chunks * 2;
    const int cper = (n_chunks + kThreads - 1) / kThreads;
    const int c0 = min(n_chunks, tid * cper), c1 = min(n_chunks, c0 + cper);
    uint64_t both[2] = {0, 0};
    for (int c = c0; c < c1; ++c) {
        both[0] += cs[2 * c];
        both[1] += cs[2 * c + 1];
    }
    const int n = kept[b];
    const uint32_t U = sample_uniform(u[(size_t)b * (k + 1) + k]);
    uint64_t S;
    uint64_t pre = block_scan_u64(both[0], s_wave, S);
    const bool fallback = S == 0;  // uniform; the bonus row's two sums are the same
    if (fallback) pre = block_scan_u64(both[1], s_wave, S);
    if (S > 0) {
        const uint64_t t = (S >> 32) * U + (((S & 0xFFFFFFFFull) * U) >> 32);
        const uint64_t mine = fallback ? both[1] : both[0];
        if (mine > 0 && pre <= t && t - pre < mine) {
            uint64_t acc = pre;
            for (int c = c0; c < c1; ++c) {
                const uint64_t x = cs[2 * c + (fallback ? 1 : 0)];
                if (t - acc < x) {
                    s_chunk = c;
                    s_t = t - acc;
                    break;
                }
                acc += x;
            }
        }
    }
    __syncthreads();
    const int chunk = s_chunk;
    if (chunk >= 0) {  // uniform
        const uint64_t t = s_t;
        const float *prow = p + ((size_t)b * (k + 1) + n) * V;
        const float *qrow = n < k && !fallback ? q + ((size_t)b * k + n) * V : nullptr;
        const int lo = chunk * kChunk, hi = min(V, lo + kChunk);
        const int v0 = lo + kPer * tid;  // 16 entries per thread, in order
        float r[kPer];
        if (vec4) {
            float4 a[kPer / 4], c[kPer / 4];
#pragma unroll
            for (int j = 0; j < kPer / 4; ++j) {
                const int e = min(v0 + 4 * j, hi - 4);
                a[j] = *reinterpret_cast<const float4 *>(prow + e);
                c[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (qrow) c[j] = *reinterpret_cast<const float4 *>(qrow + e);
            }
#pragma unroll
            for (int j = 0; j < kPer / 4; ++j) {
                const bool in = v0 + 4 * j < hi;
                r[4 * j] = in ? a[j].x - c[j].x : 0.0f;
                r[4 * j + 1] = in ? a[j].y - c[j].y : 0.0f;
                r[4 * j + 2] = in ? a[j].z - c[j].z : 0.0f;
                r[4 * j + 3] = in ? a[j].w - c[j].w : 0.0f;
            }
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const int e = min(v0 + j, hi - 1);
                const float x = qrow ? prow[e] - qrow[e] : prow[e];
                r[j] = v0 + j < hi ? x : 0.0f;
            }
        }
        uint64_t mine = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) mine += sample_weight(r[j]);
        uint64_t tot;
        const uint64_t before = block_scan_u64(mine, s_wave, tot);
        if (mine > 0 && before <= t && t - before < mine) {
            uint64_t acc = before;
            int tok = -1;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                acc += sample_weight(r[j]);
                if (tok < 0 && acc > t) tok = v0 + j;
            }
            s_tok = tok;
        }
    }
    __syncthreads();
    if (tid == 0) {
        accepted[b] = n;
        next_token[b] = s_tok;
    }
}

}  // namespace

int spec_accept_chunks(int vocab) { return (vocab + kChunk - 1) / kChunk; }

hipError_t launch_spec_accept_sample(int B, int k, int vocab, const float *p, const float *q,
                                     const int32_t *drafts, const float *u, int32_t *accepted,
                                     int32_t *next_token, void *workspace, hipStream_t stream) {
    const int n_chunks = spec_accept_chunks(vocab);
    // sums [B][n_chunks][2], then the drafts kept [B]: within the workspace of
    // B (k + 1) n_chunks pairs, as k >= 1
    uint64_t *sums = reinterpret_cast<uint64_t *>(workspace);
    int *kept = reinterpret_cast<int *>(sums + (size_t)B * n_chunks * 2);
    const int vec4 = (vocab % 4 == 0 && (reinterpret_cast<uintptr_t>(p) & 15u) == 0 &&
                      (reinterpret_cast<uintptr_t>(q) & 15u) == 0) ? 1 : 0;
    hipLaunchKernelGGL(sample_chunk_kernel, dim3(n_chunks, B), dim3(kThreads), 0, stream, p, q, drafts, u, k,
                       vocab, n_chunks, vec4, sums, kept);
    hipLaunchKernelGGL(sample_pick_kernel, dim3(B), dim3(kThreads), 0, stream, p, q, u, k, vocab, n_chunks,
                       vec4, sums, kept, accepted, next_token);
    return hipGetLastError();
}

hipError_t launch_spec_accept_greedy(int B, int k, int vocab, const float *logits,
                                     const int32_t *drafts, int32_t *accepted,
                                     int32_t *next_token, void *workspace, hipStream_t stream) {
    const int n_chunks = spec_accept_chunks(vocab);
    float *part_v = reinterpret_cast<float *>(workspace);
    int *part_i = reinterpret_cast<int *>(part_v + (size_t)B * (k + 1) * n_chunks);
    const int vec4 = (vocab % 4 == 0 && (reinterpret_cast<uintptr_t>(logits) & 15u) == 0) ? 1 : 0;
    hipLaunchKernelGGL(argmax_chunk_kernel, dim3(n_chunks, k + 1, B), dim3(kThreads), 0, stream,
                       logits, vocab, n_chunks, vec4, part_v, part_i);
    hipLaunchKernelGGL(accept_kernel, dim3(B), dim3(kThreads), 0, stream, part_v, part_i, k, n_chunks,
                       drafts, accepted, next_token);
    return hipGetLastError();
}

}  // namespace lynx
