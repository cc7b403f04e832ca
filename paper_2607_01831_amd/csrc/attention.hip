// Attention over the split-stream KV cache for gfx950: planning and launch of
// the anchor-only decode (Sec. 4.2 Anchor phase; anchor_decode.hip) and of
// the verification pass over the merged 8-bit cache (Sec. 4.3; verify.hip),
// both O = softmax(q K^T / sqrt(128)) V (Sec. 2) cut along the context,
// and the combine kernel that merges their partials (max, sum,
// unnormalised output) and attends the BF16 tail: the drafts, causal among
// themselves, in verification, and the generated tokens in decode.
#include "lane_ops.h"
#include "lynx_internal.h"
#include "split_merge.h"
#include "work_list.h"

#include <float.h>
#include <math.h>

#include <algorithm>
#include <mutex>

namespace lynx {
namespace {

constexpr float kLog2e = 1.4426950408889634f;

struct AttnArgs {
    Geometry geo;
    int B, Hq, nq, G, max_seq_len;
    int rows_total, direct, workers, n_seg, max_live;
    int tail;             // attend the BF16 tail
    int tail_count;       // tokens of the tail every query sees; -1: query i sees i + 1 (drafts)
    int tail_stride;      // tail tokens stored per sequence in k_new / v_new
    const int32_t *seq_lens;
    const uint16_t *q;
    const uint16_t *k_new;
    const uint16_t *v_new;
    float *ws_o;    // [Hkv][rows_total][n_seg][128]
    float2 *ws_ml;  // [Hkv][rows_total][n_seg]
};

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ void unpack8_bf16(const uint4 &u, float *x) {
    x[0] = bf16_lo(u.x); x[1] = bf16_hi(u.x);
    x[2] = bf16_lo(u.y); x[3] = bf16_hi(u.y);
    x[4] = bf16_lo(u.z); x[5] = bf16_hi(u.z);
    x[6] = bf16_lo(u.w); x[7] = bf16_hi(u.w);
}

constexpr int kCombineThreads = 256;

// One workgroup per (row, kv head, sequence), for many partials and few rows:
// merge the sequence's partials ("splits") and the BF16 tail tokens,
// normalise, round to BF16, write lse.
// Thread (split group sg, float4 column d4) folds every 8th split into a
// running (max, sum, output), loading kBatch splits' partial outputs and
// (max, sum) pairs together (8 when 64 splits or fewer, so no load is a
// clamped repeat; 16 above), then every 8th tail token the same way, as a
// partial of weight 1.  The 8 running triples meet in LDS.  Every load the
// kernel needs first (the first kBatch splits' partials, the tail's values,
// and the query and tail keys for the tail scores) is issued before any of
// them is used, so the kernel waits for memory once for up to 8 kBatch
// splits.
template <int kBatch>
__global__ __launch_bounds__(kCombineThreads) void attn_combine_kernel(AttnArgs a, uint16_t *out,
                                                                       float *lse) {
    const int gr = blockIdx.x;
    const int h = blockIdx.y;
    const int b = blockIdx.z;
    const int tid = threadIdx.x;
    const int Hkv = a.geo.Hkv;
    constexpr int kGroups = kCombineThreads / (kHeadDim / 4);  // 8 split groups
    constexpr int kTailMax = 64;                   // tail tokens attended at most
    constexpr int kTailPer = kTailMax / kGroups;   // per split group
    __shared__ float4 s_acc[kGroups][kHeadDim / 4];
    __shared__ float s_m[kGroups][kHeadDim / 4], s_l[kGroups][kHeadDim / 4];
    __shared__ float s_ts[kTailMax];  // tail scores (log2 units)

    // query row gr <-> (query qi, head qg); with a tail, query qi also sees
    // the BF16 tokens of the tail: drafts 0..qi in verification (causal among
    // the drafts), all tail_count generated tokens in decode
    const int qi = gr / a.G;
    const int qg = gr % a.G;
    const size_t qrow = ((size_t)b * a.nq + qi) * a.Hq + (size_t)h * a.G + qg;
    const int n_tail = a.tail ? (a.tail_count < 0 ? qi + 1 : a.tail_count) : 0;

    const int d4 = tid % (kHeadDim / 4);
    const int sg = tid / (kHeadDim / 4);
    // this thread's tail values: tokens sg, sg + 8, ... (dims 4 d4 .. + 3)
    uint2 tvw[kTailPer];
    if (n_tail > 0) {
#pragma unroll
        for (int u = 0; u < kTailPer; ++u) {
            const int j = min(sg + kGroups * u, n_tail - 1);
            tvw[u] = *reinterpret_cast<const uint2 *>(
                a.v_new + (((size_t)b * a.tail_stride + j) * Hkv + h) * kHeadDim + 4 * d4);
        }
    }
    // The sequence's partials stand from the row's number seg0 on (work_list.h).
    // Where that is known without the list, the first batch is loaded, up to
    // the most there can be, before the sequence's length is in.
    using List = WorkList<kWorkUnit, false>;
    int n = a.max_live, seg0 = b * a.direct;
    const bool listed = !a.direct && a.B > 1;
    if (listed) List(a.seq_lens, a.B, a.max_seq_len, a.workers).partials(b, seg0, n);
    const size_t base = ((size_t)h * a.rows_total + gr) * a.n_seg + seg0;
    // a batch of partials: splits s0, s0 + 8, ... (clamped to the last split)
    float4 v[kBatch];
    float2 ml[kBatch];
    bool live[kBatch];
    auto load_batch = [&](int s0) {
        const float4 *o4 = reinterpret_cast<const float4 *>(a.ws_o) + base * (kHeadDim / 4) + d4;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int s = min(s0 + kGroups * u, n - 1);
            v[u] = o4[(size_t)s * (kHeadDim / 4)];
            ml[u] = a.ws_ml[base + s];
        }
    };
    auto set_live = [&](int s0) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) live[u] = s0 + kGroups * u < n;
    };
    load_batch(sg);
    if (!listed) n = min(a.max_live, List::units(max(0, min(a.seq_lens[b], a.max_seq_len))));
    set_live(sg);
    if (n_tail > 0) {
        // tail scores, 16 tokens per pass: thread (token tid / 16, dims
        // 8 (tid % 16) .. + 7), summed over the 16 lanes of a token
        const int piece = tid & 15;
        float qv[8];
        unpack8_bf16(*reinterpret_cast<const uint4 *>(a.q + qrow * kHeadDim + 8 * piece), qv);
        const float sm = kLog2e * rsqrtf((float)kHeadDim);
        uint4 kw[kTailMax / 16];
#pragma unroll
        for (int p = 0; p < kTailMax / 16; ++p) {
            const int j = min(16 * p + (tid >> 4), n_tail - 1);
            kw[p] = *reinterpret_cast<const uint4 *>(
                a.k_new + (((size_t)b * a.tail_stride + j) * Hkv + h) * kHeadDim + 8 * piece);
        }
#pragma unroll
        for (int p = 0; p < kTailMax / 16; ++p) {
            const int j = 16 * p + (tid >> 4);
            float kv[8];
            unpack8_bf16(kw[p], kv);
            float d = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) d = fmaf(qv[e], kv[e], d);
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) d += __shfl_xor(d, off);
            if (piece == 0 && j < n_tail) s_ts[j] = d * sm;
        }
        __syncthreads();
    }

    float m_t = -INFINITY, l_t = 0.0f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    bool nan = false;
    // fold N partials (max mlv.x, sum mlv.y, output vv) into the running triple
    auto fold = [&](const auto &vv, auto &mlv, const auto &lv) {
        constexpr int N = sizeof(lv) / sizeof(lv[0]);
        float mb = m_t;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            if (!lv[u]) mlv[u] = make_float2(-INFINITY, 0.0f);
            mb = fmaxf(mb, mlv[u].x);
        }
        const float sc = m_t == -INFINITY ? 0.0f : exp2f(m_t - mb);
        acc.x *= sc;
        acc.y *= sc;
        acc.z *= sc;
        acc.w *= sc;
        l_t *= sc;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const float e = mlv[u].x == -INFINITY ? 0.0f : exp2f(mlv[u].x - mb);
            nan |= isnan(mlv[u].y);
            l_t = fmaf(mlv[u].y, e, l_t);
            // a split with weight 0 may hold no partial output at all
            const float4 x = e != 0.0f ? vv[u] : make_float4(0.f, 0.f, 0.f, 0.f);
            acc.x = fmaf(x.x, e, acc.x);
            acc.y = fmaf(x.y, e, acc.y);
            acc.z = fmaf(x.z, e, acc.z);
            acc.w = fmaf(x.w, e, acc.w);
        }
        m_t = mb;
    };
    for (int s0 = sg; s0 < n; s0 += kGroups * kBatch) {
        if (s0 != sg) {
            load_batch(s0);
            set_live(s0);
        }
        fold(v, ml, live);
    }
    // the tail tokens: partials (score, 1, value)
    if (n_tail > 0) {
        float4 tv[kTailPer];
        float2 tml[kTailPer];
        bool tlive[kTailPer];
#pragma unroll
        for (int u = 0; u < kTailPer; ++u) {
            const int j = sg + kGroups * u;
            tlive[u] = j < n_tail;
            tv[u] = make_float4(bf16_lo(tvw[u].x), bf16_hi(tvw[u].x), bf16_lo(tvw[u].y), bf16_hi(tvw[u].y));
            tml[u] = make_float2(tlive[u] ? s_ts[j] : -INFINITY, 1.0f);
        }
        fold(tv, tml, tlive);
    }
    s_acc[sg][d4] = acc;
    s_m[sg][d4] = m_t;
    s_l[sg][d4] = nan ? NAN : l_t;
    __syncthreads();
    if (sg == 0) {
        float M = -INFINITY;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) M = fmaxf(M, s_m[g][d4]);
        float4 O = make_float4(0.f, 0.f, 0.f, 0.f);
        float L = 0.0f;
        bool any_nan = false;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const float f = s_m[g][d4] == -INFINITY ? 0.0f : exp2f(s_m[g][d4] - M);
            // (of weight 0: it may hold a weightless tail token's infinity)
            const float4 o = f != 0.0f ? s_acc[g][d4] : make_float4(0.f, 0.f, 0.f, 0.f);
            O.x = fmaf(o.x, f, O.x);
            O.y = fmaf(o.y, f, O.y);
            O.z = fmaf(o.z, f, O.z);
            O.w = fmaf(o.w, f, O.w);
            any_nan |= isnan(s_l[g][d4]);
            L = fmaf(s_l[g][d4], f, L);
        }
        write_row4(out, lse, qrow, d4, O, M, any_nan ? NAN : L);
    }
}

// The same for few partials or many rows: one workgroup
// per (ROWS rows, kv head, sequence), a row per 32 threads.  Thread (row r,
// float4 column d4) folds all of the row's partials, 8 loaded at a time, so
// nothing meets in LDS but the tail, whose keys and values the rows share: a
// thread holds a quarter of a token's key against every row's query, and the
// values are staged once.  A workgroup per row reads the tail once a row, and
// spends a third of its time on its first wait (verification of 5 drafts for 16
// paged sequences: 17.1 -> 8.1 us).
// FIND: how the row's partials are found: 0 without the list, 1 by the list of a
// batch whose sequences have a lane each, 2 by any list (32 sequences of 1K-8K:
// 5.5 us, 5.7 by one kernel for all three).
template <int ROWS, int FIND>
__global__ __launch_bounds__(32 * ROWS) void attn_combine_rows_kernel(AttnArgs a, uint16_t *out, float *lse) {
    if (FIND == 1) __builtin_assume(a.B > 1 && a.B <= 64);
    constexpr int kThreads = 32 * ROWS;
    constexpr int kTailMax = 64;
    constexpr int kTokens = kThreads / 4;  // tail tokens scored per pass, four threads each
    constexpr int kPasses = kTailMax / kTokens;
    constexpr int kValues = kTailMax * (kHeadDim / 8) / kThreads;  // 16-byte value pieces per thread
    constexpr int kBatch = 8;
    const int h = blockIdx.y;
    const int b = blockIdx.z;
    const int tid = threadIdx.x;
    const int Hkv = a.geo.Hkv;
    const int d4 = tid % 32;
    const int r = tid / 32;
    const int row0 = blockIdx.x * ROWS;
    const bool row_live = row0 + r < a.rows_total;
    const int gr = min(row0 + r, a.rows_total - 1);
    const int qi = gr / a.G;
    const size_t qrow = ((size_t)b * a.nq + qi) * a.Hq + (size_t)h * a.G + gr % a.G;
    // tail tokens of this row, and of any row of the workgroup
    const int n_tail = a.tail ? (a.tail_count < 0 ? qi + 1 : a.tail_count) : 0;
    const int tail_most =
        a.tail ? (a.tail_count < 0 ? (min(row0 + ROWS, a.rows_total) - 1) / a.G + 1 : a.tail_count) : 0;
    __shared__ __attribute__((aligned(16))) uint4 s_v[kTailMax * (kHeadDim / 8)];  // tail values
    // queries, a thread's 32 dims 4 floats past the last's: other banks
    __shared__ __attribute__((aligned(16))) float s_q[ROWS][kHeadDim + 16];
    __shared__ float s_t[ROWS][kTailMax];  // tail scores (log2 units), then weights

    // the length of the lane's sequence for the list, else of this one
    const int own = a.seq_lens[FIND == 0 ? b : min((int)(threadIdx.x & 63), a.B - 1)];
    // ---- the tail's loads ----
    uint4 kw[kPasses][4];
    if (tail_most > 0) {
        const size_t t0 = (size_t)b * a.tail_stride * Hkv + h;
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int j = min(kTokens * p + tid / 4, tail_most - 1);
            const uint4 *k = reinterpret_cast<const uint4 *>(a.k_new + (t0 + (size_t)j * Hkv) * kHeadDim) + 4 * (tid % 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) kw[p][e] = k[e];
        }
#pragma unroll
        for (int i = 0; i < kValues; ++i) {
            const int piece = kThreads * i + tid, j = piece / (kHeadDim / 8);
            if (j < tail_most)
                s_v[piece] = reinterpret_cast<const uint4 *>(
                    a.v_new + (t0 + (size_t)j * Hkv) * kHeadDim)[piece % (kHeadDim / 8)];
        }
        const uint2 qw = reinterpret_cast<const uint2 *>(a.q + qrow * kHeadDim)[d4];
        *reinterpret_cast<float4 *>(&s_q[r][4 * d4 + 4 * (d4 / 8)]) =
            make_float4(bf16_lo(qw.x), bf16_hi(qw.x), bf16_lo(qw.y), bf16_hi(qw.y));
    }
    // ---- the row's partials (work_list.h): n of them from segment seg0 on ----
    int n, seg0;
    if (FIND == 0) {
        n = WorkList<kWorkUnit, false>::units(max(0, min(own, a.max_seq_len)));
        seg0 = b * a.direct;
    } else {
        const WorkList<kWorkUnit, false> list(a.seq_lens, a.B, a.max_seq_len, a.workers, own);
        list.partials(b, seg0, n);
    }
    const size_t base = ((size_t)h * a.rows_total + gr) * a.n_seg + seg0;
    const float4 *o4 = reinterpret_cast<const float4 *>(a.ws_o) + base * (kHeadDim / 4) + d4;
    float M = -INFINITY, L = 0.0f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < n; s0 += kBatch) {
        float4 v[kBatch];
        float2 ml[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int s = min(s0 + u, n - 1);
            v[u] = o4[(size_t)s * (kHeadDim / 4)];
            ml[u] = a.ws_ml[base + s];
        }
        float mb = M;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (s0 + u >= n) ml[u] = make_float2(-INFINITY, 0.0f);
            mb = fmaxf(mb, ml[u].x);
        }
        const float sc = M == -INFINITY ? 0.0f : exp2f(M - mb);
        acc.x *= sc;
        acc.y *= sc;
        acc.z *= sc;
        acc.w *= sc;
        L *= sc;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const float e = ml[u].x == -INFINITY ? 0.0f : exp2f(ml[u].x - mb);
            L = fmaf(ml[u].y, e, L);  // a NaN sum (bad block id) stays NaN
            // a partial of weight 0 may hold no output at all
            const float4 x = e != 0.0f ? v[u] : make_float4(0.f, 0.f, 0.f, 0.f);
            acc.x = fmaf(x.x, e, acc.x);
            acc.y = fmaf(x.y, e, acc.y);
            acc.z = fmaf(x.z, e, acc.z);
            acc.w = fmaf(x.w, e, acc.w);
        }
        M = mb;
    }
    // ---- the tail ----
    if (tail_most > 0) {  // uniform
        __syncthreads();  // queries and values are staged
        const float sm = kLog2e * rsqrtf((float)kHeadDim);
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            if (kTokens * p >= tail_most) break;
            float kv[32];
#pragma unroll
            for (int e = 0; e < 4; ++e) unpack8_bf16(kw[p][e], kv + 8 * e);
#pragma unroll
            for (int rr = 0; rr < ROWS; ++rr) {
                const float4 *q = reinterpret_cast<const float4 *>(&s_q[rr][36 * (tid % 4)]);
                float d = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float4 x = q[e];
                    d = fmaf(x.x, kv[4 * e], d);
                    d = fmaf(x.y, kv[4 * e + 1], d);
                    d = fmaf(x.z, kv[4 * e + 2], d);
                    d = fmaf(x.w, kv[4 * e + 3], d);
                }
                d += dpp<0xB1>(d);
                d += dpp<0x4E>(d);  // over the token's four threads
                if (tid % 4 == 0) s_t[rr][kTokens * p + tid / 4] = d * sm;
            }
        }
        __syncthreads();
        // the row's 32 threads: tokens d4 and d4 + 32
        const float t0 = d4 < n_tail ? s_t[r][d4] : -INFINITY;
        const float t1 = d4 + 32 < n_tail ? s_t[r][d4 + 32] : -INFINITY;
        const float Mt = fmaxf(M, row_max<32>(fmaxf(t0, t1)));
        const float p0 = t0 == -INFINITY ? 0.0f : exp2f(t0 - Mt);
        const float p1 = t1 == -INFINITY ? 0.0f : exp2f(t1 - Mt);
        s_t[r][d4] = p0;
        s_t[r][d4 + 32] = p1;
        const float sc = M == -INFINITY ? 0.0f : exp2f(M - Mt);
        L = fmaf(L, sc, row_sum<32>(p0 + p1));
        M = Mt;
        __syncthreads();
        acc.x *= sc;
        acc.y *= sc;
        acc.z *= sc;
        acc.w *= sc;
        const uint2 *v2 = reinterpret_cast<const uint2 *>(s_v) + d4;
#pragma unroll 4
        for (int j = 0; j < n_tail; ++j) {
            const float p = s_t[r][j];
            // a token of weight 0 may hold an infinity
            const uint2 w = p != 0.0f ? v2[j * (kHeadDim / 4)] : make_uint2(0u, 0u);
            acc.x = fmaf(p, bf16_lo(w.x), acc.x);
            acc.y = fmaf(p, bf16_hi(w.x), acc.y);
            acc.z = fmaf(p, bf16_lo(w.y), acc.z);
            acc.w = fmaf(p, bf16_hi(w.y), acc.w);
        }
    }
    if (row_live) write_row4(out, lse, qrow, d4, acc, M, L);
}

// Compute units of the current device (0 if unknown), queried once per device.
int compute_units() {
    constexpr int kMaxDevices = 64;
    static std::once_flag once[kMaxDevices];
    static int cus[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    std::call_once(once[dev], [dev]() {
        int n = 0;
        cus[dev] = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess ? n : 0;
    });
    return cus[dev];
}

}  // namespace

namespace {

// Workgroups of the attention kernels that the device holds at once, two per CU.
long long resident_workgroups() {
    const int cus = compute_units();
    return 2ll * (cus > 0 ? cus : 256);
}

// 512-token units of a sequence of at most T tokens (work_list.h).
long long work_units(int T) { return T > 0 ? ((long long)T + kWorkUnit * kKGroup - 1) / (kWorkUnit * kKGroup) : 1; }

constexpr size_t kPartialBytes = kHeadDim * sizeof(float) + sizeof(float2);

}  // namespace

// One round of workgroups, whatever the batch: as many workers per (kv head,
// row chunk) as the chip holds at once, each with an equal share of the
// batch's units.  Against splits of up to 2048 tokens per workgroup (several
// rounds, a combine kernel): see work_list.h.
AttnPlan plan_attention(KvMode mode, const Geometry &g, int B, int Hq, int nq, int max_seq_len,
                        size_t most) {
    AttnPlan p{};
    p.rows_total = nq * (Hq / g.Hkv);
    const int tile = mode == KvMode::kCodes && p.rows_total > 16 ? 32 : 16;  // rows per workgroup
    const long long chunks = (p.rows_total + tile - 1) / tile;
    const long long slots = resident_workgroups();
    const long long units = (long long)B * work_units(max_seq_len);
    const size_t row_bytes = (size_t)g.Hkv * p.rows_total * kPartialBytes;
    // A workgroup per unit of the longest sequence where those of all sequences
    // fit one round: nothing to balance, and the list's start and walk cost 1 us
    // of a 10 us call (decode, 4 sequences of 4K: 10.7 us, by the list 11.5;
    // verification of 2 drafts, 2 of 2K: 14.0 and 15.3; 6-bit anchors, 8 of 4K:
    // 15.2 and 16.4).  Past one round the list balances (decodes of one
    // sequence of 33000: 17.2 us, by direct workgroups 19.9; 5 of 8K: 18.5 and 19.7;
    // 5 ragged ones of up to 8K, not all units there: 13.7 and 12.9).
    const bool direct = units * g.Hkv * chunks <= slots &&
                        (most == SIZE_MAX || kCounterBytes + units * row_bytes <= most);
    p.direct = direct ? (int)work_units(max_seq_len) : 0;
    long long w = slots / (g.Hkv * chunks);
    w = direct || w > units ? units : w;
    // fewer partials where the workspace is given (lynx_attn_anchor_decode_noalloc)
    if (!direct && most < SIZE_MAX) {
        const long long fit = (long long)((most - kCounterBytes) / row_bytes) - (B - 1);
        w = w < fit ? w : fit;
    }
    // the shares are found in 32-bit arithmetic (workers x units)
    if (units * w > 0xffffffffll) w = 0xffffffffll / units;
    p.workers = (int)(w > 1 ? w : 1);
    p.n_seg = p.workers + (B > 0 && !direct ? B - 1 : 0);
    p.max_live = (int)(work_units(max_seq_len) < p.workers ? work_units(max_seq_len) : p.workers);
    p.o_bytes = (size_t)g.Hkv * p.rows_total * p.n_seg * kHeadDim * sizeof(float);
    p.ml_bytes = (size_t)g.Hkv * p.rows_total * p.n_seg * sizeof(float2);
    p.row_chunks = (p.rows_total + 15) / 16;
    p.counters_fit = (long long)B * g.Hkv * p.row_chunks <= kCounters;
    return p;
}

// rows_total x workers is at most a row tile per resident workgroup (a row per
// kv head where there are more of those), and at most a partial per unit; the
// sum with a partial per sequence grows with each of the arguments, so a
// workspace serves every smaller call too.
size_t attention_workspace_bound(const Geometry &g, int B, int Hq, int nq, int max_seq_len) {
    const size_t rows = (size_t)nq * (Hq / g.Hkv) * g.Hkv;
    const size_t resident = (size_t)resident_workgroups() * (nq * (Hq / g.Hkv) > 16 ? 32 : 16);
    const size_t by_slots = resident > rows ? resident : rows;
    const size_t by_units = rows * B * (size_t)work_units(max_seq_len);
    return kCounterBytes + ((by_slots < by_units ? by_slots : by_units) + rows * B) * kPartialBytes;
}

// A partial per split of every sequence, splits of 512 tokens, longer (to 2048)
// while 1024 workgroups remain, and to 8192 where a contiguous batch of at most
// 8 heads per kv head then fits two workgroups per CU: the need of a plan of
// fixed splits, by which the no-allocation decode has taken and refused calls.
// The work list needs less (plan_attention makes any call within the limit fit
// the scratch); the limit stays, so that no call changes sides, and is reported,
// so that a caller who asks first is told the same.
size_t decode_limit_bytes(const Geometry &g, int B, int Hq, int max_seq_len) {
    const int G = Hq / g.Hkv;
    const long long heads = (long long)g.Hkv * B;
    auto splits = [&](long long tokens) { return max_seq_len > 0 ? (max_seq_len + tokens - 1) / tokens : 1ll; };
    long long tokens = 512;
    while (tokens < (G > 8 ? 512 : 2048) && splits(2 * tokens) * heads >= 1024 && max_seq_len > 0) tokens *= 2;
    const int cus = compute_units();
    if (g.max_blocks == 1 && G <= 8 && cus > 0)
        for (long long st = tokens; st <= 8192; st *= 2)
            if (splits(st) * heads <= 2ll * cus) {
                tokens = st;
                break;
            }
    return kCounterBytes + (size_t)(heads * G * splits(tokens)) * kPartialBytes;
}

template <int ROWS>
static void launch_combine_rows(int find, const AttnArgs &a, uint16_t *out, float *lse, hipStream_t stream) {
    const dim3 grid((a.rows_total + ROWS - 1) / ROWS, a.geo.Hkv, a.B), block(32 * ROWS);
    if (find == 0)
        hipLaunchKernelGGL((attn_combine_rows_kernel<ROWS, 0>), grid, block, 0, stream, a, out, lse);
    else if (find == 1)
        hipLaunchKernelGGL((attn_combine_rows_kernel<ROWS, 1>), grid, block, 0, stream, a, out, lse);
    else
        hipLaunchKernelGGL((attn_combine_rows_kernel<ROWS, 2>), grid, block, 0, stream, a, out, lse);
}

hipError_t launch_attention(KvMode mode, const Geometry &g, const AttnPlan &plan, int B, int Hq,
                            int nq, int max_seq_len, const int32_t *seq_lens,
                            const int32_t *block_table, const uint8_t *k_plane,
                            const uint8_t *v_plane, MetaPtrs meta, const uint16_t *q,
                            const uint16_t *k_new, const uint16_t *v_new, int tail_count,
                            uint16_t *out,
                            float *lse, void *workspace, hipStream_t stream, int anchor_bits) {
    if (B == 0) return hipSuccess;
    AttnArgs a;
    a.geo = g;
    a.B = B;
    a.Hq = Hq;
    a.nq = nq;
    a.G = Hq / g.Hkv;
    a.max_seq_len = max_seq_len;
    a.rows_total = plan.rows_total;
    a.direct = plan.direct;
    a.workers = plan.workers;
    a.n_seg = plan.n_seg;
    a.max_live = plan.max_live;
    a.tail = k_new != nullptr ? 1 : 0;
    a.tail_count = mode == KvMode::kCodes ? -1 : tail_count;
    a.tail_stride = mode == KvMode::kCodes ? nq : tail_count;
    a.seq_lens = seq_lens;
    a.q = q;
    a.k_new = k_new;
    a.v_new = v_new;
    a.ws_o = reinterpret_cast<float *>(reinterpret_cast<char *>(workspace) + kCounterBytes);
    a.ws_ml = reinterpret_cast<float2 *>(reinterpret_cast<char *>(workspace) + kCounterBytes +
                                         plan.o_bytes);
    if (mode == KvMode::kAnchor && nq == 1) {
        // matrix-core decode over the anchor nibbles
        DecodeArgs d;
        d.geo = g;
        d.B = B;
        d.Hq = Hq;
        d.G = a.G;
        d.max_seq_len = max_seq_len;
        d.direct = plan.direct;
        d.workers = plan.workers;
        d.chunk_heads = a.G < 16 ? a.G : 16;
        d.bt_shift = -1;
        for (int sh = 0; sh < 31; ++sh)
            if ((1 << sh) == g.bt) d.bt_shift = sh;
        d.seq_lens = seq_lens;
        d.block_table = block_table;
        d.k_anc = k_plane;
        d.v_anc = v_plane;
        d.meta = meta;
        d.q = q;
        d.ws_o = a.ws_o;
        d.ws_ml = a.ws_ml;
        d.rows_total = plan.rows_total;
        d.n_seg = plan.n_seg;
        // Without a tail the last workgroup of each (sequence, kv head, head
        // chunk) merges its partials itself: no second launch.  The merge
        // holds up to two partials' (max, sum) per thread: 256 / GP threads per
        // row, GP = 4, 8 or 16 rows padded.
        const int gp = d.chunk_heads <= 4 ? 4 : d.chunk_heads <= 8 ? 8 : 16;
        d.fused = (k_new == nullptr && plan.counters_fit && plan.max_live <= 2 * (256 / gp)) ? 1 : 0;
        d.row_chunks = plan.row_chunks;
        d.counters = reinterpret_cast<unsigned *>(workspace);
        d.out = out;
        d.lse = lse;
        const int chunks = (a.G + d.chunk_heads - 1) / d.chunk_heads;
        hipError_t e = launch_anchor_decode_mfma(d, chunks, stream);
        if (e != hipSuccess) return e;
        if (d.fused) return hipSuccess;
    } else if (mode == KvMode::kAnchorSplit && nq == 1 && k_new == nullptr) {
        // matrix-core decode over A-bit anchors; the combine kernel below
        // merges its splits
        SplitDecodeArgs d;
        d.geo = g;
        d.B = B;
        d.Hq = Hq;
        d.G = a.G;
        d.max_seq_len = max_seq_len;
        d.anchor_bits = anchor_bits;
        d.direct = plan.direct;
        d.workers = plan.workers;
        d.bt_shift = -1;
        for (int sh = 0; sh < 31; ++sh)
            if ((1 << sh) == g.bt) d.bt_shift = sh;
        d.rows_total = plan.rows_total;
        d.n_seg = plan.n_seg;
        d.seq_lens = seq_lens;
        d.block_table = block_table;
        d.k_anc = k_plane;
        d.v_anc = v_plane;
        d.meta = meta;
        d.q = q;
        d.ws_o = a.ws_o;
        d.ws_ml = a.ws_ml;
        // the merge in the same launch, under the 4-bit decode's rule
        const int gp = a.G <= 4 ? 4 : a.G <= 8 ? 8 : 16;
        d.fused = (plan.counters_fit && plan.max_live <= 2 * (256 / gp)) ? 1 : 0;
        d.row_chunks = plan.row_chunks;
        d.counters = reinterpret_cast<unsigned *>(workspace);
        d.out = out;
        d.lse = lse;
        hipError_t e = launch_anchor_split_decode(d, stream);
        if (e != hipSuccess) return e;
        if (d.fused) return hipSuccess;
    } else if (mode == KvMode::kCodes) {
        // matrix-core verification over the context ...
        VerifyArgs v;
        v.geo = g;
        v.B = B;
        v.Hq = Hq;
        v.G = a.G;
        v.nq = nq;
        v.max_seq_len = max_seq_len;
        v.rows_total = plan.rows_total;
        v.direct = plan.direct;
        v.workers = plan.workers;
        v.n_seg = plan.n_seg;
        v.bt_shift = -1;
        for (int sh = 0; sh < 31; ++sh)
            if ((1 << sh) == g.bt) v.bt_shift = sh;
        v.seq_lens = seq_lens;
        v.block_table = block_table;
        v.k_codes = k_plane;
        v.v_codes = v_plane;
        v.meta = meta;
        v.q = q;
        v.ws_o = a.ws_o;
        v.ws_ml = a.ws_ml;
        hipError_t e = launch_verify_mfma(v, stream);
        if (e != hipSuccess) return e;
        // the BF16 draft tail is attended by the combine kernel below
    } else {
        return hipErrorInvalidValue;  // anchor attention with several queries: no entry point asks for it
    }
    // Many partials a sequence: a row per workgroup, 8 threads deep in them, while
    // those workgroups are resident at once; else the rows share workgroups.
    // Many are more than the 8 that a thread loads together where the partials
    // are found without the list (2 sequences of 8K, 2 drafts, 128 rows of 16
    // partials: 16.8 us, shared 18.2; 2048 such rows: 33.9, shared 26.4), and
    // more than 16 with it (8 of 1.5K-5K, 2 drafts, 9 partials: 20.6, shared
    // 19.9; 2 of 19K, 33 partials: 26.1, shared 29.8).  A single sequence's rows
    // of more than 16 go alone whatever their number (32K, 20 drafts, 640 rows:
    // 46.2, shared 47.7).
    const int each = plan.direct ? plan.direct : std::min(plan.max_live, plan.workers / B + 1);
    const long long rows_all = (long long)plan.rows_total * g.Hkv * B;
    const bool deep = (each > (plan.direct ? 8 : 16) && rows_all <= resident_workgroups()) || (B == 1 && each > 16);
    if (!deep) {
        const int find = plan.direct ? 0 : B > 1 && B <= 64 ? 1 : 2;
        if (plan.rows_total <= 4)
            launch_combine_rows<4>(find, a, out, lse, stream);
        else
            launch_combine_rows<8>(find, a, out, lse, stream);
    } else if (plan.max_live <= 64) {
        hipLaunchKernelGGL(attn_combine_kernel<8>, dim3(plan.rows_total, g.Hkv, B), dim3(kCombineThreads),
                           0, stream, a, out, lse);
    } else {
        hipLaunchKernelGGL(attn_combine_kernel<16>, dim3(plan.rows_total, g.Hkv, B), dim3(kCombineThreads),
                           0, stream, a, out, lse);
    }
    return hipGetLastError();
}

}  // namespace lynx
