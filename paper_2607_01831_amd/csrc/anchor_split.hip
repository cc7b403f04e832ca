// Anchor-phase decode over the anchors of the other split widths (gfx950,
// fp16 matrix cores).
//
// What it computes (Sec. 4.2 Anchor phase with the widths of Sec. 8): the
// uniform 8-bit code c of every K/V element split into an A-bit anchor
// a = c >> R and an R-bit residual (R = 8 - A, A in 2, 4, 6); before the
// residual arrives the anchor alone stands for code 2^R a + (2^R - 1) / 2,
// the middle of the codes it covers, so the cache reads
//   k = z' + a s',  s' = 2^R s,  z' = z + (2^R - 1) / 2 s,
// and one query per sequence attends it: o = softmax(q K^T / sqrt(128)) V.
// Planes hold a token's 128 anchors as a little-endian bit string of 16 A
// bytes (element e at bits e A .. e A + A - 1).
//
// Operands: a field is never unpacked to a value of its own.  Two fields 16
// bits apart in a word are masked where they lie or after one shift, which is
// a pair of fp16 subnormals a 2^(sh - 24) (sh the field's bit position in its
// half): a v_and for two values and a shift for about every fourth.  The
// matrix cores take subnormals exactly, but align a sum's terms by the
// exponent a subnormal is written with, 2^-14: a field in the lowest bits
// loses the bits it is below that (rms error of a sum of 2,048 products of
// 2-bit values at bit 0, 4, 6, 8: 1.4e-5, 2.6e-7, 9.4e-8, 1.0e-7 of the sum's
// spread; plain values 1.0e-7).  So every field's top bit is put at bit 7 or
// above.  The position's factor 2^sh is a
// constant of the dimension, so on the K side it is folded into the query
// with the K scale (y_d = q_d s_d 2^(15 - E - sh), fp16 hi + lo, |y| < 2^15, E
// the exponent of the row's largest fp32 product |q_d s_d| of the group), and
// on the V side into the output's scale at the end.
// V is read transposed by bytes (ds_read_b64_tr_b8): a byte of the plane holds
// the same 4 (A = 2) or 2 (A = 4) dimensions for every token.  For A = 6 a
// byte holds the end of one field and the start of another, which part being
// where a matter of its index mod 3; P V is linear in V, so the low and the
// high part of each byte are multiplied on their own (12 products instead of
// 8, masks per lane) and the parts of a field added at the end.
// The first form (bytes built from the fields, fp16 values 1024 + a less
// 1024) spent about 1,100 instructions on a 32-token tile: a paged batch of 16
// sequences of 4K-32K tokens took 207 us with 2-bit anchors, six times the
// time of its bytes; now 65 us (6-bit anchors, a batch of 16K-64K: 296 -> 178).
// The V scale rides on the softmax weight, pw_t = p_t s_t 2^-Ev in fp16 (Ev
// per wavefront from the largest V scale of its tokens), z' is summed in fp32.
//
// Work split: as in the 4-bit decode, grid = (worker, kv head x chunk of 16
// query heads) or (unit, the same, sequence), the kv head fastest for paged layouts, each worker with an
// equal share of the batch's 512-token units (work_list.h); 4 wavefronts per
// workgroup, two workgroups per CU, wavefront w owning a segment's groups w,
// w + 4, ...  The 32-token tiles stream into a private
// LDS ring by global-to-LDS copies, each with its V metadata, a group's K
// metadata with its first tile; the softmax reference is the maximum of the
// wavefront's first tile, and a wavefront whose sums leave the safe range
// redoes its tiles with a running maximum.  The four wavefronts merge through
// LDS into one partial per segment, and the last workgroup of a (sequence, kv
// head, row chunk) merges those in the same launch; the combine kernel where
// there are more sequences than counters.
#include "f16_ops.h"
#include "lane_ops.h"
#include "lynx_internal.h"
#include "split_merge.h"
#include "work_list.h"

#include <float.h>
#include <math.h>

namespace lynx {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kTile = 32;
constexpr int kRows = 16;  // query rows (heads) per workgroup
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kKMetaBytes = 2 * kHeadDim * 4;  // K scales [128], zeros [128] of a group

// The K operand's place of each dimension.  A lane holds 32 dimensions of a
// token in A words; operand kk (of 4) holds the pairs p = 0..3: dimensions
// first(kk, p) and first(kk, p) + kApart, both at bit shift(kk, p) of a half.
template <int A>
struct KPlace {
    static constexpr int kApart = A == 4 ? 4 : 8;
    static constexpr int first(int kk, int p) { return A == 4 ? 8 * kk + p : 16 * (kk >> 1) + 4 * (kk & 1) + p; }
    static constexpr int shift_of(int d) {  // of dimension d
        for (int kk = 0; kk < 4; ++kk)
            for (int p = 0; p < 4; ++p)
                if (first(kk, p) == d || first(kk, p) + kApart == d) return shift(kk, p);
        return 0;
    }
    static constexpr int shift(int kk, int p) {
        const int j = 4 * (kk & 1) + p;  // field of its half (A = 2), of its 48 bits (A = 6)
        if (A == 2) return j == 2 || j == 4 || j == 6 || j == 7 ? 8 : 6;
        if (A == 4) return 4;
        return j == 1 || j == 4 || j >= 6 ? 4 : 2;
    }
};

// The lane's 32 fields of A bits (words w) -> four operands of fp16 subnormal
// pairs, placed as KPlace says.
template <int A>
__device__ __forceinline__ void k_operands(const uint32_t (&w)[A], u32x4_t (&av)[4]) {
    if constexpr (A == 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t x = w[i], l4 = x << 4, r4 = x >> 4;
            av[2 * i] = u32x4_t{(x << 6) & 0x00C000C0u, l4 & 0x00C000C0u, l4 & 0x03000300u, x & 0x00C000C0u};
            av[2 * i + 1] = u32x4_t{x & 0x03000300u, r4 & 0x00C000C0u, r4 & 0x03000300u, (x >> 6) & 0x03000300u};
        }
    } else if constexpr (A == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t x = w[i];
            av[i] = u32x4_t{(x << 4) & 0x00F000F0u, x & 0x00F000F0u, (x >> 4) & 0x00F000F0u, (x >> 8) & 0x00F000F0u};
        }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            // the first and the second 48 bits of 16 fields, a half of each per word
            const uint32_t x0 = w[3 * i], x1 = w[3 * i + 1], x2 = w[3 * i + 2];
            const uint32_t p0 = __builtin_amdgcn_perm(x1, x0, 0x07060100u);
            const uint32_t p1 = __builtin_amdgcn_perm(x2, x0, 0x05040302u);
            const uint32_t p2 = __builtin_amdgcn_perm(x2, x1, 0x07060100u);
            av[2 * i] = u32x4_t{(p0 << 2) & 0x00FC00FCu, (p0 >> 2) & 0x03F003F0u,
                                ((p0 >> 10) & 0x003C003Cu) | ((p1 & 0x00030003u) << 6), p1 & 0x00FC00FCu};
            av[2 * i + 1] = u32x4_t{(p1 >> 4) & 0x03F003F0u,
                                    ((p1 >> 12) & 0x000C000Cu) | ((p2 & 0x000F000Fu) << 4), p2 & 0x03F003F0u,
                                    (p2 >> 6) & 0x03F003F0u};
        }
    }
}

// A tile in the ring: K rows (32 x 16 A bytes), V rows, V scales [32] and
// zeros [32].  Row t's 16-byte chunk q sits at chunk q ^ swizzle(t), so that
// the lanes of one LDS read phase touch different banks.
template <int A>
struct Ring {
    // 2-bit tiles are small (2.25 KB): three in flight, one for the others
    static constexpr int kDepth = A == 2 ? 4 : 2;
    static constexpr int kRow = 16 * A;
    static constexpr int kPlane = kTile * kRow;
    static constexpr int kVMeta = 2 * kPlane;
    static constexpr int kSlot = kVMeta + 2 * kTile * 4;
    static constexpr int kCopies = kPlane / 1024;  // per plane and tile
    static __device__ __forceinline__ int k_swizzle(int t) {
        return A == 2 ? 0 : A == 4 ? (t >> 1) & 3 : (t >> 3) & 1;
    }
    static __device__ __forceinline__ int v_swizzle(int t) {
        return A == 4 ? ((t >> 2) & 1) | ((t >> 4) & 1) << 1 : (t >> 4) & 1;
    }
};

// LAYOUT 0: one block per sequence (contiguous); 1: paged, block_tokens a
// multiple of 16; 2: any other paging.
// One segment of a worker's share, for kv head h and a chunk of 16 query rows.
// ONE: the segment is a single unit, a group per wavefront.
template <int A, int LAYOUT, int UNIT, bool ONE>
__device__ __forceinline__ void attend_segment(const SplitDecodeArgs &a, const Segment<UNIT> &seg, int h, int chunk,
                                               const int tid) {
    static_assert(UNIT == kWaves, "a group per wavefront and unit");
    using RG = Ring<A>;
    using KP = KPlace<A>;
    constexpr int R = 8 - A;
    constexpr int kDepth = RG::kDepth;
    constexpr int kChunks = A;                  // 16-byte chunks of a row
    constexpr int kParts = A == 2 ? 4 : 2;      // parts a byte is multiplied in
    constexpr int kAcc = kChunks * kParts;      // 8, 8 or 12 accumulators
    constexpr int kCols = 16 * kAcc;            // output columns before parts are added
    constexpr float centre = (float)((1 << R) - 1) * 0.5f;
    const int Hkv = a.geo.Hkv;
    const int lane = tid & 63;
    const int w = tid >> 6;
    const int col = lane & 15;
    const int kg = lane >> 4;
    const int b = seg.b, T = seg.T, g0 = seg.g0, n_groups = seg.n_groups, live = seg.live;
    const int row_base = chunk * kRows;
    const float kscore = kLog2e * rsqrtf((float)kHeadDim);
    const int heads = min(kRows, a.rows_total - row_base);  // live query rows of the chunk
    const size_t orow0 = (size_t)b * a.Hq + (size_t)h * a.G + row_base;
    const size_t prow0 = (size_t)h * a.rows_total + row_base;
    if (n_groups == 0) {
        // an empty sequence: zero output, lse -inf; or, for the combine kernel,
        // (max, sum) = (-inf, 0)
        if (a.fused) {
            for (int idx = tid; idx < heads * (kHeadDim / 4); idx += kThreads)
                *reinterpret_cast<uint2 *>(a.out + (orow0 + idx / (kHeadDim / 4)) * kHeadDim +
                                           4 * (idx % (kHeadDim / 4))) = make_uint2(0u, 0u);
            if (a.lse && tid < heads) a.lse[orow0 + tid] = -INFINITY;
        } else if (tid < heads) {
            a.ws_ml[(prow0 + tid) * a.n_seg + seg.number] = make_float2(-INFINITY, 0.0f);
        }
        return;
    }

    // LDS: 45-60 KB, two workgroups per CU; the epilogue reuses the ring
    constexpr int kRingBytes = kWaves * kDepth * RG::kSlot;
    __shared__ __attribute__((aligned(16))) uint8_t s_ring[kRingBytes];
    __shared__ __attribute__((aligned(16))) uint8_t s_km[kWaves][kKMetaBytes];
    __shared__ __attribute__((aligned(16))) uint8_t s_q[kRows * kHeadDim * 2];  // BF16 query rows
    __shared__ int s_ev[kWaves];
    __shared__ float s_ML[kRows][2];
    static_assert((kWaves * kRows * kCols + 4 * kWaves * kRows) * 4 <= kRingBytes,
                  "the epilogue's arrays must fit in the ring");
    // LAYOUT 1: the blocks of a group's eight 16-token runs, for two groups
    __shared__ int32_t s_ids[LAYOUT == 1 ? kWaves : 1][2][8];
    __shared__ int s_last;

    bool bad = false;
    const int32_t *bt_row = a.block_table + (size_t)b * a.geo.max_blocks;
    const size_t vmeta = ((size_t)b * Hkv + h) * a.geo.max_tokens;
    const size_t kmeta = ((size_t)b * Hkv + h) * a.geo.n_groups * kHeadDim;
    const size_t blk0_rows =
        LAYOUT == 0 ? ((size_t)min(max(bt_row[0], 0), a.geo.num_blocks - 1) * Hkv + h) * a.geo.bt : 0;
    if (LAYOUT == 0 && (bt_row[0] < 0 || bt_row[0] >= a.geo.num_blocks)) bad = true;
    // plane row of token t (tokens past the context are clamped by the caller)
    auto row_of = [&](int t) -> size_t {
        if (LAYOUT == 0) return blk0_rows + (size_t)t;
        const int bi = a.bt_shift >= 0 ? (t >> a.bt_shift) : t / a.geo.bt;
        int blk = bt_row[bi];
        if (blk < 0 || blk >= a.geo.num_blocks) {
            bad = true;
            blk = 0;
        }
        return ((size_t)blk * Hkv + h) * a.geo.bt + (size_t)(t - bi * a.geo.bt);
    };

    // this wavefront's tiles: tile j is tile j % 4 of its group j / 4, the
    // split's group w + 4 (j / 4)
    const int n_mine = ONE ? (n_groups > w ? 1 : 0) : n_groups > w ? (n_groups - w + kWaves - 1) / kWaves : 0;
    auto tile_t0 = [&](int j) { return (g0 + w + kWaves * (j >> 2)) * kKGroup + kTile * (j & 3); };
    auto tile_valid = [&](int j) { return (j >> 2) < n_mine && tile_t0(j) < T; };

    // ---- plain loads, all issued before the first copy: the query rows (16
    // threads per 256-byte row; rows past the chunk's heads repeat the last)
    // and the V scales of the wavefront's first group, for Ev ----
    uint4 q4;
    {
        const int hh = min(row_base + (tid >> 4), a.rows_total - 1);
        const size_t qrow = (size_t)b * a.Hq + (size_t)h * a.G + hh;
        q4 = reinterpret_cast<const uint4 *>(a.q + qrow * kHeadDim)[tid & 15];
    }
    auto v_scale_at = [&](int u, int k) {
        const int t = (g0 + w + kWaves * u) * kKGroup + 64 * k + lane;
        return u < n_mine && t < T ? a.meta.v_scale[vmeta + t] : 0.0f;
    };
    const float vs_first[2] = {v_scale_at(0, 0), v_scale_at(0, 1)};

    // ---- copies into the ring ----
    // Lane l of copy i fills 16-byte slot 64 i + l of the plane's tile: row
    // slot / A, physical chunk slot % A.
    const uint32_t ring = lds_addr(s_ring) + (uint32_t)w * kDepth * RG::kSlot;
    const uint8_t *ring_p = s_ring + (size_t)w * kDepth * RG::kSlot;
    const uint32_t km = lds_addr(&s_km[w][0]);
    int crow[RG::kCopies];          // row of the tile
    uint32_t kq[RG::kCopies], vq[RG::kCopies];  // byte offset of the logical chunk in its row
#pragma unroll
    for (int i = 0; i < RG::kCopies; ++i) {
        const int slot = 64 * i + lane;
        crow[i] = slot / A;
        const int pq = slot - crow[i] * A;
        kq[i] = 16u * (uint32_t)(pq ^ RG::k_swizzle(crow[i]));
        vq[i] = 16u * (uint32_t)(pq ^ RG::v_swizzle(crow[i]));
    }

    // LAYOUT 1: the blocks of the wavefront's group u, run r in lane r, into
    // s_ids, one group ahead of its tiles.  Past the wavefront's groups the
    // entries are clamped and unused.
    auto issue_ids = [&](int u) {
        if (LAYOUT != 1) return;
        const int tr = (g0 + w + kWaves * u) * kKGroup + 16 * lane;
        const int bi = a.bt_shift >= 0 ? (tr >> a.bt_shift) : tr / a.geo.bt;
        if (lane < 8) lds_copy4(bt_row + min(bi, a.geo.max_blocks - 1), lds_addr(&s_ids[LAYOUT == 1 ? w : 0][u & 1][0]));
    };
    // Tile j of this wavefront into ring slot j % kDepth.
    int ids = 0;  // LAYOUT 1: block ids of the group being issued, run r in lane r
    auto issue_tile = [&](int j) {
        const int t0 = __builtin_amdgcn_readfirstlane(tile_t0(j));
        if (LAYOUT == 1 && (j & 3) == 0) ids = s_ids[LAYOUT == 1 ? w : 0][(j >> 2) & 1][lane & 7];
        const uint32_t slot = ring + (uint32_t)(j % kDepth) * RG::kSlot;
        if (LAYOUT == 0 && t0 + kTile <= T) {
            const size_t rb = (blk0_rows + (size_t)t0) * RG::kRow;
#pragma unroll
            for (int i = 0; i < RG::kCopies; ++i) {
                const uint32_t off = (uint32_t)crow[i] * RG::kRow;
                lds_copy16(a.k_anc + rb, off + kq[i], slot + 1024u * i);
                lds_copy16(a.v_anc + rb, off + vq[i], slot + RG::kPlane + 1024u * i);
            }
        } else if (LAYOUT == 1 && t0 + kTile <= T) {
            // two 16-token runs, each inside one block: byte offset of run r's
            // row 0, less 16 r rows
            size_t rb[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int tr = t0 + 16 * r;
                const int bi = a.bt_shift >= 0 ? (tr >> a.bt_shift) : tr / a.geo.bt;
                int blk = __builtin_amdgcn_readlane(ids, 2 * (j & 3) + r);
                if (blk < 0 || blk >= a.geo.num_blocks) {
                    bad = true;
                    blk = 0;
                }
                rb[r] = (((size_t)blk * Hkv + h) * a.geo.bt + (size_t)(tr - bi * a.geo.bt)) * RG::kRow;
            }
#pragma unroll
            for (int i = 0; i < RG::kCopies; ++i) {
                const int r = crow[i] >> 4;
                const size_t at = (r ? rb[1] : rb[0]) + (uint32_t)((crow[i] & 15) * RG::kRow);
                lds_copy16(a.k_anc + at + kq[i], slot + 1024u * i);
                lds_copy16(a.v_anc + at + vq[i], slot + RG::kPlane + 1024u * i);
            }
        } else {
            // per-lane rows; rows past the context repeat the last token
#pragma unroll
            for (int i = 0; i < RG::kCopies; ++i) {
                const size_t at = row_of(min(t0 + crow[i], T - 1)) * RG::kRow;
                lds_copy16(a.k_anc + at + kq[i], slot + 1024u * i);
                lds_copy16(a.v_anc + at + vq[i], slot + RG::kPlane + 1024u * i);
            }
        }
        // V scale (lanes 0..31) and zero (lanes 32..63) of the tile's tokens;
        // tokens past the context repeat the last one
        {
            const int t = min(t0 + (lane & 31), T - 1);
            lds_copy4((lane < 32 ? a.meta.v_scale : a.meta.v_zero) + vmeta + t, slot + RG::kVMeta);
        }
        // K scale (lanes 0..31) and zero (lanes 32..63) of the group
        if ((j & 3) == 0) {
            const int g = g0 + min(w + kWaves * (j >> 2), n_groups - 1);
            const float *src = (lane < 32 ? a.meta.k_scale : a.meta.k_zero) + kmeta + (size_t)g * kHeadDim;
            lds_copy16(src + 4 * (lane & 31), km);
            if (!ONE && n_mine > 1) issue_ids((j >> 2) + 1);  // (a wavefront's only group has no next)
        }
    };
    static_assert(kDepth - 1 < 4, "a group's K metadata may not arrive before the last group's fold");
    auto issue_first = [&]() {
        if (n_mine > 0) {
#pragma unroll
            for (int c = 0; c < kDepth - 1; ++c) issue_tile(c);  // all in the first group
        }
    };
    // The first group's block ids are needed before its tiles; elsewhere the
    // first tiles go out before the plain loads above are waited for.
    if (LAYOUT == 1) {
        issue_ids(0);
        wait_vmcnt<0>();
    }
    issue_first();

    // The exponent of the largest V scale, from the wavefront's first group: a
    // later, larger one gives weights above 1, and past the fp16 range an
    // infinity that sends the wavefront to the slow path, which looks at all
    // of its scales, as does a first group without any.
    int Ev = 0;
    auto set_ev = [&](float vm) {
        vm = max_kg(row16_max(vm));
        Ev = 0;
        if (vm > 0.0f) frexpf(vm, &Ev);
        Ev = max(Ev, -100);
        return vm > 0.0f;
    };
    auto set_ev_all = [&]() {
        float vm = 0.0f;
        for (int u = 0; u < n_mine; ++u) vm = fmax2(vm, fmax2(v_scale_at(u, 0), v_scale_at(u, 1)));
        set_ev(vm);
    };
    if (!set_ev(fmax2(vs_first[0], vs_first[1]))) set_ev_all();
    reinterpret_cast<uint4 *>(s_q)[tid] = q4;
    __syncthreads();

    // ---- per-wavefront online-softmax state: lane (col = query row, kg);
    // the reference carries the 2^-Ev factor of the V weights ----
    float m_run = -INFINITY, m_ref = -INFINITY, l_part = 0.0f, ob_part = 0.0f;
    f32x4_t acc[kAcc];
    auto reset_state = [&]() {
        m_run = m_ref = -INFINITY;
        l_part = ob_part = 0.0f;
#pragma unroll
        for (int n = 0; n < kAcc; ++n) acc[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    reset_state();
    // Rows past the chunk's heads repeat the last one; their results go nowhere.
    // Fold of a group (K scales and zeros from the K-metadata buffer, BF16 query
    // rows from LDS): the operands y_d, hi and lo, the products' scale
    // bsc = kscore 2^(24 + R + E - 15) and the bias bb = kscore sum_d q_d z'_d.
    u32x4_t bq[8];
    float bsc = 0.0f, bb = 0.0f;
    auto fold = [&]() {
        const float4 *ks = reinterpret_cast<const float4 *>(&s_km[w][0]) + 8 * kg;
        const float4 *kz = ks + kHeadDim / 4;
        const uint4 *qp = reinterpret_cast<const uint4 *>(s_q + col * (kHeadDim * 2) + 64 * kg);
        float y[32], mx = 0.0f, bias = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint4 u = qp[k];
            const float4 s0 = ks[2 * k], s1 = ks[2 * k + 1], z0 = kz[2 * k], z1 = kz[2 * k + 1];
            const uint32_t qw[4] = {u.x, u.y, u.z, u.w};
            const float sv[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
            const float zv[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float q = e & 1 ? bf16_hi(qw[e / 2]) : bf16_lo(qw[e / 2]);
                y[8 * k + e] = q * sv[e];
                bias = fmaf(q, fmaf(centre, sv[e], zv[e]), bias);
            }
#pragma unroll
            for (int e = 0; e < 8; e += 2) mx = fmax3_abs(mx, y[8 * k + e], y[8 * k + e + 1]);
            asm volatile("" : "+v"(bias));  // summed here: later, all its terms would be held in registers
        }
        mx = max_kg(mx);
        int E = 0;
        if (mx > 0.0f) frexpf(mx, &E);
#pragma unroll
        for (int d = 0; d < 32; ++d) y[d] = ldexpf(y[d], 15 - E - KP::shift_of(d));
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            u32x4_t hi, lo;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const float y0 = y[KP::first(kk, p)], y1 = y[KP::first(kk, p) + KP::kApart];
                const uint32_t hp = pack_f16(y0, y1);
                hi[p] = hp;
                lo[p] = pack_f16(less_f16_lo(y0, hp), less_f16_hi(y1, hp));  // exact differences
            }
            bq[2 * kk] = hi;
            bq[2 * kk + 1] = lo;
        }
        // positive and finite: times the -inf of a token past the context and
        // times a product of 0 it must not be a NaN
        bsc = __builtin_amdgcn_fmed3f(ldexpf(kscore, 9 + R + E), FLT_MIN, FLT_MAX);
        bb = kscore * sum_kg(bias);
    };

    // This lane's K words of a tile: dims 32 kg .. + 31 of token 16 r + col.
    const uint32_t kswz = (uint32_t)RG::k_swizzle(col);
    auto load_k = [&](const uint8_t *slot_p, int r, uint32_t (&kw)[A]) {
        const uint8_t *row = slot_p + (16 * r + col) * RG::kRow;
        if constexpr (A == 4) {
            const uint4 u = *reinterpret_cast<const uint4 *>(row + 16 * ((uint32_t)kg ^ kswz));
            kw[0] = u.x;
            kw[1] = u.y;
            kw[2] = u.z;
            kw[3] = u.w;
        } else {
#pragma unroll
            for (int i = 0; i < A / 2; ++i) {
                const uint32_t unit = (uint32_t)(A / 2 * kg + i);  // 8-byte units
                const uint2 u = *reinterpret_cast<const uint2 *>(row + 16 * ((unit >> 1) ^ kswz) + 8 * (unit & 1));
                kw[2 * i] = u.x;
                kw[2 * i + 1] = u.y;
            }
        }
    };
    // Products of tile j (scores are bsc times them, plus bb): lane (col, kg)
    // gets token t0 + 16 r + 4 kg + i of query row col in x[4 r + i]; tokens
    // past the context get -inf.
    auto tile_products = [&](const uint8_t *slot_p, int j, float (&x)[8]) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            uint32_t kw[A];
            load_k(slot_p, r, kw);
            u32x4_t av[4];
            k_operands<A>(kw, av);
            f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                sc = mfma_f16(av[kk], bq[2 * kk + 0], sc);
                sc = mfma_f16(av[kk], bq[2 * kk + 1], sc);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * r + i] = sc[i];
        }
        const int t0 = tile_t0(j);
        if (t0 + kTile > T) {
            asm volatile("" ::: "memory");  // keep the masking out of full tiles
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int t = t0 + 16 * (i >> 2) + 4 * kg + (i & 3);
                x[i] = t < T ? x[i] : -INFINITY;
            }
        }
    };
    // the row's largest score of a tile (bsc > 0)
    auto tile_max = [&](const float (&x)[8]) {
        return fmaf(max_kg(fmax3(fmax3(x[0], x[1], x[2]), fmax3(x[3], x[4], x[5]), fmax2(x[6], x[7]))), bsc, bb);
    };

    // Transposed V reads: lane (col, kg) names row tau(kg, col / 2) =
    // 16 (col / 8) + 4 kg + (col / 2) % 4 and 8-byte half col % 2 of a chunk,
    // and receives byte col of the chunk for the tokens tau(kg, 0..7).
    uint32_t v_off[kChunks];
    {
        const int tr = 16 * (col >> 3) + 4 * kg + ((col >> 1) & 3);
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
            v_off[c] = (uint32_t)(RG::kPlane + tr * RG::kRow + 16 * (c ^ RG::v_swizzle(tr)) + 8 * (col & 1));
    }
    // A = 6: the low part of byte 16 c + col is 6, 4 or 2 bits by its index
    // mod 3; it is moved up by 4, 4 or 6 and masked, the rest is masked in place.
    uint32_t lowm[3] = {0, 0, 0}, highm[3] = {0, 0, 0}, up[3] = {0, 0, 0};
    if (A == 6) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int m = (c + col) % 3;
            lowm[c] = m == 0 ? 0x03F003F0u : m == 1 ? 0x00F000F0u : 0x00C000C0u;
            highm[c] = m == 0 ? 0x00C000C0u : m == 1 ? 0x00F000F0u : 0x00FC00FCu;
            up[c] = m == 2 ? 6 : 4;
        }
    }
    // Part p of the bytes of four tokens (word v): pairs of tokens 0, 2 (e) and
    // 1, 3 (o), both at the part's place in a half.
    auto part_of = [&](uint32_t v, int c, int p, uint32_t &e, uint32_t &o) {
        if constexpr (A == 2) {  // at bits 8, 6, 8, 6
            const uint32_t m = p & 1 ? 0x00C000C0u : 0x03000300u;
            e = (p == 0 ? v << 8 : p == 3 ? v : v << 4) & m;
            o = (p == 0 ? v : p == 3 ? v >> 8 : v >> 4) & m;
        } else if constexpr (A == 4) {  // at bit 4
            e = (p == 0 ? v << 4 : v) & 0x00F000F0u;
            o = (p == 0 ? v >> 4 : v >> 8) & 0x00F000F0u;
        } else if (p == 0) {
            e = (v << up[c % 3]) & lowm[c % 3];
            o = (v >> (8 - up[c % 3])) & lowm[c % 3];
        } else {
            e = v & highm[c % 3];
            o = (v >> 8) & highm[c % 3];
        }
    };
    // Weights against m_ref, then P V for the tile.
    auto tile_accumulate = [&](const uint8_t *slot_p, const float (&x)[8]) {
        const float *vsm = reinterpret_cast<const float *>(slot_p + RG::kVMeta) + 4 * kg;
        const float4 vs0 = *reinterpret_cast<const float4 *>(vsm);
        const float4 vs1 = *reinterpret_cast<const float4 *>(vsm + 16);
        const float4 vz0 = *reinterpret_cast<const float4 *>(vsm + kTile);
        const float4 vz1 = *reinterpret_cast<const float4 *>(vsm + kTile + 16);
        const float vsv[8] = {vs0.x, vs0.y, vs0.z, vs0.w, vs1.x, vs1.y, vs1.z, vs1.w};
        const float vzv[8] = {vz0.x, vz0.y, vz0.z, vz0.w, vz1.x, vz1.y, vz1.z, vz1.w};
        const float c0 = bb - m_ref;
        float pw[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float p = __builtin_amdgcn_exp2f(fmaf(x[i], bsc, c0));
            l_part += p;
            ob_part = fmaf(p, fmaf(centre, vsv[i], vzv[i]), ob_part);
            pw[i] = p * vsv[i];
        }
        // token pairs as the masks leave them: (0, 2), (1, 3), (4, 6), (5, 7)
        const u32x4_t pa = {pack_f16_rne(pw[0], pw[2]), pack_f16_rne(pw[1], pw[3]), pack_f16_rne(pw[4], pw[6]),
                            pack_f16_rne(pw[5], pw[7])};
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const intx2_t vt = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                (__attribute__((address_space(3))) intx2_t *)(slot_p + v_off[c]));
            const uint32_t v0 = (uint32_t)vt[0], v1 = (uint32_t)vt[1];
#pragma unroll
            for (int p = 0; p < kParts; ++p) {
                uint32_t e0, o0, e1, o1;
                part_of(v0, c, p, e0, o0);
                part_of(v1, c, p, e1, o1);
                acc[kParts * c + p] = mfma_f16(pa, u32x4_t{e0, o0, e1, o1}, acc[kParts * c + p]);
            }
        }
    };

    // Fast path: a fixed softmax reference, the maximum of the wavefront's
    // first tile; the next tiles are in flight while one is attended.
    auto copies_at = [](int c) { return 2 * RG::kCopies + ((c & 3) == 0 ? (LAYOUT == 1 ? 3 : 2) : 1); };
    for (int u = 0; u < (ONE ? min(n_mine, 1) : n_mine); ++u) {
        const bool next_group = !ONE && u + 1 < n_mine;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = 4 * u + c;
            if (c + kDepth - 1 < 4 || next_group) issue_tile(j + kDepth - 1);
            // tile j is in once only the later tiles' copies may remain in flight
            int later_here = 0, later_next = 0;
#pragma unroll
            for (int k = 1; k < kDepth; ++k) {
                later_next += copies_at(c + k);
                if (c + k < 4) later_here += copies_at(c + k);
            }
            if (next_group) {
                wait_vmcnt_folded(later_next);
            } else {
                wait_vmcnt_folded(later_here);
            }
            const uint8_t *slot_p = ring_p + (c % kDepth) * RG::kSlot;
            if (c == 0) fold();
            if (tile_valid(j)) {
                float x[8];
                tile_products(slot_p, j, x);
                if (j == 0) {
                    m_run = tile_max(x);
                    m_ref = m_run + (float)Ev;
                }
                tile_accumulate(slot_p, x);
            }
            // the slot and the K-metadata buffer are rewritten by later
            // copies: their reads must be done
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    }
    bool unsafe = !(l_part < 1e30f) || !(fabsf(ob_part) < 1e30f);
#pragma unroll
    for (int n = 0; n < kAcc; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) unsafe |= !(fabsf(acc[n][i]) < 1e30f);
    if (__any(unsafe)) {
        // Slow path (this wavefront only): running maximum with rescaling,
        // one tile fetched and waited for at a time.
        reset_state();
        set_ev_all();
        issue_ids(0);
        wait_vmcnt<0>();
        for (int j = 0; j < 4 * n_mine; ++j) {
            issue_tile(j);
            wait_vmcnt<0>();
            const uint8_t *slot_p = ring_p + (j % kDepth) * RG::kSlot;
            if ((j & 3) == 0) fold();
            if (tile_valid(j)) {
                float x[8];
                tile_products(slot_p, j, x);
                const float mx = tile_max(x);
                if (__any(mx > m_run)) {
                    const float m_new = fmaxf(mx, m_run);
                    const float alpha = (m_run == -INFINITY) ? 0.0f : exp2f(m_run - m_new);
                    m_run = m_new;
                    m_ref = m_new + (float)Ev;
                    l_part *= alpha;
                    ob_part *= alpha;
                    float af[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) af[i] = __shfl(alpha, 4 * kg + i);
#pragma unroll
                    for (int n = 0; n < kAcc; ++n)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[n][i] *= af[i];
                }
                tile_accumulate(slot_p, x);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    }
    wait_vmcnt<0>();  // no copy may land in the ring once it is reused below

    // ---- per-wavefront totals -> LDS (still scaled by 2^-Ev) ----
    __syncthreads();  // every wavefront is done with its ring
    // ring reused: o [wave][row][kCols] (A = 2, 4: dims in order; A = 6: the
    // low parts of bytes 0..95, then their high parts), then max, sum,
    // sum p z' and merge factors [wave][row]
    float *s_o = reinterpret_cast<float *>(s_ring);
    float(*s_m)[kRows] = reinterpret_cast<float(*)[kRows]>(s_o + kWaves * kRows * kCols);
    float(*s_l)[kRows] = s_m + kWaves;
    float(*s_ob)[kRows] = s_l + kWaves;
    float(*s_f)[kRows] = s_ob + kWaves;
    {
        const float l = sum_kg(l_part);
        const float ob = sum_kg(ob_part);
        if (kg == 0) {
            s_m[w][col] = m_run;
            s_l[w][col] = l;
            s_ob[w][col] = ob;
        }
        constexpr float kUnit = (float)(1u << 24) * (float)(1 << R);  // the operand's 2^-24, s' = 2^R s
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (4 * kg + i < heads) {
                float *o = s_o + (w * kRows + 4 * kg + i) * kCols;
#pragma unroll
                for (int c = 0; c < kChunks; ++c) {
                    if constexpr (A == 2) {
                        *reinterpret_cast<float4 *>(o + 4 * (16 * c + col)) =
                            make_float4(acc[4 * c][i] * (kUnit / 256.0f), acc[4 * c + 1][i] * (kUnit / 64.0f),
                                        acc[4 * c + 2][i] * (kUnit / 256.0f), acc[4 * c + 3][i] * (kUnit / 64.0f));
                    } else if constexpr (A == 4) {
                        *reinterpret_cast<float2 *>(o + 2 * (16 * c + col)) =
                            make_float2(acc[2 * c][i] * (kUnit / 16.0f), acc[2 * c + 1][i] * (kUnit / 16.0f));
                    } else {
                        o[16 * c + col] = acc[2 * c][i] * (kUnit / 16.0f);  // a byte's third kind: at 64
                        o[96 + 16 * c + col] = acc[2 * c + 1][i] * kUnit;
                    }
                }
            }
        }
    }
    if (lane == 0) s_ev[w] = Ev;
    const bool any_bad = __syncthreads_or(bad);
    if (tid < heads) {
        float M = -INFINITY;
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) M = fmaxf(M, s_m[ww][tid]);
        float L = 0.0f;
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) {
            const float f = (M == -INFINITY || s_m[ww][tid] == -INFINITY)
                                ? 0.0f
                                : exp2f(s_m[ww][tid] - M) * ldexpf(1.0f, s_ev[ww]);
            s_f[ww][tid] = f;
            L = fmaf(s_l[ww][tid], f, L);
        }
        s_ML[tid][0] = M;
        s_ML[tid][1] = any_bad ? NAN : L;
    }
    __syncthreads();
    // the sequence's partials, from its first on, rows n_seg partials apart
    const size_t pseg0 = prow0 * a.n_seg + seg.number0;
    const uint32_t prows = (uint32_t)(heads - 1) * a.n_seg + live;
    const __amdgpu_buffer_rsrc_t pair_o = buffer_rsrc(a.ws_o + pseg0 * kHeadDim, prows * kHeadDim * 4);
    const __amdgpu_buffer_rsrc_t pair_ml = buffer_rsrc(a.ws_ml + pseg0, prows * 8);
    const bool merge = a.fused && live > 1;
    for (int idx = tid; idx < heads * (kHeadDim / 4); idx += kThreads) {
        const int rr = idx / (kHeadDim / 4);
        const int d4 = idx % (kHeadDim / 4);
        float4 O = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) {
            const float f = s_f[ww][rr];
            const float ob = s_ob[ww][rr];
            const float *row = s_o + (ww * kRows + rr) * kCols;
            float4 o;
            if constexpr (A == 6) {
                // dims 4 d4 .. + 3 lie in bytes 3 d4 .. + 2: field 0 is byte 0's
                // low six bits; field 1 byte 0's top two (at bit 6) and byte 1's
                // low four; field 2 byte 1's top four (at bit 4) and byte 2's low
                // two; field 3 byte 2's top six (at bit 2)
                const float *lo = row + 3 * d4, *hi = row + 96 + 3 * d4;
                o = make_float4(lo[0], fmaf(hi[0], 1.0f / 64.0f, 4.0f * lo[1]),
                                fmaf(hi[1], 1.0f / 16.0f, 4.0f * lo[2]), 0.25f * hi[2]);
            } else {
                o = reinterpret_cast<const float4 *>(row)[d4];
            }
            O.x = fmaf(o.x + ob, f, O.x);
            O.y = fmaf(o.y + ob, f, O.y);
            O.z = fmaf(o.z + ob, f, O.z);
            O.w = fmaf(o.w + ob, f, O.w);
        }
        if (any_bad) O = make_float4(NAN, NAN, NAN, NAN);
        if (merge) {
            const uint32_t sp = (uint32_t)rr * a.n_seg + (seg.number - seg.number0);
            store16_agent(pair_o, (sp * kHeadDim + 4 * d4) * 4, O);
            if (d4 == 0) store8_agent(pair_ml, sp * 8, make_float2(s_ML[rr][0], s_ML[rr][1]));
        } else if (a.fused) {  // the whole sequence is this worker's
            write_row4(a.out, a.lse, orow0 + rr, d4, O, s_ML[rr][0], s_ML[rr][1]);
        } else {
            const size_t pi = (prow0 + rr) * a.n_seg + seg.number;
            reinterpret_cast<float4 *>(a.ws_o + pi * kHeadDim)[d4] = O;
            if (d4 == 0) a.ws_ml[pi] = make_float2(s_ML[rr][0], s_ML[rr][1]);
        }
    }
    if (!merge) return;

    // ---- split merge: count in; the chunk's last workgroup merges ----
    unsigned *ctr = a.counters + (((size_t)b * Hkv + h) * a.row_chunks + chunk) * kCounterStride;
    if (!last_to_arrive(ctr, live, &s_last)) return;
    if (heads <= 4)
        merge_pair<4>(a, pair_o, pair_ml, orow0, heads, live, s_ring);
    else if (heads <= 8)
        merge_pair<8>(a, pair_o, pair_ml, orow0, heads, live, s_ring);
    else
        merge_pair<16>(a, pair_o, pair_ml, orow0, heads, live, s_ring);
}

// LANES: a lane for each sequence (B <= 64).
template <int A, int LAYOUT, int UNIT, bool LANES>
__global__ __launch_bounds__(kThreads, 2) void anchor_split_decode_batch_kernel(SplitDecodeArgs a) {
    if (LANES) __builtin_assume(a.B > 1 && a.B <= 64);
    const int worker = LAYOUT == 0 ? blockIdx.x : blockIdx.y;
    const int hc = LAYOUT == 0 ? blockIdx.y : blockIdx.x;
    const WorkList<UNIT, true> list(a.seq_lens, a.B, a.max_seq_len, a.workers);
    Segment<UNIT> seg;
    if (!seg.start(list, worker)) return;
    for (;;) {
        attend_segment<A, LAYOUT, UNIT, false>(a, seg, fresh_uniform(hc % a.geo.Hkv), fresh_uniform(hc / a.geo.Hkv), fresh_tid());
        if (!seg.next(list, worker)) return;
        __syncthreads();  // the segment's LDS is free again
    }
}

// A single sequence of more units than workers: one segment each, no walk.
template <int A, int LAYOUT, int UNIT>
__global__ __launch_bounds__(kThreads, 2) void anchor_split_decode_long_kernel(SplitDecodeArgs a) {
    const int worker = LAYOUT == 0 ? blockIdx.x : blockIdx.y;
    const int hc = LAYOUT == 0 ? blockIdx.y : blockIdx.x;
    const WorkList<UNIT, false> list(a.seq_lens, 1, a.max_seq_len, a.workers);
    Segment<UNIT> seg;
    if (!seg.start(list, worker)) return;
    attend_segment<A, LAYOUT, UNIT, false>(a, seg, hc % a.geo.Hkv, hc / a.geo.Hkv, threadIdx.x);
}

// A unit per workgroup, for sequence blockIdx.z.
template <int A, int LAYOUT, int UNIT>
__global__ __launch_bounds__(kThreads, 2) void anchor_split_decode_kernel(SplitDecodeArgs a) {
    const int unit = LAYOUT == 0 ? blockIdx.x : blockIdx.y;
    const int hc = LAYOUT == 0 ? blockIdx.y : blockIdx.x;
    Segment<UNIT> seg;
    if (!seg.set_unit(a.seq_lens, a.max_seq_len, a.direct, blockIdx.z, unit)) return;
    attend_segment<A, LAYOUT, UNIT, true>(a, seg, hc % a.geo.Hkv, hc / a.geo.Hkv, threadIdx.x);
}

template <int A, int LAYOUT>
void launch_layout(const SplitDecodeArgs &args, dim3 grid, hipStream_t stream) {
    if (args.direct)
        hipLaunchKernelGGL((anchor_split_decode_kernel<A, LAYOUT, kWorkUnit>), grid, dim3(kThreads), 0, stream, args);
    else if (args.B == 1)
        hipLaunchKernelGGL((anchor_split_decode_long_kernel<A, LAYOUT, kWorkUnit>), grid, dim3(kThreads), 0, stream, args);
    else if (args.B <= 64)
        hipLaunchKernelGGL((anchor_split_decode_batch_kernel<A, LAYOUT, kWorkUnit, true>), grid, dim3(kThreads), 0,
                           stream, args);
    else
        hipLaunchKernelGGL((anchor_split_decode_batch_kernel<A, LAYOUT, kWorkUnit, false>), grid, dim3(kThreads), 0,
                           stream, args);
}

template <int A>
void launch_a(const SplitDecodeArgs &args, dim3 grid, hipStream_t stream) {
    if (args.geo.max_blocks == 1)
        launch_layout<A, 0>(args, grid, stream);
    else if (args.geo.bt % 16 == 0)
        launch_layout<A, 1>(args, grid, stream);
    else
        launch_layout<A, 2>(args, grid, stream);
}

}  // namespace

hipError_t launch_anchor_split_decode(const SplitDecodeArgs &args, hipStream_t stream) {
    const bool paged = args.geo.max_blocks != 1;
    if (args.workers < 1 || args.workers > 65535) return hipErrorInvalidValue;
    const unsigned hc = (unsigned)(args.geo.Hkv * ((args.rows_total + kRows - 1) / kRows));
    // kv head fastest for paged layouts (the kernel reads the grid the same way)
    const unsigned n = args.direct ? args.direct : args.workers, nz = args.direct ? args.B : 1;
    const dim3 grid = paged ? dim3(hc, n, nz) : dim3(n, hc, nz);
    switch (args.anchor_bits) {
        case 2:
            launch_a<2>(args, grid, stream);
            break;
        case 4:
            launch_a<4>(args, grid, stream);
            break;
        case 6:
            launch_a<6>(args, grid, stream);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace lynx
