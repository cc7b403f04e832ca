// Verification attention on matrix cores (gfx950 MFMA, fp16 operands).
//
// What it computes (Sec. 4.3; attention of Sec. 2): the k draft queries of a
// sequence attend, in one pass, over the merged 8-bit cache, with K and V
// reconstructed as zero + code * scale.  This kernel covers the context
// tokens; the combine kernel of attention.hip merges its splits and attends
// the drafts' own BF16 K/V (the causal tail) as one more partial.
//
// Why matrix cores: with k * G query rows per kv head (32 for 8 drafts and
// G = 4) every context token costs 2 x 128 x 32 multiply-adds against 272
// bytes, above what fp32 vector arithmetic sustains at HBM speed; the
// contraction is dense, so Q K^T and P V run as v_mfma_f32_16x16x32_f16.
//
// Exactness of the operands:
//  * a code byte c stands as the fp16 subnormal c 2^-24, one v_perm per two
//    values; the 2^24 goes into the scales below.
//  * the K scale is folded into the query per 128-token group: the products
//    q_d s_d in fp32, scaled by the exponent E of the row's largest one,
//    y_d = q_d s_d 2^(15 - E), |y| < 2^15, as fp16 hi + lo through two MFMAs;
//    the zeros enter a per-(group, row) bias sum_d q_d z_d.  E comes from the
//    products themselves: a large query value where K is flat, or a large K
//    channel where the query is small, leaves the others their bits.
//  * the V scale is folded into the softmax weight, pw_t = p_t s_t 2^-Ev
//    (fp16, rounded to nearest; Ev per wavefront, so that pw <= 1 while p <= 1,
//    and a weight beyond the fp16 range becomes infinite and sends the
//    wavefront to the running-maximum path); sum_t p_t z_t is summed in fp32.
//    The 2^-Ev factor rides on the softmax reference, so l, sum p z and the
//    products all carry it and one multiply restores it when the wavefronts
//    are merged.
//
// Work split: grid = (worker, kv head x chunk of 16 RT query rows), as many
// workers as the chip holds at once (two workgroups of 4 wavefronts per CU),
// each with an equal share of the batch's 512-token units (work_list.h), a
// segment per sequence it touches; or, where one round holds them all, (unit,
// kv head x chunk, sequence).  Wavefront w owns a segment's groups w, w + 4, ...
// and serves all RT row tiles from each of their 32-token tiles, so every
// K/V byte is fetched once per workgroup and the query fold of a group
// (y for the wavefront's own MFMA operand lanes) lives in its registers:
// no barrier inside the loop.  Tiles, each with its V metadata, stream
// into a private 2-slot LDS ring by global-to-LDS copies, one tile ahead
// of the one being attended (no registers held by loads in flight); a
// group's K metadata rides with its first tile, and the query rows are
// copied into LDS once.  At the end the four wavefronts merge through LDS
// into one partial per row and segment.
#include "f16_ops.h"
#include "lane_ops.h"
#include "lynx_internal.h"
#include "work_list.h"

#include <float.h>
#include <math.h>

namespace lynx {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kTile = 32;      // tokens per wavefront step
constexpr float kLog2e = 1.4426950408889634f;

constexpr int kDepth = 2;                          // ring slots per wavefront
constexpr int kTileBytes = kTile * kCodeRow;       // one plane's 32 rows: 4 KB
constexpr int kVMetaOff = 2 * kTileBytes;          // V scale[32] | V zero[32] of the tile
constexpr int kSlotBytes = kVMetaOff + 2 * kTile * 4;  // 8.25 KB
constexpr int kKMetaBytes = 2 * kHeadDim * 4;      // K scale[128] | K zero[128] of a group

// K tile rows in LDS: 16-byte chunk q of row t sits at chunk q ^ (t & 7), so
// the 8 lanes of one ds_read_b128 phase (8 consecutive rows, same chunk)
// touch 8 different bank groups.
__device__ __forceinline__ uint32_t k_slot(int t, int q) {
    return (uint32_t)t * kCodeRow + (uint32_t)((q ^ (t & 7)) * 16);
}

// LAYOUT 0: one block per sequence; 1: paged, block_tokens a multiple of 16;
// 2: any other paging.  RT: 16-row query tiles per workgroup (1 or 2), all
// served by every wavefront.  UNIT: 128-token groups per unit of the work list.
// One segment of a worker's share, for kv head h and a chunk of 16 RT rows.
// ONE: the segment is a single unit, a group per wavefront.
template <int RT, int LAYOUT, int UNIT, bool ONE>
__device__ __forceinline__ void verify_segment(const VerifyArgs &a, const Segment<UNIT> &seg, int h, int chunk,
                                               const int tid) {
    constexpr int kRows = RT * 16;
    constexpr int NQ = kWaves;             // wavefront w takes groups w, w + 4, ...
    static_assert(UNIT == NQ, "a group per wavefront and unit");
    const int Hkv = a.geo.Hkv;
    const int lane = tid & 63;
    const int w = tid >> 6;
    const int col = lane & 15;
    const int kg = lane >> 4;
    const int gq = w;  // this wavefront's groups: gq, gq + NQ, ...
    const int b = seg.b, T = seg.T, g0 = seg.g0, n_groups = seg.n_groups;
    const int row_base = chunk * kRows;  // first query row of the workgroup
    const float kscore = kLog2e * rsqrtf((float)kHeadDim);

    // query row r <-> (draft r / G, head r % G); its partial-output row
    auto partial_index = [&](int r) {
        return ((size_t)h * a.rows_total + r) * a.n_seg + seg.number;
    };

    if (n_groups == 0) {  // an empty sequence: (max, sum) = (-inf, 0)
        for (int r = tid; r < kRows; r += kThreads)
            if (row_base + r < a.rows_total) a.ws_ml[partial_index(row_base + r)] = make_float2(-INFINITY, 0.0f);
        return;
    }

    // LDS: under 80 KB for RT = 2, so two workgroups share a CU; the
    // epilogue reuses the ring
    __shared__ __attribute__((aligned(16))) uint8_t s_ring[kWaves * kDepth * kSlotBytes];
    __shared__ __attribute__((aligned(16))) uint8_t s_km[kWaves][kKMetaBytes];
    __shared__ __attribute__((aligned(16))) uint8_t s_q[kRows * kHeadDim * 2];  // BF16 query rows
    __shared__ int s_ev[kWaves];
    __shared__ float s_ML[kRows][2];
    static_assert(kWaves * kRows * (kHeadDim + 4) * 4 <= kWaves * kDepth * kSlotBytes,
                  "the epilogue's arrays must fit in the ring");
    // LAYOUT 1: the blocks of a group's eight 16-token runs, for two groups
    __shared__ int32_t s_ids[LAYOUT == 1 ? kWaves : 1][2][8];

    bool bad = false;
    const int32_t *bt_row = a.block_table + (size_t)b * a.geo.max_blocks;
    const size_t vmeta = ((size_t)b * Hkv + h) * a.geo.max_tokens;
    const size_t kmeta = ((size_t)b * Hkv + h) * a.geo.n_groups * kHeadDim;
    const size_t blk0_rows =
        LAYOUT == 0 ? ((size_t)min(max(bt_row[0], 0), a.geo.num_blocks - 1) * Hkv + h) * a.geo.bt : 0;
    if (LAYOUT == 0 && (bt_row[0] < 0 || bt_row[0] >= a.geo.num_blocks)) bad = true;

    // Row index (not bytes) of token t in the code planes.
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

    // This wavefront's tiles: tile j is tile j % 4 of its group j / 4, the
    // split's group gq + NQ (j / 4).
    const int n_mine = ONE ? (n_groups > gq ? 1 : 0) : n_groups > gq ? (n_groups - gq + NQ - 1) / NQ : 0;  // its groups
    auto group_of = [&](int j) { return gq + NQ * (j >> 2); };
    auto tile_t0 = [&](int j) { return (g0 + group_of(j)) * kKGroup + kTile * (j & 3); };
    auto tile_valid = [&](int j) { return (j >> 2) < n_mine && tile_t0(j) < T; };

    // ---- the exponent of the largest V scale, from the wavefront's first
    // group (plain loads, consumed before the first copy): a later, larger one
    // gives weights above 1, and past the fp16 range an infinity that sends the
    // wavefront to the slow path, which looks at all of its scales, as does a
    // first group without any ----
    int Ev = 0;
    auto v_scale_at = [&](int u, int k) {
        const int t = (g0 + gq + NQ * u) * kKGroup + 64 * k + lane;
        return u < n_mine && t < T ? a.meta.v_scale[vmeta + t] : 0.0f;
    };
    auto set_ev = [&](float vm) {
        vm = max_kg(row16_max(vm));
        Ev = 0;
        if (vm > 0.0f) frexpf(vm, &Ev);
        // V scales below 2^-100 contribute below 255 * 2^-100 per token; the
        // clamp keeps 2^-Ev, and so the weights p 2^-Ev, finite
        Ev = max(Ev, -100);
        return vm > 0.0f;
    };
    auto set_ev_all = [&]() {
        float vm = 0.0f;
        for (int u = 0; u < n_mine; ++u) vm = fmax2(vm, fmax2(v_scale_at(u, 0), v_scale_at(u, 1)));
        set_ev(vm);
    };
    if (!set_ev(fmax2(v_scale_at(0, 0), v_scale_at(0, 1)))) set_ev_all();
    // every plain load has been consumed (Ev depends on all of them): nothing
    // of the compiler's own is in flight once the copies start
    asm volatile("" ::"v"(Ev) : "memory");
    wait_vmcnt<0>();

    // ---- copies into the ring ----
    // Lane l of a 1 KB tile copy fills row 8 i + l / 8, physical chunk l % 8
    // of the slot (i = instruction); these are the logical chunks it fetches.
    const int crow = lane >> 3;
    const int kq = (lane & 7) ^ crow;  // K, and V rows 0..15
    const uint32_t ring = lds_addr(s_ring) + (uint32_t)w * kDepth * kSlotBytes;
    const uint8_t *ring_p = s_ring + (size_t)w * kDepth * kSlotBytes;
    // copies per tile: 4 K + 4 V + 1 V metadata; with a group's first tile
    // also its K metadata (into the wavefront's K-metadata buffer) and, for
    // LAYOUT 1, the next group's block ids
    const uint32_t km = lds_addr(&s_km[w][0]);
    constexpr int kFirst = LAYOUT == 1 ? 11 : 10;  // copies of a group's first tile

    // LAYOUT 1: the blocks of the wavefront's group u, run r in lane r, into
    // s_ids, one group ahead of its tiles, whose copies then take them by readlane
    // instead of waiting on a block-table load each.  Past the
    // wavefront's groups the entries are clamped and unused.
    auto issue_ids = [&](int u) {
        if (LAYOUT != 1) return;
        const int tr = (g0 + gq + NQ * u) * kKGroup + 16 * lane;
        const int bi = a.bt_shift >= 0 ? (tr >> a.bt_shift) : tr / a.geo.bt;
        if (lane < 8) lds_copy4(bt_row + min(bi, a.geo.max_blocks - 1), lds_addr(&s_ids[LAYOUT == 1 ? w : 0][u & 1][0]));
    };

    // Tile j of this wavefront into ring slot j % kDepth.
    int ids = 0;  // LAYOUT 1: block ids of the group being issued, run r in lane r
    auto issue_tile = [&](int j) {
        const int t0 = __builtin_amdgcn_readfirstlane(tile_t0(j));
        if (LAYOUT == 1 && (j & 3) == 0) ids = s_ids[LAYOUT == 1 ? w : 0][(j >> 2) & 1][lane & 7];
        const uint32_t slot = ring + (uint32_t)(j % kDepth) * kSlotBytes;
        if (LAYOUT != 2 && t0 + kTile <= T) {
            // two 16-token runs, each inside one block
#pragma unroll
            for (int run = 0; run < 2; ++run) {
                size_t row0;
                if (LAYOUT == 0) {
                    row0 = blk0_rows + (size_t)(t0 + 16 * run);
                } else {
                    const int tr = t0 + 16 * run;
                    const int bi = a.bt_shift >= 0 ? (tr >> a.bt_shift) : tr / a.geo.bt;
                    // run 2 (j % 4) + run of the wavefront's group j / 4
                    int blk = __builtin_amdgcn_readlane(ids, 2 * (j & 3) + run);
                    if (blk < 0 || blk >= a.geo.num_blocks) {
                        bad = true;
                        blk = 0;
                    }
                    row0 = ((size_t)blk * Hkv + h) * a.geo.bt + (size_t)(tr - bi * a.geo.bt);
                }
                const uint32_t vq = (uint32_t)(kq ^ (run << 2));
#pragma unroll
                for (int i2 = 0; i2 < 2; ++i2) {
                    const int i = 2 * run + i2;
                    const size_t rb = (row0 + 8 * i2) * kCodeRow;
                    const uint32_t off = (uint32_t)crow * kCodeRow;
                    lds_copy16(a.k_codes + rb, off + 16u * kq, slot + 1024u * i);
                    lds_copy16(a.v_codes + rb, off + 16u * vq, slot + kTileBytes + 1024u * i);
                }
            }
        } else {
            // per-lane rows; rows past the context repeat the last token
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = min(t0 + 8 * i + crow, T - 1);
                const size_t rb = row_of(t) * kCodeRow;
                lds_copy16(a.k_codes + rb + 16 * kq, slot + 1024u * i);
                lds_copy16(a.v_codes + rb + 16 * (kq ^ ((i >> 1) << 2)), slot + kTileBytes + 1024u * i);
            }
        }
        // V scale (lanes 0..31) and zero (lanes 32..63) of the tile's tokens;
        // tokens past the context repeat the last one
        {
            const int t = min(t0 + (lane & 31), T - 1);
            lds_copy4((lane < 32 ? a.meta.v_scale : a.meta.v_zero) + vmeta + t, slot + kVMetaOff);
        }
        // K scale (lanes 0..31) and zero (lanes 32..63) of the group; the
        // previous group's values were consumed by its fold three tiles ago
        if ((j & 3) == 0) {
            const int g = g0 + min(group_of(j), n_groups - 1);
            const float *src = (lane < 32 ? a.meta.k_scale : a.meta.k_zero) + kmeta + (size_t)g * kHeadDim;
            lds_copy16(src + 4 * (lane & 31), km);
            if (!ONE && n_mine > 1) issue_ids((j >> 2) + 1);  // (a wavefront's only group has no next)
        }
    };

    // query rows of the workgroup into LDS: copy m holds rows 4 m .. 4 m + 3
    // (RT copies per wavefront; rows past the last repeat it)
#pragma unroll
    for (int k = 0; k < RT; ++k) {
        const int m = w + 4 * k;
        const int r = min(row_base + 4 * m + (lane >> 4), a.rows_total - 1);
        const int G = fresh_uniform(a.G);
        const size_t qrow = ((size_t)b * a.nq + r / G) * a.Hq + (size_t)h * G + r % G;
        lds_copy16(a.q + qrow * kHeadDim + 8 * (lane & 15), lds_addr(s_q) + 1024u * m);
    }

    // ---- per-wavefront online-softmax state: lane (col = query row of the
    // row tile, kg); the reference carries the 2^-Ev factor of the V weights ----
    float m_run[RT], m_ref[RT], l_part[RT], ob_part[RT];
    f32x4_t acc[RT][8];
    auto reset_state = [&]() {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            m_run[rt] = m_ref[rt] = -INFINITY;
            l_part[rt] = ob_part[rt] = 0.0f;
#pragma unroll
            for (int n = 0; n < 8; ++n) acc[rt][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    };
    reset_state();

    // Fold of a group (K scales and zeros from the wavefront's K-metadata
    // buffer, BF16 query rows from LDS), per row tile: the operands
    // y_d = q_d s_d 2^(15 - E), hi and lo, E the exponent of the row's largest
    // |q_d s_d|; the products' scale bsc = kscore 2^(E + 9) and the bias
    // bb = kscore sum_d q_d z_d.  Lane (col, kg) holds dims 32 kg .. + 31 of
    // row col of each row tile, the dims of its operand pieces.
    u32x4_t bq[RT][8];
    float bsc[RT], bb[RT];
    auto fold = [&]() {
        const float4 *ks = reinterpret_cast<const float4 *>(&s_km[w][0]) + 8 * kg;
        const float4 *kz = ks + kHeadDim / 4;
        float y[RT][32], mx[RT], bias[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) mx[rt] = bias[rt] = 0.0f;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const float4 s0 = ks[2 * kk], s1 = ks[2 * kk + 1], z0 = kz[2 * kk], z1 = kz[2 * kk + 1];
            const float sv[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
            const float zv[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const uint4 u =
                    reinterpret_cast<const uint4 *>(s_q + (rt * 16 + col) * (kHeadDim * 2) + 64 * kg)[kk];
                const uint32_t qw[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float q0 = bf16_lo(qw[e]), q1 = bf16_hi(qw[e]);
                    const float y0 = q0 * sv[2 * e], y1 = q1 * sv[2 * e + 1];
                    bias[rt] = fmaf(q0, zv[2 * e], bias[rt]);
                    bias[rt] = fmaf(q1, zv[2 * e + 1], bias[rt]);
                    mx[rt] = fmax3_abs(mx[rt], y0, y1);
                    y[rt][8 * kk + 2 * e] = y0;
                    y[rt][8 * kk + 2 * e + 1] = y1;
                }
                asm volatile("" : "+v"(bias[rt]));  // summed here: later, all its terms would be held in registers
            }
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            mx[rt] = max_kg(mx[rt]);
            int E = 0;
            if (mx[rt] > 0.0f) frexpf(mx[rt], &E);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float y0 = ldexpf(y[rt][2 * e], 15 - E), y1 = ldexpf(y[rt][2 * e + 1], 15 - E);
                const uint32_t hp = pack_f16(y0, y1);
                bq[rt][2 * (e / 4)][e % 4] = hp;
                bq[rt][2 * (e / 4) + 1][e % 4] = pack_f16(less_f16_lo(y0, hp), less_f16_hi(y1, hp));  // exact differences
            }
            // positive and finite: times the -inf of a token past the context
            // and times a product of 0 it must not be a NaN
            bsc[rt] = __builtin_amdgcn_fmed3f(ldexpf(kscore, E + 9), FLT_MIN, FLT_MAX);
            bb[rt] = kscore * sum_kg(bias[rt]);
        }
    };
    // Products of tile j (scores in log2 units are bsc times them, plus bb):
    // lane (col, kg) gets token t0 + 16 r + 4 kg + i in x[4 r + i]; tokens past
    // the context get -inf.
    auto tile_products = [&](const uint8_t *slot_p, int j, float (&x)[RT][8]) {
        f32x4_t sc[RT][2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int t = 16 * r + col;
            const uint4 u0 = *reinterpret_cast<const uint4 *>(slot_p + k_slot(t, 2 * kg));
            const uint4 u1 = *reinterpret_cast<const uint4 *>(slot_p + k_slot(t, 2 * kg + 1));
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) sc[rt][r] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const uint4 &u = (kk >> 1) ? u1 : u0;
                const u32x4_t av = (kk & 1) ? codes_to_f16(u.z, u.w) : codes_to_f16(u.x, u.y);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    sc[rt][r] = mfma_f16(av, bq[rt][2 * kk + 0], sc[rt][r]);
                    sc[rt][r] = mfma_f16(av, bq[rt][2 * kk + 1], sc[rt][r]);
                }
            }
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < 8; ++i) x[rt][i] = sc[rt][i >> 2][i & 3];
        const int t0 = tile_t0(j);
        if (t0 + kTile > T) {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int t = t0 + 16 * (i >> 2) + 4 * kg + (i & 3);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) x[rt][i] = t < T ? x[rt][i] : -INFINITY;
            }
        }
    };
    // the row's largest score of a tile (bsc > 0)
    auto tile_max = [&](const float (&x)[8], int rt) {
        const float mx = max_kg(fmax3(fmax3(x[0], x[1], x[2]), fmax3(x[3], x[4], x[5]), fmax2(x[6], x[7])));
        return fmaf(mx, bsc[rt], bb[rt]);
    };
    // Weights against m_ref, then P V for the tile (V rows from the slot,
    // transposed on read).
    auto tile_accumulate = [&](const uint8_t *slot_p, const float (&x)[RT][8]) {
        const float *vsm = reinterpret_cast<const float *>(slot_p + kVMetaOff) + 4 * kg;
        const float4 vs0 = *reinterpret_cast<const float4 *>(vsm);
        const float4 vs1 = *reinterpret_cast<const float4 *>(vsm + 16);
        const float4 vz0 = *reinterpret_cast<const float4 *>(vsm + kTile);
        const float4 vz1 = *reinterpret_cast<const float4 *>(vsm + kTile + 16);
        const float vsv[8] = {vs0.x, vs0.y, vs0.z, vs0.w, vs1.x, vs1.y, vs1.z, vs1.w};
        const float vzv[8] = {vz0.x, vz0.y, vz0.z, vz0.w, vz1.x, vz1.y, vz1.z, vz1.w};
        u32x4_t pa[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            float pw[8];
            const float c0 = bb[rt] - m_ref[rt];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float p = __builtin_amdgcn_exp2f(fmaf(x[rt][i], bsc[rt], c0));
                l_part[rt] += p;
                ob_part[rt] = fmaf(p, vzv[i], ob_part[rt]);
                pw[i] = p * vsv[i];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) pa[rt][e] = pack_f16_rne(pw[2 * e], pw[2 * e + 1]);
        }
        // V values of the 8 tokens tau(kg, e) = 16 (e / 4) + 4 kg + e % 4 for
        // dims 16 c + col, read transposed from LDS
        const uint8_t *vl = slot_p + kTileBytes;
        const int tr = 16 * ((col >> 1) >> 2) + 4 * kg + ((col >> 1) & 3);
        const int half = col & 1;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const intx2_t vt = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                (__attribute__((address_space(3))) intx2_t *)(vl + v_slot(tr, c) + 8 * half));
            const u32x4_t bv = codes_to_f16((uint32_t)vt[0], (uint32_t)vt[1]);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt][c] = mfma_f16(pa[rt], bv, acc[rt][c]);
        }
    };

    // Fast path: the softmax reference of each row is the maximum of the
    // wavefront's first tile and stays fixed.  If any sum leaves the safe
    // range the wavefront redoes its tiles below with a running maximum.
    // Tile j + 1 is in flight while tile j is attended; no barriers.
    if (LAYOUT == 1) {
        issue_ids(0);
        wait_vmcnt<0>();
    }
    if (n_mine > 0) issue_tile(0);
    // the query rows are in once only tile 0's copies may remain in flight
    // (LAYOUT 1 waited for them above)
    if (LAYOUT != 1) {
        if (n_mine > 0) {
            wait_vmcnt<kFirst>();
        } else {
            wait_vmcnt<0>();
        }
    }
    __syncthreads();
    for (int u = 0; u < (ONE ? min(n_mine, 1) : n_mine); ++u) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = 4 * u + c;
            // the next tile: inside this group, or the next group's first
            const bool more = c < 3 || (!ONE && u + 1 < n_mine);
            if (more) issue_tile(j + 1);
            // tile j is in once only tile j + 1's copies may remain in flight
            if (!more) {
                wait_vmcnt<0>();
            } else if (c == 3) {
                wait_vmcnt<kFirst>();
            } else {
                wait_vmcnt<9>();
            }
            const uint8_t *slot_p = ring_p + (c % kDepth) * kSlotBytes;
            if (c == 0) fold();
            if (tile_valid(j)) {
                float x[RT][8];
                tile_products(slot_p, j, x);
                if (j == 0) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
                        m_run[rt] = tile_max(x[rt], rt);
                        m_ref[rt] = m_run[rt] + (float)Ev;
                    }
                }
                tile_accumulate(slot_p, x);
            }
            // the slot and the K-metadata buffer are rewritten by later
            // copies: their reads must be done
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    }
    bool unsafe = false;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        unsafe |= !(l_part[rt] < 1e30f) || !(fabsf(ob_part[rt]) < 1e30f);
#pragma unroll
        for (int n = 0; n < 8; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) unsafe |= !(fabsf(acc[rt][n][i]) < 1e30f);
    }
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
            const uint8_t *slot_p = ring_p + (j % kDepth) * kSlotBytes;
            if ((j & 3) == 0) fold();
            if (tile_valid(j)) {
                float x[RT][8];
                tile_products(slot_p, j, x);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const float mx = tile_max(x[rt], rt);
                    if (__any(mx > m_run[rt])) {
                        const float m_new = fmaxf(mx, m_run[rt]);
                        const float alpha = (m_run[rt] == -INFINITY) ? 0.0f : exp2f(m_run[rt] - m_new);
                        m_run[rt] = m_new;
                        m_ref[rt] = m_new + (float)Ev;
                        l_part[rt] *= alpha;
                        ob_part[rt] *= alpha;
                        float af[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) af[i] = __shfl(alpha, 4 * kg + i);
#pragma unroll
                        for (int n = 0; n < 8; ++n)
#pragma unroll
                            for (int i = 0; i < 4; ++i) acc[rt][n][i] *= af[i];
                    }
                }
                tile_accumulate(slot_p, x);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    }
    wait_vmcnt<0>();  // no copy may land in the ring once it is reused below

    // The epilogue's lane numbers are its own: kept through the loop they would
    // take registers that it has none of.
    [&](const int tid) {
    const int lane = tid & 63, w = tid >> 6, col = lane & 15, kg = lane >> 4;
    // ---- per-wavefront totals -> LDS (still scaled by 2^-Ev) ----
    // o' = sum p' z + 2^24 sum pw c 2^-24
    __syncthreads();  // every wavefront is done with its ring
    // ring reused: o [wave][kRows][128], then max, sum, sum p z and merge
    // factors [wave][kRows]
    float *s_o = reinterpret_cast<float *>(s_ring);
    float(*s_m)[kRows] = reinterpret_cast<float(*)[kRows]>(s_o + kWaves * kRows * kHeadDim);
    float(*s_l)[kRows] = s_m + kWaves;
    float(*s_ob)[kRows] = s_l + kWaves;
    float(*s_f)[kRows] = s_ob + kWaves;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const float l = sum_kg(l_part[rt]);
        const float ob = sum_kg(ob_part[rt]);
        if (kg == 0) {
            s_m[w][rt * 16 + col] = m_run[rt];
            s_l[w][rt * 16 + col] = l;
            s_ob[w][rt * 16 + col] = ob;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 8; ++c)
                s_o[(w * kRows + rt * 16 + 4 * kg + i) * kHeadDim + 16 * c + col] = acc[rt][c][i] * 16777216.0f;
    }
    if (lane == 0) s_ev[w] = Ev;
    const bool any_bad = __syncthreads_or(bad);

    // ---- merge the four wavefronts, write this segment's partial: per-row
    // factors first, then float4 multiply-adds ----
    if (tid < kRows) {
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
    for (int idx = tid; idx < kRows * (kHeadDim / 4); idx += kThreads) {
        const int rr = idx / (kHeadDim / 4);  // row within the workgroup
        const int d4 = idx % (kHeadDim / 4);
        const int row = row_base + rr;
        if (row >= a.rows_total) continue;
        float4 O = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) {
            const float f = s_f[ww][rr];
            const float ob = s_ob[ww][rr];
            const float4 o = reinterpret_cast<const float4 *>(s_o + (ww * kRows + rr) * kHeadDim)[d4];
            O.x = fmaf(o.x + ob, f, O.x);
            O.y = fmaf(o.y + ob, f, O.y);
            O.z = fmaf(o.z + ob, f, O.z);
            O.w = fmaf(o.w + ob, f, O.w);
        }
        if (any_bad) O = make_float4(NAN, NAN, NAN, NAN);
        // nontemporal: the combine kernel reads the partials back faster when
        // they did not go through the last-level cache (32K layer 30.3 ->
        // 29.8 us per call, 128K 65.2 -> 63.9 us)
        const size_t pi = partial_index(row);
        const f32x4_t ov = {O.x, O.y, O.z, O.w};
        __builtin_nontemporal_store(ov, reinterpret_cast<f32x4_t *>(a.ws_o + pi * kHeadDim) + d4);
        if (d4 == 0) {
            const f32x2_t mlv = {s_ML[rr][0], s_ML[rr][1]};
            __builtin_nontemporal_store(mlv, reinterpret_cast<f32x2_t *>(a.ws_ml + pi));
        }
    }
    }(fresh_tid());
}

// Grid (worker, kv head x chunk) for the contiguous layout.  A paged block
// holds the rows of every kv head for its tokens side by side, so paged
// layouts make the kv head the fastest grid index: workgroups reading the
// same blocks run together and share DRAM pages.
// LANES: a lane for each sequence (B <= 64).
template <int RT, int LAYOUT, int UNIT, bool LANES>
__global__ __launch_bounds__(kThreads, 2) void verify_batch_kernel(VerifyArgs a) {
    if (LANES) __builtin_assume(a.B > 1 && a.B <= 64);
    const int worker = LAYOUT == 0 ? blockIdx.x : blockIdx.y;
    const int hc = LAYOUT == 0 ? blockIdx.y : blockIdx.x;
    const WorkList<UNIT, true> list(a.seq_lens, a.B, a.max_seq_len, a.workers);
    Segment<UNIT> seg;
    if (!seg.start(list, worker)) return;
    for (;;) {
        verify_segment<RT, LAYOUT, UNIT, false>(a, seg, fresh_uniform(hc % a.geo.Hkv), fresh_uniform(hc / a.geo.Hkv), fresh_tid());
        if (!seg.next(list, worker)) return;
        __syncthreads();  // the segment's LDS is free again
    }
}

// A single sequence of more units than workers: one segment each, no walk.
template <int RT, int LAYOUT, int UNIT>
__global__ __launch_bounds__(kThreads, 2) void verify_long_kernel(VerifyArgs a) {
    const int worker = LAYOUT == 0 ? blockIdx.x : blockIdx.y;
    const int hc = LAYOUT == 0 ? blockIdx.y : blockIdx.x;
    const WorkList<UNIT, false> list(a.seq_lens, 1, a.max_seq_len, a.workers);
    Segment<UNIT> seg;
    if (!seg.start(list, worker)) return;
    verify_segment<RT, LAYOUT, UNIT, false>(a, seg, hc % a.geo.Hkv, hc / a.geo.Hkv, threadIdx.x);
}

// A unit per workgroup, for sequence blockIdx.z.
template <int RT, int LAYOUT, int UNIT>
__global__ __launch_bounds__(kThreads, 2) void verify_kernel(VerifyArgs a) {
    const int unit = LAYOUT == 0 ? blockIdx.x : blockIdx.y;
    const int hc = LAYOUT == 0 ? blockIdx.y : blockIdx.x;
    Segment<UNIT> seg;
    if (!seg.set_unit(a.seq_lens, a.max_seq_len, a.direct, blockIdx.z, unit)) return;
    verify_segment<RT, LAYOUT, UNIT, true>(a, seg, hc % a.geo.Hkv, hc / a.geo.Hkv, threadIdx.x);
}

template <int RT, int LAYOUT>
void launch_rt(const VerifyArgs &args, dim3 grid, hipStream_t stream) {
    if (args.direct)
        hipLaunchKernelGGL((verify_kernel<RT, LAYOUT, kWorkUnit>), grid, dim3(kThreads), 0, stream, args);
    else if (args.B == 1)
        hipLaunchKernelGGL((verify_long_kernel<RT, LAYOUT, kWorkUnit>), grid, dim3(kThreads), 0, stream, args);
    else if (args.B <= 64)
        hipLaunchKernelGGL((verify_batch_kernel<RT, LAYOUT, kWorkUnit, true>), grid, dim3(kThreads), 0, stream, args);
    else
        hipLaunchKernelGGL((verify_batch_kernel<RT, LAYOUT, kWorkUnit, false>), grid, dim3(kThreads), 0, stream, args);
}

template <int RT>
void launch_layout(const VerifyArgs &args, dim3 grid, hipStream_t stream) {
    if (args.geo.max_blocks == 1)
        launch_rt<RT, 0>(args, grid, stream);
    else if (args.geo.bt % 16 == 0)
        launch_rt<RT, 1>(args, grid, stream);
    else
        launch_rt<RT, 2>(args, grid, stream);
}

}  // namespace

hipError_t launch_verify_mfma(const VerifyArgs &args, hipStream_t stream) {
    if (args.rows_total < 1 || args.workers < 1 || args.workers > 65535) return hipErrorInvalidValue;
    const int rt = args.rows_total <= 16 ? 1 : 2;
    const unsigned hc = (unsigned)(args.geo.Hkv * ((args.rows_total + 16 * rt - 1) / (16 * rt)));
    // kv head fastest for paged layouts (the kernel reads the grid the same way)
    const unsigned n = args.direct ? args.direct : args.workers, nz = args.direct ? args.B : 1;
    const dim3 grid = args.geo.max_blocks == 1 ? dim3(n, hc, nz) : dim3(hc, n, nz);
    if (rt == 1)
        launch_layout<1>(args, grid, stream);
    else
        launch_layout<2>(args, grid, stream);
    return hipGetLastError();
}

}  // namespace lynx
