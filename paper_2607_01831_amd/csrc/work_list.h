// Work list of the attention kernels (gfx950): the batch's context cut into
// equal shares, one per resident workgroup.
//
// A launch has as many workgroups per (kv head, row chunk) as fit the chip in
// one round (plan_attention).  The sequences' units of UNIT 128-token groups
// (at least one unit each, so that an empty sequence has an owner) stand in
// one list, and worker p of W takes the units [p total / W, (p + 1) total / W)
// of it, whichever sequences they belong to (or a share inside one sequence, see
// inner_share): one segment per sequence that it touches, one partial per
// segment.  A grid of fixed splits per sequence leaves a ragged batch's last
// round partly empty and pays a prologue and an epilogue per split (16 paged
// sequences of 16K-64K tokens: 166 us for the decode and its combine in splits
// of 2048 tokens, 154 us so; 32 of 1K-8K with a tail 58.5 -> 45.6 us).
// The worker that owns unit x is floor(((x + 1) W - 1) / total), so each side
// finds the others' shares without tables.  Segment (p, b) is number p + b of
// its (kv head, row): the two never go down along the list and one of them
// goes up with every segment, so no two share a number, and a sequence's
// segments are consecutive.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lane_ops.h"
#include "lynx_internal.h"

namespace lynx {

// WALK: the kernel loops over segments (see fresh_tid in lane_ops.h).
template <int UNIT, bool WALK>
struct WorkList {
    static constexpr int kTokens = UNIT * kKGroup;
    const int32_t *lens;
    int B, max_len;
    int own_T;    // tokens of the lane's sequence (B <= 64)
    int upto;     // units of the sequences up to the lane's (B <= 64)
    int only;     // tokens of a single sequence
    int total;    // units of all sequences
    int workers;  // workers with a share: min(asked, total)

    __device__ __forceinline__ int tokens(int b) const { return max(0, min(lens[b], max_len)); }
    // The same where b is uniform, in a scalar register.
    __device__ __forceinline__ int tokens_of(int b) const {
        if (B == 1) return only;
        return B <= 64 ? __builtin_amdgcn_readlane(own_T, b) : __builtin_amdgcn_readfirstlane(tokens(b));
    }
    static __device__ __forceinline__ int units(int T) { return max(1, (T + kTokens - 1) / kTokens); }

    // Sum over the wavefront's lanes up to and with this one (DPP shifts inside
    // the 16-lane rows, then the rows' last lanes broadcast on).
    template <int CTRL, int ROWS>
    static __device__ __forceinline__ int add_dpp(int v) {
        return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false);
    }
    static __device__ __forceinline__ int scan(int v) {
        v = add_dpp<0x111, 0xF>(v);  // row_shr 1, 2, 4, 8
        v = add_dpp<0x112, 0xF>(v);
        v = add_dpp<0x114, 0xF>(v);
        v = add_dpp<0x118, 0xF>(v);
        v = add_dpp<0x142, 0xA>(v);  // row_bcast 15 into rows 1 and 3
        return add_dpp<0x143, 0xC>(v);  // row_bcast 31 into rows 2 and 3
    }
    // Units of the 64 sequences from i0, a lane each; those of lanes past the
    // batch count 0.
    __device__ __forceinline__ int units_at(int i0) const {
        const int i = i0 + (int)(threadIdx.x & 63);
        const int T = B <= 64 ? own_T : tokens(min(i, B - 1));
        return i < B ? units(T) : 0;
    }

    // The lane's entry of the lengths, for a kernel that has other loads to issue
    // before it waits for this one.
    static __device__ __forceinline__ int load_own(const int32_t *seq_lens, int batch) {
        return batch <= 64 ? seq_lens[min((int)(threadIdx.x & 63), batch - 1)] : 0;
    }
    __device__ __forceinline__ WorkList(const int32_t *seq_lens, int batch, int max_seq_len, int asked)
        : WorkList(seq_lens, batch, max_seq_len, asked, batch > 1 ? load_own(seq_lens, batch) : 0) {}
    __device__ __forceinline__ WorkList(const int32_t *seq_lens, int batch, int max_seq_len, int asked, int own)
        : lens(seq_lens), B(batch), max_len(max_seq_len), own_T(0), upto(0), only(0), total(0) {
        if (B == 1) {
            only = tokens(0);
            total = units(only);
        } else if (B <= 64) {
            own_T = max(0, min(own, max_len));
            upto = scan(units_at(0));
            total = __builtin_amdgcn_readlane(upto, 63);
        } else {
            for (int i0 = 0; i0 < B; i0 += 64) total += __builtin_amdgcn_readlane(scan(units_at(i0)), 63);
        }
        workers = min(asked, total);
    }
    static __device__ __forceinline__ int opaque(int v) { return WALK ? fresh_uniform(v) : v; }
    // First unit of worker p's share (p = workers: the end of the list).
    __device__ __forceinline__ int begin(int p) const {
        if (workers == total) return p;  // a unit each: no division in a short call
        return (int)((uint32_t)p * (uint32_t)total / (uint32_t)opaque(workers));
    }
    // The worker that owns unit x.
    __device__ __forceinline__ int owner(int x) const {
        if (workers == total) return x;
        return (int)(((uint32_t)(x + 1) * (uint32_t)workers - 1u) / (uint32_t)opaque(total));
    }
    // The sequence that holds unit x, and the number of its first unit.
    __device__ __forceinline__ void find(int x, int &b, int &first) const {
        b = 0;
        first = 0;
        if (B == 1) return;
        if (B <= 64) {
            b = __ffsll((long long)__ballot(upto > x)) - 1;
            first = __builtin_amdgcn_readlane(upto, b) - units(__builtin_amdgcn_readlane(own_T, b));
            return;
        }
        for (int i0 = 0; i0 < B; i0 += 64) {
            const int own = units_at(i0);
            const int last = first + scan(own);
            const uint64_t past = __ballot(last > x);
            if (past) {  // uniform across the wavefront
                const int l = __ffsll((long long)past) - 1;
                b = i0 + l;
                first = __builtin_amdgcn_readlane(last - own, l);
                return;
            }
            first = __builtin_amdgcn_readlane(last, 63);
        }
    }
    // A share across a boundary costs a second prologue, epilogue and merge, as
    // long as a unit itself.  So shares of few units stay inside their
    // sequences, of `s` units at most (0: the shares of begin() and owner()),
    // where that takes no more workers and no larger share than the equal ones
    // (decode of 15 sequences of 2500 tokens: 18.4 us, by equal shares 24.5; 16
    // of 1K-5K: 18.7 and 22.2).  Of more than four units a share hides the
    // boundary, and the look for whole ones, mostly in vain, costs 2% (32 of
    // 1K-8K with a tail, five units: 46.0 us, without it 45.0).  segs: the
    // shares of the sequences up to the lane's.
    __device__ __forceinline__ int inner_share(int &segs) const {
        if (B == 1 || B > 64 || workers == total || total > 4 * workers) return 0;
        const uint32_t s = ((uint32_t)total + workers - 1) / (uint32_t)opaque(workers);
        segs = scan((int)(((uint32_t)units_at(0) + s - 1) / s));
        return __builtin_amdgcn_readlane(segs, 63) <= workers ? (int)s : 0;
    }
    // Sequence b's partials: n from number seg0 on.
    __device__ __forceinline__ void partials(int b, int &seg0, int &n) const {
        int segs;
        if (inner_share(segs)) {
            seg0 = b > 0 ? __builtin_amdgcn_readlane(segs, b - 1) : 0;
            n = __builtin_amdgcn_readlane(segs, b) - seg0;
        } else {
            const int first = B == 1 ? 0 : first_unit(b);
            seg0 = owner(first);
            n = owner(first + units(tokens_of(b)) - 1) - seg0 + 1;
        }
        seg0 += b;
    }
    // The number of sequence b's first unit.
    __device__ __forceinline__ int first_unit(int b) const {
        if (B <= 64) return __builtin_amdgcn_readlane(upto, b) - units(__builtin_amdgcn_readlane(own_T, b));
        int first = 0;
        for (int i0 = 0; i0 < b; i0 += 64)
            first += __builtin_amdgcn_readlane(scan(i0 + (int)(threadIdx.x & 63) < b ? units_at(i0) : 0), 63);
        return first;
    }
};

// A worker's walk over its share.
template <int UNIT>
struct Segment {
    int b;        // sequence
    int T;        // its tokens
    int g0;       // first 128-token group of the segment
    int n_groups; // its groups that hold tokens
    int number;   // of the worker's partial
    int number0;  // of the sequence's first partial
    int live;     // the sequence's partials
    int pos, end; // units of the worker's share: the segment's first, the share's end
    int first;    // the sequence's first unit
    int n_units;  // the segment's units

    template <bool WALK>
    __device__ __forceinline__ void set(const WorkList<UNIT, WALK> &wl, int p) {
        T = wl.tokens_of(b);
        const int all = wl.units(T);
        n_units = min(end, first + all) - pos;
        g0 = (pos - first) * UNIT;
        n_groups = max(0, min(n_units * UNIT, (T + kKGroup - 1) / kKGroup - g0));
        // a single sequence is every worker's; no division either
        const int w0 = wl.B == 1 ? 0 : __builtin_amdgcn_readfirstlane(wl.owner(first));
        const int w1 = wl.B == 1 ? wl.workers - 1 : __builtin_amdgcn_readfirstlane(wl.owner(first + all - 1));
        number = p + b;
        number0 = w0 + b;
        live = w1 - w0 + 1;
    }
    // The first segment of worker p; false where it has none.
    template <bool WALK>
    __device__ __forceinline__ bool start(const WorkList<UNIT, WALK> &wl, int p) {
        if (p >= wl.workers) return false;
        int segs;
        if (const int s = wl.inner_share(segs)) {
            const uint64_t past = __ballot(segs > p);
            if (!past) return false;
            b = __ffsll((long long)past) - 1;
            const int w0 = b > 0 ? __builtin_amdgcn_readlane(segs, b - 1) : 0;
            T = wl.tokens_of(b);
            const int u0 = (p - w0) * s;
            n_units = min(s, wl.units(T) - u0);
            g0 = u0 * UNIT;
            n_groups = max(0, min(n_units * UNIT, (T + kKGroup - 1) / kKGroup - g0));
            number = p + b;
            number0 = w0 + b;
            live = __builtin_amdgcn_readlane(segs, b) - w0;
            pos = end = first = 0;  // no second one
            return true;
        }
        pos = __builtin_amdgcn_readfirstlane(wl.begin(p));
        end = __builtin_amdgcn_readfirstlane(wl.begin(p + 1));
        wl.find(pos, b, first);
        set(wl, p);
        return true;
    }
    // Without a list, where every unit has a worker (AttnPlan::direct): unit
    // `unit` of sequence `seq`, whose partials stand from direct seq on; false
    // past the sequence's end.
    __device__ __forceinline__ bool set_unit(const int32_t *lens, int max_len, int direct, int seq, int unit) {
        b = seq;
        T = max(0, min(lens[seq], max_len));
        live = WorkList<UNIT, false>::units(T);
        g0 = unit * UNIT;
        n_groups = max(0, min(UNIT, (T + kKGroup - 1) / kKGroup - g0));
        number0 = seq * direct;
        number = number0 + unit;
        return unit < live;
    }
    // The next one; false past the share's end.
    template <bool WALK>
    __device__ __forceinline__ bool next(const WorkList<UNIT, WALK> &wl, int p) {
        pos += n_units;
        if (pos >= end) return false;
        first += wl.units(T);
        ++b;
        set(wl, p);
        return true;
    }
};

}  // namespace lynx
