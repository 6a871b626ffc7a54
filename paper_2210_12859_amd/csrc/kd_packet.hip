// kd_packet.hip -- kNN by packets: one wave answers 64 neighbouring queries.
//
// The queries are sorted along the tree (kd_sort.hip), so the 64 queries of a
// wave lie close together and need nearly the same nodes.  Instead of 64
// independent walks, the wave makes one walk over groups of nodes and tests
// whole groups against all its queries on the matrix cores:
//   * group: the top levels of a subtree.  The tree of H levels is cut at
//     depth Td (leaves: subtrees of at most 6 levels) and above it into groups
//     of 5 levels (31 points), so a group has at most 32 child groups.
//   * expansion: lane l loads the bounding box of child group l % 32 and tests
//     it against the box of 32 of the wave's queries (lanes 0-31: queries
//     0-31, lanes 32-63: queries 32-63) grown by their largest search radius;
//     the children that pass are then tested against every single query, the
//     box read from its lane.
//   * scan: 32 points against 64 queries.  With coordinates taken from the
//     middle c of the packet (p' = p - c, q' = q - c), the sign of
//     |p'|^2 - 2 p'.q' + (|q'|^2 - worst - slack) says whether the point can
//     be among the query's k best.  The numbers are split into two
//     half-precision parts each, which makes it a product of a 32 x 16 and a 16 x 64 matrix
//     (two v_mfma_f32_32x32x16_f16) whose sign bits are collected into one
//     32-bit mask per query.  slack covers the rounding of that product (see
//     packet_slack), so no point of the result is ever lost; points that pass
//     are read back from LDS, their squared distance is computed as
//     everywhere else (binary32, left to right) and inserted into the lane's
//     sorted (d2, index) list.  Results are therefore the lane-by-lane
//     traversal's, bit for bit.
// Two walks per packet: the first visits the few leaves that hold the queries
// and finds for each query an upper bound of its k-th distance (the k-th
// smallest product, kept in a list of floats: one v_med3 per slot); the
// second visits every group within those bounds.
//
// Packets that would need many leaves (queries far apart, or far from the
// data) and queries that are not finite are appended, with the bound found so
// far, to a list that the one-wave-per-query kernel finishes (kd_wave.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kd_groups.h"
#include "kd_internal.h"
#include "kd_list.h"

namespace kd {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Pairs of chunks held in LDS until their candidates are inserted and the bounds
// refreshed: until a query has FLUSH candidates, but two at least and four at
// most.  More pairs fill the insertions better, which few candidates (uniform
// points) gain by; a sooner refresh spares the next chunks' candidates, which many
// (clusters) gain by.  1M points and queries, always 4 / always 2 / by candidates,
// ms: 3-D, k = 1 mixture 0.410 / 0.381 / 0.368, k = 8 uniform 0.466 / 0.474 / 0.467,
// mixture 0.668 / 0.660 / 0.648, clusters of many widths 1.237 / 1.197 / 1.143, k =
// 32 clusters 3.436 / 3.275 / 3.195; 4-D, k = 8 uniform 0.939 / 0.955 / 0.935, clusters 2.639 / 2.570 /
// 2.552, k = 16 uniform 1.328 / 1.349 / 1.317.  3 or 5 candidates instead of 4 are
// within 1 % of it, 8 up to 2 % slower on clusters.
constexpr uint32_t NPEND = 4;
constexpr uint32_t FLUSH = 4;
// Entry of the chunks held that a queue byte names.  Lanes without a candidate
// read bytes that nothing wrote, so every byte has to name one of the entries.
__host__ __device__ constexpr uint32_t held_entry(uint32_t byte, uint32_t entries) { return byte & (entries - 1u); }
constexpr bool held_entries_hold(uint32_t entries) {
    for (uint32_t b = 0; b < 256u; ++b)
        if (held_entry(b, entries) >= entries || (b < entries && held_entry(b, entries) != b)) return false;
    return entries <= 256u;  // a queue entry is a byte
}
static_assert(held_entries_hold(NPEND * 64), "queue bytes");
constexpr int QCAP = 16;        // candidates a query can hold until then
constexpr uint32_t MAX_HOME = 8;          // chunk pairs of the first walk
constexpr uint32_t NO_KEY = 0x7fe00000u;  // high word above every key's
// scaled |p'|^2 of an empty slot: never a candidate, as the query side of the
// product is at least -2 |p'| |q'| - r^2 - slack > -2 240 64 - 4200
constexpr float PT_NONE = 60000.0f;
constexpr float BOUND_MAX = 30000.0f;  // larger products stand for no point
constexpr float COORD_MAX = 1.0e18f;  // larger queries are left over

struct PacketArgs {
    const void* nodes;       // TreeRec<D>[N + 2]
    const float* boxes;      // subtree boxes by node id
    int32_t N;
    GroupShape shape;
    const void* sq;          // NodeRec<D>[Q], sorted
    uint32_t Q;
    int k;
    float R2;
    int32_t* out_idx;
    float* out_d2;
    int vec_store;
    uint32_t leaf_limit;
    uint32_t* fb_count;      // queries left to the one-wave-per-query kernel
    void* fb_recs;           // their records, NodeRec<D>[Q] (jobs: class slots)
    float* fb_w0;            // and upper bounds of their k-th squared distance
    // jobs: what describes the tree and the outputs comes from the packet's job
    const BatchJob* jobs;
    int njobs;
    uint32_t packets;
    const uint32_t* perm;    // class slots in sorted order (NULL: slot order)
};

// Rounding of the matrix test.  A number is cut into two half-precision parts
// (error below 2^-20 of it); of a product of two cut numbers the low-by-low
// part is left out.  With A = |q'| + |p'| the coordinate terms are off by at
// most 3.1 2^-20 2 |p'| |q'| <= 1.6 2^-20 A^2, |p'|^2 and the threshold by
// 2^-20 A^2 each, and the binary32 steps (shifted and scaled coordinates,
// squares, accumulation, the squared distance itself) by less than 60 2^-24
// A^2: 7.4 2^-20 A^2 = 7.0e-6 A^2 together.  A candidate has |p'| <= |q'| + r
// (r the search radius), so 8e-6 (2 |q'| + r)^2 covers it.  Numbers are
// scaled so that PACKET_SCALE covers |q'| + r of every query; the constant, in
// scaled units, covers low parts that are not normal half-precision numbers
// (2^-24 each, times at most 2 PACKET_SCALE, at most 10 of them: 8e-5).
constexpr float PACKET_SCALE = 64.0f;
constexpr float COORD_CLAMP = 120.0f;  // scaled coordinates of points beyond every query's reach
__device__ __forceinline__ float packet_slack(float qn, float r) {
    const float a = 2.0f * qn + r;
    return a * a * 8.0e-6f + 2.0e-4f;
}

// Maximum over the lane's 32-lane half: four exchanges inside rows of 16
// lanes (quad_perm, half mirror, mirror), one between the two rows.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float half_max(float v) {
    v = fmaxf(v, dpp<0xb1>(v));   // quad_perm 1,0,3,2
    v = fmaxf(v, dpp<0x4e>(v));   // quad_perm 2,3,0,1
    v = fmaxf(v, dpp<0x141>(v));  // row_half_mirror
    v = fmaxf(v, dpp<0x140>(v));  // row_mirror
    const u32x2 s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(s.x), __uint_as_float(s.y));
}
__device__ __forceinline__ float half_min(float v) { return -half_max(-v); }
__device__ __forceinline__ float both_halves_max(float v) {
    const u32x2 s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(s.x), __uint_as_float(s.y));
}

__device__ __forceinline__ uint32_t pack_half(float first, float second) {
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(first, second));
}
__device__ __forceinline__ float half_rest(float x) {  // x minus its half-precision part
    return x - float(__builtin_amdgcn_cvt_pkrtz(x, 0.0f)[0]);
}

// Lowest set bit of m (any value when there is none).
__device__ __forceinline__ uint32_t first_bit(uint64_t m) {
    uint32_t lo, hi;
    asm("v_ffbl_b32 %0, %1" : "=v"(lo) : "v"(uint32_t(m)));
    asm("v_ffbl_b32 %0, %1" : "=v"(hi) : "v"(uint32_t(m >> 32)));
    hi += 32u;
    return lo < hi ? lo : hi;
}

__device__ __forceinline__ uint32_t sign_bits(const f32x16& acc) {
    uint32_t m = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) m = __builtin_amdgcn_alignbit(m, __float_as_uint(acc[r]), 31);
    return m;  // result r at bit 15 - r
}

// Operands of the product: k-slots 0-7 of a 32 x 16 tile come from lanes 0-31,
// slots 8-15 from lanes 32-63.
//   points  (row = lane % 32): xh yh zh wh Ph Pl 1  1  | xl yl zl wl xh yh zh wh
//   queries (column):          xh yh zh wh 1  1  th tl | xh yh zh wh xl yl zl wl
// with P = |p'|^2, the query's -2 q' as x..w and its threshold t, all scaled.
template <int D>
struct Packet {
    float q[D];
    bool active;
    float c[D];            // wave-uniform middle of the packet
    float scale;           // wave-uniform
    float qq, qn;          // scaled |q'|^2 and |q'|
    float lo[D], hi[D];    // box of the lane's half of the packet
    u32x4 b_lo, b_hi;      // query operands of queries 0-31 and 32-63
    uint32_t w3;           // the lane's own k-slots 14, 15
    int32_t slot, slot_lv, slot_off;  // the chunk point the lane loads

    // one word of both query operands from the lane's own query's words of
    // k-slots 2w, 2w+1 and 8 + 2w, 9 + 2w
    template <int W>
    __device__ __forceinline__ void operand_word(uint32_t low, uint32_t high) {
        const u32x2 s = __builtin_amdgcn_permlane32_swap(low, high, false, false);
        b_lo[W] = s.x;
        b_hi[W] = s.y;
    }
    __device__ __forceinline__ void set_query(float sc) {
        scale = sc;
        float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        qq = 0.0f;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float d = active ? (q[j] - c[j]) * sc : 0.0f;
            qq = __builtin_fmaf(d, d, qq);
            x[j] = -2.0f * d;
        }
        qn = __builtin_amdgcn_sqrtf(qq);
        const uint32_t xy = pack_half(x[0], x[1]), zw = pack_half(x[2], x[3]);
        operand_word<0>(xy, xy);
        operand_word<1>(zw, zw);
        operand_word<2>(0x3c003c00u, pack_half(half_rest(x[0]), half_rest(x[1])));
        w3 = pack_half(half_rest(x[2]), half_rest(x[3]));
    }
    // lanes without a query keep every point out
    __device__ __forceinline__ void set_threshold(float t) {
        const float u = active ? t : PT_NONE;
        operand_word<3>(pack_half(u, half_rest(u)), w3);
    }

    // Operands of the 32 points of lanes 0-31 (pa) and of lanes 32-63 (pb),
    // each lane's own point p.  Coordinates beyond COORD_CLAMP are clamped,
    // which keeps every number finite; with EXACT_ONLY such points are
    // dropped.
    template <bool EXACT_ONLY>
    __device__ __forceinline__ void point_operands(const float (&p)[D], bool valid, u32x4& pa, u32x4& pb) const {
        float d[4] = {0.0f, 0.0f, 0.0f, 0.0f}, l[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float pp = 0.0f;
        bool in = valid;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float x = (p[j] - c[j]) * scale;
            d[j] = __builtin_amdgcn_fmed3f(x, -COORD_CLAMP, COORD_CLAMP);
            if (EXACT_ONLY) in = in & (x == d[j]);
            pp = __builtin_fmaf(d[j], d[j], pp);
        }
        pp = in ? pp : PT_NONE;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            // a dropped point's product is PT_NONE alone
            if (EXACT_ONLY) d[j] = in ? d[j] : 0.0f;
            l[j] = half_rest(d[j]);
        }
        const uint32_t xy = pack_half(d[0], d[1]), zw = pack_half(d[2], d[3]);
        const uint32_t low[4] = {xy, zw, pack_half(pp, half_rest(pp)), 0x3c003c00u};
        const uint32_t high[4] = {pack_half(l[0], l[1]), pack_half(l[2], l[3]), xy, zw};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const u32x2 s = __builtin_amdgcn_permlane32_swap(low[w], high[w], false, false);
            pa[w] = s.x;
            pb[w] = s.y;
        }
    }
};

__device__ __forceinline__ f32x16 products(const u32x4& a, const u32x4& b) {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.0f;
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), z, 0, 0,
                                                  0);
}

// Bound by vector issue (72 % of the SIMDs' cycles; 11.6K instructions a
// packet at k = 8, uniform 1M: 47 chunks scanned, 63 boxes tested against the
// queries).  One wave per workgroup, so
// that a slow packet holds no other's place; with five instead of four per
// SIMD where the registers of short lists allow it without spills: the 1M call
// 0.458 -> 0.411 ms.  Half-precision parts instead of
// v_mfma_f32_32x32x2_f32 on binary32 numbers: 64 instead of 384 matrix cycles
// a chunk.  Lists over 32 are left to the other kernels: the allocator would
// copy live registers inside divergent regions, which loses them in the
// inactive lanes.
// Where a packet's queries come from: one call's sorted records, or the class
// slots of jobs.
enum Source { CALL, JOBS };
template <int D, int K, Source SRC>
__global__ __launch_bounds__(64, K <= 8 ? (D == 4 || K <= 2 || SRC != CALL ? 4 : 5) : 1) void knn_packet(PacketArgs a) {
    __shared__ float4 pt[NPEND * 64];                    // points of the chunks held
    __shared__ int32_t pid[D == 4 ? NPEND * 64 : 1];     // their caller indices where w is a coordinate
    __shared__ uint8_t queue[(QCAP + 1) * 64];           // candidate i of lane l at 64 i + l
    const uint32_t lane = __lane_id();
    // workgroups of one XCD (blockIdx % 8) take neighbouring packets
    const uint32_t pk = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    uint32_t first = pk * 64u, end = a.Q;
    uint32_t slot_base = 0;
    const float* queries = nullptr;
    if constexpr (SRC == JOBS) {
        if (pk >= a.packets) return;
        int lo = 0, hi = a.njobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.jobs[mid].packet_base <= pk) lo = mid;
            else hi = mid - 1;
        }
        const BatchJob& J = a.jobs[lo];
        a.nodes = J.nodes;
        a.boxes = J.boxes;
        a.N = J.N;
        a.shape = job_shape(J);
        a.k = J.k;
        a.R2 = J.R2;
        a.out_idx = J.out_idx;
        a.out_d2 = J.out_d2;
        a.vec_store = (J.k & 3) == 0 &&
                      ((reinterpret_cast<uintptr_t>(J.out_idx) | reinterpret_cast<uintptr_t>(J.out_d2)) & 15u) == 0;
        queries = J.queries;
        slot_base = J.slot_base;
        first = J.slot_base + (pk - J.packet_base) * 64u;
        end = J.slot_base + J.Q;
    }
    if (first >= end) return;
    const TreeRec<D>* __restrict__ g1 = reinterpret_cast<const TreeRec<D>*>(a.nodes);
    const int32_t* __restrict__ ids =
        rec_has_idx(D) ? nullptr : reinterpret_cast<const int32_t*>(g1 + (int64_t(a.N) + 2));
    const uint32_t slot = first + lane;
    const bool have = slot < end;

    Packet<D> s;
    int32_t row = 0;
    if constexpr (SRC == JOBS) {
        const uint32_t at = have ? slot : first;
        row = int32_t((a.perm ? a.perm[at] : at) - slot_base);
#pragma unroll
        for (int j = 0; j < D; ++j) s.q[j] = queries[size_t(row) * D + j];
    } else {
        const NodeRec<D>* r = reinterpret_cast<const NodeRec<D>*>(a.sq) + (have ? slot : first);
#pragma unroll
        for (int j = 0; j < D; ++j) s.q[j] = r->c[j];
        row = r->idx;
    }
    bool finite = true;
#pragma unroll
    for (int j = 0; j < D; ++j) finite = finite & (fabsf(s.q[j]) <= COORD_MAX);
    s.active = have & finite;

    // queries left to the one-wave-per-query kernel, with bound w0
    auto hand_over = [&](bool mine, float w0) {
        const uint64_t m = wave_ballot(mine);
        if (!m) return;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(a.fb_count, uint32_t(__popcll(m)));
        base = __builtin_amdgcn_readfirstlane(base);
        if (mine) {
            const uint32_t pos = base + __popcll(m & ((uint64_t(1) << lane) - 1));
            if constexpr (SRC == JOBS) {
                reinterpret_cast<uint32_t*>(a.fb_recs)[pos] = slot_base + uint32_t(row);
            } else {
                NodeRec<D>* o = reinterpret_cast<NodeRec<D>*>(a.fb_recs) + pos;
                NodeRec<D> rec;
#pragma unroll
                for (int j = 0; j < D; ++j) rec.c[j] = s.q[j];
                rec.idx = row;
                *o = rec;
            }
            a.fb_w0[pos] = w0;
        }
    };
    hand_over(have & !finite, a.R2);
    if (!wave_any(s.active)) return;

    // boxes of the two halves and the middle of the packet
#pragma unroll
    for (int j = 0; j < D; ++j) {
        s.lo[j] = half_min(s.active ? s.q[j] : __builtin_inff());
        s.hi[j] = half_max(s.active ? s.q[j] : -__builtin_inff());
        const float l = -both_halves_max(-s.lo[j]), h = both_halves_max(s.hi[j]);
        s.c[j] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(0.5f * l + 0.5f * h)));
    }
    // |q'|: the coordinates' largest and the length
    float qmax = 0.0f, qlen = 0.0f;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        const float d = s.active ? fabsf(s.q[j] - s.c[j]) : 0.0f;
        qmax = fmaxf(qmax, d);
        qlen = __builtin_fmaf(d, d, qlen);
    }
    qmax = both_halves_max(half_max(qmax));
    qlen = __builtin_amdgcn_sqrtf(qlen);
    {
        // row rho of a tile's result sits at bit 16 h + 15 - r of the query's
        // mask (h = rho / 4 % 2, r = 4 (rho / 8) + rho % 4): the lane that
        // loads row rho takes the chunk's point of that number, so bit b of
        // a mask is point b
        const int32_t rho = int32_t(lane & 31u);
        s.slot = (((rho >> 2) & 1) << 4) + 15 - (((rho >> 3) << 2) | (rho & 3));
        s.slot_lv = s.slot ? 31 - __builtin_clz(uint32_t(s.slot)) : 0;
        s.slot_off = s.slot - (1 << s.slot_lv);
    }
    // A chunk is up to 32 points of a group: the top nlev levels of its
    // subtree (slot j >= 1: the j-th node in level order), or (sixth) its
    // sixth level.  Two chunks are read at a time, one by each half of the
    // wave; load() starts reading.
    struct ChunkId {
        int32_t r, nlev;  // r = 0: no chunk
        bool sixth;
    };
    struct Chunks {
        float p[D];
        int32_t idx;
        bool ok;
    };
    const bool upper = lane >= 32;
    auto load = [&](const ChunkId& c0, const ChunkId& c1) -> Chunks {
        Chunks ch;
        const int32_t r = upper ? c1.r : c0.r;
        const bool sixth = upper ? c1.sixth : c0.sixth;
        const int32_t id = sixth ? (r << GL) + s.slot : (r << s.slot_lv) + s.slot_off;
        ch.ok = (sixth | ((s.slot > 0) & (s.slot_lv < (upper ? c1.nlev : c0.nlev)))) & (r != 0) & (id <= a.N);
        load_point<D>(g1, ids, ch.ok ? id : 1, ch.p, ch.idx);
        return ch;
    };

    // Box of child group lane % 32 of group r, and its gap to the lane's half
    // of the packet (NaN where there is no such child: every comparison fails).
    float bl[D], bh[D];
    auto child_gap = [&](int32_t r, int32_t lv) -> float {
        const int32_t ch = int32_t(lane & 31u);
        const bool none = (ch >> lv) != 0;
        const int32_t id = none ? r : (r << lv) + ch;
        load_box<D>(a.boxes, id, bl, bh);
        const float gap = box_gap<D>(bl, bh, s.lo, s.hi);
        return none ? __builtin_nanf("") : gap;
    };
    // lanes without a query are out of reach of every box
    float qb[D];
#pragma unroll
    for (int j = 0; j < D; ++j) qb[j] = s.active ? s.q[j] : __builtin_inff();
    // Children of m (bit = child, boxes in bl / bh) that some query reaches
    // within `reach` (its own squared radius).
    auto test_children = [&](uint32_t m, float reach) -> uint32_t {
        uint32_t out = 0;
        while (m) {
            const int32_t ch = int32_t(__builtin_ctz(m));
            const uint32_t bit = m & (0u - m);
            m ^= bit;
            float l[D], h[D];
#pragma unroll
            for (int j = 0; j < D; ++j) {
                l[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(bl[j]), ch));
                h[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(bh[j]), ch));
            }
            if (wave_any(box_gap<D>(l, h, qb, qb) <= reach)) out |= bit;
        }
        return out;
    };

    // Walk over the groups from the root.  expand(r, lv, to_leaves) gives the
    // children of group r to visit; chunk(data, last) takes 32 points.  The
    // next chunk is read while one is worked on.  The first nfirst leaves of
    // `home` come first.  own: the points of the groups above the leaves are
    // taken too.  Ends early when enough() says so.
    uint32_t stack = 0;   // lane g: children of group level g still to visit
    int32_t home = 0;     // lane i: the i-th leaf of the first walk
    uint32_t nhome = 0;
    auto walk = [&](uint32_t nfirst, bool own, auto&& expand, auto&& chunk, auto&& enough) {
        const bool six = a.shape.leaf_levels > GL;
        int32_t g = -1, r = 1;
        uint32_t leaf_m = a.shape.leaf_group == 0 ? 1u : 0u;  // leaves still to read: base + bit
        int32_t base = 1;
        int32_t part = 0;  // the sixth level of this leaf comes next
        uint32_t m = 0;
        uint32_t at_first = 0;
        ChunkId c0 = {0, 0, false}, c1 = {0, 0, false};
        Chunks cur;
        bool loaded = false;
        bool cut = false;  // the chunks at hand end the leaves of `home`
        for (;;) {
            ChunkId c = {0, GL, false};
            bool more = true;
            bool ends = false;
            if (part) {
                c.r = part;
                c.sixth = true;
                part = 0;
                ends = nfirst != 0 && at_first == nfirst;
            } else if (at_first < nfirst) {
                c.r = int32_t(__builtin_amdgcn_readlane(uint32_t(home), at_first));
                ++at_first;
                if (six && (c.r << GL) <= a.N) part = c.r;
                ends = part == 0 && at_first == nfirst;
            } else if (leaf_m) {
                c.r = base + int32_t(__builtin_ctz(leaf_m));
                leaf_m &= leaf_m - 1;
                if (six && (c.r << GL) <= a.N) part = c.r;
            } else if (a.shape.leaf_group == 0) {
                more = false;
            } else {
                // the next group: the root, or the next child of the deepest
                // level with children left
                if (g < 0) {
                    g = 0;
                } else {
                    m = g + 1 == a.shape.leaf_group ? 0u : __builtin_amdgcn_readlane(stack, uint32_t(g));
                    while (m == 0 && g > 0) {
                        --g;
                        r >>= g == 0 ? a.shape.top_levels : GL;
                        m = __builtin_amdgcn_readlane(stack, uint32_t(g));
                    }
                    if (m) {
                        stack = lane == uint32_t(g) ? m & (m - 1) : stack;
                        r = (r << (g == 0 ? a.shape.top_levels : GL)) + int32_t(__builtin_ctz(m));
                        ++g;
                    } else {
                        more = false;
                    }
                }
                if (more) {
                    c.nlev = g == 0 ? a.shape.top_levels : GL;
                    const bool to_leaves = g + 1 == a.shape.leaf_group;
                    const uint32_t in = expand(r, c.nlev, to_leaves);
                    if (to_leaves) {
                        leaf_m = in;
                        base = r << c.nlev;
                    } else {
                        stack = lane == uint32_t(g) ? in : stack;
                    }
                    if (enough()) return;
                    if (!own) continue;
                    c.r = r;
                }
            }
            // two chunks make a pair; the last leaf of `home` and the last
            // chunk of all close theirs
            const bool closes = c0.r != 0 || ends || !more;
            if (c0.r == 0) c0 = c;
            else c1 = c;
            if (!closes) continue;
            if (ends) {
                nfirst = 0;
                at_first = 0;
            }
            const bool pair = c0.r != 0;
            Chunks next;
            if (pair) next = load(c0, c1);
            if (loaded) chunk(cur, !pair || cut);
            if (!pair || enough()) return;
            cur = next;
            loaded = true;
            cut = ends;
            c0.r = 0;
            c1.r = 0;
        }
    };

    float worst = a.R2;
    uint64_t L[K];
    uint32_t leaves = 0;
    bool over = false;
    // ---- first walk: an upper bound of every query's k-th distance
    {
        // Short lists take one result for every 2 RUN points, the smallest: this
        // loosens the bound little where few of the points are among the k
        // nearest, and cannot tighten it.  fcp, 1M uniform / mixture points: 0.318
        // -> 0.302 / 0.462 -> 0.451 ms with RUN 4 instead of 1; k = 8 with RUN 2:
        // 0.472 -> 0.486, with 4: 0.585 ms.
        constexpr int RUN = K <= 2 ? 4 : 1;
        float F[K];
#pragma unroll
        for (int j = 0; j < K; ++j) F[j] = j < K - a.k ? -PT_NONE : PT_NONE;
        uint32_t seen = 0;
        bool scaled = false;
        // scale of the first leaves found: their boxes and the queries within
        // half of COORD_CLAMP (points of later leaves beyond it are left out)
        auto set_scale = [&](float extent) {
            const float e = fmaxf(extent, qmax);
            s.set_query(0.5f * COORD_CLAMP / fmaxf(e, 1.0e-15f));
            s.set_threshold(0.0f);
            scaled = true;
        };
        auto insert = [&](float x) {
            if (K <= 8 || wave_any(x < F[K - 1])) {
#pragma unroll
                for (int j = K - 1; j > 0; --j) F[j] = __builtin_amdgcn_fmed3f(F[j - 1], x, F[j]);
                F[0] = fminf(F[0], x);
            }
        };
        auto bound_chunks = [&](const Chunks& ch, bool) {
            ++seen;
            u32x4 pa[2];
            s.template point_operands<true>(ch.p, ch.ok, pa[0], pa[1]);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const f32x16 acc_lo = products(pa[c], s.b_lo), acc_hi = products(pa[c], s.b_hi);
#pragma unroll
                for (int i = 0; i < 16; i += RUN) {
                    float lo = acc_lo[i], hi = acc_hi[i];
#pragma unroll
                    for (int e = 1; e < RUN; ++e) {
                        lo = fminf(lo, acc_lo[i + e]);
                        hi = fminf(hi, acc_hi[i + e]);
                    }
                    // both halves' results of the lane's own query
                    const u32x2 v = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi),
                                                                     false, false);
                    if (K <= 8) {
                        insert(fminf(__uint_as_float(v.x), __uint_as_float(v.y)));
                    } else {
                        insert(__uint_as_float(v.x));
                        insert(__uint_as_float(v.y));
                    }
                }
            }
        };
        auto expand_home = [&](int32_t r, int32_t lv, bool to_leaves) -> uint32_t {
            const float gap = child_gap(r, lv);
            uint64_t m = wave_ballot(gap <= 0.0f);
            uint32_t out;
            if (m) {
                const uint32_t all = uint32_t(m) | uint32_t(m >> 32);
                const uint32_t in = test_children(all, 0.0f);
                out = in ? in : all;
            } else {
                // no child overlaps the packet: the nearest one
                const float best = -both_halves_max(half_max(-gap));
                m = wave_ballot(gap == best);
                m &= ~(m - 1);
                out = uint32_t(m) | uint32_t(m >> 32);
            }
            if (to_leaves) {
                // a leaf holds 15 points or more: with longer lists its
                // sibling, then its cousins come along
                if (K > 8) out |= (out & 0x55555555u) << 1 | (out & 0xaaaaaaaau) >> 1;
                if (K > 16) out |= (out & 0x33333333u) << 2 | (out & 0xccccccccu) >> 2;
                if (lv < GL) out &= (1u << (1 << lv)) - 1u;
                for (uint32_t rest = out; rest && nhome < 32; rest &= rest - 1, ++nhome)
                    home = lane == nhome ? (r << lv) + int32_t(__builtin_ctz(rest)) : home;
                if (!scaled) {
                    float e = 0.0f;
#pragma unroll
                    for (int j = 0; j < D; ++j) e = fmaxf(e, fmaxf(fabsf(bl[j] - s.c[j]), fabsf(bh[j] - s.c[j])));
                    const bool mine = (out >> (lane & 31u)) & 1u;
                    set_scale(both_halves_max(half_max(mine ? e : 0.0f)));
                }
            }
            return out;
        };
        if (a.shape.leaf_group == 0) {
            float e = 0.0f;
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const float* b = a.boxes + box_words(D);
                e = fmaxf(e, fmaxf(fabsf(b[j] - s.c[j]), fabsf(b[box_words(D) / 2 + j] - s.c[j])));
            }
            set_scale(e);
        }
        walk(0, false, expand_home, bound_chunks, [&]() { return seen >= MAX_HOME; });
        // back from scaled units; the last terms cover the rounding and
        // underflow of that
        const float d = fmaxf(F[K - 1] + s.qq, 0.0f);
        const float inv = 1.0f / s.scale;
        const float b = (d + packet_slack(s.qn, __builtin_amdgcn_sqrtf(d) + 0.02f)) * inv * inv * 1.00001f + 1.0e-37f;
        worst = F[K - 1] < BOUND_MAX ? fminf(worst, b) : worst;
    }
    // queries that found too few points to be bounded are left over
    {
        const bool open = s.active & !(worst <= COORD_MAX);
        hand_over(open, a.R2);
        s.active = s.active & !open;
        if (!wave_any(s.active)) return;
        worst = s.active ? worst : 0.0f;
    }

    // ---- second walk: every group within the bounds
    {
        const uint64_t sent = make_key(worst, SENT_IDX);
#pragma unroll
        for (int j = 0; j < K; ++j) L[j] = j < K - a.k ? uint64_t(0) : sent;
    }
    {
        const float reach = s.active ? qlen + __builtin_amdgcn_sqrtf(worst) : 0.0f;
        s.set_query(PACKET_SCALE / fmaxf(1.001f * both_halves_max(half_max(reach)), 1.0e-15f));
    }
    auto refresh = [&]() {
        worst = key_d2(L[K - 1]);
        const float r = __builtin_amdgcn_sqrtf(worst) * s.scale;
        s.set_threshold(s.qq - r * r - packet_slack(s.qn, r));
    };
    refresh();
    uint32_t ncand = 0;  // candidates of the lane's query in the queue
    uint32_t npend = 0;  // chunks held
    auto insert_queue = [&]() {
        // every lane takes its next candidates, two at a time; lanes without
        // one read some held point and insert the largest key, which changes
        // nothing
        auto key_at = [&](uint32_t i) -> uint64_t {
            const uint32_t at = held_entry(queue[i * 64u + lane], NPEND * 64u);
            const float4 w = pt[at];
            float p[D];
            p[0] = w.x;
            p[1] = w.y;
            p[2] = w.z;
            if (D > 3) p[D > 3 ? 3 : 0] = w.w;
            const float dx0 = s.q[0] - p[0];
            float d2 = dx0 * dx0;
#pragma unroll
            for (int j = 1; j < D; ++j) {
                const float dx = s.q[j] - p[j];
                d2 = d2 + dx * dx;
            }
            const int32_t idx = D == 3 ? __float_as_int(w.w) : pid[at];
            return (uint64_t(i < ncand ? __float_as_uint(d2) : NO_KEY) << 32) | uint32_t(idx);
        };
        for (uint32_t i = 0; wave_any(i < ncand); i += 2) {
            const uint64_t k0 = key_at(i), k1 = key_at(i + 1);
            list_insert<K>(L, k0);
            list_insert<K>(L, k1);
        }
        ncand = 0;
    };
    auto scan_chunks = [&](const Chunks& ch, bool last) {
        const uint32_t base = npend * 64u;
        lds_order();  // other lanes read the entries held before
        {
            const uint32_t at = base + (lane & 32u) + uint32_t(s.slot);
            float4 w;
            w.x = ch.p[0];
            w.y = ch.p[1];
            w.z = ch.p[2];
            w.w = D == 3 ? __int_as_float(ch.idx) : (D == 4 ? ch.p[D > 3 ? 3 : 0] : 0.0f);
            pt[at] = w;
            if (D == 4) pid[at] = ch.idx;
        }
        lds_order();
        u32x4 pa[2];
        s.template point_operands<false>(ch.p, ch.ok, pa[0], pa[1]);
        uint32_t mask[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t m_lo = sign_bits(products(pa[c], s.b_lo)), m_hi = sign_bits(products(pa[c], s.b_hi));
            const u32x2 m = __builtin_amdgcn_permlane32_swap(m_lo, m_hi, false, false);
            mask[c] = m.x | (m.y << 16);
        }
        ++npend;
        bool batch = npend == NPEND || last;
        uint64_t todo = uint64_t(mask[0]) | (uint64_t(mask[1]) << 32);
        for (;;) {
            // every lane queues its candidates, until one lane's share is full
            while (wave_any(todo != 0)) {
                queue[ncand * 64u + lane] = uint8_t(base + first_bit(todo));
                ncand += todo != 0 ? 1u : 0u;
                todo &= todo - 1;
                if (wave_any(ncand == QCAP)) break;
            }
            const bool left = wave_any(todo != 0);
            batch = batch || left || (npend >= 2 && wave_any(ncand >= FLUSH));
            if (batch || wave_any(ncand == QCAP)) insert_queue();
            if (!left) break;
        }
        if (batch) {
            npend = 0;
            refresh();
        }
    };
    auto expand_in = [&](int32_t r, int32_t lv, bool to_leaves) -> uint32_t {
        const float gap = child_gap(r, lv);
        const uint64_t m = wave_ballot(gap <= half_max(worst));
        uint32_t mm = uint32_t(m) | uint32_t(m >> 32);
        if (to_leaves) {
            // leaves already taken
            for (uint32_t i = 0; i < nhome; ++i) {
                const uint32_t off = __builtin_amdgcn_readlane(uint32_t(home), i) - uint32_t(r << lv);
                mm &= off < 32u ? ~(1u << off) : ~0u;
            }
        }
        const uint32_t in = test_children(mm, worst);
        if (to_leaves) {
            leaves += uint32_t(__popc(in));
            over = leaves > a.leaf_limit;
            if (over) return 0;
        }
        return in;
    };
    walk(nhome, true, expand_in, scan_chunks, [&]() { return over; });
    if (over) {
        hand_over(s.active, worst);
        return;
    }
    // results
    if (!s.active) return;
    int32_t* oi = a.out_idx + int64_t(row) * a.k;
    float* od = a.out_d2 ? a.out_d2 + int64_t(row) * a.k : nullptr;
    const int off = K - a.k;
    if (K >= 4 && a.vec_store) {
#pragma unroll
        for (int j = 0; j < K; j += 4) {
            if (j >= off) {
                int32_t vi[4];
                float vd[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint64_t key = L[j + e < K ? j + e : 0];
                    const bool empty = uint32_t(key) == SENT_IDX;
                    vi[e] = empty ? -1 : int32_t(uint32_t(key));
                    vd[e] = empty ? __builtin_inff() : key_d2(key);
                }
                *reinterpret_cast<int4*>(oi + (j - off)) = make_int4(vi[0], vi[1], vi[2], vi[3]);
                if (od) *reinterpret_cast<float4*>(od + (j - off)) = make_float4(vd[0], vd[1], vd[2], vd[3]);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (j >= off) {
                const uint32_t id = uint32_t(L[j]);
                const bool empty = id == SENT_IDX;
                oi[j - off] = empty ? -1 : int32_t(id);
                if (od) od[j - off] = empty ? __builtin_inff() : key_d2(L[j]);
            }
        }
    }
}

template <int D, Source SRC>
hipError_t launch_packet_k(int K, const PacketArgs& a, int64_t packets, hipStream_t st) {
    // a multiple of 8 workgroups, so that the XCDs' shares cover every packet
    const dim3 g(unsigned((packets + 7) / 8 * 8)), b(64);
    switch (K) {
        case 1: hipLaunchKernelGGL((knn_packet<D, 1, SRC>), g, b, 0, st, a); break;
        case 2: hipLaunchKernelGGL((knn_packet<D, 2, SRC>), g, b, 0, st, a); break;
        case 4: hipLaunchKernelGGL((knn_packet<D, 4, SRC>), g, b, 0, st, a); break;
        case 8: hipLaunchKernelGGL((knn_packet<D, 8, SRC>), g, b, 0, st, a); break;
        case 16: hipLaunchKernelGGL((knn_packet<D, 16, SRC>), g, b, 0, st, a); break;
        case 32: hipLaunchKernelGGL((knn_packet<D, 32, SRC>), g, b, 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

// Leaves a packet may visit before its queries are handed over: about three
// times what a packet of uniform queries visits (k = 8: 38 in 3-D, 93 in 4-D),
// more in long calls, where a slow packet is not the call's tail.  3-D, k = 8,
// 1M Gaussian-mixture points and queries, limit 48 / 96 / 144 / 320 / 640:
// 0.84 / 0.70 / 0.80 / 1.01 / 1.03 ms; k = 16, 10M clustered: 45.2 / 31.4 /
// 27.3 / 24.4 / 24.3 ms; 4-D, k = 16, 1M mixture: 3.50 / 2.80 / 1.63 / 1.78 /
// 2.07 ms.
static uint32_t packet_leaf_limit(int dim, int K, uint32_t Q) {
    return (dim == 4 ? 192u : 96u) * (K > 16 ? 4u : (K > 8 ? 3u : 2u)) / 2u + Q / 49152u;
}

bool packet_tree(kd_tree t) {
    if (t->d_dims || t->N < 1) return false;
    for (int j = 0; j < t->dim; ++j)
        if (!(t->lo[j] >= -COORD_MAX) || !(t->hi[j] <= COORD_MAX)) return false;
    return true;
}

hipError_t launch_knn_packet(kd_tree t, int K, const PacketCall& c, hipStream_t st) {
    if (c.Q == 0) return hipSuccess;
    PacketArgs a = {};
    a.nodes = t->d_nodes;
    a.boxes = static_cast<const float*>(t->d_boxes);
    a.N = int32_t(t->N);
    a.shape = group_shape(t->N);
    a.sq = c.sq;
    a.Q = c.Q;
    a.k = c.k;
    a.R2 = c.R2;
    a.out_idx = c.out_idx;
    a.out_d2 = c.out_d2;
    a.vec_store = c.vec_store;
    a.leaf_limit = packet_leaf_limit(t->dim, K, c.Q);
    a.fb_count = c.fb_count;
    a.fb_recs = c.fb_recs;
    a.fb_w0 = c.fb_w0;
    const int64_t packets = (int64_t(c.Q) + 63) / 64;
    switch (t->dim) {
        case 3: return launch_packet_k<3, CALL>(K, a, packets, st);
        case 4: return launch_packet_k<4, CALL>(K, a, packets, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_knn_packet_jobs(int dim, int K, const PacketJobs& c, hipStream_t st) {
    if (c.packets == 0) return hipSuccess;
    PacketArgs a = {};
    a.leaf_limit = packet_leaf_limit(dim, K, c.n);
    a.fb_count = c.fb_count;
    a.fb_recs = c.fb_slot;
    a.fb_w0 = c.fb_w0;
    a.jobs = c.jobs;
    a.njobs = c.njobs;
    a.packets = c.packets;
    a.perm = c.perm;
    switch (dim) {
        case 3: return launch_packet_k<3, JOBS>(K, a, c.packets, st);
        case 4: return launch_packet_k<4, JOBS>(K, a, c.packets, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace kd
