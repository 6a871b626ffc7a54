// kd_range_packet.hip -- radius and box queries by packets: one wave answers 64
// neighbouring queries with one walk.
//
// The queries are sorted along the tree (kd_sort.hip), so the 64 regions of a
// wave lie close together and reach nearly the same nodes.  Lane by lane every
// query walks alone: a chain of node loads, and all lanes step as often as the
// longest walk.  Here the wave walks once, over groups of levels (kd_groups.h)
// in the order of the tree's pre-order:
//   * A group of l levels and its 2^l child groups, or a leaf of up to six
//     levels, is a complete tree of at most 63 items; lane j takes the item of
//     pre-order rank j.  It loads the item's point (or a child's bounding box)
//     and tests it against the bounding boxes of the regions of the wave's two
//     halves; children that pass are tested against every single region.
//   * The items that pass are then taken in rank order: a point, read back from
//     LDS, is tested by all 64 lanes against their own regions; a child is
//     entered, and the rest of its parent's items wait on a stack.
// So points are met in the traversal's order, which is the order the indices of
// the variable-length results have, whatever is left out on the way.
//
// Rows are the lane-by-lane kernel's: a point is in range by the same binary32
// expression, the k best keys are kept in the same sorted list, and what is left
// out cannot be in range (box distances are computed like point distances and
// rounding is monotone; the regions' bounding boxes are widened by more than
// the rounding of their corners).  Points that can enter a list wait in LDS
// until some lane's share is full; all lanes then insert together.
//
// Bound by vector and scalar issue (a point costs about 20 instructions for all
// 64 queries, an entered group about 150 and 18 for each child tested; in 3-D and
// 4-D the compiler chooses between an item's point and box by address, through 28
// and 48 bytes of private memory a lane).  Bounding
// boxes of 16 regions each: with 32 a call takes up to 4 % longer, with 8 up to
// 8 %, and without the test against every region 10 times as long on mixtures
// (packets across clusters).  Lane by lane -> here, 1M 3-D points and queries,
// the 8 best and the count at 8 in range: 0.85 -> 0.58 ms; all points of 300,007
// boxes over 400,000 mixture points, 48 each: 2.18 -> 0.93 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kd_groups.h"
#include "kd_internal.h"
#include "kd_list.h"

namespace kd {

namespace {

constexpr int QUEUE = 8;       // list candidates a lane holds before all are inserted
constexpr int ITEMS = 64;      // LDS slots per group level

struct RangePacketArgs {
    const void* nodes;         // TreeRec<D>[N + 2]
    const float* sboxes;       // subtree boxes by node id
    int32_t N;
    GroupShape shape;
    const void* recs;          // NodeRec<D>[Q], sorted: the query point or the box's centre
    const float* boxes;        // box queries: caller float [Q][2][D]
    uint32_t Q;
    float R2;
    int cap;
    int vec_store;
    int32_t* out_idx;
    float* out_d2;
    uint32_t* out_count;
    const int64_t* fill_off;
    int64_t fill_cap;
    int32_t* fill_idx;
};

// A query's region: load() tells whether any point can be in it, bounds() a box
// around it, reaches() whether a box can hold a point of it, has() whether a
// point is in it and the high word of its list key.
template <int D>
struct Ball {
    static constexpr bool kBox = false;
    static constexpr int kUnroll = 1;  // 2: counts up to 9 % slower
    float q[D];
    __device__ __forceinline__ bool load(const NodeRec<D>& r, const float*, float R2) {
        bool ok = true;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            q[j] = r.c[j];
            // NaN: nothing; infinite: nothing, or everything without a bound
            ok = ok & (fabsf(q[j]) < __builtin_inff() || (q[j] == q[j] && R2 == __builtin_inff()));
        }
        return ok;
    }
    __device__ __forceinline__ void bounds(float R2, float (&lo)[D], float (&hi)[D]) const {
        // the added term covers squares that underflow
        const float r = __builtin_amdgcn_sqrtf(R2) * 1.000001f + 1.0e-18f;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float l = q[j] - r, h = q[j] + r;
            const bool all = R2 == __builtin_inff();
            lo[j] = all ? -__builtin_inff() : l - fabsf(l) * 2.4e-7f;
            hi[j] = all ? __builtin_inff() : h + fabsf(h) * 2.4e-7f;
        }
    }
    __device__ __forceinline__ bool reaches(const float (&l)[D], const float (&h)[D], float R2) const {
        return box_gap<D>(l, h, q, q) <= R2;
    }
    __device__ __forceinline__ bool has(const float (&p)[D], float R2, uint32_t& key_hi) const {
        float d2 = 0.0f;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float dx = q[j] - p[j];
            d2 = j == 0 ? dx * dx : d2 + dx * dx;
        }
        key_hi = __float_as_uint(d2);
        return d2 <= R2;
    }
    static __device__ __forceinline__ uint64_t empty_key(float R2) { return make_key(R2, SENT_IDX); }
};

template <int D>
struct Box {
    static constexpr bool kBox = true;
    static constexpr int kUnroll = 2;  // 400,000 mixture points, 300,007 boxes: 0.98 -> 0.89 ms (4: 0.89, 8: 0.99)
    float lo[D], hi[D];
    __device__ __forceinline__ bool load(const NodeRec<D>& r, const float* boxes, float) {
        const float* b = boxes + size_t(r.idx) * 2 * D;
        bool ok = true;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            lo[j] = b[j];
            hi[j] = b[D + j];
            ok = ok & (lo[j] <= hi[j]);  // empty, or a NaN bound: nothing
        }
        return ok;
    }
    __device__ __forceinline__ void bounds(float, float (&l)[D], float (&h)[D]) const {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            l[j] = lo[j];
            h[j] = hi[j];
        }
    }
    __device__ __forceinline__ bool reaches(const float (&l)[D], const float (&h)[D], float) const {
        bool in = true;
#pragma unroll
        for (int j = 0; j < D; ++j) in = in & (l[j] <= hi[j]) & (h[j] >= lo[j]);
        return in;
    }
    // the list key is (1, index), above the spare slots' key 0
    __device__ __forceinline__ bool has(const float (&p)[D], float, uint32_t& key_hi) const {
        bool in = true;
#pragma unroll
        for (int j = 0; j < D; ++j) in = in & (lo[j] <= p[j]) & (p[j] <= hi[j]);
        key_hi = 1u;
        return in;
    }
    static __device__ __forceinline__ uint64_t empty_key(float) { return (uint64_t(2) << 32) | SENT_IDX; }
};

// Largest of the SUB lanes around the lane.
constexpr int SUB = 16;
__device__ __forceinline__ float sub_max(float v) {
#pragma unroll
    for (int m = 1; m < SUB; m <<= 1) v = fmaxf(v, __shfl_xor(v, m));
    return v;
}
__device__ __forceinline__ float lane_value(float v, uint32_t l) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l));
}

// The node of pre-order rank j in a complete tree of `levels` levels: level and
// place in it; level 31 beyond the last.
__device__ __forceinline__ void preorder_item(uint32_t j, int32_t levels, int32_t& lv, int32_t& off) {
    lv = 0;
    off = 0;
    uint32_t rest = j;
    uint32_t size = (1u << levels) - 1u;  // of the subtree entered
    if (j >= size) {
        lv = 31;
        return;
    }
#pragma unroll
    for (int i = 0; i < GL; ++i) {
        size >>= 1;
        const bool down = rest != 0;
        const bool right = rest > size;
        rest = down ? rest - 1u - (right ? size : 0u) : 0u;
        lv += down ? 1 : 0;
        off = down ? 2 * off + (right ? 1 : 0) : off;
    }
}

enum Mode { COUNT, FILL, LIST };

template <int D, int K, class Qy, Mode MODE>
__global__ __launch_bounds__(64) void range_packet(RangePacketArgs a) {
    // the items' points, ITEMS per group level of the tree, then (4-D) their
    // caller indices
    extern __shared__ float4 pt[];
    int32_t* const pid = reinterpret_cast<int32_t*>(pt + (a.shape.leaf_group + 1) * ITEMS);
    __shared__ uint64_t queue[MODE == LIST ? (QUEUE + Qy::kUnroll) * 64 : 1];
    const TreeRec<D>* __restrict__ g1 = reinterpret_cast<const TreeRec<D>*>(a.nodes);
    const int32_t* __restrict__ ids =
        rec_has_idx(D) ? nullptr : reinterpret_cast<const int32_t*>(g1 + (int64_t(a.N) + 2));
    const uint32_t lane = __lane_id();
    // workgroups of one XCD (blockIdx % 8) take neighbouring packets
    const uint32_t first = ((blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * 64u;
    if (first >= a.Q) return;
    if (MODE == FILL && a.fill_off[a.Q] > a.fill_cap) return;
    const bool have = first + lane < a.Q;
    const NodeRec<D> rec = reinterpret_cast<const NodeRec<D>*>(a.recs)[have ? first + lane : first];
    const int32_t row = rec.idx;
    Qy s;
    const bool active = s.load(rec, a.boxes, a.R2) & have;
    // bounding boxes of the regions of every SUB lanes, wave-uniform
    float blo[64 / SUB][D], bhi[64 / SUB][D];
    {
        float l[D], h[D];
        s.bounds(a.R2, l, h);
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float lo = -sub_max(active ? -l[j] : -__builtin_inff());
            const float hi = sub_max(active ? h[j] : -__builtin_inff());
#pragma unroll
            for (int i = 0; i < 64 / SUB; ++i) {
                blo[i][j] = lane_value(lo, SUB * i);
                bhi[i][j] = lane_value(hi, SUB * i);
            }
        }
    }
    uint32_t count = 0;
    int64_t pos = MODE == FILL ? a.fill_off[row] : 0;
    const int64_t end = MODE == FILL ? a.fill_off[row + 1] : 0;
    uint64_t L[MODE == LIST ? K : 1];
    uint32_t held = 0;
    if constexpr (MODE == LIST) {
        // spare slots (beyond cap) hold key 0 in front
#pragma unroll
        for (int j = 0; j < K; ++j) L[j] = j < K - a.cap ? uint64_t(0) : Qy::empty_key(a.R2);
    }
    auto insert_held = [&]() {
        if constexpr (MODE == LIST) {
            for (uint32_t i = 0; wave_any(i < held); ++i) {
                const uint64_t key = queue[i * 64u + lane];
                list_insert<K>(L, i < held ? key : (uint64_t(0x7fe00000u) << 32));
            }
            held = 0;
        }
    };

    // this lane's item of a six-level tree, and of the root group's tree
    const int32_t top = a.shape.top_levels;
    int32_t lv6, off6, lvt, offt;
    preorder_item(lane, GL + 1, lv6, off6);
    preorder_item(lane, a.shape.leaf_group == 0 ? GL + 1 : top + 1, lvt, offt);
    const uint64_t child6 = wave_ballot(lv6 == GL), childt = wave_ballot(lvt == top);

    uint32_t stack_lo = 0, stack_hi = 0;  // lane g: items of group level g still to take
    int32_t g = 0, r = 1;
    uint64_t m;          // items of the current group still to take
    uint64_t children;   // those of its items that are child groups
    auto enter = [&]() {
        lds_order();  // other lanes read the items of the group here before
        const bool leaf = g == a.shape.leaf_group;
        const int32_t lv = g == 0 ? lvt : lv6, off = g == 0 ? offt : off6;
        children = leaf ? 0 : (g == 0 ? childt : child6);
        const bool child = !leaf & (lv == (g == 0 ? top : GL));
        const bool some = lv < 31;
        const int32_t id = some ? (r << lv) + off : r;
        const bool valid = some & (id <= a.N);
        float l[D], h[D];
        int32_t idx;
        load_point<D>(g1, ids, (valid & !child) ? id : r, l, idx);
        {
            float4 w;
            w.x = l[0];
            w.y = l[1];
            w.z = D == 2 ? __int_as_float(idx) : l[D > 2 ? 2 : 0];
            w.w = D == 3 ? __int_as_float(idx) : l[D > 3 ? 3 : 0];
            pt[g * ITEMS + int32_t(lane)] = w;
            if (D == 4) pid[g * ITEMS + int32_t(lane)] = idx;
        }
#pragma unroll
        for (int j = 0; j < D; ++j) h[j] = l[j];
        if (!leaf) {
            float bl[D], bh[D];
            load_box<D>(a.sboxes, child ? id : r, bl, bh);
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const float x = bl[j], y = bh[j];
                l[j] = child ? x : l[j];
                h[j] = child ? y : h[j];
            }
        }
        bool near = false;
#pragma unroll
        for (int i = 0; i < 64 / SUB; ++i) {
            bool in = valid;
#pragma unroll
            for (int j = 0; j < D; ++j) in = in & (l[j] <= bhi[i][j]) & (h[j] >= blo[i][j]);
            near = near | in;
        }
        m = wave_ballot(near);
        for (uint64_t c = m & children; c; c &= c - 1) {
            const uint32_t j = uint32_t(__builtin_ctzll(c));
            float cl[D], ch[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                cl[d] = lane_value(l[d], j);
                ch[d] = lane_value(h[d], j);
            }
            if (!wave_any(active & s.reaches(cl, ch, a.R2))) m &= ~(uint64_t(1) << j);
        }
        lds_order();  // (not between the loads above: that cost 3 to 4 % of a call)
    };
    enter();
    for (;;) {
        // points before the next child
        const uint64_t next = m & children;
        uint64_t run = next ? m & ((next & (0 - next)) - 1) : m;
        m &= ~run;
        while (run) {
            // kUnroll points at a time, so that their reads overlap; beyond the
            // last one it is repeated, and left out
            constexpr int UNROLL = Qy::kUnroll;
            float4 w[UNROLL];
            int32_t wi[UNROLL];
            bool some[UNROLL];
            uint32_t j = 0;
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                some[u] = run != 0;
                j = run ? uint32_t(__builtin_ctzll(run)) : j;
                run &= run - 1;
                w[u] = pt[g * ITEMS + int32_t(j)];
                if (D == 4 && MODE != COUNT) wi[u] = pid[g * ITEMS + int32_t(j)];
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                float p[D];
                p[0] = w[u].x;
                p[1] = w[u].y;
                if (D > 2) p[D > 2 ? 2 : 0] = w[u].z;
                if (D > 3) p[D > 3 ? 3 : 0] = w[u].w;
                uint32_t key_hi;
                const bool in = active & some[u] & s.has(p, a.R2, key_hi);
                count += in ? 1u : 0u;
                if constexpr (MODE != COUNT) {
                    const int32_t idx =
                        D == 2 ? __float_as_int(w[u].z) : (D == 3 ? __float_as_int(w[u].w) : wi[u]);
                    if constexpr (MODE == FILL) {
                        if (in & (pos < end)) a.fill_idx[pos] = idx;
                        pos += in ? 1 : 0;
                    } else {
                        const uint64_t key = (uint64_t(key_hi) << 32) | uint32_t(idx);
                        queue[held * 64u + lane] = key;
                        held += (in & (key < L[K - 1])) ? 1u : 0u;
                    }
                }
            }
            if (MODE == LIST && wave_any(held >= uint32_t(QUEUE))) insert_held();
        }
        if (m) {
            const uint32_t j = uint32_t(__builtin_ctzll(m));
            m &= m - 1;
            stack_lo = lane == uint32_t(g) ? uint32_t(m) : stack_lo;
            stack_hi = lane == uint32_t(g) ? uint32_t(m >> 32) : stack_hi;
            r = (r << (g == 0 ? top : GL)) + int32_t(__builtin_amdgcn_readlane(uint32_t(g == 0 ? offt : off6), j));
            ++g;
            enter();
        } else {
            if (g == 0) break;
            --g;
            r >>= g == 0 ? top : GL;
            m = uint64_t(uint32_t(__builtin_amdgcn_readlane(stack_lo, uint32_t(g)))) |
                uint64_t(uint32_t(__builtin_amdgcn_readlane(stack_hi, uint32_t(g)))) << 32;
            children = g == 0 ? childt : child6;
        }
    }
    insert_held();
    if (!have) return;
    a.out_count[row] = count;
    if constexpr (MODE == LIST) {
        int32_t* oi = a.out_idx + int64_t(row) * a.cap;
        float* od = (!Qy::kBox && a.out_d2) ? a.out_d2 + int64_t(row) * a.cap : nullptr;
        const int off = K - a.cap;
#pragma unroll
        for (int j = 0; j < K; j += 4) {
            int32_t vi[4];
            float vd[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t key = L[j + e];
                const bool empty = uint32_t(key) == SENT_IDX;
                vi[e] = empty ? -1 : int32_t(uint32_t(key));
                vd[e] = empty ? __builtin_inff() : key_d2(key);
            }
            if (a.vec_store) {
                if (j >= off) {
                    *reinterpret_cast<int4*>(oi + (j - off)) = make_int4(vi[0], vi[1], vi[2], vi[3]);
                    if (od) *reinterpret_cast<float4*>(od + (j - off)) = make_float4(vd[0], vd[1], vd[2], vd[3]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (j + e >= off) {
                        oi[j + e - off] = vi[e];
                        if (od) od[j + e - off] = vd[e];
                    }
            }
        }
    }
}

template <int D, class Qy>
hipError_t launch_mode(const RangePacketArgs& a, int grid, hipStream_t st) {
    const dim3 g(grid), b(64);
    const unsigned lds = unsigned(a.shape.leaf_group + 1) * ITEMS * (D == 4 ? 20 : 16);
    if (a.fill_idx) hipLaunchKernelGGL((range_packet<D, 1, Qy, FILL>), g, b, lds, st, a);
    else if (a.cap == 0) hipLaunchKernelGGL((range_packet<D, 1, Qy, COUNT>), g, b, lds, st, a);
    else if (a.cap <= 8) hipLaunchKernelGGL((range_packet<D, 8, Qy, LIST>), g, b, lds, st, a);
    else if (a.cap <= 16) hipLaunchKernelGGL((range_packet<D, 16, Qy, LIST>), g, b, lds, st, a);
    else if (a.cap <= 32) hipLaunchKernelGGL((range_packet<D, 32, Qy, LIST>), g, b, lds, st, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_range_packet(kd_tree t, const RangePacketCall& c, hipStream_t st) {
    if (c.Q == 0) return hipSuccess;
    RangePacketArgs a = {};
    a.nodes = t->d_nodes;
    a.sboxes = static_cast<const float*>(t->d_boxes);
    a.N = int32_t(t->N);
    a.shape = group_shape(t->N);
    a.recs = c.recs;
    a.boxes = c.boxes;
    a.Q = c.Q;
    a.R2 = c.R2;
    a.cap = c.cap;
    a.out_idx = c.out_idx;
    a.out_d2 = c.out_d2;
    a.out_count = c.out_count;
    a.fill_off = c.fill_off;
    a.fill_cap = c.fill_cap;
    a.fill_idx = c.fill_idx;
    auto aligned = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    a.vec_store = c.cap % 4 == 0 && aligned(c.out_idx) && aligned(c.out_d2);
    // a multiple of 8 workgroups, so that the XCDs' shares cover every packet
    const int grid = int(((c.Q + 63u) / 64u + 7u) / 8u * 8u);
    const bool box = c.boxes != nullptr;
    switch (t->dim) {
        case 2: return box ? launch_mode<2, Box<2>>(a, grid, st) : launch_mode<2, Ball<2>>(a, grid, st);
        case 3: return box ? launch_mode<3, Box<3>>(a, grid, st) : launch_mode<3, Ball<3>>(a, grid, st);
        case 4: return box ? launch_mode<4, Box<4>>(a, grid, st) : launch_mode<4, Ball<4>>(a, grid, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace kd
