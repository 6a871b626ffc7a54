// kd_wave.hip -- kNN with one wave per query: the answer's latency instead of
// its throughput.
//
// For calls with too few queries to fill the GPU with one lane each, for lists
// over 32 and for the queries the packet kernel leaves over.  A lane-by-lane
// walk is a chain of ~130 dependent node loads; here the wave's 64 lanes share
// the query:
//   * groups of levels (kd_groups.h): lane l tests the bounding box of child
//     group l % 32, so one load descends five levels;
//   * 64 points at a time (two leaves, one in each half of the wave), one lane
//     each: squared distances as everywhere (binary32, left to right), and
//     a vote for those that can enter the list;
//   * the k-best list lies across the lanes (lane i: the i-th smallest
//     (d2, index) key, so any k <= 64), an insertion is one shift of the lanes
//     behind its place; many candidates at once are sorted over the lanes and
//     merged (bitonic networks of DPP exchanges).
// Children are taken nearest first and again tested against the current k-th
// distance; a group's own points come after its children, when the radius is
// small.  Box distances are computed like point distances and rounding is
// monotone, so no point of the result is passed over (ties included): rows are
// the lane-by-lane traversal's, bit for bit.
//
// Bound by the latency of the group and point loads (a k = 8 query over 10K
// 3-D points: 6 box loads and about 8 pairs of leaves in sequence), then by
// vector issue once ~8 waves per SIMD run.  250 queries over 10K points, k =
// 8: 156 us lane by lane (sort, walk, hand-off: 8 launches), 13 us here.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kd_groups.h"
#include "kd_internal.h"
#include "kd_list.h"

namespace kd {

namespace {

struct WaveArgs {
    const void* nodes;       // TreeRec<D>[N + 2]
    const float* boxes;      // subtree boxes by node id
    int32_t N;
    GroupShape shape;
    const float* queries;    // caller [n][D] (NULL: recs)
    const void* recs;        // NodeRec<D>[]
    const float* w0;         // with recs: upper bounds of the k-th squared distances (NULL: R2)
    uint32_t n;
    const uint32_t* n_dev;   // number of recs, on the device (NULL: n)
    int k;
    float R2;
    int32_t* out_idx;
    float* out_d2;
    // jobs: what describes the tree and the outputs comes from the slot's job
    const BatchJob* jobs;
    int njobs;
    const uint32_t* slots;   // class slots (NULL: 0 .. n - 1)
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t NO_KEY = 0x7fe00000u;  // high word above every key's
// Candidates of 64 points that enter the list together: one by one they cost
// about 10 vector and 8 scalar instructions each, together 170.  In lists of 8
// and more the first points of a query and most of what a long list meets are
// that many.  150,001 2-D queries, k = 50: 0.377 -> 0.294 ms (from 12 on: 0.301,
// from 8 on: 0.313), 1M 3-D queries, k = 50: 3.45 -> 2.59, 250,000, k = 32: 0.684
// -> 0.560, 100,000, k = 8: 0.170 -> 0.166.
constexpr int MANY = 20;
constexpr int MERGE_K = 8;  // in shorter lists the test for it costs 8 %

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(int(old), int(v), CTRL, 0xf, 0xf, false));
}
// The value of the lane below; 0 in lane 0 (wave_shr:1).
__device__ __forceinline__ uint32_t shift_up(uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ uint32_t min_u32(uint32_t a, uint32_t b) { return a < b ? a : b; }

// Smallest of lanes 0-31, wave-uniform.
__device__ __forceinline__ uint32_t min_low_half(uint32_t v) {
    v = min_u32(v, dpp_u32<0xb1>(v, v));   // quad_perm 1,0,3,2
    v = min_u32(v, dpp_u32<0x4e>(v, v));   // quad_perm 2,3,0,1
    v = min_u32(v, dpp_u32<0x141>(v, v));  // row_half_mirror
    v = min_u32(v, dpp_u32<0x140>(v, v));  // row_mirror
    const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    return a < b ? a : b;
}

// The key of lane l ^ X (X = 1, 2, 3, 4, 7, 8, 15, 16, 31, 32, 63): DPP inside
// rows of 16 lanes, row and half swaps beyond.
template <int X>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    if constexpr (X == 1) return dpp_u32<0xb1>(v, v);
    else if constexpr (X == 2) return dpp_u32<0x4e>(v, v);
    else if constexpr (X == 3) return dpp_u32<0x1b>(v, v);
    else if constexpr (X == 7) return dpp_u32<0x141>(v, v);
    else if constexpr (X == 15) return dpp_u32<0x140>(v, v);
    else if constexpr (X == 8) return dpp_u32<0x128>(v, v);  // row_ror:8
    else if constexpr (X == 4) return lane_xor<3>(lane_xor<7>(v));
    else if constexpr (X == 16) {
        // x: every even row twice, y: every odd one
        const u32x2 s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (__lane_id() & 16u) ? s.x : s.y;
    } else if constexpr (X == 32) {
        const u32x2 s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (__lane_id() & 32u) ? s.x : s.y;
    } else if constexpr (X == 31) return lane_xor<16>(lane_xor<15>(v));
    else return lane_xor<32>(lane_xor<31>(v));
}
template <int X>
__device__ __forceinline__ uint64_t key_xor(uint64_t k) {
    return (uint64_t(lane_xor<X>(uint32_t(k >> 32))) << 32) | lane_xor<X>(uint32_t(k));
}
// One exchange with lane l ^ X: the lane without bit B keeps the smaller key.
template <int X, int B>
__device__ __forceinline__ uint64_t exchange(uint64_t k) {
    const uint64_t p = key_xor<X>(k);
    const uint64_t lo = key_min(k, p), hi = key_max(k, p);
    return (__lane_id() & uint32_t(B)) ? hi : lo;
}
// Ascending order of a bitonic sequence over the lanes of every group of 2 B.
template <int B>
__device__ __forceinline__ uint64_t bitonic(uint64_t k) {
    k = exchange<B, B>(k);
    if constexpr (B > 1) k = bitonic<B / 2>(k);
    return k;
}
// Ascending order over the lanes of every group of 2 B, from any order: the
// first exchange of a merge is with the mirrored lane.
template <int B>
__device__ __forceinline__ uint64_t sort_lanes(uint64_t k) {
    if constexpr (B > 1) k = sort_lanes<B / 2>(k);
    k = exchange<2 * B - 1, B>(k);
    if constexpr (B > 1) k = bitonic<B / 2>(k);
    return k;
}

template <int D, bool JOBS, bool MERGE>
__global__ __launch_bounds__(64) void knn_wave(WaveArgs a) {
    __shared__ float s_gap[MAX_GROUP_LEVELS][64];
    const uint32_t lane = __lane_id();
    const bool upper = lane >= 32;
    // chunk slot of the lane (see kd_groups.h)
    const int32_t slot = int32_t(lane & 31u);
    const int32_t slot_lv = slot ? 31 - __builtin_clz(uint32_t(slot)) : 0;
    const int32_t slot_off = slot - (1 << slot_lv);
    const uint32_t n = a.n_dev ? *a.n_dev : a.n;

    // workgroups of one XCD (blockIdx % 8) take neighbouring records
    const uint32_t part = (n + 7u) >> 3;
    for (uint32_t b = blockIdx.x; b < 8u * part; b += gridDim.x) {
        const uint32_t i = a.queries ? b : (b & 7u) * part + (b >> 3);
        if (i >= n) continue;
        uint32_t row = i;
        if constexpr (JOBS) {
            const uint32_t at = a.slots ? a.slots[i] : i;
            int lo = 0, hi = a.njobs - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (a.jobs[mid].slot_base <= at) lo = mid;
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
            a.recs = J.queries;
            row = at - J.slot_base;
        }
        const TreeRec<D>* __restrict__ g1 = reinterpret_cast<const TreeRec<D>*>(a.nodes);
        const int32_t* __restrict__ ids =
            rec_has_idx(D) ? nullptr : reinterpret_cast<const int32_t*>(g1 + (int64_t(a.N) + 2));
        const int32_t top_levels = a.shape.top_levels, leaf_group = a.shape.leaf_group;
        const bool six = a.shape.leaf_levels > GL;
        float q[D];
        float bound = a.R2;
        if constexpr (JOBS) {
#pragma unroll
            for (int j = 0; j < D; ++j) q[j] = static_cast<const float*>(a.recs)[size_t(row) * D + j];
            if (a.w0) bound = a.w0[i];
        } else if (a.queries) {
#pragma unroll
            for (int j = 0; j < D; ++j) q[j] = a.queries[size_t(i) * D + j];
        } else {
            const NodeRec<D>* r = reinterpret_cast<const NodeRec<D>*>(a.recs) + i;
#pragma unroll
            for (int j = 0; j < D; ++j) q[j] = r->c[j];
            row = uint32_t(r->idx);
            if (a.w0) bound = a.w0[i];
        }
        bool ordered = true;  // no NaN
#pragma unroll
        for (int j = 0; j < D; ++j) ordered = ordered & (q[j] == q[j]);

        uint64_t key = make_key(bound, SENT_IDX);  // lane i: the i-th smallest
        float worst = bound;                       // wave-uniform

        // 64 points, one a lane; the candidates enter one by one
        auto take = [&](const int32_t r0, const int32_t lv0, const bool six0, const int32_t r1, const int32_t lv1,
                        const bool six1) {
            const int32_t r = upper ? r1 : r0, lv = upper ? lv1 : lv0;
            const bool sx = upper ? six1 : six0;
            const int32_t id = sx ? (r << GL) + slot : (r << slot_lv) + slot_off;
            const bool ok = (sx | ((slot > 0) & (slot_lv < lv))) & (r != 0) & (id <= a.N);
            float p[D];
            int32_t idx;
            load_point<D>(g1, ids, ok ? id : 1, p, idx);
            const float dx0 = q[0] - p[0];
            float d2 = dx0 * dx0;
#pragma unroll
            for (int j = 1; j < D; ++j) {
                const float dx = q[j] - p[j];
                d2 = d2 + dx * dx;
            }
            uint64_t cand = wave_ballot(ok & (d2 <= worst));
            if (MERGE && __popcll(cand) >= MANY) {
                // all at once: sorted over the lanes, the smaller of the list and
                // the reversed candidates, and that bitonic sequence sorted
                uint64_t c = (ok & (d2 <= worst)) ? make_key(d2, idx) : uint64_t(NO_KEY) << 32;
                c = sort_lanes<32>(c);
                key = bitonic<32>(key_min(key, key_xor<63>(c)));
                worst = __uint_as_float(__builtin_amdgcn_readlane(uint32_t(key >> 32), a.k - 1));
                cand = 0;
            }
            while (cand) {
                const int l = __builtin_ctzll(cand);
                cand &= cand - 1;
                const uint64_t ck = (uint64_t(__builtin_amdgcn_readlane(__float_as_uint(d2), l)) << 32) |
                                    __builtin_amdgcn_readlane(uint32_t(idx), l);
                // the sorted list of the lane helpers, one slot a lane: slot j
                // becomes the candidate clamped to slots j - 1 and j
                const uint64_t prev = (uint64_t(shift_up(uint32_t(key >> 32))) << 32) | shift_up(uint32_t(key));
                key = key_max(prev, key_min(ck, key));
                worst = __uint_as_float(__builtin_amdgcn_readlane(uint32_t(key >> 32), a.k - 1));
                cand &= wave_ballot(d2 <= worst);
            }
        };

        if (ordered && leaf_group == 0) {
            take(1, GL, false, six && (1 << GL) <= a.N ? 1 : 0, GL, true);
        } else if (ordered) {
            uint32_t stack = 0;  // lane g: children of group level g still to visit
            int32_t g = 0, r = 1;
            bool fresh = true;   // the group at hand was just entered
            float gap = 0.0f;
            for (;;) {
                const int32_t lv = g == 0 ? top_levels : GL;
                uint32_t m;
                if (fresh) {
                    float bl[D], bh[D];
                    const bool none = (slot >> lv) != 0;
                    load_box<D>(a.boxes, none ? r : (r << lv) + slot, bl, bh);
                    gap = box_gap<D>(bl, bh, q, q);
                    m = uint32_t(wave_ballot(!none & (gap <= worst)));
                } else {
                    gap = s_gap[g][lane];
                    m = __builtin_amdgcn_readlane(stack, uint32_t(g)) & uint32_t(wave_ballot(gap <= worst));
                }
                if (g + 1 == leaf_group) {
                    // leaves nearest first, two chunks at a time, then the
                    // group's own points
                    int32_t part = 0;
                    bool own = true;
                    const uint32_t order = (__float_as_uint(gap) & ~31u) | uint32_t(slot);
                    while (m | uint32_t(part) | uint32_t(own)) {
                        int32_t cr[2] = {0, 0}, cl[2] = {GL, GL};
                        bool cs[2] = {false, false};
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            if (part) {
                                cr[h] = part;
                                cs[h] = true;
                                part = 0;
                            } else if (m) {
                                const uint32_t best = min_low_half((m >> slot) & 1u ? order : ~0u) & 31u;
                                m &= ~(1u << best);
                                cr[h] = (r << lv) + int32_t(best);
                                if (six && (cr[h] << GL) <= a.N) part = cr[h];
                            } else if (own) {
                                own = false;
                                cr[h] = r;
                                cl[h] = lv;
                            }
                        }
                        take(cr[0], cl[0], cs[0], cr[1], cl[1], cs[1]);
                        m &= uint32_t(wave_ballot(gap <= worst));
                    }
                } else if (m) {
                    if (fresh) s_gap[g][lane] = gap;
                    const uint32_t order = (__float_as_uint(gap) & ~31u) | uint32_t(slot);
                    const uint32_t best = min_low_half((m >> slot) & 1u ? order : ~0u) & 31u;
                    stack = lane == uint32_t(g) ? m & ~(1u << best) : stack;
                    r = (r << lv) + int32_t(best);
                    ++g;
                    fresh = true;
                    continue;
                } else {
                    take(r, lv, false, 0, 0, false);
                }
                // the group is done
                if (g == 0) break;
                --g;
                r >>= g == 0 ? top_levels : GL;
                fresh = false;
            }
        }
        if (lane < uint32_t(a.k)) {
            const bool empty = uint32_t(key) == SENT_IDX;
            a.out_idx[int64_t(row) * a.k + lane] = empty ? -1 : int32_t(uint32_t(key));
            if (a.out_d2) a.out_d2[int64_t(row) * a.k + lane] = empty ? __builtin_inff() : key_d2(key);
        }
    }
}

template <bool JOBS, bool MERGE>
hipError_t launch_wave_m(int dim, const WaveArgs& a, int grid, hipStream_t st) {
    const dim3 g(grid), b(64);
    switch (dim) {
        case 2: hipLaunchKernelGGL((knn_wave<2, JOBS, MERGE>), g, b, 0, st, a); break;
        case 3: hipLaunchKernelGGL((knn_wave<3, JOBS, MERGE>), g, b, 0, st, a); break;
        case 4: hipLaunchKernelGGL((knn_wave<4, JOBS, MERGE>), g, b, 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <bool JOBS>
hipError_t launch_wave(int dim, bool merge, const WaveArgs& a, int grid, hipStream_t st) {
    return merge ? launch_wave_m<JOBS, true>(dim, a, grid, st) : launch_wave_m<JOBS, false>(dim, a, grid, st);
}

}  // namespace

hipError_t launch_knn_wave(kd_tree t, const WaveCall& c, hipStream_t st) {
    if (c.n == 0) return hipSuccess;
    WaveArgs a = {};
    a.nodes = t->d_nodes;
    a.boxes = static_cast<const float*>(t->d_boxes);
    a.N = int32_t(t->N);
    a.shape = group_shape(t->N);
    a.queries = c.queries;
    a.recs = c.recs;
    a.w0 = c.w0;
    a.n = c.n;
    a.n_dev = c.n_dev;
    a.k = c.k;
    a.R2 = c.R2;
    a.out_idx = c.out_idx;
    a.out_d2 = c.out_d2;
    const int g = int(std::min<uint32_t>((c.n + 7u) / 8u * 8u, 1u << 22));
    return launch_wave<false>(t->dim, c.k >= MERGE_K, a, g, st);
}

hipError_t launch_knn_wave_jobs(int dim, int K, const WaveJobs& c, hipStream_t st) {
    if (c.n == 0) return hipSuccess;
    WaveArgs a = {};
    a.w0 = c.w0;
    a.n = c.n;
    a.n_dev = c.n_dev;
    a.jobs = c.jobs;
    a.njobs = c.njobs;
    a.slots = c.slots;
    const int g = int(std::min<uint32_t>((c.n + 7u) / 8u * 8u, 1u << 22));
    return launch_wave<true>(dim, K >= MERGE_K, a, g, st);
}

}  // namespace kd
