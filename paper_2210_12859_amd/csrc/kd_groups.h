// kd_groups.h -- the tree cut into groups of levels, for the kernels that
// take many nodes at a time.
//
// The tree of H levels is cut at depth Td: below it lie the leaves, subtrees
// of 5 or 6 levels (17 to 33 points on average); above it groups of GL = 5
// levels (31 points), the root group having the 1 to 5 levels left over.  A
// group of l levels has 2^l child groups, all of them present (Td is above the
// last two levels).  Points of a subtree are read in chunks of up to 32: slot
// j of a chunk (1 <= j < 2^l) is the j-th node of the subtree's top l <= 5
// levels in level order, id (r << floor(log2 j)) + j - 2^floor(log2 j) for
// root r; a leaf's sixth level, ids (r << 5) + j, is a chunk of its own.
#pragma once

#include <hip/hip_runtime.h>

#include "kd_internal.h"

namespace kd {

struct GroupShape {
    int32_t leaf_levels;  // levels of a leaf (1..6)
    int32_t top_levels;   // levels of the root group when it is no leaf (1..GL)
    int32_t leaf_group;   // group level of the leaves (0: the root is one)
};

namespace {

constexpr int GL = 5;
constexpr int MAX_GROUP_LEVELS = 8;  // N < 2^30: Td <= 25, at most 6 group levels

inline GroupShape group_shape(int64_t N) {
    GroupShape s;
    int H = 0, Td = 0;
    while (H < 31 && (int64_t(1) << H) <= N) ++H;
    while ((N >> Td) > 32) ++Td;
    s.leaf_levels = H - Td;
    s.top_levels = Td == 0 ? GL : (Td - 1) % GL + 1;
    s.leaf_group = Td == 0 ? 0 : (Td - s.top_levels) / GL + 1;
    return s;
}

inline void set_shape(BatchJob& j, int64_t N) {
    const GroupShape s = group_shape(N);
    j.leaf_levels = s.leaf_levels;
    j.top_levels = s.top_levels;
    j.leaf_group = s.leaf_group;
}
__device__ __forceinline__ GroupShape job_shape(const BatchJob& j) {
    return GroupShape{j.leaf_levels, j.top_levels, j.leaf_group};
}

template <int D>
__device__ __forceinline__ void load_point(const TreeRec<D>* g1, const int32_t* ids, int32_t id, float (&p)[D],
                                           int32_t& idx) {
    const uint4 w = *reinterpret_cast<const uint4*>(g1 + id);
    p[0] = __uint_as_float(w.x);
    p[1] = __uint_as_float(w.y);
    if constexpr (D == 2) {
        idx = int32_t(w.z);
    } else if constexpr (D == 3) {
        p[2] = __uint_as_float(w.z);
        idx = ids[id];
    } else {
        p[2] = __uint_as_float(w.z);
        p[3] = __uint_as_float(w.w);
        idx = int32_t(reinterpret_cast<const uint32_t*>(g1 + id)[4]);
    }
}

template <int D>
__device__ __forceinline__ void load_box(const float* boxes, int32_t id, float (&lo)[D], float (&hi)[D]) {
    const uint4* p = reinterpret_cast<const uint4*>(boxes + int64_t(id) * box_words(D));
    float w[8];
    const uint4 u = p[0];
    w[0] = __uint_as_float(u.x); w[1] = __uint_as_float(u.y); w[2] = __uint_as_float(u.z); w[3] = __uint_as_float(u.w);
    if (box_words(D) == 8) {
        const uint4 v = p[1];
        w[4] = __uint_as_float(v.x); w[5] = __uint_as_float(v.y); w[6] = __uint_as_float(v.z); w[7] = __uint_as_float(v.w);
    }
#pragma unroll
    for (int j = 0; j < D; ++j) {
        lo[j] = w[j];
        hi[j] = w[box_words(D) / 2 + j];
    }
}

// Squared distance from the box [qlo, qhi] (a point: qlo = qhi) to the box
// [lo, hi], summed like a point distance; never above the distance of any
// point of the second box from any query in the first (rounding is monotone).
template <int D>
__device__ __forceinline__ float box_gap(const float (&lo)[D], const float (&hi)[D], const float (&qlo)[D],
                                         const float (&qhi)[D]) {
    float d2 = 0.0f;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        const float o = fmaxf(fmaxf(lo[j] - qhi[j], qlo[j] - hi[j]), 0.0f);
        d2 = j == 0 ? o * o : d2 + o * o;
    }
    return d2;
}

}  // namespace

}  // namespace kd
