// kd_build_gpu.hip -- the canonical left-balanced k-d tree built on the GPU.
//
// The tree is the one every correct builder produces (Sec. 4): at level-order
// position n (split dimension floor(log2(n+1)) mod D) sits the element of
// rank leftSize(|S|) of the node's subtree set S, ordered by (split
// coordinate, caller index); smaller elements form the left subtree, larger
// ones the right.
//
// For each dimension d the points are sorted once by (coordinate d, caller
// index) into the list L_d (stable radix sorts of all dimensions together,
// starting from caller order); a point's place there is its rank in d.  Ranks
// are unique, so from here on a split is one rank and a side one comparison.
//
// Every point not yet placed belongs to one node of the current level (its
// segment).  The segments' sizes and starts follow from N alone (the tree is
// complete): with W = 2^(H-1-l) last-level slots under each node of level l
// and `last` nodes on the last level, segment s starts at
// s (W - 1) + min(last, s W) and holds (W - 1) + clamp(last - s W, 0, W)
// points.  Its root is the point of rank leftSize(size) among them.
//   * The top levels, until segments have at most 2047 points: two kernels a
//     level.  level_count sends every point to its child segment (its rank
//     against the last split) and counts segments per tile of L_d;
//     level_locate finds each segment's root: the tile where the counts reach
//     its rank, then the point in it.
//   * The lists are then grouped by segment (one stable radix sort of all D on
//     the segment number), and build_subtree finishes each segment in one
//     workgroup: the D lists in LDS, per level one look at L_d for the sides
//     and a stable partition of all lists.
//   * Trees with more than ten top levels group their lists after the tenth as
//     well, so that a tile of a list never holds more than two of its groups'
//     segments and the counts stay small.
// The result equals the host builder's and the oracle's byte for byte.  Bound
// by the chain of launches (41 at 300K 3-D points, 3 to 15 us each, the
// finishing one 45).  With a sort of the level's list by segment on every level
// instead it was 190 launches; kd_build, allocations and read-back included,
// sorts -> now, us: 1000 3-D points 540 -> 150, 100K 1220 -> 390, 300K 2180 ->
// 540, 1M 3040 -> 1450, 10M 24.3 -> 13.9 ms.
//
// Stored split dimensions (the widest rule): every segment of the level
// picks its own dimension, so all D lists are sorted by segment each level.
// In list L_d a segment's points are in coordinate order, so its extent in d
// is the coordinate of its last point minus that of its first; the largest
// extent (the lowest d on ties) is the segment's dimension, and its points
// are ranked in that dimension's list.  Each point is assigned once, by the
// list of its segment's dimension.  H levels of D sorts.
//
// Node records and subtree boxes are then written on the device as well.
#include <hip/hip_runtime.h>

#include "kd_internal.h"

namespace kd {

namespace {

constexpr uint32_t PLACED = 0xffffffffu;

// Radix key of a coordinate: unsigned order equals float order (-0 == +0).
__device__ __forceinline__ uint32_t coord_key(float f) {
    uint32_t b = __float_as_uint(f);
    if (b == 0x80000000u) b = 0;  // -0 orders as +0, ties then go by index
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Size of the left subtree of a complete tree of n nodes (the rank of the
// subtree root in its ordered set).
__device__ __forceinline__ int64_t left_size_dev(int64_t n) {
    if (n < 2) return 0;
    const int h = 63 - __builtin_clzll(uint64_t(n));   // n has h + 1 levels
    const int64_t full_above = (int64_t(1) << h) - 1;  // nodes above the last level
    const int64_t on_last = n - full_above;
    const int64_t half = int64_t(1) << (h - 1);        // last-level slots under the left child
    return (half - 1) + (on_last < half ? on_last : half);
}

// Segments of a level: W last-level slots under each, `last` nodes on the last
// level (of the whole tree, or of one subtree).
struct Shape {
    int64_t W, last;
    __device__ int64_t start(int64_t s) const {
        const int64_t sW = s * W;
        return s * (W - 1) + (last < sW ? last : sW);
    }
    __device__ int64_t size(int64_t s) const {
        const int64_t extra = last - s * W;
        return (W - 1) + (extra < 0 ? 0 : (extra > W ? W : extra));
    }
    // the segment of position j (segments of at least one point)
    __device__ int64_t at(int64_t j) const {
        const int64_t full = last / W;  // segments of 2 W - 1 points; then one between, then W - 1
        if (j < full * (2 * W - 1)) return j / (2 * W - 1);
        const int64_t beyond = j - full * (2 * W - 1) - size(full);
        return beyond < 0 ? full : full + 1 + beyond / (W > 1 ? W - 1 : 1);
    }
};

// of dimensions d0, d0 + 1, ...
__global__ void dim_keys(const float* __restrict__ pts, uint32_t N, int D, int d0, size_t stride,
                         uint32_t* __restrict__ k, uint32_t* __restrict__ v, uint32_t* __restrict__ bad) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const float f = pts[size_t(i) * D + d0 + blockIdx.y];
    if (!__builtin_isfinite(f)) *bad = 1u;
    k[blockIdx.y * stride + i] = coord_key(f);
    v[blockIdx.y * stride + i] = i;
}

// rank[d][p] = place of point p in L_d
__global__ void list_ranks(const uint32_t* __restrict__ L, uint32_t N, size_t stride, uint32_t* __restrict__ rank) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < N) rank[blockIdx.y * stride + L[blockIdx.y * stride + j]] = j;
}

// Splits of a level whose list is grouped by segment.
__global__ void grouped_splits(const uint32_t* __restrict__ Ld, const uint32_t* __restrict__ rank_d, uint32_t nseg,
                               Shape sh, uint32_t* __restrict__ split) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < nseg) split[s] = rank_d[Ld[sh.start(s) + left_size_dev(sh.size(s))]];
}

// The last split, not yet applied: point p of segment s goes to 2 s or 2 s + 1,
// or is the segment's root.  Several points at once, their loads in step.
struct Pending {
    const uint32_t* rank;   // in the split's dimension
    const uint32_t* split;  // by segment
    const uint32_t* seg;    // NULL: all points are in segment 0
    int32_t* order;         // of the level's first node
    template <int M>
    __device__ void children(const uint32_t (&p)[M], const bool (&valid)[M], bool write, uint32_t (&s)[M]) const {
        uint32_t r[M], at[M];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            s[i] = !valid[i] ? PLACED : (seg ? seg[p[i]] : 0u);
            r[i] = valid[i] ? rank[p[i]] : 0u;
        }
#pragma unroll
        for (int i = 0; i < M; ++i) at[i] = split[s[i] == PLACED ? 0u : s[i]];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const bool open = s[i] != PLACED;
            if (write && open && r[i] == at[i]) order[s[i]] = int32_t(p[i]);
            s[i] = !open || r[i] == at[i] ? PLACED : 2 * s[i] + (r[i] > at[i] ? 1u : 0u);
        }
    }
};

constexpr uint32_t TILE = 1024;        // list entries a workgroup counts
constexpr int TILE_ROUNDS = TILE / 256;
constexpr uint32_t MAX_COUNTERS = 512; // segments of a tile: 2^9 of one group, or 2^8 of each of two

// Counts of the level's segments in each tile of its list; the groups of
// segments the list is sorted by have at least TILE - 1 entries, so a tile
// touches at most two.
__global__ __launch_bounds__(256) void level_count(const uint32_t* __restrict__ Ld, uint32_t R, Pending pend,
                                                   Shape group, int base, int level, uint32_t counters,
                                                   uint32_t* seg, uint32_t* __restrict__ segL,
                                                   uint32_t* __restrict__ hist) {
    __shared__ uint32_t cnt[MAX_COUNTERS];
    const uint32_t t = threadIdx.x;
    const uint32_t j0 = blockIdx.x * TILE;
    cnt[t] = 0;
    cnt[t + 256] = 0;
    uint32_t p[TILE_ROUNDS], s[TILE_ROUNDS];
    bool valid[TILE_ROUNDS];
#pragma unroll
    for (int r = 0; r < TILE_ROUNDS; ++r) {
        const uint32_t j = j0 + r * 256 + t;
        valid[r] = j < R;
        p[r] = Ld[valid[r] ? j : R - 1];
    }
    const uint32_t c0 = base ? uint32_t(group.at(j0)) << (level - base) : 0u;
    pend.children(p, valid, true, s);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TILE_ROUNDS; ++r) {
        if (valid[r]) {
            seg[p[r]] = s[r];
            segL[j0 + r * 256 + t] = s[r];
        }
        if (counters <= 8) {
            for (uint32_t c = 0; c < counters; ++c) {
                const uint32_t m = uint32_t(__popcll(__ballot(s[r] - c0 == c)));
                if ((t & 63) == 0 && m) atomicAdd(&cnt[c], m);
            }
        } else if (s[r] - c0 < counters) {
            atomicAdd(&cnt[s[r] - c0], 1u);
        }
    }
    __syncthreads();
    for (uint32_t c = t; c < counters; c += 256) hist[size_t(blockIdx.x) * counters + c] = cnt[c];
}

// Exclusive prefix over the 256 threads of a workgroup, and the sum.
__device__ __forceinline__ uint32_t prefix256(uint32_t v, uint32_t* part, uint32_t* sum) {
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off);
        if (lane >= uint32_t(off)) x += y;
    }
    __syncthreads();  // part may still be read
    if (lane == 63) part[w] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (uint32_t i = 0; i < 4; ++i) {
        before += i < w ? part[i] : 0u;
        all += part[i];
    }
    *sum = all;
    return before + x - v;
}

// One workgroup per segment: the rank (in the level's dimension) of its root.
__global__ __launch_bounds__(256) void level_locate(const uint32_t* __restrict__ Ld, const uint32_t* __restrict__ rank,
                                                    const uint32_t* __restrict__ segL,
                                                    const uint32_t* __restrict__ hist, uint32_t R, Shape sh,
                                                    Shape group, int base, int level, uint32_t counters,
                                                    uint32_t* __restrict__ split) {
    __shared__ uint32_t part[4];
    __shared__ uint32_t found[2];
    const uint32_t s = blockIdx.x, g = s >> (level - base);
    const uint32_t lo = base ? uint32_t(group.start(g)) : 0u;
    const uint32_t hi = base ? lo + uint32_t(group.size(g)) : R;
    const uint32_t m = uint32_t(left_size_dev(sh.size(s)));
    const uint32_t t0 = lo / TILE, t1 = (hi - 1) / TILE;
    uint32_t before = 0, sum;
    if (threadIdx.x == 0) found[0] = t1 + 1;
    for (uint32_t tb = t0; tb <= t1; tb += 256) {
        const uint32_t t = tb + threadIdx.x;
        uint32_t v = 0;
        if (t <= t1) {
            // a tile's counters start at the group of its first entry
            const uint32_t g0 = base && t * TILE < lo ? g - 1 : g;
            v = hist[size_t(t) * counters + (s - (g0 << (level - base)))];
        }
        const uint32_t at = before + prefix256(v, part, &sum);
        if (at <= m && m < at + v) {
            found[0] = t;
            found[1] = m - at;
        }
        before += sum;
        if (before > m) break;
    }
    __syncthreads();
    const uint32_t tile = found[0];
    if (tile > t1) return;  // never: the counts are of these entries
    const uint32_t want = found[1];
    // each thread four entries in a row
    uint32_t hits = 0;
#pragma unroll
    for (uint32_t i = 0; i < TILE / 256; ++i) {
        const uint32_t j = tile * TILE + threadIdx.x * (TILE / 256) + i;
        if (j < R && segL[j] == s) hits |= 1u << i;
    }
    uint32_t at = prefix256(uint32_t(__popc(hits)), part, &sum);
    if (at <= want && want < at + uint32_t(__popc(hits))) {
        for (; at < want; ++at) hits &= hits - 1;
        split[s] = rank[Ld[tile * TILE + threadIdx.x * (TILE / 256) + uint32_t(__ffs(int(hits)) - 1)]];
    }
}

// Sort keys that group the lists by segment (placed points last).  applied:
// seg_out holds the segments after the last split already (it may be the
// split's own array).
__global__ void group_keys(const uint32_t* __restrict__ L, uint32_t R, size_t stride, Pending pend, bool applied,
                           uint32_t placed_key, uint32_t* seg_out, uint32_t* __restrict__ k) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= R) return;
    const uint32_t p[1] = {L[blockIdx.y * stride + j]};
    const bool valid[1] = {true};
    uint32_t s[1];
    if (applied) s[0] = seg_out[p[0]];
    else pend.children(p, valid, blockIdx.y == 0, s);
    k[blockIdx.y * stride + j] = s[0] == PLACED ? placed_key : s[0];
    if (blockIdx.y == 0 && !applied) seg_out[p[0]] = s[0];
}

// The levels from `top` on, one segment of that level per workgroup: its
// points, at most MAX_SUB, are entries [start, start + size) of every list.
// Bound by vector issue and the chain of LDS steps and barriers (3 a level).
// Two workgroups of 16 waves fill a CU; with 2047 points they take 27 (2-D) to 43
// KB (4-D) of LDS each, with 4095 two would still fit in 2-D and 3-D, one in 4-D.
// 16 waves a workgroup instead of 8: 55 -> 45 us at 300K points.
constexpr int SUB_LEVELS = 11;
constexpr int MAX_SUB = (1 << SUB_LEVELS) - 1;
constexpr int SUB_ROWS = (MAX_SUB + 63) / 64;      // rows of 64 list entries
constexpr int SUB_WAVES = 16;
constexpr int SUB_ROUNDS = SUB_ROWS / SUB_WAVES;   // rows of a wave
template <int D>
__global__ __launch_bounds__(64 * SUB_WAVES) void build_subtree(const uint32_t* __restrict__ S, size_t stride,
                                                                uint32_t* __restrict__ slot, int top, int H,
                                                                int64_t last, int32_t* __restrict__ order) {
    __shared__ uint32_t point[MAX_SUB + 1];             // caller index of local point i
    __shared__ uint16_t list[2][D][MAX_SUB + 1];        // local points by coordinate, segment by segment
    __shared__ uint8_t side[MAX_SUB + 1];               // 0 left, 1 right, 2 placed on this level
    __shared__ uint32_t count[D][SUB_ROWS];             // lefts | rights << 16 of a row
    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint32_t s = blockIdx.x;
    const Shape whole{int64_t(1) << (H - 1 - top), last};
    const int64_t start = whole.start(s);
    const int32_t n = int32_t(whole.size(s));
    const int32_t slast = n - int32_t(whole.W - 1);     // this subtree's points on the last level
    if (n <= 0 || n > MAX_SUB) return;                  // never: every node of level `top` exists
    for (int32_t i = int32_t(t); i < n; i += 64 * SUB_WAVES) {
        const uint32_t p = S[start + i];
        point[i] = p;
        list[0][0][i] = uint16_t(i);
        slot[p] = uint32_t(i);
    }
    __threadfence_block();
    __syncthreads();
#pragma unroll
    for (int d = 1; d < D; ++d)
        for (int32_t i = int32_t(t); i < n; i += 64 * SUB_WAVES)
            list[0][d][i] = uint16_t(slot[S[d * stride + start + i]]);
    __syncthreads();

    int cur = 0, d = top % D;
    for (int l = top; l < H; ++l, d = d + 1 == D ? 0 : d + 1, cur ^= 1) {
        const int lgW = H - 1 - l;
        const int32_t W = 1 << lgW;
        const int32_t R = n - ((1 << (l - top)) - 1);   // points not yet placed
        const int32_t full = slast >> lgW;              // segments of 2 W - 1 points
        const float inv_full = 1.0f / float(2 * W - 1), inv_rest = 1.0f / float(W > 1 ? W - 1 : 1);
        const int32_t full_end = full * (2 * W - 1);
        const int32_t mid = (W - 1) + (slast - full * W);  // size of the segment between
        const int32_t rows = (R + 63) >> 6;
        // per entry of this thread: its segment and the segment's start and root
        int32_t sg[SUB_ROUNDS], first[SUB_ROUNDS], root[SUB_ROUNDS];
#pragma unroll
        for (int r = 0; r < SUB_ROUNDS; ++r) {
            const int32_t row = r * SUB_WAVES + int32_t(wave);
            const int32_t j = row * 64 + int32_t(lane);
            if (row >= rows) break;
            // j < 2048 and quotients of whole numbers: half a unit of margin
            // covers the rounding of the product
            int32_t sl;
            if (j < full_end) {
                sl = int32_t((float(j) + 0.5f) * inv_full);
            } else {
                const int32_t beyond = j - full_end - mid;
                sl = beyond < 0 ? full : full + 1 + int32_t((float(beyond) + 0.5f) * inv_rest);
            }
            const int32_t sW = sl * W;
            int32_t extra = slast - sW;
            extra = extra < 0 ? 0 : (extra > W ? W : extra);
            const int32_t half = W >> 1;
            sg[r] = sl;
            first[r] = sl * (W - 1) + (slast < sW ? slast : sW);
            root[r] = W > 1 ? (half - 1) + (extra < half ? extra : half) : 0;  // size of the left subtree
            if (j < R) {
                const uint32_t i = list[cur][d][j];
                const int32_t o = j - first[r];
                if (o == root[r]) {
                    order[((int64_t(1) << l) - 1) + (int64_t(s) << (l - top)) + sl] = int32_t(point[i]);
                    side[i] = 2;
                } else {
                    side[i] = o < root[r] ? 0 : 1;
                }
            }
        }
        if (l + 1 == H) break;
        __syncthreads();
        uint16_t it[D][SUB_ROUNDS];
        uint8_t sd[D][SUB_ROUNDS];
#pragma unroll
        for (int r = 0; r < SUB_ROUNDS; ++r) {
            const int32_t row = r * SUB_WAVES + int32_t(wave);
            const int32_t j = row * 64 + int32_t(lane);
            if (row >= rows) break;
#pragma unroll
            for (int e = 0; e < D; ++e) {
                it[e][r] = 0;
                sd[e][r] = 2;
                if (j < R) {
                    it[e][r] = list[cur][e][j];
                    sd[e][r] = side[it[e][r]];
                }
                const uint32_t c = uint32_t(__popcll(__ballot(sd[e][r] == 0))) |
                                   uint32_t(__popcll(__ballot(sd[e][r] == 1))) << 16;
                if (lane == 0) count[e][row] = c;
            }
        }
        __syncthreads();
        // lefts and rights of the rows before: lane i holds row i's
        uint32_t pre[D];
#pragma unroll
        for (int e = 0; e < D; ++e) {
            uint32_t c = int32_t(lane) < rows ? count[e][lane & (SUB_ROWS - 1)] : 0u, x = c;
#pragma unroll
            for (int off = 1; off < SUB_ROWS; off <<= 1) {
                const uint32_t y = __shfl_up(x, off);
                if (lane >= uint32_t(off)) x += y;
            }
            pre[e] = x - c;
        }
        const int32_t half = W >> 1;
        const int32_t lrest = slast - full * W;
#pragma unroll
        for (int r = 0; r < SUB_ROUNDS; ++r) {
            const int32_t row = r * SUB_WAVES + int32_t(wave);
            if (row >= rows) break;
            const int32_t sl = sg[r];
            // next level: starts of the two children, and how many lefts and
            // rights the segments before this one have
            const int32_t cl = 2 * sl * half, cr = cl + half;
            const int32_t startL = 2 * sl * (half - 1) + (slast < cl ? slast : cl);
            const int32_t startR = (2 * sl + 1) * (half - 1) + (slast < cr ? slast : cr);
            const int32_t lefts = sl * (half - 1) + (sl < full ? sl : full) * half +
                                  (sl > full ? (lrest < half ? lrest : half) : 0);
            const int32_t rights = startL - lefts;
#pragma unroll
            for (int e = 0; e < D; ++e) {
                const uint32_t p = __builtin_amdgcn_readlane(pre[e], row);
                const uint64_t b0 = __ballot(sd[e][r] == 0), b1 = __ballot(sd[e][r] == 1);
                const uint64_t lt = (uint64_t(1) << lane) - 1;
                const int32_t nl = int32_t(p & 0xffffu) + __popcll(b0 & lt);
                const int32_t nr = int32_t(p >> 16) + __popcll(b1 & lt);
                const int32_t to = sd[e][r] == 0 ? startL + nl - lefts : startR + nr - rights;
                if (sd[e][r] != 2) list[cur ^ 1][e][to & MAX_SUB] = it[e][r];
            }
        }
        __syncthreads();
    }
}

__global__ void fill_u32(uint32_t* __restrict__ p, uint32_t n, uint32_t v) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Widest rule: the lists' entries and their segments, for all lists.
__global__ void level_keys(const uint32_t* __restrict__ L, const uint32_t* __restrict__ seg, uint32_t N, size_t stride,
                           uint32_t placed_key, uint32_t* __restrict__ k, uint32_t* __restrict__ v) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= N) return;
    const size_t at = blockIdx.y * stride + j;
    const uint32_t p = L[at];
    const uint32_t s = seg[p];
    k[at] = s == PLACED ? placed_key : s;
    v[at] = p;
}

// Split dimension of each node of the level (widest rule): the extent of
// segment s in d is the coordinate of its last point minus its first's in
// the segment-sorted list S_d.
__global__ void segment_dims(const float* __restrict__ pts, int D, const uint32_t* __restrict__ S, size_t stride,
                             uint32_t nseg, int64_t W, int64_t last, int64_t first,
                             uint8_t* __restrict__ segdim, uint8_t* __restrict__ pos_dims) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nseg) return;
    const int64_t sW = int64_t(s) * W;
    const int64_t start = int64_t(s) * (W - 1) + (last < sW ? last : sW);
    int64_t extra = last - sW;
    extra = extra < 0 ? 0 : (extra > W ? W : extra);
    const int64_t size = (W - 1) + extra;  // >= 1: node first + s exists
    int best = 0;
    float best_ext = -1.0f;
    for (int d = 0; d < D; ++d) {
        const float lo = pts[size_t(S[d * stride + start]) * D + d];
        const float hi = pts[size_t(S[d * stride + start + size - 1]) * D + d];
        const float ext = hi - lo;
        if (ext > best_ext) {
            best_ext = ext;
            best = d;
        }
    }
    segdim[s] = uint8_t(best);
    pos_dims[first + s] = uint8_t(best);
}

// The points of list d whose segment splits in d (points in (segment,
// coordinate, index) order): place each segment's root, send the rest to the
// child segments.  The new segments go to seg_next, as the other lists still
// read seg.
__global__ void level_assign_widest(const uint32_t* __restrict__ S, size_t stride, const uint8_t* __restrict__ segdim,
                                    const uint32_t* __restrict__ seg, uint32_t R, int64_t W, int64_t last,
                                    int64_t first, int32_t* __restrict__ order, uint32_t* __restrict__ seg_next) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= R) return;
    const uint32_t d = blockIdx.y;
    const uint32_t p = S[d * stride + j];
    const int64_t s = seg[p];  // unplaced: the first R entries of the list
    if (segdim[s] != d) return;
    const int64_t sW = s * W;
    const int64_t start = s * (W - 1) + (last < sW ? last : sW);
    int64_t extra = last - sW;
    extra = extra < 0 ? 0 : (extra > W ? W : extra);
    const int64_t size = (W - 1) + extra;
    const int64_t m = left_size_dev(size);
    const int64_t o = int64_t(j) - start;
    if (o == m) {
        order[first + s] = int32_t(p);
        seg_next[p] = PLACED;
    } else {
        seg_next[p] = uint32_t(o < m ? 2 * s : 2 * s + 1);
    }
}

// Per node id: the split dimensions of the node and its three nearest
// ancestors, 2 bits each (own dimension in bits 0-1).
__global__ void pack_dims(const uint8_t* __restrict__ pos_dims, uint32_t N, uint8_t* __restrict__ out) {
    const uint32_t pos = blockIdx.x * blockDim.x + threadIdx.x;
    if (pos >= N) return;
    uint32_t a = pos + 1, b = 0;
    for (int m = 0; m < 4 && a >= 1; ++m, a >>= 1) b |= uint32_t(pos_dims[a - 1]) << (2 * m);
    out[pos + 1] = uint8_t(b);
}

// Node record of id pos + 1 (see TreeRec): coordinates, caller index (in the
// record or in the index array), ancestor splits (parent first).
template <int D>
__device__ __forceinline__ void pack_record(const float* __restrict__ pts, const int32_t* __restrict__ order,
                                            uint32_t N, const uint8_t* __restrict__ pos_dims, uint32_t pos,
                                            TreeRec<D>* __restrict__ r, float (&p)[D]) {
    constexpr int A0 = D + (rec_has_idx(D) ? 1 : 0);
    TreeRec<D> rec;
#pragma unroll
    for (int w = 0; w < rec_words(D); ++w) rec.w[w] = 0;
    const int32_t i = order[pos];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        p[j] = pts[size_t(i) * D + j];
        rec.w[j] = __float_as_uint(p[j]);
    }
    if constexpr (rec_has_idx(D)) rec.w[D] = uint32_t(i);
    else reinterpret_cast<int32_t*>(r + (size_t(N) + 2))[pos + 1] = i;
    uint32_t a = (pos + 1) >> 1;
#pragma unroll
    for (int m = 0; m < rec_ancestors(D); ++m) {
        if (a >= 1) {
            const int lvl = 31 - __builtin_clz(a);
            const int d = pos_dims ? int(pos_dims[a - 1]) : lvl % D;
            rec.w[A0 + m] = __float_as_uint(pts[size_t(order[a - 1]) * D + d]);
        }
        a >>= 1;
    }
    r[pos + 1] = rec;
}

// Records and subtree bounding boxes of levels [lo, hi), one subtree of level lo
// per workgroup: all its records first, each node's box begun as its point in
// LDS, then the levels bottom up: a box is the own point and the children's
// boxes (below the last level here: of the launch before).  One launch per
// level, through memory, cost 78 us at 300K points; this 24.
constexpr int PACK_LEVELS = 11;
template <int D>
__global__ __launch_bounds__(512) void pack_levels(const float* __restrict__ pts, const int32_t* __restrict__ order,
                                                   uint32_t N, const uint8_t* __restrict__ pos_dims, int lo, int hi,
                                                   TreeRec<D>* __restrict__ recs, float* boxes,
                                                   float* __restrict__ root_box) {
    constexpr int BW = box_words(D), HB = BW / 2;
    __shared__ float lds[2 * D][1 << PACK_LEVELS];  // box words of local node i (1-based)
    if (blockIdx.x == 0 && threadIdx.x == 0 && lo == 0) {
        // the padding before the first and behind the last node
        for (uint32_t id = 0; id <= N + 1; id += N + 1) {
            for (int w = 0; w < rec_words(D); ++w) recs[id].w[w] = 0;
            if constexpr (!rec_has_idx(D)) reinterpret_cast<int32_t*>(recs + (size_t(N) + 2))[id] = 0;
            for (int w = 0; w < BW; ++w) boxes[size_t(id) * BW + w] = 0.0f;
        }
    }
    const uint32_t top = (uint32_t(1) << lo) + blockIdx.x;
    const uint32_t nodes = uint32_t(1) << (hi - lo);
    // node id of local node i
    auto node = [&](uint32_t i) {
        const int l = 31 - __clz(int(i));
        return (top << l) + (i - (1u << l));
    };
    for (uint32_t i = 1 + threadIdx.x; i < nodes; i += 512) {
        const uint32_t id = node(i);
        if (id > N) continue;
        float p[D];
        pack_record<D>(pts, order, N, pos_dims, id - 1, recs, p);
#pragma unroll
        for (int j = 0; j < D; ++j) lds[j][i] = lds[D + j][i] = p[j];
    }
    __syncthreads();
    for (int l = hi - lo - 1; l >= 0; --l) {
        for (uint32_t i = (1u << l) + threadIdx.x; i < (2u << l); i += 512) {
            const uint32_t id = node(i);
            if (id > N) continue;
            float b[2 * D];
#pragma unroll
            for (int w = 0; w < 2 * D; ++w) b[w] = lds[w][i];
            for (uint32_t c = 0; c < 2 && 2 * id + c <= N; ++c) {
                float lows[D], highs[D];
                const float* cb = boxes + size_t(2 * id + c) * BW;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    lows[j] = 2 * i < nodes ? lds[j][2 * i + c] : cb[j];
                    highs[j] = 2 * i < nodes ? lds[D + j][2 * i + c] : cb[HB + j];
                }
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    // keep the current value unless the child's is strictly beyond it
                    // (the host builder's rule, so -0 / +0 come out the same)
                    b[j] = lows[j] < b[j] ? lows[j] : b[j];
                    b[D + j] = b[D + j] < highs[j] ? highs[j] : b[D + j];
                }
            }
            float out[BW] = {};
#pragma unroll
            for (int j = 0; j < D; ++j) {
                lds[j][i] = out[j] = b[j];
                lds[D + j][i] = out[HB + j] = b[D + j];
            }
            float4* o = reinterpret_cast<float4*>(boxes + size_t(id) * BW);
#pragma unroll
            for (int w = 0; w < BW / 4; ++w) {
                const float4 v = make_float4(out[4 * w], out[4 * w + 1], out[4 * w + 2], out[4 * w + 3]);
                o[w] = v;
                if (id == 1) {
                    root_box[4 * w] = v.x;
                    root_box[4 * w + 1] = v.y;
                    root_box[4 * w + 2] = v.z;
                    root_box[4 * w + 3] = v.w;
                }
            }
        }
        __syncthreads();
    }
    if (lo == 0 && int64_t(N) > FILL_POINTS) {
        // the boxes of FILL_LEVEL are this launch's or the one's before
        float rl[D], rh[D], sum = 0.0f;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            rl[j] = lds[j][1];
            rh[j] = lds[D + j][1];
        }
        for (uint32_t i = (1u << FILL_LEVEL) + threadIdx.x; i < (2u << FILL_LEVEL); i += 512) {
            float l[D], h[D];
#pragma unroll
            for (int j = 0; j < D; ++j) {
                l[j] = hi > FILL_LEVEL ? lds[j][i] : boxes[size_t(i) * BW + j];
                h[j] = hi > FILL_LEVEL ? lds[D + j][i] : boxes[size_t(i) * BW + HB + j];
            }
            sum += box_share<D>(l, h, rl, rh);
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) lds[0][threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < 8; ++w) sum += lds[0][w];
            root_box[ROOT_FILL] = sum;
        }
    }
}

inline dim3 grid_for(uint64_t n) { return dim3(unsigned((n + 255) / 256)); }

size_t pad(size_t bytes) { return (bytes + 255) & ~size_t(255); }

int tree_levels(int64_t N) {  // floor(log2 N) + 1
    int H = 0;
    while (H < 31 && (int64_t(1) << H) <= N) ++H;
    return H;
}

constexpr int GROUP_LEVELS = 10;  // top levels before the lists are grouped a first time

// The lists of all dimensions are sorted together, or one after another: where
// each fills the GPU, and where memory is short.  One after another needs keys
// and values to sort into for one list only.  Together / one by one, ms: by level
// 2.1M 2-D to 4-D points 2.77 / 2.79, 3.07 / 3.20, 3.45 / 3.62; 4.2M 5.30 / 5.19,
// 6.00 / 5.88, 6.82 / 6.57; 10M 12.9 / 12.3, 15.1 / 14.0, 17.3 / 15.6; 3-D by the
// widest rule 2.1M 7.95 / 9.56, 4.2M 17.6 / 18.9, 10M 50.8 / 48.7.
bool one_by_one(int64_t N, bool widest, bool tight) { return tight || N >= int64_t(1) << (widest ? 23 : 22); }

// Workspace of a build by level: lists, ranks and a segment array; all lists
// together: keys and values to sort them into (keys in the place of the ranks
// unless the lists are grouped twice), two more segment arrays and tile counts;
// one by one: three arrays for the sort, two of which the levels use too.  Then
// two levels of splits and sort counts.
struct LevelLayout {
    size_t stride, lists, one, splits, hist, sort, total;
    int top;
    bool single, spare;
    LevelLayout(int64_t N, int D, bool tight) {
        const int H = tree_levels(N);
        top = H > SUB_LEVELS ? H - SUB_LEVELS : 0;
        single = one_by_one(N, false, tight);
        spare = top > GROUP_LEVELS;
        stride = pad(size_t(N) * 4) / 4;
        lists = stride * 4 * size_t(D);
        one = stride * 4;
        splits = pad((size_t(1) << top) * 4);
        hist = top > 1 ? pad((size_t(N) / TILE + 1) * 4 * (spare ? MAX_COUNTERS : 1u << (top - 1))) : 0;
        sort = pad(sort_pairs_scratch_bytes(uint32_t(N)) * size_t(single ? 1 : D));
        total = (single ? lists * 2 + one * 4 : lists * (spare ? 5 : 4) + one * 3 + hist) + splits * 2 + sort;
    }
};

// Workspace of a build by the widest rule: lists sorted by coordinate and by
// segment, what the sorts need, two segment arrays, segment dimensions.
struct WidestLayout {
    size_t stride, lists, one, dims, sort, total;
    bool single;
    WidestLayout(int64_t N, int D, bool tight) {
        single = one_by_one(N, true, tight);
        stride = pad(size_t(N) * 4) / 4;
        lists = stride * 4 * size_t(D);
        one = stride * 4;
        dims = pad(size_t(N));
        sort = pad(sort_pairs_scratch_bytes(uint32_t(N)) * size_t(single ? 1 : D));
        total = lists * 2 + (single ? one : lists) * 3 + one * 2 + dims + sort;
    }
};

struct Carve {
    char* p;
    template <typename T = uint32_t>
    T* take(size_t bytes) {
        T* r = reinterpret_cast<T*>(p);
        p += bytes;
        return r;
    }
};

// L_d for every dimension, in L (ka, kb, vb are workspace).
kd_status sorted_lists(const float* d_pts, uint32_t n, int D, size_t stride, bool single, uint32_t* ka, uint32_t* L,
                       uint32_t* kb, uint32_t* vb, void* sort, uint32_t* d_bad, hipStream_t st) {
    const int step = single ? 1 : D;
    for (int d = 0; d < D; d += step) {
        uint32_t* va = L + size_t(d) * stride;
        hipLaunchKernelGGL(dim_keys, dim3(grid_for(n).x, step), dim3(256), 0, st, d_pts, n, D, d, stride, ka, va,
                           d_bad);
        KD_HIP(hipGetLastError());
        bool second = false;  // four passes: back in the first pair
        const kd_status s = sort_pairs(ka, va, kb, vb, n, 32, sort, st, &second, step, stride);
        if (s != KD_OK) return s;
    }
    return KD_OK;
}

kd_status build_widest_device(const float* d_pts, int64_t N, int D, int32_t* d_order, uint32_t* d_bad, void* ws,
                              uint8_t* d_pos_dims, bool tight, hipStream_t st) {
    const uint32_t n = uint32_t(N);
    const WidestLayout lay(N, D, tight);
    const size_t stride = lay.stride;
    Carve c{static_cast<char*>(ws)};
    uint32_t* L = c.take(lay.lists);   // by coordinate
    uint32_t* v0 = c.take(lay.lists);  // by segment
    uint32_t* k0 = c.take(lay.single ? lay.one : lay.lists);
    uint32_t* k1 = c.take(lay.single ? lay.one : lay.lists);
    uint32_t* v1 = c.take(lay.single ? lay.one : lay.lists);
    uint32_t* seg = c.take(lay.one);
    uint32_t* seg_next = c.take(lay.one);
    uint8_t* segdim = c.take<uint8_t>(lay.dims);
    void* sort = c.p;
    const dim3 g = grid_for(n), b(256);
    kd_status s = sorted_lists(d_pts, n, D, stride, lay.single, k0, L, k1, v1, sort, d_bad, st);
    if (s != KD_OK) return s;
    hipLaunchKernelGGL(fill_u32, g, b, 0, st, seg, n, 0u);
    KD_HIP(hipGetLastError());
    const int H = tree_levels(N);
    const int64_t last = N - ((int64_t(1) << (H - 1)) - 1);
    const int step = lay.single ? 1 : D;
    for (int l = 0; l < H; ++l) {
        const int64_t first = (int64_t(1) << l) - 1;
        const uint32_t R = uint32_t(N - first);
        const int64_t W = int64_t(1) << (H - 1 - l);
        const uint32_t* S = v0;
        for (int d = 0; d < D; d += step) {
            uint32_t* vd = v0 + size_t(d) * stride;
            // one by one the sorted list has to end in v0: with an odd number of
            // passes it starts in v1
            const bool odd = lay.single && ((l + 1 + 7) / 8) % 2 == 1;
            uint32_t *ka = odd ? k1 : k0, *va = odd ? v1 : vd, *kb = odd ? k0 : k1, *vb = odd ? vd : v1;
            hipLaunchKernelGGL(level_keys, dim3(g.x, step), b, 0, st, L + size_t(d) * stride, seg, n, stride,
                               uint32_t(1) << l, ka, va);
            KD_HIP(hipGetLastError());
            bool second = false;
            s = sort_pairs(ka, va, kb, vb, n, l + 1, sort, st, &second, step, stride);
            if (s != KD_OK) return s;
            // (one point is not sorted at all, and lies where it was written)
            if (!lay.single) S = second ? v1 : v0;
            else if (odd && !second) KD_HIP(hipMemcpyAsync(vd, va, size_t(n) * 4, hipMemcpyDeviceToDevice, st));
        }
        const int64_t nodes = std::min<int64_t>(int64_t(1) << l, N - first);
        hipLaunchKernelGGL(segment_dims, grid_for(uint64_t(nodes)), b, 0, st, d_pts, D, S, stride, uint32_t(nodes), W,
                           last, first, segdim, d_pos_dims);
        KD_HIP(hipGetLastError());
        KD_HIP(hipMemcpyAsync(seg_next, seg, size_t(n) * 4, hipMemcpyDeviceToDevice, st));
        hipLaunchKernelGGL(level_assign_widest, dim3(grid_for(R).x, D), b, 0, st, S, stride, segdim, seg, R, W, last,
                           first, d_order, seg_next);
        KD_HIP(hipGetLastError());
        std::swap(seg, seg_next);
    }
    return KD_OK;
}

template <int D>
kd_status build_by_level(const float* d_pts, int64_t N, int32_t* d_order, uint32_t* d_bad, void* ws, bool tight,
                         hipStream_t st) {
    const uint32_t n = uint32_t(N);
    const LevelLayout lay(N, D, tight);
    const size_t stride = lay.stride;
    const bool single = lay.single;
    Carve c{static_cast<char*>(ws)};
    uint32_t* L = c.take(lay.lists);
    uint32_t* rank = c.take(lay.lists);
    uint32_t* seg = c.take(lay.one);
    // the sorts' keys, and the keys and values they sort into; segments by list
    // entry, a second array of segments by point, tile counts
    uint32_t *k0, *k1, *v1, *segL, *seg2, *hist;
    if (single) {
        k0 = segL = c.take(lay.one);
        k1 = hist = c.take(lay.one);  // (N / 1024 + 1) 512 counts fit: N > 2047 where there are any
        v1 = c.take(lay.one);
        seg2 = seg;                   // each list's keys are made before the next list's
    } else {
        k0 = c.take(lay.lists);
        // before the ranks are made, and when they are not needed any more
        k1 = lay.spare ? c.take(lay.lists) : rank;
        v1 = c.take(lay.lists);
        segL = c.take(lay.one);
        seg2 = c.take(lay.one);
        hist = c.take(lay.hist);
    }
    uint32_t* split = c.take(lay.splits);
    uint32_t* split2 = c.take(lay.splits);
    void* sort = c.p;
    kd_status s = sorted_lists(d_pts, n, D, stride, single, k0, L, k1, v1, sort, d_bad, st);
    if (s != KD_OK) return s;
    const int H = tree_levels(N), top = lay.top;
    const int64_t last = N - ((int64_t(1) << (H - 1)) - 1);  // nodes on the last level
    auto shape = [&](int l) { return Shape{int64_t(1) << (H - 1 - l), last}; };
    uint32_t R = n;      // list entries
    int base = 0;        // the lists are grouped by the segments of this level
    const uint32_t* seg_now = nullptr;
    // the split of level l - 1 (in `split`)
    auto pending = [&](int l) {
        return Pending{rank + size_t((l - 1) % D) * stride, split, seg_now, d_order + ((int64_t(1) << (l - 1)) - 1)};
    };
    auto group_lists = [&](int l) -> kd_status {
        const int step = single ? 1 : D;
        for (int d = 0; d < D; d += step) {
            uint32_t* Ld = L + size_t(d) * stride;
            hipLaunchKernelGGL(group_keys, dim3(grid_for(R).x, step), dim3(256), 0, st, Ld, R, stride, pending(l),
                               d > 0, uint32_t(1) << l, seg2, k0);
            KD_HIP(hipGetLastError());
            bool second = false;
            const kd_status gs = sort_pairs(k0, Ld, k1, v1, R, l + 1, sort, st, &second, step, stride);
            if (gs != KD_OK) return gs;
            if (second && single) KD_HIP(hipMemcpyAsync(Ld, v1, size_t(R) * 4, hipMemcpyDeviceToDevice, st));
            else if (second) std::swap(L, v1);
        }
        seg_now = seg2;
        std::swap(seg, seg2);
        base = l;
        R = uint32_t(N - ((int64_t(1) << l) - 1));
        return KD_OK;
    };
    if (top > 0) {
        hipLaunchKernelGGL(list_ranks, dim3(grid_for(n).x, D), dim3(256), 0, st, L, n, stride, rank);
        KD_HIP(hipGetLastError());
    }
    for (int l = 0; l < top; ++l) {
        if (l == GROUP_LEVELS) {
            s = group_lists(l);
            if (s != KD_OK) return s;
        }
        const uint32_t* Ld = L + size_t(l % D) * stride;
        const uint32_t* rd = rank + size_t(l % D) * stride;
        const uint32_t nseg = uint32_t(1) << l;
        if (l == base) {
            hipLaunchKernelGGL(grouped_splits, grid_for(nseg), dim3(256), 0, st, Ld, rd, nseg, shape(l), split);
        } else {
            const uint32_t tiles = (R + TILE - 1) / TILE;
            const uint32_t counters = (uint32_t(1) << (l - base)) * (base ? 2u : 1u);
            hipLaunchKernelGGL(level_count, dim3(tiles), dim3(256), 0, st, Ld, R, pending(l), shape(base), base, l,
                               counters, seg, segL, hist);
            KD_HIP(hipGetLastError());
            seg_now = seg;
            hipLaunchKernelGGL(level_locate, dim3(nseg), dim3(256), 0, st, Ld, rd, segL, hist, R, shape(l), shape(base),
                               base, l, counters, split2);
            std::swap(split, split2);
        }
        KD_HIP(hipGetLastError());
    }
    if (top > 0) {
        s = group_lists(top);
        if (s != KD_OK) return s;
    }
    hipLaunchKernelGGL((build_subtree<D>), dim3(1u << top), dim3(64 * SUB_WAVES), 0, st, L, stride, segL, top, H, last,
                       d_order);
    KD_HIP(hipGetLastError());
    return KD_OK;
}

template <int D>
kd_status pack_tree(const float* d_pts, const int32_t* d_order, int64_t N, void* d_nodes, float* d_boxes,
                    float* root_box, const uint8_t* d_pos_dims, hipStream_t st) {
    for (int hi = tree_levels(N); hi > 0;) {
        const int lo = hi > PACK_LEVELS ? hi - PACK_LEVELS : 0;
        hipLaunchKernelGGL((pack_levels<D>), dim3(1u << lo), dim3(512), 0, st, d_pts, d_order, uint32_t(N), d_pos_dims,
                           lo, hi, static_cast<TreeRec<D>*>(d_nodes), d_boxes, root_box);
        KD_HIP(hipGetLastError());
        hi = lo;
    }
    return KD_OK;
}

}  // namespace

size_t build_scratch_bytes(int64_t N, int dim, bool widest, bool tight) {
    return widest ? WidestLayout(N, dim, tight).total : LevelLayout(N, dim, tight).total;
}

kd_status build_level_order_device(const float* d_pts, int64_t N, int D, int32_t* d_order, uint32_t* d_bad, void* ws,
                                   bool tight, hipStream_t st, uint8_t* d_pos_dims) {
    if (N <= 0) return KD_OK;
    if (d_pos_dims) return build_widest_device(d_pts, N, D, d_order, d_bad, ws, d_pos_dims, tight, st);
    switch (D) {
        case 2: return build_by_level<2>(d_pts, N, d_order, d_bad, ws, tight, st);
        case 3: return build_by_level<3>(d_pts, N, d_order, d_bad, ws, tight, st);
        default: return build_by_level<4>(d_pts, N, d_order, d_bad, ws, tight, st);
    }
}

kd_status pack_tree_device(const float* d_pts, const int32_t* d_order, int64_t N, int D, void* d_nodes,
                           float* d_boxes, float* root_box, hipStream_t st, const uint8_t* d_pos_dims,
                           uint8_t* d_dims) {
    if (N <= 0) return KD_OK;
    if (d_dims) {
        KD_HIP(hipMemsetAsync(d_dims, 0, size_t(N) + 2, st));
        hipLaunchKernelGGL(pack_dims, grid_for(uint64_t(N)), dim3(256), 0, st, d_pos_dims, uint32_t(N), d_dims);
        KD_HIP(hipGetLastError());
    }
    switch (D) {
        case 2: return pack_tree<2>(d_pts, d_order, N, d_nodes, d_boxes, root_box, d_pos_dims, st);
        case 3: return pack_tree<3>(d_pts, d_order, N, d_nodes, d_boxes, root_box, d_pos_dims, st);
        default: return pack_tree<4>(d_pts, d_order, N, d_nodes, d_boxes, root_box, d_pos_dims, st);
    }
}

}  // namespace kd
