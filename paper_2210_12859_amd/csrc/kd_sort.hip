// kd_sort.hip -- reorders query batches along a Z-order (Morton) curve, or by
// their paths down the tree (queries answered in packets), so that queries
// served together (one wave, one CU, one XCD) traverse the same
// parts of the tree.  The reorder changes only which lane serves a query and
// when, never a result.
//
// Stable LSD radix sort of (Morton code or path, caller row) on the top sort_bits
// bits, 8 bits per pass; one pass is three kernels:
//   radix_hist    per-tile digit counts                  -> hist[digit][tile]
//   radix_scan    per digit, exclusive scan over tiles (in place) + totals
//   radix_scatter stable rank of every key inside its tile (wave ballots over
//                 the digit bits + LDS counts over waves and rounds), written
//                 at digit base + tile offset + rank
// A tile is 2048 keys, 512 threads x 4 rounds; round r covers keys
// [r*512, (r+1)*512) of the tile.  The scatter first reorders its tile by
// digit in LDS and then writes each digit's run of keys to consecutive
// addresses, so the stores coalesce (about 8 keys per digit and tile for
// random digits) instead of touching a different cache line per key.
// (Measured against 4096-key tiles: equal at 1M and 10M queries, 20 % less
// sort time at 16K, where the larger tiles leave most CUs idle.)
//
// For a single tree the keys travel with the 16/32-byte traversal records
// (coordinates + caller row) instead of a row index, so no pass gathers at
// random: the first pass reads the queries and computes the codes itself, the
// last pass writes only the records, and the first kernel also clears the
// traversal's work counters.  A 16-bit sort is 6 kernels.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kd_internal.h"

namespace kd {

namespace {

constexpr int SCAN_THREADS = 256;    // radix_scan: one workgroup per digit
#ifndef KD_SORT_THREADS
#define KD_SORT_THREADS 512
#endif
#ifndef KD_SORT_ROUNDS
#define KD_SORT_ROUNDS 4
#endif
constexpr int TILE_THREADS = KD_SORT_THREADS;  // radix_hist / radix_scatter (>= 256: one thread per digit)
constexpr int TILE_WAVES = TILE_THREADS / 64;
constexpr int TILE_ROUNDS = KD_SORT_ROUNDS;
constexpr int SORT_TILE = TILE_THREADS * TILE_ROUNDS;  // keys per tile
static_assert(TILE_THREADS >= 256 && TILE_THREADS <= 1024 && TILE_THREADS % 64 == 0, "tile threads");

uint32_t sort_tiles(uint32_t n) { return (n + SORT_TILE - 1) / SORT_TILE; }
// Words of one list's counts and totals.
__host__ __device__ constexpr size_t list_words(uint32_t ntiles) { return 256 * size_t(ntiles) + 256 + 128; }

__device__ __forceinline__ uint32_t spread_bits(uint32_t v, int D) {
    // insert D-1 zero bits between the low bits of v
    if (D == 2) {
        v &= 0xffffu;
        v = (v | (v << 8)) & 0x00ff00ffu;
        v = (v | (v << 4)) & 0x0f0f0f0fu;
        v = (v | (v << 2)) & 0x33333333u;
        v = (v | (v << 1)) & 0x55555555u;
    } else if (D == 3) {
        v &= 0x3ffu;
        v = (v | (v << 16)) & 0x030000ffu;
        v = (v | (v << 8)) & 0x0300f00fu;
        v = (v | (v << 4)) & 0x030c30c3u;
        v = (v | (v << 2)) & 0x09249249u;
    } else {
        v &= 0xffu;
        v = (v | (v << 12)) & 0x000f000fu;
        v = (v | (v << 6)) & 0x03030303u;
        v = (v | (v << 3)) & 0x11111111u;
    }
    return v;
}

struct MortonArgs {
    const float* queries;
    uint32_t Q;
    float lo[4];
    float scale[4];  // (2^bits) / extent, 0 for a flat axis
};

// 32-bit code of D coordinates, most significant spatial bit in bit 31
// (D = 3 uses bits 2..31).  NaN maps to cell 0, outside the box clamps.
template <int D>
__device__ __forceinline__ uint32_t morton_code(const float* c, const float* lo, const float* scale) {
    constexpr int bits = D == 2 ? 16 : (D == 3 ? 10 : 8);
    const float maxc = float((1u << bits) - 1);
    uint32_t code = 0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        float u = (c[j] - lo[j]) * scale[j];
        u = u != u ? 0.0f : fminf(fmaxf(u, 0.0f), maxc);
        code |= spread_bits(uint32_t(u), D) << (D - 1 - j);
    }
    if (D == 3) code <<= 2;
    return code;
}

// One radix pass.  D = 0: keys and rows come from kin/vin and go to
// kout/vout.  D > 0: keys travel with NodeRec<D> records (coordinates +
// caller row) kin/rin -> kout/rout; FROM_Q computes the keys and records from
// the queries (row = slot), TO_REC writes only the records, to `rec`.
// (Kept within 152 bytes: a longer argument costs every launch another line of
// host memory, 0.3 us.)
struct SortPass {
    const uint32_t* kin;  // tree order, first pass: the paths, written by radix_hist
    const uint32_t* vin;
    const void* rin;      // tree order, first pass: TreeRec<D>[N + 2]
    uint32_t* kout;
    uint32_t* vout;
    void* rout;
    void* rec;
    MortonArgs m;
    uint32_t n;
    int shift;
    uint32_t ntiles;
    uint32_t stride;  // pair sorts: elements from one list to the next (grid.y lists)
    uint32_t* hist;
    uint32_t* totals;
    uint32_t* zero;   // cleared by radix_hist (nzero words), may be NULL
    uint32_t nzero;
    int32_t N;        // tree order: points,
    int levels;       // and levels of the paths (0: Morton codes)
};

template <int D>
__device__ __forceinline__ void load_query(const MortonArgs& m, uint32_t row, float* c) {
#pragma unroll
    for (int j = 0; j < D; ++j) c[j] = m.queries[size_t(row) * D + j];
}

// Paths of a thread's queries from the root, `levels` steps to the close child
// (left: 0), at the top of the key (3-D and 4-D: 2-D calls sort by Morton
// code).  The order is the tree's own, so it is as fine as the data is dense;
// the walks of a thread's queries go in step, so their loads overlap.  Bound by the gathers (64 lines a load once the paths
// part): the split coordinates of the first TOP_LEVELS levels are therefore
// staged in LDS.  1M queries: 30 us from the nodes alone, 22 us here.
constexpr int TOP_LEVELS = 12;  // a multiple of every D
template <int D>
__device__ __forceinline__ void tree_paths(const SortPass& p, uint32_t base, uint32_t (&key)[TILE_ROUNDS]) {
    __shared__ float top[1 << TOP_LEVELS];
    const TreeRec<D>* g1 = static_cast<const TreeRec<D>*>(p.rin);
    const int staged = p.levels < TOP_LEVELS ? p.levels : TOP_LEVELS;
    float c[TILE_ROUNDS][D];
    int32_t id[TILE_ROUNDS];
#pragma unroll
    for (int r = 0; r < TILE_ROUNDS; ++r) {
        const uint32_t i = base + r * TILE_THREADS + threadIdx.x;
        load_query<D>(p.m, i < p.n ? i : p.n - 1, c[r]);
        id[r] = 1;
    }
#pragma unroll
    for (int32_t i0 = 0; i0 < (1 << TOP_LEVELS); i0 += TILE_THREADS) {
        const int32_t i = i0 + int32_t(threadIdx.x);
        const int lv = 31 - __clz(i | 1);
        if (i < (1 << TOP_LEVELS)) top[i] = __uint_as_float(g1[i > 0 && i <= p.N ? i : 1].w[lv % D]);
    }
    __syncthreads();
    // levels [from, to), from a multiple of D: the split dimension is a constant
    auto descend = [&](int from, int to, auto split) {
        for (int l = from; l < to; l += D)
#pragma unroll
            for (int j = 0; j < D; ++j) {
                if (l + j >= to) break;
                float sv[TILE_ROUNDS];
#pragma unroll
                for (int r = 0; r < TILE_ROUNDS; ++r) sv[r] = split(id[r], j);
                // below the last level (incomplete): to the left
#pragma unroll
                for (int r = 0; r < TILE_ROUNDS; ++r)
                    id[r] = (id[r] << 1) | (id[r] <= p.N && c[r][j] - sv[r] > 0.0f ? 1 : 0);
            }
    };
    descend(0, staged, [&](int32_t i, int) { return top[i]; });
    descend(staged, p.levels, [&](int32_t i, int j) { return __uint_as_float(g1[i <= p.N ? i : 1].w[j]); });
#pragma unroll
    for (int r = 0; r < TILE_ROUNDS; ++r) key[r] = uint32_t(id[r]) << (32 - p.levels);
}

template <int D, bool FROM_Q, bool TREE = false>
__global__ __launch_bounds__(TILE_THREADS) void radix_hist(SortPass p) {
    __shared__ uint32_t cnt[256];
    const uint32_t t = threadIdx.x;
    if (t < 256) cnt[t] = 0;
    for (uint32_t i = blockIdx.x * TILE_THREADS + t; i < p.nzero; i += gridDim.x * TILE_THREADS) p.zero[i] = 0;
    __syncthreads();
    const uint32_t base = blockIdx.x * uint32_t(SORT_TILE);
    uint32_t path[TILE_ROUNDS];
    if constexpr (TREE) tree_paths<D>(p, base, path);
#pragma unroll
    for (int r = 0; r < TILE_ROUNDS; ++r) {
        const uint32_t i = base + r * TILE_THREADS + t;
        if (i < p.n) {
            uint32_t key;
            if constexpr (TREE) {
                key = path[r];
                const_cast<uint32_t*>(p.kin)[i] = key;
            } else if constexpr (FROM_Q) {
                float c[D > 0 ? D : 1];
                load_query<D>(p.m, i, c);
                key = morton_code<D>(c, p.m.lo, p.m.scale);
            } else {
                key = p.kin[D == 0 ? size_t(blockIdx.y) * p.stride + i : i];
            }
            atomicAdd(&cnt[(key >> p.shift) & 0xffu], 1u);
        }
    }
    __syncthreads();
    if constexpr (D == 0) p.hist += blockIdx.y * list_words(p.ntiles);
    if (t < 256) p.hist[size_t(t) * p.ntiles + blockIdx.x] = cnt[t];
}

// One block per digit: exclusive scan of hist[digit][0..ntiles) in place;
// totals[digit] = sum.
__global__ __launch_bounds__(SCAN_THREADS) void radix_scan(uint32_t* __restrict__ hist, uint32_t ntiles,
                                                           uint32_t* __restrict__ totals, size_t list_stride) {
    __shared__ uint32_t part[SCAN_THREADS];
    hist += blockIdx.y * list_stride;
    totals += blockIdx.y * list_stride;
    uint32_t* row = hist + size_t(blockIdx.x) * ntiles;
    const uint32_t per = (ntiles + SCAN_THREADS - 1) / SCAN_THREADS;
    const uint32_t b = threadIdx.x * per;
    const uint32_t e = b + per < ntiles ? b + per : ntiles;
    uint32_t s = 0;
    for (uint32_t i = b; i < e; ++i) s += row[i];
    part[threadIdx.x] = s;
    __syncthreads();
    // inclusive scan of part (Hillis-Steele)
    for (int off = 1; off < SCAN_THREADS; off <<= 1) {
        uint32_t v = threadIdx.x >= off ? part[threadIdx.x - off] : 0u;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    uint32_t run = threadIdx.x ? part[threadIdx.x - 1] : 0u;
    for (uint32_t i = b; i < e; ++i) {
        uint32_t v = row[i];
        row[i] = run;
        run += v;
    }
    if (threadIdx.x == SCAN_THREADS - 1) totals[blockIdx.x] = part[SCAN_THREADS - 1];
}

// Inclusive scan of v over the first 256 threads; every thread of the block
// takes part in the barriers.
__device__ __forceinline__ uint32_t scan256(uint32_t* buf, uint32_t v) {
    const uint32_t t = threadIdx.x;
    if (t < 256) buf[t] = v;
    __syncthreads();
    for (uint32_t off = 1; off < 256; off <<= 1) {
        uint32_t x = 0;
        if (t < 256 && t >= off) x = buf[t - off];
        __syncthreads();
        if (t < 256) buf[t] += x;
        __syncthreads();
    }
    return t < 256 ? buf[t] : 0u;
}

template <int D, bool FROM_Q, bool TO_REC>
__global__ __launch_bounds__(TILE_THREADS) void radix_scatter(SortPass p) {
    static_assert(D > 0 || (!FROM_Q && !TO_REC), "queries need a dimension");
    __shared__ uint32_t gbase[256];              // output position of the tile's first key of digit d
    __shared__ uint32_t lstart[256];             // tile position of the first key of digit d
    __shared__ uint32_t lnext[256];              // next free tile position of digit d
    __shared__ uint32_t sbuf[256];
    __shared__ uint32_t wcnt[TILE_WAVES][256];   // digit counts per wave -> prefix over waves
    __shared__ uint32_t skey[SORT_TILE];
    __shared__ uint32_t sval[SORT_TILE];         // tile index of the key
    const uint32_t t = threadIdx.x;
    const uint32_t w = t >> 6;
    const size_t list = D == 0 ? size_t(blockIdx.y) * p.stride : 0;
    if constexpr (D == 0) {
        p.hist += blockIdx.y * list_words(p.ntiles);
        p.totals += blockIdx.y * list_words(p.ntiles);
    }
    const uint32_t tile = blockIdx.x;
    const uint32_t tile0 = tile * uint32_t(SORT_TILE);
    const uint32_t tile_n = p.n - tile0 < uint32_t(SORT_TILE) ? p.n - tile0 : uint32_t(SORT_TILE);

    // digit bases: global (all smaller digits + this digit in earlier tiles)
    // and local (smaller digits in this tile)
    uint32_t tot = 0, before = 0, mine = 0;
    if (t < 256) {
        tot = p.totals[t];
        before = p.hist[size_t(t) * p.ntiles + tile];
        const uint32_t after = tile + 1 < p.ntiles ? p.hist[size_t(t) * p.ntiles + tile + 1] : tot;
        mine = after - before;
    }
    const uint32_t incl_tot = scan256(sbuf, tot);
    if (t < 256) gbase[t] = incl_tot - tot + before;
    __syncthreads();
    const uint32_t incl_mine = scan256(sbuf, mine);
    if (t < 256) {
        lstart[t] = incl_mine - mine;
        lnext[t] = incl_mine - mine;
    }
    for (uint32_t j = t; j < uint32_t(TILE_WAVES * 256); j += TILE_THREADS) (&wcnt[0][0])[j] = 0;
    __syncthreads();

    // rank the tile's keys stably by digit; LDS gets (key, tile index)
    const uint64_t lt_mask = (uint64_t(1) << (t & 63)) - 1;
#pragma unroll
    for (int r = 0; r < TILE_ROUNDS; ++r) {
        const uint32_t li = r * TILE_THREADS + t;
        const bool valid = li < tile_n;
        uint32_t key = 0, d = 0;
        if (valid) {
            const uint32_t i = tile0 + li;
            if constexpr (FROM_Q) {
                if (p.levels) {
                    key = p.kin[i];
                } else {
                    float c[D > 0 ? D : 1];
                    load_query<D>(p.m, i, c);
                    key = morton_code<D>(c, p.m.lo, p.m.scale);
                }
            } else {
                key = p.kin[list + i];
            }
            d = (key >> p.shift) & 0xffu;
        }
        // lanes of this wave holding the same digit
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t m = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? m : ~m;
        }
        const uint32_t rank = __popcll(peers & lt_mask);
        if (valid && rank == 0) wcnt[w][d] = __popcll(peers);
        __syncthreads();
        uint32_t round_total = 0;
        if (t < 256) {
            for (int ww = 0; ww < TILE_WAVES; ++ww) {
                const uint32_t c = wcnt[ww][t];
                wcnt[ww][t] = round_total;
                round_total += c;
            }
        }
        __syncthreads();
        if (valid) {
            const uint32_t pos = lnext[d] + wcnt[w][d] + rank;
            if (pos < uint32_t(SORT_TILE)) {  // always, as the counts come from the same keys
                skey[pos] = key;
                sval[pos] = li;
            }
        }
        __syncthreads();
        if (t < 256) {
            lnext[t] += round_total;
            for (int ww = 0; ww < TILE_WAVES; ++ww) wcnt[ww][t] = 0;
        }
        __syncthreads();
    }

    // write the digit runs out: consecutive tile positions of one digit go
    // to consecutive output positions; the payload is read from this tile's
    // slice of the input (a window of SORT_TILE entries)
    for (uint32_t j = t; j < tile_n; j += TILE_THREADS) {
        const uint32_t key = skey[j];
        const uint32_t src = tile0 + sval[j];
        const uint32_t d = (key >> p.shift) & 0xffu;
        const uint32_t off = gbase[d] + (j - lstart[d]);
        if (off >= p.n) continue;  // never, as above
        if constexpr (D == 0) {
            p.kout[list + off] = key;
            p.vout[list + off] = p.vin[list + src];
        } else {
            NodeRec<D> rec;
            if constexpr (FROM_Q) {
                load_query<D>(p.m, src, rec.c);
                rec.idx = int32_t(src);
            } else {
                rec = static_cast<const NodeRec<D>*>(p.rin)[src];
            }
            if constexpr (TO_REC) {
                static_cast<NodeRec<D>*>(p.rec)[off] = rec;
            } else {
                p.kout[off] = key;
                static_cast<NodeRec<D>*>(p.rout)[off] = rec;
            }
        }
    }
}

// Identity order: copy the queries into records, clear the work counters.
template <int D>
__global__ void copy_records(SortPass p) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < p.nzero) p.zero[i] = 0;
    if (i >= p.n) return;
    NodeRec<D> rec;
    load_query<D>(p.m, i, rec.c);
    rec.idx = int32_t(i);
    static_cast<NodeRec<D>*>(p.rec)[i] = rec;
}

// Job of class slot i (jobs sorted by slot_base).
__device__ __forceinline__ int find_job(const BatchJob* jobs, int njobs, uint32_t i) {
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].slot_base <= i) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// key = job index in the top jb bits, the job-local Morton code below
__global__ void batch_morton_codes(const BatchJob* __restrict__ jobs, int njobs, int D, int jb, uint32_t n,
                                   uint32_t* __restrict__ codes, uint32_t* __restrict__ vals) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int j = find_job(jobs, njobs, i);
    const BatchJob& J = jobs[j];
    const uint32_t row = i - J.slot_base;
    float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int d = 0; d < D; ++d) c[d] = J.queries[size_t(row) * D + d];
    uint32_t code;
    switch (D) {
        case 2: code = morton_code<2>(c, J.lo, J.scale); break;
        case 3: code = morton_code<3>(c, J.lo, J.scale); break;
        default: code = morton_code<4>(c, J.lo, J.scale); break;
    }
    codes[i] = jb > 0 ? (uint32_t(j) << (32 - jb)) | (code >> jb) : code;
    vals[i] = i;
}

// key = job index in the top jb bits, the path from the job's root below it
// (as many levels as the tree has whole ones and `bits` holds)
template <int D>
__global__ void batch_path_codes(const BatchJob* __restrict__ jobs, int njobs, int jb, int bits, uint32_t n,
                                 uint32_t* __restrict__ codes, uint32_t* __restrict__ vals) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int j = find_job(jobs, njobs, i);
    const BatchJob& J = jobs[j];
    const TreeRec<D>* g1 = static_cast<const TreeRec<D>*>(J.nodes);
    const float* q = J.queries + size_t(i - J.slot_base) * D;
    float c[D];
#pragma unroll
    for (int d = 0; d < D; ++d) c[d] = q[d];
    const int whole = 31 - __clz(J.N);
    const int levels = whole < bits ? whole : bits;
    uint32_t id = 1;
    for (int l = 0; l < levels; l += D) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (l + d < levels) id = (id << 1) | (c[d] - __uint_as_float(g1[id].w[d]) > 0.0f ? 1u : 0u);
    }
    const uint32_t path = levels ? (id - (1u << levels)) << (32 - levels) : 0u;
    codes[i] = jb > 0 ? (uint32_t(j) << (32 - jb)) | (path >> jb) : path;
    vals[i] = i;
}

template <int D>
hipError_t launch_pass(const SortPass& p, bool first, bool last, hipStream_t st, unsigned lists = 1) {
    const dim3 g(p.ntiles), b(TILE_THREADS), bs(SCAN_THREADS);
    if constexpr (D == 0) {
        const dim3 gl(p.ntiles, lists);
        hipLaunchKernelGGL((radix_hist<0, false>), gl, b, 0, st, p);
        hipLaunchKernelGGL(radix_scan, dim3(256, lists), bs, 0, st, p.hist, p.ntiles, p.totals, list_words(p.ntiles));
        hipLaunchKernelGGL((radix_scatter<0, false, false>), gl, b, 0, st, p);
    } else {
        if (D > 2 && first && p.levels) hipLaunchKernelGGL((radix_hist<(D < 3 ? 3 : D), true, true>), g, b, 0, st, p);
        else if (first) hipLaunchKernelGGL((radix_hist<D, true>), g, b, 0, st, p);
        else hipLaunchKernelGGL((radix_hist<D, false>), g, b, 0, st, p);
        hipLaunchKernelGGL(radix_scan, dim3(256), bs, 0, st, p.hist, p.ntiles, p.totals, size_t(0));
        if (first && last) hipLaunchKernelGGL((radix_scatter<D, true, true>), g, b, 0, st, p);
        else if (first) hipLaunchKernelGGL((radix_scatter<D, true, false>), g, b, 0, st, p);
        else if (last) hipLaunchKernelGGL((radix_scatter<D, false, true>), g, b, 0, st, p);
        else hipLaunchKernelGGL((radix_scatter<D, false, false>), g, b, 0, st, p);
    }
    return hipGetLastError();
}

}  // namespace

size_t batch_sort_scratch_bytes(int64_t n) {
    const size_t ntiles = sort_tiles(uint32_t(n));
    return 4 * size_t(n) * sizeof(uint32_t) + (256 * ntiles + 256) * sizeof(uint32_t) + 256;
}

kd_status batch_sort(const BatchJob* d_jobs, int njobs, int dim, uint32_t n, int sort_bits, void* ws,
                     hipStream_t st, const uint32_t** perm_out, bool tree_order) {
    *perm_out = nullptr;
    if (n <= 1) return KD_OK;
    int jb = 0;
    while ((1 << jb) < njobs) ++jb;
    if (sort_bits <= 0) return KD_OK;  // class slots are already in job order
    SortPass p = {};
    p.n = n;
    p.ntiles = sort_tiles(n);
    uint32_t* k0 = reinterpret_cast<uint32_t*>(ws);
    uint32_t* v0 = k0 + n;
    uint32_t* k1 = v0 + n;
    uint32_t* v1 = k1 + n;
    p.hist = v1 + n;
    p.totals = p.hist + size_t(256) * p.ntiles;
    // the job bits must take part in the sort: sort on at least jb top bits
    int bits = sort_bits < jb ? ((jb + 7) / 8) * 8 : sort_bits;
    if (bits > 32) bits = 32;
    const dim3 g((n + 255) / 256), b(256);
    if (tree_order && dim == 3)
        hipLaunchKernelGGL(batch_path_codes<3>, g, b, 0, st, d_jobs, njobs, jb, bits - jb, n, k0, v0);
    else if (tree_order && dim == 4)
        hipLaunchKernelGGL(batch_path_codes<4>, g, b, 0, st, d_jobs, njobs, jb, bits - jb, n, k0, v0);
    else
        hipLaunchKernelGGL(batch_morton_codes, g, b, 0, st, d_jobs, njobs, dim, jb, n, k0, v0);
    KD_HIP(hipGetLastError());
    for (int q = 0; q < bits / 8; ++q) {
        p.shift = 32 - bits + 8 * q;
        p.kin = k0;
        p.vin = v0;
        p.kout = k1;
        p.vout = v1;
        KD_HIP(launch_pass<0>(p, false, false, st));
        uint32_t* tk = k0; k0 = k1; k1 = tk;
        uint32_t* tv = v0; v0 = v1; v1 = tv;
    }
    *perm_out = v0;
    return KD_OK;
}

size_t sort_pairs_scratch_bytes(uint32_t n) {
    return list_words(sort_tiles(n)) * sizeof(uint32_t);
}

kd_status sort_pairs(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, uint32_t n, int bits, void* ws,
                     hipStream_t st, bool* in_second, int lists, size_t stride) {
    *in_second = false;
    if (n <= 1 || bits <= 0) return KD_OK;
    SortPass p = {};
    p.n = n;
    p.ntiles = sort_tiles(n);
    p.stride = uint32_t(stride);
    p.hist = static_cast<uint32_t*>(ws);
    p.totals = p.hist + size_t(256) * p.ntiles;
    const int passes = (bits + 7) / 8;
    for (int q = 0; q < passes; ++q) {
        p.shift = 8 * q;
        p.kin = k0;
        p.vin = v0;
        p.kout = k1;
        p.vout = v1;
        KD_HIP(launch_pass<0>(p, false, false, st, unsigned(lists)));
        uint32_t* tk = k0; k0 = k1; k1 = tk;
        uint32_t* tv = v0; v0 = v1; v1 = tv;
        *in_second = !*in_second;
    }
    return KD_OK;
}

size_t sort_scratch_bytes(int64_t Q, int dim) {
    const size_t ntiles = sort_tiles(uint32_t(Q));
    const size_t rb = dim == 4 ? 32 : 16;
    return 2 * size_t(Q) * (sizeof(uint32_t) + rb) + (256 * ntiles + 256) * sizeof(uint32_t) + 512;
}

kd_status reorder_queries(kd_tree t, const float* queries, int64_t Q, int sort_bits, void* ws, void* sq,
                          uint32_t* zero, uint32_t nzero, hipStream_t st, bool tree_order) {
    const uint32_t n = uint32_t(Q);
    SortPass p = {};
    p.rec = sq;
    p.n = n;
    p.zero = zero;
    p.nzero = nzero;
    p.m.queries = queries;
    p.m.Q = n;
    const int bits = t->dim == 2 ? 16 : (t->dim == 3 ? 10 : 8);
    for (int j = 0; j < 4; ++j) {
        const float ext = t->hi[j] - t->lo[j];
        p.m.lo[j] = t->lo[j];
        p.m.scale[j] = (j < t->dim && ext > 0.0f) ? float(1u << bits) / ext : 0.0f;
    }
    if (sort_bits <= 0 || n <= 1) {
        const uint32_t m = n > nzero ? n : nzero;
        const dim3 g((m + 255) / 256), b(256);
        if (m == 0) return KD_OK;
        switch (t->dim) {
            case 2: hipLaunchKernelGGL(copy_records<2>, g, b, 0, st, p); break;
            case 3: hipLaunchKernelGGL(copy_records<3>, g, b, 0, st, p); break;
            default: hipLaunchKernelGGL(copy_records<4>, g, b, 0, st, p); break;
        }
        KD_HIP(hipGetLastError());
        return KD_OK;
    }
    p.ntiles = sort_tiles(n);
    const size_t rb = t->dim == 4 ? 32 : 16;
    char* w = static_cast<char*>(ws);
    void* r0 = w;
    void* r1 = w + size_t(n) * rb;
    uint32_t* k0 = reinterpret_cast<uint32_t*>(w + 2 * size_t(n) * rb);
    uint32_t* k1 = k0 + n;
    p.hist = k1 + n;
    p.totals = p.hist + size_t(256) * p.ntiles;
    if (tree_order) {
        int levels = 0;
        while (levels < 31 && (int64_t(2) << levels) <= t->N) ++levels;  // floor(log2 N)
        // Levels: cells of 16 to 32 queries, or 32 to 64 where the 16 levels of two
        // passes would leave more.  k = 8, 14 / 16 levels, ms: 300K uniform points
        // and queries 0.280 / 0.296, 1M 0.470 / 0.452; 16 / 18 / 20: 8M 3.58 / 3.41
        // / 3.54, 10M clustered, k = 16, 24.1 / 23.5 / 23.0; 17 levels at 2M and 4M
        // 4 % slower than 16 (the third pass).
        int q = 31 - __builtin_clz(n);  // floor(log2 Q)
        q = q >= 23 ? q - 5 : std::min(q - 4, 16);
        p.levels = std::max(1, std::min(levels, q));
        sort_bits = (p.levels + 7) / 8 * 8;
        p.N = int32_t(t->N);
    }
    const int passes = sort_bits / 8;
    for (int q = 0; q < passes; ++q) {
        p.shift = 32 - sort_bits + 8 * q;
        p.kin = k0;
        p.rin = q == 0 && p.levels ? t->d_nodes : r0;
        p.kout = k1;
        p.rout = r1;
        const bool first = q == 0, last = q == passes - 1;
        hipError_t e = t->dim == 2 ? launch_pass<2>(p, first, last, st)
                     : t->dim == 3 ? launch_pass<3>(p, first, last, st) : launch_pass<4>(p, first, last, st);
        KD_HIP(e);
        p.zero = nullptr;
        p.nzero = 0;
        uint32_t* tk = k0; k0 = k1; k1 = tk;
        void* tr = r0; r0 = r1; r1 = tr;
    }
    return KD_OK;
}

}  // namespace kd
