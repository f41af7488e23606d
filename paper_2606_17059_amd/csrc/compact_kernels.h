// compact_kernels.h -- rebuild the device forest without the records and
// labels that no peer's tree uses any more.
//
// Merges leave the old child blocks of rebuilt parents behind, and cleared or
// evicted peers leave nodes that no peer holds.  A node some peer holds has
// an ancestor chain of nodes that peer holds (masks never grow away from the
// root), so the live forest is the root plus every node with a non-empty mask
// that is reachable through such nodes.  The rebuild copies it level by level
// into fresh arrays.  New ids are given in that order (a level's nodes by their
// parents, children by token), so a level's frontier is a range of new ids and
// needs only the old id of each:
//   1. count: a wave per frontier node counts the children some peer holds; a
//      workgroup keeps its sixteen nodes' prefix and its total;
//   2. scan: one workgroup scans the totals and moves the range on;
//   3. copy: the kept children's records, first tokens, mask words and access
//      times go to their new ids, and the parent's record is pointed at them;
//   4. after the last level, a scan of label lengths gives every node a span of
//      the new pool; labels are copied, with their narrow copy, and wide blocks
//      get their separators.
// Ranges and totals stay on the device: levels are enqueued several at a time
// (levels past the last find an empty range) and read back once, where a
// readback, a rocPRIM scan and a wait a level cost about 45 us each.
// A forest of at most kCompactSmall records takes steps 1 to 3 for all levels,
// and the label scan, in one workgroup and one launch.
// Measured, call included (with the arrays of the last compaction reused):
// 256,000 records and 23 M label tokens 1.8 -> 0.23 ms; 500 nodes, 15 levels 514 -> 98 us.
// The root stays node 0.  Match results, exports and access times are those of
// the old forest.
#ifndef PR_COMPACT_KERNELS_H
#define PR_COMPACT_KERNELS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "forest_layout.h"
#include "merge_kernels.h"

namespace pr {

constexpr int kCompactWaves = 16;                  // frontier nodes a workgroup counts together
constexpr int kCompactThreads = 64 * kCompactWaves;
constexpr int kCompactUnroll = 4;                  // 64-child chunks a wave has in flight
constexpr int kCompactLabTile = 4 * kCompactThreads;  // label lengths a workgroup scans
constexpr int64_t kCompactSmall = 8192;

struct CompactState {
    long long lo, hi;    // new ids of the next level's frontier
    long long flo, fhi;  // of the one being copied
    long long n_pool;    // label tokens of the new image
    unsigned long long hi_tokens, wide_tokens;  // a live label token is in [65536, 131071], past it
    long long bad;       // more live nodes than records
};

// Peer words of old node x: whether some peer holds it.  r: its record.
__device__ __forceinline__ bool node_has_peers(const DevForest &F, int64_t x, const Node &r) {
    uint64_t any = r.mask0;
    for (int w = 1; w < F.W; w++) any |= F.mext[x * (F.W - 1) + (w - 1)];
    return any != 0;
}

__device__ __forceinline__ void compact_copy_node(const DevForest &O, const DevForest &N, int64_t src, int64_t dst,
                                                  Node r, int32_t *old_of) {
    r.aux = 0;
    N.nodes[dst] = r;  // ct_beg, ct_cnt and lab_off follow
    N.ntok[dst] = r.tok;
    for (int w = 1; w < O.W; w++) N.mext[dst * (O.W - 1) + (w - 1)] = O.mext[src * (O.W - 1) + (w - 1)];
    if (O.ltime && N.ltime) N.ltime[dst] = O.ltime[src];
    old_of[dst] = (int32_t)src;
}

__device__ __forceinline__ void compact_root(const DevForest &O, const DevForest &N, int32_t *old_of) {
    compact_copy_node(O, N, 0, 0, O.nodes[0], old_of);
    N.ntok[0] = O.ntok[0];
}

__global__ void compact_init_kernel(DevForest O, DevForest N, int32_t *old_of, CompactState *S) {
    compact_root(O, N, old_of);
    *S = CompactState{0, 1, 0, 0, 0, 0, 0, 0};
}

// Exclusive scan over the workgroup's threads of kCompactThreads values.
__device__ __forceinline__ long long compact_scan(long long v, long long *tmp, long long *total) {
    return plan_block_excl<long long>(v, 0, [](long long a, long long b) { return a + b; }, tmp, total);
}

// Frontier nodes of a tile.  A wave per node suits a level of parents; the
// leaves, most of a forest's nodes, have no children to look at, so a level of
// more than kCompactLeafLevel nodes (which cannot all have many) takes a thread
// per node to find the few that do.  The last level of 256,000 records, half of
// them live: count 34 -> 10 us, copy 27 -> 11 us.
constexpr int64_t kCompactLeafLevel = 16384;
__device__ __forceinline__ int compact_tile(int64_t n) { return n > kCompactLeafLevel ? kCompactThreads : kCompactWaves; }

// Children of old node x that some peer holds (wave-cooperative).
__device__ __forceinline__ int32_t compact_kept(const DevForest &O, int32_t beg, int32_t cnt, int lane) {
    int32_t k = 0;
    for (int32_t j0 = 0; j0 < cnt; j0 += 64 * kCompactUnroll) {
        bool keep[kCompactUnroll];
#pragma unroll
        for (int u = 0; u < kCompactUnroll; u++) {
            const int32_t j = j0 + 64 * u + lane;
            keep[u] = j < cnt && node_has_peers(O, beg + j, O.nodes[beg + j]);
        }
#pragma unroll
        for (int u = 0; u < kCompactUnroll; u++) k += (int32_t)__popcll(__ballot(keep[u]));
    }
    return k;
}

// Step 1 (grid-stride over tiles): start[i] = kept children of the tile's
// earlier nodes, blk[tile] = the tile's total.
__global__ __launch_bounds__(kCompactThreads) void compact_count_kernel(DevForest O, const int32_t *__restrict__ old_of,
                                                                       const CompactState *__restrict__ S,
                                                                       int32_t *__restrict__ start,
                                                                       int64_t *__restrict__ blk) {
    __shared__ int32_t s_cnt[kCompactWaves];
    __shared__ long long s_tmp[kCompactWaves];
    const int t = (int)threadIdx.x, lane = t & 63, wv = uniform((int32_t)(threadIdx.x >> 6));
    const int64_t lo = S->lo, n = S->hi - lo;
    const int tile = compact_tile(n);
    for (int64_t b = blockIdx.x; b * tile < n; b += gridDim.x) {
        if (tile == kCompactThreads) {
            const int64_t i = b * tile + t;
            int32_t beg = 0, cnt = 0;
            if (i < n) {
                const Node &x = O.nodes[old_of[lo + i]];
                beg = x.ct_beg;
                cnt = x.ct_cnt;
            }
            int32_t mine = 0;
            for (uint64_t m = __ballot(cnt > 0); m; m &= m - 1) {
                const int l = __ffsll((unsigned long long)m) - 1;
                const int32_t k = compact_kept(O, __builtin_amdgcn_readlane(beg, l), __builtin_amdgcn_readlane(cnt, l), lane);
                if (lane == l) mine = k;
            }
            long long total;
            const long long pre = compact_scan(mine, s_tmp, &total);
            if (i < n) start[lo + i] = (int32_t)pre;
            if (t == 0) blk[b] = total;
            continue;
        }
        const int64_t i = b * tile + wv;
        int32_t k = 0;
        if (i < n) {
            const Node x = O.nodes[old_of[lo + i]];
            k = compact_kept(O, x.ct_beg, x.ct_cnt, lane);
        }
        if (lane == 0) s_cnt[wv] = k;
        __syncthreads();
        int32_t pre = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kCompactWaves; w++) {
            pre += w < wv ? s_cnt[w] : 0;
            all += s_cnt[w];
        }
        if (i < n && lane == 0) start[lo + i] = pre;
        if (t == 0) blk[b] = all;
        __syncthreads();
    }
}

// Exclusive scan of blk[0, n) in place by one workgroup; returns the total.
__device__ __forceinline__ long long compact_scan_tiles(int64_t *blk, int64_t n, long long *tmp) {
    constexpr int kPer = 16;
    long long base = 0;
    for (int64_t i0 = 0; i0 < n; i0 += (int64_t)kPer * kCompactThreads) {
        long long v[kPer], sum = 0, total;
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int64_t i = i0 + (int64_t)threadIdx.x * kPer + k;
            v[k] = i < n ? blk[i] : 0;
            sum += v[k];
        }
        long long run = base + compact_scan(sum, tmp, &total);
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int64_t i = i0 + (int64_t)threadIdx.x * kPer + k;
            if (i < n) blk[i] = run;
            run += v[k];
        }
        base += total;
    }
    return base;
}

// Step 2 (one workgroup): the level's totals, and the range moves on.
__global__ __launch_bounds__(kCompactThreads) void compact_scan_kernel(CompactState *S, int64_t *blk, int64_t n_old) {
    __shared__ long long s_tmp[kCompactWaves];
    const long long lo = S->lo, hi = S->hi;
    const int tile = compact_tile(hi - lo);
    const long long total = compact_scan_tiles(blk, (hi - lo + tile - 1) / tile, s_tmp);
    if (threadIdx.x == 0) {
        // live nodes are distinct old records: more than n_old means a malformed forest
        const bool bad = hi + total > n_old;
        S->flo = bad ? hi : lo;
        S->fhi = hi;
        S->lo = hi;
        S->hi = bad ? hi : hi + total;
        if (bad) S->bad = 1;
    }
}

// Kept children of the frontier node with old block [cbeg, cbeg + ccnt) and new
// id i to new ids from beg on (wave-cooperative).
__device__ __forceinline__ void compact_copy_children(const DevForest &O, const DevForest &N, int32_t *old_of,
                                                      int32_t cbeg, int32_t ccnt, int64_t i, int64_t beg, int lane) {
    const uint64_t below = (1ull << lane) - 1ull;
    int64_t pos = beg;
    for (int32_t j0 = 0; j0 < ccnt; j0 += 64 * kCompactUnroll) {
        Node r[kCompactUnroll];
        bool keep[kCompactUnroll];
#pragma unroll
        for (int u = 0; u < kCompactUnroll; u++) {
            const int32_t j = j0 + 64 * u + lane;
            keep[u] = false;
            if (j < ccnt) {
                r[u] = O.nodes[cbeg + j];
                keep[u] = node_has_peers(O, cbeg + j, r[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < kCompactUnroll; u++) {
            const uint64_t b = __ballot(keep[u]);
            if (keep[u]) compact_copy_node(O, N, cbeg + j0 + 64 * u + lane, pos + __popcll(b & below), r[u], old_of);
            pos += __popcll(b);
        }
    }
    if (lane == 0) {
        N.nodes[i].ct_beg = (int32_t)beg;
        N.nodes[i].ct_cnt = (int32_t)(pos - beg);
    }
}

// Step 3 (grid-stride; a wave per frontier node, or per 64 of a level of leaves,
// whose records already say that they have no children).
__global__ __launch_bounds__(kCompactThreads) void compact_copy_kernel(DevForest O, DevForest N, int32_t *old_of,
                                                                      const CompactState *__restrict__ S,
                                                                      const int32_t *__restrict__ start,
                                                                      const int64_t *__restrict__ blk) {
    const int lane = (int)(threadIdx.x & 63);
    const int64_t lo = S->flo, n = S->fhi - lo, next = S->fhi;
    const int tile = compact_tile(n);
    const int per = tile / kCompactWaves;  // frontier nodes of a wave
    for (int64_t i0 = ((int64_t)blockIdx.x * kCompactWaves + uniform((int32_t)(threadIdx.x >> 6))) * per; i0 < n;
         i0 += (int64_t)gridDim.x * kCompactWaves * per) {
        const int64_t i = i0 + lane;
        int32_t cbeg = 0, ccnt = 0, pre = 0;
        if (lane < per && i < n) {
            const Node &x = O.nodes[old_of[lo + i]];
            cbeg = x.ct_beg;
            ccnt = x.ct_cnt;
            pre = start[lo + i];
        }
        for (uint64_t m = __ballot(ccnt > 0); m; m &= m - 1) {
            const int l = __ffsll((unsigned long long)m) - 1;
            compact_copy_children(O, N, old_of, __builtin_amdgcn_readlane(cbeg, l), __builtin_amdgcn_readlane(ccnt, l),
                                  lo + i0 + l, next + blk[(i0 + l) / tile] + __builtin_amdgcn_readlane(pre, l), lane);
        }
    }
}

// Step 4a (tiles of kCompactLabTile nodes, grid-stride): off[i] = label tokens
// of the tile's earlier nodes, blk[tile] = the tile's total.
__global__ __launch_bounds__(kCompactThreads) void compact_lab_kernel(DevForest N, const CompactState *__restrict__ S,
                                                                     int64_t *__restrict__ off,
                                                                     int64_t *__restrict__ blk) {
    __shared__ long long s_tmp[kCompactWaves];
    constexpr int kPer = kCompactLabTile / kCompactThreads;
    const int64_t n = S->hi;
    for (int64_t b = blockIdx.x; b * kCompactLabTile < n; b += gridDim.x) {
        long long v[kPer], sum = 0, total;
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int64_t i = b * kCompactLabTile + (int64_t)threadIdx.x * kPer + k;
            v[k] = i < n ? N.nodes[i].lab_len : 0;
            sum += v[k];
        }
        long long run = compact_scan(sum, s_tmp, &total);
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int64_t i = b * kCompactLabTile + (int64_t)threadIdx.x * kPer + k;
            if (i < n) off[i] = run;
            run += v[k];
        }
        if (threadIdx.x == 0) blk[b] = total;
    }
}

// Step 4b (one workgroup).
__global__ __launch_bounds__(kCompactThreads) void compact_lab_scan_kernel(CompactState *S, int64_t *blk) {
    __shared__ long long s_tmp[kCompactWaves];
    const long long total = compact_scan_tiles(blk, (S->hi + kCompactLabTile - 1) / kCompactLabTile, s_tmp);
    if (threadIdx.x == 0) S->n_pool = total;
}

// Step 4c (a workgroup per kCompactSeg tokens of the new pool): labels, their
// narrow copy, and for the nodes whose labels start there the new label offset
// and a wide block's separators.  The segment's nodes are found by a search over
// the label offsets and listed in LDS with a bit per token that starts a label;
// every token finds its own by counting the bits before it.  Short labels cost
// no more than long ones, every store is a full line, segments are alike however
// the lengths are spread, and the bit plane is written in whole words.  230 MB
// for 23 M tokens: 160 us with a wave per node (most have one or two 64-token
// chunks), 104 us with a search per token, four loads in flight and 32 KB of LDS
// (five workgroups a CU), 58 us with all sixteen loads in flight and 17 KB.
// blk nullptr: off holds whole offsets.
constexpr int kCompactSeg = 4096;
constexpr int kCompactSegThreads = 256;
__global__ __launch_bounds__(kCompactSegThreads) void compact_labels_kernel(DevForest O, DevForest N, NarrowDst D,
                                                                           const int32_t *__restrict__ old_of,
                                                                           CompactState *S,
                                                                           const int64_t *__restrict__ off,
                                                                           const int64_t *__restrict__ blk) {
    constexpr int T = kCompactSegThreads, kUnroll = kCompactSeg / T, kWords = kCompactSeg / 64;
    __shared__ uint32_t s_delta[kCompactSeg];        // per label in order: its source in the old pool less its start
    __shared__ unsigned long long s_start[kWords];   // a bit per token that starts a label
    __shared__ int s_before[kWords];                 // label starts in the words before
    static_assert(kWords == 64, "a lane per word");
    const int t = (int)threadIdx.x, lane = t & 63;
    const int64_t n = S->hi, base = (int64_t)blockIdx.x * kCompactSeg;
    const int64_t end = min<int64_t>(S->n_pool, base + kCompactSeg);
    if (base >= end) return;
    const auto at = [&](int64_t i) { return off[i] + (blk ? blk[i / kCompactLabTile] : 0); };
    // the last node whose label starts at or before the segment (only the root's
    // label is empty, so it is the one that holds its first token)
    int64_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const int64_t stride = (hi - lo + 63) / 64, j = lo + lane * stride;
        const int c = (int)__popcll(__ballot(j < hi && at(j) <= base));  // lane 0 always: at(lo) <= base
        hi = min(lo + c * stride, hi);
        lo += (c - 1) * stride;
    }
    const auto separators = [&](int32_t b, int32_t c) {
        if (c > kSepCount) N.nsep[b + lane] = N.ntok[b + PR_SEP_INDEX(lane, c)];
        if (c >= kSep2Min) sep2_write(N.nsep + b, N.ntok + b, c, lane);
    };
    if (base == 0 && t < 64) separators(N.nodes[0].ct_beg, N.nodes[0].ct_cnt);  // the root has no label to list it by
    if (t < kWords) s_start[t] = 0;
    __syncthreads();
    for (int64_t i0 = lo;; i0 += T) {
        const int64_t i = i0 + t;
        const int64_t o = i < n ? at(i) : end;
        int32_t beg = 0, cnt = 0;
        if (o < end) {
            // the source is the old record's; a label that starts before the
            // segment is listed from the segment's start on
            const int32_t skip = (int32_t)max<int64_t>(base - o, 0);
            const uint32_t k = (uint32_t)(o + skip - base);
            s_delta[i - lo] = O.nodes[old_of[i]].lab_off + (uint32_t)skip - k;
            atomicOr(&s_start[k >> 6], 1ull << (k & 63u));
            if (o >= base) {
                N.nodes[i].lab_off = (uint32_t)o;
                beg = N.nodes[i].ct_beg;
                cnt = N.nodes[i].ct_cnt;
            }
        }
        for (uint64_t wide = __ballot(cnt > kSepCount); wide; wide &= wide - 1) {
            const int l = __ffsll((unsigned long long)wide) - 1;
            separators(__builtin_amdgcn_readlane(beg, l), __builtin_amdgcn_readlane(cnt, l));
        }
        if (__syncthreads_or(o >= end)) break;  // offsets ascend: the rest start past the segment
    }
    if (t < kWords) {
        const uint32_t c = (uint32_t)__popcll(s_start[t]);
        s_before[t] = (int)(wave_incl_add_u32(c) - c);
    }
    __syncthreads();
    // a wave takes 64 tokens of the new pool at a time, all of its loads in flight
    const int len = (int)(end - base);
    uint32_t all = 0, v[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; u++) {
        const int k = u * T + t;
        v[u] = 0;
        if (k < len) {
            // the last label that starts at or before k
            const int a = s_before[k >> 6] + (int)__popcll(s_start[k >> 6] & (~0ull >> (63 - lane))) - 1;
            v[u] = (uint32_t)O.pool[s_delta[a] + (uint32_t)k];
        }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; u++) {
        const int k = u * T + t;
        if (k < len) {
            N.pool[base + k] = (int32_t)v[u];
            if (D.p16) D.p16[base + k] = (uint16_t)v[u];
            all |= v[u];
        }
        const uint64_t bits = __ballot((v[u] >> 16) & 1u);
        if (D.p16 && lane < 2 && k - lane + 32 * lane < len)
            D.hib[(base + k - lane + 32 * lane) >> 5] = (uint32_t)(bits >> (32 * lane));
    }
    // (a wider token may raise the 17-bit flag too; it drops the narrow copy)
    if (__ballot((all >> 16) & 1u) && lane == 0 && !fresh_u64(&S->hi_tokens)) atomicOr(&S->hi_tokens, 1ull);
    if (__ballot(all > 0x1FFFFu) && lane == 0 && !fresh_u64(&S->wide_tokens)) atomicOr(&S->wide_tokens, 1ull);
}

// Steps 1 to 4b for a small forest in one workgroup: each level a thousand
// frontier nodes at a time, whose children a scan spreads over the threads.
__global__ __launch_bounds__(kCompactThreads) void compact_small_kernel(DevForest O, DevForest N, int32_t *old_of,
                                                                       int64_t *off, int64_t n_old, CompactState *S) {
    __shared__ int32_t s_pre[kCompactThreads + 1], s_beg[kCompactThreads], s_kept[kCompactThreads];
    __shared__ int32_t s_wave[kCompactWaves];
    __shared__ long long s_tmp[kCompactWaves];
    const int t = (int)threadIdx.x, lane = t & 63, wv = t >> 6;
    const uint64_t below = (1ull << lane) - 1ull;
    if (t == 0) compact_root(O, N, old_of);
    __syncthreads();
    long long lo = 0, hi = 1;
    bool bad = false;
    while (lo < hi && !bad) {
        long long next = hi;
        for (long long f0 = lo; f0 < hi && !bad; f0 += kCompactThreads) {
            const int m = (int)min<long long>(kCompactThreads, hi - f0);
            Node x{};
            if (t < m) x = O.nodes[old_of[f0 + t]];
            long long total;
            const long long pre = compact_scan(t < m ? x.ct_cnt : 0, s_tmp, &total);
            if (total > n_old) {  // children are distinct old records
                bad = true;
                break;
            }
            s_pre[t] = (int32_t)pre;
            s_beg[t] = x.ct_beg;
            s_kept[t] = 0;
            if (t == 0) s_pre[kCompactThreads] = (int32_t)total;
            __syncthreads();
            for (int j0 = 0; j0 < (int)total; j0 += kCompactThreads) {
                const int j = j0 + t;
                int own = 0;
                bool keep = false;
                int64_t src = 0;
                Node r{};
                if (j < (int)total) {
                    int a = 0, b = m;  // the last frontier node with s_pre <= j
                    while (b - a > 1) {
                        const int mid = (a + b) >> 1;
                        if (s_pre[mid] <= j)
                            a = mid;
                        else
                            b = mid;
                    }
                    own = a;
                    src = (int64_t)s_beg[own] + (j - s_pre[own]);
                    r = O.nodes[src];
                    keep = node_has_peers(O, src, r);
                }
                const uint64_t bal = __ballot(keep);
                if (lane == 0) s_wave[wv] = (int32_t)__popcll(bal);
                __syncthreads();
                int32_t before = 0, all = 0;
#pragma unroll
                for (int w = 0; w < kCompactWaves; w++) {
                    before += w < wv ? s_wave[w] : 0;
                    all += s_wave[w];
                }
                if (next + all > n_old) bad = true;
                if (keep && !bad) {
                    compact_copy_node(O, N, src, next + before + __popcll(bal & below), r, old_of);
                    atomicAdd(&s_kept[own], 1);
                }
                next += all;
                __syncthreads();
                if (bad) break;
            }
            // each frontier node's kept children follow the earlier ones'
            long long kept_all;
            const long long kept_pre = compact_scan(s_kept[t], s_tmp, &kept_all);
            if (t < m) {
                N.nodes[f0 + t].ct_beg = (int32_t)(next - kept_all + kept_pre);
                N.nodes[f0 + t].ct_cnt = s_kept[t];
            }
            __syncthreads();
        }
        lo = hi;
        hi = next;
    }
    long long n_pool = 0;
    if (!bad) {
        for (long long i0 = 0; i0 < hi; i0 += kCompactThreads) {
            const long long i = i0 + t;
            long long total;
            const long long pre = compact_scan(i < hi ? N.nodes[i].lab_len : 0, s_tmp, &total);
            if (i < hi) off[i] = n_pool + pre;
            n_pool += total;
        }
    }
    if (t == 0) *S = bad ? CompactState{0, 0, 0, 0, 0, 0, 0, 1} : CompactState{hi, hi, hi, hi, n_pool, 0, 0, 0};
}

}  // namespace pr

#endif
