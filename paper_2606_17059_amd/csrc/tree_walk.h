// tree_walk.h -- one peer's tree walked in one launch: its size, its export's
// sequences, and the eviction of its least recently used tokens.
//
// A tree of a few thousand nodes is far too small to fill the chip, and walking
// it a level per launch with the frontier read back each time costs about 20 us
// a level (an LRU-cut tree of 100 nodes is 15 levels deep: 320 us for its size).
// tree_walk_kernel runs every level in one workgroup: the frontier (its nodes
// that have children) lives in LDS, a scan of the child counts spreads the
// level's children over the threads, four of a thread's children in flight, so
// a level of up to 4,096 children costs about one load's latency.  Measured,
// calls included: the export of a tree of 4,000 prompts (16,000 children looked
// at) 410 -> 127 us.  Sizes, and evictions among few records, need no walk
// (below).
//
// A walk whose frontier, level or leaf list is too large ends without having
// changed anything, and the level-by-level kernels (export_kernels.h,
// lru_kernels.h) do the work.
#ifndef PR_TREE_WALK_H
#define PR_TREE_WALK_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "forest_layout.h"
#include "lru_kernels.h"
#include "merge_kernels.h"
#include "wave_ops.h"

namespace pr {

constexpr int kWalkThreads = 1024;
constexpr int kWalkFront = 4096;       // frontier nodes in LDS
constexpr int kWalkUnroll = 4;         // children a thread has in flight
constexpr int kWalkChildren = 1 << 17; // children of one level: more are worth a chip-wide launch
constexpr int kWalkLeaves = 8192;      // leaves ordered in LDS (exports)
constexpr int kWalkBits = 1 << 18;     // records up to which a bitmap orders them

// Device and host copies of what a walk found.
struct WalkStatus {
    uint32_t done;     // 0: too large for one workgroup, nothing was written that counts
    uint32_t nodes;    // visited nodes (the root excluded)
    uint32_t leaves;   // sequences an export has
    uint32_t fits;     // the export's buffers hold it
    unsigned long long tokens, leaf_tokens;  // tokens of the tree, of the export
};

// What a walk writes besides the status (nullptr: not wanted).
struct WalkOut {
    int64_t *depth;    // per node id: tokens from the root through its label
    int32_t *parent;   // per node id
    int32_t *all;      // visited nodes
    int32_t *leaves;   // leaves, then (sorted) by node id
    int32_t *sorted;
    // an export's offsets: written if the export fits seqs_cap offsets and tokens_cap tokens
    int64_t *offsets;
    int64_t seqs_cap, tokens_cap;
};

// Sum over the workgroup, in every thread (kWalkThreads threads; tmp: 16 words).
__device__ __forceinline__ long long walk_block_sum(long long v, long long *tmp) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();  // tmp's readers of the last call are through
    if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = v;
    __syncthreads();
    long long s = 0;
#pragma unroll
    for (int k = 0; k < kWalkThreads / 64; k++) s += tmp[k];
    return s;
}

__device__ __forceinline__ void walk_report(const WalkStatus &r, WalkStatus *dev, WalkStatus *host) {
    *dev = r;
    const uint64_t *w = reinterpret_cast<const uint64_t *>(&r);
    for (int k = 0; k < (int)(sizeof(r) / 8); k++)
        __hip_atomic_store(reinterpret_cast<uint64_t *>(host) + k, w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(kWalkThreads) void tree_walk_kernel(DevForest F, int64_t n_nodes, int32_t p, WalkOut O,
                                                                WalkStatus *dev, WalkStatus *host) {
    // frontier nodes with children: id, first child, children before its own in
    // the level, depth; two of each (this level, the next)
    __shared__ int32_t s_id[2][kWalkFront], s_beg[2][kWalkFront], s_pre[2][kWalkFront], s_dep[2][kWalkFront];
    __shared__ uint8_t s_found[2][kWalkFront];
    __shared__ int s_next[2], s_total, s_leaves, s_nodes, s_over;
    __shared__ int s_tmp[kPlanWaves];
    __shared__ long long s_sum[kPlanWaves];
    const int t = (int)threadIdx.x, lane = t & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    const int32_t w = p >> 6;
    const auto plus = [](int a, int b) { return a + b; };
    long long tokens = 0, leaf_tokens = 0;
    if (t == 0) {
        const Node root = F.nodes[0];
        s_id[0][0] = 0;
        s_beg[0][0] = root.ct_beg;
        s_pre[0][0] = root.ct_cnt;
        s_dep[0][0] = 0;
        s_leaves = s_nodes = s_over = 0;
        s_next[0] = root.ct_cnt > 0 ? 1 : 0;
    }
    __syncthreads();
    int m = s_next[0];
    // a slot of a list for every lane that wants one: one LDS atomic per wave
    const auto slot = [&](int *ctr, bool want) -> int {
        const uint64_t b = __ballot(want);
        int base = 0;
        if (b && lane == 0) base = atomicAdd(ctr, (int)__popcll(b));
        base = __builtin_amdgcn_readfirstlane(base);
        return base + (int)__popcll(b & below);
    };
    const auto leaf = [&](bool want, int32_t id, int32_t dep) {
        const int k = slot(&s_leaves, want);
        if (want) {
            leaf_tokens += dep;
            if (O.leaves && k < n_nodes) O.leaves[k] = id;
        }
    };
    for (int cur = 0; m > 0; cur ^= 1) {
        // children before each frontier node's (its own count is in s_pre).
        // Two barriers a level: what a late thread of the last level still reads
        // (s_next, s_found) has another copy in this one.
        int total;
        if (t == 0) s_next[cur ^ 1] = 0;
        if (m <= 64) {
            if (t < 64) {
                const int c = t < m ? s_pre[cur][t] : 0;
                const int inc = (int)wave_incl_add_u32((uint32_t)c);
                if (t < m) {
                    s_pre[cur][t] = inc - c;
                    s_found[cur][t] = 0;
                }
                if (t == 63) s_total = inc;
            }
            __syncthreads();
            total = s_total;
        } else {
            constexpr int kPer = kWalkFront / kWalkThreads;
            int c[kPer], sum = 0;
#pragma unroll
            for (int k = 0; k < kPer; k++) {
                const int i = t * kPer + k;
                c[k] = i < m ? s_pre[cur][i] : 0;
                sum += c[k];
            }
            int run = plan_block_excl<int>(sum, 0, plus, s_tmp, &total);
#pragma unroll
            for (int k = 0; k < kPer; k++) {
                const int i = t * kPer + k;
                if (i < m) {
                    s_pre[cur][i] = run;
                    s_found[cur][i] = 0;
                }
                run += c[k];
            }
            __syncthreads();
        }
        if (total > kWalkChildren || total < 0) {
            if (t == 0) s_over = 1;
            break;
        }
        for (int j0 = 0; j0 < total; j0 += kWalkThreads * kWalkUnroll) {
            int own[kWalkUnroll];
            int32_t id[kWalkUnroll];
            Node r[kWalkUnroll];
            uint64_t word[kWalkUnroll];
#pragma unroll
            for (int u = 0; u < kWalkUnroll; u++) {
                const int j = j0 + u * kWalkThreads + t;
                own[u] = 0;
                id[u] = 0;
                r[u] = Node{};
                word[u] = 0;
                if (j >= total) continue;
                int lo = 0, hi = m;  // the last frontier node with s_pre <= j
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_pre[cur][mid] <= j)
                        lo = mid;
                    else
                        hi = mid;
                }
                own[u] = lo;
                id[u] = s_beg[cur][lo] + (j - s_pre[cur][lo]);
                if (id[u] >= 0 && id[u] < n_nodes) {
                    r[u] = F.nodes[id[u]];
                    word[u] = w == 0 ? r[u].mask0 : F.mext[(int64_t)id[u] * (F.W - 1) + (w - 1)];
                }
            }
#pragma unroll
            for (int u = 0; u < kWalkUnroll; u++) {
                if (j0 + u * kWalkThreads >= total) break;
                const bool held = (word[u] >> (p & 63)) & 1ull;
                const int32_t dep = s_dep[cur][own[u]] + r[u].lab_len;
                if (held) {
                    s_found[cur][own[u]] = 1;
                    tokens += r[u].lab_len;
                    if (O.depth) O.depth[id[u]] = dep;
                    if (O.parent) O.parent[id[u]] = s_id[cur][own[u]];
                }
                const int v = slot(&s_nodes, held);
                if (held && O.all && v < n_nodes) O.all[v] = id[u];
                const int f = slot(&s_next[cur ^ 1], held && r[u].ct_cnt > 0);
                if (held && r[u].ct_cnt > 0) {
                    if (f < kWalkFront) {
                        s_id[cur ^ 1][f] = id[u];
                        s_beg[cur ^ 1][f] = r[u].ct_beg;
                        s_pre[cur ^ 1][f] = r[u].ct_cnt;
                        s_dep[cur ^ 1][f] = dep;
                    } else {
                        s_over = 1;
                    }
                }
                leaf(held && r[u].ct_cnt <= 0, id[u], dep);
            }
        }
        __syncthreads();
        // a frontier node none of whose children holds p
        for (int i0 = 0; i0 < m; i0 += kWalkThreads) {
            const int i = i0 + t;
            const bool is = i < m && !s_found[cur][i] && s_id[cur][i] != 0;
            leaf(is, is ? s_id[cur][i] : 0, is ? s_dep[cur][i] : 0);
        }
        m = s_next[cur ^ 1];
        if (s_over != 0 || s_nodes > n_nodes) {
            __syncthreads();
            if (t == 0) s_over = 1;
            break;
        }
    }
    __syncthreads();
    const long long all_tokens = walk_block_sum(tokens, s_sum), all_leaf = walk_block_sum(leaf_tokens, s_sum);
    const int n = s_leaves;
    bool done = s_over == 0 && n <= n_nodes;
    bool fits = O.offsets && (int64_t)n + 1 <= O.seqs_cap && all_leaf <= O.tokens_cap;
    if (O.offsets && n > kWalkLeaves) done = false;
    if (done && fits) {
        // leaves by node id, then the offsets of their depths.  Ids differ, so
        // up to kWalkBits records a bit each in LDS (the frontier's, which is
        // free) and a scan of the words' counts put them in order; a bitonic sort
        // in LDS beyond.
        int32_t *key = &s_id[0][0];
        static_assert(2 * kWalkFront >= kWalkLeaves && kWalkBits <= 32 * 2 * kWalkFront, "they fit the frontier's LDS");
        if (n_nodes <= kWalkBits) {
            uint32_t *bits = reinterpret_cast<uint32_t *>(&s_beg[0][0]);
            const int words = (int)((n_nodes + 31) >> 5), each = (words + kWalkThreads - 1) / kWalkThreads;
            for (int i = t; i < words; i += kWalkThreads) bits[i] = 0;
            __syncthreads();
            for (int i = t; i < n; i += kWalkThreads) atomicOr(&bits[O.leaves[i] >> 5], 1u << (O.leaves[i] & 31));
            __syncthreads();
            const int w0 = min(t * each, words), w1 = min(w0 + each, words);
            int c = 0, total;
            for (int i = w0; i < w1; i++) c += __popc(bits[i]);
            int r = plan_block_excl<int>(c, 0, plus, s_tmp, &total);
            for (int i = w0; i < w1; i++)
                for (uint32_t v = bits[i]; v; v &= v - 1) key[r++] = 32 * i + __ffs((int)v) - 1;
            __syncthreads();
        } else {
            int np = 1;
            while (np < n) np <<= 1;
            for (int i = t; i < np; i += kWalkThreads) key[i] = i < n ? O.leaves[i] : INT32_MAX;
            __syncthreads();
            for (int k = 2; k <= np; k <<= 1)
                for (int j = k >> 1; j > 0; j >>= 1) {
                    for (int q = t; q < np / 2; q += kWalkThreads) {
                        const int a = ((q & ~(j - 1)) << 1) | (q & (j - 1)), b = a + j;
                        const int32_t x = key[a], y = key[b];
                        if ((x > y) == ((a & k) == 0)) {
                            key[a] = y;
                            key[b] = x;
                        }
                    }
                    __syncthreads();
                }
        }
        constexpr int kPer = kWalkLeaves / kWalkThreads;
        long long d[kPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int i = t * kPer + k;
            d[k] = i < n ? O.depth[key[i]] : 0;
            sum += d[k];
        }
        long long total;
        long long run = plan_block_excl<long long>(sum, 0, [](long long a, long long b) { return a + b; }, s_sum, &total);
        if (t == 0) O.offsets[0] = 0;
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int i = t * kPer + k;
            run += d[k];
            if (i < n) {
                O.offsets[i + 1] = run;
                O.sorted[i] = key[i];
            }
        }
    }
    if (t == 0)
        walk_report(WalkStatus{done ? 1u : 0u, (uint32_t)s_nodes, (uint32_t)n, fits ? 1u : 0u,
                               (unsigned long long)all_tokens, (unsigned long long)all_leaf},
                    dev, host);
}

// ---- the size of a tree ------------------------------------------------------
// Records hold everything a tree's size needs: a record in use has not moved
// (moved is 0) and peers hold all of a path or none of it, so the size is the
// sum of the labels of the records that have the peer's bit and have not moved,
// in one pass over the records without a level waiting for another (records of
// refused allocations have no peers).  What it moves is 40 bytes a record of the
// forest, whosever it is, so past kSizeRecords records the walk is tried first: of
// 20 M records, 196 us for any tree, where a walk finds one of 450 nodes in 53 us,
// one of 4,200 in 175, and turns back from a larger one after 22 (at 8 M: 110, 41,
// 84 and 20).  A tree of 15
// levels among 1,500 records 33 -> 2.9 us, one of 4,000 prompts in a forest of
// 65,000 records 33 -> 6.3 us (the walk's kernel -> this one).
constexpr int kSizeThreads = 256;
constexpr int kSizePer = 4;  // records a thread has in flight
constexpr unsigned kSizeBlocks = 1024;
constexpr int64_t kSizeRecords = 1 << 23;

// Zero between calls: the last workgroup to finish clears it.
struct SizeState {
    unsigned long long tokens;
    uint32_t blocks, pad;
};

__global__ __launch_bounds__(kSizeThreads) void tree_size_kernel(DevForest F, int64_t n_nodes, int32_t p, SizeState *acc,
                                                                 unsigned long long *host) {
    __shared__ unsigned long long s_sum[kSizeThreads / 64];
    const int32_t w = p >> 6;
    const int64_t step = (int64_t)gridDim.x * kSizeThreads;
    unsigned long long sum = 0;
    for (int64_t i0 = (int64_t)blockIdx.x * kSizeThreads + threadIdx.x; i0 < n_nodes; i0 += step * kSizePer) {
        uint64_t word[kSizePer];
        int32_t len[kSizePer];
        long long mv[kSizePer];
#pragma unroll
        for (int k = 0; k < kSizePer; k++) {
            const int64_t i = i0 + k * step;
            word[k] = 0;
            len[k] = 0;
            mv[k] = 0;
            if (i < n_nodes) {
                word[k] = w == 0 ? F.nodes[i].mask0 : F.mext[i * (F.W - 1) + (w - 1)];
                len[k] = F.nodes[i].lab_len;
                mv[k] = F.moved[i];
            }
        }
#pragma unroll
        for (int k = 0; k < kSizePer; k++)
            if (((word[k] >> (p & 63)) & 1ull) && mv[k] == 0) sum += (unsigned long long)len[k];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x != 0) return;
    sum = 0;
    for (int k = 0; k < kSizeThreads / 64; k++) sum += s_sum[k];
    if (gridDim.x > 1) {
        atomicAdd(&acc->tokens, sum);
        __threadfence();
        if (atomicAdd(&acc->blocks, 1u) + 1 < gridDim.x) return;
        __threadfence();
        sum = atomicAdd(&acc->tokens, 0ull);
        acc->tokens = 0;
        acc->blocks = 0;
    }
    __hip_atomic_store(reinterpret_cast<uint64_t *>(host), (uint64_t)sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---- eviction ----------------------------------------------------------------
// The eviction of lru_kernels.h in one workgroup, a thread with several nodes
// in registers.  SCAN: among at most kEvictScan records the nodes are found as
// for the tree's size; each writes its place to its children's parent words in
// LDS, and depths are sums along the parents by pointer jumping (four rounds
// for 15 levels, where a walk waits for memory level by level), and the class's
// tokens above a depth by two scans over depths in place of a bisection: walk
// and eviction of such a tree took 33 + 20 us, this launch takes 20.
// Otherwise the kernel comes after a walk (whose status on the device says
// whether it is whole) and takes at most kEvictNodes nodes.  The time class where the
// budget runs out is found by a radix selection over the times' bytes that
// differ, weighted by label tokens; the cut depth by bisection over sums; the
// order of the paths at the cut depth by comparing pairs.  Nothing is changed
// before the cuts are known to fit the node capacity.
constexpr int kEvictNodes = 4 * kWalkThreads;
constexpr int kEvictScan = 8 * kWalkThreads;
constexpr int kEvictLevel = 512;  // nodes at the cut depth

struct EvictStatus {
    uint32_t done;  // 0: nothing was changed
    uint32_t pad;
    unsigned long long evicted, n_nodes;
};

// walk, all, depth, parent: of the walk (SCAN: not used).
template <bool SCAN>
__global__ __launch_bounds__(kWalkThreads) void evict_kernel(DevForest F, const WalkStatus *walk,
                                                            const int32_t *__restrict__ all,
                                                            const int64_t *__restrict__ depth,
                                                            const int32_t *__restrict__ parent, int64_t max_tokens,
                                                            MergeCounters *ctr, EvictStatus *out) {
    constexpr int kEvictPer = SCAN ? kEvictScan / kWalkThreads : kEvictNodes / kWalkThreads;
    __shared__ unsigned long long s_hist[256];
    __shared__ int32_t s_level[kEvictLevel], s_rank[kEvictLevel];
    __shared__ long long s_sum[kPlanWaves];
    __shared__ unsigned long long s_prefix, s_rem, s_class;
    __shared__ int s_n;
    const int t = (int)threadIdx.x;
    const unsigned long long n0 = ctr->n_nodes;
    const auto report = [&](bool done, unsigned long long evicted, unsigned long long n_nodes) {
        if (t != 0) return;
        const EvictStatus r{done ? 1u : 0u, 0u, evicted, n_nodes};
        const uint64_t *w = reinterpret_cast<const uint64_t *>(&r);
        for (int k = 0; k < (int)(sizeof(r) / 8); k++)
            __hip_atomic_store(reinterpret_cast<uint64_t *>(out) + k, w[k], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
    };
    int32_t id[kEvictPer], e[kEvictPer], len[kEvictPer];
    unsigned long long time[kEvictPer];
    long long total = 0;
    // SCAN: per record its parent, its depth, and the ancestor its depth counts
    // from so far (later the class's tokens per depth)
    constexpr int kLds = SCAN ? kEvictScan : 1;
    __shared__ int32_t s_par[kLds], s_dep[kLds], s_anc[kLds];
    if constexpr (SCAN) {
        if (n0 > (unsigned long long)kEvictScan) {
            report(false, 0, n0);
            return;
        }
        const int n = (int)n0, lane = t & 63, w = F.local >> 6;
        for (int q = t; q < n; q += kWalkThreads) s_anc[q] = -1;
        int32_t beg[kEvictPer], cnt[kEvictPer];
#pragma unroll
        for (int k = 0; k < kEvictPer; k++) {
            const int i = t + k * kWalkThreads;
            id[k] = -1;
            e[k] = len[k] = beg[k] = cnt[k] = 0;
            time[k] = 0;
            if (i < n) {
                const Node r = F.nodes[i];
                const uint64_t word = w == 0 ? r.mask0 : F.mext[(int64_t)i * (F.W - 1) + (w - 1)];
                const bool held = i > 0 && ((word >> (F.local & 63)) & 1ull) && F.moved[i] == 0;
                time[k] = F.ltime[i];
                if (held) {
                    id[k] = i;
                    len[k] = r.lab_len;
                }
                if (held || i == 0) {
                    beg[k] = r.ct_beg;
                    cnt[k] = r.ct_cnt;
                }
            }
        }
        __syncthreads();
        // every record is in one block of children; blocks past a few children
        // are written by the whole wave
#pragma unroll
        for (int k = 0; k < kEvictPer; k++) {
            const int i = t + k * kWalkThreads;
            if (cnt[k] <= 8)
                for (int j = 0; j < cnt[k]; j++)
                    if ((uint32_t)(beg[k] + j) < (uint32_t)n) s_anc[beg[k] + j] = i;
            for (uint64_t m = __ballot(cnt[k] > 8); m; m &= m - 1) {
                const int l = __ffsll((unsigned long long)m) - 1;
                const int32_t b = __builtin_amdgcn_readlane(beg[k], l), c = __builtin_amdgcn_readlane(cnt[k], l);
                for (int j = lane; j < c; j += 64)
                    if ((uint32_t)(b + j) < (uint32_t)n) s_anc[b + j] = i - lane + l;
            }
        }
        __syncthreads();
        int lost = 0;
        if (t == 0) s_anc[0] = s_dep[0] = 0;
#pragma unroll
        for (int k = 0; k < kEvictPer; k++) {
            if (id[k] < 0) continue;
            s_dep[id[k]] = len[k];
            lost |= s_anc[id[k]] < 0;
            s_par[id[k]] = s_anc[id[k]];
        }
        if (__syncthreads_or(lost)) {
            report(false, 0, n0);
            return;
        }
        for (int round = 0; round < 16; round++) {  // 13 for a chain of 8,192
            int32_t add[kEvictPer], up[kEvictPer];
            int more = 0;
#pragma unroll
            for (int k = 0; k < kEvictPer; k++) {
                const int32_t a = id[k] >= 0 ? s_anc[id[k]] : 0;
                add[k] = a > 0 ? s_dep[a] : 0;
                up[k] = a > 0 ? s_anc[a] : 0;
                more |= up[k] > 0;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kEvictPer; k++)
                if (id[k] >= 0) {
                    s_dep[id[k]] += add[k];
                    s_anc[id[k]] = up[k];
                }
            if (!__syncthreads_or(more)) break;
        }
        long long mine = 0;
#pragma unroll
        for (int k = 0; k < kEvictPer; k++)
            if (id[k] >= 0) {
                e[k] = s_dep[id[k]];
                mine += len[k];
            }
        total = walk_block_sum(mine, s_sum);
    } else {
        const int V = (int)walk->nodes;
        if (!walk->done || V > kEvictNodes) {
            report(false, 0, n0);
            return;
        }
        total = (long long)walk->tokens;
#pragma unroll
        for (int k = 0; k < kEvictPer; k++) {
            const int i = t + k * kWalkThreads;
            id[k] = -1;
            e[k] = len[k] = 0;
            time[k] = 0;
            if (i < V) {
                id[k] = all[i];
                e[k] = (int32_t)depth[id[k]];
                len[k] = F.nodes[id[k]].lab_len;
                time[k] = F.ltime[id[k]];
            }
        }
    }
    unsigned long long lo = ~0ull, hi = 0;
#pragma unroll
    for (int k = 0; k < kEvictPer; k++)
        if (id[k] >= 0) {
            lo = min(lo, time[k]);
            hi = max(hi, time[k]);
        }
    if (max_tokens >= total) {  // everything goes
#pragma unroll
        for (int k = 0; k < kEvictPer; k++)
            if (id[k] >= 0) lru_clear(F, id[k], F.local);
        report(true, (unsigned long long)total, n0);
        return;
    }
    // the bytes in which the times differ: the smallest time K whose tokens and
    // the earlier ones' reach the budget
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = min(lo, (unsigned long long)__shfl_xor(lo, off));
        hi = max(hi, (unsigned long long)__shfl_xor(hi, off));
    }
    if ((t & 63) == 0) {
        s_hist[t >> 6] = lo;
        s_hist[64 + (t >> 6)] = hi;
    }
    __syncthreads();
    for (int k = 0; k < kWalkThreads / 64; k++) {
        lo = min(lo, s_hist[k]);
        hi = max(hi, s_hist[64 + k]);
    }
    int top = 0;  // bits above which every time is the same
    while (top < 64 && (lo >> top) != (hi >> top)) top += 8;
    unsigned long long prefix = top < 64 ? lo >> top << top : 0ull;
    unsigned long long rem = (unsigned long long)max_tokens, cls = (unsigned long long)total;
    for (int sh = top - 8; sh >= 0; sh -= 8) {
        __syncthreads();
        if (t < 256) s_hist[t] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kEvictPer; k++)
            if (id[k] >= 0 && (sh + 8 >= 64 || (time[k] >> (sh + 8)) == (prefix >> (sh + 8))))
                atomicAdd(&s_hist[(time[k] >> sh) & 255u], (unsigned long long)len[k]);
        __syncthreads();
        if (t < 64) {
            unsigned long long v[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                v[k] = s_hist[4 * t + k];
                sum += v[k];
            }
            unsigned long long run = plan_wave_incl(sum, [](unsigned long long a, unsigned long long b) { return a + b; }) - sum;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                if (run < rem && rem <= run + v[k]) {
                    s_prefix = prefix | ((unsigned long long)(4 * t + k) << sh);
                    s_rem = rem - run;
                    s_class = v[k];
                }
                run += v[k];
            }
        }
        __syncthreads();
        prefix = s_prefix;
        rem = s_rem;
        cls = s_class;
    }
    // rem of the class's cls tokens go (rem >= 1)
    const bool whole = rem == cls;
    long long D = 0, r_at = 0;
    int rank_slot[kEvictPer];
#pragma unroll
    for (int k = 0; k < kEvictPer; k++) rank_slot[k] = -1;
    if (!whole) {
        // class tokens at depth x and deeper
        const auto deeper = [&](long long x) {
            long long v = 0;
#pragma unroll
            for (int k = 0; k < kEvictPer; k++)
                if (id[k] >= 0 && time[k] == prefix && e[k] >= x) v += min((long long)len[k], e[k] - x + 1);
            return walk_block_sum(v, s_sum);
        };
        int maxd = 0;
#pragma unroll
        for (int k = 0; k < kEvictPer; k++) maxd = max(maxd, e[k]);
        for (int off = 32; off >= 1; off >>= 1) maxd = max(maxd, __shfl_xor(maxd, off));
        if (t == 0) s_n = 0;
        __syncthreads();
        if ((t & 63) == 0) atomicMax(&s_n, maxd);
        __syncthreads();
        const int deepest = s_n;
        // the deepest D whose tokens and the deeper ones' reach rem
        if (SCAN && deepest + 2 <= kEvictScan) {
            // class tokens per depth: a node's first and the one past its last
            // token step the count, summed over depths, then the tokens above
            constexpr int kPer = kLds / kWalkThreads > 0 ? kLds / kWalkThreads : 1;
            for (int q = t; q < kLds; q += kWalkThreads) s_anc[q] = 0;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kEvictPer; k++)
                if (id[k] >= 0 && time[k] == prefix) {
                    atomicAdd(&s_anc[e[k] - len[k] + 1], 1);
                    atomicAdd(&s_anc[e[k] + 1], -1);
                }
            __syncthreads();
            const auto plus = [](long long x, long long y) { return x + y; };
            long long c[kPer], step = 0, all_c, above = 0;
#pragma unroll
            for (int k = 0; k < kPer; k++) step += c[k] = s_anc[t * kPer + k];
            long long at = plan_block_excl<long long>(step, 0, plus, s_sum, &all_c);
#pragma unroll
            for (int k = 0; k < kPer; k++) above += c[k] = at += c[k];
            long long left = (long long)cls - plan_block_excl<long long>(above, 0, plus, s_sum, &all_c);
#pragma unroll
            for (int k = 0; k < kPer; k++) {
                if (left >= (long long)rem && left - c[k] < (long long)rem) {  // one depth of all
                    s_prefix = (unsigned long long)(t * kPer + k);
                    s_rem = rem - (unsigned long long)(left - c[k]);
                }
                left -= c[k];
            }
            __syncthreads();
            D = (long long)s_prefix;
            r_at = (long long)s_rem;
        } else {
            long long a = 1, b = deepest;
            while (a < b) {
                const long long mid = (a + b + 1) / 2;
                if (deeper(mid) >= (long long)rem)
                    a = mid;
                else
                    b = mid - 1;
            }
            D = a;
            r_at = (long long)rem - deeper(D + 1);
        }
        if (t == 0) s_n = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kEvictPer; k++)
            if (id[k] >= 0 && time[k] == prefix && e[k] - len[k] + 1 <= D && D <= e[k]) {
                rank_slot[k] = atomicAdd(&s_n, 1);
                if (rank_slot[k] < kEvictLevel) {
                    s_level[rank_slot[k]] = id[k];
                    s_rank[rank_slot[k]] = 0;
                }
            }
        __syncthreads();
        const int c = s_n;
        if (c > kEvictLevel) {
            report(false, 0, n0);
            return;
        }
        if (r_at < c)
            for (int q = t; q < c * c; q += kWalkThreads) {
                const int i = q / c, j = q % c;
                if (i < j) {
                    bool first;
                    if constexpr (SCAN)
                        first = lru_path_before(F.ntok, s_par, s_dep, s_level[j], s_level[i]);
                    else
                        first = lru_path_before(F.ntok, parent, depth, s_level[j], s_level[i]);
                    atomicAdd(&s_rank[first ? i : j], 1);
                }
            }
        __syncthreads();
    }
    // tokens each node keeps (up to depth `keep`), and the cuts' records
    if (t == 0) s_n = 0;
    __syncthreads();
    int32_t cut[kEvictPer];
    bool gone[kEvictPer];
#pragma unroll
    for (int k = 0; k < kEvictPer; k++) {
        cut[k] = -1;
        gone[k] = false;
        if (id[k] < 0 || time[k] > prefix) continue;
        const long long s = (long long)e[k] - len[k] + 1;
        long long keep = s - 1;
        if (time[k] == prefix && !whole) {
            if (rank_slot[k] >= 0)
                keep = s_rank[rank_slot[k]] < r_at ? D - 1 : D;
            else
                keep = s > D ? s - 1 : e[k];
        }
        gone[k] = keep < s;
        if (keep >= s && keep < e[k]) {
            cut[k] = atomicAdd(&s_n, 1);
            len[k] = (int32_t)(keep - s + 1);  // tokens the upper part keeps
        }
    }
    __syncthreads();
    const int n_cut = s_n;
    if ((long long)n0 + n_cut > F.cap_nodes) {
        report(false, 0, n0);
        return;
    }
#pragma unroll
    for (int k = 0; k < kEvictPer; k++) {
        if (gone[k]) lru_clear(F, id[k], F.local);
        if (cut[k] >= 0) lru_cut(F, id[k], len[k], (int32_t)(n0 + (unsigned long long)cut[k]), F.local);
    }
    if (t == 0) ctr->n_nodes = n0 + (unsigned long long)n_cut;
    report(true, (unsigned long long)max_tokens, n0 + (unsigned long long)n_cut);
}

}  // namespace pr

#endif
