// small_merge.h -- a merge (or touch) of at most 64 sequences in one launch,
// and the last unfinished ones of a larger batch.
//
// A node that serves requests one at a time merges and touches batches of one
// or a few sequences.  The rounds of merge_kernels.h take two dozen dependent
// launches for them, each a few microseconds long; here one workgroup of
// sixteen waves runs the rounds itself, with barriers in place of launches:
//   walk     a wave per insert (m_walk);
//   plan     one wave, one lane per insert: the winners of each slot and edge
//            are found by comparing every pair of lanes, and prefix sums over
//            the lanes give each winner its records and label span;
//   build    waves share the 64-child chunks of the rebuilt parents' old blocks
//            and the winners' leaves;
//   finish   separators of wide blocks, parents pointed at their new blocks;
//   cut      a wave per winning cut.
// The rules are those of merge_kernels.h (lowest batch index wins a slot or an
// edge, adds before cuts in a round, losers walk again).  Labels are written to
// the narrow copy as they are written to the pool.  What does not fit (the
// capacity, or rebuilt parents with more than kSmallChunks chunks, which more
// than one workgroup should move) ends the launch between two rounds with the
// forest consistent, and the caller goes on with the other kernels; batches of
// long sequences (kSmallWork) are left to them from the start.
//
// One insert into the 57-topic trees of the request-at-a-time simulation, call
// included: 106 us with the rounds' launches, 33 us here; touching one request 157 us
// (a route, a gather and those launches), 22 us.
//
// Records read here may have been changed by atomics of this launch (peer bits,
// times), which do not update lines the CU's first-level cache holds: such
// reads go past it (fresh_*).
#ifndef PR_SMALL_MERGE_H
#define PR_SMALL_MERGE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "forest_layout.h"
#include "merge_kernels.h"
#include "wave_ops.h"

namespace pr {

constexpr int kSmallWaves = 16;
constexpr int kSmallMax = 64;      // inserts: one lane each
constexpr int kSmallChunks = 256;  // chunks of 64 old children one round moves
constexpr int kSmallGather = 16;   // inserts a thread looks at for the unfinished ones of a larger batch
constexpr int64_t kSmallBatch = 64 * kSmallWaves * kSmallGather;
static_assert(kPlanMaxBatch <= kSmallBatch, "the rounds' batches are looked at whole for what they left");
// Inserts past a wave each are worked off one after the other, on one CU; launches
// give each a wave and spread their labels over the chip, for 17 us more, since
// this one then ends at once.  Sequences times their tokens up to which one
// workgroup is the faster (us here / in launches, a merge of new sequences, call
// included):
//   24 of  5,000 tokens  89 /  98    10,000 tokens  148 / 137
//   32 of  5,000         98 / 123    10,000         201 / 171
//   48 of  1,200         73 /  87     5,000         133 / 111
//   64 of  1,200         89 /  87     2,500         121 / 101    20,000 tokens 587 / 271
// and up to a wave each at any length (16 of 20,000: 142 / 154).
constexpr int64_t kSmallWork = 5500000;

// Written to pinned host memory when the launch ends.
struct SmallStatus {
    uint32_t done;  // 1: every insert is in; 0: the other kernels go on
    uint32_t hi, wide;  // an appended token is in [65536, 131071], past 131071 (or negative)
    uint32_t stamps;    // stamps taken
    uint32_t left;      // unfinished inserts found at the start
    uint32_t rounds;    // the last round in which one walked
    uint32_t overflow, fallback;  // the counters' of the rounds before
    unsigned long long n_nodes, n_pool;
};

// A barrier that also waits for this wave's own stores and atomics.
__device__ __forceinline__ void small_sync() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// Sum over lower lanes (exclusive); *total gets the wave's sum.
__device__ __forceinline__ int64_t lane_excl(int64_t v, int lane, int64_t *total) {
    int64_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t u = __shfl_up(inc, off);
        if (lane >= off) inc += u;
    }
    *total = __shfl(inc, 63);
    return inc - v;
}

// One workgroup.  stamp0: the first stamp not used yet; a round that moves
// records takes one.  st: nullptr for a batch of at most kSmallMax sequences,
// else the states that rounds of launches left of one of at most kSmallBatch:
// at most kSmallMax unfinished ones are done here, more are left to further
// rounds.  Either way the round counters are cleared for the next call.
__global__ __launch_bounds__(64 *kSmallWaves) void small_merge_kernel(DevForest F, Batch B, NarrowDst N,
                                                                     MergeCounters *ctr,
                                                                     unsigned long long *skipped_acc,
                                                                     const InsState *st, long long stamp0,
                                                                     SmallStatus *out) {
    __shared__ InsState s_st[kSmallMax];
    __shared__ int64_t s_off[kSmallMax], s_len[kSmallMax], s_pb[kSmallMax];
    __shared__ int32_t s_peer[kSmallMax];
    // winners of the round (per insert): 0 none, 1 add, 2 cut; an add winner's
    // ordinal in its group and the group's head; records of a cut
    __shared__ int32_t s_win[kSmallMax], s_ord[kSmallMax], s_head[kSmallMax], s_nb[kSmallMax];
    // per group head: the parent's old block, its chunks' prefix, new leaves
    __shared__ int32_t s_beg[kSmallMax], s_cnt[kSmallMax], s_c0[kSmallMax], s_nw[kSmallMax];
    __shared__ int32_t s_idx[kSmallMax];
    __shared__ int s_tmp[kSmallWaves];
    __shared__ int s_state, s_chunks;  // s_state: 0 go on, 1 done, 2 leave the rest
    __shared__ uint32_t s_seen, s_skip;
    const int lane = (int)(threadIdx.x & 63);
    const int wv = uniform((int32_t)(threadIdx.x / 64));
    int n = (int)B.n, left = n;
    unsigned long long n_nodes = ctr->n_nodes, n_pool = ctr->n_pool;  // wave 0 keeps them
    uint32_t seen = 0;
    long long stamp = stamp0;

    const bool broken = st && (ctr->overflow || ctr->plan_fallback);
    if (st) {
        // the unfinished inserts, in batch order
        int c = 0, at[kSmallGather];
#pragma unroll
        for (int k = 0; k < kSmallGather; k++) {
            const int i = (int)threadIdx.x * kSmallGather + k;
            const int32_t kind = i < n ? st[i].kind : kInsSkip;
            at[k] = kind == kInsSkip || kind == kInsDone ? -1 : c++;
        }
        const int before = plan_block_excl<int>(c, 0, [](int a, int b) { return a + b; }, s_tmp, &left);
#pragma unroll
        for (int k = 0; k < kSmallGather; k++)
            if (at[k] >= 0 && before + at[k] < kSmallMax) s_idx[before + at[k]] = (int)threadIdx.x * kSmallGather + k;
        n = min(left, kSmallMax);
    } else if (wv == 0) {
        s_idx[lane] = lane;
    }
    __syncthreads();
    if (wv == 0) {
        bool ok = false, bad = false;
        if (lane < n) {
            const int32_t i = s_idx[lane];
            const int64_t b = B.offsets[i], e = B.offsets[i + 1];
            const int32_t p = batch_peer(B, i);
            ok = p >= 0 && p < B.P && b >= 0 && e >= b && e <= B.num_tokens && e - b <= (int64_t)INT32_MAX;
            bad = !ok && !B.touch;
            s_off[lane] = ok ? b : 0;
            s_len[lane] = ok ? e - b : 0;
            s_peer[lane] = ok ? p : 0;
            s_st[lane].kind = ok ? kInsActive : kInsSkip;
        }
        const uint32_t skip = (uint32_t)__popcll(__ballot(bad));
        bool large = false;
        if (n > kSmallWaves && !B.touch) {
            int64_t tokens;
            (void)lane_excl(ok ? s_len[lane] : 0, lane, &tokens);
            large = tokens > kSmallWork / n;
        }
        if (lane == 0) {
            s_state = left > kSmallMax || broken || large ? 2 : 0;
            s_seen = 0;
            s_skip = st ? (uint32_t)ctr->skipped : skip;
        }
    }
    small_sync();

    // every round finishes at least the lowest unfinished insert
    for (int round = 0; round < 2 * kSmallMax && s_state == 0; round++) {
        // walk
        for (int i = wv; i < n; i += kSmallWaves) {
            const int32_t kind = s_st[i].kind;
            if (kind == kInsSkip || kind == kInsDone) continue;
            const int32_t p = s_peer[i];
            const InsState r = m_walk(F, B.tokens + s_off[i], s_len[i], p, B.touch, stamps_path(F, p), lane);
            if (lane == 0) s_st[i] = r;
        }
        small_sync();
        // plan
        if (wv == 0) {
            InsState r{};
            r.kind = kInsSkip;
            if (lane < n) r = s_st[lane];
            const bool add = r.kind == kInsAdd, cut = r.kind == kInsSplit;
            const uint64_t addm = __ballot(add), cutm = __ballot(cut);
            bool win = add || cut;
            for (uint64_t m = addm; m; m &= m - 1) {
                const int j = __ffsll((unsigned long long)m) - 1;
                const int32_t xj = __builtin_amdgcn_readlane(r.x, j), tj = __builtin_amdgcn_readlane(r.t, j);
                if (add && j < lane && xj == r.x && tj == r.t) win = false;  // the slot's lowest index wins
            }
            for (uint64_t m = cutm; m; m &= m - 1) {
                const int j = __ffsll((unsigned long long)m) - 1;
                const int32_t cj = __builtin_amdgcn_readlane(r.c, j);
                if (cut && j < lane && cj == r.c) win = false;  // the edge's
            }
            // groups of add winners by parent: head (lowest index), ordinal by token, size
            int32_t head = lane, ord = 0, size = 0;
            for (uint64_t m = __ballot(win && add); m; m &= m - 1) {
                const int j = __ffsll((unsigned long long)m) - 1;
                const int32_t xj = __builtin_amdgcn_readlane(r.x, j), tj = __builtin_amdgcn_readlane(r.t, j);
                if (xj == r.x) {
                    head = min(head, j);
                    ord += tj < r.t;
                    size++;
                }
            }
            const bool is_head = win && add && head == lane;
            int32_t beg = 0, cnt = 0;
            if (is_head) {
                const Node x = fresh_node(&F.nodes[r.x]);
                beg = x.ct_beg;
                cnt = x.ct_cnt;
            }
            const int64_t rest = win ? (B.touch ? 0 : s_len[lane] - r.d - (cut ? r.l : 0)) : 0;
            const int64_t recs = is_head ? cnt + size : (win && cut ? (rest > 0 ? 2 : 1) : 0);
            int64_t t_recs, t_pool, t_chunks;
            const int64_t nb = lane_excl(recs, lane, &t_recs), pb = lane_excl(rest, lane, &t_pool);
            const int64_t c0 = lane_excl(is_head ? (cnt + 63) / 64 : 0, lane, &t_chunks);
            // a first-token match guarantees a cut past the label's first token
            const bool odd = __ballot(win && cut && r.l <= 0) != 0;
            int state = 0;
            if (!addm && !cutm)
                state = 1;
            else if (odd || t_chunks > kSmallChunks || (int64_t)n_nodes + t_recs > F.cap_nodes ||
                     (int64_t)n_pool + t_pool > F.cap_pool)
                state = 2;
            if (lane < n) {
                s_win[lane] = win ? (add ? 1 : 2) : 0;
                s_ord[lane] = ord;
                s_head[lane] = head;
                s_nb[lane] = (int32_t)((int64_t)n_nodes + nb);
                s_pb[lane] = (int64_t)n_pool + pb;
                s_beg[lane] = beg;
                s_cnt[lane] = cnt;
                s_c0[lane] = (int32_t)c0;
                s_nw[lane] = is_head ? size : 0;
            }
            if (state == 0) {
                n_nodes += (unsigned long long)t_recs;
                n_pool += (unsigned long long)t_pool;
            }
            if (lane == 0) {
                s_state = state;
                s_chunks = (int)t_chunks;
            }
        }
        small_sync();
        if (s_state != 0) break;
        // build: old children move up by the new leaves below them, stamped
        // with their new position
        const uint64_t heads = __ballot(lane < n && s_nw[lane < n ? lane : 0] > 0);
        for (int q = wv; q < s_chunks; q += kSmallWaves) {
            const int l = lane < n ? lane : 0;
            const int c0 = s_c0[l], nc = (s_cnt[l] + 63) / 64;
            const int h = __ffsll((unsigned long long)__ballot(((heads >> lane) & 1ull) && q >= c0 && q < c0 + nc)) - 1;
            const int32_t j = (q - s_c0[h]) * 64 + lane;
            if (j < s_cnt[h]) {
                const int32_t src = s_beg[h] + j;
                const int32_t tok = F.ntok[src];
                int32_t up = 0;
                for (int i = 0; i < n; i++)
                    if (s_win[i] == 1 && s_head[i] == h) up += s_st[i].t < tok;
                const int64_t dst = (int64_t)s_nb[h] + j + up;
                F.nodes[dst] = fresh_node(&F.nodes[src]);
                F.ntok[dst] = tok;
                if (F.ltime) F.ltime[dst] = fresh_u64(&F.ltime[src]);
                for (int w = 0; w < F.W - 1; w++)
                    F.mext[dst * (F.W - 1) + w] = fresh_u64(&F.mext[(int64_t)src * (F.W - 1) + w]);
                F.moved[src] = (stamp << 32) | (long long)(uint32_t)dst;
            }
        }
        for (int i = wv; i < n; i += kSmallWaves) {
            if (s_win[i] != 1) continue;
            const int h = s_head[i];
            const int32_t d = s_st[i].d, p = s_peer[i];
            const int64_t rest = s_len[i] - d;
            const int32_t *s = B.tokens + s_off[i] + d;
            const int64_t dst = (int64_t)s_nb[h] + s_ord[i] + lower_count(F.ntok + s_beg[h], s_cnt[h], s[0]);
            copy_tokens_narrow(F, N, s_pb[i], s, rest, lane, seen);
            leaf_mext(F, dst, p, lane);
            if (lane == 0) {
                const Node leaf{s[0], (uint32_t)s_pb[i], (int32_t)rest, 0, 0, 0, p < 64 ? 1ull << p : 0ull};
                F.nodes[dst] = leaf;
                F.ntok[dst] = leaf.tok;
                if (F.ltime) F.ltime[dst] = stamps_path(F, p) ? F.now : 0ull;
                s_st[i].kind = kInsDone;
            }
        }
        small_sync();
        // finish
        for (int h = wv; h < n; h += kSmallWaves) {
            if (s_nw[h] == 0) continue;
            const int32_t nb = s_nb[h], c = s_cnt[h] + s_nw[h];
            if (c > kSepCount) F.nsep[nb + lane] = F.ntok[nb + PR_SEP_INDEX(lane, c)];
            if (c >= kSep2Min) sep2_write(F.nsep + nb, F.ntok + nb, c, lane);
            if (lane == 0) {
                const int32_t x = current_pos(F, s_st[h].x, stamp);
                F.nodes[x].ct_beg = nb;
                F.nodes[x].ct_cnt = c;
            }
        }
        small_sync();
        // cut
        for (int i = wv; i < n; i += kSmallWaves) {
            if (s_win[i] != 2) continue;
            InsState r = s_st[i];
            r.c = current_pos(F, r.c, stamp);
            const int64_t rest = B.touch ? 0 : s_len[i] - (int64_t)r.d - r.l;
            cut_edge(F, N, fresh_node(&F.nodes[r.c]), r.c, r.l, B.tokens + s_off[i] + r.d + r.l, rest, s_peer[i],
                     stamps_path(F, s_peer[i]), s_nb[i], s_pb[i], lane, seen);
            if (lane == 0) s_st[i].kind = kInsDone;
        }
        if (s_chunks) stamp++;
        small_sync();
    }
    const uint32_t f = (__ballot(seen & 1u) ? 1u : 0u) | (__ballot(seen & 2u) ? 2u : 0u);
    if (lane == 0 && f) atomicOr(&s_seen, f);
    small_sync();
    if (threadIdx.x == 0) {
        const bool done = s_state == 1;
        SmallStatus r{};
        r.done = done;
        r.hi = (s_seen & 1u) || ctr->hi_tokens;
        r.wide = (s_seen & 2u) || ctr->wide_tokens;
        r.stamps = (uint32_t)(stamp - stamp0);
        r.left = (uint32_t)left;
        r.rounds = (uint32_t)ctr->rounds;
        r.overflow = ctr->overflow != 0;
        r.fallback = ctr->plan_fallback != 0;
        r.n_nodes = n_nodes;
        r.n_pool = n_pool;
        // the rounds after these do not look at the entries they skip again
        if (done || st) *skipped_acc += s_skip;
        *ctr = MergeCounters{};
        ctr->n_nodes = n_nodes;
        ctr->n_pool = n_pool;
        // system scope: straight to the pinned buffer
        const uint64_t *w = reinterpret_cast<const uint64_t *>(&r);
        for (int k = 0; k < (int)(sizeof(r) / 8); k++)
            __hip_atomic_store(reinterpret_cast<uint64_t *>(out) + k, w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

}  // namespace pr

#endif
