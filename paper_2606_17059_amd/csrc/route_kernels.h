// route_kernels.h -- gfx950 kernel of the batched router (device code).
//
// One wavefront (64 lanes) serves one query and walks the union forest from
// the root.  Per tree level the wave
//   1. locates the child whose first label token is the next query token: the
//      node's child block was already loaded into the lanes (its first tokens
//      for up to 64 children, else its 64 separators, two cache lines either
//      way), a ballot finds the slot (for a wide block, the sub-range whose
//      first tokens one more load brings), and one scalar load fetches the
//      child's 32-byte record;
//   2. issues, in one batch, the loads of the query token after the label, of
//      the child's mask words, of the child's own first-token array
//      (speculatively, for the next level), and of the label and query tokens
//      it compares: raw buffer loads ranged to the step, 64 tokens per
//      instruction, all of a step in flight at once; query tokens are read
//      once, so their loads are non-temporal (except the first level's, which
//      come with the query's first token, before the walk starts);
//   3. narrows the wave-uniform set of peers still matching by the child's peer
//      mask; every peer that drops out records the depth reached so far (lane
//      i owns peers i, i+64, ...), and takes the common-prefix length of label
//      and query from a ballot of mismatches.
// Peers still in the set at the end matched the whole walked depth.  A wave
// reduction then takes the largest match and the lowest peer id holding it
// (the argmax of Algorithm 1, ties to the lowest id).  Rows of whole cache
// lines are stored non-temporally, so that they do not evict labels.
// When the root has a single child (a prompt prefix every stored sequence
// shares), its record is loaded before the walk and the first level's batch
// goes out without waiting for the query's first token.  The first level
// compares its label against a window of the query's first 128 tokens, or 256
// when the host chose the wide window for a long shared prefix.  Batches of long
// queries can be served in an order computed on the device (longest first,
// route_order.h).
// Labels are read from the int32 pool, or, while every label token lies in
// [0, 65535], from a 16-bit copy of it (half the label bytes and requests; a
// query token outside that range equals no label token either way), or,
// while every label token lies in [0, 131071], from that copy of the low 16
// bits plus a plane of bit 16 (one 32-bit word per 32 tokens, loaded once per
// compare step and handed to the lanes by cross-lane permutes).
#ifndef PR_ROUTE_KERNELS_H
#define PR_ROUTE_KERNELS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "forest_layout.h"
#include "lcp.h"
#include "route_launch.h"
#include "wave_ops.h"

#ifndef PR_FIRST_WINDOW
#define PR_FIRST_WINDOW 1
#endif
#ifndef PR_ROUTE_WAVES_PER_EU
#define PR_ROUTE_WAVES_PER_EU 8
#endif
#ifndef PR_OUT_NT
#define PR_OUT_NT 1
#endif
#ifndef PR_WIN_POLICY
#define PR_WIN_POLICY 0
#endif

namespace pr {

// Output stores of the match rows.  They are written once and never read by
// the kernel; when a row fills whole 128-byte lines (P a multiple of 32),
// non-temporal stores keep them from pushing the labels, which every query
// reads, out of the L2.  Shorter rows share lines with their neighbours, which
// plain stores let the L2 merge (as for the 4-byte chosen peer).  The
// non-temporal path is a raw buffer store over the row (a different operation
// from the plain store, so the compiler cannot fold the two paths into one
// store and lose the policy); lanes past the row are dropped by its range.
template <int W>
__device__ __forceinline__ void store_row(int32_t *row, const int32_t (&m)[W], int32_t P, int lane) {
#if PR_OUT_NT
    if ((P & 31) == 0) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(row, (short)0, P * 4, 0x00020000);
#pragma unroll
        for (int w = 0; w < W; w++) __builtin_amdgcn_raw_buffer_store_b32(m[w], r, (lane + 64 * w) * 4, 0, 2);
        return;
    }
#endif
#pragma unroll
    for (int w = 0; w < W; w++) {
        const int p = lane + 64 * w;
        if (p < P) row[p] = m[w];
    }
}

#if PR_FIRST_WINDOW
// First-level window: the query's first 64 * WV tokens are loaded into
// registers together with its first token, whose HBM round trip the walk
// waits for anyway, so that the first level's compare waits only on its label,
// which the L2 holds.  Lane l of vector j holds token 64 j + l (0 past the
// query).  The loads use the default cache policy: they also bring the lines
// that the first level's next-token load reads.  A window wider than the first
// level's label reads tokens that the second level reads again, so the wide
// window (kWideWinVectors) is for forests whose root has one child with a
// label of at least that many tokens (a long shared system prompt).

template <int WV>
__device__ __forceinline__ void load_window(int32_t (&win)[WV], const int32_t *p, int32_t cnt, int lane) {
    const __amdgpu_buffer_rsrc_t r = token_rsrc(p, cnt * 4);
    int32_t off = lane * 4;  // opaque, as in lcp_step
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int j = 0; j < WV; j++)
        win[j] = __builtin_amdgcn_raw_buffer_load_b32(r, off + j * kWave * 4, 0, PR_WIN_POLICY);
}

// Label tokens [0, cnt) (ra, LT wide, cnt <= 64 * NL) against the window,
// which may hold query tokens past cnt: only lanes below cnt count.  Returns
// the first mismatch, or -1.
template <int NL, typename LT, bool HB, int WV>
__device__ __forceinline__ int32_t lcp_step_win(__amdgpu_buffer_rsrc_t ra, const int32_t (&win)[WV],
                                                int32_t cnt, int lane, const uint32_t *hib, uint32_t A) {
    int32_t va[NL];
    int32_t off = lane * (int32_t)sizeof(LT);  // opaque, as in lcp_step
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int j = 0; j < NL; j++) va[j] = load_label<LT>(ra, off + j * kWave * (int32_t)sizeof(LT));
    if constexpr (HB) {
        HiBits hb = hb_load(hib, A, cnt, lane);
        hb_trim(hb, A, cnt, lane);
#pragma unroll
        for (int j = 0; j < NL; j++) va[j] |= hb_take(hb, j);
    }
    // both sides of the & are evaluated, so no label load becomes conditional
    uint32_t mm = 0;
#pragma unroll
    for (int j = 0; j < NL; j++) mm |= (uint32_t)((j * kWave + lane < cnt) & (va[j] != win[j])) << j;
    if (!__ballot(mm != 0)) return -1;
#pragma unroll
    for (int j = 0; j < NL; j++) {
        const uint64_t bal = __ballot((mm >> j) & 1u);
        if (bal) return j * kWave + (int32_t)(__ffsll((unsigned long long)bal) - 1);
    }
    return -1;
}

// wave_lcp for the first level, whose first query tokens are in win.
template <typename LT, bool HB, int WV>
__device__ __forceinline__ int64_t wave_lcp_first(const LabelSrc<LT, HB> &lab, const int32_t *__restrict__ b,
                                                  int64_t n, const int32_t (&win)[WV], int lane) {
    constexpr int32_t kTokens = kWave * WV;
    const int32_t cnt = (int32_t)min(n, (int64_t)kTokens);
    const __amdgpu_buffer_rsrc_t ra = label_rsrc(lab.p, cnt);
    const int32_t r = cnt <= 2 * kWave ? lcp_step_win<2, LT, HB, WV>(ra, win, cnt, lane, lab.hib, lab.abs)
                                       : lcp_step_win<WV, LT, HB, WV>(ra, win, cnt, lane, lab.hib, lab.abs);
    if (r >= 0 && r < cnt) return r;
    return wave_lcp<LT, HB>(lab, b, n, kTokens, (int64_t)kWave * kLcpVectors, lane);
}
#endif

// A node's child block as held by the wave: lane j holds the first token of
// child beg + j (cnt <= 64) or the block's separator j (cnt > 64).
struct ChildBlock {
    int32_t beg, cnt;  // uniform
    int32_t tok;
};

// Uniform view of the located child.
struct Child {
    int32_t id, lab_off, lab_len, ct_beg, ct_cnt;
    uint64_t mask0;
};

__device__ __forceinline__ void load_block(ChildBlock &cb, const int32_t *__restrict__ ntok,
                                           const int32_t *__restrict__ nsep, int32_t beg, int32_t cnt, int lane) {
    cb.beg = beg;
    cb.cnt = cnt;
    cb.tok = 0;
    if (cnt > kSepCount)
        cb.tok = nsep[beg + lane];
    else if (lane < cnt)
        cb.tok = ntok[beg + lane];
}

// Find the child whose first token is t.  Returns false if there is none.
__device__ __forceinline__ bool locate(const ChildBlock &cb, int32_t t, const Node *__restrict__ nodes,
                                       const int32_t *__restrict__ ntok, const int32_t *__restrict__ nsep, int lane,
                                       Child &c) {
    int32_t idx = -1;
    if (cb.cnt <= kSepCount) {
        const uint64_t b = __ballot(lane < cb.cnt && cb.tok == t);
        if (b) idx = (int32_t)(__ffsll((unsigned long long)b) - 1);
    } else {
        // separators ascend, so the lanes with sep <= t form a prefix
        const uint64_t b = __ballot(cb.tok <= t);
        if (!b) return false;  // t is below every first token
        const int32_t k = (int32_t)__popcll(b) - 1;
        int32_t lo = PR_SEP_INDEX(k, cb.cnt);
        int32_t hi = PR_SEP_HI(k, cb.cnt);
        if (cb.cnt >= kSep2Min) {
            // blocks of 4,160 children or more: the sub-range's own 64
            // separators, two contiguous lines (lane 0's is the first level's
            // k-th, <= t); the rest is at most ceil(span / 64) first tokens
            const int32_t span = hi - lo;
            const uint64_t b2 = __ballot(nsep[cb.beg + kSepCount + kSepCount * k + lane] <= t);
            const int32_t j = (int32_t)__popcll(b2) - 1;
            hi = lo + PR_SEP_HI(j, span);
            lo += PR_SEP_INDEX(j, span);
        }
        while (hi - lo > kWave) {  // sub-ranges of more than 64 children (blocks over 262,144): 64-ary search
            const int32_t stride = (hi - lo + kWave - 1) / kWave;
            const int32_t j = lo + lane * stride;
            bool le = false;
            if (j < hi) le = ntok[cb.beg + j] <= t;
            const uint64_t bl = __ballot(le);
            if (!bl) return false;
            lo = lo + (__popcll(bl) - 1) * stride;
            hi = min(lo + stride, hi);
        }
        const int32_t j = lo + lane;
        bool eq = false;
        if (j < hi) eq = ntok[cb.beg + j] == t;
        const uint64_t be = __ballot(eq);
        if (be) idx = lo + (int32_t)(__ffsll((unsigned long long)be) - 1);
    }
    if (idx < 0) return false;
    const Node r = nodes[cb.beg + idx];  // wave-uniform address: a scalar load
    c.id = cb.beg + idx;
    c.lab_off = (int32_t)r.lab_off;
    c.lab_len = r.lab_len;
    c.ct_beg = r.ct_beg;
    c.ct_cnt = r.ct_cnt;
    c.mask0 = r.mask0;
    return true;
}


// Order key of a candidate: larger is earlier; 0 for peers that are not
// candidates (every real key is above 2^32 - 1026).
__device__ __forceinline__ uint64_t select_key(int32_t m, int32_t p, const Select &sel) {
    const uint32_t tie = (sel.prefer_local && p == sel.local) ? 0u : (uint32_t)p + 1u;
    return ((uint64_t)(uint32_t)m << 32) | (uint64_t)(0xFFFFFFFFu - tie);
}

__device__ __forceinline__ int32_t select_decode(uint64_t key, const Select &sel) {
    if (key == 0) return -1;
    const uint32_t tie = 0xFFFFFFFFu - (uint32_t)key;
    return tie == 0 ? sel.local : (int32_t)(tie - 1u);
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint64_t o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    return v;
}

// elig: the eligibility words, loaded by the caller (all ones for every peer).
template <int W>
__device__ __forceinline__ int32_t select_peers(const int32_t (&m)[W], int32_t P, int lane, const Select &sel,
                                                const uint64_t (&elig)[W], bool want_second, int32_t &second) {
    uint64_t key[W];
#pragma unroll
    for (int w = 0; w < W; w++) {
        const int p = lane + 64 * w;
        const bool ok = p < P && (((elig[w] >> lane) & 1ull) || p == sel.local);
        key[w] = ok ? select_key(m[w], p, sel) : 0ull;
    }
    uint64_t k1 = 0;
#pragma unroll
    for (int w = 0; w < W; w++) k1 = key[w] > k1 ? key[w] : k1;
    k1 = wave_max_u64(k1);
    second = -1;
    if (want_second) {
        uint64_t k2 = 0;
#pragma unroll
        for (int w = 0; w < W; w++) k2 = (key[w] != k1 && key[w] > k2) ? key[w] : k2;
        second = select_decode(wave_max_u64(k2), sel);
    }
    return select_decode(k1, sel);
}

// A team's compare of a long label: its waves take a share each of up to 64 *
// kLcpVectors tokens, all in flight together, and meet at a barrier with the
// first mismatch each has found.  Every wave returns the same value, so the
// waves of a team walk in step; the two rows of `first` alternate, so that a
// wave that is ahead does not overwrite what another still reads.
// What bounds a batch that leaves most of the chip idle is the chain of round
// trips of its longest query, about 1 us for every 1,024 tokens of a label.
struct Team {
    int32_t *first;  // LDS, [2][kTeamMax]
    int wv, lg, row;  // 1 << lg waves
};

template <typename LT, bool HB>
__device__ __forceinline__ int64_t team_lcp(const LabelSrc<LT, HB> &lab, const int32_t *__restrict__ b, int64_t n,
                                            int lane, Team &team) {
    constexpr int64_t kMost = (int64_t)kWave * kLcpVectors;
    for (int64_t base = 0; base < n;) {
        // an equal share of what is left, in whole lines
        const int64_t each = min(((((n - base - 1) >> team.lg) + 1) + 31) & ~(int64_t)31, kMost);
        const int64_t from = base + team.wv * each, to = min(from + each, n);
        int32_t at = INT32_MAX;
        if (from < to) {
            const int64_t r = wave_lcp<LT, HB>(lab, b, to, from, kMost, lane);
            if (r < to) at = (int32_t)r;
        }
        int32_t *row = team.first + team.row * kTeamMax;
        team.row ^= 1;
        if (lane == 0) row[team.wv] = at;
        __syncthreads();
        const int32_t f = (lane >> team.lg) == 0 ? row[lane] : INT32_MAX;
        const uint64_t bal = __ballot(f != INT32_MAX);
        if (bal) return __builtin_amdgcn_readlane(f, (int)(__ffsll((unsigned long long)bal) - 1));
        base += each << team.lg;
    }
    return n;
}

// SEL = false: plain routing (every peer eligible, ties to the lowest id, no
// second pick); the selection options are compiled out.  LT: the label
// pool's token type (int32_t, or uint16_t for the 16-bit copy); HB (with
// uint16_t): bit 16 of every label token comes from the bit plane hib
// (17-bit labels).  WV: vectors of the first-level window.  TEAM: a workgroup
// of up to kTeamMax waves serves one query (team_lcp).
template <int W, bool SEL, typename LT, bool HB = false, int WV = kWinVectors, bool TEAM = false>
__global__ __launch_bounds__(TEAM ? kWave * kTeamMax : kWave * kRouteWavesPerBlock)
__attribute__((amdgpu_waves_per_eu(PR_ROUTE_WAVES_PER_EU))) void route_kernel(
    const Node *__restrict__ nodes, const int32_t *__restrict__ ntok, const int32_t *__restrict__ nsep,
    const uint64_t *__restrict__ mext, const LT *__restrict__ pool, const uint32_t *__restrict__ hib,
    const int32_t *__restrict__ qtok, int64_t num_tokens,
    const int64_t *__restrict__ qoff, int64_t nq, int32_t P, const Select sel_in, int32_t *__restrict__ match_len,
    int32_t *__restrict__ chosen, const int32_t *__restrict__ order) {
    const Select sel = SEL ? sel_in : Select{nullptr, -1, 0, nullptr};
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wv = uniform((int32_t)(threadIdx.x / kWave));
    const int64_t slot = TEAM ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * kRouteWavesPerBlock + wv;
    if (slot >= nq) return;
    Team team{nullptr, wv, TEAM ? 31 - __clz((int)(blockDim.x / kWave)) : 0, 0};
    if constexpr (TEAM) {
        __shared__ int32_t s_first[2][kTeamMax];
        team.first = &s_first[0][0];
    }
    // order (optional) is a permutation of the queries: the dispatcher starts
    // slots in index order, so slot i serves query order[i]
    const int64_t q = order ? (int64_t)order[slot] : slot;
    int32_t *row = match_len + q * (int64_t)P;
    // The offsets and the root's record are loaded together, and a query with
    // bad offsets runs as an empty one (its row is written as -1 at the end),
    // so that no branch on the offsets sits between those loads and the
    // walk's first loads.
    int64_t qb0 = qoff[q], qe0 = qoff[q + 1];
    const Node root = nodes[0];
    int32_t root_beg = root.ct_beg, root_cnt = root.ct_cnt;
    // both loads are issued before anything waits on either (the compiler
    // would otherwise sink the offsets' load below the root's branches)
    asm volatile("" : "+s"(qb0), "+s"(qe0), "+s"(root_beg), "+s"(root_cnt));
    const bool bad = qb0 < 0 || qe0 < qb0 || qe0 > num_tokens || qe0 - qb0 > (int64_t)INT32_MAX;
    const int64_t qb = bad ? 0 : qb0;
    const int64_t qlen = bad ? 0 : qe0 - qb0;
    const int32_t *qs = qtok + qb;
    // the eligibility words are read now and used after the walk, so their
    // load is not one more round trip at the end
    uint64_t elig[W];
#pragma unroll
    for (int w = 0; w < W; w++) elig[w] = (SEL && sel.eligible) ? sel.eligible[w] : ~0ull;

    int32_t m[W];
    uint64_t alive[W];
#pragma unroll
    for (int w = 0; w < W; w++) {
        m[w] = 0;
        const int rem = P - 64 * w;
        alive[w] = rem >= 64 ? ~0ull : (rem > 0 ? ((1ull << rem) - 1ull) : 0ull);
    }

    int64_t d = 0;
    // The root's child block and, when the root has a single child (every
    // stored sequence starts with the same token, as behind a shared system
    // prompt), that child's record: the first level then issues its batch of
    // loads without waiting for the query's first token or a record load.
    ChildBlock cb;
    load_block(cb, ntok, nsep, root_beg, root_cnt, lane);
    const bool single = root_cnt == 1;
    const int32_t c0_id = single ? root_beg : 0;  // node 0 always exists
    const Node r0 = nodes[c0_id];
    const Child c0{c0_id, (int32_t)r0.lab_off, r0.lab_len, r0.ct_beg, r0.ct_cnt, r0.mask0};
    const int32_t c0_tok = r0.tok;
#if PR_FIRST_WINDOW
    // the query's first token comes with the window (lane 0 of its first
    // vector), read where the first level needs it
    int32_t t = 0;
#else
    int32_t t = qlen > 0 ? qs[0] : 0;
#endif
    // One tree level; returns whether the walk goes on.  The first level is a
    // separate instance (FIRST), so that the window's registers die after it.
    // With `known` the level's child is the root's single child c0, taken on
    // the assumption that the query starts with its first token; the check
    // waits until the level's loads are issued.
    auto level = [&](auto first_tag, const auto &win, auto known_tag) __attribute__((always_inline)) -> bool {
        constexpr bool FIRST = decltype(first_tag)::value;
        constexpr bool KNOWN = FIRST && decltype(known_tag)::value;
        Child c;
        if constexpr (KNOWN) {
            c = c0;
        } else {
            if constexpr (FIRST && PR_FIRST_WINDOW) t = uniform(win[0]);
            if (!locate(cb, t, nodes, ntok, nsep, lane, c)) return false;
        }
        if (c.lab_len <= 0) return false;  // only the root has an empty label
        // one batch of loads per level: next token, ext mask words, the next
        // child block (used if the label matches in full) and the label compare
        const int64_t end = d + c.lab_len;
        const int32_t tnext = end < qlen ? qs[end] : 0;
        uint64_t mx[W];
        mx[0] = c.mask0;
#pragma unroll
        for (int w = 1; w < W; w++) mx[w] = mext[(int64_t)c.id * (W - 1) + (w - 1)];
        load_block(cb, ntok, nsep, c.ct_beg, c.ct_cnt, lane);
        const int64_t n = min((int64_t)c.lab_len, qlen - d);
        const LabelSrc<LT, HB> lab{pool + (uint32_t)c.lab_off, hib, (uint32_t)c.lab_off};
        int64_t l;
        if (TEAM && n > kTeamSplit && team.lg > 0)
            l = team_lcp<LT, HB>(lab, qs + d, n, lane, team);
        else if constexpr (FIRST)
            l = wave_lcp_first<LT, HB, WV>(lab, qs, n, win, lane);
        else
            l = wave_lcp<LT, HB>(lab, qs + d, n, 0, (int64_t)kWave * kLcpFirstVectors, lane);
        if constexpr (KNOWN) {
            if constexpr (PR_FIRST_WINDOW) t = uniform(win[0]);
            if (t != c0_tok) return false;  // no child starts with the query's first token
        }
        bool any = false;
#pragma unroll
        for (int w = 0; w < W; w++) {
            const uint64_t nm = alive[w] & mx[w];
            if (((alive[w] & ~nm) >> lane) & 1ull) m[w] = (int32_t)d;
            alive[w] = nm;
            any |= nm != 0ull;
        }
        if (!any) return false;  // no peer holds this edge (left behind by a replaced snapshot)
        d += l;
        if (l < c.lab_len) return false;
        t = tnext;
        return d < qlen;
    };
    struct NoWindow {};
#if PR_FIRST_WINDOW
    int32_t win[WV];
    load_window<WV>(win, qs, (int32_t)min(qlen, (int64_t)kWave * WV), lane);
    if constexpr (TEAM) {
        // the host knows the batch's mean at most (its buffer may be larger than its
        // queries): a query keeps the waves that its own length pays for, and the
        // rest end here, past the loads that the walk waits for first (a barrier
        // waits for the waves that are left)
        if (qlen < team_least(W) || qlen < kTeamTokens << team.lg) {
            team.lg = qlen < team_least(W) ? 0 : 31 - __clz((int32_t)qlen / (int32_t)kTeamTokens);
            if ((wv >> team.lg) != 0) return;
        }
    }
    bool more = false;
    if (qlen > 0) more = single ? level(std::true_type{}, win, std::true_type{})
                                : level(std::true_type{}, win, std::false_type{});
#else
    bool more = qlen > 0 && level(std::false_type{}, NoWindow{}, std::false_type{});
#endif
    while (more) more = level(std::false_type{}, NoWindow{}, std::false_type{});

    if (TEAM && wv != 0) return;  // every wave of a team has the same result
    if (bad) {
        if (match_len)
            for (int p = lane; p < P; p += kWave) row[p] = -1;
        if (lane == 0) {
            chosen[q] = -1;
            if (sel.second) sel.second[q] = -1;
        }
        return;
    }
    // peers still holding the walked path matched all of it
#pragma unroll
    for (int w = 0; w < W; w++)
        if ((alive[w] >> lane) & 1ull) m[w] = (int32_t)d;

    if (match_len) store_row<W>(row, m, P, lane);
    int32_t second;
    const int32_t best = select_peers<W>(m, P, lane, sel, elig, sel.second != nullptr, second);
    if (lane == 0) {
        chosen[q] = best;  // 4 bytes a query: plain stores, which the L2 merges into whole lines
        if (sel.second) sel.second[q] = second;
    }
}

}  // namespace pr

#endif
