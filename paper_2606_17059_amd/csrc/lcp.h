// lcp.h -- the common prefix of an edge label and a sequence, compared by a
// wave (routes and merge walks): raw buffer loads ranged to a step, 64 tokens
// per instruction, all of a step in flight at once.
#ifndef PR_LCP_H
#define PR_LCP_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#ifndef PR_LCP_VECTORS
#define PR_LCP_VECTORS 16
#endif
#ifndef PR_LCP_FIRST_VECTORS
#define PR_LCP_FIRST_VECTORS 9
#endif
#ifndef PR_QUERY_NT
#define PR_QUERY_NT 1
#endif
#ifndef PR_ALIGN_STEPS
#define PR_ALIGN_STEPS 1
#endif

namespace pr {

constexpr int kWave = 64;
constexpr int kLcpVectors = PR_LCP_VECTORS;               // 64-token vectors per compare step
constexpr int kLcpFirstVectors = PR_LCP_FIRST_VECTORS;    // ... in a label's first step

// Raw buffer resource over bytes [p, p + bytes): loads past the end return 0
// without touching memory (the hardware range check of stride-0 buffers).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t token_rsrc(const int32_t *p, int32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(p), (short)0, bytes, 0x00020000);
}

// Cache policy of the query loads: non-temporal (read once).
#ifdef PR_QUERY_POLICY
constexpr int kQueryPolicy = PR_QUERY_POLICY;
#else
constexpr int kQueryPolicy = PR_QUERY_NT ? 2 : 0;
#endif

// Label tokens: int32, or uint16 (the 16-bit copy of the pool).  Raw buffer
// resources over the label bytes and loads of one token per lane.
template <typename LT>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t label_rsrc(const LT *p, int32_t cnt) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<LT *>(p), (short)0, cnt * (int32_t)sizeof(LT), 0x00020000);
}

template <typename LT>
__device__ __forceinline__ int32_t load_label(__amdgpu_buffer_rsrc_t r, int32_t off) {
    if constexpr (sizeof(LT) == 2)
        return (int32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
    else
        return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
}

// Where a compare step reads its labels.  p: the label's first token in the
// pool (int32), or in its 16-bit copy.  HB (17-bit labels, with the 16-bit
// copy): bit 16 of pool token i is bit i % 32 of hib[i / 32], and abs is the
// label's offset in the pool, so that a step knows which bit words to load.
template <typename LT, bool HB>
struct LabelSrc {
    const LT *p;
    const uint32_t *hib;
    uint32_t abs;
};

// The bit words of a step over pool tokens [A, A + cnt), A = abs + base: lane w
// holds word A / 32 + w (w <= 32 for cnt <= 1024), with the bits of tokens at
// or past A + cnt cleared, so that lanes past the step compare equal as with
// plain labels.  Lane l of every 64-token vector j then takes bit
// (A % 32 + l) % 32 of lane 2 j + (A % 32 + l) / 32's word (hb_take).
struct HiBits {
    uint32_t word;   // this lane's bit word
    int32_t addr;    // ds_bpermute byte address of vector 0's source lane
    uint32_t shift;  // bit position inside it
};

// The load is issued by hb_load; hb_trim, called once every load of the step
// has been issued, clears the bits past the step (so that the first use of
// the word does not make the compiler wait on it before the other loads).
__device__ __forceinline__ HiBits hb_load(const uint32_t *hib, uint32_t A, int32_t cnt, int lane) {
    const uint32_t a0 = A & 31u;
    const int32_t nwords = (int32_t)((a0 + (uint32_t)cnt + 31u) >> 5);
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(hib + (A >> 5)), (short)0, nwords * 4, 0x00020000);
    HiBits h;
    h.word = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, lane * 4, 0, 0);
    h.addr = (int32_t)(((a0 + (uint32_t)lane) >> 5) << 2);
    h.shift = (a0 + (uint32_t)lane) & 31u;
    return h;
}

__device__ __forceinline__ void hb_trim(HiBits &h, uint32_t A, int32_t cnt, int lane) {
    const int32_t lim = cnt + (int32_t)(A & 31u) - 32 * lane;  // bits of this lane's word inside the step
    h.word = lim >= 32 ? h.word : (lim <= 0 ? 0u : h.word & ((1u << lim) - 1u));
}

// Bit 16 of the label token lane `lane` holds in vector j.
__device__ __forceinline__ int32_t hb_take(const HiBits &h, int j) {
    const uint32_t w = (uint32_t)__builtin_amdgcn_ds_bpermute(h.addr + 8 * j, (int32_t)h.word);
    return (int32_t)(((w >> h.shift) & 1u) << 16);
}

// One compare step over cnt <= 64 * NV tokens: ra holds the label tokens
// (LT wide), rb the query tokens, both ranged to cnt tokens so that lanes past
// the end read 0 on both sides and compare equal.  Returns the first
// mismatch, or -1.
template <int NV, typename LT, bool HB = false>
__device__ __forceinline__ int32_t lcp_step(__amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb, int lane,
                                            const uint32_t *hib = nullptr, uint32_t A = 0, int32_t cnt = 0) {
    int32_t va[NV], vb[NV];
    // opaque lane offset: with its range unknown the per-vector constant stays
    // an add, which folds into the loads' immediate offsets; and as each step
    // size gets its own opaque value, the compiler cannot merge the first loads
    // of the short and the long step into one block that waits before the long
    // step issues the rest
    int32_t off = lane * 4;
    asm volatile("" : "+v"(off));
    // 16-bit labels take their own (opaque) lane offset
    int32_t offa = off;
    if constexpr (sizeof(LT) != 4) {
        offa = lane * (int32_t)sizeof(LT);
        asm volatile("" : "+v"(offa));
    }
#pragma unroll
    for (int j = 0; j < NV; j++) {
        va[j] = load_label<LT>(ra, offa + j * kWave * (int32_t)sizeof(LT));
        vb[j] = __builtin_amdgcn_raw_buffer_load_b32(rb, off + j * kWave * 4, 0, kQueryPolicy);
    }
    if constexpr (HB) {
        HiBits hb = hb_load(hib, A, cnt, lane);
        hb_trim(hb, A, cnt, lane);
#pragma unroll
        for (int j = 0; j < NV; j++) va[j] |= hb_take(hb, j);
    }
    // fold every vector's mismatches into a lane mask before branching, so
    // that no load of the step can be deferred behind an early exit
    uint32_t mm = 0;
#pragma unroll
    for (int j = 0; j < NV; j++) mm |= (uint32_t)(va[j] != vb[j]) << j;
    if (!__ballot(mm != 0)) return -1;
#pragma unroll
    for (int j = 0; j < NV; j++) {
        const uint64_t bal = __ballot((mm >> j) & 1u);
        if (bal) return j * kWave + (int32_t)(__ffsll((unsigned long long)bal) - 1);
    }
    return -1;
}

// Length of the common prefix of a[0..n) (a label) and b[0..n) (query
// tokens), from position base on: the first i in [base, n) with a[i] != b[i],
// or n.  Wave-cooperative; every lane returns the same value.  The first step
// compares up to `first` tokens (a label's first step: 64 * kLcpFirstVectors,
// which bounds what a mismatch early in a long label reads in vain), later
// steps up to 64 * kLcpVectors, which halves the round trips over long labels
// that match in full.  Every step but a label's last ends at a query line, 0 to
// 31 tokens short of its nominal size; the nine-vector first step leaves the
// rest of a 1024-token label to an eight-vector step.  Steps of at most 128
// and 512 tokens take two- and eight-vector forms.
template <typename LT, bool HB>
__device__ __forceinline__ int64_t wave_lcp(const LabelSrc<LT, HB> &lab, const int32_t *__restrict__ b,
                                            int64_t n, int64_t base, int64_t first, int lane) {
    const LT *__restrict__ a = lab.p;
    for (int64_t step = first; base < n; step = (int64_t)kWave * kLcpVectors) {
        int32_t cnt = (int32_t)min(n - base, step);
#if PR_ALIGN_STEPS
        // a step that is not the label's last ends at a 128-byte line of the
        // query, so no line is split between two steps: its non-temporal read
        // would not keep the line in the L2 for the next step
        if (n - base > step) cnt -= (int32_t)(((uint32_t)((uintptr_t)(b + base) >> 2) + (uint32_t)step) & 31u);
#endif
        const __amdgpu_buffer_rsrc_t ra = label_rsrc(a + base, cnt);
        const __amdgpu_buffer_rsrc_t rb = token_rsrc(b + base, cnt * 4);
        const uint32_t A = lab.abs + (uint32_t)base;
        int32_t r;
        if (cnt <= 2 * kWave)
            r = lcp_step<2, LT, HB>(ra, rb, lane, lab.hib, A, cnt);
        else if (cnt <= 8 * kWave)
            r = lcp_step<8, LT, HB>(ra, rb, lane, lab.hib, A, cnt);
        else if (kLcpFirstVectors > 8 && kLcpVectors > kLcpFirstVectors && cnt <= kWave * kLcpFirstVectors)
            r = lcp_step<kLcpFirstVectors, LT, HB>(ra, rb, lane, lab.hib, A, cnt);
        else
            r = lcp_step<kLcpVectors, LT, HB>(ra, rb, lane, lab.hib, A, cnt);
        if (r >= 0 && r < cnt) return base + r;
        base += cnt;
    }
    return n;
}

}  // namespace pr

#endif
