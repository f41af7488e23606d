// route_launch.h -- what the host code needs to launch the route kernels
// (route_kernels.h, compiled in route.hip): sizes, argument structs, launches.
#ifndef PR_ROUTE_LAUNCH_H
#define PR_ROUTE_LAUNCH_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "forest_layout.h"
#include "lcp.h"

#ifndef PR_ROUTE_WAVES_PER_BLOCK
#define PR_ROUTE_WAVES_PER_BLOCK 1
#endif
#ifndef PR_WIN_VECTORS
#define PR_WIN_VECTORS 2
#endif

namespace pr {

constexpr int kRouteWavesPerBlock = PR_ROUTE_WAVES_PER_BLOCK;
constexpr int kWinVectors = PR_WIN_VECTORS;  // 64-token vectors of the first-level window
constexpr int kWideWinVectors = 4;           // ... of the wide one
constexpr int kTeamMax = 16;                 // waves of a query's team at most
constexpr int64_t kTeamSplit = 256;          // labels beyond this many tokens are split over the team
constexpr int64_t kTeamTokens = 512;         // ... and a query has a wave for every so many tokens at most
static_assert(kWinVectors >= 2 && kWinVectors <= 16, "window of 2 to 16 vectors");

// Tokens of the shortest query that a team serves.  Meeting at a barrier for each
// label costs about 0.3 us of the 0.5 us that 1,000 tokens take a wave; with more
// mask words a level has more to do in every wave, and sixteen spill in a team
// (us with 1 / 4 waves, 8 past 4,000 tokens; 48 queries each):
//   mask words    1,800 tokens  2,400          4,400          6,300
//       2          4.28 / 4.60   5.41 /  4.56   6.96 /  4.91   8.24 /  5.46
//       8          5.34 / 5.84   6.47 /  5.94   7.91 /  6.28   8.18 /  6.26
//      16          6.57 / 7.81   7.62 /  8.11   9.39 /  8.61  10.74 /  8.94
//      16, 512     8.00 / 10.3   9.03 / 10.10  10.98 / 13.17  12.94 / 13.53   queries
// One mask word: 4.79 / 4.49 at 1,300 tokens, 4.34 / 4.44 at 1,100.
constexpr int64_t team_least(int W) { return W == 1 ? 1024 : (W < 16 ? 2048 : 5120); }

// Peer selection (the argmax of Algorithm 1, with the push-back and failover
// rules of Sections "Hot specialist push-back" and "In-flight forwarded
// request failure").  Candidates are ordered by larger match, then, when
// prefer_local is set, the local peer, then the lower id; best is the first
// eligible candidate and second the next (-1 when there is none).  The local
// peer is always eligible.  Plain routing is the case "every peer eligible,
// no local peer, no second".
struct Select {
    const uint64_t *eligible;  // ceil(P / 64) words, bit p % 64 of word p / 64; nullptr: every peer
    int32_t local;             // -1: none
    int32_t prefer_local;
    int32_t *second;           // nullptr: not wanted
};

// The longest-first order (route_order_count_kernel, route_order_scatter_kernel).
constexpr int kOrderThreads = 1024;
constexpr int kOrderWaves = kOrderThreads / kWave;
constexpr int kOrderPerThread = 4;
constexpr int kOrderChunk = kOrderThreads * kOrderPerThread;  // queries per workgroup
constexpr int kOrderBuckets = 16;
constexpr int kOrderMaxBlocks = 16;
constexpr int32_t kOrderMaxQueries = kOrderChunk * kOrderMaxBlocks;  // 65,536

// The forest's arrays as a route reads them.
struct RouteForest {
    const Node *nodes;
    const int32_t *ntok, *nsep;
    const uint64_t *mext;
    const int32_t *pool;
    const uint16_t *pool16;  // nullptr: labels are read from pool
    const uint32_t *hib;     // bit plane of 17-bit labels, nullptr: 16-bit (or int32) labels
    int32_t P, W;
    bool wide_window;
};

struct RouteBatch {
    const int32_t *tokens;
    int64_t num_tokens;
    const int64_t *offsets;
    int64_t n;
    int32_t *match_len, *chosen;
    const int32_t *order;  // nullptr: index order
};

// Enqueue the route kernel: plain routing, or selection when sel asks for it.
hipError_t launch_route(const RouteForest &F, const RouteBatch &B, const Select &sel, hipStream_t s);

// The launch of a batch with a team of `waves` waves for every query (route_team.hip).
void launch_route_team(const RouteForest &F, const RouteBatch &B, const Select &sel, int waves, hipStream_t s);

// Enqueue the two order launches; bkt, blockcnt and order as in route.hip.
hipError_t launch_route_order(const int64_t *q_offsets, int64_t nq, int64_t ntok, hipStream_t s, uint8_t *bkt,
                              int32_t *blockcnt, int32_t *order);

}  // namespace pr

#endif
