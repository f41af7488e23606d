// route.hip -- launches of the route kernels (a translation unit of its own:
// its 60 kernel instances compile beside the rest of the library).
#include "route_kernels.h"
#include "route_order.h"

#include <algorithm>

namespace pr {

namespace {

template <int W, bool SEL, typename LT, bool HB>
void launch_t(const RouteForest &F, const LT *pool, const RouteBatch &B, const Select &sel, hipStream_t s) {
    const int64_t blocks = (B.n + kRouteWavesPerBlock - 1) / kRouteWavesPerBlock;
    if (F.wide_window)
        hipLaunchKernelGGL((route_kernel<W, SEL, LT, HB, kWideWinVectors>), dim3((unsigned)blocks),
                           dim3(kWave * kRouteWavesPerBlock), 0, s, F.nodes, F.ntok, F.nsep, F.mext, pool, F.hib,
                           B.tokens, B.num_tokens, B.offsets, B.n, F.P, sel, B.match_len, B.chosen, B.order);
    else
        hipLaunchKernelGGL((route_kernel<W, SEL, LT, HB>), dim3((unsigned)blocks), dim3(kWave * kRouteWavesPerBlock),
                           0, s, F.nodes, F.ntok, F.nsep, F.mext, pool, F.hib, B.tokens, B.num_tokens, B.offsets, B.n,
                           F.P, sel, B.match_len, B.chosen, B.order);
}

// Over the narrow labels when they are current.
template <int W, bool SEL>
void launch_l(const RouteForest &F, const RouteBatch &B, const Select &sel, hipStream_t s) {
    if (F.pool16 && F.hib)
        launch_t<W, SEL, uint16_t, true>(F, F.pool16, B, sel, s);
    else if (F.pool16)
        launch_t<W, SEL, uint16_t, false>(F, F.pool16, B, sel, s);
    else
        launch_t<W, SEL, int32_t, false>(F, F.pool, B, sel, s);
}

template <int W>
void launch_w(const RouteForest &F, const RouteBatch &B, const Select &sel, hipStream_t s) {
    const bool plain = !sel.eligible && !sel.prefer_local && !sel.second;
    if (plain)
        launch_l<W, false>(F, B, sel, s);
    else
        launch_l<W, true>(F, B, sel, s);
}

// Waves launched for each query (a power of two); a query shorter than the mean
// that tokens gives, as where they are a buffer that the batch only starts, ends
// the ones it does not pay for (512 queries of 300 tokens in a buffer of 32 M: 3.6
// us with a wave each, 6.2 with sixteen, 4.1 with fifteen that end).  A small batch of long queries takes
// as long as its longest query's chain of compare steps, so a team shares them,
// a wave for every 512 tokens of the mean query: 48 queries of 20,000 tokens
// 34.4 -> 8.4 us, one 33.2 -> 8.0, 512 of 5,300 10.9 -> 7.1.  Past 8,192 waves
// (the chip's slots) or half as many queries as tokens a query, teams read as
// much more as they wait less (us with 1, 2, 4, 8, 16 waves):
//   20,700 tokens   512 queries  48.1  32.2  21.3  16.7  17.2
//                 2,048          56.0  51.4  48.5  48.4  53.5
//                 4,096          78.9  86.9  81.0  85.6  97.4
//    5,300 tokens 2,048          13.4  13.5  13.3  16.0  24.7
//    2,500 tokens 1,024           7.9   7.8   7.5  10.0  16.5
//                 2,048           8.8   9.6  10.5  16.9  29.2
//    1,400 tokens   512           5.6   5.3   5.6   6.2   8.4
//                 1,024           5.4   5.6   6.4   9.0  14.2
int team_waves(int64_t n, int64_t tokens, int W) {
    if (n <= 0 || n > 2048) return 1;
    const int64_t mean = tokens / n;
    if (2 * n > mean || mean < team_least(W) || (W >= 16 && n > 256 && mean < 8192)) return 1;
    int waves = 1;
    while (waves < kTeamMax && 2 * kTeamTokens * waves <= mean && 2 * waves * n <= 8192) waves *= 2;
    return waves;
}

}  // namespace

hipError_t launch_route(const RouteForest &F, const RouteBatch &B, const Select &sel, hipStream_t s) {
    if (const int waves = team_waves(B.n, B.num_tokens, F.W); waves > 1) {
        launch_route_team(F, B, sel, waves, s);
        return hipGetLastError();
    }
    switch (F.W) {
        case 1: launch_w<1>(F, B, sel, s); break;
        case 2: launch_w<2>(F, B, sel, s); break;
        case 4: launch_w<4>(F, B, sel, s); break;
        case 8: launch_w<8>(F, B, sel, s); break;
        default: launch_w<16>(F, B, sel, s); break;
    }
    return hipGetLastError();
}

// The two order launches (at most 16 workgroups each) on stream s: bkt gets
// every query's length bucket (a quarter of the mean query wide), blockcnt
// the per-workgroup bucket counts, order the queries longest first.  Every
// entry read is written earlier in the same two launches, so the buffers need
// no clearing.  nq <= kOrderMaxQueries.
hipError_t launch_route_order(const int64_t *q_offsets, int64_t nq, int64_t ntok, hipStream_t s, uint8_t *bkt,
                              int32_t *blockcnt, int32_t *order) {
    const uint32_t unit = (uint32_t)std::min<int64_t>(std::max<int64_t>(1, ntok / nq / 4), INT32_MAX);
    const unsigned blocks = (unsigned)((nq + kOrderChunk - 1) / kOrderChunk);
    hipLaunchKernelGGL(route_order_count_kernel, dim3(blocks), dim3(kOrderThreads), 0, s, q_offsets, (int32_t)nq,
                       unit, bkt, blockcnt);
    hipLaunchKernelGGL(route_order_scatter_kernel, dim3(blocks), dim3(kOrderThreads), 0, s, bkt, (int32_t)nq,
                       blockcnt, order);
    return hipGetLastError();
}

}  // namespace pr
