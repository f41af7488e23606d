// route.hip -- launches of the route kernels (a translation unit of its own:
// its 60 kernel instances compile beside the rest of the library).
#include "route_kernels.h"

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

}  // namespace

hipError_t launch_route(const RouteForest &F, const RouteBatch &B, const Select &sel, hipStream_t s) {
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
