// route_team.hip -- launches of the route kernels that serve a query with a team
// of waves (a translation unit of its own, compiled beside route.hip).
#include "route_kernels.h"

namespace pr {

namespace {

template <int W, bool SEL, typename LT, bool HB>
void launch_t(const RouteForest &F, const LT *pool, const RouteBatch &B, const Select &sel, int waves, hipStream_t s) {
    hipLaunchKernelGGL((route_kernel<W, SEL, LT, HB, kWinVectors, true>), dim3((unsigned)B.n), dim3(kWave * waves), 0,
                       s, F.nodes, F.ntok, F.nsep, F.mext, pool, F.hib, B.tokens, B.num_tokens, B.offsets, B.n, F.P,
                       sel, B.match_len, B.chosen, B.order);
}

template <int W, bool SEL>
void launch_l(const RouteForest &F, const RouteBatch &B, const Select &sel, int waves, hipStream_t s) {
    if (F.pool16 && F.hib)
        launch_t<W, SEL, uint16_t, true>(F, F.pool16, B, sel, waves, s);
    else if (F.pool16)
        launch_t<W, SEL, uint16_t, false>(F, F.pool16, B, sel, waves, s);
    else
        launch_t<W, SEL, int32_t, false>(F, F.pool, B, sel, waves, s);
}

template <int W>
void launch_w(const RouteForest &F, const RouteBatch &B, const Select &sel, int waves, hipStream_t s) {
    if (!sel.eligible && !sel.prefer_local && !sel.second)
        launch_l<W, false>(F, B, sel, waves, s);
    else
        launch_l<W, true>(F, B, sel, waves, s);
}

}  // namespace

void launch_route_team(const RouteForest &F, const RouteBatch &B, const Select &sel, int waves, hipStream_t s) {
    switch (F.W) {
        case 1: launch_w<1>(F, B, sel, waves, s); break;
        case 2: launch_w<2>(F, B, sel, waves, s); break;
        case 4: launch_w<4>(F, B, sel, waves, s); break;
        case 8: launch_w<8>(F, B, sel, waves, s); break;
        default: launch_w<16>(F, B, sel, waves, s); break;
    }
}

}  // namespace pr
