// The LDS-tiled 2D smoothing launches of the FP64 hierarchy (the finest level's
// in chhs_tile2d_l0.hip).
#include "chhs_tile2d.hpp"

namespace chhs {

template <>
void launch_tile2d<double>(const Batch<double>& b, const TileTask* t, int nt, bool level0, int ns,
                           int epi, bool pro, int threads, bool rhs, int ty, bool zero,
                           double* partial, hipStream_t st) {
    (void)zero;
    if (nt <= 0) return;
    if (level0) {
        if (!rhs) launch_tile2d_l0(b, t, nt, ns, epi, pro, threads, ty, partial, st);
        return;
    }
    if (rhs) {
        // first pre-smoothing launch of a coarse level (no prolongation)
        if (pro || epi == 2) return;
#define CHHS_TILE_RHS(NS, EPI)                                                    \
    if (ns == NS && epi == EPI) {                                                 \
        launch_one<double, false, NS, EPI, false, false, true>(b, t, nt, threads, ty, partial, st); \
        return;                                                                   \
    }
        CHHS_TILE_RHS(1, 0)
        CHHS_TILE_RHS(1, 1)
        CHHS_TILE_RHS(2, 0)
        CHHS_TILE_RHS(2, 1)
#undef CHHS_TILE_RHS
        return;
    }
    // the restriction follows pre-smoothing (no prolongation), the norm partials
    // are the finest level's
#define CHHS_TILE_CASE(NS, EPI, PRO)                                              \
    if (ns == NS && epi == EPI && pro == PRO) {                                   \
        launch_one<double, false, NS, EPI, PRO, false>(b, t, nt, threads, ty, partial, st); \
        return;                                                                   \
    }
    CHHS_TILE_CASE(1, 0, false)
    CHHS_TILE_CASE(1, 0, true)
    CHHS_TILE_CASE(1, 1, false)
    CHHS_TILE_CASE(2, 0, false)
    CHHS_TILE_CASE(2, 0, true)
    CHHS_TILE_CASE(2, 1, false)
#undef CHHS_TILE_CASE
}

}  // namespace chhs
