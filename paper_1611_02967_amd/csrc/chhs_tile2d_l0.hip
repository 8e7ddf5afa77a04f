// The LDS-tiled 2D smoothing launches of the finest FP64 level.
#include "chhs_tile2d.hpp"

namespace chhs {

void launch_tile2d_l0(const Batch<double>& b, const TileTask* t, int nt, int ns, int epi, bool pro,
                      int threads, int ty, double* partial, hipStream_t st) {
#define CHHS_TILE_CASE(NS, EPI, PRO)                                              \
    if (ns == NS && epi == EPI && pro == PRO) {                                   \
        launch_one<double, true, NS, EPI, PRO, false>(b, t, nt, threads, ty, partial, st); \
        return;                                                                   \
    }
#define CHHS_TILE_NS(NS)         \
    CHHS_TILE_CASE(NS, 0, false) \
    CHHS_TILE_CASE(NS, 0, true)  \
    CHHS_TILE_CASE(NS, 1, false) \
    CHHS_TILE_CASE(NS, 2, false) \
    CHHS_TILE_CASE(NS, 2, true)
    CHHS_TILE_NS(1)
    CHHS_TILE_NS(2)
#undef CHHS_TILE_NS
#undef CHHS_TILE_CASE
}

}  // namespace chhs
