// The LDS-tiled 2D smoothing launches of the FP32 correction hierarchy.
#include "chhs_tile2d.hpp"

namespace chhs {

// FP32 correction form (mixed-precision inner solve): general right-hand
// sides, no norm epilogue.
template <>
void launch_tile2d<float>(const Batch<float>& b, const TileTask* t, int nt, bool level0, int ns,
                          int epi, bool pro, int threads, bool rhs, int ty, bool zero,
                          double* partial, hipStream_t st) {
    (void)level0;
    if (nt <= 0) return;
    if (zero) {
        // first launch of a correction cycle on the finest level (64 x 16 or
        // 64 x 32 tiles)
        if (pro || rhs || epi == 2 || (ty != kTileY && ty != kTileYTall)) return;
#define CHHS_TILE_ZERO(NS, EPI)                                                   \
    if (ns == NS && epi == EPI) {                                                 \
        launch_one<float, false, NS, EPI, false, true, false, true>(b, t, nt, threads, ty, partial, st); \
        return;                                                                   \
    }
        CHHS_TILE_ZERO(1, 0)
        CHHS_TILE_ZERO(1, 1)
        CHHS_TILE_ZERO(2, 0)
        CHHS_TILE_ZERO(2, 1)
#undef CHHS_TILE_ZERO
        return;
    }
    if (rhs) {
        if (pro || epi == 2) return;
#define CHHS_TILE_RHS(NS, EPI)                                                    \
    if (ns == NS && epi == EPI) {                                                 \
        launch_one<float, false, NS, EPI, false, true, true>(b, t, nt, threads, ty, partial, st); \
        return;                                                                   \
    }
        CHHS_TILE_RHS(1, 0)
        CHHS_TILE_RHS(1, 1)
        CHHS_TILE_RHS(2, 0)
        CHHS_TILE_RHS(2, 1)
#undef CHHS_TILE_RHS
        return;
    }
#define CHHS_TILE_CASE(NS, EPI, PRO)                                              \
    if (ns == NS && epi == EPI && pro == PRO) {                                   \
        launch_one<float, false, NS, EPI, PRO, true>(b, t, nt, threads, ty, partial, st); \
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
