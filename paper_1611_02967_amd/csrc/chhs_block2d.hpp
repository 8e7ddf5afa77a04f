// Tiles of FP64 2D levels with a thread for every pair of cells.
//
// The work and the result of k_tile2d's FP64 form (fused red-black steps on a 64 x
// TY tile with its halo in LDS, the same optional parts and the same bits), for
// levels of few tiles, where the time of one workgroup is the time of the launch:
// a chain of dependent loads, phases and barriers, not bandwidth.  Against
// k_tile2d's loop over the region's pairs:
//   - slots (pairs of x-adjacent cells, x even) are only those within H faces of
//     the tile, not the whole padded rectangle, and every slot has its thread;
//   - the slots of the tile come first, row by row, so that lanes l and l ^ 32 of
//     a wave are the two rows of a coarse cell: the residual and the restriction
//     take phi^m and f from the registers of the thread that smoothed the pair,
//     where k_tile2d read them from memory again (after RHS, what another wave
//     had just written);
//   - the halo's slots follow by distance, so whole waves drop out of the later
//     phases.
// In LDS a row's even columns precede its odd ones (k_tile2d's layout).
// Measured, k_tile2d with 1024 threads / this kernel: a call at 512^2 4629 / 4013 us,
// 448 x 320 4324 / 4004, 1024^2 2705 / 2576, 2048^2 (its coarse levels) 6525 / 6430,
// 32 small grids 2687 / 2596, 64^2 1794 / 1757.
#pragma once

#include "chhs_cell.hpp"

namespace chhs {
namespace {

constexpr int block_dist(int v, int n) { return v < 0 ? -v : (v >= n ? v - n + 1 : 0); }

template <int H, int TY>
struct BlockSlots {
    static constexpr int TX = kTileX;
    static constexpr int HX = (H + 1) & ~1;        // x halo padded to keep pairs aligned
    static constexpr int R = TY + 2 * H;
    static constexpr int PW = (TX + 2 * HX) / 2;   // pairs per row
    static constexpr int kFar = 15;                // a member beyond H
    static constexpr int pair_dist(int p, int y) {
        const int a = block_dist(2 * p - HX, TX), b = block_dist(2 * p + 1 - HX, TX);
        return (a < b ? a : b) + block_dist(y - H, TY);
    }
    static constexpr int count() {
        int n = 0;
        for (int y = 0; y < R; ++y)
            for (int p = 0; p < PW; ++p) n += pair_dist(p, y) <= H ? 1 : 0;
        return n;
    }
    static constexpr int N = count();
    static constexpr int kThreads = (N + 63) & ~63;
    unsigned v[N] = {};     // pair | row << 8 | distance of the members << 16, << 20
    constexpr BlockSlots() {
        int n = 0;
        for (int d = 0; d <= H; ++d)
            for (int y = 0; y < R; ++y)
                for (int p = 0; p < PW; ++p) {
                    if (pair_dist(p, y) != d) continue;
                    const int a = block_dist(2 * p - HX, TX) + block_dist(y - H, TY);
                    const int b = block_dist(2 * p + 1 - HX, TX) + block_dist(y - H, TY);
                    v[n++] = unsigned(p) | unsigned(y) << 8 | unsigned(a > H ? kFar : a) << 16 |
                             unsigned(b > H ? kFar : b) << 20;
                }
    }
};
template <int H, int TY>
__constant__ constexpr BlockSlots<H, TY> kBlockSlots{};

template <bool L0, int NS, int EPI, bool PRO, bool RHS, int TY>
__global__ __launch_bounds__((BlockSlots<(EPI ? 1 : 0) + 2 * NS, TY>::kThreads)) void k_block2d(
    Batch<double> bt, const TileTask* __restrict__ tasks, int ntiles, double* partial) {
    typedef double D2 __attribute__((ext_vector_type(2)));
    constexpr int X = EPI ? 1 : 0, H = X + 2 * NS, TX = kTileX;
    using G = BlockSlots<H, TY>;
    constexpr int PW = G::PW, SY = 2 * PW, kTile = TX * TY / 2;     // slots of the tile
    __shared__ double s_phi[SY * G::R], s_mu[SY * G::R], s_p[SY * G::R], s_ps[SY * G::R];

    // XCD x takes a contiguous range of tasks (a bijection on [0, ntiles))
    const int bid = blockIdx.x;
    const int xcd = bid % 8, jj = bid / 8;
    const int q8 = ntiles / 8, rem = ntiles % 8;
    const int tile = xcd * q8 + (xcd < rem ? xcd : rem) + jj;
    const TileTask tk = tasks[tile];
    if (bt.active != nullptr && bt.active[tk.inst] == 0) return;
    const Level<double> L = make_view(bt.desc[tk.inst * kMaxLevels + bt.level], bt.cur);
    const Level<double> C = make_view(bt.desc[tk.inst * kMaxLevels + bt.level + 1], bt.cur_c);
    const int nx = L.nx, ny = L.ny;
    const int tid = threadIdx.x;
    const double psh = bt.pshift != nullptr ? bt.pshift[tk.inst * kResStride + 4] : 0.0;

    const unsigned sl = kBlockSlots<H, TY>.v[tid < G::N ? tid : 0];
    const int rp = int(sl & 255), ry = int(sl >> 8 & 255);
    const int gx = tk.bx * TX - G::HX + 2 * rp, gy = tk.by * TY - H + ry;
    // the extents are even: a pair is in the grid or not as a whole
    const bool in = tid < G::N && gx >= 0 && gx < nx && gy >= 0 && gy < ny;
    const int g = gy * nx + gx, c = (gy >> 1) * C.nx + (gx >> 1);
    const int w0 = ry * SY + rp, w1 = w0 + PW;      // the members' words
    const int da = in ? int(sl >> 16 & 15) : G::kFar, db = in ? int(sl >> 20 & 15) : G::kFar;

    D2 phi = {0, 0}, mu = {0, 0}, p = {0, 0}, ps = {0, 0}, psi = {0, 0}, f0 = {0, 0}, f1 = {0, 0},
       f2 = {0, 0};
    if (in) {
        auto ld = [&](const double* a) { return gload(reinterpret_cast<const D2*>(a), g >> 1); };
        phi = ld(L.phi);
        mu = ld(L.mu);
        p = ld(L.p) - psh;
        ps = ld(L.pstar);
        psi = ld(L.psi);
        f1 = ld(RHS ? L.fr1 : L.f1);
        if (!L0) {
            f0 = ld(RHS ? L.fr0 : L.f0);
            f2 = ld(RHS ? L.fr2 : L.f2);
        }
        if (PRO) {
            phi += gload(C.phi, c) - gload(C.ub0, c);
            mu += gload(C.mu, c) - gload(C.ub1, c);
            p += gload(C.p, c) - gload(C.ub2, c);
        }
        if (L0) f0 = psi;
        s_phi[w0] = phi.x, s_phi[w1] = phi.y;
        s_mu[w0] = mu.x, s_mu[w1] = mu.y;
        s_p[w0] = p.x, s_p[w1] = p.y;
        s_ps[w0] = ps.x, s_ps[w1] = ps.y;
    }
    __syncthreads();

    const double lam = L.lam, kap = L.kap, gam = L.gamma;
    const double inv_lam = 1.0 / lam;
    const bool hy0 = gy > 0, hy1 = gy < ny - 1;
    // fn(word) for the interior faces of member e in the order x - 1, x + 1, y - 1, y + 1
    auto faces = [&](int e, auto&& fn) {
        const int w = e ? w1 : w0, wl = w + (e ? -PW : PW - 1);
        if (gx + e > 0) fn(wl);
        if (gx + e < nx - 1) fn(wl + 1);
        if (hy0) fn(w - SY);
        if (hy1) fn(w + SY);
    };
    auto apply = [&](int e, double (&n)[3]) {
        const int w = e ? w1 : w0;
        const double phic = s_phi[w], muc = s_mu[w], pc = s_p[w], ps_e = e ? ps.y : ps.x;
        CellDiffs d;
        faces(e, [&](int wn) {
            d.face(gam, ps_e, s_ps[wn], s_mu[wn] - muc, s_p[wn] - pc, s_phi[wn] - phic);
        });
        cell_apply(d, lam, kap, gam, phic, muc, e ? psi.y : psi.x, n);
    };

    if (RHS) {
        double n[3];
        if (da <= H - 1) {
            apply(0, n);
            f0.x += n[0], f1.x += n[1], f2.x += n[2];
        }
        if (db <= H - 1) {
            apply(1, n);
            f0.y += n[0], f1.y += n[1], f2.y += n[2];
        }
        if (tid < kTile && in) {
            gstore(reinterpret_cast<D2*>(L.f0), g >> 1, f0);
            gstore(reinterpret_cast<D2*>(L.f1), g >> 1, f1);
            gstore(reinterpret_cast<D2*>(L.f2), g >> 1, f2);
        }
        // the first phase overwrites what other waves still read here
        __syncthreads();
    }

    const int nfy = int(hy0) + int(hy1);
#pragma unroll
    for (int ph = 0; ph < 2 * NS; ++ph) {
        const int e = (gy & 1) ^ (ph & 1);          // the member of the phase's color
        if ((e ? db : da) <= X + 2 * NS - 1 - ph) {
            const int w = e ? w1 : w0;
            const double ps_e = e ? ps.y : ps.x;
            CellSums q;
            faces(e, [&](int wn) { q.face(gam, ps_e, s_ps[wn], s_mu[wn], s_p[wn], s_phi[wn]); });
            const int nf = nfy + (gx + e > 0 ? 1 : 0) + (gx + e < nx - 1 ? 1 : 0);
            double phin, mun, pn;
            cell_update(q, nf, lam, inv_lam, kap, gam, s_phi[w], e ? psi.y : psi.x, e ? f0.y : f0.x,
                        e ? f1.y : f1.x, e ? f2.y : f2.x, phin, mun, pn);
            s_phi[w] = phin;
            s_mu[w] = mun;
            s_p[w] = pn;
        }
        __syncthreads();
    }

    // the tile: whole waves
    __shared__ double red[4][EPI == 2 ? TY / 2 : 1];
    if (tid < kTile) {
        const D2 uphi = {s_phi[w0], s_phi[w1]}, umu = {s_mu[w0], s_mu[w1]}, up = {s_p[w0], s_p[w1]};
        if (in) {
            gstore(reinterpret_cast<D2*>(L.phi_alt), g >> 1, uphi);
            gstore(reinterpret_cast<D2*>(L.mu_alt), g >> 1, umu);
            gstore(reinterpret_cast<D2*>(L.p_alt), g >> 1, up);
        }
        if constexpr (EPI != 0) {
            double ra[3] = {0, 0, 0}, rb[3] = {0, 0, 0};
            if (in) {
                apply(0, ra);
                apply(1, rb);
                ra[0] = f0.x - ra[0], ra[1] = f1.x - ra[1], ra[2] = f2.x - ra[2];
                rb[0] = f0.y - rb[0], rb[1] = f1.y - rb[1], rb[2] = f2.y - rb[2];
            }
            if constexpr (EPI == 1) {
                // the two rows of a coarse cell (lane ^ 32), two fields per exchange:
                // lanes 0-31 then hold r0, r2, mu and lanes 32-63 r1, phi, p of the cell
                const double q0 = swap_sum(ra[0] + rb[0], ra[1] + rb[1], true) * 0.25;
                const double q1 = swap_sum(ra[2] + rb[2], in ? uphi.x + uphi.y : 0.0, true) * 0.25;
                const double q2 =
                    swap_sum(in ? umu.x + umu.y : 0.0, in ? up.x + up.y : 0.0, true) * 0.25;
                const bool lo = (tid & 32) == 0;
                if (in) {
                    if (lo) gstore(C.fr0, c, q0);
                    if (!lo) gstore(C.fr1, c, q0);
                    if (lo) gstore(C.fr2, c, q1);
                    if (!lo) gstore(C.phi, c, q1);
                    if (!lo) gstore(C.ub0, c, q1);
                    if (lo) gstore(C.mu, c, q2);
                    if (lo) gstore(C.ub1, c, q2);
                    if (!lo) gstore(C.p, c, q2);
                    if (!lo) gstore(C.ub2, c, q2);
                }
            } else {
                double v[4] = {__builtin_fma(rb[0], rb[0], ra[0] * ra[0]),
                               __builtin_fma(rb[1], rb[1], ra[1] * ra[1]),
                               __builtin_fma(rb[2], rb[2], ra[2] * ra[2]), in ? up.x + up.y : 0.0};
                for (int off = 32; off > 0; off >>= 1)
                    for (int k = 0; k < 4; ++k) v[k] += __shfl_xor(v[k], off, 64);
                if ((tid & 63) == 0)
                    for (int k = 0; k < 4; ++k) red[k][tid >> 6] = v[k];
            }
        }
    }
    if constexpr (EPI == 2) {
        // one partial per 64 x 4 cells, whatever the tile's height (as k_tile2d)
        __syncthreads();
        const int r4 = tid >> 2, k = tid & 3;
        if (r4 < TY / 4 && (tk.by * (TY / 4) + r4) * 4 < ny) {
            const int tx = (nx + TX - 1) / TX;
            gstore(partial, (tk.part + r4 * tx) * kNormStride + k, red[k][2 * r4] + red[k][2 * r4 + 1]);
        }
    }
}

}  // namespace
}  // namespace chhs
