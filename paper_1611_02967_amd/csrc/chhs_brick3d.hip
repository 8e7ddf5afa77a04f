// Smoothing of small 3D levels in bricks, batched over instances: FP64, or (T =
// float) the correction form.
//
// One workgroup owns a brick of 8 x 4 x 4 cells of one instance (a BrickTask)
// and stages it in LDS with the cells around it that its result depends on.  It
// runs NS red-black smoothing steps (the update of cell_update, as the per-color
// launches): phase q of the 2 NS phases updates every cell within X + 2 NS - 1 -
// q faces of the brick, so after the last phase the brick (and with X = 1 the
// cells that share a face with it) hold what per-color launches produce, bit for
// bit: cells around the brick are recomputed by the neighbouring bricks with
// identical arithmetic.  Out of place: u is read from one copy and the brick
// written to the other, so no brick loads what another has overwritten.
//
// Fused around the steps, each otherwise a launch of its own:
//   PRO    u += P(u_c - ub_c), piecewise constant, as u loads
//   RHS    first launch on a coarse level: its right-hand side f = fr + N(u)
//          on every cell a phase may update, the brick's cells written back
//   EPI 1  the residual of the brick restricted into the next coarser level
//          (k_restrict_residual's sums): u_c = ub_c = R u, fr_c = R(f - N(u))
//   EPI 2  finest level: norm partials of the brick (R_phi^2, R_mu^2, R_p^2, p),
//          one per brick whatever NS, so an instance's sums do not depend on NS
//
// What bounds it: latency.  On these levels a launch of one color takes 3.6-4.4
// us whatever it does (launch, task and descriptor loads, seven dependent cell
// reads, one update), and a V-cycle had 8 of them plus restriction, right-hand
// side and prolongation on every level.  Here a level takes two to four launches
// with all loads issued at once and phases at LDS latency.  The recomputation
// around small bricks costs little while the level does not fill the device, and
// 8 x 4 x 4 gives the most workgroups whose slots still fit one per thread.
// Measured, per-color launches / bricks: two steps of 32^3 1565 / 949 us, of 48 x
// 32 x 64 2100 / 1300, of 128^3 (its three coarse levels) 7670 / 7035.
//
// A slot is a pair of x-adjacent cells (x even) within H faces of the brick;
// every slot has its own thread.  Slots are ordered by their distance from the
// brick, so the waves of the outer ones drop out of the later phases whole, and
// the first 64 slots, one wave, are the brick.  In LDS a row's even columns
// precede its odd ones: the pairs of a row update the same member in a phase and
// touch consecutive words.
#include "chhs_cell.hpp"

#include <type_traits>

namespace chhs {
namespace {

constexpr int TX = kBrickX, TY = kBrickY, TZ = kBrickZ;
template <typename T>
using V2 = T __attribute__((ext_vector_type(2)));

constexpr int dist1(int v, int n) { return v < 0 ? -v : (v >= n ? v - n + 1 : 0); }

// Slots within H faces of the brick: cell offsets from the brick's first cell
// and distances of the two members (kFar: beyond H).
constexpr int kFar = 15;
template <int H>
struct Slots {
    static constexpr int HX = (H + 1) & ~1;        // x halo padded to keep pairs aligned
    static constexpr int R = TY + 2 * H, D = TZ + 2 * H;
    static constexpr int PW = (TX + 2 * HX) / 2;   // pairs per row
    static constexpr int W = 2 * PW * R * D;       // words of a field
    static constexpr int pair_dist(int p, int y, int z) {
        const int x = 2 * p - HX;
        const int a = dist1(x, TX), b = dist1(x + 1, TX);
        return (a < b ? a : b) + dist1(y - H, TY) + dist1(z - H, TZ);
    }
    static constexpr int count() {
        int n = 0;
        for (int z = 0; z < D; ++z)
            for (int y = 0; y < R; ++y)
                for (int p = 0; p < PW; ++p) n += pair_dist(p, y, z) <= H ? 1 : 0;
        return n;
    }
    static constexpr int N = count();
    unsigned v[N] = {};     // pair | row << 4 | plane << 8 | distance of the members << 12, << 16
    constexpr Slots() {
        int n = 0;
        for (int d = 0; d <= H; ++d)
            for (int z = 0; z < D; ++z)
                for (int y = 0; y < R; ++y)
                    for (int p = 0; p < PW; ++p) {
                        if (pair_dist(p, y, z) != d) continue;
                        const int yz = dist1(y - H, TY) + dist1(z - H, TZ);
                        const int a = dist1(2 * p - HX, TX) + yz, b = dist1(2 * p + 1 - HX, TX) + yz;
                        v[n++] = unsigned(p) | unsigned(y) << 4 | unsigned(z) << 8 |
                                 unsigned(a > H ? kFar : a) << 12 | unsigned(b > H ? kFar : b) << 16;
                    }
    }
};
template <int H>
__constant__ constexpr Slots<H> kSlots{};

template <typename T, bool L0, int NS, int EPI, bool PRO, bool RHS>
__global__ __launch_bounds__((Slots<(EPI ? 1 : 0) + 2 * NS>::N + 63) & ~63) void k_brick3d(
    Batch<T> bt, const BrickTask* __restrict__ tasks, int ntasks, double* partial) {
    constexpr bool CORR = std::is_same<T, float>::value;
    using D2 = V2<T>;
    constexpr int X = EPI ? 1 : 0, H = X + 2 * NS;
    using G = Slots<H>;
    constexpr int PW = G::PW, SY = 2 * PW, SZ = 2 * PW * G::R;
    static_assert(PW <= 16 && G::R <= 16 && G::D <= 16, "slot fields");
    __shared__ T s_phi[G::W], s_mu[G::W], s_p[G::W], s_ps[G::W];

    // XCD x takes a contiguous range of tasks (a bijection on [0, ntasks)):
    // neighbouring bricks share their halo through one L2
    const int bid = blockIdx.x;
    const int xcd = bid % 8, jj = bid / 8;
    const int q8 = ntasks / 8, rem = ntasks % 8;
    const int task = xcd * q8 + (xcd < rem ? xcd : rem) + jj;
    const BrickTask tk = tasks[task];
    if (bt.active != nullptr && bt.active[tk.inst] == 0) return;
    const Level<T> L = make_view(bt.desc[tk.inst * kMaxLevels + bt.level], bt.cur);
    const Level<T> C = make_view(bt.desc[tk.inst * kMaxLevels + bt.level + 1], bt.cur_c);
    const int nx = L.nx, ny = L.ny, nz = L.nz;
    const int tid = threadIdx.x;
    const double psh = !CORR && bt.pshift != nullptr ? bt.pshift[tk.inst * kResStride + 4] : 0.0;

    const unsigned sl = kSlots<H>.v[tid < G::N ? tid : 0];
    const int rp = int(sl & 15), ry = int(sl >> 4 & 15), rz = int(sl >> 8 & 15);
    const int gx = tk.bx * TX - G::HX + 2 * rp, gy = tk.by * TY - H + ry, gz = tk.bz * TZ - H + rz;
    // extents are even: a pair is in the grid or not as a whole
    const bool in = tid < G::N && gx >= 0 && gx < nx && gy >= 0 && gy < ny && gz >= 0 && gz < nz;
    const int g = (gz * ny + gy) * nx + gx;
    const int w0 = (rz * G::R + ry) * SY + rp, w1 = w0 + PW;     // the members' words
    // per color: 1 where the member of that color is the right one
    const int e0 = (gy ^ gz) & 1;
    const int da = in ? int(sl >> 12 & 15) : kFar, db = in ? int(sl >> 16 & 15) : kFar;

    D2 phi = {0, 0}, mu = {0, 0}, p = {0, 0}, ps = {0, 0}, psi = {0, 0}, f0 = {0, 0}, f1 = {0, 0},
       f2 = {0, 0}, bs = {0, 0};
    if (in) {
        auto ld = [&](const T* a) { return gload(reinterpret_cast<const D2*>(a), g >> 1); };
        phi = ld(L.phi);
        mu = ld(L.mu);
        p = ld(L.p);
        ps = ld(L.pstar);
        psi = ld(L.psi);
        f1 = ld(RHS ? L.fr1 : L.f1);
        if (!L0) {
            f0 = ld(RHS ? L.fr0 : L.f0);
            f2 = ld(RHS ? L.fr2 : L.f2);
        }
        if (CORR) bs = ld(L.b);
        if (PRO) {
            const int c = ((gz >> 1) * C.ny + (gy >> 1)) * C.nx + (gx >> 1);
            phi += gload(C.phi, c) - gload(C.ub0, c);
            mu += gload(C.mu, c) - gload(C.ub1, c);
            p += gload(C.p, c) - gload(C.ub2, c);
        }
        if (L0) f0 = psi;
        if (!CORR) p -= T(psh);
        s_phi[w0] = phi.x, s_phi[w1] = phi.y;
        s_mu[w0] = mu.x, s_mu[w1] = mu.y;
        s_p[w0] = p.x, s_p[w1] = p.y;
        s_ps[w0] = ps.x, s_ps[w1] = ps.y;
    }
    __syncthreads();

    const T lam = L.lam, kap = L.kap, gam = L.gamma;
    const T inv_lam = T(1) / lam;
    const bool hy0 = gy > 0, hy1 = gy < ny - 1, hz0 = gz > 0, hz1 = gz < nz - 1;
    // fn(word) for the interior faces of member e in the order x - 1, x + 1,
    // y - 1, y + 1, z - 1, z + 1
    auto faces = [&](int e, auto&& fn) {
        const int w = e ? w1 : w0, wl = w + (e ? -PW : PW - 1);
        if (gx + e > 0) fn(wl);
        if (gx + e < nx - 1) fn(wl + 1);
        if (hy0) fn(w - SY);
        if (hy1) fn(w + SY);
        if (hz0) fn(w - SZ);
        if (hz1) fn(w + SZ);
    };
    auto apply = [&](int e, T (&n)[3]) {
        const int w = e ? w1 : w0;
        const T phic = s_phi[w], muc = s_mu[w], pc = s_p[w];
        const T ps_e = e ? ps.y : ps.x, psi_e = e ? psi.y : psi.x;
        Diffs<T> d;
        faces(e, [&](int wn) {
            d.face(gam, ps_e, s_ps[wn], s_mu[wn] - muc, s_p[wn] - pc, s_phi[wn] - phic);
        });
        if constexpr (CORR)
            cell_apply(d, lam, kap, gam, phic, muc, psi_e, e ? bs.y : bs.x, n);
        else
            cell_apply(d, lam, kap, gam, phic, muc, psi_e, n);
    };

    if (RHS) {
        T n[3];
        if (da <= H - 1) {
            apply(0, n);
            f0.x += n[0], f1.x += n[1], f2.x += n[2];
        }
        if (db <= H - 1) {
            apply(1, n);
            f0.y += n[0], f1.y += n[1], f2.y += n[2];
        }
        if (tid < 64 && in) {
            gstore(reinterpret_cast<D2*>(L.f0), g >> 1, f0);
            gstore(reinterpret_cast<D2*>(L.f1), g >> 1, f1);
            gstore(reinterpret_cast<D2*>(L.f2), g >> 1, f2);
        }
        // the first phase overwrites what other waves still read here
        __syncthreads();
    }

    const int nfyz = int(hy0) + int(hy1) + int(hz0) + int(hz1);
#pragma unroll
    for (int ph = 0; ph < 2 * NS; ++ph) {
        const int e = e0 ^ (ph & 1);
        if ((e ? db : da) <= X + 2 * NS - 1 - ph) {
            const int w = e ? w1 : w0;
            const T ps_e = e ? ps.y : ps.x, psi_e = e ? psi.y : psi.x;
            const T f0_e = e ? f0.y : f0.x, f1_e = e ? f1.y : f1.x, f2_e = e ? f2.y : f2.x;
            Sums<T> q;
            faces(e, [&](int wn) { q.face(gam, ps_e, s_ps[wn], s_mu[wn], s_p[wn], s_phi[wn]); });
            const int nf = nfyz + (gx + e > 0 ? 1 : 0) + (gx + e < nx - 1 ? 1 : 0);
            T phin, mun, pn;
            if constexpr (CORR)
                cell_update(q, nf, lam, inv_lam, kap, gam, s_phi[w], psi_e, e ? bs.y : bs.x, f0_e,
                            f1_e, f2_e, phin, mun, pn);
            else
                cell_update(q, nf, lam, inv_lam, kap, gam, s_phi[w], psi_e, f0_e, f1_e, f2_e, phin,
                            mun, pn);
            s_phi[w] = phin;
            s_mu[w] = mun;
            s_p[w] = pn;
        }
        __syncthreads();
    }

    // the brick: the first wave, lane = z 16 + y 4 + pair
    if (tid >= 64) return;
    const D2 uphi = {s_phi[w0], s_phi[w1]}, umu = {s_mu[w0], s_mu[w1]}, up = {s_p[w0], s_p[w1]};
    if (in) {
        gstore(reinterpret_cast<D2*>(L.phi_alt), g >> 1, uphi);
        gstore(reinterpret_cast<D2*>(L.mu_alt), g >> 1, umu);
        gstore(reinterpret_cast<D2*>(L.p_alt), g >> 1, up);
    }
    if (EPI == 0) return;
    T ra[3] = {0, 0, 0}, rb[3] = {0, 0, 0};
    if (in) {
        apply(0, ra);
        apply(1, rb);
        ra[0] = f0.x - ra[0], ra[1] = f1.x - ra[1], ra[2] = f2.x - ra[2];
        rb[0] = f0.y - rb[0], rb[1] = f1.y - rb[1], rb[2] = f2.y - rb[2];
    }
    if (EPI == 1) {
        // children of a coarse cell: the pair, lanes ^ 4 (y) and ^ 16 (z)
        T v[7] = {ra[0] + rb[0], ra[1] + rb[1], ra[2] + rb[2], uphi.x + uphi.y,
                  umu.x + umu.y, up.x + up.y,   bs.x + bs.y};
#pragma unroll
        for (int k = 0; k < (CORR ? 7 : 6); ++k) {
            v[k] += __shfl_xor(v[k], 4, 64);
            v[k] += __shfl_xor(v[k], 16, 64);
            v[k] *= T(0.125);
        }
        if (!in) return;
        const int c = ((gz >> 1) * C.ny + (gy >> 1)) * C.nx + (gx >> 1);
        const int sub = (tid >> 2 & 1) | (tid >> 3 & 2);     // the lane's y and z within the cell
        if (sub == 0) {
            gstore(C.fr0, c, v[0]);
            gstore(C.fr1, c, v[1]);
            gstore(C.fr2, c, v[2]);
        }
        if (sub == 1) gstore(C.phi, c, v[3]), gstore(C.ub0, c, v[3]);
        if (sub == 2) gstore(C.mu, c, v[4]), gstore(C.ub1, c, v[4]);
        if (sub == 3) gstore(C.p, c, v[5]), gstore(C.ub2, c, v[5]);
        if (CORR && sub == 1) gstore(C.b, c, v[6]);
    }
    if constexpr (EPI == 2) {
        double v[4] = {__builtin_fma(rb[0], rb[0], ra[0] * ra[0]),
                       __builtin_fma(rb[1], rb[1], ra[1] * ra[1]),
                       __builtin_fma(rb[2], rb[2], ra[2] * ra[2]), in ? up.x + up.y : 0.0};
        for (int off = 32; off > 0; off >>= 1)
            for (int k = 0; k < 4; ++k) v[k] += __shfl_xor(v[k], off, 64);
        if (tid < 4) gstore(partial, task * kNormStride + tid,
                            tid == 0 ? v[0] : (tid == 1 ? v[1] : (tid == 2 ? v[2] : v[3])));
    }
}

template <typename T, bool L0, int NS, int EPI, bool PRO, bool RHS>
void launch(const Batch<T>& b, const BrickTask* t, int nt, double* partial, hipStream_t st) {
    constexpr int threads = (Slots<(EPI ? 1 : 0) + 2 * NS>::N + 63) & ~63;
    hipLaunchKernelGGL((k_brick3d<T, L0, NS, EPI, PRO, RHS>), dim3(nt), dim3(threads), 0, st, b, t,
                       nt, partial);
}

template <typename T, bool L0, int NS>
void launch_ns(const Batch<T>& b, const BrickTask* t, int nt, int epi, bool pro, bool rhs,
               double* partial, hipStream_t st) {
    if constexpr (L0) {
        if (epi == 2) {
            if (pro)
                launch<T, L0, NS, 2, true, false>(b, t, nt, partial, st);
            else
                launch<T, L0, NS, 2, false, false>(b, t, nt, partial, st);
            return;
        }
    } else if (rhs) {
        if (epi == 1)
            launch<T, L0, NS, 1, false, true>(b, t, nt, partial, st);
        else
            launch<T, L0, NS, 0, false, true>(b, t, nt, partial, st);
        return;
    }
    if (epi == 1)
        launch<T, L0, NS, 1, false, false>(b, t, nt, partial, st);
    else if (pro)
        launch<T, L0, NS, 0, true, false>(b, t, nt, partial, st);
    else
        launch<T, L0, NS, 0, false, false>(b, t, nt, partial, st);
}

}  // namespace

template <typename T>
void launch_brick3d(const Batch<T>& b, const BrickTask* t, int nt, bool level0, int ns, int epi,
                    bool pro, bool rhs, double* partial, hipStream_t st) {
    if (nt == 0) return;
    if constexpr (std::is_same<T, double>::value)
        if (level0) {
            if (ns == 2)
                launch_ns<T, true, 2>(b, t, nt, epi, pro, rhs, partial, st);
            else
                launch_ns<T, true, 1>(b, t, nt, epi, pro, rhs, partial, st);
            return;
        }
    if (ns == 2)
        launch_ns<T, false, 2>(b, t, nt, epi, pro, rhs, partial, st);
    else
        launch_ns<T, false, 1>(b, t, nt, epi, pro, rhs, partial, st);
}
template void launch_brick3d(const Batch<double>&, const BrickTask*, int, bool, int, int, bool, bool,
                             double*, hipStream_t);
template void launch_brick3d(const Batch<float>&, const BrickTask*, int, bool, int, int, bool, bool,
                             double*, hipStream_t);

}  // namespace chhs
