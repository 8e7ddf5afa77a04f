// Coarse tail of the V-cycle in one workgroup, every pair of cells owned by a
// thread.
//
// One workgroup per instance runs every level from the instance's tail level
// down to the coarsest grid: smoothing, residual + restriction, FAS coarse
// right-hand side, the coarsest-grid smoothing steps, prolongation +
// correction.  Where the finest level itself is here (FP64), the cycle ends with
// the norm of its residual, and when that holds for every instance of the
// context one launch runs the cycles of a whole step up to the tolerance.
//
// What bounds it is latency: the V-cycle over these levels is a chain of about
// fifty dependent phases, each a few cells per lane.  So a phase is kept
// short.  Every pair of x-adjacent cells of every level has an owner thread
// for the whole launch, which keeps in registers what does not change between
// phases: the face coefficients, the eliminated diagonal, the right-hand
// side, phi^m and the pair's own iterate (the x neighbour inside the pair is a
// register too).  The face coefficients of all levels are formed once, by all
// levels' owners at the same time.  LDS holds what neighbours read: the
// iterate, as one (phi, mu, p) record per cell so that a neighbour costs one
// address, and a record of zeros that stands in for the neighbour beyond a
// boundary face.  The right-hand side of a level is formed in the same phase
// as its first red update, reading the restricted iterate (which no phase
// overwrites) instead of the iterate.  Levels of at most 64 pairs are packed
// into one wave, which orders its own phases without workgroup barriers while
// the other waves wait at the next one.
//
// Measured per V-cycle (MI355X), k_tail -> this kernel: from 32^2 FP64 53 -> 22
// us, from 16^2 FP64 37 -> 15, from 8^3 FP64 39 -> 16, from 32^2 FP32 47 -> 26.  A
// phase takes 0.22 us whether its level fills half a wave or eight waves: the
// dependent chain of one cell update (LDS read, four faces, reciprocal), not
// the number of cells.
#include "chhs_cell.hpp"

namespace chhs {
namespace {

// What the owner of a pair keeps; arrays [2] are indexed by color (0 the red
// member, 1 the black one) so that a phase uses compile-time indices.  Faces
// of a member: `mid` between the two members, then K outer ones: the other x
// face, y - 1, y + 1 (, z - 1, z + 1).
//
// FP64: the nonlinear term is kept as a polynomial of phi,
//   chi(phi, psi) = psi^3 / 4 + phi (d0 + phi (c1 / 2 + phi / 4)),
//   d0 = psi^2 / 4,  c1 = psi / 2,
// so that chi' = d0 + phi (c1 + 3/4 phi), chi - chi' phi = psi^3 / 4 - phi^2 (c1 +
// phi) / 2; the constant goes into the right-hand side f[1].  The first-order
// step's chi = phi^3 is d0 = c1 = 0 with the phi terms times k3 = 4 (k3 = 1
// otherwise).  f[2] is kept divided by lam, sn is sum a / nF.
// FP32 correction form: d0 holds b, c1 holds psi, sn holds sum a, and every
// expression and every sum is that of cell_solve / cell_operator in the same
// order, with the multiply-adds that k_tail fuses written out: the rounding of
// the corrections shows in the refined pressure (at 1e-8 of it, where its error
// is 1e-5), and so it is the same in both tail kernels.
template <int DIM, typename T>
struct Pair {
    static constexpr int K = 2 * DIM - 1;
    T a[2][K], amid;            // A_h phi_* on the faces (0 on boundary faces)
    T ared[2], sn[2];           // reduced off-diagonal, sum of a over the faces / their number
    T inv_nf[2];
    T d0[2], c1[2], f[2][3], u[2][3];
    int cell0, nb[2][K];       // the left cell; LDS words of the outer neighbours' records
    unsigned fl;                // TailOwner::fl
    __device__ __forceinline__ bool alive(int c) const { return (fl >> c) & 1u; }
    __device__ __forceinline__ bool has(int c, int k) const { return (fl >> (2 + c * K + k)) & 1u; }
    __device__ __forceinline__ int cell(int c) const { return cell0 + (c ^ int((fl >> kOwnRed) & 1u)); }
    __device__ __forceinline__ int w(int c) const { return 3 * cell(c); }     // its record
    __device__ __forceinline__ bool kap_first() const { return (fl >> kOwnKapFirst) & 1u; }
    __device__ __forceinline__ bool mid() const { return (fl >> kOwnMid) & 1u; }
    // member c is the right one of the pair
    __device__ __forceinline__ bool right(int c) const { return ((fl >> kOwnRed) & 1u) != unsigned(c); }
    __device__ __forceinline__ int nf(int c) const {
        return __popc(fl & ((1u << kOwnMid) | (((1u << K) - 1u) << (2 + c * K))));
    }
};

// Scalars of a level.
template <typename T>
struct Coef {
    T lam, inv_lam, kap, gam, k3;
};

// Lane exchange within groups of four lanes (quad permutation, VALU only).
template <int CTRL>
__device__ __forceinline__ double quad(double v) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_mov_dpp(int(unsigned(x)), CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_mov_dpp(int(unsigned(x >> 32)), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}
template <int CTRL>
__device__ __forceinline__ float quad(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf,
                                                              0xf, true));
}
constexpr int kLane1 = 0xB1;    // lane ^ 1: quad_perm [1, 0, 3, 2]
constexpr int kLane2 = 0x4E;    // lane ^ 2: quad_perm [2, 3, 0, 1]

// The same value, opaque to the compiler: what is computed from it stays where
// it is written.  A phase forms M = 1 + gamma a^2 anew from the register that
// holds a; kept across the phases, those products would not fit the registers
// of the workgroup.
template <typename T>
__device__ __forceinline__ T opaque(T v) {
    asm volatile("" : "+v"(v));
    return v;
}

// The collective cell update of member C (cell_solve with the coefficients
// held by the owner).  U: the level's records in LDS.
template <int DIM, typename T, bool CORR, int C>
__device__ __forceinline__ void relax(Pair<DIM, T>& P, T* U, const Coef<T>& q) {
    constexpr int K = Pair<DIM, T>::K;
    const T gam = opaque(q.gam);
    T xphi[K], xmu[K], xp[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const T* r = U + P.nb[C][k];
        xphi[k] = r[0];
        xmu[k] = r[1];
        xp[k] = r[2];
    }
    T phi, mu, p;
    if constexpr (CORR) {
#pragma clang fp contract(off)
        // faces in the order x - 1, x + 1, y - 1, y + 1 (, z - 1, z + 1)
        const bool r = P.right(C);
        T smmu = 0, sphi = 0, sp = 0, sap = 0, samu = 0;
        auto add = [&](T a, T nphi, T nmu, T np) {
#pragma clang fp contract(off)
            smmu = fma_of(fma_of(a, gam * a, T(1)), nmu, smmu);
            sphi = sphi + nphi;
            sp = sp + np;
            sap = fma_of(a, np, sap);
            samu = fma_of(a, nmu, samu);
        };
        const T ophi = P.u[1 - C][0], omu = P.u[1 - C][1], op = P.u[1 - C][2];
        add(r ? P.amid : P.a[C][0], r ? ophi : xphi[0], r ? omu : xmu[0], r ? op : xp[0]);
        add(r ? P.a[C][0] : P.amid, r ? xphi[0] : ophi, r ? xmu[0] : omu, r ? xp[0] : op);
#pragma unroll
        for (int k = 1; k < K; ++k) add(P.a[C][k], xphi[k], xmu[k], xp[k]);
        const T fnf = T(P.nf(C)), lam = q.lam, kap = q.kap;
        const T x = P.u[C][0], psi = P.c1[C], b = P.d0[C], y = b + x;
        const T dchi = T(0.25) * fma_of(psi, psi, fma_of(y, T(3) * y, psi * (y + y)));
        const T b1 = fma_of(lam, sap, fma_of(lam, smmu, P.f[C][0]));
        const T b2 = fma_of(-kap, sphi, fma_of(-x, dchi, fma_of(T(0.25) * x, chi_sum(x, psi, b), P.f[C][1])));
        const T b3 = fma_of(-(lam * gam), samu, fma_of(-lam, sp, P.f[C][2]));
        const T b1r = fma_of(P.sn[C] * P.inv_nf[C], b3, b1);
        const T bb = P.kap_first() ? dchi + kap * fnf : fma_of(kap, fnf, dchi);
        const T inv_det = recip_ge1(fma_of(P.ared[C], bb, T(1)));
        mu = fma_of(bb, b1r, b2) * inv_det;
        phi = fma_of(-P.ared[C], b2, b1r) * inv_det;
        p = -(P.inv_nf[C] * fma_of(q.inv_lam, b3, (gam * P.sn[C]) * mu));
    } else {
        const T x = P.u[C][0];
        const T bb = q.kap * T(P.nf(C)) + P.d0[C] + x * (P.c1[C] + T(0.75) * q.k3 * x);
        const T inv_det = recip_ge1(T(1) + P.ared[C] * bb);
        // a missing partner's record is zero and its face coefficient too
        const T pmu = P.u[1 - C][1], pp = P.u[1 - C][2];
        T sphi = P.u[1 - C][0], sp = pp;
        T smmu = (T(1) + gam * P.amid * P.amid) * pmu;
        T sap = P.amid * pp, samu = P.amid * pmu;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const T a = P.a[C][k];
            smmu += (T(1) + gam * a * a) * xmu[k];
            sphi += xphi[k];
            sp += xp[k];
            sap += a * xp[k];
            samu += a * xmu[k];
        }
        const T b2 = P.f[C][1] - q.kap * sphi - (T(0.5) * x * x) * (P.c1[C] + q.k3 * x);
        const T b3 = P.f[C][2] - sp - gam * samu;                       // / lam
        const T b1r = P.f[C][0] + q.lam * (smmu + sap + P.sn[C] * b3);
        mu = (b2 + bb * b1r) * inv_det;
        phi = (b1r - P.ared[C] * b2) * inv_det;
        p = -(b3 * P.inv_nf[C] + gam * P.sn[C] * mu);
    }
    if (P.alive(C)) {
        P.u[C][0] = phi;
        P.u[C][1] = mu;
        P.u[C][2] = p;
        T* r = U + P.w(C);
        r[0] = phi;
        r[1] = mu;
        r[2] = p;
    }
}

// N(u) of member C (cell_operator; FP64: without chi's constant and the third
// row divided by lam), the neighbours read from the records V.
template <int DIM, typename T, bool CORR, int C>
__device__ __forceinline__ void apply_n(const Pair<DIM, T>& P, const T* V, const Coef<T>& q,
                                        T (&n)[3]) {
    constexpr int K = Pair<DIM, T>::K;
    const T gam = opaque(q.gam);
    const unsigned fl = opaque(P.fl);       // the words below are formed anew, not kept
    const T x = P.u[C][0], muc = P.u[C][1], pc = P.u[C][2];
    T smm = 0, sap = 0, sphi = 0, sp = 0, samu = 0;
    auto add = [&](T a, T xphi, T xmu, T xp) {
        const T dmu = xmu - muc, dp = xp - pc, dphi = xphi - x;
        smm = fma_of(fma_of(a, gam * a, T(1)), dmu, smm);
        sap = fma_of(a, dp, sap);
        sphi = sphi + dphi;
        sp = sp + dp;
        samu = fma_of(a, dmu, samu);
    };
    // across a boundary face the cell's own values: zero differences
    const T ophi = P.mid() ? P.u[1 - C][0] : x, omu = P.mid() ? P.u[1 - C][1] : muc;
    const T op = P.mid() ? P.u[1 - C][2] : pc;
    if constexpr (CORR) {
        const bool r = P.right(C);
        const T* v = V + (((fl >> (2 + C * K)) & 1u) ? P.nb[C][0] : P.w(C));
        const T xphi = v[0], xmu = v[1], xp = v[2];
        add(r ? P.amid : P.a[C][0], r ? ophi : xphi, r ? omu : xmu, r ? op : xp);
        add(r ? P.a[C][0] : P.amid, r ? xphi : ophi, r ? xmu : omu, r ? xp : op);
    } else {
        add(P.amid, ophi, omu, op);
    }
#pragma unroll
    for (int k = CORR ? 1 : 0; k < K; ++k) {
        const T* r = V + (((fl >> (2 + C * K + k)) & 1u) ? P.nb[C][k] : P.w(C));
        add(P.a[C][k], r[0], r[1], r[2]);
    }
    if constexpr (CORR) {
#pragma clang fp contract(off)
        n[0] = fma_of(-q.lam, sap, fma_of(-q.lam, smm, x));
        n[1] = fma_of(q.kap, sphi, fma_of(T(-0.25) * x, chi_sum(x, P.c1[C], P.d0[C]), muc));
        n[2] = fma_of(q.lam, sp, (q.lam * gam) * samu);
    } else {
        n[0] = x - q.lam * (smm + sap);
        n[1] = muc + q.kap * sphi - x * (P.d0[C] + x * (T(0.5) * P.c1[C] + T(0.25) * q.k3 * x));
        n[2] = sp + gam * samu;
    }
}

// An instance's results and flags, also into the host's mirror (fresh: new
// results o, else those it has).
__device__ __forceinline__ void write_results(const TailSolve& q, int inst, bool fresh,
                                              const double* o, int act, int cycles) {
    double* r = q.out.res + inst * kResStride;
    double* m = q.out.mirror + inst * kResStride;
    int* flags = reinterpret_cast<int*>(q.out.mirror + size_t(gridDim.x) * kResStride);
    for (int k = 0; k < 6; ++k) {
        if (fresh) r[k] = o[k];
        m[k] = fresh ? o[k] : r[k];
    }
    if (fresh) {
        q.out.act[inst] = act;
        q.out.cycles[inst] = cycles;
    }
    flags[inst] = fresh ? act : 0;
    flags[gridDim.x + inst] = fresh ? cycles : q.out.cycles[inst];
}

template <int DIM, typename T, bool CORR, int NT>
__global__ __launch_bounds__(NT) void k_tail_own(const TailDesc<T>* __restrict__ tails,
                                             const TailOwner* __restrict__ owners, int stride,
                                             const int* __restrict__ active, CycleShape shape,
                                             TailSolve solve) {
    extern __shared__ __align__(16) unsigned char own_lds[];
    __shared__ double sums[2][NT / 64][4];      // two, so that a slow wave may still read the last
    T* const base = reinterpret_cast<T*>(own_lds);
    constexpr int K = Pair<DIM, T>::K;
    const int inst = blockIdx.x, tid = threadIdx.x;
    // the pair's place and geometry come ready from a table, and the level data
    // in one descriptor, so that the staging loads are two dependent accesses
    // away from the launch
    const TailOwner own = owners[inst * stride + tid];
    const TailDesc<T>& G = tails[inst];
    if (active != nullptr && active[inst] == 0) {
        if (solve.cycles > 0 && tid == 0) write_results(solve, inst, false, nullptr, 0, 0);
        return;
    }
    if (G.levels == 0) return;          // the instance's tail is worked by k_tail
    // the mean of the initial p, taken out by a step's first cycle (the finest
    // level here; later cycles carry what they add to it, of the size of p)
    const int before = CORR ? 0 : solve.out.cycles[inst];     // cycles of the step so far
    const T mean = CORR ? T(0) : T(solve.out.res[inst * kResStride + 4]);
    const T psh = before == 0 && G.finest != 0 ? mean : T(0);
    const bool owner = (own.fl >> kOwnValid) & 1u;
    const int my = owner ? int((own.fl >> kOwnLevel) & 7u) : -1;       // level below the tail's top one
    const int last = G.levels - 1;
    const bool finest = G.finest != 0;
    Coef<T> cf;
    {
        // spacing 2^l h: lam and kap are those of the top level times 4^-l
        const T s = ldexp(T(1), my > 0 ? -2 * my : 0);
        cf.lam = G.lam * s;
        cf.kap = G.kap * s;
        cf.inv_lam = T(1) / cf.lam;
        cf.gam = G.gamma;
        cf.k3 = G.cubic ? T(4) : T(1);
    }
    const int nx = own.nx, n = own.n;
    T* const U = base + own.off;
    T* const UB = U + 3 * (n + 1);
    T* const FR = UB + 3 * n;
    T* const PS = FR + 3 * n;
    T* const B = PS + n;                // correction form
    const int e0 = (own.fl >> kOwnRed) & 1u;    // the red member
    const int par = own.par;

    Pair<DIM, T> P;
    P.fl = own.fl;
    P.cell0 = own.cell0;
    T ps[2] = {T(0), T(0)};
    if (owner) {
        // every global load of the pair, then the LDS stores: phi_* of every
        // level, the iterate of the top one
        T g[2][7], psi[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int e = P.alive(c) ? c ^ e0 : 0;
            ps[c] = gload(G.pstar, own.ps + e);
            psi[c] = gload(G.psi, own.psi + e);
            if (my == 0) {
                // below the finest level f holds the restricted residual, from
                // which f = fr + N(u) is formed after the staging
                const int cell = own.cell0 + e;
                for (int k = 0; k < 3; ++k) g[c][k] = gload(G.u[k], cell);
                for (int k = 0; k < 3; ++k) g[c][3 + k] = gload(G.f[k], cell);
                if (CORR) g[c][6] = gload(G.b, cell);
            }
        }
        if (own.cell0 == 0)
            for (int k = 0; k < 3; ++k) U[3 * n + k] = T(0);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const bool live = P.alive(c);
            if (live) PS[P.cell(c)] = ps[c];
            for (int k = 0; k < 3; ++k) P.u[c][k] = P.f[c][k] = T(0);
            if (CORR) {
                P.c1[c] = psi[c];
                P.d0[c] = T(0);
            } else {
                P.c1[c] = G.cubic ? T(0) : T(0.5) * psi[c];
                P.d0[c] = G.cubic ? T(0) : T(0.25) * psi[c] * psi[c];
            }
            if (my == 0 && live) {
                P.u[c][0] = g[c][0];
                P.u[c][1] = g[c][1];
                P.u[c][2] = CORR ? g[c][2] : g[c][2] - psh;
                P.f[c][0] = g[c][3];
                P.f[c][1] = g[c][4];
                P.f[c][2] = CORR ? g[c][5] : g[c][5] * cf.inv_lam;
                if (!CORR && finest && !G.cubic)
                    P.f[c][1] += T(0.25) * psi[c] * psi[c] * psi[c];
                if (CORR) P.d0[c] = g[c][6];
                for (int k = 0; k < 3; ++k) U[P.w(c) + k] = P.u[c][k];
            }
        }
    }
    __syncthreads();
    if (owner) {
        // face coefficients of the pair
        P.amid = P.mid() ? T(0.5) * (ps[0] + ps[1]) : T(0);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int e = c ^ e0;
            const int cell = own.cell0 + e;
            // outer x face: of the left member x - 1, of the right one x + 1
            T sa = 0, sa2 = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int o = k == 0 ? (e == 0 ? -1 : 1)
                            : (k == 1 ? -nx : (k == 2 ? nx : (k == 3 ? -own.nxy : own.nxy)));
                const bool in_k = P.has(c, k);
                const int nbc = in_k ? cell + o : n;
                P.nb[c][k] = 3 * nbc;
                const T a = in_k ? T(0.5) * (ps[c] + PS[in_k ? nbc : 0]) : T(0);
                P.a[c][k] = a;
            }
            // in the order x - 1, x + 1, y - 1, y + 1 (, z - 1, z + 1)
            const bool r = P.right(c);
            const T axm = r ? P.amid : P.a[c][0], axp = r ? P.a[c][0] : P.amid;
            auto square = [&](T a) {
                sa = sa + a;
                sa2 = fma_of(a, a, sa2);
            };
            square(axm);
            square(axp);
#pragma unroll
            for (int k = 1; k < K; ++k) square(P.a[c][k]);
            const int nf = P.nf(c);
            P.inv_nf[c] = nf == 6 ? T(1) / T(6)
                        : (nf == 5 ? T(1) / T(5)
                        : (nf == 4 ? T(0.25) : (nf == 3 ? T(1) / T(3) : (nf == 2 ? T(0.5) : T(1)))));
            const T fnf = T(nf), inv_nf = P.inv_nf[c];
            P.sn[c] = CORR ? sa : sa * inv_nf;
            P.ared[c] = cf.lam * fma_of(cf.gam, fma_of(-(sa * sa), inv_nf, sa2), fnf);
        }
    }

    // Order of the phases.  A level of one wave orders its own phases (a wave's
    // LDS accesses are performed in the order issued); the other waves have
    // nothing to do until the next workgroup barrier.
    auto sync = [&](bool wave) {
        if (wave) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
    };
    const unsigned single = G.single, joined = G.joined;
    auto is = [](unsigned mask, int l) { return ((mask >> l) & 1u) != 0; };
    auto smooth = [&](int l, int steps) {
        const bool wave = is(single, l);
        for (int s = 0; s < steps; ++s) {
            if (my == l) relax<DIM, T, CORR, 0>(P, U, cf);
            sync(wave);
            if (my == l) relax<DIM, T, CORR, 1>(P, U, cf);
            sync(wave);
        }
    };
    const int nu1 = finest ? shape.nu1f : shape.nu1c, nu2 = finest ? shape.nu2f : shape.nu2c;

    if (!finest) {
        if (my == 0) {
            T n0[3], n1[3];
            apply_n<DIM, T, CORR, 0>(P, U, cf, n0);
            apply_n<DIM, T, CORR, 1>(P, U, cf, n1);
            for (int k = 0; k < 3; ++k) {
                P.f[0][k] += n0[k];
                P.f[1][k] += n1[k];
            }
        }
        // the first phase overwrites records that other waves still read here
        sync(is(single, 0));
    }

    for (int cycle = 1;; ++cycle) {
        // nothing derived from these is kept over the whole loop (registers)
        P.cell0 = opaque(P.cell0);
        P.fl = opaque(P.fl);
        cf.lam = opaque(cf.lam);
        cf.kap = opaque(cf.kap);
        for (int l = 0; l <= last; ++l) {
            if (l > 0 && my == l) {
                // the restricted iterate and f = fr + N(u); the neighbours' values
                // come from UB, which the first phase does not overwrite (the record
                // of a missing second member is not used)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const bool live = P.alive(c);
                    const int w = live ? P.w(c) : 0;
                    T v[7];
                    for (int k = 0; k < 3; ++k) v[k] = UB[w + k];
                    for (int k = 0; k < 3; ++k) v[3 + k] = FR[w + k];
                    if (CORR) v[6] = B[live ? P.cell(c) : 0];
                    for (int k = 0; k < 3; ++k) P.u[c][k] = live ? v[k] : T(0);
                    P.f[c][0] = live ? v[3] : T(0);
                    P.f[c][1] = live ? v[4] : T(0);
                    P.f[c][2] = live ? (CORR ? v[5] : v[5] * cf.inv_lam) : T(0);
                    if (CORR) P.d0[c] = live ? v[6] : T(0);
                }
                T n0[3], n1[3];
                apply_n<DIM, T, CORR, 0>(P, UB, cf, n0);
                apply_n<DIM, T, CORR, 1>(P, UB, cf, n1);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    P.f[0][k] += n0[k];
                    P.f[1][k] += n1[k];
                }
            }
            smooth(l, l == last ? shape.coarse : (l == 0 ? nu1 : shape.nu1c));
            if (l == last) break;
            if (my == l) {
                // residual of the pair, restricted by cell averaging with the other
                // pairs of the coarse cell (lanes of one group of 2 or 4)
                T n0[3], n1[3], v[7];
                apply_n<DIM, T, CORR, 0>(P, U, cf, n0);
                apply_n<DIM, T, CORR, 1>(P, U, cf, n1);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    v[k] = (P.f[0][k] - n0[k]) + (P.f[1][k] - n1[k]);
                    v[3 + k] = P.u[0][k] + P.u[1][k];
                }
                if (!CORR) v[2] *= cf.lam;
                v[6] = P.d0[0] + P.d0[1];           // b
                const T wgt = DIM == 3 ? T(0.125) : T(0.25);
#pragma unroll
                for (int k = 0; k < 7; ++k) {
                    if (!CORR && k == 6) continue;
                    v[k] += quad<kLane1>(v[k]);
                    if (DIM == 3) v[k] += quad<kLane2>(v[k]);
                    v[k] *= wgt;
                }
                const int cn = n >> DIM;
                T* const CU = U + own_words(n, CORR);
                T* const CUB = CU + 3 * (cn + 1);
                T* const CFR = CUB + 3 * cn;
                if ((own.fl >> kOwnFirst) & 1u) {
                    for (int k = 0; k < 3; ++k) {
                        CU[3 * par + k] = v[3 + k];
                        CUB[3 * par + k] = v[3 + k];
                        CFR[3 * par + k] = v[k];
                    }
                    if (CORR) CFR[4 * cn + par] = v[6];
                }
            }
            sync(is(joined, l));
        }

        for (int l = last - 1; l >= 0; --l) {
            // a coarser level of one wave other than this level's
            if (is(single, l + 1) && !is(joined, l)) __syncthreads();
            if (my == l) {
                const int cn = n >> DIM;
                const T* const CU = U + own_words(n, CORR);
                const T* const CUB = CU + 3 * (cn + 1);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if (shape.bilinear != 0) {
                        const int* g = &owners[inst * stride + tid].nx;     // nx, nx ny
                        const int fx = g[0], fxy = g[1];
                        int i, j, k;
                        decode<DIM>(P.cell(c), fx, fxy / fx, i, j, k);
                        for (int m = 0; m < 3; ++m)
                            P.u[c][m] += bilinear_corr<DIM, T, 3>(CU + m, CUB + m, fx >> 1,
                                                                  (fxy / fx) >> 1, (n / fxy) >> 1, i, j, k);
                    } else {
                        for (int m = 0; m < 3; ++m) P.u[c][m] += CU[3 * par + m] - CUB[3 * par + m];
                    }
                    for (int m = 0; m < 3; ++m) U[P.w(c) + m] = P.u[c][m];
                }
            }
            sync(is(single, l));
            smooth(l, l == 0 ? nu2 : shape.nu2c);
        }

        // The finest level is here (FP64): the norm of its residual.  Sums over
        // each wave of its owners, then over the waves, in a fixed order.
        if constexpr (CORR) {
            break;
        } else {
            if (!finest || solve.partial == nullptr) break;
            // The waves of its owners whole: the lanes without a pair of it add zero.
            if (tid < 64 * G.top_waves) {
                double v[4] = {0.0, 0.0, 0.0, 0.0};
                if (my == 0) {
                    T n[3];
                    apply_n<DIM, T, CORR, 0>(P, U, cf, n);
                    v[3] = P.u[0][2] + P.u[1][2];
                    auto add = [&](int c) {
                        for (int k = 0; k < 3; ++k) {
                            const T r = (k == 2 ? cf.lam : T(1)) * (P.f[c][k] - n[k]);
                            v[k] += r * r;
                        }
                    };
                    add(0);
                    __builtin_amdgcn_sched_barrier(0);      // one member at a time (registers)
                    apply_n<DIM, T, CORR, 1>(P, U, cf, n);
                    add(1);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
                    if ((tid & 63) == 0) sums[cycle & 1][tid >> 6][k] = v[k];
                }
            }
            __syncthreads();
            double t[4] = {0.0, 0.0, 0.0, 0.0};
            for (int w = 0; w < G.top_waves; ++w)
                for (int k = 0; k < 4; ++k) t[k] += sums[cycle & 1][w][k];
            if (solve.cycles == 0) {
                // one cycle: the partial for the reduction that ends it
                if (tid == 0)
                    for (int k = 0; k < 4; ++k)
                        gstore(solve.partial, G.part * kNormStride + k, t[k]);
                break;
            }
            // cycles up to the tolerance: the stopping test of k_inst_reduce; an
            // instance that the launch leaves active goes on in the next one
            const InstInfo& in = solve.info[inst];
            const double hd = in.dim == 3 ? in.h * in.h * in.h : in.h * in.h;
            const double tot = combined_norm(t, hd);
            const bool more =
                tot > solve.tol && tot < 1e300 && before + cycle < solve.max_cycles;
            if (more && cycle < solve.cycles) continue;
            if (tid == 0) {
                const double o[6] = {sqrt(t[0] * hd), sqrt(t[1] * hd), sqrt(t[2] * hd), tot,
                                     t[3] / double(in.n0), tot < 1e300 ? 0.0 : 1.0};
                write_results(solve, inst, true, o, more ? 1 : 0, before + cycle);
            }
            break;
        }
    }

    if (my == 0)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            if (P.alive(c))
                for (int k = 0; k < 3; ++k) gstore(G.u[k], P.cell(c), P.u[c][k]);
}

template <typename T>
__global__ void k_spread_owners(const TailDesc<T>* __restrict__ tails, TailOwner* owners) {
    const int inst = blockIdx.x, from = tails[inst].own_from;
    if (tails[inst].levels == 0 || from == inst) return;
    owners[inst * blockDim.x + threadIdx.x] = owners[from * blockDim.x + threadIdx.x];
}

}  // namespace

namespace {

// The kernel for workgroups of `threads`, compiled for several sizes because
// fewer waves leave each lane more registers (512 threads: 256, 768: 168, 1024:
// 128); a size is built only for the forms that fit it without spilling.
template <typename T, bool CORR>
auto own_kernel(int dim, int threads) {
    if constexpr (CORR) {
        if (threads <= 512) return dim == 2 ? &k_tail_own<2, T, CORR, 512> : &k_tail_own<3, T, CORR, 512>;
        return dim == 2 ? &k_tail_own<2, T, CORR, 1024> : &k_tail_own<3, T, CORR, 1024>;
    } else {
        if (dim == 3) return &k_tail_own<3, T, CORR, 512>;
        return threads <= 512 ? &k_tail_own<2, T, CORR, 512> : &k_tail_own<2, T, CORR, 768>;
    }
}

}  // namespace

template <typename T, bool CORR>
int prepare_tail_own(int dim, int threads, size_t lds_bytes) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(own_kernel<T, CORR>(dim, threads)),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_bytes));
    return e == hipSuccess ? 0 : -1;
}

template <typename T, bool CORR>
void launch_tail_own(int dim, const TailDesc<T>* tails, const TailOwner* owners, int ninst,
                 const int* active, const CycleShape& shape, const TailSolve& solve,
                 int threads, size_t lds_bytes, hipStream_t st) {
    if (ninst <= 0) return;
    hipLaunchKernelGGL((own_kernel<T, CORR>(dim, threads)), dim3(ninst), dim3(threads), lds_bytes,
                       st, tails, owners, threads, active, shape, solve);
}

template <typename T>
void launch_spread_owners(const TailDesc<T>* tails, TailOwner* owners, int ninst, int threads,
                          hipStream_t st) {
    hipLaunchKernelGGL(k_spread_owners<T>, dim3(ninst), dim3(threads), 0, st, tails, owners);
}

template void launch_spread_owners<double>(const TailDesc<double>*, TailOwner*, int, int, hipStream_t);
template void launch_spread_owners<float>(const TailDesc<float>*, TailOwner*, int, int, hipStream_t);
template int prepare_tail_own<double, false>(int, int, size_t);
template int prepare_tail_own<float, true>(int, int, size_t);
template void launch_tail_own<double, false>(int, const TailDesc<double>*, const TailOwner*, int,
                                         const int*, const CycleShape&, const TailSolve&, int,
                                     size_t, hipStream_t);
template void launch_tail_own<float, true>(int, const TailDesc<float>*, const TailOwner*, int,
                                       const int*, const CycleShape&, const TailSolve&, int,
                                     size_t, hipStream_t);

}  // namespace chhs
