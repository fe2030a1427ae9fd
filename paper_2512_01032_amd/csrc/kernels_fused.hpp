// kernels_fused.hpp -- the time step as one kernel (gfx950), for lattices in the
// fused layout (pflbm.hpp).
//
// The separate passes (kernels_impl.hpp) form phi in a kernel of its own,
// because the in-place sweep overwrites the h of a tile's neighbours.  Here h
// has two buffers: step t reads hb[t & 1] and writes hb[(t + 1) & 1], so any
// tile can form phi of its halo from h entries that nobody writes during the
// step.  That makes the phi pass, the wall pass, the ghost pass and the step
// counter parts of the sweep: one launch instead of three to five.  g stays in
// place (AA pattern).
//
// Rounding.  The sign term of Eq. 5 and the eps-regularised unit vectors turn a
// last-bit difference into a visible one within tens of steps, so a lattice
// must not round differently because it runs fused.  The arithmetic below and the
// near-wall functions that both layouts use (wall_normal, wall_sums) have every
// rounding explicit: contraction off, fma where one is meant.  The separate sweep is
// compiled with contraction; its node arithmetic is repeated here in the order and
// with the fused multiply-adds that it has, so the two layouts agree bitwise, which
// the tests hold for every option.
//
// What bounds it.  While the populations stay in the 256 MB Infinity Cache a step
// was bound by its three to five dependent launches (4 to 9 us each) and by the
// second pass over h: FP32 cap 128 x 128 x 96 76.0 -> 52.0 us a step, channel
// 1024 x 32 x 32 68.1 -> 43.4, FP64 droplet 32^3 16.3 -> 8.1, 2-D channel
// 25.0 -> 10.7, FP16 g cap 119 x 101 x 67 with hysteresis 48.7 -> 29.6.  Beyond it
// HBM bounds the step (4.5 TB/s, duct 256 x 256 x 512, 1083 -> 1027 with plane_order).  Vector
// instructions come next (900 to 1050 per wave): the cells' indexes are shifts and
// masks and the ring rows wave-uniform (with division by the ring length
// instead 1000 to 1140, the cap 55.7 us, FP16 g duct 192 x 192 x 384 483 us against
// 414), and h in blocks of a tile width puts a thread's seven accesses at
// immediate offsets of one address (414 -> 394 us; h as seven separate rows
// before).  One node per thread: marching two planes per thread needs more than
// 128 registers, two planes per 512-thread tile lose more in the barrier than the
// shared halo gives (the cap 59.3 against 55.7 us).
#pragma once

#include <type_traits>

#include "kernels_impl.hpp"

namespace pflbm {

// ------------------------------------------------------ h of the fused layout
// Blocks of one tile width: f_i of node (x, y, z) is at
//   (x / TX) TX Q SZ + i TX SZ + (x % TX) SZ   of the row (y, z),
// so the Q populations of a wave's nodes lie together, and its Q accesses differ
// in the instruction's immediate offset alone.
template <typename S_, int Q_, int TX> struct HArr {
    typedef S_ S;
    static constexpr int Q = Q_;
    static constexpr uint32_t SZ = (uint32_t)sizeof(S), DIR = (uint32_t)TX * SZ, BLK = DIR * (uint32_t)Q;
    __amdgpu_buffer_rsrc_t r;
    uint32_t row, plane;      // bytes between y-rows and between z-planes
    __device__ void load(const void* base, int64_t bytes, int nxh, int ny) {
        row = (uint32_t)nxh * (uint32_t)Q * SZ;
        plane = row * (uint32_t)ny;
        r = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)(uint32_t)bytes, BUF_FLAGS);
    }
    __device__ __amdgpu_buffer_rsrc_t rs(int) const { return r; }
    __device__ static uint32_t xo(int x) { return (uint32_t)x / (uint32_t)TX * BLK + (uint32_t)x % (uint32_t)TX * SZ; }
    __device__ uint32_t at(int x, int y, int z) const { return xo(x) + (uint32_t)y * row + (uint32_t)z * plane; }
};
// Byte offsets of a node and of its x and y neighbours, periodic wrap, and the
// three z-planes around it, in h.
template <typename H> struct HNbr {
    uint32_t x[3], y[3], z[3];
    __device__ void init(const H& h, int xx, int yy, int zz, int nx, int ny, int nz) {
        x[0] = H::xo(xx == 0 ? nx - 1 : xx - 1); x[1] = H::xo(xx); x[2] = H::xo(xx == nx - 1 ? 0 : xx + 1);
        y[1] = (uint32_t)yy * h.row;
        y[0] = yy == 0 ? (uint32_t)(ny - 1) * h.row : y[1] - h.row;
        y[2] = yy == ny - 1 ? 0u : y[1] + h.row;
        z[0] = (uint32_t)(zz == 0 ? nz - 1 : zz - 1) * h.plane;
        z[1] = (uint32_t)zz * h.plane;
        z[2] = (uint32_t)(zz == nz - 1 ? 0 : zz + 1) * h.plane;
    }
};
// Post-collision h of a node into the buffer of the next step: f*_i to
// (x + c_i, i), or to (x, opp(i)) where x + c_i is solid (half-way
// bounce-back), so every step reads its own entries only.
template <typename H, typename T>
__device__ inline void push_h(const H& a, const HNbr<H>& nb, uint32_t solid, bool wsolid, const T* d) {
    typedef typename H::S S;
    const uint32_t own = nb.x[1] + nb.y[1];
    Store<S>::stx(a, 0, own, nb.z[1], d[0]);
    if (!wsolid) {
#pragma unroll
        for (int i = 1; i < H::Q; ++i)
            Store<S>::stx(a, i, nb.x[CX[i] + 1] + nb.y[CY[i] + 1] + (uint32_t)i * H::DIR, nb.z[CZ[i] + 1], d[i]);
        return;
    }
#pragma unroll
    for (int i = 1; i < H::Q; ++i) {
        const uint32_t to = nb.x[CX[i] + 1] + nb.y[CY[i] + 1] + nb.z[CZ[i] + 1] + (uint32_t)i * H::DIR;
        const uint32_t back = own + nb.z[1] + (uint32_t)OPP[i] * H::DIR;
        Store<S>::stx(a, i, ((solid >> i) & 1u) ? back : to, 0u, d[i]);
    }
}

// ------------------------------------------------- g of the fused layout
// The blocked form of the separate passes, g alone.  A node's z-plane is uniform
// over a wave, so an access is a per-lane (x, y) offset plus a scalar holding
// plane and direction.  A pair (i, opp(i)) never straddles the two groups of the
// FP64 layout.
template <typename LAY> struct GNbr {
    uint32_t x[3], y[3], z[3];
    __device__ void init(int xx, int yy, int zz, int nx, int ny, int nz, int nxp) {
        const int xs[3] = {xx == 0 ? nx - 1 : xx - 1, xx, xx == nx - 1 ? 0 : xx + 1};
#pragma unroll
        for (int c = 0; c < 3; ++c)
            x[c] = (uint32_t)(xs[c] >> 6) * (uint32_t)LAY::BLK + (uint32_t)(xs[c] & 63) * (uint32_t)LAY::SZG;
        const uint32_t row = (uint32_t)(nxp >> 6) * (uint32_t)LAY::BLK, plane = (uint32_t)ny * row;
        y[1] = (uint32_t)yy * row;
        y[0] = yy == 0 ? (uint32_t)(ny - 1) * row : y[1] - row;
        y[2] = yy == ny - 1 ? 0u : y[1] + row;
        z[0] = (uint32_t)(zz == 0 ? nz - 1 : zz - 1) * plane;
        z[1] = (uint32_t)zz * plane;
        z[2] = (uint32_t)(zz == nz - 1 ? 0 : zz + 1) * plane;
    }
    __device__ uint32_t xy(int i, int s) const { return x[s * CX[i] + 1] + y[s * CY[i] + 1]; }
    // offset of the plane of x + s c_i
    __device__ uint32_t zs(int i, int s) const { return z[s * CZ[i] + 1]; }
};
// Keeps a wave-uniform branch a branch.
__device__ inline void keep_branch() { asm volatile(""); }
// Deviations of the populations g_i(x) entering the node's collision: even step
// (x, i); odd step (x - c_i, opp(i)), or (x, i) where x - c_i is solid.  wsolid:
// some lane of the wave has a solid neighbour.
template <typename T, int PAR, typename PA, typename LAY>
__device__ inline void read_g(const PA& a, const GNbr<LAY>& nb, uint32_t solid, bool wsolid, T inv_scale, T* d) {
    typedef typename PA::S S;
    const uint32_t own = nb.xy(0, 0);
    d[0] = (T)Store<S>::ldx(a, 0, own, nb.z[1] + PA::so(0));
    if (PAR == 0 || !wsolid) {
#pragma unroll
        for (int i = 1; i < QG; ++i) {
            if (PAR == 0) d[i] = (T)Store<S>::ldx(a, i, own, nb.z[1] + PA::so(i));
            else d[i] = (T)Store<S>::ldx(a, OPP[i], nb.xy(i, -1), nb.zs(i, -1) + PA::so(OPP[i]));
        }
    } else {
        keep_branch();
#pragma unroll
        for (int i = 1; i < QG; ++i) {
            const bool so = (solid >> OPP[i]) & 1u;
            const uint32_t off = so ? own + nb.z[1] + PA::so(i) : nb.xy(i, -1) + nb.zs(i, -1) + PA::so(OPP[i]);
            d[i] = (T)Store<S>::ldx(a, i, off, 0u);
        }
    }
    if (Store<S>::scaled) {
#pragma unroll
        for (int i = 0; i < QG; ++i) d[i] *= inv_scale;
    }
}
// Post-collision g_i of a node: even step to (x, opp(i)); odd step to
// (x + c_i, i), or to (x, opp(i)) where x + c_i is solid (half-way bounce-back).
template <int PAR, typename PA, typename LAY, typename V>
__device__ inline void put_g1(const PA& a, const GNbr<LAY>& nb, uint32_t solid, bool wsolid, int i, V v) {
    typedef typename PA::S S;
    const uint32_t own = nb.xy(0, 0);
    if (PAR == 0 || i == 0) {
        Store<S>::stx(a, OPP[i], own, nb.z[1] + PA::so(OPP[i]), v);
    } else if (!wsolid) {
        Store<S>::stx(a, i, nb.xy(i, 1), nb.zs(i, 1) + PA::so(i), v);
    } else {
        keep_branch();
        const uint32_t off = ((solid >> i) & 1u) ? own + nb.z[1] + PA::so(OPP[i]) : nb.xy(i, 1) + nb.zs(i, 1) + PA::so(i);
        Store<S>::stx(a, i, off, 0u, v);
    }
}

// ------------------------------------------------------- node arithmetic
// One node's quantities between the stages below (compute precision T).
template <typename T> struct FNode {
    T pc, rho, pb;            // phi, density, clamped phi
    T gr[3], lap;             // gradient and Laplacian of phi
    T mu;                     // chemical potential
    T u[3], uu, pdev;
    T mf[3];                  // mu grad + F
};

// Gradient and Laplacian sums (Eq. 16) in the paper's difference form, each +-c
// pair once: a neighbourhood symmetric about x gives an exactly zero component.
template <typename T, typename NB>
__device__ inline void f_stencil(T pc, const NB& nbv, T* sum) {
#pragma clang fp contract(off)
    T gx = T(0), gy = T(0), gz = T(0), lap = T(0);
#pragma unroll
    for (int i = 1; i < 19; i += 2) {
        const T vp = nbv(i), vm = nbv(i + 1);
        const T dv = vp - vm;
        if (CX[i]) gx = fm(dv, T(wg(i) * CX[i]), gx);
        if (CY[i]) gy = fm(dv, T(wg(i) * CY[i]), gy);
        if (CZ[i]) gz = fm(dv, T(wg(i) * CZ[i]), gz);
        lap = fm((vp - pc) + (vm - pc), T(wg(i)), lap);
    }
    sum[0] = gx; sum[1] = gy; sum[2] = gz; sum[3] = lap;
}

// Local scalars (Eq. 9, Eqs. 10-12) from phi and the stencil sums.
template <typename T>
__device__ inline void f_scalars(FNode<T>& s, const Phys<T>& ph, const T* sum) {
#pragma clang fp contract(off)
    s.gr[0] = sum[0] * T(3); s.gr[1] = sum[1] * T(3); s.gr[2] = sum[2] * T(3);
    s.lap = sum[3] * T(6);
    s.pb = clamp01(s.pc);
    s.rho = fm(ph[PI_RDIF], s.pb, ph[PI_RHO_G]);
    const T ml = s.lap * ph[PI_MULAP];
    s.mu = fm(s.pc + T(-0.5), (s.pc + T(-1)) * (s.pc * ph[PI_MU3]), -ml);
}

// Mass s, momentum j and second moments m (xx yy zz xy xz yz) of the incoming
// populations, by pairs (i, opp(i)).
template <typename T>
__device__ inline void f_moments(const T* d, T& s, T* j, T* m) {
#pragma clang fp contract(off)
    s = d[0];
    j[0] = j[1] = j[2] = T(0);
    m[0] = m[1] = m[2] = m[3] = m[4] = m[5] = T(0);
#pragma unroll
    for (int i = 1; i < QG; i += 2) {
        const T ev = d[i] + d[i + 1], od = d[i] - d[i + 1];
        s += ev;
        if (CX[i]) j[0] += T(CX[i]) * od;
        if (CY[i]) j[1] += T(CY[i]) * od;
        if (CZ[i]) j[2] += T(CZ[i]) * od;
        if (CX[i]) m[0] += ev;
        if (CY[i]) m[1] += ev;
        if (CZ[i]) m[2] += ev;
        if (CX[i] * CY[i]) m[3] += T(CX[i] * CY[i]) * ev;
        if (CX[i] * CZ[i]) m[4] += T(CX[i] * CZ[i]) * ev;
        if (CY[i] * CZ[i]) m[5] += T(CY[i] * CZ[i]) * ev;
    }
}

// u, then P (text of Eq. 15).
template <typename T>
__device__ inline void f_velocity(FNode<T>& n, const Phys<T>& ph, T s, const T* j, T& ug) {
#pragma clang fp contract(off)
    const T irho = dev_div(T(1), n.rho);
    const T F[3] = {ph[PI_FX], ph[PI_FY], ph[PI_FZ]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        n.mf[a] = fm(n.gr[a], n.mu, F[a]);
        n.u[a] = irho * fm(n.mf[a], T(0.5), j[a]);
    }
    ug = fm(n.gr[2], n.u[2], fm(n.gr[0], n.u[0], n.gr[1] * n.u[1]));
    n.pdev = fm(ph[PI_RDIF] * T(0.5), ug, s);
    n.uu = fm(n.u[2], n.u[2], fm(n.u[0], n.u[0], n.u[1] * n.u[1]));
}

// What the outgoing pairs of the filtered collision (Eqs. 6-8, 13-15) share:
// w_i (E +- O) with E = e2 B + a r + C0 + om c_i c_i:Pi, O = a B + e2 r + c,
// a = 3/2 c_i.u, b = rdif c_i.grad, c = c_i.V / 2, r = b + 2 c, e2 = a a + k2.
template <typename T> struct FPair {
    T u15[3], rg[3], vh[3], V[3], Pi[6], om, k2, B, C0;
};
template <typename T>
__device__ inline void f_collision(FPair<T>& q, const FNode<T>& n, const Phys<T>& ph, T ug, const T* m) {
#pragma clang fp contract(off)
    const T rdif = ph[PI_RDIF], Tg = T(TGc);
#pragma unroll
    for (int a = 0; a < 3; ++a) q.V[a] = n.mf[a] * T(3);
    const T* u = n.u;
    const T* g = n.gr;
    const T* V = q.V;
    const T uV = fm(V[2], u[2], fm(V[0], u[0], V[1] * u[1]));
    const T cuu = fm(rdif, ug, uV);
    const T tp = n.pdev * Tg, rt = rdif * Tg;
    const T ru[3] = {n.rho * u[0], n.rho * u[1], n.rho * u[2]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T gu = g[a] * u[a], vu = V[a] * u[a];
        const T k = fm(fm(rdif, gu + gu, vu + vu), Tg, -(cuu * (u[a] * u[a])));
        const T cck = fm(rt, ug, k);
        q.Pi[a] = m[a] + fm(cck, T(0.5), -fm(ru[a], u[a], tp));
    }
    constexpr int IA[3] = {0, 0, 1}, IB[3] = {1, 2, 2};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int a = IA[c], b = IB[c];
        const T gu = fm(u[a], g[b], g[a] * u[b]), vu = fm(u[a], V[b], u[b] * V[a]);
        const T k = fm(fm(rdif, gu, vu), Tg, -(cuu * (u[a] * u[b])));
        q.Pi[3 + c] = m[3 + c] + fm(k + T(0), T(0.5), -fm(ru[a], u[b], T(0)));
    }
    T Fm;
    if (ph.mix) Fm = half_tanh1((n.pb - ph[PI_MIX_PHI]) * ph[PI_MIX_INVW]);
    else Fm = n.pb;
    const T tau = fm(T(1) - Fm, ph[PI_TAU_G], Fm * ph[PI_TAU_L]);
    q.om = (T(1) - dev_div(T(1), tau)) * T(4.5);
    const T trPi = ((q.Pi[0] + q.Pi[1]) + q.Pi[2]) * Tg;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        q.u15[a] = u[a] * T(1.5);
        q.rg[a] = rdif * g[a];
        q.vh[a] = V[a] * T(0.5);
    }
    q.k2 = n.uu * T(-0.75);
    q.B = fm(n.rho, T(2), -cuu);
    q.C0 = fm(-trPi, q.om, fm(uV, T(-0.5), n.pdev));
}
template <typename T>
__device__ inline T f_rest(const FPair<T>& q) {
#pragma clang fp contract(off)
    return fm(q.k2, q.B, q.C0) * T(wg(0));
}
// Outgoing pair (i, opp(i)).  The even step's kernel forms the sums over two
// axes from the unrounded second term and rounds w O first; the odd step's adds
// rounded terms and, in FP32 for every pair and in FP64 for the z axis, rounds
// w E first and subtracts rounded products.
template <typename T, int PAR>
__device__ inline void f_pair(int i, const FPair<T>& q, const FNode<T>& n, T rdif, T& vp, T& vm) {
#pragma clang fp contract(off)
    T a, b, c, cc;
    bool yaxis = false;
    const int nz = (CX[i] != 0) + (CY[i] != 0) + (CZ[i] != 0);
    if (nz == 1) {
        const int k = CX[i] ? 0 : (CY[i] ? 1 : 2);
        a = q.u15[k]; b = q.rg[k]; c = q.vh[k]; cc = q.Pi[k];
        yaxis = k == 1;
    } else {
        // f: the axis whose rounded term comes first, s: the other one
        const int lo = CX[i] ? 0 : 1, hi = CZ[i] ? 2 : 1;
        const int sg = (CX[i] ? CX[i] : CY[i]) * (CZ[i] ? CZ[i] : CY[i]);
        const int pi = CX[i] ? (CY[i] ? 3 : 4) : 5;
        if (PAR == 0) {
            const int f = CX[i] && CZ[i] && sg > 0 ? 0 : (CZ[i] ? 2 : 0), s = f == lo ? hi : lo;
            // xy: x +- y; xz: x + z, -z + x; yz: +-z + y
            const T sf = f == 2 && sg < 0 ? T(-1) : T(1), ss = f == 0 && sg < 0 ? T(-1) : T(1);
            a = fm(n.u[s], ss * T(1.5), sf * q.u15[f]);
            b = fm(ss * rdif, n.gr[s], sf * q.rg[f]);
            c = fm(q.V[s], ss * T(0.5), sf * q.vh[f]);
        } else {
            const T ss = T(sg);
            a = q.u15[lo] + ss * q.u15[hi];
            b = q.rg[lo] + ss * q.rg[hi];
            c = q.vh[lo] + ss * q.vh[hi];
        }
        cc = fm(q.Pi[pi], T(2 * sg), q.Pi[lo] + q.Pi[hi]);
    }
    const T e2 = fm(a, a, q.k2);
    const T r = PAR == 0 && yaxis ? fm(rdif, n.gr[1], c + c) : fm(c, T(2), b);
    const T E = fm(q.B, e2, fm(a, r, fm(q.om, cc, q.C0)));
    const T O = fm(q.B, a, fm(e2, r, c));
    const T w = T(wg(i));
    if (PAR == 1 && (sizeof(T) == 4 || i == 5)) {
        const T wE = E * w, wO = O * w;
        vp = fm(O, w, wE);
        vm = wE - wO;
    } else {
        const T wO = O * w;
        vp = fm(E, w, wO);
        vm = fm(E, w, -wO);
    }
}

// Phase field (Eqs. 1-5): w_i X_i is the equilibrium deviation of direction i,
// handed over as set(i, X_i, w_i).
template <typename T, int QP, typename SET>
__device__ inline void f_phase_eq(const FNode<T>& n, const Phys<T>& ph, const SET& set) {
#pragma clang fp contract(off)
    const T pc = n.pc;
    const T gnorm = dev_sqrt(fm(n.gr[2], n.gr[2], fm(n.gr[1], n.gr[1], n.gr[0] * n.gr[0])));
    const T ph5 = pc + T(-0.5);
    T theta = fm(ph5, ph5 * T(-4), T(1)) * ph[PI_THETA0];
    if (ph.mobility_corr) {
        const T y1a = clamp01((pc - ph[PI_MC_PHI_M]) * ph[PI_MC_INVD]);
        const T y1b = clamp01((T(1) - pc) * ph[PI_MC_INVD]);
        const T y2a = clamp01(pc * ph[PI_MC_INVD]);
        const T y2b = clamp01((ph[PI_MC_PHI_m] - pc) * ph[PI_MC_INVD]);
        const T Y1 = y1a < y1b ? y1a : y1b;
        const T Y2 = y2a < y2b ? y2a : y2b;
        T sp, sm;   // 1 +- lap / (|lap| + eps)
        const T den = fabs(n.lap) + ph[PI_EPS];
        if constexpr (sizeof(T) == 4) {
            const T r = __builtin_amdgcn_rcpf(den);
            sp = fm(n.lap, r, T(1));
            sm = fm(-n.lap, r, T(1));
        } else {
            const T sgn = n.lap / den;
            sp = T(1) + sgn;
            sm = T(1) - sgn;
        }
        theta = fm(gnorm * ph[PI_MC_K], fm(sp, Y1, sm * Y2), theta);
    }
    const T ign = dev_div(theta, gnorm + ph[PI_EPS]);   // theta n = theta grad / (|grad| + eps)
    const T hr = pc - ph[PI_HREF], uu2 = n.uu + n.uu;
    set(0, fm(-pc, uu2, hr), T(wp<QP>(0)));
#pragma unroll
    for (int i = 1; i < QP; i += 2) {
        const int k = CX[i] ? 0 : (CY[i] ? 1 : 2);
        const T e = fm(pc, fm(n.u[k], n.u[k] * T(8), -uu2), hr);
        const T o = fm(n.gr[k], ign, (pc * T(4)) * n.u[k]);
        set(i, o + e, T(wp<QP>(i)));
        set(i + 1, e - o, T(wp<QP>(i)));
    }
}

// FP64 diagnostics of one node: its terms of the summed quantities (max |u| as its
// square: the root is monotone and taken once per tile) and its kind.  The kinds are
// flags, counted over a wave by ballots: as counters beside the sums, their equal
// increments were merged into one through an index, which put them into scratch
// memory (lbm_reduce of the duct 256 x 256 x 512: FP32 756 us, 679 without; FP16 g
// 866, 630; FP64 1821, 1455).
struct DiagKind { bool nan, liq, gas; };
template <typename T>
__device__ inline DiagKind f_diag(double* acc, const FNode<T>& n, const Phys<T>& ph) {
    const T pc = n.pc;
    const double uu = (double)n.uu;
    const double P = (double)(T(TGc) * (ph[PI_GREF] + n.pdev));
    const bool bad = isnan((double)pc) || isnan(uu) || isnan(P);
    const DiagKind k = {bad, !bad && pc > T(0.99), !bad && pc < T(0.01)};
    if (!bad) {
        acc[P_PHI] += (double)pc;
        acc[P_MX] += (double)(n.rho * n.u[0]);
        acc[P_MY] += (double)(n.rho * n.u[1]);
        acc[P_MZ] += (double)(n.rho * n.u[2]);
        acc[P_UMAX] = fmax(acc[P_UMAX], uu);
    }
    if (k.liq) acc[P_PLIQ] += P;
    if (k.gas) acc[P_PGAS] += P;
    return k;
}

// Equilibria of one node at step 0 (MODE_INIT): g with K_i (Eqs. 7-8) through
// put_g(i, g_eq_i - w_i gref), from the node's phi, stencil (sum: unscaled
// gradient sums), u and P.
template <typename T, typename PUT>
__device__ inline void f_init_g(const FNode<T>& n, const Phys<T>& ph, const T* sum, const PUT& put_g) {
#pragma clang fp contract(off)
    const T rdif = ph[PI_RDIF];
    const T* u = n.u;
    const T* g = n.gr;
    const T V[3] = {n.mf[0] * T(3), n.mf[1] * T(3), n.mf[2] * T(3)};
    const T ug = fm(g[2], u[2], fm(g[1], u[1], g[0] * u[0]));
    const T uV = fm(u[2], V[2], fm(u[0], V[0], u[1] * V[1]));
    const T k2 = n.uu * T(-1.5);
    // w (rho gam + pdev) - K / 2, K = w (gam rdif (b - ug) + (1 + gam) (c - uV))
    auto eq = [&](T gam, T bu, T cv, T w) -> T {
        const T K = fm(bu, rdif * gam, cv * (gam + T(1))) * w;
        return fm(fm(n.rho, gam, n.pdev), w, K * T(-0.5));
    };
    put_g(0, eq(fm(n.uu, T(-1.5), T(0)), T(0) - ug, T(0) - uV, T(wg(0))));
#pragma unroll
    for (int i = 1; i < QG; i += 2) {
        const int nz = (CX[i] != 0) + (CY[i] != 0) + (CZ[i] != 0);
        const T w = T(wg(i));
        T a, bp, bm, cp, cm;
        if (nz == 1) {
            const int k = CX[i] ? 0 : (CY[i] ? 1 : 2);
            a = u[k];
            bp = fm(sum[k], T(3), -ug); bm = fm(sum[k], T(-3), -ug);
            cp = fm(n.mf[k], T(3), -uV); cm = fm(n.mf[k], T(-3), -uV);
        } else {
            const int lo = CX[i] ? 0 : 1, hi = CZ[i] ? 2 : 1;
            const int sg = (CX[i] ? CX[i] : CY[i]) * (CZ[i] ? CZ[i] : CY[i]);
            a = u[lo] + T(sg) * u[hi];
            T b, c;
            if (lo == 1 && sg < 0) {
                b = fm(sum[1], T(3), -g[2]);
                c = fm(n.mf[1], T(3), -V[2]);
            } else {
                b = fm(sum[hi], T(3 * sg), g[lo]);
                c = fm(n.mf[hi], T(3 * sg), V[lo]);
            }
            bp = b - ug; bm = -b - ug;
            cp = c - uV; cm = -c - uV;
        }
        const T e = fm(a, a * T(4.5), k2);
        put_g(i, eq(fm(a, T(3), e), bp, cp, w));
        put_g(i + 1, eq(fm(a, T(-3), e), bm, cm, w));
    }
}

__device__ inline int wrap1(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// Pressure ghosts of an owner node at the end of its step t: for each ghost
// g = x - n it feeds (n the face's inward normal), the equilibria at its phi and
// u and the face pressure of step t + 1, without forcing and without the
// counter-term, in the directions that point into a fluid node, in the entries
// step t + 1 reads: h (g + c_i, i) of the next buffer, g (g + c_i, i) when t + 1
// is even and (g, opp(i)) when it is odd.  No other node reads or writes these
// entries at step t: only g itself, which is no fluid node, would.
template <typename T, int PAR, typename LAY, typename GB, typename HR, typename FL>
__device__ inline void feed_ghosts(const Desc* D, const GB& gb, const HR& hn, const Phys<T>& pp, const T* u, T pc,
                                   int x, int y, int z, int nx, int ny, int nz, int nxp,
                                   int64_t next, const FL& flag_at) {
#pragma clang fp contract(off)
    typedef typename GB::S SG;
    typedef typename HR::S SH;
    constexpr int QP = HR::Q;
    const T uu = fm(u[2], u[2], fm(u[0], u[0], u[1] * u[1]));
    const T rho = fm(clamp01(pc), pp[PI_RDIF], pp[PI_RHO_G]);
    const T uug = uu * T(1.5), uuh = uu * T(i2tp<QP>()), hr = pc - pp[PI_HREF];
    const uint32_t row = (uint32_t)(nxp >> 6) * (uint32_t)LAY::BLK;
    auto goff = [&](int xa, int ya, int za, uint32_t size) -> uint32_t {
        return (uint32_t)(xa >> 6) * (uint32_t)LAY::BLK + (uint32_t)(xa & 63) * size +
               ((uint32_t)ya + (uint32_t)ny * (uint32_t)za) * row;
    };
#pragma clang loop unroll(disable)
    for (int face = 0; face < 6; ++face) {
        const int sgn = (face & 1) ? -1 : 1;
        const int nf[3] = {(face >> 1) == 0 ? sgn : 0, (face >> 1) == 1 ? sgn : 0, (face >> 1) == 2 ? sgn : 0};
        const uint8_t fg = flag_at(-nf[0], -nf[1], -nf[2]);
        if (flag_kind(fg) != KIND_GHOST || flag_sub(fg) != face) continue;
        const double Pb = __builtin_fma(D->face_ramp[face], (double)(next - D->t0), D->face_P[face]);
        T pdb;
        if constexpr (sizeof(T) == 8) pdb = fm(Pb, 3.0, -pp[PI_GREF]);
        else pdb = (T)(Pb * 3.0) - pp[PI_GREF];
#pragma unroll
        for (int i = 1; i < QG; ++i) {
            if (CX[i] * nf[0] + CY[i] * nf[1] + CZ[i] * nf[2] <= 0) continue;
            // the target g + c_i lies beside the owner, in the plane of the face
            const int lx = CX[i] - nf[0], ly = CY[i] - nf[1], lz = CZ[i] - nf[2];
            if (flag_kind(flag_at(lx, ly, lz)) != KIND_FLUID) continue;
            const int xn = wrap1(x + lx, nx), yn = wrap1(y + ly, ny), zn = wrap1(z + lz, nz);
            const T cu = cdot(i, u[0], u[1], u[2]), cu2 = cu * cu;
            const T vg = T(wg(i)) * fm(rho, fm(cu, T(3), cu2 * T(4.5)) - uug, pdb);
            const T vs = Store<SG>::scaled ? vg * pp[PI_SG] : vg;
            if (PAR == 1) Store<SG>::st(gb, i, goff(xn, yn, zn, sizeof(SG)), vs);
            else Store<SG>::st(gb, OPP[i], goff(x - nf[0], y - nf[1], z - nf[2], sizeof(SG)), vs);
            if (i < QP) {
                const T gh = fm(cu, T(itp<QP>()), cu2 * T(i2tp2<QP>())) - uuh;
                const T vh = T(wp<QP>(i)) * fm(pc, gh, hr);
                Store<SH>::stx(hn, i, hn.at(xn, yn, zn) + (uint32_t)i * HR::DIR, 0u, vh);
            }
        }
    }
}

// The near-wall threads of a workgroup as a list, one segment per wave (barrier between
// wall_gather and wall_entry), so that a tile side with one wall node per row costs one
// wave instead of all.  wall_entry: thread of entry e.
__device__ inline void wall_gather(uint8_t* list, uint32_t* link, int* cnt, int tid, uint32_t solid) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(solid != 0u);
    if ((tid & 63) == 0) cnt[tid >> 6] = __builtin_popcountll(m);
    if (solid) {
        const int r = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        list[(tid & ~63) + r] = (uint8_t)tid;
        link[tid] = solid;
    }
}
__device__ inline int wall_total(const int* cnt) {
    int total = 0;
#pragma unroll
    for (int g = 0; g < NTHREADS / 64; ++g) total += cnt[g];
    return uni(total);
}
__device__ inline int wall_entry(const uint8_t* list, const int* cnt, int e) {
    int g = 0, r = e;
#pragma unroll
    for (int j = 0; j < NTHREADS / 64 - 1; ++j) {
        const int c = cnt[j];
        if (g == j && r >= c) { r -= c; g = j + 1; }
    }
    return list[g * 64 + r];
}

// One time step of a tile (MODE_STEP), or its read-back (MODE_READ) or
// initialisation (MODE_INIT).  A tile is TX x (256 / TX) nodes of one z-plane, one
// per thread.
//
// phi of the tile and of its one-node halo is formed from the h entries of the
// step (each node's own entries): every thread forms its column of three planes,
// then the rings around them, in an order whose indexes are shifts and masks;
// near-wall nodes are gathered into a list and their stencil sums with the
// wetting values (Eqs. 16-19) formed from the LDS planes, so that a tile side
// with one wall node per row costs one wave instead of all; then every node is
// updated.  Owners feed their pressure ghosts, and the lattice's first tile the
// step counter (each parity reads one entry and writes the other, so no tile
// waits).
template <typename T, typename SH, typename SG, int MODE, bool DIAG, int TX, int PAR>
__global__ void __launch_bounds__(NTHREADS)
step_kernel(Desc* __restrict__ descs, const Tile* __restrict__ tiles, bool back, ReadOut ro, InitIn in) {
    static_assert(!Store<SH>::scaled, "h is stored unscaled");
    constexpr int QP = QH, TY = NTHREADS / TX, WAVES = NTHREADS / 64;
    constexpr int LW = TX + 2, LN = (TX + 2) * (TY + 2);
    __shared__ T s_phi[3][LN];
    __shared__ uint8_t s_flag[3][LN];
    __shared__ T s_ws[4][NTHREADS];           // near-wall nodes: stencil sums
    __shared__ uint32_t s_wlink[NTHREADS];    // and solid links
    __shared__ uint8_t s_wlist[NTHREADS];     // their threads, one segment per wave
    __shared__ int s_wcnt[WAVES];
    __shared__ T s_cs[2][16];                 // cos and sin of each material's contact angle
    __shared__ double s_acc[DIAG ? 7 : 1][DIAG ? NTHREADS : 1];
    __shared__ int s_cnt[3][WAVES];

    const Tile tl = load_tile(tiles, back);
    Desc* D = descs + tl.lat;
    const int tid = threadIdx.x;
    const int64_t step = uni(D->step2[PAR]);
    const bool stopped = MODE == MODE_STEP && step >= uni(D->stop_step);
    if (MODE == MODE_STEP && tl.tile_in_lat == 0 && tid == 0) D->step2[PAR ^ 1] = stopped ? step : step + 1;
    if (stopped) return;
    const int64_t time = step - uni(D->t0);
    const int nx = uni(D->nx), ny = uni(D->ny), nz = uni(D->nz);
    const int nxy = nx * ny;
    const int tx = tid & (TX - 1), ty = tid / TX;
    const int x = tl.x0 + tx, y = tl.y0 + ty, z = tl.z0;
    const bool active = x < nx && y < ny;
    const int64_t N = uni(D->N);
    const int64_t dev = uni(D->diag_every);
    const bool diag = DIAG && (MODE == MODE_READ || (dev > 0 && (time % dev) == 0));
    Phys<T> ph;
    ph.load(D);
    const uint8_t* __restrict__ flg = unip(D->flag);
    const uint32_t* __restrict__ lnk = unip(D->link);
    const __attribute__((address_space(4))) Desc* DC = (const __attribute__((address_space(4))) Desc*)D;
    typedef Lay<SG, SG, 0> LAYT;
    const auto gb = pop_array<SG, QG, 0, LAYT>(D);
    const int nxp = uni(D->nxp), nxh = uni(D->nxh);
    typedef HArr<SH, QP, TX> HR;
    HR hc, hn;   // h entering this step, h of the next one
    hc.load(unip((char*)D->hb[PAR]), uni(D->hbytes), nxh, ny);
    hn.load(unip((char*)D->hb[MODE == MODE_INIT ? PAR : PAR ^ 1]), uni(D->hbytes), nxh, ny);
    const bool walls = DC->n_wall > 0, ghosts = DC->gface_count > 0, linked = walls || ghosts;

    // ---- the node's link word first (the odd step's addresses need it)
    const int n = x + nx * y + nxy * z;
    uint32_t links = 0u;
    if (linked && active) links = lnk[n];

    // ---- cells.  0 .. 2: the node's column in the planes below, at and above the
    //      tile; then the rings.  Lanes past x = nx or y = ny form some node's phi
    //      into a cell that nobody reads.
    constexpr int NRING = 6 * TX + 6 * TY + 4, NR = (NRING + NTHREADS - 1) / NTHREADS, NCELL = 3 + NR;
    const int zp[3] = {z == 0 ? nz - 1 : z - 1, z, z == nz - 1 ? 0 : z + 1};
    const int xa = tl.x0 == 0 ? nx - 1 : tl.x0 - 1, xb = tl.x0 + TX < nx ? tl.x0 + TX : 0;
    const int ya = tl.y0 == 0 ? ny - 1 : tl.y0 - 1, yb = tl.y0 + TY < ny ? tl.y0 + TY : 0;
    const int xw = x < nx ? x : 0, yw = y < ny ? y : 0;
    int cidx[NCELL], cxy[NCELL], cz[NCELL];   // LDS cell (-1: none), column, plane
    uint32_t cho[NCELL];                      // h offset
    auto set_cell = [&](int j, int p, int cell, int cx, int cy, int czz) {
        cidx[j] = p * LN + cell;
        cxy[j] = cx + nx * cy;
        cz[j] = czz;
        cho[j] = hc.at(cx, cy, czz);
    };
#pragma unroll
    for (int j = 0; j < 3; ++j) set_cell(j, j, (ty + 1) * LW + tx + 1, xw, yw, zp[j]);
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        // rows below and above the tile in each plane, its columns left and
        // right, the corners of its own plane (no node uses the others)
        const int e = tid + j * NTHREADS;
        if ((TX == 64 ? uni(e >> 6) * 64 : e) < 6 * TX) {
            const int seg = TX == 64 ? uni(e >> 6) : e / TX, p = seg >> 1, c = e & (TX - 1);
            const bool up = seg & 1;
            set_cell(3 + j, p, (up ? (TY + 1) * LW : 0) + c + 1, tl.x0 + c < nx ? tl.x0 + c : 0, up ? yb : ya,
                     p == 0 ? zp[0] : (p == 1 ? zp[1] : zp[2]));
        } else {
            const int e2 = e - 6 * TX, k = e2 - 6 * TY;
            const bool corner = k >= 0;
            const int side = e2 / TY, p = corner ? 1 : side >> 1, r = e2 & (TY - 1);
            const bool right = (corner ? k : side) & 1;
            const int row = corner ? (k & 2 ? TY + 1 : 0) : r + 1;
            const int cy = corner ? (k & 2 ? yb : ya) : (tl.y0 + r < ny ? tl.y0 + r : 0);
            set_cell(3 + j, p, row * LW + (right ? TX + 1 : 0), right ? xb : xa, cy,
                     p == 0 ? zp[0] : (p == 1 ? zp[1] : zp[2]));
            if (k > 3) cidx[3 + j] = -1;
        }
    }
    uint32_t cf[NCELL];
    T cv[NCELL][MODE == MODE_INIT ? 1 : QP];
    if (linked) {
#pragma unroll
        for (int j = 0; j < NCELL; ++j)
            if (j < 3 || cidx[j] >= 0) cf[j] = flg[(uint32_t)(cxy[j] + nxy * cz[j])];
    }
#pragma unroll
    for (int j = 0; j < NCELL; ++j) {
        if (j >= 3 && cidx[j] < 0) continue;
        if constexpr (MODE == MODE_INIT) {
            cv[j][0] = ((const T*)in.phi)[(uint32_t)(cxy[j] + nxy * cz[j])];
        } else {
#pragma unroll
            for (int i = 0; i < QP; ++i) cv[j][i] = (T)Store<SH>::ldx(hc, i, cho[j] + (uint32_t)i * HR::DIR, 0u);
        }
    }
    if (walls && tid < 32) s_cs[tid >> 4][tid & 15] = (T)(tid < 16 ? DC->cos_t[tid] : DC->sin_t[tid - 16]);
    const uint32_t solid = links & SOLID_MASK;
    T B[QP];
    if constexpr (MODE != MODE_INIT) {
#pragma unroll
        for (int i = 0; i < QP; ++i) B[i] = cv[1][i];
        if (ghosts) {
            // a pressure ghost takes its owner's phi: one step inward
#pragma unroll
            for (int j = 0; j < NCELL; ++j) {
                if ((j >= 3 && cidx[j] < 0) || flag_kind((uint8_t)cf[j]) != KIND_GHOST) continue;
                const int face = flag_sub((uint8_t)cf[j]), ax = face >> 1;
                // (x faces lie at x = 0 and x = nx - 1)
                const uint32_t dx = (face & 1) ? HR::xo(nx - 1) - HR::xo(nx - 2) : HR::xo(1) - HR::xo(0);
                const uint32_t d = ax == 0 ? dx : (ax == 1 ? hc.row : hc.plane);
                const uint32_t off = (face & 1) ? cho[j] - d : cho[j] + d;
#pragma unroll
                for (int i = 0; i < QP; ++i) cv[j][i] = (T)Store<SH>::ldx(hc, i, off + (uint32_t)i * HR::DIR, 0u);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NCELL; ++j) {
        T v = cv[j][0];
        if constexpr (MODE != MODE_INIT) {
            T sum = T(0);
#pragma unroll
            for (int i = 0; i < QP; ++i) sum += cv[j][i];
            v = ph[PI_HREF] + sum;
        }
        if (j < 3 || cidx[j] >= 0) (&s_phi[0][0])[cidx[j]] = v;
    }
    // (a lattice without walls and faces has fluid nodes only)
    uint32_t f = KIND_FLUID;
    if (linked) {
        f = cf[1];
#pragma unroll
        for (int j = 0; j < NCELL; ++j)
            if (j < 3 || cidx[j] >= 0) (&s_flag[0][0])[cidx[j]] = (uint8_t)cf[j];
    }
    const bool fluid = active && flag_kind((uint8_t)f) == KIND_FLUID;
    if (walls) wall_gather(s_wlist, s_wlink, s_wcnt, tid, solid);
    lds_barrier();
    if (walls) {
        const int total = wall_total(s_wcnt);
        // neighbouring tiles start on different waves (and so SIMDs)
        for (int e = (tid + 64 * tl.tile_in_lat) & (NTHREADS - 1); e < total; e += NTHREADS) {
            const int id = wall_entry(s_wlist, s_wcnt, e);
            const int wx = id & (TX - 1), wy = id / TX;
            const int cw = (wy + 1) * LW + wx + 1;
            const uint32_t sol = s_wlink[id];
            uint32_t mw[3] = {0u, 0u, 0u};
            T nv[19];
#pragma unroll
            for (int i = 1; i < 19; ++i) {
                const int p = 1 + CZ[i], c = cw + CY[i] * LW + CX[i];
                const bool so = (sol >> i) & 1u;
                nv[i] = so ? T(0) : s_phi[p][c];
                mw[(i - 1) / 6] |= so ? (uint32_t)flag_sub(s_flag[p][c]) << (4 * ((i - 1) % 6)) : 0u;
            }
            const int hmode = DC->hysteresis;
            const int64_t nwl = DC->n_wall;
            T* hist = nullptr;
            if (hmode) hist = unip((T*)DC->hyst) + unip(D->wslot)[tl.x0 + wx + nx * (tl.y0 + wy) + nxy * z];
            T nw[3];
            wall_normal(sol, nw);
            const bool record = MODE == MODE_INIT || (MODE == MODE_READ && DC->hyst_reset != 0);
            T sums[4];
            wall_sums<T, MODE>(sol, s_phi[1][cw], nv, mw, nw, s_cs, ph, hmode, record, hist, nwl, sums);
#pragma unroll
            for (int j = 0; j < 4; ++j) s_ws[j][id] = sums[j];
        }
        if (total) lds_barrier();
    }

    double acc[NPART];
#pragma unroll
    for (int j = 0; j < NPART; ++j) acc[j] = 0.0;
    DiagKind kind = {false, false, false};
    const int c0 = (ty + 1) * LW + tx + 1;
    if (MODE == MODE_READ && active && !fluid) {
        double pv = 0.0, Pv = 0.0;
        if (flag_kind((uint8_t)f) == KIND_GHOST) {
            const int face = flag_sub((uint8_t)f);
            pv = (double)s_phi[1][c0];
            Pv = D->face_P[face] + D->face_ramp[face] * (double)time;
        }
        if (ro.phi) ro.phi[n] = pv;
        if (ro.P) ro.P[n] = Pv;
        if (ro.u) { ro.u[n] = 0.0; ro.u[N + n] = 0.0; ro.u[2 * N + n] = 0.0; }
        if (ro.pops)
            for (int i = 0; i < QP + QG; ++i) ro.pops[(int64_t)i * N + n] = 0.0;
    }
    if (fluid) {
        GNbr<LAYT> nb;
        nb.init(x, y, z, nx, ny, nz, nxp);
        const bool wsolid = __builtin_amdgcn_ballot_w64(solid != 0u) != 0u;
        const T pc = s_phi[1][c0];
        T sum[4];
        f_stencil(pc, [&](int i) -> T { return s_phi[1 + CZ[i]][c0 + CY[i] * LW + CX[i]]; }, sum);
        if (solid) { sum[0] = s_ws[0][tid]; sum[1] = s_ws[1][tid]; sum[2] = s_ws[2][tid]; sum[3] = s_ws[3][tid]; }
        FNode<T> nd;
        nd.pc = pc;
        f_scalars(nd, ph, sum);
        if constexpr (MODE == MODE_INIT) {
            const T F[3] = {ph[PI_FX], ph[PI_FY], ph[PI_FZ]};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                nd.u[a] = in.u ? (T)in.u[a * N + n] : T(0);
                nd.mf[a] = fm(nd.gr[a], nd.mu, F[a]);
            }
            nd.uu = fm(nd.u[2], nd.u[2], fm(nd.u[1], nd.u[1], nd.u[0] * nd.u[0]));
            nd.pdev = in.P ? fm((T)in.P[n], T(3), -ph[PI_GREF]) : ph[PI_PREF_DEV];
            const T sgs = ph[PI_SG];
            f_init_g(nd, ph, sum, [&](int i, T v) {
                put_g1<0>(gb, nb, 0u, false, OPP[i], Store<SG>::scaled ? v * sgs : v);
            });
            const uint32_t ho = hn.at(x, y, z);
            f_phase_eq<T, QP>(nd, ph, [&](int i, T X, T w) { Store<SH>::stx(hn, i, ho + (uint32_t)i * HR::DIR, 0u, X * w); });
        } else {
            T dg[QG], s, j[3], m[6], ug;
            read_g<T, PAR>(gb, nb, solid, wsolid, ph[PI_INV_SG], dg);
            f_moments(dg, s, j, m);
            f_velocity(nd, ph, s, j, ug);
            if (MODE == MODE_READ) {
                const T P = T(TGc) * (ph[PI_GREF] + nd.pdev);
                if (ro.phi) ro.phi[n] = (double)pc;
                if (ro.P) ro.P[n] = (double)P;
                if (ro.u) { ro.u[n] = (double)nd.u[0]; ro.u[N + n] = (double)nd.u[1]; ro.u[2 * N + n] = (double)nd.u[2]; }
                if (ro.pops) {
                    for (int i = 0; i < QP; ++i)
                        ro.pops[(int64_t)i * N + n] = (double)(T(wp<QP>(i)) * ph[PI_HREF] + B[i]);
                    for (int i = 0; i < QG; ++i)
                        ro.pops[(int64_t)(QP + i) * N + n] = (double)(T(wg(i)) * ph[PI_GREF] + dg[i]);
                }
            }
            if (DIAG && diag) kind = f_diag(acc, nd, ph);
            if constexpr (MODE == MODE_STEP) {
                FPair<T> q;
                f_collision(q, nd, ph, ug, m);
                // free-slip band (Sec. III.A): at a wall link the wall moves with
                // the tangential fluid velocity u_w (times the slip factor for
                // partial slip), and the bounced-back population loses the
                // moving-wall term 6 w_i rho (c_i . u_w)
                T ruw[3] = {T(0), T(0), T(0)};   // u_w
                bool slip = false;
                if (solid && ph.friction && pc >= ph[PI_SLIP_LO] && pc <= ph[PI_SLIP_HI]) {
                    T nw[3];
                    wall_normal(solid, nw);
                    const T un = fm(nw[2], nd.u[2], fm(nw[0], nd.u[0], nw[1] * nd.u[1]));
#pragma unroll
                    for (int a = 0; a < 3; ++a) ruw[a] = fm(-nw[a], un, nd.u[a]);
                    slip = true;
                }
                const bool wslip = __builtin_amdgcn_ballot_w64(slip) != 0u;
                const T rho6 = nd.rho * ph[PI_SLIP_W6], sgs = ph[PI_SG], rdif = ph[PI_RDIF];
                auto put = [&](int i, T v) {
                    put_g1<PAR>(gb, nb, solid, wsolid, i, Store<SG>::scaled ? v * sgs : v);
                };
                put(0, f_rest(q));
#pragma unroll
                for (int i = 1; i < QG; i += 2) {
                    T vp, vm;
                    f_pair<T, PAR>(i, q, nd, rdif, vp, vm);
                    if (wslip) {
                        keep_branch();
                        if (slip && ((solid >> i) & 1u))
                            vp = fm(rho6 * cdot(i, ruw[0], ruw[1], ruw[2]), -T(wg(i)), vp);
                        if (slip && ((solid >> (i + 1)) & 1u))
                            vm = fm(rho6 * cdot(i + 1, ruw[0], ruw[1], ruw[2]), -T(wg(i)), vm);
                    }
                    put(i, vp);
                    put(i + 1, vm);
                }
                const T itau = ph[PI_ITAU_H];
                f_phase_eq<T, QP>(nd, ph, [&](int i, T X, T w) { B[i] = fm(itau, fm(X, w, -B[i]), B[i]); });
                HNbr<HR> hnb;
                hnb.init(hn, x, y, z, nx, ny, nz);
                push_h(hn, hnb, solid, wsolid, B);
                if (links >> LINK_OWNER_SHIFT)
                    feed_ghosts<T, PAR, LAYT>(D, gb, hn, ph, nd.u, pc, x, y, z, nx, ny, nz, nxp, step + 1,
                                              [&](int cx, int cy, int cz) -> uint8_t {
                                                  return s_flag[1 + cz][c0 + cy * LW + cx];
                                              });
            }
        }
    }
    if constexpr (DIAG && MODE != MODE_INIT) {
        if (!diag) return;
        // Counts are ballots.  The other seven quantities go through LDS, so that a
        // wave sums one or two of them over the tile's 256 nodes: a tree per wave
        // and quantity exchanged seven times as much and bound the pass
        // (lbm_reduce, FP16 g duct 256 x 256 x 512, 803 us).
        constexpr int NSUM = 7;
        const int lane = tid & 63, w = uni(tid >> 6);
        auto part = [](int j) -> int { return j < P_PLIQ - 1 ? j : (j == P_PLIQ - 1 ? P_PLIQ : P_PGAS); };
#pragma unroll
        for (int j = 0; j < NSUM; ++j) s_acc[j][tid] = acc[part(j)];
        const bool is[3] = {kind.nan, kind.liq, kind.gas};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(is[j]);
            if (lane == 0) s_cnt[j][w] = __builtin_popcountll(m);
        }
        lds_barrier();
        double* __restrict__ out = D->partials + tl.tile_in_lat;
        const int64_t nt = uni(D->ntiles);
        for (int j = w; j < NSUM; j += WAVES) {
            double v = s_acc[j][lane];
#pragma unroll
            for (int k = 1; k < WAVES; ++k) {
                const double o = s_acc[j][lane + 64 * k];
                v = j == P_UMAX ? fmax(v, o) : v + o;
            }
            v = j == P_UMAX ? sqrt(wave_max(v)) : wave_sum(v);
            if (lane == 0) out[part(j) * nt] = v;
        }
        if (tid < 3) {
            int c = 0;
            for (int k = 0; k < WAVES; ++k) c += s_cnt[tid][k];
            out[(tid == 0 ? P_NAN : (tid == 1 ? P_NLIQ : P_NGAS)) * nt] = (double)c;
        }
    }
}

// Phi of every node [N] into the h buffer of the next step, whose live entries that
// step writes anyway.
template <typename T, typename SH>
__global__ void __launch_bounds__(NTHREADS)
fused_phi_kernel(const Desc* __restrict__ descs, const Tile* __restrict__ tiles, int par) {
    const Tile tl = load_tile(tiles);
    const Desc* D = descs + tl.lat;
    const int nx = uni(D->nx), ny = uni(D->ny), TX = uni(D->tx), nxh = uni(D->nxh);
    const int x = tl.x0 + (threadIdx.x & (TX - 1)), y = tl.y0 + threadIdx.x / TX;
    if (x >= nx || y >= ny) return;
    const bool linked = uni((int)(D->n_wall > 0 || D->gface_count > 0)) != 0;
    const uint8_t* __restrict__ flg = unip(D->flag);
    const SH* __restrict__ h = (const SH*)unip((char*)D->hb[par]);
    T* __restrict__ out = unip((T*)D->hb[par ^ 1]);
    const T href = unip(param_block<T>(D))[PI_HREF];
    for (int k = 0; k < tl.zn; ++k) {
        const int z = tl.z0 + k, n = x + nx * (y + ny * z);
        int ox = x, oy = y, oz = z;
        if (linked) {
            const uint8_t f = flg[n];
            if (flag_kind(f) == KIND_SOLID) continue;
            if (flag_kind(f) == KIND_GHOST) {   // its owner's
                const int face = flag_sub(f), in = (face & 1) ? -1 : 1;
                if (face >> 1 == 0) ox += in;
                else if (face >> 1 == 1) oy += in;
                else oz += in;
            }
        }
        const SH* const own = h + (int64_t)QH * (nxh * ((int64_t)oy + (int64_t)ny * oz) + ox / TX * TX) + ox % TX;
        T v[QH], sum = T(0);
#pragma unroll
        for (int i = 0; i < QH; ++i) v[i] = (T)own[i * TX];
#pragma unroll
        for (int i = 0; i < QH; ++i) sum += v[i];
        out[n] = href + sum;
    }
}

// Populations f_i(x) of a step of parity PAR (canonical [26][N] doubles) into the
// entries that step reads: h its own, g the AA slots.
template <typename T, typename SH, typename SG, int PAR>
__global__ void __launch_bounds__(NTHREADS)
fused_restore_kernel(const Desc* __restrict__ descs, const Tile* __restrict__ tiles,
                     const double* __restrict__ pops) {
    constexpr int QP = QH;
    const Tile tl = load_tile(tiles);
    const Desc* D = descs + tl.lat;
    const int nx = uni(D->nx), ny = uni(D->ny), nz = uni(D->nz), TX = uni(D->tx);
    const int tx = threadIdx.x & (TX - 1), ty = threadIdx.x / TX;
    const int x = tl.x0 + tx, y = tl.y0 + ty;
    if (x >= nx || y >= ny) return;
    Phys<T> ph;
    ph.load(D);
    const int64_t N = uni(D->N);
    typedef Lay<SG, SG, 0> LAYT;
    const auto gb = pop_array<SG, QG, 0, LAYT>(D);
    const int nxp = uni(D->nxp), nxh = uni(D->nxh);
    SH* const h = (SH*)unip((char*)D->hb[PAR]);
    const uint8_t* __restrict__ flg = unip(D->flag);
    const uint32_t* __restrict__ lnk = unip(D->link);
    for (int k = 0; k < tl.zn; ++k) {
        const int z = tl.z0 + k;
        const int n = x + nx * (y + ny * z);
        const uint8_t f = flg[n];
        if (flag_kind(f) != KIND_FLUID) continue;
        const uint32_t solid = (f & F_NEAR_WALL) ? (lnk[n] & SOLID_MASK) : 0u;
        Nbr nb;
        nb.init<LAYT>(x, y, z, nx, ny, nz, nxp);
        SH* const own = h + (int64_t)QP * (nxh * ((int64_t)y + (int64_t)ny * z) + x / TX * TX) + x % TX;
        for (int i = 0; i < QP; ++i) own[i * TX] = (SH)(T)(pops[(int64_t)i * N + n] - wp<QP>(i) * D->href);
        T dg[QG];
        for (int i = 0; i < QG; ++i) dg[i] = (T)(pops[(int64_t)(QP + i) * N + n] - wg(i) * D->gref);
        place_pops<T, PAR>(gb, nb, solid, ph[PI_SG], dg);
    }
}

// ---------------------------------------------------------------- launchers
template <typename T, typename SH, typename SG, int TX, int PAR>
hipError_t launch_step_tp(bool back, int mode, Desc* d, const Tile* tiles, int ntiles, int diag, ReadOut ro, InitIn in,
                          hipStream_t s) {
    dim3 grid(ntiles), block(NTHREADS);
    switch (mode) {
        case MODE_STEP:
            if (diag) step_kernel<T, SH, SG, MODE_STEP, true, TX, PAR><<<grid, block, 0, s>>>(d, tiles, back, ro, in);
            else step_kernel<T, SH, SG, MODE_STEP, false, TX, PAR><<<grid, block, 0, s>>>(d, tiles, back, ro, in);
            break;
        case MODE_READ:
            step_kernel<T, SH, SG, MODE_READ, true, TX, PAR><<<grid, block, 0, s>>>(d, tiles, back, ro, in);
            break;
        case MODE_READ_MARCH:
            sweep_kernel<T, SH, SG, MODE_READ, true, TX, PAR, QH, false, true><<<grid, block, 0, s>>>(d, tiles, ro, in);
            break;
        case MODE_INIT:
            // (a lattice starts at step 0)
            if constexpr (PAR == 0) step_kernel<T, SH, SG, MODE_INIT, false, TX, 0><<<grid, block, 0, s>>>(d, tiles, back, ro, in);
            else return hipErrorInvalidValue;
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// back: the tile list backwards
template <typename T, typename SH, typename SG>
hipError_t launch_step(bool back, int mode, int tx, int parity, Desc* d, const Tile* tiles, int ntiles, int diag, ReadOut ro,
                       InitIn in, hipStream_t s) {
    switch (tx * 2 + (parity & 1)) {
        case 128: return launch_step_tp<T, SH, SG, 64, 0>(back, mode, d, tiles, ntiles, diag, ro, in, s);
        case 129: return launch_step_tp<T, SH, SG, 64, 1>(back, mode, d, tiles, ntiles, diag, ro, in, s);
        case 64: return launch_step_tp<T, SH, SG, 32, 0>(back, mode, d, tiles, ntiles, diag, ro, in, s);
        case 65: return launch_step_tp<T, SH, SG, 32, 1>(back, mode, d, tiles, ntiles, diag, ro, in, s);
        case 32: return launch_step_tp<T, SH, SG, 16, 0>(back, mode, d, tiles, ntiles, diag, ro, in, s);
        case 33: return launch_step_tp<T, SH, SG, 16, 1>(back, mode, d, tiles, ntiles, diag, ro, in, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace pflbm
