// fdtd_adj_pass.h -- the single-pass adjoint step for gfx950: the transposes
// of the H and of the E update of a domain in one launch, from adjoint set rs
// into set ws; then dJ/deps from the forward state, and the dispersive cells'
// histories, in launches of their own.
//
// What bounds it: HBM bytes.  The split pair reads both cotangent fields twice
// and passes U = S coef Ebar_pre through memory (21 field words per cell, and
// the gradient's); one pass reads and writes each once (12).  The dependences
// are those of the forward step, so the march is too (fdtd_pass.hip): per
// plane k a thread takes Hbar(k), forms the raw-difference cotangents of its
// H terms once (its own absorber memories only) and exchanges them with the
// nodes one step forward; Ebar(k) and the cotangents of its E terms follow,
// which the H nodes of plane k-1 collect from one step forward.
//
// Measured (us per step with the gradient, the split pair before): 101^3 f64
// with absorbers 142 -> 52; 160^3 f32 155 -> 102; 212^3 f32 327 -> 213; 256 x 256 x
// 280 f32 Bloch cell 640 -> 392; 280^3 f32 diagonal eps, all cells in the
// gradient 1045 -> 920 (of that the FP64 gradient 345, at 4.1 TB/s); 536^3 f32
// 3401 -> 2226.
//
// The arithmetic of every node is that of the split kernels, operation by
// operation, so both families give the same bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "fdtd_dev.h"
#include "fdtd_launch.h"
#include "fdtd_pass.h"

namespace fdtd {

namespace {

// LDS of a block: exchange buffers, and the absorber coefficients of its
// columns, rows and planes (from the plane below the first)
template <typename T, int V, int NT>
struct AdjLds {
    Grp<T, V> hxy[2][NT], hzy[2][NT];   // H terms along y: (Hx, 0), (Hz, 1)
    T hzx[2][NT], hyx[2][NT];           // along x, last node of the group: (Hz, 0), (Hy, 1)
    Grp<T, V> exy[2][NT], ezy[2][NT];   // E terms along y: (Ex, 0), (Ez, 1)
    T ezx[2][NT], eyx[2][NT];           // along x, first node of the group: (Ez, 0), (Ey, 1)
    T cx[6][kAdjMaxGroups * V];
    T cy[6][kPassMaxRows];
    T cz[6][kPassMaxPlanes + 2];
};

template <typename T, int V>
struct AdjCtx {
    Const<DomDev<T>>* d;
    const DomDev<T>* dg;         // the same, for the node code it shares with the split kernels
    TileMap<V> m;
    SlabMap<V> s;
    int tid, k0, k1, nz;
    bool seam;                   // the domain has a periodic axis
    unsigned vh, ve, vs, vp;     // byte offsets in a plane: H loads, E loads, stores; in a plane of the eps box
    bool inb[V];                 // node inside the eps box' x and y range
    int ez0, ez1;
    T S, bg;
    long long so, wo;            // offsets of the sets read and written (elements)
    T fl, fr, fd, fu;            // Bloch factors of the four neighbours (1 off a seam)
    bool lx[V];                  // node in the dispersive box' x and y range
    int lz0, lz1;                // its planes
};

// raw-difference cotangent of a term from ybar and its memory cotangent (tr_term of the split kernels)
template <typename T>
__device__ __forceinline__ T tr(bool in, T ki, T c, T psi, T ybar) {
    return in ? fma(ki, ybar, c * (psi + ybar)) : ybar;
}

// The march.  M: what the tile and its halo may meet (AdjMask); each variant
// keeps the registers of what it does not meet.  ND: eps^-1 and gradient
// arrays (1 isotropic, 3 diagonal).
template <typename T, int V, int NT, int M, int ND>
__device__ __forceinline__ void adj_march(const AdjCtx<T, V>& c, AdjLds<T, V, NT>& L) {
    using G = Grp<T, V>;
    constexpr bool X = M & kPassX, Y = M & kPassY, Z = M & kPassZ, PER = M & kAdjPer, LOR = M & kAdjLor;
    constexpr unsigned ts = sizeof(T);
    Const<DomDev<T>>& d = *c.d;
    const unsigned pbytes = (unsigned)(d.plane * (long long)ts);
    const long long pl = d.plane;
    // cotangent arrays lie fd elements apart in the order Ex Hx Ey Hy Ez Hz, as the forward ones
    const long long fd = d.Ha[0] - d.Ea[0], ed = ND > 1 ? d.epsinv[1] - d.epsinv[0] : 0;
    const long long epl = (long long)d.exs * (d.ehi[1] - d.elo[1]);
    const unsigned ebytes = (unsigned)(epl * (long long)ts);
    const T* rnext = uniform(d.Ea[0] + c.so + c.k0 * pl);                   // plane to fetch, set read
    const T* enext = uniform(d.epsinv[0] + (c.k0 - c.ez0) * epl);
    T* wcur = uniform(d.Ea[0] + c.wo + c.k0 * pl);                          // plane of the E nodes, set written
    const int nz = c.nz, tid = c.tid;
    const long long setd = (c.wo - c.so) * (long long)ts;          // from the read set to the written one
    const char *bx = nullptr, *by = nullptr, *bz = nullptr;        // absorber memories, read set
    unsigned sx = 0, sy = 0, sz = 0, zhi = 0, za0 = 0, za1 = 0, zpl = 0;
    if constexpr (X) {
        const PsiAxis p = psi_range<true>(d, 0);
        bx = p.base + c.so * (long long)ts;
        sx = p.span;
    }
    if constexpr (Y) {
        const PsiAxis p = psi_range<true>(d, 1);
        by = p.base + c.so * (long long)ts;
        sy = p.span;
    }
    if constexpr (Z) {
        const PsiAxis p = psi_range<true>(d, 2);
        bz = p.base + c.so * (long long)ts;
        sz = p.span;
        zhi = p.hi;
        za0 = p.a[0];
        za1 = p.a[1];
        zpl = (unsigned)(d.n[1] * d.ppx) * ts;
    }
    const T S = c.S, mS = -c.S;
    auto zslab = [&](int k) { return k < d.L[2][0] ? 0 : (k >= nz - d.L[2][1] && k < nz ? 1 : -1); };
    auto zoff = [&](int k, int s, int q) {   // offset of array q of side s at plane k
        const int kk = s ? k - (nz - d.L[2][1]) : k;
        return c.s.vz + (s ? zhi + (unsigned)q * za1 : (unsigned)q * za0) + (unsigned)kk * zpl;
    };
    // memory cotangents at plane k: H side (at every node of the tile), E side
    G pxe[2], pxh[2], pye[2], pyh[2], pze[2], pzh[2];
    auto mem = [&](int k, int h, G (&px)[2], G (&py)[2], G (&pz)[2]) {
        if (X && c.s.wx)
            for (int r = 0; r < 2; ++r)
                px[r] = ld_g<T, V>(make_rsrc(bx, sx), c.s.vx == kOob ? kOob : c.s.vx + k * c.s.dx + (2 * r + h) * c.s.ax);
        if (Y && c.s.wy)
            for (int r = 0; r < 2; ++r)
                py[r] = ld_g<T, V>(make_rsrc(by, sy), c.s.iny ? c.s.vy + k * c.s.dy + (2 * r + h) * c.s.ay : kOob);
        if constexpr (Z) {
            const int s = zslab(k);
            if (s >= 0)
                for (int r = 0; r < 2; ++r) pz[r] = ld_g<T, V>(make_rsrc(bz, sz), c.vh != kOob ? zoff(k, s, 2 * r + h) : kOob);
        }
    };
    G Hk[3], Pe[3], Ph[3], Pi[ND];
    G Cz, Dz;                                      // H terms along z of the plane below: (Hy, 0), (Hx, 1)
    G x0, x1, y0, y1, z0, z1;                      // E terms of the plane below: component, term
    for (int v = 0; v < V; ++v) {
        x0.v[v] = x1.v[v] = y0.v[v] = y1.v[v] = z0.v[v] = z1.v[v] = T(0);
        Cz.v[v] = Dz.v[v] = T(0);
        for (int q = 0; q < 3; ++q) Hk[q].v[v] = T(0);
    }
    {   // (no branches: they cost the plane pointers their scalar registers)
        const unsigned nb = c.k0 > 0 ? pbytes : 0u;
        const long long back = c.k0 > 0 ? pl : 0;
        const T* h = rnext + fd - back;
        Hk[0] = ld_g<T, V>(make_rsrc(h, nb), c.vh);
        Hk[1] = ld_g<T, V>(make_rsrc(h + 2 * fd, nb), c.vh);
        for (int v = 0; v < V; ++v) {
            Cz.v[v] = mS * Hk[1].v[v];
            Dz.v[v] = S * Hk[0].v[v];
        }
        if constexpr (Z) {
            const int s = c.k0 > 0 ? zslab(c.k0 - 1) : -1;
            for (int r = 0; r < 2; ++r)
                pzh[r] = ld_g<T, V>(make_rsrc(bz, s >= 0 ? sz : 0u), c.vh != kOob ? zoff(c.k0 - 1, s > 0, 2 * r + 1) : kOob);
            const T cc = L.cz[4][0], kk = L.cz[5][0];
            for (int v = 0; v < V; ++v) {
                Cz.v[v] = tr(s >= 0, kk, cc, pzh[0].v[v], Cz.v[v]);
                Dz.v[v] = tr(s >= 0, kk, cc, pzh[1].v[v], Dz.v[v]);
            }
        }
    }
    // (uniform(): a descriptor whose pointer or size the compiler keeps in
    // vector registers costs a loop over the lanes per access)
    auto fetch = [&](int k) {   // operands of plane k (zeros past the march and past the domain)
        const unsigned nb = uniform(k <= c.k1 && k < nz ? pbytes : 0u), ne = uniform(nb && k >= c.ez0 && k < c.ez1 ? ebytes : 0u);
        const T* f = uniform(rnext);
        for (int q = 0; q < 3; ++q) {
            Pe[q] = ld_g<T, V>(make_rsrc(f, nb), c.ve);
            f += fd;
            Ph[q] = ld_g<T, V>(make_rsrc(f, nb), c.vh);
            f += fd;
        }
        const T* e = uniform(enext);
        for (int q = 0; q < ND; ++q) {
            Pi[q] = ld_g<T, V>(make_rsrc(e, ne), c.vp);
            e += ed;
        }
        rnext += pl;
        enext += epl;
    };
    fetch(c.k0);
    if constexpr ((M & 7) != 0) {
        mem(c.k0, 1, pxh, pyh, pzh);
        mem(c.k0, 0, pxe, pye, pze);
    }
    int b = 0;
    for (int kn = c.k0; kn <= c.k1; ++kn, b ^= 1) {
        const bool first = kn > c.k0, last = kn == c.k1;
        G Hn[3], Eo[3], Ei[3];
        for (int q = 0; q < 3; ++q) {
            Hn[q] = Ph[q];
            Eo[q] = Pe[q];
        }
        const bool ekin = kn >= c.ez0 && kn < c.ez1;
        for (int q = 0; q < ND; ++q)
            for (int v = 0; v < V; ++v) Ei[q].v[v] = c.inb[v] && ekin ? Pi[q].v[v] : c.bg;
        for (int q = ND; q < 3; ++q) Ei[q] = Ei[0];
        // ---- H terms of plane kn: ybar = -S Hbar (term 0), S Hbar (term 1)
        const int sk = Z ? zslab(kn) : -1;
        G hxy, hzy, hzx, hyx, hyz, hxz;   // (Hx,0) y; (Hz,1) y; (Hz,0) x; (Hy,1) x; (Hy,0) z; (Hx,1) z
        for (int v = 0; v < V; ++v) {
            hxy.v[v] = mS * Hn[0].v[v];
            hzy.v[v] = S * Hn[2].v[v];
            hzx.v[v] = mS * Hn[2].v[v];
            hyx.v[v] = S * Hn[1].v[v];
            hyz.v[v] = mS * Hn[1].v[v];
            hxz.v[v] = S * Hn[0].v[v];
        }
        G n0, n1;                          // new memories
        if (Y && c.s.wy) {
            const T bb = L.cy[3][c.m.row], cc = L.cy[4][c.m.row], kk = L.cy[5][c.m.row];
            for (int v = 0; v < V; ++v) {
                n0.v[v] = bb * (pyh[0].v[v] + hxy.v[v]);
                n1.v[v] = bb * (pyh[1].v[v] + hzy.v[v]);
                hxy.v[v] = tr(c.s.iny, kk, cc, pyh[0].v[v], hxy.v[v]);
                hzy.v[v] = tr(c.s.iny, kk, cc, pyh[1].v[v], hzy.v[v]);
            }
            const unsigned o = c.s.iny && c.vs != kOob && !last ? c.s.vy + kn * c.s.dy + c.s.ay : kOob;
            st_g<T, V>(make_rsrc(by + setd, sy), o, n0);
            st_g<T, V>(make_rsrc(by + setd, sy), o == kOob ? kOob : o + 2 * c.s.ay, n1);
        }
        if (Z && sk >= 0) {
            const int z = kn - c.k0 + 1;
            const T bb = L.cz[3][z], cc = L.cz[4][z], kk = L.cz[5][z];
            for (int v = 0; v < V; ++v) {
                n0.v[v] = bb * (pzh[0].v[v] + hyz.v[v]);
                n1.v[v] = bb * (pzh[1].v[v] + hxz.v[v]);
                hyz.v[v] = tr(true, kk, cc, pzh[0].v[v], hyz.v[v]);
                hxz.v[v] = tr(true, kk, cc, pzh[1].v[v], hxz.v[v]);
            }
            const bool w = c.vs != kOob && !last;
            st_g<T, V>(make_rsrc(bz + setd, sz), w ? zoff(kn, sk, 1) : kOob, n0);
            st_g<T, V>(make_rsrc(bz + setd, sz), w ? zoff(kn, sk, 3) : kOob, n1);
        }
        if (X && c.s.wx) {
            for (int v = 0; v < V; ++v) {
                const int x = c.m.col * V + v;
                const T bb = L.cx[3][x], cc = L.cx[4][x], kk = L.cx[5][x];
                n0.v[v] = c.s.inx[v] ? bb * (pxh[0].v[v] + hzx.v[v]) : T(0);   // zeros beside the slab
                n1.v[v] = c.s.inx[v] ? bb * (pxh[1].v[v] + hyx.v[v]) : T(0);
                hzx.v[v] = tr(c.s.inx[v], kk, cc, pxh[0].v[v], hzx.v[v]);
                hyx.v[v] = tr(c.s.inx[v], kk, cc, pxh[1].v[v], hyx.v[v]);
            }
            const unsigned o = c.s.vx != kOob && c.vs != kOob && !last ? c.s.vx + kn * c.s.dx + c.s.ax : kOob;
            st_g<T, V>(make_rsrc(bx + setd, sx), o, n0);
            st_g<T, V>(make_rsrc(bx + setd, sx), o == kOob ? kOob : o + 2 * c.s.ax, n1);
        }
        L.hxy[b][tid] = hxy;
        L.hzy[b][tid] = hzy;
        L.hzx[b][tid] = hzx.v[V - 1];
        L.hyx[b][tid] = hyx.v[V - 1];
        if constexpr ((M & 7) != 0) mem(kn + 1, 1, pxh, pyh, pzh);
        fetch(kn + 1);
        lds_barrier();
        // ---- Ebar at plane kn: the terms of the node one step back less its own
        G hxd = L.hxy[b][c.m.id], hzd = L.hzy[b][c.m.id];
        T hzl = L.hzx[b][c.m.il], hyl = L.hyx[b][c.m.il];
        if constexpr (PER) {
            for (int v = 0; v < V; ++v) {
                hxd.v[v] = c.fd * hxd.v[v];
                hzd.v[v] = c.fd * hzd.v[v];
            }
            hzl = c.fl * hzl;
            hyl = c.fl * hyl;
        }
        if (c.m.wd)
            for (int v = 0; v < V; ++v) hxd.v[v] = hzd.v[v] = T(0);
        if (c.m.wl) hzl = hyl = T(0);
        const bool kwall = kn == 0 || kn >= nz;   // Ex, Ey held at zero there; no E past the last plane
        bool fx[V], fy[V], fz[V];
        for (int v = 0; v < V; ++v) {
            const bool xw = v == 0 && c.m.wl, out = (v > 0 && c.m.tail) || kn >= nz;
            fx[v] = !(c.m.wd || kwall || out);
            fy[v] = !(xw || kwall || out);
            fz[v] = !(xw || c.m.wd || out);
        }
        G En[3], U[3];
        for (int v = 0; v < V; ++v) {
            const T hzm = v ? hzx.v[v ? v - 1 : 0] : hzl, hym = v ? hyx.v[v ? v - 1 : 0] : hyl;
            T a = Eo[0].v[v];
            a += Cz.v[v] - hyz.v[v];
            a += hzd.v[v] - hzy.v[v];
            En[0].v[v] = fx[v] ? a : T(0);
            a = Eo[1].v[v];
            a += hzm - hzx.v[v];
            a += Dz.v[v] - hxz.v[v];
            En[1].v[v] = fy[v] ? a : T(0);
            a = Eo[2].v[v];
            a += hxd.v[v] - hxy.v[v];
            a += hym - hyx.v[v];
            En[2].v[v] = fz[v] ? a : T(0);
            for (int q = 0; q < 3; ++q) U[q].v[v] = S * Ei[q].v[v] * En[q].v[v];
            U[0].v[v] = fx[v] ? U[0].v[v] : T(0);
            U[1].v[v] = fy[v] ? U[1].v[v] : T(0);
            U[2].v[v] = fz[v] ? U[2].v[v] : T(0);
        }
        Cz = hyz;
        Dz = hxz;
        // a dispersive node: each pole's W^{n+1} roll feeds E^{n+1}; Ebar keeps
        // the cotangent before the source, which k_adj_lor takes further
        if constexpr (LOR) {
            if (kn >= c.lz0 && kn < c.lz1)
                for (int v = 0; v < V; ++v)
                    if (c.lx[v]) {
                        const long long q = lidx(*c.dg, c.m.i + v, c.m.j, kn) + c.so;
                        for (int e = 0; e < 3; ++e) {
                            T ep = En[e].v[v];
                            const FDTD_GLOBAL T* w = gp(c.dg->lora[1][e]) + q;
                            for (int p = 0; p < c.dg->npole; ++p) ep = fma(T(0.5) * c.dg->lg[p], w[p * c.dg->lbox], ep);
                            const T invden = T(1) / (T(1) / Ei[e].v[v] + T(0.25) * c.dg->lgs);
                            const bool f = e == 0 ? fx[v] : e == 1 ? fy[v] : fz[v];
                            En[e].v[v] = f ? ep : T(0);
                            U[e].v[v] = f ? S * invden * ep : T(0);
                        }
                    }
        }
        // ---- E terms of plane kn (ybar = U for term 0, -U for term 1), memory cotangents
        G nx0, nx1, ny0, ny1, nz0, nz1;
        for (int v = 0; v < V; ++v) {
            nx0.v[v] = U[0].v[v];
            nx1.v[v] = -U[0].v[v];
            ny0.v[v] = U[1].v[v];
            ny1.v[v] = -U[1].v[v];
            nz0.v[v] = U[2].v[v];
            nz1.v[v] = -U[2].v[v];
        }
        if (Y && c.s.wy) {
            const T bb = L.cy[0][c.m.row], cc = L.cy[1][c.m.row], kk = L.cy[2][c.m.row];
            for (int v = 0; v < V; ++v) {
                n0.v[v] = fx[v] ? bb * (pye[0].v[v] + nx0.v[v]) : T(0);
                n1.v[v] = fz[v] ? bb * (pye[1].v[v] + nz1.v[v]) : T(0);
                nx0.v[v] = fx[v] ? tr(c.s.iny, kk, cc, pye[0].v[v], nx0.v[v]) : T(0);
                nz1.v[v] = fz[v] ? tr(c.s.iny, kk, cc, pye[1].v[v], nz1.v[v]) : T(0);
            }
            const unsigned o = c.s.iny && c.vs != kOob && !last ? c.s.vy + kn * c.s.dy : kOob;
            st_g<T, V>(make_rsrc(by + setd, sy), o, n0);
            st_g<T, V>(make_rsrc(by + setd, sy), o == kOob ? kOob : o + 2 * c.s.ay, n1);
        }
        if (Z && sk >= 0) {
            const int z = kn - c.k0 + 1;
            const T bb = L.cz[0][z], cc = L.cz[1][z], kk = L.cz[2][z];
            for (int v = 0; v < V; ++v) {
                n0.v[v] = fy[v] ? bb * (pze[0].v[v] + ny0.v[v]) : T(0);
                n1.v[v] = fx[v] ? bb * (pze[1].v[v] + nx1.v[v]) : T(0);
                ny0.v[v] = fy[v] ? tr(true, kk, cc, pze[0].v[v], ny0.v[v]) : T(0);
                nx1.v[v] = fx[v] ? tr(true, kk, cc, pze[1].v[v], nx1.v[v]) : T(0);
            }
            const bool w = c.vs != kOob && !last;
            st_g<T, V>(make_rsrc(bz + setd, sz), w ? zoff(kn, sk, 0) : kOob, n0);
            st_g<T, V>(make_rsrc(bz + setd, sz), w ? zoff(kn, sk, 2) : kOob, n1);
        }
        if (X && c.s.wx) {
            for (int v = 0; v < V; ++v) {
                const int x = c.m.col * V + v;
                const T bb = L.cx[0][x], cc = L.cx[1][x], kk = L.cx[2][x];
                n0.v[v] = c.s.inx[v] && fz[v] ? bb * (pxe[0].v[v] + nz0.v[v]) : T(0);
                n1.v[v] = c.s.inx[v] && fy[v] ? bb * (pxe[1].v[v] + ny1.v[v]) : T(0);
                nz0.v[v] = fz[v] ? tr(c.s.inx[v], kk, cc, pxe[0].v[v], nz0.v[v]) : T(0);
                ny1.v[v] = fy[v] ? tr(c.s.inx[v], kk, cc, pxe[1].v[v], ny1.v[v]) : T(0);
            }
            const unsigned o = c.s.vx != kOob && c.vs != kOob && !last ? c.s.vx + kn * c.s.dx : kOob;
            st_g<T, V>(make_rsrc(bx + setd, sx), o, n0);
            st_g<T, V>(make_rsrc(bx + setd, sx), o == kOob ? kOob : o + 2 * c.s.ax, n1);
        }
        if constexpr ((M & 7) != 0) mem(kn + 1, 0, pxe, pye, pze);
        {
            const unsigned nb = uniform(last ? 0u : pbytes);
            const T* f = uniform(wcur);
            for (int q = 0; q < 3; ++q) {
                st_g<T, V>(make_rsrc(f, nb), c.vs, En[q]);
                f += 2 * fd;
            }
        }
        // ---- Hbar at plane kn - 1: its own terms less those of the node one step forward
        G xyu = L.exy[b ^ 1][c.m.iu], zyu = L.ezy[b ^ 1][c.m.iu];
        T zxr = L.ezx[b ^ 1][c.m.ir], yxr = L.eyx[b ^ 1][c.m.ir];
        if constexpr (PER) {
            for (int v = 0; v < V; ++v) {
                xyu.v[v] = c.fu * xyu.v[v];
                zyu.v[v] = c.fu * zyu.v[v];
            }
            zxr = c.fr * zxr;
            yxr = c.fr * yxr;
        }
        if (c.m.wu)
            for (int v = 0; v < V; ++v) xyu.v[v] = zyu.v[v] = T(0);
        if (c.m.wr) zxr = yxr = T(0);
        G Hw[3];
        for (int v = 0; v < V; ++v) {
            const T zr = v + 1 < V ? z0.v[v + 1 < V ? v + 1 : v] : zxr, yr = v + 1 < V ? y1.v[v + 1 < V ? v + 1 : v] : yxr;
            const T p[3] = {y0.v[v] - ny0.v[v], z0.v[v] - zr, x0.v[v] - xyu.v[v]};
            const T r[3] = {z1.v[v] - zyu.v[v], x1.v[v] - nx1.v[v], y1.v[v] - yr};
            // (the order of the sum is that of the split kernels of either kind of domain)
            for (int q = 0; q < 3; ++q) Hw[q].v[v] = c.seam ? (Hk[q].v[v] + p[q]) + r[q] : Hk[q].v[v] + (p[q] + r[q]);
        }
        {
            const unsigned nb = uniform(first ? pbytes : 0u);
            const T* f = uniform(wcur + fd - (first ? pl : 0));
            for (int q = 0; q < 3; ++q) {
                st_g<T, V>(make_rsrc(f, nb), c.vs, Hw[q]);
                f += 2 * fd;
            }
        }
        wcur += pl;
        L.exy[b][tid] = nx0;
        L.ezy[b][tid] = nz1;
        L.ezx[b][tid] = nz0.v[0];
        L.eyx[b][tid] = ny1.v[0];
        for (int q = 0; q < 3; ++q) Hk[q] = Hn[q];
        x0 = nx0;
        x1 = nx1;
        y0 = ny0;
        y1 = ny1;
        z0 = nz0;
        z1 = nz1;
    }
}

// One tile: a function of its own per variant (not inlined), so that the lean
// variants do not inherit the spills and scalar pressure of the others.
template <typename T, int V, int NT, int M, int ND>
__device__ __attribute__((noinline, noreturn)) void adj_tile(const DomDev<T>* doms_, const int4* tab_, int rs_, int ws_) {
    extern __shared__ __align__(16) char smem[];
    AdjLds<T, V, NT>& L = *(AdjLds<T, V, NT>*)smem;
    const DomDev<T>* doms = uniform(doms_);
    Const<int4>* tab = as_const(uniform(tab_));
    const int rs = uniform(rs_), ws = uniform(ws_);
    const int dom = tab[2 * blockIdx.x].x, q0 = tab[2 * blockIdx.x].z, q1 = tab[2 * blockIdx.x].w;
    const int y0 = tab[2 * blockIdx.x + 1].x, y1 = tab[2 * blockIdx.x + 1].y;
    Const<DomDev<T>>& d = as_const(doms)[dom];
    AdjCtx<T, V> c;
    c.d = &d;
    c.dg = doms + dom;
    const int nx = d.n[0], ny = d.n[1], nz = c.nz = d.n[2];
    const bool perx = d.per[0], pery = d.per[1];
    c.k0 = tab[2 * blockIdx.x + 1].z;
    c.k1 = tab[2 * blockIdx.x + 1].w;
    const int tid = c.tid = threadIdx.x;
    c.m = map_tile<T, V, (M & kPassX) != 0>(d, tid, q0, q1, y0, y1);
    const int i = c.m.i, j = c.m.j, wt = c.m.wt, rt = c.m.rt;
    c.vh = c.m.act ? c.m.f : kOob;
    c.ve = c.m.has_e ? c.m.f : kOob;
    c.vs = c.m.own ? c.m.f : kOob;
    bool any = false;
    for (int v = 0; v < V; ++v) {
        c.inb[v] = c.m.has_e && i + v >= d.elo[0] && i + v < d.ehi[0] && j >= d.elo[1] && j < d.ehi[1];
        any |= c.inb[v];
    }
    c.vp = any ? ((unsigned)(j - d.elo[1]) * (unsigned)d.exs + (unsigned)(i - d.exa)) * (unsigned)sizeof(T) : kOob;
    c.ez0 = d.elo[2];
    c.ez1 = d.ehi[2];
    c.S = d.S;
    c.bg = d.epsinv_bg;
    c.so = (long long)rs * d.as;
    c.wo = (long long)ws * d.as;
    c.seam = perx || pery;
    if constexpr (M & kAdjPer) {
        c.fl = perx && i == 0 ? d.bsign[0] : T(1);
        c.fr = perx && i + V >= nx ? d.bsign[0] : T(1);
        c.fd = pery && j == 0 ? d.bsign[1] : T(1);
        c.fu = pery && j == ny - 1 ? d.bsign[1] : T(1);
    }
    if constexpr (M & kAdjLor) {
        for (int v = 0; v < V; ++v)
            c.lx[v] = c.m.has_e && d.has_lor && i + v >= d.llo[0] && i + v < d.lhi[0] && j >= d.llo[1] && j < d.lhi[1];
        c.lz0 = d.has_lor ? d.llo[2] : 0;
        c.lz1 = d.has_lor ? d.lhi[2] : 0;
    }
    if constexpr ((M & 7) != 0) {
        c.s = map_slabs<T, V, true>(d, c.m, c.m.act);
        if constexpr (M & kPassX)
            for (int s = tid; s < 6 * wt * V; s += NT) {
                const int tb = s / (wt * V), x = s - tb * (wt * V);
                const int gx = (q0 - c.m.hl) * V + x;
                L.cx[tb][x] = gx >= 0 && gx < nx ? gp(d.tab[0])[tb * nx + gx] : T(0);
            }
        if constexpr (M & kPassY)
            for (int s = tid; s < 6 * rt; s += NT) {
                const int tb = s / rt, r = s - tb * rt, gy = y0 - c.m.hb + r;
                L.cy[tb][r] = gy >= 0 && gy < ny ? gp(d.tab[1])[tb * ny + gy] : T(0);
            }
        if constexpr (M & kPassZ) {
            const int nzc = c.k1 - c.k0 + 2;
            for (int s = tid; s < 6 * nzc; s += NT) {
                const int tb = s / nzc, r = s - tb * nzc, gz = c.k0 - 1 + r;
                L.cz[tb][r] = gz >= 0 && gz < nz ? gp(d.tab[2])[tb * nz + gz] : T(0);
            }
        }
        __syncthreads();
    }
    adj_march<T, V, NT, M, ND>(c, L);
    __builtin_amdgcn_endpgm();
}

template <typename T, int V, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_adj_pass(const DomDev<T>* __restrict__ doms, const int4* __restrict__ tab, int rs, int ws) {
    const int4 ta = tab[2 * blockIdx.x];
    if (ta.x < 0) return;
    const DomDev<T>& d = doms[ta.x];
    auto go = [&](auto m) {
        constexpr int MM = decltype(m)::value;
        if (d.eps_diag) adj_tile<T, V, NT, MM, 3>(doms, tab, rs, ws);
        else adj_tile<T, V, NT, MM, 1>(doms, tab, rs, ws);
    };
#define FDTD_ADJ_CASE(M) \
    case (M): go(std::integral_constant<int, (M)>{}); break
    switch (ta.y) {
    FDTD_ADJ_CASE(0);
    FDTD_ADJ_CASE(1);
    FDTD_ADJ_CASE(2);
    FDTD_ADJ_CASE(3);
    FDTD_ADJ_CASE(4);
    FDTD_ADJ_CASE(5);
    FDTD_ADJ_CASE(6);
    FDTD_ADJ_CASE(7);
    FDTD_ADJ_CASE(kAdjPer | kPassZ);
    FDTD_ADJ_CASE(kAdjLor);
    default: go(std::integral_constant<int, kAdjAll>{}); break;
    }
#undef FDTD_ADJ_CASE
}

// dJ/deps of the gradient box from the stored Ebar (set ws; before the source
// in dispersive cells) and the forward state (set fsr).  A launch of its own:
// inside the march it took the registers of the prefetch (spills), and cost more
// than the one more read of Ebar here.  One thread per column of kz planes; the plane below is carried.
// spread: deal the blocks to the XCDs in turn instead of in runs, for domains with a dispersive box, whose
// costlier blocks lie side by side (256^3 f32, a box of 96 cells, 16 poles: a step 1835 -> 1630 us by it).
template <typename T>
__global__ void __launch_bounds__(256) k_adj_grad(const DomDev<T>* __restrict__ doms, const int* __restrict__ gbs, int ndom, int kz,
                                                  int ws, int fsr, int spread) {
    const int nb = gbs[ndom], blk = spread ? (int)blockIdx.x : xcd_remap(blockIdx.x, gridDim.x);
    if (blk >= nb) return;
    const int dom = find_domain(gbs, ndom, blk);
    const DomDev<T>& d = doms[dom];
    const int gw = d.ghi[0] - d.glo[0], gh = d.ghi[1] - d.glo[1];
    const int per = (gw * gh + 255) / 256, b = blk - gbs[dom];   // blocks per chunk of planes
    const int r = b % per * 256 + threadIdx.x;
    if (r >= gw * gh) return;
    const int j = d.glo[1] + r / gw, i = d.glo[0] + r % gw;
    const int k0 = d.glo[2] + b / per * kz, k1 = min(k0 + kz, d.ghi[2]);
    const long long wo = (long long)ws * d.as, fo = (long long)fsr * d.fs, pl = d.plane;
    const FDTD_GLOBAL T *hx = gp(d.H[0]) + fo, *hy = gp(d.H[1]) + fo, *hz = gp(d.H[2]) + fo;
    const T S = d.S;
    const bool xs = slab_side(d, 0, i) >= 0 || slab_side(d, 1, j) >= 0;
    const bool xl = d.has_lor && i >= d.llo[0] && i < d.lhi[0] && j >= d.llo[1] && j < d.lhi[1];
    long long f = fidx(d, i, j, k0);
    T xk = T(0), yk = T(0);   // forward Hx, Hy of the plane below
    if (k0 > 0) {
        xk = hx[f - pl];
        yk = hy[f - pl];
    }
#pragma unroll 2
    for (int k = k0; k < k1; ++k, f += pl) {
        const T x = hx[f], y = hy[f], z = hz[f];
        const T zy = nb_back(d, hz, f, 1, j), xy = nb_back(d, hx, f, 1, j);
        const T zx = nb_back(d, hz, f, 0, i), yx = nb_back(d, hy, f, 0, i);
        const T e[3] = {gp(d.Ea[0])[f + wo], gp(d.Ea[1])[f + wo], gp(d.Ea[2])[f + wo]};
        double g[3] = {0, 0, 0};
        if (xs || slab_side(d, 2, k) >= 0 || (xl && k >= d.llo[2] && k < d.lhi[2])) {
            if (!e_masked_d(d, 0, i, j, k)) g[0] = grad_term(d, 0, i, j, k, f, e[0], z, zy, y, yk, fsr);
            if (!e_masked_d(d, 1, i, j, k)) g[1] = grad_term(d, 1, i, j, k, f, e[1], x, xk, z, zx, fsr);
            if (!e_masked_d(d, 2, i, j, k)) g[2] = grad_term(d, 2, i, j, k, f, e[2], y, yx, x, xy, fsr);
        } else {
            const T c[3] = {(z - zy) - (y - yk), (x - xk) - (z - zx), (y - yx) - (x - xy)};
            for (int q = 0; q < 3; ++q) {
                const T ei = epsinv_at(d, q, i, j, k);
                if (!e_masked_d(d, q, i, j, k)) g[q] = -(double)e[q] * (double)(S * ei * ei * c[q]);
            }
        }
        grad_store(d, i, j, k, g);
        xk = x;
        yk = y;
    }
}

// The E-update transpose of the dispersive cells beyond the cotangent before
// the source (in set ws): the histories' transposes and Ebar^n (et_node's
// recursion).  One thread per cell and component.
template <typename T>
__global__ void __launch_bounds__(256) k_adj_lor(const DomDev<T>* __restrict__ doms, const int* __restrict__ lbs, int ndom, int rs,
                                                 int ws) {
    const int dom = find_domain(lbs, ndom, blockIdx.x);
    const DomDev<T>& d = doms[dom];
    const long long q = (long long)(blockIdx.x - lbs[dom]) * 256 + threadIdx.x;
    const int c = blockIdx.y;
    if (!d.apass || q >= d.lbox) return;
    const int bx = d.lhi[0] - d.llo[0], by = d.lhi[1] - d.llo[1];
    const int i = d.llo[0] + (int)(q % bx), j = d.llo[1] + (int)(q / bx % by), k = d.llo[2] + (int)(q / ((long long)bx * by));
    const long long ro = (long long)rs * d.as, wo = (long long)ws * d.as;
    if (e_masked_d(d, c, i, j, k)) {
        gp(d.lora[0][c])[q + wo] = T(0);
        for (int p = 0; p < d.npole; ++p) gp(d.lora[1][c])[q + p * d.lbox + wo] = gp(d.lora[2][c])[q + p * d.lbox + wo] = T(0);
        return;
    }
    const long long f = fidx(d, i, j, k) + wo;
    const T einf = T(1) / epsinv_at(d, c, i, j, k);
    const T invden = T(1) / (einf + T(0.25) * d.lgs);
    const T s = gp(d.Ea[c])[f] * invden;
    gp(d.Ea[c])[f] = fma(einf, s, gp(d.lora[0][c])[q + ro]);
    T enm1 = T(0);
    for (int p = 0; p < d.npole; ++p) {
        const long long o = q + p * d.lbox;
        const T wb = gp(d.lora[1][c])[o + ro], wob = gp(d.lora[2][c])[o + ro];
        T wn = fma(d.lal[p], wb, wob);
        T wnm1 = d.lxi[p] * wb;
        enm1 = p == 0 ? -T(0.5) * d.lg[0] * wb : fma(-T(0.5) * d.lg[p], wb, enm1);
        wn = fma(-T(0.5) * (T(1) + d.lal[p]), s, wn);
        wnm1 = fma(-T(0.5) * d.lxi[p], s, wnm1);
        gp(d.lora[1][c])[o + wo] = wn;
        gp(d.lora[2][c])[o + wo] = wnm1;
    }
    gp(d.lora[0][c])[q + wo] = fma(T(0.25) * d.lgs, s, enm1);
}

}  // namespace

template <typename T>
void launch_adj_pass(const LaunchCfg& c, const void* doms, int rs, int ws, hipStream_t s) {
    constexpr int V = kPassGroup<T>;
    const DomDev<T>* dd = (const DomDev<T>*)doms;
    if (c.ant == 512)
        hipLaunchKernelGGL((k_adj_pass<T, V, 512>), dim3(c.agrid), dim3(512), sizeof(AdjLds<T, V, 512>), s, dd, c.atab, rs, ws);
    else
        hipLaunchKernelGGL((k_adj_pass<T, V, 256>), dim3(c.agrid), dim3(256), sizeof(AdjLds<T, V, 256>), s, dd, c.atab, rs, ws);
}

template <typename T>
void launch_adj_grad(const LaunchCfg& c, const void* doms, int rs, int ws, int fsr, hipStream_t s) {
    const DomDev<T>* dd = (const DomDev<T>*)doms;
    if (c.ngrad) hipLaunchKernelGGL(k_adj_grad<T>, dim3(c.ngrad), dim3(256), 0, s, dd, c.gbs, c.ndom, c.gkz, ws, fsr,
                                    c.nalor ? 1 : 0);
    if (c.nalor) hipLaunchKernelGGL(k_adj_lor<T>, dim3(c.nlor, 3), dim3(256), 0, s, dd, c.lbs, c.ndom, rs, ws);
}

}  // namespace fdtd
