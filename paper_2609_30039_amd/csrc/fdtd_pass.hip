// fdtd_pass.hip -- the single-pass forward step for gfx950: E^{n+1} and
// H^{n+3/2} of a domain in one launch, from state set rs into set ws.
//
// What bounds it: HBM bytes.  The split pair reads the fields twice (21 field
// words per cell); one pass reads and writes each once (12).  A block covers
// a tile of column groups by rows and marches z; every thread owns a group of
// V neighbouring x nodes (8 bytes: one dwordx2 per array and plane).  Per
// plane k a thread holds H(k) and H(k-1), computes E^{n+1}(k), then
// H^{n+3/2}(k-1).  Neighbours come from LDS (H(k) one row and one column
// back, E^{n+1}(k-1) one row and one column forward; double buffers, one
// barrier per plane) and the tile carries a halo of one row and one column
// group on each inner side: the low ones supply H, the high ones recompute
// E^{n+1}.  The next plane's loads are issued before the barrier, so a plane
// of loads is in flight while one is computed.
//
// All field traffic goes through buffer descriptors of one plane: lanes
// outside the domain, halo lanes of a store and planes past the end get an
// offset (or a descriptor) out of range, for which the hardware returns zero
// and drops the store.  The loop has no branches around memory operations, so
// the compiler's waits on the prefetched loads do not wait for later stores.
//
// Measured (us per step, captured chunks, the split pair before): 32^3 f64 box
// 20.6 -> 6.2; 70 x 87 x 123 f64 with absorbers and 3 poles 65 -> 41; 148^3
// f32 with absorbers and a pole 88 -> 60; 212^3 f32 with absorbers 237 -> 187;
// 256 x 256 x 280 f32 Bloch cell 387 -> 283; 536^3 f32 diagonal eps 2717 ->
// 2133 in a closed box (4.4 TB/s of the 9.2 GB it must move; a copy of 4 GiB
// reaches 4.9), 3033 -> 2450 with absorbers, 3194 -> 2716 with a dispersive
// box too.  What remains over the floor is the absorbers: their waves carry
// more loads, stores and instructions per plane, and the block waits for them.
//
// The arithmetic of every node is that of the split kernels, operation by
// operation, so both families give the same bits.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "fdtd_dev.h"
#include "fdtd_launch.h"
#include "fdtd_pass.h"

namespace fdtd {

namespace {

// A group of the dispersive histories, whose rows are not aligned to groups: a
// load may take one node before or after the box (inside the state set, which
// is padded for it, and not used); a store writes the nodes in[v] only.
template <typename T, int V>
__device__ __forceinline__ Grp<T, V> ld_u(const T* p) {
    if constexpr (V == 1) {
        return Grp<T, V>{{gp(p)[0]}};
    } else {
        typedef T U __attribute__((ext_vector_type(2), aligned(sizeof(T))));
        const U u = *(const FDTD_GLOBAL U*)p;
        return Grp<T, V>{{u.x, u.y}};
    }
}

template <typename T, int V>
__device__ __forceinline__ void st_u(T* p, Grp<T, V> x, const bool (&in)[V]) {
    bool all = true;
    for (int v = 0; v < V; ++v) all = all && in[v];
    if constexpr (V == 2) {
        typedef T U __attribute__((ext_vector_type(2), aligned(sizeof(T))));
        if (all) {
            *(FDTD_GLOBAL U*)p = U{x.v[0], x.v[1]};
            return;
        }
    }
    for (int v = 0; v < V; ++v)
        if (in[v]) gp(p)[v] = x.v[v];
}

// LDS of a block: exchange buffers, and the absorber coefficients of its
// columns, rows and planes (tables bE cE kiE bH cH kiH)
template <typename T, int V, int NT>
struct PassLds {
    Grp<T, V> hx[2][NT], hz[2][NT];
    T hy[2][NT];                      // last node of the group
    Grp<T, V> ex[2][NT], ez[2][NT];
    T ey[2][NT];                      // first node of the group
    T cx[6][kPassMaxGroups * V];
    T cy[6][kPassMaxRows];
    T cz[6][kPassMaxPlanes + 1];
};

// the absorber recursion of one term (as st_pref in the split kernels): in
// the slab psi <- b psi + c D and D -> ki D + psi, outside it D unchanged
template <typename T>
__device__ __forceinline__ T slab_term(bool in, T b, T c, T ki, T psi, T D, T& pn) {
    pn = fma(b, psi, c * D);
    return in ? fma(ki, D, pn) : D;
}

// What the march needs, fixed per block or per thread.
template <typename T, int V>
struct PassCtx {
    Const<DomDev<T>>* d;
    int tid, row, col, i, j, k0, k1, nz;
    int il, ir, id, iu;          // threads of the neighbouring groups: left, right, row below, row above
    bool wl, wr, wd, wu;         // the neighbour past a wall: left, right, row below, row above
    bool tail;                   // the group's last node lies past nx
    unsigned vh, ve, vs;         // byte offsets in a plane: H loads, E loads, stores
    unsigned vp;                 // in a plane of the eps box
    bool inb[V];                 // node inside the eps box' x and y range
    int ez0, ez1;
    T S, bg;
    long long so, wo;            // set offsets (elements)
    int t, slot;
    bool own;
    // planes k0 + bit with sources, plane-monitor samples and probes
    unsigned long long src_planes, smp_planes, prb_planes;
    T fl, fr, fd, fu;            // Bloch factors of the four neighbours (1 off a seam)
    bool inx[V], iny;            // node in an x slab; thread in a y slab
    unsigned vx, dx, ax, vy, dy, ay, vz;   // memory offsets at plane 0, per plane, per array
    bool wx, wy;                 // some thread of the wave is in an x slab, a y slab
    bool lx[V];                  // node in the dispersive box' x and y range
    int lz0, lz1;                // its planes
};

// The march.  M: what the tile and its halo may meet (PassMask); each variant
// keeps the registers of what it does not meet.  The absorber memories of the
// next plane are fetched right after the last use of this plane's.  ND: eps^-1 arrays (1 isotropic, 3 diagonal).
template <typename T, int V, int NT, int M, int ND>
__device__ __forceinline__ void pass_march(const PassCtx<T, V>& c, PassLds<T, V, NT>& L) {
    using G = Grp<T, V>;
    constexpr bool X = M & kPassX, Y = M & kPassY, Z = M & kPassZ, MIX = M & kPassMix;
    constexpr unsigned ts = sizeof(T);
    Const<DomDev<T>>& d = *c.d;
    const unsigned pbytes = (unsigned)(d.plane * (long long)ts);
    const long long pl = d.plane;
    // the six field arrays of a set lie fd elements apart in the order Ex Hx Ey
    // Hy Ez Hz, the eps^-1 arrays ed apart: one base each, stepped plane by
    // plane, keeps the scalar registers (a descriptor is four) within their file
    const long long fd = d.H[0] - d.E[0], ed = ND > 1 ? d.epsinv[1] - d.epsinv[0] : 0;
    const long long epl = (long long)d.exs * (d.ehi[1] - d.elo[1]);
    const unsigned ebytes = (unsigned)(epl * (long long)ts);
    const T* rnext = d.E[0] + c.so + c.k0 * pl;                    // plane to fetch, set read
    const T* enext = d.epsinv[0] + (c.k0 - c.ez0) * epl;
    T* wcur = d.E[0] + c.wo + c.k0 * pl;                           // plane of the E update, set written
    const int nz = c.nz, tid = c.tid;
    const long long setd = (c.wo - c.so) * (long long)ts;          // from the read set to the written one
    const char *bx = nullptr, *by = nullptr, *bz = nullptr;        // absorber memories, read set
    unsigned sx = 0, sy = 0, sz = 0, zhi = 0, za0 = 0, za1 = 0, zpl = 0;
    if constexpr (X) {
        const PsiAxis p = psi_range<false>(d, 0);
        bx = p.base + c.so * (long long)ts;
        sx = p.span;
    }
    if constexpr (Y) {
        const PsiAxis p = psi_range<false>(d, 1);
        by = p.base + c.so * (long long)ts;
        sy = p.span;
    }
    if constexpr (Z) {
        const PsiAxis p = psi_range<false>(d, 2);
        bz = p.base + c.so * (long long)ts;
        sz = p.span;
        zhi = p.hi;
        za0 = p.a[0];
        za1 = p.a[1];
        zpl = (unsigned)(d.n[1] * d.ppx) * ts;
    }
    G Hk[3], Ek[3], Ph[3], Pe[3], Pi[ND];
    for (int q = 0; q < 3; ++q)
        for (int v = 0; v < V; ++v) Hk[q].v[v] = Ek[q].v[v] = T(0);
    {
        const unsigned nb = c.k0 > 0 ? pbytes : 0u;
        const T* h = rnext + fd - (c.k0 > 0 ? pl : 0);
        Hk[0] = ld_g<T, V>(make_rsrc(h, nb), c.vh);
        Hk[1] = ld_g<T, V>(make_rsrc(h + 2 * fd, nb), c.vh);
    }
    auto fetch = [&](int k) {   // operands of plane k (zeros past the march and past the domain)
        const unsigned nb = k <= c.k1 && k < nz ? pbytes : 0u, ne = nb && k >= c.ez0 && k < c.ez1 ? ebytes : 0u;
        const T* f = rnext;
        for (int q = 0; q < 3; ++q) {
            Pe[q] = ld_g<T, V>(make_rsrc(f, nb), c.ve);
            f += fd;
            Ph[q] = ld_g<T, V>(make_rsrc(f, nb), c.vh);
            f += fd;
        }
        const T* e = enext;
        for (int q = 0; q < ND; ++q) {
            Pi[q] = ld_g<T, V>(make_rsrc(e, ne), c.vp);
            e += ed;
        }
        rnext += pl;
        enext += epl;
    };
    // absorber memories of the E update of plane k and of the H update of plane k
    G pxe[2], pxh[2], pye[2], pyh[2], pze[2], pzh[2];
    auto zslab = [&](int k) { return k < d.L[2][0] ? 0 : (k >= nz - d.L[2][1] && k < nz ? 1 : -1); };
    auto zoff = [&](int k, int s, int q) {   // offset of array q of side s at plane k
        const int kk = s ? k - (nz - d.L[2][1]) : k;
        return c.vz + (s ? zhi + (unsigned)q * za1 : (unsigned)q * za0) + (unsigned)kk * zpl;
    };
    auto mem_e = [&](int k) {
        if (X && c.wx)
            for (int r = 0; r < 2; ++r) pxe[r] = ld_g<T, V>(make_rsrc(bx, sx), c.vx == kOob ? kOob : c.vx + k * c.dx + 2 * r * c.ax);
        if (Y && c.wy)
            for (int r = 0; r < 2; ++r) pye[r] = ld_g<T, V>(make_rsrc(by, sy), c.iny ? c.vy + k * c.dy + 2 * r * c.ay : kOob);
        if constexpr (Z) {
            const int s = zslab(k);
            if (s >= 0)
                for (int r = 0; r < 2; ++r) pze[r] = ld_g<T, V>(make_rsrc(bz, sz), c.ve != kOob ? zoff(k, s, 2 * r) : kOob);
        }
    };
    auto mem_h = [&](int k) {
        if (X && c.wx)
            for (int r = 0; r < 2; ++r) pxh[r] = ld_g<T, V>(make_rsrc(bx, sx), c.vx == kOob ? kOob : c.vx + k * c.dx + (2 * r + 1) * c.ax);
        if (Y && c.wy)
            for (int r = 0; r < 2; ++r) pyh[r] = ld_g<T, V>(make_rsrc(by, sy), c.iny ? c.vy + k * c.dy + (2 * r + 1) * c.ay : kOob);
        if constexpr (Z) {
            const int s = k >= c.k0 ? zslab(k) : -1;
            if (s >= 0)
                for (int r = 0; r < 2; ++r) pzh[r] = ld_g<T, V>(make_rsrc(bz, sz), c.vs != kOob ? zoff(k, s, 2 * r + 1) : kOob);
        }
    };
    fetch(c.k0);
    if constexpr (M != 0) {
        mem_e(c.k0);
        mem_h(c.k0 - 1);
    }
    int b = 0;
    for (int kn = c.k0; kn <= c.k1; ++kn, b ^= 1) {
        const int kp = kn - 1;
        G Hn[3], Eo[3], Ei[3];
        for (int q = 0; q < 3; ++q) {
            Hn[q] = Ph[q];
            Eo[q] = Pe[q];
        }
        const bool ekin = kn >= c.ez0 && kn < c.ez1;
        for (int q = 0; q < ND; ++q)
            for (int v = 0; v < V; ++v) Ei[q].v[v] = c.inb[v] && ekin ? Pi[q].v[v] : c.bg;
        for (int q = ND; q < 3; ++q) Ei[q] = Ei[0];
        L.hx[b][tid] = Hn[0];
        L.hz[b][tid] = Hn[2];
        L.hy[b][tid] = Hn[1].v[V - 1];
        fetch(kn + 1);
        lds_barrier();
        // ---- E^{n+1} at plane kn
        G hxd = L.hx[b][c.id], hzd = L.hz[b][c.id];
        T hyl = L.hy[b][c.il], hzl = L.hz[b][c.il].v[V - 1];
        if constexpr (MIX) {
            for (int v = 0; v < V; ++v) {
                hxd.v[v] = c.fd * hxd.v[v];
                hzd.v[v] = c.fd * hzd.v[v];
            }
            hyl = c.fl * hyl;
            hzl = c.fl * hzl;
        }
        if (c.wd)
            for (int v = 0; v < V; ++v) hxd.v[v] = hzd.v[v] = T(0);
        if (c.wl) hyl = hzl = T(0);
        const bool kwall = kn == 0 || kn >= nz;   // Ex, Ey held at zero there; no E past the last plane
        const bool first = kn > c.k0, last = kn == c.k1;
        const int sze = Z ? zslab(kn) : -1;
        G En[3], cu[3];
        G n0, n1;                                  // new memories
        bool fx[V], fy[V], fz[V];
        for (int v = 0; v < V; ++v) {
            const bool xw = v == 0 && c.wl, out = (v > 0 && c.tail) || kn >= nz;
            fx[v] = !(c.wd || kwall || out);
            fy[v] = !(xw || kwall || out);
            fz[v] = !(xw || c.wd || out);
        }
        G Dx0, Dx1, Dy0, Dy1, Dz0, Dz1;
        for (int v = 0; v < V; ++v) {
            const T hx = Hn[0].v[v], hy = Hn[1].v[v], hz = Hn[2].v[v];
            const T hyx = v ? Hn[1].v[v ? v - 1 : 0] : hyl, hzx = v ? Hn[2].v[v ? v - 1 : 0] : hzl;
            Dx0.v[v] = hz - hzd.v[v], Dx1.v[v] = hy - Hk[1].v[v];   // Ex: Hz along y, Hy along z
            Dy0.v[v] = hx - Hk[0].v[v], Dy1.v[v] = hz - hzx;        // Ey: Hx along z, Hz along x
            Dz0.v[v] = hy - hyx, Dz1.v[v] = hx - hxd.v[v];          // Ez: Hy along x, Hx along y
        }
        if (Y && c.wy) {
            const T bb = L.cy[0][c.row], cc = L.cy[1][c.row], kk = L.cy[2][c.row];
            for (int v = 0; v < V; ++v) {
                T p0, p1;
                Dx0.v[v] = slab_term(c.iny, bb, cc, kk, pye[0].v[v], Dx0.v[v], p0);
                Dz1.v[v] = slab_term(c.iny, bb, cc, kk, pye[1].v[v], Dz1.v[v], p1);
                n0.v[v] = fx[v] ? p0 : T(0);
                n1.v[v] = fz[v] ? p1 : T(0);
            }
            const unsigned o = c.iny && c.vs != kOob && !last ? c.vy + kn * c.dy : kOob;
            st_g<T, V>(make_rsrc(by + setd, sy), o, n0);
            st_g<T, V>(make_rsrc(by + setd, sy), o == kOob ? kOob : o + 2 * c.ay, n1);
        }
        if (Z && sze >= 0) {
            const T bb = L.cz[0][kn - c.k0], cc = L.cz[1][kn - c.k0], kk = L.cz[2][kn - c.k0];
            for (int v = 0; v < V; ++v) {
                T p0, p1;
                Dy0.v[v] = slab_term(true, bb, cc, kk, pze[0].v[v], Dy0.v[v], p0);
                Dx1.v[v] = slab_term(true, bb, cc, kk, pze[1].v[v], Dx1.v[v], p1);
                n0.v[v] = fy[v] ? p0 : T(0);
                n1.v[v] = fx[v] ? p1 : T(0);
            }
            const bool w = c.vs != kOob && !last;
            st_g<T, V>(make_rsrc(bz + setd, sz), w ? zoff(kn, sze, 0) : kOob, n0);
            st_g<T, V>(make_rsrc(bz + setd, sz), w ? zoff(kn, sze, 2) : kOob, n1);
        }
        if (X && c.wx) {
            for (int v = 0; v < V; ++v) {
                const int x = c.col * V + v;
                const T bb = L.cx[0][x], cc = L.cx[1][x], kk = L.cx[2][x];
                T p0, p1;
                Dz0.v[v] = slab_term(c.inx[v], bb, cc, kk, pxe[0].v[v], Dz0.v[v], p0);
                Dy1.v[v] = slab_term(c.inx[v], bb, cc, kk, pxe[1].v[v], Dy1.v[v], p1);
                n0.v[v] = c.inx[v] && fz[v] ? p0 : T(0);   // zeros beside the slab
                n1.v[v] = c.inx[v] && fy[v] ? p1 : T(0);
            }
            const unsigned o = c.vx != kOob && c.vs != kOob && !last ? c.vx + kn * c.dx : kOob;
            st_g<T, V>(make_rsrc(bx + setd, sx), o, n0);
            st_g<T, V>(make_rsrc(bx + setd, sx), o == kOob ? kOob : o + 2 * c.ax, n1);
        }
        if constexpr (M != 0) mem_e(kn + 1);
        for (int v = 0; v < V; ++v) {
            cu[0].v[v] = Dx0.v[v] - Dx1.v[v];
            cu[1].v[v] = Dy0.v[v] - Dy1.v[v];
            cu[2].v[v] = Dz0.v[v] - Dz1.v[v];
            for (int q = 0; q < 3; ++q) En[q].v[v] = fma(c.S * Ei[q].v[v], cu[q].v[v], Eo[q].v[v]);
        }
        // dispersive cells (the arithmetic of e_update_v)
        bool lor = false;
        if constexpr (MIX) {
            if (kn >= c.lz0 && kn < c.lz1) {
                for (int v = 0; v < V; ++v) lor |= c.lx[v];
            }
        }
        G eold[3], wn[3];
        long long lq = 0;
        if constexpr (MIX) {
            if (lor && d.lorpre) {   // E^{n+1} and the histories are in set ws already
                for (int q = 0; q < 3; ++q) eold[q] = ld_g<T, V>(make_rsrc(wcur + 2 * q * fd, pbytes), c.ve);
                for (int v = 0; v < V; ++v)
                    for (int q = 0; q < 3; ++q)
                        if (c.lx[v]) En[q].v[v] = eold[q].v[v];
            } else if (lor) {        // one pole
                lq = ((long long)(kn - d.llo[2]) * (d.lhi[1] - d.llo[1]) + (c.j - d.llo[1])) * (d.lhi[0] - d.llo[0]) + (c.i - d.llo[0]);
                const bool own = c.own && !last;
                G w[3], wo[3];
                for (int q = 0; q < 3; ++q) {
                    eold[q] = ld_u<T, V>(d.lor[0][q] + lq + c.so);
                    w[q] = ld_u<T, V>(d.lor[1][q] + lq + c.so);
                    wo[q] = ld_u<T, V>(d.lor[2][q] + lq + c.so);
                }
                for (int q = 0; q < 3; ++q) {
                    G a, e;
                    for (int v = 0; v < V; ++v) {
                        const bool f = q == 0 ? fx[v] : q == 1 ? fy[v] : fz[v];   // zero on walls
                        T n = fma(T(1) / Ei[q].v[v], Eo[q].v[v], T(0.25) * d.lgs * eold[q].v[v]);
                        n = fma(c.S, cu[q].v[v], n);
                        n -= T(0.5) * fma(T(1) + d.lal[0], w[q].v[v], d.lxi[0] * wo[q].v[v]);
                        if (c.lx[v]) En[q].v[v] = n * (T(1) / (T(1) / Ei[q].v[v] + T(0.25) * d.lgs));
                        wn[q].v[v] = fma(d.lal[0], w[q].v[v], d.lxi[0] * wo[q].v[v]);
                        a.v[v] = f ? Eo[q].v[v] : T(0);
                        e.v[v] = f ? w[q].v[v] : T(0);
                    }
                    if (own) {
                        st_u<T, V>(d.lor[0][q] + lq + c.wo, a, c.lx);
                        st_u<T, V>(d.lor[2][q] + lq + c.wo, e, c.lx);
                    }
                }
            }
        }
        if (c.src_planes >> (kn - c.k0) & 1)
            for (int q = 0; q < d.nsrc; ++q) {
                Const<SrcDev<T>>& sr = d.src[q];
                if (c.t < sr.nwave && kn == sr.k) {
                    const T w = gp(sr.wave)[c.t];
                    for (int v = 0; v < V; ++v)
                        if ((sr.kind == 1 || (c.i + v == sr.i && c.j == sr.j)) && !(MIX && lor && d.lorpre && c.lx[v])) {
                            if (sr.comp == 0) En[0].v[v] += w;
                            else if (sr.comp == 1) En[1].v[v] += w;
                            else En[2].v[v] += w;
                        }
                }
            }
        for (int v = 0; v < V; ++v) {
            En[0].v[v] = fx[v] ? En[0].v[v] : T(0);
            En[1].v[v] = fy[v] ? En[1].v[v] : T(0);
            En[2].v[v] = fz[v] ? En[2].v[v] : T(0);
        }
        if constexpr (MIX) {
            if (lor && !d.lorpre && c.own && !last)   // W^{n+1} of the owned dispersive nodes
                for (int q = 0; q < 3; ++q) {
                    G a;
                    for (int v = 0; v < V; ++v) {
                        const bool f = q == 0 ? fx[v] : q == 1 ? fy[v] : fz[v];
                        a.v[v] = f ? fma(T(0.5) * d.lg[0], En[q].v[v] - eold[q].v[v], wn[q].v[v]) : T(0);
                    }
                    st_u<T, V>(d.lor[1][q] + lq + c.wo, a, c.lx);
                }
        }
        {
            const unsigned nb = last ? 0u : pbytes;
            const T* f = wcur;
            for (int q = 0; q < 3; ++q) {
                st_g<T, V>(make_rsrc(f, nb), c.vs, En[q]);
                f += 2 * fd;
            }
        }
        // ---- H^{n+3/2} at plane kp
        G exu = L.ex[b ^ 1][c.iu], ezu = L.ez[b ^ 1][c.iu];
        T eyr = L.ey[b ^ 1][c.ir], ezr = L.ez[b ^ 1][c.ir].v[0];
        if constexpr (MIX) {
            for (int v = 0; v < V; ++v) {
                exu.v[v] = c.fu * exu.v[v];
                ezu.v[v] = c.fu * ezu.v[v];
            }
            eyr = c.fr * eyr;
            ezr = c.fr * ezr;
        }
        if (c.wu)
            for (int v = 0; v < V; ++v) exu.v[v] = ezu.v[v] = T(0);
        if (c.wr) eyr = ezr = T(0);
        const int szh = Z && first ? zslab(kp) : -1;
        for (int v = 0; v < V; ++v) {
            const T ex = Ek[0].v[v], ey = Ek[1].v[v], ez = Ek[2].v[v];
            const T eyx = v + 1 < V ? Ek[1].v[v + 1 < V ? v + 1 : v] : eyr, ezx = v + 1 < V ? Ek[2].v[v + 1 < V ? v + 1 : v] : ezr;
            // Hx: d+_y Ez - d+_z Ey ; Hy: d+_z Ex - d+_x Ez ; Hz: d+_x Ey - d+_y Ex
            Dx0.v[v] = ezu.v[v] - ez, Dx1.v[v] = En[1].v[v] - ey;
            Dy0.v[v] = En[0].v[v] - ex, Dy1.v[v] = ezx - ez;
            Dz0.v[v] = eyx - ey, Dz1.v[v] = exu.v[v] - ex;
        }
        if (Y && c.wy) {
            const T bb = L.cy[3][c.row], cc = L.cy[4][c.row], kk = L.cy[5][c.row];
            for (int v = 0; v < V; ++v) {
                Dx0.v[v] = slab_term(c.iny, bb, cc, kk, pyh[0].v[v], Dx0.v[v], n0.v[v]);
                Dz1.v[v] = slab_term(c.iny, bb, cc, kk, pyh[1].v[v], Dz1.v[v], n1.v[v]);
            }
            const unsigned o = c.iny && c.vs != kOob && first ? c.vy + kp * c.dy + c.ay : kOob;
            st_g<T, V>(make_rsrc(by + setd, sy), o, n0);
            st_g<T, V>(make_rsrc(by + setd, sy), o == kOob ? kOob : o + 2 * c.ay, n1);
        }
        if (Z && szh >= 0) {
            const int z = kp - c.k0;
            const T bb = L.cz[3][z], cc = L.cz[4][z], kk = L.cz[5][z];
            for (int v = 0; v < V; ++v) {
                Dy0.v[v] = slab_term(true, bb, cc, kk, pzh[0].v[v], Dy0.v[v], n0.v[v]);
                Dx1.v[v] = slab_term(true, bb, cc, kk, pzh[1].v[v], Dx1.v[v], n1.v[v]);
            }
            const bool w = c.vs != kOob;
            st_g<T, V>(make_rsrc(bz + setd, sz), w ? zoff(kp, szh, 1) : kOob, n0);
            st_g<T, V>(make_rsrc(bz + setd, sz), w ? zoff(kp, szh, 3) : kOob, n1);
        }
        if (X && c.wx) {
            for (int v = 0; v < V; ++v) {
                const int x = c.col * V + v;
                const T bb = L.cx[3][x], cc = L.cx[4][x], kk = L.cx[5][x];
                T p0, p1;
                Dz0.v[v] = slab_term(c.inx[v], bb, cc, kk, pxh[0].v[v], Dz0.v[v], p0);
                Dy1.v[v] = slab_term(c.inx[v], bb, cc, kk, pxh[1].v[v], Dy1.v[v], p1);
                n0.v[v] = c.inx[v] ? p0 : T(0);
                n1.v[v] = c.inx[v] ? p1 : T(0);
            }
            const unsigned o = c.vx != kOob && c.vs != kOob && first ? c.vx + kp * c.dx + c.ax : kOob;
            st_g<T, V>(make_rsrc(bx + setd, sx), o, n0);
            st_g<T, V>(make_rsrc(bx + setd, sx), o == kOob ? kOob : o + 2 * c.ax, n1);
        }
        if constexpr (M != 0) mem_h(kn);
        G Hw[3];
        for (int v = 0; v < V; ++v) {
            Hw[0].v[v] = fma(-c.S, Dx0.v[v] - Dx1.v[v], Hk[0].v[v]);
            Hw[1].v[v] = fma(-c.S, Dy0.v[v] - Dy1.v[v], Hk[1].v[v]);
            Hw[2].v[v] = fma(-c.S, Dz0.v[v] - Dz1.v[v], Hk[2].v[v]);
        }
        {
            const unsigned nb = first ? pbytes : 0u;
            const T* f = wcur + fd - (first ? pl : 0);
            for (int q = 0; q < 3; ++q) {
                st_g<T, V>(make_rsrc(f, nb), c.vs, Hw[q]);
                f += 2 * fd;
            }
        }
        wcur += pl;
        if (first && c.smp_planes >> (kp - c.k0) & 1 && c.own)
            for (int v = 0; v < V; ++v)
                if (!(v > 0 && c.tail))
                    sample_node<T>(d, c.slot, c.i + v, c.j, kp, Ek[0].v[v], Ek[1].v[v], Ek[2].v[v], Hw[0].v[v], Hw[1].v[v],
                                Hw[2].v[v]);
        if (first && c.prb_planes >> (kp - c.k0) & 1 && c.own)
            for (int q = 0; q < d.nprb; ++q) {
                Const<PrbDev>& m = d.prb[q];
                if (m.k != kp || m.j != c.j || c.t >= m.ntrace) continue;
                for (int v = 0; v < V; ++v)
                    if (m.i == c.i + v) {
                        const T x = m.comp == 0 ? Ek[0].v[v] : m.comp == 1 ? Ek[1].v[v] : m.comp == 2 ? Ek[2].v[v]
                                    : m.comp == 3 ? Hw[0].v[v] : m.comp == 4 ? Hw[1].v[v] : Hw[2].v[v];
                        gp(m.trace)[c.t] = (double)x;
                    }
            }
        L.ex[b][tid] = En[0];
        L.ez[b][tid] = En[2];
        L.ey[b][tid] = En[1].v[0];
        for (int q = 0; q < 3; ++q) {
            Hk[q] = Hn[q];
            Ek[q] = En[q];
        }
    }
}

// One tile.  A function of its own per variant (not inlined), so that the
// lean variants do not inherit the spills and scalar pressure of the others.
template <typename T, int V, int NT, int M, int ND>
__device__ __attribute__((noinline, noreturn)) void pass_tile(const DomDev<T>* doms_, const int4* tab_, int rs_, int ws_, int t_,
                                                    int slot_, int rec_) {
    extern __shared__ __align__(16) char smem[];
    PassLds<T, V, NT>& L = *(PassLds<T, V, NT>*)smem;
    const DomDev<T>* doms = uniform(doms_);
    Const<int4>* tab = as_const(uniform(tab_));
    const int rs = uniform(rs_), ws = uniform(ws_), t = uniform(t_), slot = uniform(slot_), rec = uniform(rec_);
    const int dom = tab[2 * blockIdx.x].x, q0 = tab[2 * blockIdx.x].z, q1 = tab[2 * blockIdx.x].w;
    const int y0 = tab[2 * blockIdx.x + 1].x, y1 = tab[2 * blockIdx.x + 1].y;
    Const<DomDev<T>>& d = as_const(doms)[dom];
    PassCtx<T, V> c;
    c.d = &d;
    const int nx = d.n[0], ny = d.n[1], nz = d.n[2];
    const bool perx = d.per[0], pery = d.per[1];
    c.nz = nz;
    c.k0 = tab[2 * blockIdx.x + 1].z;
    c.k1 = tab[2 * blockIdx.x + 1].w;
    const int tid = c.tid = threadIdx.x;
    const TileMap<V> m = map_tile<T, V, (M & kPassX) != 0>(d, tid, q0, q1, y0, y1);
    const int i = c.i = m.i, j = c.j = m.j, wt = m.wt, rt = m.rt;
    const bool has_e = m.has_e;
    c.row = m.row;
    c.col = m.col;
    c.il = m.il;
    c.ir = m.ir;
    c.id = m.id;
    c.iu = m.iu;
    c.own = m.own;
    c.vh = m.act ? m.f : kOob;
    c.ve = has_e ? m.f : kOob;
    c.vs = c.own ? m.f : kOob;
    c.wl = m.wl;
    c.wr = m.wr;
    c.wd = m.wd;
    c.wu = m.wu;
    c.tail = m.tail;
    bool any = false;
    for (int v = 0; v < V; ++v) {
        c.inb[v] = has_e && i + v >= d.elo[0] && i + v < d.ehi[0] && j >= d.elo[1] && j < d.ehi[1];
        any |= c.inb[v];
    }
    c.vp = any ? ((unsigned)(j - d.elo[1]) * (unsigned)d.exs + (unsigned)(i - d.exa)) * (unsigned)sizeof(T) : kOob;
    c.ez0 = d.elo[2];
    c.ez1 = d.ehi[2];
    c.S = d.S;
    c.bg = d.epsinv_bg;
    c.so = (long long)rs * d.fs;
    c.wo = (long long)ws * d.fs;
    c.t = t;
    c.slot = slot;
    c.src_planes = c.smp_planes = c.prb_planes = 0;
    auto mark = [&](unsigned long long& b, int k, int last) {
        if (k >= c.k0 && k < c.k0 + 64 && k <= last) b |= 1ull << (k - c.k0);
    };
    for (int s = 0; s < d.nsrc; ++s) mark(c.src_planes, d.src[s].k, c.k1);
    if (slot >= 0)
        for (int s = 0; s < d.nsmp; ++s) {
            mark(c.smp_planes, d.smp[s].k, c.k1 - 1);
            mark(c.smp_planes, d.smp[s].k - 1, c.k1 - 1);   // flux monitors sample H one plane below too
        }
    if (rec)
        for (int s = 0; s < d.nprb; ++s) mark(c.prb_planes, d.prb[s].k, c.k1 - 1);
    if constexpr (M != 0) {
        c.fl = perx && i == 0 ? d.bsign[0] : T(1);
        c.fr = perx && i + V >= nx ? d.bsign[0] : T(1);
        c.fd = pery && j == 0 ? d.bsign[1] : T(1);
        c.fu = pery && j == ny - 1 ? d.bsign[1] : T(1);
        for (int v = 0; v < V; ++v)
            c.lx[v] = d.has_lor && i + v >= d.llo[0] && i + v < d.lhi[0] && j >= d.llo[1] && j < d.lhi[1];
        c.lz0 = d.has_lor ? d.llo[2] : 0;
        c.lz1 = d.has_lor ? d.lhi[2] : 0;
        const SlabMap<V> sl = map_slabs<T, V, false>(d, m, has_e);
        for (int v = 0; v < V; ++v) c.inx[v] = sl.inx[v];
        c.iny = sl.iny;
        c.wx = sl.wx;
        c.wy = sl.wy;
        c.vx = sl.vx;
        c.dx = sl.dx;
        c.ax = sl.ax;
        c.vy = sl.vy;
        c.dy = sl.dy;
        c.ay = sl.ay;
        c.vz = sl.vz;
        // coefficient tables of the tile into LDS
        if constexpr (M & kPassX)
            for (int s = tid; s < 6 * wt * V; s += NT) {
                const int tb = s / (wt * V), x = s - tb * (wt * V);
                const int gx = (q0 - m.hl) * V + x;
                L.cx[tb][x] = gx >= 0 && gx < nx ? gp(d.tab[0])[tb * nx + gx] : T(0);
            }
        if constexpr (M & kPassY)
            for (int s = tid; s < 6 * rt; s += NT) {
                const int tb = s / rt, r = s - tb * rt, gy = y0 - m.hb + r;
                L.cy[tb][r] = gy >= 0 && gy < ny ? gp(d.tab[1])[tb * ny + gy] : T(0);
            }
        if constexpr (M & kPassZ) {
            const int nzc = c.k1 - c.k0 + 1;
            for (int s = tid; s < 6 * nzc; s += NT) {
                const int tb = s / nzc, r = s - tb * nzc, gz = c.k0 + r;
                L.cz[tb][r] = gz < nz ? gp(d.tab[2])[tb * nz + gz] : T(0);
            }
        }
        __syncthreads();
    }
    pass_march<T, V, NT, M, ND>(c, L);
    __builtin_amdgcn_endpgm();
}

template <typename T, int V, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_pass(const DomDev<T>* __restrict__ doms, const int4* __restrict__ tab, int rs, int ws, int t,
       const int* __restrict__ tdev, int slot, int rec) {
    const int4 ta = tab[2 * blockIdx.x];
    if (ta.x < 0) return;
    graph_args(tdev, t, rs, ws);
    const DomDev<T>& d = doms[ta.x];
    const int mask = ta.y;
    auto go = [&](auto m) {
        constexpr int MM = decltype(m)::value;
        if (d.eps_diag) pass_tile<T, V, NT, MM, 3>(doms, tab, rs, ws, t, slot, rec);
        else pass_tile<T, V, NT, MM, 1>(doms, tab, rs, ws, t, slot, rec);
    };
    switch (mask) {
    case 0: go(std::integral_constant<int, 0>{}); break;
    case kPassX: go(std::integral_constant<int, kPassX>{}); break;
    case kPassY: go(std::integral_constant<int, kPassY>{}); break;
    case kPassZ: go(std::integral_constant<int, kPassZ>{}); break;
    case kPassX | kPassY: go(std::integral_constant<int, kPassX | kPassY>{}); break;
    case kPassX | kPassZ: go(std::integral_constant<int, kPassX | kPassZ>{}); break;
    case kPassY | kPassZ: go(std::integral_constant<int, kPassY | kPassZ>{}); break;
    case kPassX | kPassY | kPassZ: go(std::integral_constant<int, kPassX | kPassY | kPassZ>{}); break;
    case kPassMix: go(std::integral_constant<int, kPassMix>{}); break;
    case kPassMix | kPassX: go(std::integral_constant<int, kPassMix | kPassX>{}); break;
    case kPassMix | kPassZ: go(std::integral_constant<int, kPassMix | kPassZ>{}); break;
    default: go(std::integral_constant<int, kPassAll>{}); break;
    }
}

}  // namespace

template <typename T>
void launch_pass(const LaunchCfg& c, const void* doms, int rs, int ws, int t, hipStream_t s, const int* tdev, int slot,
                 bool rec) {
    constexpr int V = kPassGroup<T>;
    const DomDev<T>* dd = (const DomDev<T>*)doms;
    if (c.pnt == 1024)
        hipLaunchKernelGGL((k_pass<T, V, 1024>), dim3(c.pgrid), dim3(1024), sizeof(PassLds<T, V, 1024>), s, dd, c.ptab, rs, ws, t, tdev, slot,
                           rec ? 1 : 0);
    else if (c.pnt == 512)
        hipLaunchKernelGGL((k_pass<T, V, 512>), dim3(c.pgrid), dim3(512), sizeof(PassLds<T, V, 512>), s, dd, c.ptab, rs, ws, t, tdev, slot,
                           rec ? 1 : 0);
    else
        hipLaunchKernelGGL((k_pass<T, V, 256>), dim3(c.pgrid), dim3(256), sizeof(PassLds<T, V, 256>), s, dd, c.ptab, rs, ws, t, tdev, slot,
                           rec ? 1 : 0);
}

template void launch_pass<float>(const LaunchCfg&, const void*, int, int, int, hipStream_t, const int*, int, bool);
template void launch_pass<double>(const LaunchCfg&, const void*, int, int, int, hipStream_t, const int*, int, bool);

}  // namespace fdtd
