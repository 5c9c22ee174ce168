// fdtd_pass.h -- what the single-pass kernels, forward and adjoint, share
// (internal): buffer descriptors of a plane, the LDS barrier, a thread's place
// in its tile and in the absorber memories.
#pragma once
#include <stdint.h>

#include "fdtd_dev.h"
#include "fdtd_launch.h"

namespace fdtd {

namespace {

using Rsrc = __amdgpu_buffer_rsrc_t;
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// an offset out of range of every descriptor here (each spans below 2 GiB)
constexpr unsigned kOob = 0x80000000u;

__device__ __forceinline__ Rsrc make_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}

// The descriptors and tables do not change during a launch: read through the
// constant address space, their fields are scalar loads and stay scalars.
template <typename P>
using Const = const __attribute__((address_space(4))) P;
template <typename P>
__device__ __forceinline__ Const<P>* as_const(const P* p) {
    return (Const<P>*)p;
}

template <typename T, int V>
struct Grp {   // V neighbouring x nodes
    T v[V];
};

template <typename T, int V>
__device__ __forceinline__ Grp<T, V> ld_g(Rsrc r, unsigned off) {
    static_assert(sizeof(Grp<T, V>) == 8, "8 bytes per thread");
    return __builtin_bit_cast(Grp<T, V>, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}

template <typename T, int V>
__device__ __forceinline__ void st_g(Rsrc r, unsigned off, Grp<T, V> x) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, (int)off, 0, 0);
}

template <typename T>
__device__ __forceinline__ T ld_1(Rsrc r, unsigned off) {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}

template <typename T>
__device__ __forceinline__ void st_1(Rsrc r, unsigned off, T x) {
    if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, (int)off, 0, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, (int)off, 0, 0);
}

// barrier that orders LDS accesses only: loads and stores in flight stay so
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One axis' absorber memories as the kernels address them: the eight arrays
// of an axis (side by side: psi_E r0, psi_H r0, psi_E r1, psi_H r1 per side)
// lie in one range of a state set, `a` bytes apart on a side.
struct PsiAxis {
    const char* base;     // first array of the first side present, set 0
    unsigned span;        // bytes of all of them (0: no slab)
    unsigned a[2];        // array distance per side
    unsigned hi;          // offset of the high side's first array
};

// ADJ: the adjoint state's memories
template <bool ADJ, typename D>
__device__ __forceinline__ PsiAxis psi_range(const D& d, int a) {
    auto at = [&](int side, int h) {
        if constexpr (ADJ) return (const char*)(h ? d.psiHa[a][side][0] : d.psiEa[a][side][0]);
        else return (const char*)(h ? d.psiH[a][side][0] : d.psiE[a][side][0]);
    };
    PsiAxis p;
    const bool lo = d.L[a][0] > 0, hi = d.L[a][1] > 0;
    p.base = lo ? at(0, 0) : at(1, 0);
    p.a[0] = lo ? (unsigned)(at(0, 1) - at(0, 0)) : 0u;
    p.a[1] = hi ? (unsigned)(at(1, 1) - at(1, 0)) : 0u;
    p.hi = lo ? (unsigned)(at(1, 0) - at(0, 0)) : 0u;
    p.span = hi ? p.hi + 4u * p.a[1] : 4u * p.a[0];
    if (!lo && !hi) p.span = 0;
    return p;
}

// a value that is the same in every lane, as a scalar
template <typename P>
__device__ __forceinline__ P uniform(P x) {
    if constexpr (sizeof(P) == 4) {
        return __builtin_bit_cast(P, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
    } else {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
        const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u),
                       hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
        return __builtin_bit_cast(P, (unsigned long long)hi << 32 | lo);
    }
}

// A thread's place in a tile of owned column groups [q0, q1) and rows
// [y0, y1), with a halo of one group and one row on each inner side (and
// across a seam).
template <int V>
struct TileMap {
    int row, col, i, j, wt, rt, hl, hb;   // place; tile width and height, low halo
    int il, ir, id, iu;          // threads of the neighbouring groups: left, right, row below, row above
    bool act, has_e, own;        // holds a node; not of the low halo; owned
    bool wl, wr, wd, wu;         // the neighbour past a wall: left, right, row below, row above
    bool tail;                   // the group's last node lies past nx
    unsigned f;                  // byte offset in a plane
};

// Threads take the tile's columns row by row.  A tile that meets x slabs (X)
// takes the slab columns (nl low, nh high) of all rows first, so that only
// the waves holding them touch the x memories.
template <typename T, int V, bool X, typename D>
__device__ __forceinline__ TileMap<V> map_tile(const D& d, int tid, int q0, int q1, int y0, int y1) {
    TileMap<V> m;
    const int nx = d.n[0], ny = d.n[1], nq = (nx + V - 1) / V;
    const bool perx = d.per[0], pery = d.per[1];
    const int hr = perx || q1 < nq, ht = pery || y1 < ny;
    m.hl = perx || q0 > 0;
    m.hb = pery || y0 > 0;
    const int wt = m.wt = q1 - q0 + m.hl + hr, rt = m.rt = y1 - y0 + m.hb + ht;
    int nl = 0, nh = 0;
    if constexpr (X) {
        const int g0 = q0 - m.hl;   // group of the tile's first column (no slab on a periodic axis)
        nl = min(max((d.L[0][0] + V - 1) / V - g0, 0), wt);
        if (d.L[0][1]) nh = min(max(g0 + wt - (nx - d.L[0][1]) / V, 0), wt - nl);
    }
    const int ns = nl + nh, wi = wt - ns;
    const bool part = tid < ns * rt;   // slab columns
    const int u = part ? tid : tid - ns * rt, wp = max(part ? ns : wi, 1);
    m.row = u / wp;
    const int cc = u - m.row * wp;
    m.col = part ? (cc < nl ? cc : cc + wi) : cc + nl;
    m.act = (part || wi > 0) && m.row < rt;
    if (!m.act) m.row = m.col = 0;   // idle threads: in range of every table, no loads, no stores
    auto at = [&](int row, int col) {
        return col < nl ? row * ns + col : col >= nl + wi ? row * ns + col - wi : ns * rt + row * wi + col - nl;
    };
    m.il = m.col > 0 ? at(m.row, m.col - 1) : 0;
    m.ir = m.col + 1 < wt ? at(m.row, m.col + 1) : 0;
    m.id = m.row > 0 ? at(m.row - 1, m.col) : 0;
    m.iu = m.row + 1 < rt ? at(m.row + 1, m.col) : 0;
    int q = q0 - m.hl + m.col, j = y0 - m.hb + m.row;
    if (q < 0) q = nq - 1;         // across a seam (a periodic axis has whole groups)
    else if (q >= nq) q = 0;
    if (j < 0) j = ny - 1;
    else if (j >= ny) j = 0;
    const int i = q * V;
    m.i = i;
    m.j = j;
    m.has_e = m.act && m.row >= m.hb && m.col >= m.hl;
    m.own = m.has_e && m.row < m.hb + (y1 - y0) && m.col < m.hl + (q1 - q0);
    m.f = ((unsigned)j * (unsigned)d.pitch + (unsigned)i) * (unsigned)sizeof(T);
    m.wl = i == 0 && !perx;
    m.wr = i + V >= nx && !perx;
    m.wd = j == 0 && !pery;
    m.wu = j == ny - 1 && !pery;
    m.tail = V > 1 && i + V > nx;
    return m;
}

// A thread's place in the absorber memories: whether its nodes lie in an x or
// y slab, its byte offsets at plane 0, per plane and per array (z slabs: in a
// plane).  in: the thread's nodes take part.
template <int V>
struct SlabMap {
    bool inx[V], iny, wx, wy;    // wx, wy: some thread of the wave is in an x slab, a y slab
    unsigned vx, dx, ax, vy, dy, ay, vz;
};

template <typename T, int V, bool ADJ, typename D>
__device__ __forceinline__ SlabMap<V> map_slabs(const D& d, const TileMap<V>& m, bool in) {
    SlabMap<V> s;
    const int nx = d.n[0], ny = d.n[1], i = m.i, j = m.j;
    {
        const PsiAxis p = psi_range<ADJ>(d, 0);
        const int xh = nx - d.L[0][1];
        const bool high = i + V > xh && !(i < d.L[0][0]);   // a group meets one slab only
        bool any = false;
        for (int v = 0; v < V; ++v) {
            s.inx[v] = in && i + v < nx && (high ? i + v >= xh : i + v < d.L[0][0]);
            any |= s.inx[v];
        }
        s.wx = __builtin_amdgcn_ballot_w64(any) != 0;
        const int Ls = d.lxp[high];
        s.ax = p.a[high];
        s.dx = (unsigned)(ny * Ls) * (unsigned)sizeof(T);
        s.vx = any ? (high ? p.hi : 0u) + (unsigned)(j * Ls + (high ? i - d.lxs : i)) * (unsigned)sizeof(T) : kOob;
    }
    {
        const PsiAxis p = psi_range<ADJ>(d, 1);
        const int yh = ny - d.L[1][1];
        const bool high = j >= yh;
        const int Ls = d.L[1][high];
        s.iny = in && (high || j < d.L[1][0]);
        s.wy = __builtin_amdgcn_ballot_w64(s.iny) != 0;
        s.ay = p.a[high];
        s.dy = (unsigned)(Ls * d.ppx) * (unsigned)sizeof(T);
        s.vy = (high ? p.hi : 0u) + (unsigned)((high ? j - yh : j) * d.ppx + i) * (unsigned)sizeof(T);
    }
    s.vz = (unsigned)(j * d.ppx + i) * (unsigned)sizeof(T);
    return s;
}

}  // namespace

}  // namespace fdtd
