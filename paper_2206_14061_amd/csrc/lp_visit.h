// Iteration over the exact stencil of a particle from its neighbour list
// (with skin) and its stencil record.  Shared by the selection, export and
// fit kernels so that every pass keeps exactly the same rows.
#pragma once

#include "lp_internal.h"

namespace lp {

struct Pt {
    double x, y, z;     // position (mirrors: reflected source)
    int32_t id;         // real id, or n + k for mirror k
    int32_t src;        // real particle carrying the state
    bool mirror;
    bool valid;
};

// Along periodic axes a point stands for its copy nearest to the particle
// at (xi, yi).
__device__ __forceinline__ void to_image(const View& v, const GridInfo& g, Pt& p,
                                         double xi, double yi)
{
    if (!v.periodic) return;
    p.x = image_coord(p.x, xi, g.Lx, g.hLx);
    p.y = image_coord(p.y, yi, g.Ly, g.hLy);
}

// Position of real particle j from its 32-byte record.
__device__ __forceinline__ void packed_pos(const View& v, int32_t j, double& x, double& y,
                                          double& z)
{
    const double* r = v.p4 + 4 * (int64_t)j;
    const double2 xy = *reinterpret_cast<const double2*>(r);
    x = xy.x;
    y = xy.y;
    z = r[2];
}

// Point of neighbour-list entry e (a real id, or MBIT | source of a
// potential mirror; the mirror exists while its source is within R of the
// wall, and is placed at (x, y, 2 wall - z)), seen from (xi, yi).
__device__ __forceinline__ Pt list_point(const View& v, const GridInfo& g,
                                         int32_t e, double xi, double yi)
{
    Pt p;
    if (e & MBIT) {
        const int32_t j = e & ~MBIT;
        const int32_t k = v.mirror_of[j];
        p.valid = k >= 0;
        packed_pos(v, j, p.x, p.y, p.z);
        p.z = dsub(dmul(2.0, g.wall), p.z);
        p.id = (int32_t)v.n + k;
        p.src = j;
        p.mirror = true;
    } else {
        p.valid = true;
        packed_pos(v, e, p.x, p.y, p.z);
        p.id = e;
        p.src = e;
        p.mirror = false;
    }
    to_image(v, g, p, xi, yi);
    return p;
}

#ifndef LP_FIT_BATCH
#define LP_FIT_BATCH 4
#endif
// Stencil rows whose loads the fits issue together (by default).
constexpr int FIT_BATCH = LP_FIT_BATCH;

// Registers of one particle's list walk: its position and the fields of
// its system's grid that a list entry needs, copied once so that stores
// made during the walk cannot force the grid table to be read again.
struct Seen {
    double xi, yi, zi;
    double wall2;               // twice the wall height (mirror plane)
    double Lx, hLx, Ly, hLy;    // periodic box, 0 on open axes
};

__device__ __forceinline__ Seen seen_from(const View& v, const GridInfo& g, int64_t i)
{
    Seen s;
    s.xi = v.x[i];
    s.yi = v.y[i];
    s.zi = v.z[i];
    s.wall2 = dmul(2.0, g.wall);
    s.Lx = g.Lx;
    s.hLx = g.hLx;
    s.Ly = g.Ly;
    s.hLy = g.hLy;
    return s;
}

// The points of U list entries (the same points as list_point).  Every
// position load is issued before the first is used, so the U gathers are
// in flight together instead of one latency after another.
template <int U>
__device__ __forceinline__ void gather_list(const View& v, const Seen& s,
                                            const int32_t (&e)[U], Pt (&p)[U])
{
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int32_t j = e[u] & ~MBIT;
        packed_pos(v, j, p[u].x, p[u].y, p[u].z);
        p[u].src = j;
        p[u].id = j;
        p[u].mirror = (e[u] & MBIT) != 0;
        p[u].valid = true;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (p[u].mirror) {
            const int32_t k = v.mirror_of[p[u].src];
            p[u].valid = k >= 0;
            p[u].id = (int32_t)v.n + k;
            p[u].z = dsub(s.wall2, p[u].z);
        }
    }
    if (v.periodic) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            p[u].x = image_coord(p[u].x, s.xi, s.Lx, s.hLx);
            p[u].y = image_coord(p[u].y, s.yi, s.Ly, s.hLy);
        }
    }
}

__device__ __forceinline__ bool key_less(double ra, int32_t ia, double rb,
                                         int32_t ib)
{
    return ra < rb || (ra == rb && ia < ib);
}

__device__ __forceinline__ int octant_of(double dx, double dy, double dz)
{
    return (dx >= 0.0 ? 1 : 0) + (dy >= 0.0 ? 2 : 0) + (dz >= 0.0 ? 4 : 0);
}

// Stencil record of one particle, in registers: kept rows, ghost mask and
// the keep bitmask over its neighbour-list entries.
struct Rec {
    int m, gm;
    uint64_t mask[MASK_WORDS];
};

__device__ __forceinline__ Rec load_rec(const View& v, int64_t i)
{
    Rec r;
    const int64_t n = v.n;
    const int32_t* q = v.rec;
    r.m = q[REC_M * n + i];
    r.gm = q[REC_GM * n + i];
#pragma unroll
    for (int w = 0; w < MASK_WORDS; ++w) r.mask[w] = v.kmask[w * n + i];
    return r;
}

// Set bits of a keep mask in ascending order (list indices).
struct MaskWalk {
    static_assert(MASK_WORDS == 4, "keep mask walk assumes four words");
    // the word being walked (entries base, base + 1, ...) and the words
    // after it
    uint64_t cur, b1, b2, b3;
    int base = 0;
    __device__ __forceinline__ explicit MaskWalk(const Rec& r)
        : cur(r.mask[0]), b1(r.mask[1]), b2(r.mask[2]), b3(r.mask[3]) {}
    __device__ __forceinline__ bool any() const { return (cur | b1 | b2 | b3) != 0; }
    // next set bit; the caller pops at most popcount times.  A lane moves
    // to the next word only when its current one is used up (a few times
    // per stencil), so the common pop is one count of trailing zeros.
    __device__ __forceinline__ int pop()
    {
        if (cur == 0) {
            cur = b1;
            b1 = b2;
            b2 = b3;
            b3 = 0;
            base += 64;
            if (cur == 0) {
                cur = b1;
                b1 = b2;
                b2 = 0;
                base += 64;
                if (cur == 0) {
                    cur = b1;
                    b1 = 0;
                    base += 64;
                }
            }
        }
        const int k = base + __builtin_ctzll(cur);
        cur &= cur - 1;
        return k;
    }
};

// Calls f(pt, dx, dy, dz) for every stencil row of real particle i, in
// ascending list order (the ghost rows are not visited: they follow from
// r.gm).  Each lane walks only its own kept entries, so a wave runs as
// many iterations as its largest stencil.  Rows are taken B at a time:
// their list words, then their positions, are loaded together, and the
// calls of f for the batch form one block, so the loads f makes for later
// rows can be issued before the earlier rows are summed.
template <int B = FIT_BATCH, class F>
__device__ __forceinline__ void visit_stencil(const View& v, const GridInfo& g,
                                              int64_t i, const Rec& r, F&& f)
{
    const int64_t n = v.n;
    const Seen s = seen_from(v, g, i);
    const double xi = s.xi, yi = s.yi, zi = s.zi;
    MaskWalk mw(r);
    int t = 0;
    for (; t + B <= r.m; t += B) {
        int32_t e[B];
#pragma unroll
        for (int u = 0; u < B; ++u) e[u] = v.vl[vl_at(n, i, mw.pop())];
        Pt p[B];
        gather_list(v, s, e, p);
#pragma unroll
        for (int u = 0; u < B; ++u)
            f(p[u], dsub(p[u].x, xi), dsub(p[u].y, yi), dsub(p[u].z, zi));
    }
    for (; t < r.m; ++t) {
        const int32_t e[1] = {v.vl[vl_at(n, i, mw.pop())]};
        Pt p[1];
        gather_list(v, s, e, p);
        f(p[0], dsub(p[0].x, xi), dsub(p[0].y, yi), dsub(p[0].z, zi));
    }
}

// The sources staged for half h of a tile: those of the half, or of the
// whole tile.  S < 0: not staged; reals: those that are no mirrors.
struct StageUnit {
    int S, reals;
    const int32_t* src;
};
__device__ __forceinline__ bool tile_split(const View& v, int64_t tile)
{
    return v.tile_cnt[2 * tile + 1] != TILE_WHOLE;
}
__device__ __forceinline__ StageUnit stage_unit(const View& v, int64_t tile, int h)
{
    const int64_t u = 2 * tile + (h && tile_split(v, tile) ? 1 : 0);
    const int32_t tc = v.tile_cnt[u];
    return StageUnit{tile_slots(tc), tile_reals(tc), v.tile_src + u * STAGE_CAP};
}

// The part of the particles a block of a staged kernel takes, P of them from
// i0 on and the unit they are staged as.  A block of a whole tile (P = BLOCK)
// takes its first half only when the tile is staged in halves; the second
// halves are those of a second grid's worth of blocks, which do nothing for
// other tiles (a loop over the two in one block costs 176 spilled registers
// in pass 1).
template <int P>
struct BlockPart {
    int64_t i0;
    int h;                      // half (P = BLOCK: 1 only in the second set)
    StageUnit unit;
    bool split;
    static unsigned blocks(int64_t n)
    {
        return (unsigned)((P == BLOCK ? 2 : 1) * ((n + P - 1) / P));
    }
    __device__ __forceinline__ BlockPart(const View& v, int rows_ok)
    {
        if (P == BLOCK) {
            const unsigned half = gridDim.x / 2;
            h = blockIdx.x >= half ? 1 : 0;
            i0 = xcd_block(blockIdx.x - (h ? half : 0u), half) * P;
        } else {
            i0 = xcd_block(blockIdx.x, gridDim.x) * P;
            h = (int)(i0 % BLOCK) / HALF;
        }
        unit = StageUnit{-1, 0, nullptr};
        split = false;
        if (rows_ok) {
            unit = stage_unit(v, i0 / BLOCK, h);
            split = tile_split(v, i0 / BLOCK);
        }
    }
    // nothing to do in this block
    __device__ __forceinline__ bool idle() const { return P == BLOCK && h == 1 && !split; }
    // is the block's particle p in the unit?
    __device__ __forceinline__ bool mine(int p) const
    {
        return P < BLOCK || !split || p / HALF == h;
    }
    static_assert(P == BLOCK || HALF % P == 0, "a tile, or a part of half of one");
};

// A staged field at a row's byte offset.
__device__ __forceinline__ double staged_at(const double* field, uint32_t off)
{
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(field) + off);
}

// visit_stencil for a particle of a staged tile: the fields of the tile's
// list sources sit in LDS in slot order, and a row's point is read from
// there at the byte offset the selection left for it.  The m rows are
// spread over LPP adjacent lanes: lane `sub` takes the chunks of four rows
// sub, sub + LPP, ... (one 8-byte load each, the next one in flight), in
// list order.  Calls f(off, dx, dy, dz).
template <int LPP, bool PERIODIC, class F>
__device__ __forceinline__ void visit_staged(const View& v, const Seen& s, int64_t i, int m,
                                             int sub, const double* sx, const double* sy,
                                             const double* sz, F&& f)
{
    auto row = [&](uint32_t off) {
        double x = staged_at(sx, off), y = staged_at(sy, off);
        const double z = staged_at(sz, off);
        if (PERIODIC) {
            x = image_coord(x, s.xi, s.Lx, s.hLx);
            y = image_coord(y, s.yi, s.Ly, s.hLy);
        }
        f(off, dsub(x, s.xi), dsub(y, s.yi), dsub(z, s.zi));
    };
    const int full = m >> 2, used = (m + 3) >> 2;
    const uint2* kp = reinterpret_cast<const uint2*>(v.ks + vs_at(v.n, i, 4 * sub));
    const int64_t step = (int64_t)LPP * v.n;
    uint2 w = make_uint2(0u, 0u);
    if (sub < used) w = *kp;
    int c = sub;
    while (c < full) {
        const uint2 cur = w;
        c += LPP;
        kp += step;
        if (c < used) w = *kp;
        row(cur.x & 0xFFFFu);
        row(cur.x >> 16);
        row(cur.y & 0xFFFFu);
        row(cur.y >> 16);
    }
    if (c == full)
        for (int u = 0; u < (m & 3); ++u)
            row(((u & 2 ? w.y : w.x) >> (16 * (u & 1))) & 0xFFFFu);
}

// visit_stencil with the rows of particle i spread over LPP adjacent lanes:
// lane `sub` takes the chunks of CH kept rows sub, sub + LPP, ...  CH = 4 are
// the rows of visit_staged.  CH = 1 is faster where every particle gathers:
// adjacent lanes read and add to adjacent sources, and a row at a time needs
// fewer registers (us at 400,000 particles, chunks of four and of one: the
// reverse kernels 2,260 and 2,190, 2,010 and 1,930; a step with two lanes in the
// fits 554, 522, with four 639, 579).
template <int LPP, int CH, class F>
__device__ __forceinline__ void visit_stencil_sub(const View& v, const GridInfo& g,
                                                  int64_t i, const Rec& r, int sub, F&& f)
{
    if (LPP == 1) {
        visit_stencil(v, g, i, r, f);
        return;
    }
    const int64_t n = v.n;
    MaskWalk mw(r);
    for (int t = 0; t < CH * sub && t < r.m; ++t) mw.pop();
    if constexpr (CH == 1) {
        const double xi = v.x[i], yi = v.y[i], zi = v.z[i];
        for (int t = sub; t < r.m; t += LPP) {
            const Pt p = list_point(v, g, v.vl[vl_at(n, i, mw.pop())], xi, yi);
            f(p, dsub(p.x, xi), dsub(p.y, yi), dsub(p.z, zi));
            for (int u = 1; u < LPP && t + u < r.m; ++u) mw.pop();
        }
        return;
    }
    const Seen s = seen_from(v, g, i);
    const double xi = s.xi, yi = s.yi, zi = s.zi;
    for (int t = CH * sub; t < r.m; t += CH * LPP) {
        for (int u = t; u < t + CH && u < r.m; ++u) {
            const int32_t e[1] = {v.vl[vl_at(n, i, mw.pop())]};
            Pt p[1];
            gather_list(v, s, e, p);
            f(p[0], dsub(p[0].x, xi), dsub(p[0].y, yi), dsub(p[0].z, zi));
        }
        for (int u = t + CH; u < t + CH * LPP && u < r.m; ++u) mw.pop();
    }
}

template <int CTRL>
__device__ __forceinline__ int dpp_move(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x)
{
    return __int_as_float(dpp_move<CTRL>(__float_as_int(x)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x)
{
    return __hiloint2double(dpp_move<CTRL>(__double2hiint(x)),
                            dpp_move<CTRL>(__double2loint(x)));
}

// sum of x over the LPP (up to 16) adjacent lanes of a particle (the same
// value in every one of them: the partners of a step add the same operands):
// swaps of neighbours and of pairs inside quads, then the half-row and row
// mirrors
template <int LPP, class T>
__device__ __forceinline__ T lane_sum(T x)
{
    static_assert(LPP == 1 || LPP == 2 || LPP == 4 || LPP == 8 || LPP == 16, "lanes of a row");
    if (LPP >= 2) x += dpp_move<0xB1>(x);
    if (LPP >= 4) x += dpp_move<0x4E>(x);
    if (LPP >= 8) x += dpp_move<0x141>(x);
    if (LPP >= 16) x += dpp_move<0x140>(x);
    return x;
}

}  // namespace lp
