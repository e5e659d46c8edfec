// Neighbour list, mirrors, stencil selection and ghost masks (Sec. 3.1
// steps 5-6 and the solid-wall mirrors and free-boundary ghosts of step 9).
//
// Neighbour list with skin: at a rebuild each particle records every real
// particle within R (1 + skin) and every potential mirror source (a real
// within R (1 + skin) of the wall whose reflection lies within R (1 + skin)).
// Until some particle has moved more than skin R / 2, the list contains
// every pair that can be closer than R, so every pass below applies the
// exact candidate test r2 = (dx*dx + dy*dy) + dz*dz < R*R to the list and
// obtains exactly the candidates a full search would.  The list is built
// with a wavefront per cell (k_list_cells: the cell's particles share the
// 27 cells they scan); k_list_build, a thread per particle, gives the same
// lists and serves as the check of the former.
//
// Stencil selection (nearest candidate of each octant, then the nearest
// others by key (r^2, id), m_max in all), a few adjacent lanes per particle,
// without storing or sorting the candidates: every list entry's exact test
// leaves a 15-bit key (r^2 in units of R^2/32766; monotone) and its octant
// in the lanes' registers, and the cut is the key value below which exactly
// m_max candidates lie, found by counting (k_select).  The result is a keep
// bitmask over the list entries (plus row count and ghost mask), which the
// exports, the refits and the fits that gather walk, and, where the tile is
// staged, the kept rows' slot words in list order, which the other fits read.
#include <algorithm>
#include <type_traits>

#include "lp_visit.h"

namespace lp {

namespace {

inline unsigned int blocks_for(int64_t n, int per = BLOCK)
{
    return (unsigned int)((n + per - 1) / per);
}

__device__ __forceinline__ void cell_clamp(const GridInfo& g, double x, double y,
                                           double z, int& cx, int& cy, int& cz)
{
    const double xw = wrap_coord(x, g.xlo, g.Lx), yw = wrap_coord(y, g.ylo, g.Ly);
    const int ix = (int)dmul(dsub(xw, g.x0), g.inv_cx);
    const int iy = (int)dmul(dsub(yw, g.y0), g.inv_cy);
    const int iz = (int)dmul(dsub(z, g.z0), g.inv_c);
    cx = ix < 0 ? 0 : (ix >= g.nx ? g.nx - 1 : ix);
    cy = iy < 0 ? 0 : (iy >= g.ny ? g.ny - 1 : iy);
    cz = iz < 0 ? 0 : (iz >= g.nz ? g.nz - 1 : iz);
}

// Orders the LDS accesses of one wavefront's lanes (no block barrier).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Neighbouring cell d in {-1, 0, 1} of cell c along an axis of nc cells:
// clipped on an open axis; wrapped on a periodic one, where fewer than
// three cells are each visited once.  -1: no cell.
__device__ __forceinline__ int nb_cell(int c, int d, int nc, bool periodic)
{
    if (!periodic) return (c + d < 0 || c + d >= nc) ? -1 : c + d;
    if (nc < 3 && (d == -1 || (nc == 1 && d == 1))) return -1;
    return (c + d + nc) % nc;
}

// ---- neighbour-list build ---------------------------------------------

// Candidates of the list build whose positions are loaded together.
constexpr int LIST_BATCH = 8;

// The candidates' positions come from their 32-byte records (x, y, z, 0),
// which the rebuild's gather writes: two loads per candidate.  Nearest
// images are taken only where some system is periodic (PERIODIC).
template <bool PERIODIC>
__global__ __launch_bounds__(BLOCK) void k_list_build(
    int64_t n, int n_sys, const int64_t* __restrict__ off,
    const GridInfo* __restrict__ grid, const double* __restrict__ x,
    const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ p4,
    const int32_t* __restrict__ cs, const int32_t* __restrict__ ce,
    int32_t* __restrict__ vl, int32_t* __restrict__ vcnt, ErrWord* err,
    const int32_t* gate)
{
    if (gate && *gate == 0) return;
    const int64_t i = xcd_block(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
    if (i >= n) return;
    const GridInfo& g = grid[sys_of(off, n_sys, i)];
    const double Rv2 = g.Rv2 * (1.0 + 1e-12);
    const double xi = x[i], yi = y[i], zi = z[i];
    int cnt = 0;
    // entry cnt goes to out[cnt % VCHUNK]; out moves to the next chunk of
    // the particle (n VCHUNK entries on) whenever one fills
    int32_t* out = vl + (int64_t)i * VCHUNK;
    const int64_t cstride = n * VCHUNK;
    // the records as a byte base with 32-bit offsets (j < 2^27)
    const char* p4b = reinterpret_cast<const char*>(p4);
    const bool px = g.Lx > 0.0, py = g.Ly > 0.0;
    auto scan = [&](double qx, double qy, double qz, bool mirror) {
        int cx, cy, cz;
        cell_clamp(g, qx, qy, qz, cx, cy, cz);
        for (int zz = cz - 1; zz <= cz + 1; ++zz) {
            if (zz < 0 || zz >= g.nz) continue;
            for (int dy0 = -1; dy0 <= 1; ++dy0) {
                const int yy = nb_cell(cy, dy0, g.ny, py);
                if (yy < 0) continue;
                const int64_t row = g.cell_base + (int64_t)g.nx * (yy + (int64_t)g.ny * zz);
                // the particle ranges of the row's three cells, loaded
                // together (a clipped or repeated cell is empty)
                int32_t b[3], len[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int xx = nb_cell(cx, q - 1, g.nx, px);
                    const int64_t c = row + (xx < 0 ? 0 : xx);
                    const int32_t cb = cs[c], cend = ce[c];
                    b[q] = cb;
                    len[q] = xx < 0 ? 0 : cend - cb;
                }
                const int l01 = len[0] + len[1];
                const int tot = l01 + len[2];
                // the row's candidates in cell order, LIST_BATCH at a time:
                // their positions loaded together, then tested in order
                for (int t0 = 0; t0 < tot; t0 += LIST_BATCH) {
                    int32_t jb[LIST_BATCH];
                    double qxs[LIST_BATCH], qys[LIST_BATCH], qzs[LIST_BATCH];
#pragma unroll
                    for (int u = 0; u < LIST_BATCH; ++u) {
                        const int t = t0 + u < tot ? t0 + u : t0;
                        const int32_t j = t < len[0] ? b[0] + t
                                          : (t < l01 ? b[1] + (t - len[0]) : b[2] + (t - l01));
                        jb[u] = j;
                        const double* r =
                            reinterpret_cast<const double*>(p4b + ((uint32_t)j << 5));
                        const double2 xy = *reinterpret_cast<const double2*>(r);
                        qxs[u] = xy.x;
                        qys[u] = xy.y;
                        qzs[u] = r[2];
                    }
#pragma unroll
                    for (int u = 0; u < LIST_BATCH; ++u) {
                        const int32_t j = jb[u];
                        if (t0 + u >= tot || (!mirror && j == (int32_t)i)) continue;
                        const double dx =
                            (PERIODIC ? image_coord(qxs[u], qx, g.Lx, g.hLx) : qxs[u]) - qx;
                        const double dy =
                            (PERIODIC ? image_coord(qys[u], qy, g.Ly, g.hLy) : qys[u]) - qy;
                        const double dz = qzs[u] - qz;
                        // the list only has to hold every pair within the
                        // list radius: fused products are fine here, their
                        // rounding far inside Rv2's 1e-12 margin
                        if (fma(dz, dz, fma(dy, dy, dx * dx)) >= Rv2) continue;
                        if (mirror && !(qzs[u] - g.wall < g.Rv)) continue;
                        if (cnt < VCAP) {
                            out[cnt & (VCHUNK - 1)] = mirror ? (j | MBIT) : j;
                            if ((cnt & (VCHUNK - 1)) == VCHUNK - 1) out += cstride;
                        }
                        ++cnt;
                    }
                }
            }
        }
    };
    scan(xi, yi, zi, false);
    // potential mirrors: reals near the wall whose reflection is near i,
    // i.e. reals near the reflection of i (reflection is an isometry)
    if (zi - g.wall < g.Rv) scan(xi, yi, dsub(dmul(2.0, g.wall), zi), true);
    if (cnt > VCAP) {
        raise_error(err, ERR_CAPACITY, i);
        cnt = VCAP;
    }
    vcnt[i] = cnt;
}

// ---- neighbour-list build, a wavefront per cell ------------------------
//
// Every particle of a cell scans the same 27 cells, so one wavefront takes
// a cell: the 27 cells' candidates, in the order the per-particle scan
// above visits them (rows by z, then y; a row's three cells by x; a cell's
// particles by index), form one sequence that is loaded 64 at a time, one
// candidate per lane, and tested against the cell's particles in turn.
// For each particle the accepted lanes append their ids in lane order (a
// ballot prefix count), so the lists are identical to the per-particle
// scan's (same entries, same order, same test on the same values).  A
// particle's potential mirror sources follow its real entries, through the
// same sequence around its reflection; the particles whose reflections fall
// in one cell take it together.  Where the cells are few, several wavefronts
// share a cell's particles.
//
// What bounds it: the chain of a cell at the wall up to 65,536 particles,
// above the instructions per particle and 64 candidates (24 vector ones; 14 %
// of the candidates are accepted, the cells' share of the sphere).  With the
// reflections scanned one particle at a time and one wavefront per cell that
// chain took 100 us at 4,096 to 131,072 particles, and the build 154 at
// 262,144 and 250 at 524,288; now 17 at 4,096, 39 at 32,768, 87 at 131,072,
// 149 and 244.  Entries gathered in LDS and written by chunks (280 us at
// 524,288: the LDS costs wavefronts) and four particles tested together
// (282) were slower.
// The cell's particles are taken 64 at a time; their positions sit in LDS
// (read with one address by the whole wavefront) and their running counts
// in lane q of `cntv`.
constexpr int LC_WAVES = BLOCK / 64;   // cells per block and pass
constexpr int LC_MAX_BLOCKS = 16384;   // grid-stride launches

__device__ __forceinline__ int sys_of_cell(const GridInfo* grid, int n_sys, int64_t c)
{
    int lo = 0, hi = n_sys - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (grid[mid].cell_base <= c) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// entry pos of particle i, as vl_at places it; cst = n VCHUNK (< 2^30)
__device__ __forceinline__ void vl_put(int32_t* vl, int32_t i, uint32_t cst, uint32_t pos,
                                       int32_t e)
{
    vl[(uint64_t)(pos / VCHUNK) * cst + (uint64_t)(uint32_t)i * VCHUNK + pos % VCHUNK] = e;
}

// The 27 cells around (ccx, ccy, ccz) in scan order, cell l = 9 (z + 1) +
// 3 (y + 1) + (x + 1) for offsets x, y, z in {-1, 0, 1}: lane l < 27
// finds its cell's particle range (empty where the cell does not exist),
// and the wavefront stores the ranges' first particles and the exclusive
// prefix sums of their lengths (lanes 27..31: the total).  Returns the
// total.
__device__ __forceinline__ int cell_seq(const GridInfo& g, const int32_t* __restrict__ cs,
                                        const int32_t* __restrict__ ce, int ccx, int ccy,
                                        int ccz, int32_t* sb, int32_t* so)
{
    const int lane = threadIdx.x & 63;
    const bool px = g.Lx > 0.0, py = g.Ly > 0.0;
    int32_t b = 0, len = 0;
    if (lane < 27) {
        const int zz = ccz + lane / 9 - 1;
        const int yy = nb_cell(ccy, (lane / 3) % 3 - 1, g.ny, py);
        const int xx = nb_cell(ccx, lane % 3 - 1, g.nx, px);
        if (zz >= 0 && zz < g.nz && yy >= 0 && xx >= 0) {
            const int64_t c = g.cell_base + xx + (int64_t)g.nx * (yy + (int64_t)g.ny * zz);
            b = cs[c];
            len = ce[c] - b;
        }
    }
    int inc = len;
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
        const int o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane < 32) {
        sb[lane] = b;
        so[lane] = inc - len;
    }
    wave_sync();
    return __builtin_amdgcn_readlane(inc, 31);
}

// Candidate t (< tot) of the sequence cell_seq stored: the last cell
// whose offset is at most t holds it (an empty cell shares its offset
// with the next one).  Lanes past the sequence take `dflt`.
__device__ __forceinline__ int32_t seq_at(const int32_t* sb, const int32_t* so, int t,
                                          int tot, int32_t dflt)
{
    int lo = 0, hi = 26;
#pragma unroll
    for (int r = 0; r < 5; ++r) {
        const int mid = (lo + hi + 1) >> 1;
        if (so[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return t < tot ? sb[lo] + (t - so[lo]) : dflt;
}

template <bool PERIODIC>
__global__ __launch_bounds__(BLOCK) void k_list_cells(
    int64_t n, int n_sys, const GridInfo* __restrict__ grid,
    const double* __restrict__ p4, const int32_t* __restrict__ cs,
    const int32_t* __restrict__ ce, int64_t n_cells, const int64_t* __restrict__ n_cells_dev,
    int split_bits, int32_t* __restrict__ vl, int32_t* __restrict__ vcnt, ErrWord* err,
    const int32_t* gate)
{
    if (gate && *gate == 0) return;
    __shared__ double4 ppos[LC_WAVES][64];
    __shared__ int32_t seqb[LC_WAVES][32], seqo[LC_WAVES][32];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t* sb = seqb[wv];
    int32_t* so = seqo[wv];
    const int64_t tc = n_cells_dev ? *n_cells_dev : n_cells;
    const int64_t units = tc << split_bits;
    const int64_t step = (int64_t)gridDim.x * LC_WAVES;
    const char* p4b = reinterpret_cast<const char*>(p4);
    const uint32_t cst = (uint32_t)(n * VCHUNK);
    auto load_pos = [&](int32_t j, double& qx, double& qy, double& qz) {
        const double* r = reinterpret_cast<const double*>(p4b + ((uint32_t)j << 5));
        const double2 xy = *reinterpret_cast<const double2*>(r);
        qx = xy.x;
        qy = xy.y;
        qz = r[2];
    };
    // a unit is one share of a cell's particles; the wavefront looks at its
    // next 64 units at once, one per lane, and takes those that hold particles
    // (in a sparse state nearly none does: one unit after another took 436 us
    // at 131,072 particles in 1.1 M cells and 394 at 33,000 in 2.2 M)
    for (int64_t u0 = xcd_block(blockIdx.x, gridDim.x) * LC_WAVES + wv; u0 < units;
         u0 += 64 * step) {
        int32_t mine = 0, mine_end = 0;
        if (u0 + lane * step < units) {
            const int64_t unit = u0 + lane * step, cell = unit >> split_bits;
            const int part = (int)(unit & ((1 << split_bits) - 1));
            const int32_t first = cs[cell], all = ce[cell] - first;
            const int share = (all + (1 << split_bits) - 1) >> split_bits;
            mine = first + part * share;
            mine_end = first + ((part + 1) * share < all ? (part + 1) * share : all);
        }
        for (uint64_t left = __ballot(mine_end > mine); left; left &= left - 1) {
        const int at = __builtin_ctzll(left);
        const int64_t cell = (u0 + at * step) >> split_bits;
        const int32_t cb = __builtin_amdgcn_readlane(mine, at);
        const int32_t cend = __builtin_amdgcn_readlane(mine_end, at);
        const GridInfo& g = grid[sys_of_cell(grid, n_sys, cell)];
        const int loc = (int)(cell - g.cell_base);
        const int cx = loc % g.nx, cy = (loc / g.nx) % g.ny, cz = loc / (g.nx * g.ny);
        const double Rv2 = g.Rv2 * (1.0 + 1e-12);
        int tot = cell_seq(g, cs, ce, cx, cy, cz, sb, so);
        for (int32_t q0 = cb; q0 < cend; q0 += 64) {
            const int nq = cend - q0 < 64 ? cend - q0 : 64;
            const int32_t mi = q0 + lane;          // this lane's particle
            if (lane < nq) {
                const double2* r = reinterpret_cast<const double2*>(p4b + ((uint32_t)mi << 5));
                const double2 a = r[0], c2 = r[1];
                ppos[wv][lane] = make_double4(a.x, a.y, c2.x, 0.0);
            }
            wave_sync();
            int cntv = 0;
            // real candidates
            for (int t0 = 0; t0 < tot; t0 += 64) {
                const bool in = t0 + lane < tot;
                const int32_t j = seq_at(sb, so, t0 + lane, tot, cb);
                double qx, qy, qz;
                load_pos(j, qx, qy, qz);
                for (int q = 0; q < nq; ++q) {
                    const double4 pq = ppos[wv][q];
                    const int32_t iq = q0 + q;
                    const double dx =
                        (PERIODIC ? image_coord(qx, pq.x, g.Lx, g.hLx) : qx) - pq.x;
                    const double dy =
                        (PERIODIC ? image_coord(qy, pq.y, g.Ly, g.hLy) : qy) - pq.y;
                    const double dz = qz - pq.z;
                    const bool acc =
                        in && j != iq && !(fma(dz, dz, fma(dy, dy, dx * dx)) >= Rv2);
                    const uint64_t m = __ballot(acc);
                    if (m) {
                        const int c0 = __builtin_amdgcn_readlane(cntv, q);
                        const uint32_t pos = (uint32_t)c0 + __builtin_amdgcn_mbcnt_hi(
                                                 (uint32_t)(m >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                        if (acc && pos < (uint32_t)VCAP) vl_put(vl, iq, cst, pos, j);
                        cntv = lane == q ? c0 + __popcll(m) : cntv;
                    }
                }
            }
            // potential mirrors of the particles near the wall: reals near the
            // wall that lie near their reflections.  The cell's particles
            // whose reflections fall in one cell (all of them, where the
            // reflections are clamped to the grid's lowest layer) scan its
            // surroundings together, as above.
            const double zq = lane < nq ? ppos[wv][lane].z : 0.0;
            int mcell = -1;
            if (lane < nq && zq - g.wall < g.Rv) {
                int mx, my, mz;
                cell_clamp(g, ppos[wv][lane].x, ppos[wv][lane].y,
                           dsub(dmul(2.0, g.wall), zq), mx, my, mz);
                mcell = mx + g.nx * (my + g.ny * mz);
            }
            uint64_t todo = __ballot(mcell >= 0);
            const bool reseq = todo != 0ull;
            while (todo) {
                const int mc = __builtin_amdgcn_readlane(mcell, __builtin_ctzll(todo));
                const uint64_t same = __ballot(mcell == mc);
                todo &= ~same;
                wave_sync();
                const int mtot = cell_seq(g, cs, ce, mc % g.nx, (mc / g.nx) % g.ny,
                                          mc / (g.nx * g.ny), sb, so);
                for (int t0 = 0; t0 < mtot; t0 += 64) {
                    const int32_t j = seq_at(sb, so, t0 + lane, mtot, cb);
                    double qx, qy, qz;
                    load_pos(j, qx, qy, qz);
                    const bool in = t0 + lane < mtot && qz - g.wall < g.Rv;
                    for (uint64_t rest = same; rest; rest &= rest - 1) {
                        const int q = __builtin_ctzll(rest);
                        const double4 pq = ppos[wv][q];
                        const int32_t iq = q0 + q;
                        const double dx =
                            (PERIODIC ? image_coord(qx, pq.x, g.Lx, g.hLx) : qx) - pq.x;
                        const double dy =
                            (PERIODIC ? image_coord(qy, pq.y, g.Ly, g.hLy) : qy) - pq.y;
                        const double dz = qz - dsub(dmul(2.0, g.wall), pq.z);
                        const bool acc = in && !(fma(dz, dz, fma(dy, dy, dx * dx)) >= Rv2);
                        const uint64_t m = __ballot(acc);
                        if (m) {
                            const int c0 = __builtin_amdgcn_readlane(cntv, q);
                            const uint32_t pos = (uint32_t)c0 + __builtin_amdgcn_mbcnt_hi(
                                                     (uint32_t)(m >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                            if (acc && pos < (uint32_t)VCAP)
                                vl_put(vl, iq, cst, pos, j | MBIT);
                            cntv = lane == q ? c0 + __popcll(m) : cntv;
                        }
                    }
                }
            }
            if (lane < nq) {
                if (cntv > VCAP) {
                    raise_error(err, ERR_CAPACITY, mi);
                    cntv = VCAP;
                }
                vcnt[mi] = cntv;
            }
            // the next chunk's positions (and the cell's own sequence, if
            // a mirror scan replaced it) overwrite the LDS words
            wave_sync();
            if (reseq && q0 + 64 < cend) tot = cell_seq(g, cs, ce, cx, cy, cz, sb, so);
        }
        wave_sync();
        }
    }
}

// ---- mirrors of the current state --------------------------------------

template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* wsum,
                                                    uint32_t& total)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t inc = v;
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
    for (int w = 0; w < NT / 64; ++w) {
        if (w < wave) pre += wsum[w];
        tot += wsum[w];
    }
    __syncthreads();
    total = tot;
    return pre + inc - v;
}

// Wall flags of the SORT_ITEMS chunks of 64 particles from wb on (chunk q:
// particles wb + 64 q + lane, false past n) as wave masks, bit l for
// particle wb + 64 q + l; all heights are loaded before any test.  s_tile:
// the system of the whole tile, or -1 when the tile spans several.
__device__ __forceinline__ void wall_masks(int64_t n, int n_sys, const int64_t* off,
                                           const GridInfo* grid, const double* z, int64_t wb,
                                           int s_tile, uint64_t (&m)[SORT_ITEMS])
{
    const int lane = threadIdx.x & 63;
    double zz[SORT_ITEMS];
#pragma unroll
    for (int q = 0; q < SORT_ITEMS; ++q) {
        const int64_t i = wb + 64 * q + lane;
        zz[q] = i < n ? z[i] : INFINITY;
    }
    if (s_tile >= 0) {
        const double wall = grid[s_tile].wall, R = grid[s_tile].R;
#pragma unroll
        for (int q = 0; q < SORT_ITEMS; ++q) m[q] = __ballot(dsub(zz[q], wall) < R);
    } else {
#pragma unroll
        for (int q = 0; q < SORT_ITEMS; ++q) {
            const int64_t i = wb + 64 * q + lane;
            bool f = false;
            if (i < n) {
                const GridInfo& g = grid[sys_of(off, n_sys, i)];
                f = dsub(zz[q], g.wall) < g.R;
            }
            m[q] = __ballot(f);
        }
    }
}

// The system holding every particle of tile `tile`, or -1.
__device__ __forceinline__ int tile_system(int64_t n, int n_sys, const int64_t* off,
                                           int64_t tile)
{
    const int64_t t0 = tile * SORT_TILE;
    const int64_t t1 = t0 + SORT_TILE - 1 < n ? t0 + SORT_TILE - 1 : n - 1;
    const int s0 = sys_of(off, n_sys, t0);
    return s0 == sys_of(off, n_sys, t1) ? s0 : -1;
}

// Mirrors are counted and numbered a tile of SORT_TILE particles per block:
// wave w takes the SORT_ITEMS chunks of 64 consecutive particles from
// t0 + 64 SORT_ITEMS w on, one particle per lane (coalesced loads of z),
// with the wall flags of a chunk as one ballot mask.
constexpr int MIRROR_WAVES = BLOCK / 64;
static_assert(SORT_TILE == MIRROR_WAVES * 64 * SORT_ITEMS, "a tile per block");

// Also clears the step's counters: the selection's list of particles for
// its second kernel, the fits' refit list and the displacement maximum of
// the next list check (read by the host before this kernel is enqueued).
__global__ void k_mirror_count(int64_t n, int n_sys, const int64_t* off,
                               const GridInfo* grid, const double* z,
                               int32_t* bsum, unsigned int* hard_n,
                               unsigned int* redo_n, Summary* sum)
{
    __shared__ uint32_t wsum[MIRROR_WAVES];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *hard_n = 0u;
        *redo_n = 0u;
        sum->disp = DISP_ZERO;
    }
    const int w = threadIdx.x >> 6;
    const int s_tile = tile_system(n, n_sys, off, blockIdx.x);
    const int64_t wb = (int64_t)blockIdx.x * SORT_TILE + (int64_t)w * 64 * SORT_ITEMS;
    uint64_t m[SORT_ITEMS];
    wall_masks(n, n_sys, off, grid, z, wb, s_tile, m);
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < SORT_ITEMS; ++q) c += (uint32_t)__popcll(m[q]);
    if ((threadIdx.x & 63) == 0) wsum[w] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tot = 0;
#pragma unroll
        for (int q = 0; q < MIRROR_WAVES; ++q) tot += wsum[q];
        bsum[blockIdx.x] = (int32_t)tot;
    }
}

// k_mirror_count and k_mirror_write in one launch, for few particles: a tile
// per block of MIRROR_NT threads, each block counting the mirrors of the
// tiles before its own again (at most MIRROR_ONE_MAX heights in all, from L2)
// instead of waiting for a launch that has.  Two launches took 2.2 and 3.6 us
// and the gap between them at 4,096 particles; one takes 3.2.
constexpr int MIRROR_NT = 1024;
constexpr int64_t MIRROR_ONE_MAX = 32768;
__global__ __launch_bounds__(MIRROR_NT) void k_mirror_one(
    int64_t n, int n_sys, const int64_t* off, const GridInfo* grid, const double* z,
    unsigned int* hard_n, unsigned int* redo_n, Summary* sum, int32_t* mirror_of, int32_t* msrc)
{
    constexpr int PER = SORT_TILE / MIRROR_NT;
    __shared__ uint32_t wsum[MIRROR_NT / 64], before;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (t == 0) {
        before = 0u;
        if (blockIdx.x == 0) {
            *hard_n = 0u;
            *redo_n = 0u;
            sum->disp = DISP_ZERO;
        }
    }
    const int64_t t0 = (int64_t)blockIdx.x * SORT_TILE;
    const bool one = n_sys == 1;
    const double wall0 = grid[0].wall, R0 = grid[0].R;
    auto near = [&](int64_t i, double zi) {
        double wall = wall0, R = R0;
        if (!one) {
            const GridInfo& g = grid[sys_of(off, n_sys, i)];
            wall = g.wall;
            R = g.R;
        }
        return dsub(zi, wall) < R;
    };
    // this tile's heights first: wavefront w takes particles 64 PER w + 64 q
    double zz[PER];
    const int64_t wb = t0 + 64 * PER * w + lane;
#pragma unroll
    for (int q = 0; q < PER; ++q) zz[q] = wb + 64 * q < n ? z[wb + 64 * q] : INFINITY;
    __syncthreads();
    uint32_t c = 0u;
#pragma unroll 4
    for (int64_t i = t; i < t0; i += MIRROR_NT) c += near(i, z[i]) ? 1u : 0u;
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d);
    if (lane == 0 && c) atomicAdd(&before, c);
    uint64_t m[PER];
    uint32_t mine = 0u;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        m[q] = __ballot(wb + 64 * q < n && near(wb + 64 * q, zz[q]));
        mine += (uint32_t)__popcll(m[q]);
    }
    if (lane == 0) wsum[w] = mine;
    __syncthreads();
    uint32_t k = before, tot = before;
    for (int q = 0; q < MIRROR_NT / 64; ++q) {
        k += q < w ? wsum[q] : 0u;
        tot += wsum[q];
    }
    if (blockIdx.x == gridDim.x - 1 && t == 0) sum->n_mirror = (int64_t)tot;
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int64_t i = wb + 64 * q;
        if (i < n) {
            const bool f = (m[q] >> lane) & 1ull;
            const uint32_t kk = k + (uint32_t)__popcll(m[q] & below);
            mirror_of[i] = f ? (int32_t)kk : -1;
            if (f) msrc[kk] = (int32_t)i;
        }
        k += (uint32_t)__popcll(m[q]);
    }
}

// Exclusive scan in place of a uint32 array (single block of 1024); the
// total goes to *total.
__global__ void k_scan_total(uint32_t* a, int64_t cnt, int64_t* total)
{
    __shared__ uint32_t part[1024];
    const int t = threadIdx.x;
    const int64_t chunk = (cnt + 1023) / 1024;
    const int64_t b = t * chunk;
    const int64_t e = (b + chunk < cnt) ? b + chunk : cnt;
    uint32_t s = 0;
    for (int64_t i = b; i < e; ++i) s += a[i];
    part[t] = s;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        uint32_t v = t >= d ? part[t - d] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    uint32_t run = part[t] - s;
    for (int64_t i = b; i < e; ++i) {
        uint32_t v = a[i];
        a[i] = run;
        run += v;
    }
    if (t == 1023) *total = (int64_t)part[1023];
}

// bsum holds the blocks' exclusive offsets (scanned) or their counts; with
// counts (few blocks) each block sums those of the blocks before it and the
// last block writes the total.  Mirror ids follow the source order.
__global__ void k_mirror_write(int64_t n, int n_sys, const int64_t* off,
                               const GridInfo* grid, const int32_t* bsum,
                               int scanned, int64_t* total, const double* z,
                               int32_t* mirror_of, int32_t* msrc)
{
    __shared__ uint32_t wsum[MIRROR_WAVES];
    __shared__ uint32_t bpre[MIRROR_WAVES];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t base;
    if (scanned) {
        base = (uint32_t)bsum[blockIdx.x];
    } else {
        uint32_t p = 0;
        for (int q = threadIdx.x; q < (int)blockIdx.x; q += BLOCK) p += (uint32_t)bsum[q];
        for (int d = 32; d > 0; d >>= 1) p += __shfl_xor(p, d);
        if (lane == 0) bpre[w] = p;
        __syncthreads();
        base = 0;
#pragma unroll
        for (int q = 0; q < MIRROR_WAVES; ++q) base += bpre[q];
    }
    const int s_tile = tile_system(n, n_sys, off, blockIdx.x);
    const int64_t wb = (int64_t)blockIdx.x * SORT_TILE + (int64_t)w * 64 * SORT_ITEMS;
    uint64_t m[SORT_ITEMS];
    wall_masks(n, n_sys, off, grid, z, wb, s_tile, m);
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < SORT_ITEMS; ++q) c += (uint32_t)__popcll(m[q]);
    if (lane == 0) wsum[w] = c;
    __syncthreads();
    uint32_t k = base, tot = 0;
#pragma unroll
    for (int q = 0; q < MIRROR_WAVES; ++q) {
        k += q < w ? wsum[q] : 0u;
        tot += wsum[q];
    }
    if (!scanned && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        *total = (int64_t)(base + tot);
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int q = 0; q < SORT_ITEMS; ++q) {
        const int64_t i = wb + 64 * q + lane;
        if (i < n) {
            const bool f = (m[q] >> lane) & 1ull;
            const uint32_t kk = k + (uint32_t)__popcll(m[q] & below);
            mirror_of[i] = f ? (int32_t)kk : -1;
            if (f) msrc[kk] = (int32_t)i;
        }
        k += (uint32_t)__popcll(m[q]);
    }
}

// ---- stencil selection ---------------------------------------------------
//
// L adjacent lanes per particle; lane `sub` takes the list entries
// 4 L c + 4 sub + u (chunk c, u = 0..3): one 16-byte load of list words (8
// bytes of slot words) per chunk, and an entry's bit of the keep mask is
// 4 L c + 4 sub + u as well.  Every entry is tested exactly once and leaves
//   - a 15-bit key, r^2 rounded down to units of R^2/32766 (0x7FFF: not a
//     candidate), two to a register,
//   - its octant, a nibble;
// and the group's OR over its entries gives the octants that hold
// candidates, those that hold one below half of R^2, and those covered.
// The cut is a key value T with exactly m_max keys below it, found by
// counting keys below trial values (three packed 16-bit operations per two
// entries; the first trial from count ~ r^3, then bisection).  The m_max
// nearest are the stencil when every octant with candidates has one below
// T, which one below half of R^2 shows for nearly every particle.  Otherwise
//   - the first of an octant without a candidate below the cut is kept for
//     itself (forced) and the others are cut again, until no octant is
//     missing (no particle of a column, 1 % of a sheared one);
//   - candidates tied at the cut (or for an octant's first) are ranked by
//     their exact keys (r^2, id) (0.2 % of the particles).
//
// What bounds it: a thread per particle (r^2 buckets in LDS, two passes)
// waited for memory up to 131,072 particles (54 us at 4,096, 60 at 33,263,
// 73 at 131,072), and above for its uncoalesced gathers and 7,300 VALU
// instructions per wavefront (106 us at 262,144, 188 at 524,288, 781 on the
// sheared 1,048,576).  With L lanes the chains are L times shorter and the
// lists are read coalesced: 9 us (L = 16), 20 (L = 8), 47 (L = 8).  Above
// that the vector ALU bounds it (L = 4: 1,840 instructions per 16 particles,
// 98 us of issue at 524,288) once the gathers go to the tile's sources in
// LDS: 66, 119 and 394 us (76, 136 and 427 from the records; 71, 131 and 410
// with the kept rows written for the fits).  There the rare
// cases take a kernel of their own (k_select_rest, 13 us): with them the
// four-lane form needs 150 registers and 87 us at 262,144.
typedef short s16x2 __attribute__((ext_vector_type(2)));

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}

// f over the L lanes of a group, the same value in every lane: swaps of
// neighbours and pairs inside quads, then the half-row and row mirrors.
template <int L, class F>
__device__ __forceinline__ uint32_t group_red(uint32_t x, F&& f)
{
    static_assert(L == 2 || L == 4 || L == 8 || L == 16, "lanes of one DPP row");
    x = f(x, dpp_u32<0xB1>(x));
    if (L >= 4) x = f(x, dpp_u32<0x4E>(x));
    if (L >= 8) x = f(x, dpp_u32<0x141>(x));
    if (L >= 16) x = f(x, dpp_u32<0x140>(x));
    return x;
}
template <int L>
__device__ __forceinline__ uint32_t group_add(uint32_t x)
{
    return group_red<L>(x, [](uint32_t a, uint32_t b) { return a + b; });
}
template <int L>
__device__ __forceinline__ uint32_t group_or(uint32_t x)
{
    return group_red<L>(x, [](uint32_t a, uint32_t b) { return a | b; });
}
template <int L>
__device__ __forceinline__ uint32_t group_min(uint32_t x)
{
    return group_red<L>(x, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
}

// f(integral_constant<int, K>) for K = B .. E-1, in order
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// A value that is the same in all active lanes, as a scalar.
__device__ __forceinline__ double scalar(double x)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                            __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// Hides a value's origin from the compiler.
__device__ __forceinline__ void hide(uint32_t& x) { asm volatile("" : "+v"(x)); }

constexpr uint32_t NO_KEY = 0x7FFFu;     // key of an entry that is no candidate
constexpr uint32_t HALF_KEY = 0x4000u;   // keys below: r^2 < R^2/2 (about)

// -1 in each half whose key is below T's (both in [0, 0x7FFF])
__device__ __forceinline__ s16x2 key_below(uint32_t pair, s16x2 T)
{
    return (__builtin_bit_cast(s16x2, pair) - T) >> 15;
}

// LDS for the tied candidates of one group (cap >= 16).
struct TieList {
    double* r2;
    int32_t* id;
    int cap;
};

// The selection of particle i by a group of L lanes (lane `sub`).  STAGED:
// the positions of the tile's list sources are in (sx, sy, sz), and an
// entry's is read through its slot word; else they are gathered from the
// 32-byte records.  FULL: with every case of the rule; else a particle that
// needs that is appended to `hard`.  write_rows (the same for the group):
// leave the kept rows' slot words, by way of the group's LDS `rows`.
template <int L, bool STAGED, bool PERIODIC, bool FULL>
__device__ __forceinline__ void select_particle(const View& v, int64_t i, int sub,
                                                const double* sx, const double* sy,
                                                const double* sz, TieList ties, int32_t* hard,
                                                unsigned int* hard_n, int force_rest,
                                                bool write_rows, uint16_t* rows)
{
    constexpr int NCH = VCAP / (4 * L);      // chunks of a full list
    const int64_t n = v.n;
    // One system after another where a wavefront's particles lie in several
    // (a group's lanes share theirs), so that its constants are scalars.
    const int sys = sys_of(v.off, v.n_sys, i);
    for (bool todo = true; todo;) {
    const int s0 = __builtin_amdgcn_readfirstlane(sys);
    if (sys != s0) continue;
    todo = false;
    const GridInfo& g = v.grid[s0];
    const double margin = scalar(dmul(v.ghost_margin, g.h));
    const double R = scalar(g.R), R2 = scalar(g.R2), wall = scalar(g.wall);
    const double kscale = scalar((1.0 - 1.0 / 16384.0) / g.R2);
    // no -0 among these (nor in the records), so that no difference is -0 and
    // an octant follows from sign bits
    Seen s;
    s.xi = v.x[i] + 0.0;
    s.yi = v.y[i] + 0.0;
    s.zi = v.z[i] + 0.0;
    s.wall2 = scalar(dmul(2.0, g.wall) + 0.0);
    s.Lx = scalar(g.Lx);
    s.hLx = scalar(g.hLx);
    s.Ly = scalar(g.Ly);
    s.hLy = scalar(g.hLy);
    const double xi = s.xi, yi = s.yi, zi = s.zi;
    // entry 4 L c + 4 sub + u is in the list when left > 4 L c + u
    const int left = v.vcnt[i] - 4 * sub;

    // ---- exact test of every entry
    uint32_t key[2 * NCH];               // entries (0, 1) and (2, 3) of a chunk
    uint32_t octs[(NCH + 1) / 2];        // octant nibbles, eight entries each
#pragma unroll
    for (int c = 0; c < (NCH + 1) / 2; ++c) octs[c] = 0u;
    // octants: bits 0-7 with candidates, 8-15 with one below HALF_KEY, 16-23
    // covered (a candidate farther than margin on every axis)
    uint32_t seen = 0u;
    int nact = 0;                        // chunks in use in this wavefront
    // a mirror exists while its source lies within R of the wall (the rule
    // that sets mirror_of) and sits at its reflection
    auto reflect = [&](double z) {
        return dsub(z, wall) < R ? dsub(s.wall2, z) : (double)INFINITY;
    };
    // the entries 2 h, 2 h + 1 of chunk c at positions (px, py, pz) of the
    // sources (infinite: no entry).  Every entry takes the same instructions
    // (no divergent branches).
    auto test2 = [&](auto C, auto Hh, const double* px, const double* py, const double* pz) {
        constexpr int c = decltype(C)::value, h = decltype(Hh)::value;
        uint32_t kk[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const double x = PERIODIC ? image_coord(px[u], xi, s.Lx, s.hLx) : px[u];
            const double y = PERIODIC ? image_coord(py[u], yi, s.Ly, s.hLy) : py[u];
            const double dx = dsub(x, xi), dy = dsub(y, yi), dz = dsub(pz[u], zi);
            const double d2 = dist2(dx, dy, dz);
            const bool cand = d2 < R2;
            // octant_of, complemented (the sign bits)
            const uint32_t no = (uint32_t)__double2hiint(dx) >> 31 |
                                ((uint32_t)__double2hiint(dy) >> 31) << 1 |
                                ((uint32_t)__double2hiint(dz) >> 31) << 2;
            const bool far = (int)cand & (int)(fabs(dx) > margin) & (int)(fabs(dy) > margin) &
                             (int)(fabs(dz) > margin);
            const uint32_t hi = (uint32_t)__double2hiint(__builtin_fma(d2, kscale, 1.0));
            const uint32_t kq = (hi >> 5) & 0x7FFFu;
            kk[u] = cand ? kq : NO_KEY;
            uint32_t w = cand ? 1u : 0u;
            w = kk[u] < HALF_KEY ? 0x101u : w;
            seen |= w << no;
            seen |= (far ? 0x10000u : 0u) << no;
            octs[c / 2] |= no << (16 * (c & 1) + 8 * h + 4 * u);
        }
        key[2 * c + h] = kk[0] | (kk[1] << 16);
    };
    // (the first chunks' words stay for the kept rows below)
    constexpr int TIER = (3 * NCH + 7) / 8;
    uint2 w[NCH];
    if constexpr (STAGED) {
        // every chunk's slot words are in flight before the first is used
        const uint2* vs0 = reinterpret_cast<const uint2*>(v.vs + vs_at(n, i, 4 * sub));
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            w[c] = make_uint2(0u, 0u);
            if (__ballot(left > 4 * L * c) == 0ull) continue;
            nact = c + 1;
            w[c] = vs0[(int64_t)c * L * n];
        }
        nact = __builtin_amdgcn_readfirstlane(nact);
        static_for<0, NCH>([&](auto C) {
            constexpr int c = decltype(C)::value;
            if (c >= nact) {
                key[2 * c] = key[2 * c + 1] = NO_KEY | (NO_KEY << 16);
                return;
            }
            // a list's last chunk is padded with STAGE_CAP, the words of
            // chunks past it are arbitrary
            constexpr uint32_t PAD = 8u * STAGE_CAP | (8u * STAGE_CAP << 16);
            const bool none = left <= 4 * L * c;
            static_for<0, 2>([&](auto Hh) {
                const uint32_t ww = none ? PAD : (Hh.value ? w[c].y : w[c].x);
                double px[2], py[2], pz[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t q = u ? ww >> 16 : ww & 0xFFFFu;
                    px[u] = staged_at(sx, q);
                    py[u] = staged_at(sy, q);
                    pz[u] = staged_at(sz, q);
                }
                test2(C, Hh, px, py, pz);
            });
        });
    } else {
        const char* base = reinterpret_cast<const char*>(v.p4);
        // list words of the next chunk are loaded ahead (every particle
        // holds VCAP list slots, so every read is in bounds)
        // (entries 4 sub + 8 a come 8 a n words after entries 4 sub)
        static_assert(4 * L % VCHUNK == 0 || L == 1, "chunks of whole list chunks");
        const int4* vl0 = reinterpret_cast<const int4*>(v.vl + vl_at(n, i, 4 * sub));
        int4 e = vl0[0];
        static_for<0, NCH>([&](auto C) {
            constexpr int c = decltype(C)::value;
            if (__ballot(left > 4 * L * c) == 0ull) {
                key[2 * c] = key[2 * c + 1] = NO_KEY | (NO_KEY << 16);
                return;
            }
            nact = c + 1;
            double px[4], py[4], pz[4];
            bool mir[4];
            const int32_t ev[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // entries past the list's end read the particle's own record;
                // the record offset j * 32 stays below 2^32 (j < 2^27)
                const int32_t ee = left > 4 * L * c + u ? ev[u] : (int32_t)i;
                const double* r = reinterpret_cast<const double*>(
                    base + ((uint32_t)(ee & ~MBIT) << 5));
                const double2 xy = *reinterpret_cast<const double2*>(r);
                px[u] = xy.x;
                py[u] = xy.y;
                pz[u] = r[2];
                mir[u] = (ee & MBIT) != 0;
            }
            if (c + 1 < NCH) e = vl0[(int64_t)(c + 1) * L * n];
            if (__ballot(mir[0] || mir[1] || mir[2] || mir[3]))
#pragma unroll
                for (int u = 0; u < 4; ++u) pz[u] = mir[u] ? reflect(pz[u]) : pz[u];
            if (__ballot(left < 4 * L * c + 4))
#pragma unroll
                for (int u = 0; u < 4; ++u) pz[u] = left > 4 * L * c + u ? pz[u] : INFINITY;
            static_for<0, 2>([&](auto Hh) {
                test2(C, Hh, px + 2 * Hh.value, py + 2 * Hh.value, pz + 2 * Hh.value);
            });
        });
        nact = __builtin_amdgcn_readfirstlane(nact);
    }
    seen = group_or<L>(seen);
    const uint32_t allo = seen & 0xFFu;
    // (octants count from the sign bits here: octant o is bit 7 - o)
    const int gm = (int)(__brev(~(seen >> 16) & 0xFFu) >> 24);
    // f over the chunks in use (and some empty ones): the first TIER chunks
    // without a branch per chunk, which lists of ordinary length fit in
    auto chunks = [&](auto&& f) {
        static_for<0, TIER>(f);
        if (nact > TIER) static_for<TIER, NCH>(f);
    };
    // f(bit 4 c + u, key, octant) for this lane's entries.  For the rare
    // passes: the words are unpacked each time, as copies whose origin the
    // compiler does not see (it would keep every unpacked entry in registers
    // from one pass to the next).
    auto entries = [&](auto&& f) {
        chunks([&](auto C) {
            constexpr int c = decltype(C)::value;
            uint32_t k0 = key[2 * c], k1 = key[2 * c + 1], oo = octs[c / 2];
            hide(k0);
            hide(k1);
            hide(oo);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                f(4 * c + u, ((u < 2 ? k0 : k1) >> (16 * (u & 1))) & 0xFFFFu,
                  (oo >> (16 * (c & 1) + 4 * u)) & 7u);
        });
    };
    // keys of the group below T
    auto below = [&](uint32_t T) -> int {
        const s16x2 t2 = {(short)T, (short)T};
        s16x2 acc = {0, 0};
        chunks([&](auto C) {
            constexpr int c = decltype(C)::value;
            acc += key_below(key[2 * c], t2);
            acc += key_below(key[2 * c + 1], t2);
        });
        return (int)group_add<L>((uint32_t)(-(int)acc.x - (int)acc.y));
    };
    int nc = below(NO_KEY);
    const int m_max = v.m_max;
    const int m = nc < m_max ? nc : m_max;
    int K = m_max;                       // candidates to keep below the cut
    uint32_t T = NO_KEY;                 // the cut
    int tied = 0, need = 0;              // candidates with key T, those kept
    auto cut = [&](bool on) {
        // invariant: below(lo) = cl < K < ch = below(hi)
        uint32_t lo = 0u, hi = NO_KEY;
        int cl = 0, ch = nc;
        bool open = on && nc > K;
        if (on) {
            T = nc <= K ? NO_KEY : 0u;
            tied = need = 0;
        }
        if (open && K == 0) open = false;            // T = 0: none
        uint32_t tr = (uint32_t)(32766.0f * exp2f(0.6666667f * __log2f((float)K / (float)nc)));
        for (int it = 0; __ballot(open) != 0ull; ++it) {
            if (it > 0) tr = (lo + hi) >> 1;
            tr = tr <= lo ? lo + 1u : (tr >= hi ? hi - 1u : tr);
            const int c = below(tr);
            if (!open) continue;
            if (c == K) {
                T = tr;
                open = false;
            } else if (c < K) {
                lo = tr;
                cl = c;
            } else {
                hi = tr;
                ch = c;
            }
            if (open && hi - lo <= 1u) {
                T = lo;
                need = K - cl;
                tied = ch - cl;
                open = false;
            }
        }
    };
    // fewer rows than octants with candidates: their firsts, in octant order
    const bool few = nc > m_max && __popc(allo) > m_max;
    if (few) T = 0u;
    if (__ballot(!few && nc > K)) cut(!few);

    uint64_t kept = 0;                   // this lane's entries kept for themselves
    if constexpr (!FULL) {
        bool rest = force_rest || few || tied > 0;
        // is there an octant whose candidates all lie above the cut?
        const bool doubt = nc > m_max && (T < HALF_KEY || ((seen >> 8) & 0xFFu) != allo);
        if (__ballot(doubt) != 0ull) {
            uint32_t ko = 0u;
            entries([&](int, uint32_t k, uint32_t o) { ko |= k < T ? 1u << o : 0u; });
            rest = rest || (doubt && group_or<L>(ko) != allo);
        }
        // one atomic per wavefront
        const uint64_t rb = __ballot(rest && sub == 0);
        if (rb) {
            const int lane = (int)(threadIdx.x & 63u), lead = __builtin_ctzll(rb);
            uint32_t at = 0u;
            if (lane == lead) at = atomicAdd(hard_n, (uint32_t)__popcll(rb));
            at = __shfl(at, lead);
            if (rest && sub == 0)
                hard[at + (uint32_t)__popcll(rb & ((1ull << lane) - 1ull))] = (int32_t)i;
            if (rest) continue;
        }
    } else {

    // of the group's cnt_mem entries `mem` (this lane's),
    // those of this lane among the `need_mem` smallest exact keys (r^2, id)
    auto smallest = [&](uint64_t mem, int cnt_mem, int need_mem) -> uint64_t {
        const int own = __popcll(mem);
        int at = own;
#pragma unroll
        for (int d = 1; d < L; d <<= 1) {
            const int o = __shfl_up(at, d, L);
            if (sub >= d) at += o;
        }
        at -= own;
        // (this is rare: the particle's own values are read again here)
        const Seen own_s = seen_from(v, g, i);
        // exact key of this group's lane ln's entry e
        auto exact = [&](int ln, int e, double& r2, int32_t& id) {
            const int32_t le[1] = {v.vl[vl_at(n, i, 4 * L * (e >> 2) + 4 * ln + (e & 3))]};
            Pt p[1];
            gather_list(v, own_s, le, p);
            r2 = dist2(dsub(p[0].x, own_s.xi), dsub(p[0].y, own_s.yi),
                       dsub(p[0].z, own_s.zi));
            id = p[0].id;
        };
        uint64_t out = 0;
        if (__ballot(cnt_mem > ties.cap) != 0ull) {
            // too many for the list (points at equal distances): every
            // member against every other, the members named in LDS
            wave_sync();
            ties.r2[sub] = __longlong_as_double((long long)mem);
            wave_sync();
            for (uint64_t b = mem; b; b &= b - 1) {
                double ra, rb;
                int32_t ia, ib;
                exact(sub, __builtin_ctzll(b), ra, ia);
                int less = 0;
                for (int ln = 0; ln < L; ++ln)
                    for (uint64_t o = (uint64_t)__double_as_longlong(ties.r2[ln]); o;
                         o &= o - 1) {
                        exact(ln, __builtin_ctzll(o), rb, ib);
                        less += key_less(rb, ib, ra, ia) ? 1 : 0;
                    }
                if (less < need_mem) out |= b & (0ull - b);
            }
            wave_sync();
            return out;
        }
        int q = at;
        for (uint64_t b = mem; b; b &= b - 1, ++q) {
            double r2;
            int32_t id;
            exact(sub, __builtin_ctzll(b), r2, id);
            ties.r2[q] = r2;
            ties.id[q] = id;
        }
        wave_sync();
        q = at;
        for (uint64_t b = mem; b; b &= b - 1, ++q) {
            const double r2 = ties.r2[q];
            const int32_t id = ties.id[q];
            int less = 0;
            for (int o = 0; o < cnt_mem; ++o)
                less += key_less(ties.r2[o], ties.id[o], r2, id) ? 1 : 0;
            if (less < need_mem) out |= b & (0ull - b);
        }
        wave_sync();
        return out;
    };

    // ---- octants without a candidate below the cut: force their first
    uint32_t fo = 0u;
    bool open = nc > m_max;
    while (__ballot(open) != 0ull) {
        uint32_t ko = 0u;
        entries([&](int, uint32_t k, uint32_t o) { ko |= k < T ? 1u << o : 0u; });
        ko = group_or<L>(ko);
        const uint32_t miss = open ? allo & ~(ko | fo) : 0u;
        open = miss != 0u && K > 0;
        if (__ballot(open) == 0ull) break;
        // (octant o is bit 7 - o here: the highest bit is the first octant)
        const uint32_t mo = open ? 31u - (uint32_t)__builtin_clz(miss) : 8u;
        uint32_t mk = NO_KEY;
        entries([&](int, uint32_t k, uint32_t o) { mk = o == mo && k < mk ? k : mk; });
        mk = group_min<L>(mk);
        uint64_t hit = 0;
        entries([&](int b, uint32_t k, uint32_t o) {
            hit |= open && o == mo && k == mk ? 1ull << b : 0ull;
        });
        const int hits = (int)group_add<L>((uint32_t)__popcll(hit));
        if (__ballot(open && hits > 1)) {
            const uint64_t f = smallest(open && hits > 1 ? hit : 0ull, hits, 1);
            if (open && hits > 1) hit = f;
        }
        if (open) {
            kept |= hit;
            fo |= 1u << mo;
            --K;
        }
        // (T falls with K, so a forced entry's key stays at or above it)
        cut(open && !few);
    }

    // ---- candidates tied at the cut: the `need` smallest exact keys
    if (__ballot(tied > 0) != 0ull) {
        uint64_t mem = 0;
        entries([&](int b, uint32_t k, uint32_t) {
            mem |= tied > 0 && k == T ? 1ull << b : 0ull;
        });
        mem &= ~kept;
        const int cm = (int)group_add<L>((uint32_t)__popcll(mem));
        kept |= smallest(mem, cm, need);
    }
    }

    // ---- keep mask: the keys below the cut, and `kept`
    uint32_t mw[2 * MASK_WORDS];
#pragma unroll
    for (int w = 0; w < 2 * MASK_WORDS; ++w) mw[w] = 0u;
    {
        const s16x2 t2 = {(short)T, (short)T};
        // first bit of a chunk in the mask, less 4 sub
        constexpr int STEP = 4 * L;
        chunks([&](auto C) {
            constexpr int c = decltype(C)::value;
            // (both halves of a pair are 0 or -1)
            const uint32_t d0 = __builtin_bit_cast(uint32_t, key_below(key[2 * c], t2));
            const uint32_t d1 = __builtin_bit_cast(uint32_t, key_below(key[2 * c + 1], t2));
            const uint32_t nib = (d0 & 1u) | ((d0 >> 16) & 2u) | (d1 & 4u) | ((d1 >> 16) & 8u);
            mw[STEP * c / 32] |= nib << (STEP * c % 32);
        });
        if (FULL && __ballot(kept != 0ull) != 0ull)
            chunks([&](auto C) {
                constexpr int c = decltype(C)::value;
                mw[STEP * c / 32] |= ((uint32_t)(kept >> (4 * c)) & 0xFu) << (STEP * c % 32);
            });
    }
    // (4 sub stays inside the chunk's 4 L bits; L = 16: across two words)
    if (L == 16) {
#pragma unroll
        for (int w = 0; w < MASK_WORDS; ++w) {
            const uint32_t x = mw[2 * w];
            mw[2 * w] = sub < 8 ? x << (4 * (sub & 7)) : 0u;
            mw[2 * w + 1] = sub < 8 ? 0u : x << (4 * (sub & 7));
        }
    } else {
#pragma unroll
        for (int w = 0; w < 2 * MASK_WORDS; ++w) mw[w] <<= 4 * sub;
    }
#pragma unroll
    for (int w = 0; w < 2 * MASK_WORDS; ++w) mw[w] = group_or<L>(mw[w]);
    if (sub == 0) {
        v.rec[REC_M * n + i] = m;
        v.rec[REC_GM * n + i] = gm;
    }
#pragma unroll
    for (int w = 0; w < MASK_WORDS; ++w)
        if (sub == w % L)
            v.kmask[w * n + i] = (uint64_t)mw[2 * w] | ((uint64_t)mw[2 * w + 1] << 32);

    // ---- the kept rows' slot words, in list order, for the fits of a staged
    // tile: ranked by the mask, gathered in LDS, written by chunks.  (It
    // costs the selection 17 us of 131 at 524,288 particles and saves the two
    // fits, which walked the mask over the list's words, some 80.)
    if (write_rows) {
        const uint2* vs0 = reinterpret_cast<const uint2*>(v.vs + vs_at(n, i, 4 * sub));
        static_for<STAGED ? TIER : 0, NCH>([&](auto C) {
            constexpr int c = decltype(C)::value;
            w[c] = make_uint2(0u, 0u);
            if (c < nact && left > 4 * L * c) w[c] = vs0[(int64_t)c * L * n];
        });
        int before = 0;                  // rows of the mask words before
        static_for<0, NCH>([&](auto C) {
            constexpr int c = decltype(C)::value;
            if (c >= nact) return;
            constexpr int W = 4 * L * c / 32;
            const uint32_t word = L == 16 && sub >= 8 ? mw[W + 1] : mw[W];
            const int sh = L == 16 ? 4 * (sub & 7) : 4 * L * c % 32 + 4 * sub;
            int row = before + __popc(word & ((1u << sh) - 1u));
            if (L == 16) row += sub >= 8 ? __popc(mw[W]) : 0;
            const uint32_t nib = word >> sh;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t e = u < 2 ? w[c].x : w[c].y;
                if ((nib >> u) & 1u)
                    rows[row] = (uint16_t)(u & 1 ? e >> 16 : e);
                row += (int)((nib >> u) & 1u);
            }
            if (L == 16) before += __popc(mw[W]) + __popc(mw[W + 1]);
            else if (4 * L * (c + 1) % 32 == 0) before += __popc(mw[W]);
        });
        wave_sync();
        for (int q = sub; 4 * q < m; q += L)
            *reinterpret_cast<uint2*>(v.ks + vs_at(n, i, 4 * q)) =
                *reinterpret_cast<const uint2*>(rows + 4 * q);
        wave_sync();
    }
    }
}

// LDS words of one particle's rows (a multiple of 4, and of a stride that
// spreads the particles over the banks)
constexpr int ROW_LDS = MMAX_LIMIT + 4;

// Do the fits read particle i's rows from its tile's staged sources?
__device__ __forceinline__ bool rows_wanted(const View& v, int64_t i)
{
    return v.map_ok && stage_unit(v, i / BLOCK, (int)(i % BLOCK) / HALF).S >= 0;
}

// Threads per block of the selection: with staging, half a tile at L = 4.
constexpr int sel_threads(bool staged) { return staged ? 512 : 256; }

// Gathers from the records, every case of the rule in one kernel.
template <int L, bool PERIODIC>
__global__ __launch_bounds__(BLOCK, 4) void k_select_full(View v)
{
    constexpr int P = BLOCK / L;
    constexpr int TIE_CAP = 64;
    __shared__ double tie_r2[P][TIE_CAP];
    __shared__ int32_t tie_id[P][TIE_CAP];
    __shared__ __align__(8) uint16_t rows[P][ROW_LDS];
    const int grp = threadIdx.x / L;
    const int64_t i = xcd_block(blockIdx.x, gridDim.x) * P + grp;
    if (i >= v.n) return;
    select_particle<L, false, PERIODIC, true>(v, i, threadIdx.x % L, nullptr, nullptr, nullptr,
                                              TieList{tie_r2[grp], tie_id[grp], TIE_CAP},
                                              nullptr, nullptr, 0, rows_wanted(v, i),
                                              rows[grp]);
}

// Leaves the rare cases to k_select_rest.  STAGED: from the tile's list
// sources staged in LDS; a tile that is not staged gathers from the records,
// as every block does without STAGED.
template <int L, bool STAGED, bool PERIODIC>
__global__ __launch_bounds__(sel_threads(STAGED), 4) void k_select(View v, int32_t* hard,
                                                                   unsigned int* hard_n,
                                                                   int force_rest)
{
    constexpr int NT = sel_threads(STAGED);
    constexpr int P = NT / L;                // particles per block
    // slot STAGE_CAP: the source of an entry past a list's end, infinitely
    // far away
    constexpr int NS = STAGED ? STAGE_CAP + 1 : 1;
    __shared__ double sx[NS], sy[NS], sz[NS];
    __shared__ __align__(8) uint16_t rows[STAGED ? P : 1][ROW_LDS];
    const int t = threadIdx.x;
    const int64_t i0 = xcd_block(blockIdx.x, gridDim.x) * P;
    const int64_t i = i0 + t / L;
    int S = -1;                              // staged sources, -1: none
    if (STAGED) {
        static_assert(P <= HALF, "a block lies in half a tile");
        const StageUnit su = stage_unit(v, i0 / BLOCK, (int)(i0 % BLOCK) / HALF);
        S = su.S;
        if (S >= 0) {
            constexpr int SP = (STAGE_CAP + NT - 1) / NT;
            const int32_t* src = su.src;
            int32_t js[SP];
#pragma unroll
            for (int u = 0; u < SP; ++u) js[u] = t + u * NT < S ? src[t + u * NT] : -1;
            double q[3][SP];
#pragma unroll
            for (int u = 0; u < SP; ++u)
                packed_pos(v, js[u] < 0 ? 0 : js[u] & ~MBIT, q[0][u], q[1][u], q[2][u]);
#pragma unroll
            for (int u = 0; u < SP; ++u) {
                if (js[u] < 0) continue;
                if (js[u] & MBIT) {
                    // a mirror exists while its source lies within R of the
                    // wall (the rule that sets mirror_of), at its reflection
                    const GridInfo& g = v.grid[sys_of(v.off, v.n_sys, js[u] & ~MBIT)];
                    q[2][u] = dsub(q[2][u], g.wall) < g.R
                                  ? dsub(dmul(2.0, g.wall) + 0.0, q[2][u]) : (double)INFINITY;
                }
                sx[t + u * NT] = q[0][u];
                sy[t + u * NT] = q[1][u];
                sz[t + u * NT] = q[2][u];
            }
            if (t == 0) sx[STAGE_CAP] = sy[STAGE_CAP] = sz[STAGE_CAP] = INFINITY;
            __syncthreads();
        }
    }
    if (i >= v.n) return;
    const TieList none{nullptr, nullptr, 0};
    if (STAGED && S >= 0)
        select_particle<L, STAGED, PERIODIC, false>(v, i, t % L, sx, sy, sz, none, hard,
                                                    hard_n, force_rest, true, rows[t / L]);
    else
        select_particle<L, false, PERIODIC, false>(v, i, t % L, sx, sy, sz, none, hard,
                                                   hard_n, force_rest, false, nullptr);
}

// The particles k_select has listed, with every case of the rule.
constexpr int REST_LANES = 16;
constexpr int REST_BLOCKS = 1024;

template <bool PERIODIC>
__global__ __launch_bounds__(BLOCK) void k_select_rest(View v, const int32_t* hard,
                                                       const unsigned int* hard_n,
                                                       Counters* cnt)
{
    constexpr int P = BLOCK / REST_LANES;
    __shared__ double tie_r2[P][VCAP];
    __shared__ int32_t tie_id[P][VCAP];
    __shared__ __align__(8) uint16_t rows[P][ROW_LDS];
    const int grp = threadIdx.x / REST_LANES, sub = threadIdx.x % REST_LANES;
    const unsigned int total = *hard_n;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        atomicAdd(&cnt->hard_stencils, (unsigned long long)total);
    for (int64_t q = (int64_t)blockIdx.x * P + grp; q < (int64_t)total;
         q += (int64_t)gridDim.x * P)
        select_particle<REST_LANES, false, PERIODIC, true>(
            v, hard[q], sub, nullptr, nullptr, nullptr, TieList{tie_r2[grp], tie_id[grp], VCAP},
            nullptr, nullptr, 0, rows_wanted(v, hard[q]), rows[grp]);
}

template <int L>
void launch_select_full(lp_ctx* c, const View& v)
{
    const dim3 gb(blocks_for(c->n, BLOCK / L)), bb(BLOCK);
    if (c->periodic)
        hipLaunchKernelGGL((k_select_full<L, true>), gb, bb, 0, c->stream, v);
    else
        hipLaunchKernelGGL((k_select_full<L, false>), gb, bb, 0, c->stream, v);
}

template <int L, bool STAGED>
void launch_select_as(lp_ctx* c, const View& v, int force)
{
    Work& w = c->w;
    constexpr int NT = sel_threads(STAGED);
    const dim3 gb(blocks_for(c->n, NT / L)), bb(NT);
    if (c->periodic)
        hipLaunchKernelGGL((k_select<L, STAGED, true>), gb, bb, 0, c->stream, v, w.hard,
                           w.hard_n, force);
    else
        hipLaunchKernelGGL((k_select<L, STAGED, false>), gb, bb, 0, c->stream, v, w.hard,
                           w.hard_n, force);
}

// The selection in one kernel (k_select_full) up to SELECT_FULL_MAX
// particles, above by k_select and k_select_rest (LP_DEBUG_SORTED_STENCIL:
// always, every particle through the rest).  Measured, us: 131,072
// particles 47 in one, 38 + 13 in two; 262,144 88 and 66 + 13.  16 lanes
// against 8: 4,096 particles 9.5 and 11.1, 12,075 13.6 and 13.5.
constexpr int64_t SELECT_L16_MAX = 8192, SELECT_FULL_MAX = 163840;

bool select_in_one(const lp_ctx* c)
{
    return c->n <= SELECT_FULL_MAX && !(c->cfg.debug_flags & LP_DEBUG_SORTED_STENCIL);
}

void launch_select(lp_ctx* c, const View& v)
{
    c->rows_ok = c->map_ok;
    if (select_in_one(c)) {
        if (c->n <= SELECT_L16_MAX) launch_select_full<16>(c, v);
        else launch_select_full<8>(c, v);
        return;
    }
    const int force = (c->cfg.debug_flags & LP_DEBUG_SORTED_STENCIL) ? 1 : 0;
    if (c->map_ok) launch_select_as<4, true>(c, v, force);
    else launch_select_as<4, false>(c, v, force);
}

void launch_select_rest(lp_ctx* c, const View& v)
{
    if (select_in_one(c)) return;
    Work& w = c->w;
    const unsigned nb = std::min(blocks_for(c->n, BLOCK / REST_LANES), (unsigned)REST_BLOCKS);
    if (c->periodic)
        hipLaunchKernelGGL(k_select_rest<true>, dim3(nb), dim3(BLOCK), 0, c->stream, v,
                           w.hard, w.hard_n, w.cnt);
    else
        hipLaunchKernelGGL(k_select_rest<false>, dim3(nb), dim3(BLOCK), 0, c->stream, v,
                           w.hard, w.hard_n, w.cnt);
}

// ---- exports -----------------------------------------------------------
//
// EXP_LANES adjacent lanes per particle: each tests or reads every
// EXP_LANES-th list entry, the group's ids are gathered in LDS in list order
// and written from there, consecutive lanes to consecutive places.  Lists run
// by rows of cells and ids by the cells' Morton order, so an id's place is the
// count of the smaller ones (unless the list is in order).  (A thread per particle, sorting by
// insertion in its global row, took 484 us for the candidates and 266 for the
// stencils of 49,569 particles, and the offsets summed by one block 105 twice;
// now 57, 37 and 13.)
constexpr int EXP_LANES = 16, EXP_P = BLOCK / EXP_LANES;

// The m ids of a group in ascending order into out.
__device__ __forceinline__ void write_ascending(const int32_t* ids, int m, int sub, int32_t* out)
{
    wave_sync();
    uint32_t bad = 0u;
    for (int q = sub; q + 1 < m; q += EXP_LANES) bad |= ids[q] > ids[q + 1] ? 1u : 0u;
    bad = group_or<EXP_LANES>(bad);
    for (int q = sub; q < m; q += EXP_LANES) {
        const int32_t id = ids[q];
        int at = q;
        if (bad) {
            at = 0;
            for (int o = 0; o < m; ++o) at += ids[o] < id || (ids[o] == id && o < q) ? 1 : 0;
        }
        out[at] = id;
    }
}

// idx null: counts[i + 1] = the candidates of particle i (counts[0] = 0);
// else they go to idx + counts[i].
template <bool WRITE>
__global__ __launch_bounds__(BLOCK) void k_candidates(View v, int64_t* counts, int32_t* idx)
{
    __shared__ int32_t ids[EXP_P][WRITE ? VCAP : 1];
    const int64_t n = v.n;
    const int grp = threadIdx.x / EXP_LANES, sub = threadIdx.x % EXP_LANES;
    const int base = (int)(threadIdx.x & 63u) & ~(EXP_LANES - 1);
    const int64_t i = xcd_block(blockIdx.x, gridDim.x) * EXP_P + grp;
    if (!WRITE && blockIdx.x == 0 && threadIdx.x == 0) counts[0] = 0;
    if (i >= n) return;
    const GridInfo& g = v.grid[sys_of(v.off, v.n_sys, i)];
    const Seen s = seen_from(v, g, i);
    const double R2 = g.R2;
    const int cnt = v.vcnt[i];
    int nc = 0;
    for (int k0 = 0; k0 < cnt; k0 += EXP_LANES) {
        const bool in = k0 + sub < cnt;
        const int32_t e[1] = {in ? v.vl[vl_at(n, i, k0 + sub)] : (int32_t)i};
        Pt p[1];
        gather_list(v, s, e, p);
        const bool cand = in && p[0].valid &&
                          dist2(dsub(p[0].x, s.xi), dsub(p[0].y, s.yi), dsub(p[0].z, s.zi)) < R2;
        const uint32_t m = (uint32_t)(__ballot(cand) >> base) & ((1u << EXP_LANES) - 1u);
        if (WRITE && cand) ids[grp][nc + __popc(m & ((1u << sub) - 1u))] = p[0].id;
        nc += __popc(m);
    }
    if (WRITE) write_ascending(ids[grp], nc, sub, idx + counts[i]);
    else if (sub == 0) counts[i + 1] = nc;
}

// Inclusive sums in place of a[1..n], SORT_TILE of them per block, in two
// launches: the blocks' sums (at most VCAP SORT_TILE each), then every block
// adds those before it (from L2) to its own running sums.
__global__ __launch_bounds__(BLOCK) void k_sum_i64(const int64_t* a, int64_t n, int32_t* bsum)
{
    __shared__ int part[BLOCK / 64];
    const int64_t b = 1 + (int64_t)blockIdx.x * SORT_TILE;
    int s = 0;
    for (int q = threadIdx.x; q < SORT_TILE; q += BLOCK) s += b + q <= n ? (int)a[b + q] : 0;
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x / 64] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int w = 0; w < BLOCK / 64; ++w) tot += part[w];
        bsum[blockIdx.x] = tot;
    }
}
__global__ __launch_bounds__(BLOCK) void k_scan_i64(int64_t* a, int64_t n, const int32_t* bsum)
{
    __shared__ long long before;
    __shared__ uint32_t wsum[BLOCK / 64];
    const int t = threadIdx.x;
    if (t == 0) before = 0;
    __syncthreads();
    long long p = 0;
    for (int q = t; q < (int)blockIdx.x; q += BLOCK) p += bsum[q];
    for (int d = 32; d > 0; d >>= 1) p += __shfl_xor(p, d);
    if ((t & 63) == 0 && p)
        atomicAdd(reinterpret_cast<unsigned long long*>(&before), (unsigned long long)p);
    const int64_t b = 1 + (int64_t)blockIdx.x * SORT_TILE + t * SORT_ITEMS;
    uint32_t c[SORT_ITEMS], mine = 0u, total = 0u;
#pragma unroll
    for (int q = 0; q < SORT_ITEMS; ++q) {
        c[q] = b + q <= n ? (uint32_t)a[b + q] : 0u;
        mine += c[q];
    }
    const uint32_t at = block_excl_scan<BLOCK>(mine, wsum, total);
    long long run = before + at;
#pragma unroll
    for (int q = 0; q < SORT_ITEMS; ++q) {
        run += c[q];
        if (b + q <= n) a[b + q] = run;
    }
}

__global__ __launch_bounds__(BLOCK) void k_export_stencils(View v, int32_t* cnt_out,
                                                           int32_t* idx_out, uint8_t* gm_out)
{
    __shared__ int32_t ids[EXP_P][MMAX_LIMIT];
    const int64_t n = v.n;
    const int grp = threadIdx.x / EXP_LANES, sub = threadIdx.x % EXP_LANES;
    const int64_t i = xcd_block(blockIdx.x, gridDim.x) * EXP_P + grp;
    if (i >= n) return;
    const Rec r = load_rec(v, i);
    if (sub == 0) {
        if (gm_out) gm_out[i] = (uint8_t)r.gm;
        if (cnt_out) cnt_out[i] = r.m;
    }
    if (!idx_out) return;
    int m = 0;
#pragma unroll
    for (int w = 0; w < MASK_WORDS; ++w) {
        if (r.mask[w] == 0) continue;
#pragma unroll
        for (int c = 0; c < 64; c += EXP_LANES) {
            const uint32_t bits = (uint32_t)(r.mask[w] >> c) & ((1u << EXP_LANES) - 1u);
            if ((bits >> sub) & 1u) {
                const int32_t e = v.vl[vl_at(n, i, 64 * w + c + sub)];
                const int at = m + __popc(bits & ((1u << sub) - 1u));
                ids[grp][at] = e & MBIT ? (int32_t)n + v.mirror_of[e & ~MBIT] : e;
            }
            m += __popc(bits);
        }
    }
    int32_t* out = idx_out + i * v.m_max;
    write_ascending(ids[grp], m, sub, out);
    for (int q = m + sub; q < v.m_max; q += EXP_LANES) out[q] = -1;
}

// ---- tile map: the distinct list sources of each tile ------------------
//
// One block per tile of BLOCK consecutive particles, MAP_SPLIT threads per
// particle (each takes every MAP_SPLIT-th batch of its list: the chains are
// that much shorter).  Sources are found in
// granules of 16 consecutive ids: a list holds runs of consecutive ids
// (the particles of a cell), so a thread looks a granule up in an LDS hash
// table only where its id's granule changes (about 40 times in 77 entries)
// and marks each source by a plain byte store, which many threads may do at
// once.  The granules present are ranked by id, a prefix sum of their marks
// numbers the sources in ascending order, and every list entry then gets the
// slot of its source (a 16-bit word).  A mirror is a source of its own, named
// MBIT | the particle it reflects, so mirrors come after the real ones.
// A tile with more than STAGE_CAP sources is numbered by halves; a half with
// too many is not staged, nor is a tile with more granules than the table
// holds.
//
// What bounds it: one tile's chain up to 131,072 particles, the list's bytes
// in and the words' bytes out (twice) above.  Inserting every entry by LDS
// compare-and-swap and sorting the sources (66 bitonic steps) took 75 us at
// 4,096 particles, 87 at 32,768, 100 at 131,072, 146 at 262,144 and 230 at
// 524,288; by granules it is 16, 20, 30, 55 and 115 (about 400 MB there,
// 80 us at the copy rate).  The map is built before the selection, which
// then reads staged positions in the passes that rebuild too; on a second
// stream beside the selection the two took longer than in line (114 us at
// 262,144 for the map alone).

constexpr int GRAN = 16;               // ids per granule
constexpr int GRAN_SLOTS = 1024;       // granules per tile (power of 2)
static_assert(GRAN * GRAN_SLOTS <= 0x10000 && STAGE_CAP < 0x2000, "16-bit places and slots");
constexpr int MAP_SPLIT = 4, MAP_NT = BLOCK * MAP_SPLIT;
static_assert(GRAN_SLOTS % MAP_NT == 0 && GRAN == 16, "tile map sizes");

__global__ __launch_bounds__(MAP_NT, 8) void k_tile_map(
    int64_t n, const int32_t* __restrict__ vl, const int32_t* __restrict__ vcnt,
    int32_t* __restrict__ tile_src, int32_t* __restrict__ tile_cnt,
    uint16_t* __restrict__ vs, int disable, const int32_t* gate)
{
    if (gate && *gate == 0) return;
    constexpr int PER = GRAN_SLOTS / MAP_NT;
    __shared__ int32_t gkey[GRAN_SLOTS];               // granule of a table place, -1: free
    // a byte per half tile and id of each place
    __shared__ uint32_t mark[2][GRAN_SLOTS * GRAN / 4];
    __shared__ int32_t list[GRAN_SLOTS];               // the places in use
    __shared__ int32_t lkey[GRAN_SLOTS];               // and their granules
    __shared__ uint32_t rcnt[GRAN_SLOTS];              // marks of the granule of each rank
    __shared__ uint32_t wsum[MAP_NT / 64];
    __shared__ int full, ng, reals;
    const int t = threadIdx.x;
    const int64_t tile = blockIdx.x;
    const int64_t i = tile * BLOCK + t % BLOCK;
    const int part = t / BLOCK;
    const int cnt = i < n ? vcnt[i] : 0;
    const int half = t % BLOCK / HALF;
    for (int h = t; h < GRAN_SLOTS; h += MAP_NT) gkey[h] = -1;
    for (int h = t; h < GRAN_SLOTS * GRAN / 4; h += MAP_NT) mark[0][h] = mark[1][h] = 0u;
    if (t == 0) {
        full = disable;
        ng = 0;
    }
    __syncthreads();
    uint8_t* markb = reinterpret_cast<uint8_t*>(mark[half]);
    // list words are loaded MAP_BATCH at a time (one memory latency per
    // batch instead of per entry)
    constexpr int MAP_BATCH = 8;
    int32_t last = -1;                     // the granule looked up last
    uint32_t place = 0u;                   // and its place
    for (int k0 = part * MAP_BATCH; k0 < cnt; k0 += MAP_SPLIT * MAP_BATCH) {
        // a full table ends the insertions (the tile is not staged)
        if (*(volatile int*)&full) break;
        int32_t jb[MAP_BATCH];
        vl_load(vl, n, i, k0, jb);
        uint32_t hb[MAP_BATCH];
#pragma unroll
        for (int u = 0; u < MAP_BATCH; ++u) {
            hb[u] = 0u;
            if (k0 + u >= cnt) continue;
            const int32_t j = jb[u];       // (with its mirror bit)
            const int32_t gr = j / GRAN;
            if (gr != last) {
                last = gr;
                uint32_t h = ((uint32_t)gr * 2654435761u) >> 22;   // top 10 bits
                static_assert(GRAN_SLOTS == 1 << 10, "hash bits");
                int probe = 0;
                for (; probe < GRAN_SLOTS; ++probe) {
                    int32_t old = *(volatile int32_t*)&gkey[h];
                    if (old == -1) old = atomicCAS(&gkey[h], -1, gr);
                    if (old == gr) break;
                    if (old == -1) {
                        const int q = atomicAdd(&ng, 1);
                        list[q] = (int32_t)h;
                        lkey[q] = gr;
                        break;
                    }
                    h = (h + 1) & (GRAN_SLOTS - 1);
                }
                if (probe == GRAN_SLOTS) full = 1;
                place = h;
            }
            // the entry's place until its source's slot is known
            hb[u] = place * GRAN + (uint32_t)(j % GRAN);
            markb[hb[u]] = 1;
        }
#pragma unroll
        for (int u = 0; u < MAP_BATCH; u += 4) vs_store4(vs, n, i, k0 + u, hb + u);
    }
    __syncthreads();
    const int G = ng;
    if (full) {
        if (t < 2) tile_cnt[2 * tile + t] = t ? TILE_WHOLE : -1;
        return;
    }
    // thread t takes the granules t, t + MAP_NT, ... of the list: their marks
    // as bits, and their rank among the granules
    uint32_t bits[2][PER];
    int32_t key[PER], rank[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int q = t + r * MAP_NT;
        bits[0][r] = bits[1][r] = 0u;
        key[r] = rank[r] = 0;
        if (q < G) {
            const int h = list[q];
            key[r] = lkey[q];
            // bytes of 0 or 1 -> four bits (byte k's bit moves to 28 + k)
            auto nib = [](uint32_t x) { return (x * 0x10204080u) >> 28; };
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const uint4 m = *reinterpret_cast<const uint4*>(&mark[w][h * GRAN / 4]);
                bits[w][r] = nib(m.x) | nib(m.y) << 4 | nib(m.z) << 8 | nib(m.w) << 12;
            }
        }
    }
    if (t < G)
#pragma unroll 8
        for (int o = 0; o < G; ++o) {
            const int32_t k = lkey[o];
#pragma unroll
            for (int r = 0; r < PER; ++r) rank[r] += k < key[r] ? 1 : 0;
        }
    uint32_t* tab = mark[0];               // (the marks have been read)
    // the whole tile (unit -1), or else its halves
    for (int unit = -1; unit < 2; ++unit) {
    uint32_t b[PER];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        b[r] = unit < 0 ? bits[0][r] | bits[1][r] : bits[unit][r];
        if (t + r * MAP_NT < G) rcnt[rank[r]] = (uint32_t)__popc(b[r]);
    }
    __syncthreads();
    // exclusive prefix sum over the ranks, thread t the ranks [t PER, ...)
    uint32_t c[PER], mine = 0u, total = 0u;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        c[r] = t * PER + r < G ? rcnt[t * PER + r] : 0u;
        mine += c[r];
    }
    uint32_t at = block_excl_scan<MAP_NT>(mine, wsum, total);
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        if (t * PER + r < G) rcnt[t * PER + r] = at;
        at += c[r];
    }
    const int S = (int)total;
    if (t == 0) reals = S;
    if (S > STAGE_CAP) {
        // (neither half staged: one unit, which gathers from memory)
        if (t == 0 && unit >= 0)
            tile_cnt[2 * tile + unit] = unit && tile_cnt[2 * tile] < 0 ? TILE_WHOLE : -1;
        continue;                          // (the same in every thread)
    }
    __syncthreads();
    // the sources, and each place's first slot with its marks
    int32_t* src = tile_src + (2 * tile + (unit < 0 ? 0 : unit)) * STAGE_CAP;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int q = t + r * MAP_NT;
        if (q >= G) continue;
        const uint32_t first = rcnt[rank[r]];
        tab[list[q]] = b[r] | (first << 16);
        if (key[r] >= MBIT / GRAN) atomicMin(&reals, (int)first);
        int32_t* out = src + first;
        for (uint32_t m = b[r]; m; m &= m - 1) *out++ = key[r] * GRAN + __builtin_ctz(m);
    }
    __syncthreads();
    if (t == 0) {
        tile_cnt[2 * tile + (unit < 0 ? 0 : unit)] = S | (reals << 16);
        if (unit < 0) tile_cnt[2 * tile + 1] = TILE_WHOLE;
    }
    // places -> slots (the thread rereads its own words); the words past the
    // list in its last chunk stand for no source
    if (unit < 0 || unit == half)
    for (int k0 = part * MAP_BATCH; k0 < cnt; k0 += MAP_SPLIT * MAP_BATCH) {
        uint32_t hb[MAP_BATCH];
#pragma unroll
        for (int u = 0; u < MAP_BATCH; u += 4) vs_load4(vs, n, i, k0 + u, hb + u);
#pragma unroll
        for (int u = 0; u < MAP_BATCH; ++u) {
            const uint32_t w = tab[hb[u] / GRAN];
            const uint32_t q = (w >> 16) + (uint32_t)__popc(w & ((1u << (hb[u] % GRAN)) - 1u));
            hb[u] = 8u * (k0 + u < cnt ? q : (uint32_t)STAGE_CAP);
        }
#pragma unroll
        for (int u = 0; u < MAP_BATCH; u += 4) vs_store4(vs, n, i, k0 + u, hb + u);
    }
    if (unit < 0) break;
    }
}

// 32-byte position records (x, y, z, 0) of the state the stencils are
// built on; every neighbour gather of the selection and the fits reads
// them (one cache line per neighbour instead of three).
__global__ __launch_bounds__(BLOCK) void k_pack_pos(int64_t n, const double* x,
                                                    const double* y, const double* z,
                                                    double* p4)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2* r = reinterpret_cast<double2*>(p4 + 4 * i);
    // (+ 0.0: no -0 in a record)
    r[0] = make_double2(x[i] + 0.0, y[i] + 0.0);
    r[1] = make_double2(z[i] + 0.0, 0.0);
}

}  // namespace

lp_status list_build(lp_ctx* c, const int32_t* gate)
{
    Work& w = c->w;
    const int64_t n = c->n;
    if (!gate) c->list_ok = false;
    if (n > 0 && (c->cfg.debug_flags & LP_DEBUG_PARTICLE_LIST)) {
        // the per-particle scan (same lists; kept to check the cell scan)
        if (c->periodic)
            hipLaunchKernelGGL(k_list_build<true>, dim3(blocks_for(n)), dim3(BLOCK), 0,
                               c->stream, n, c->n_sys, w.off, w.grid, w.sst[0], w.sst[1],
                               w.sst[2], w.p4, w.cs, w.ce, w.vl, w.vcnt, w.err, gate);
        else
            hipLaunchKernelGGL(k_list_build<false>, dim3(blocks_for(n)), dim3(BLOCK), 0,
                               c->stream, n, c->n_sys, w.off, w.grid, w.sst[0], w.sst[1],
                               w.sst[2], w.p4, w.cs, w.ce, w.vl, w.vcnt, w.err, gate);
    } else if (n > 0) {
        // a wavefront per cell: the eager build knows the cell count; a
        // gated build reads it on the device and strides over the tables
        // with a grid sized by the particle count
        const int64_t tc = gate ? w.cells_max : c->total_cells;
        const int64_t* tdev = gate ? &w.summary->total_cells : nullptr;
        // Wavefronts per cell, until the cells alone fill the chip.  Measured
        // with 1, 2, 4 and 8, us: 4,096 particles 52, 32, 22, 17; 12,075 53,
        // 33, 23, 22; 32,768 54, 41, 39, 43; 65,536 63, 58, 59, 66; 131,072
        // 95, 87, 97, 112; 262,144 150, 149, 167, 279.
        const int split_bits = n <= 16384 ? 3 : n <= 65536 ? 2 : n <= 262144 ? 1 : 0;
        const int64_t groups = ((tc << split_bits) + LC_WAVES - 1) / LC_WAVES;
        const int64_t cap =
            gate ? (2 * (int64_t)blocks_for(n)) << split_bits : (int64_t)LC_MAX_BLOCKS;
        const unsigned nb = (unsigned)std::max<int64_t>(1, std::min(groups, cap));
        if (c->periodic)
            hipLaunchKernelGGL(k_list_cells<true>, dim3(nb), dim3(BLOCK), 0, c->stream, n,
                               c->n_sys, w.grid, w.p4, w.cs, w.ce, tc, tdev, split_bits, w.vl,
                               w.vcnt, w.err, gate);
        else
            hipLaunchKernelGGL(k_list_cells<false>, dim3(nb), dim3(BLOCK), 0, c->stream, n,
                               c->n_sys, w.grid, w.p4, w.cs, w.ce, tc, tdev, split_bits, w.vl,
                               w.vcnt, w.err, gate);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(c, e, "list build launch");
    c->list_ok = true;
    ++c->list_gen;
    // an eager build leaves the tile map stale (captured steps rebuild the
    // map under the same gate right after the list)
    if (!gate) c->map_ok = false;
    return LP_OK;
}

lp_status tile_map_build(lp_ctx* c, const int32_t* gate)
{
    Work& w = c->w;
    const int64_t n = c->n;
    if (!c->list_ok) {
        c->err = "the neighbour list has not been built";
        return LP_E_STATE;
    }
    if (n > 0)
        hipLaunchKernelGGL(k_tile_map, dim3(blocks_for(n)), dim3(MAP_NT), 0, c->stream,
                           n, w.vl, w.vcnt, w.tile_src, w.tile_cnt, w.vs,
                           (c->cfg.debug_flags & LP_DEBUG_GLOBAL_GATHER) ? 1 : 0, gate);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(c, e, "tile map launch");
    c->map_ok = true;
    return LP_OK;
}

lp_status stencils_build(lp_ctx* c, const double* const st[7], bool packed, int part)
{
    Work& w = c->w;
    const int64_t n = c->n;
    c->stencils_ok = false;
    if (!c->list_ok) {
        c->err = "the neighbour list has not been built";
        return LP_E_STATE;
    }
    View v = make_view(c, st);
    hipStream_t s = c->stream;
    if (n > 0 && part != STENCIL_TAIL) {
        // (the state copy or the re-sort of a step has packed them already)
        if (!packed)
            hipLaunchKernelGGL(k_pack_pos, dim3(blocks_for(n)), dim3(BLOCK), 0, s, n, st[0],
                               st[1], st[2], w.p4);
        // mirrors of the current state (ids n + k in ascending source order)
        const int64_t nb = (n + SORT_TILE - 1) / SORT_TILE;
        if (n <= MIRROR_ONE_MAX && !(c->cfg.debug_flags & LP_DEBUG_MIRROR_SCAN)) {
            hipLaunchKernelGGL(k_mirror_one, dim3((unsigned)nb), dim3(MIRROR_NT), 0, s, n,
                               c->n_sys, w.off, w.grid, st[2], w.hard_n, w.redo_n, w.summary,
                               w.mirror_of, w.msrc);
        } else {
            hipLaunchKernelGGL(k_mirror_count, dim3((unsigned)nb), dim3(BLOCK), 0, s, n,
                               c->n_sys, w.off, w.grid, st[2], w.bsum, w.hard_n, w.redo_n,
                               w.summary);
            // up to MIRROR_SUM_BLOCKS blocks each add the counts before them
            // (at most that many words per block, from L2) instead of a scan
            const int scanned =
                (nb > MIRROR_SUM_BLOCKS || (c->cfg.debug_flags & LP_DEBUG_MIRROR_SCAN)) ? 1 : 0;
            if (scanned)
                hipLaunchKernelGGL(k_scan_total, dim3(1), dim3(1024), 0, s,
                                   (uint32_t*)w.bsum, nb, &w.summary->n_mirror);
            hipLaunchKernelGGL(k_mirror_write, dim3((unsigned)nb), dim3(BLOCK), 0, s, n,
                               c->n_sys, w.off, w.grid, w.bsum, scanned, &w.summary->n_mirror,
                               st[2], w.mirror_of, w.msrc);
        }
        // the select phase times the selection kernel alone
        prof_mark(c, 1, false);
        launch_select(c, v);
        prof_mark(c, 1, true);
    }
    if (n > 0 && part != STENCIL_HEAD) {
        prof_mark(c, 2, false);
        launch_select_rest(c, v);
        prof_mark(c, 2, true);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(c, e, "stencil launch");
    if (part != STENCIL_HEAD) c->stencils_ok = true;
    // k_mirror_count cleared the refit list and the displacement maximum
    if (n > 0 && part != STENCIL_TAIL) c->redo_clear = c->disp_clear = true;
    return LP_OK;
}

lp_status stencils_export(lp_ctx* c, const double* const st[7],
                          int64_t* cand_off, int32_t* cand_idx, int64_t cap,
                          int64_t* needed, int32_t* sten_cnt,
                          int32_t* sten_idx, uint8_t* ghost_mask,
                          int64_t* n_mirror)
{
    Work& w = c->w;
    const int64_t n = c->n;
    View v = make_view(c, st);
    hipStream_t s = c->stream;
    if (n_mirror) {
        hipError_t e = hipMemcpyAsync(w.h_summary, w.summary, sizeof(Summary),
                                      hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_fail(c, e, "mirror count");
        *n_mirror = w.h_summary->n_mirror;
        c->n_mirror = *n_mirror;
    }
    if (cand_off || cand_idx || needed) {
        int64_t* off = cand_off ? cand_off : w.coff;
        const unsigned nb = std::max(1u, blocks_for(n, SORT_TILE));
        hipLaunchKernelGGL(k_candidates<false>, dim3(std::max(1u, blocks_for(n, EXP_P))),
                           dim3(BLOCK), 0, s, v, off, (int32_t*)nullptr);
        hipLaunchKernelGGL(k_sum_i64, dim3(nb), dim3(BLOCK), 0, s, off, n, w.bsum);
        hipLaunchKernelGGL(k_scan_i64, dim3(nb), dim3(BLOCK), 0, s, off, n, w.bsum);
        int64_t total = 0;
        hipError_t e = hipMemcpyAsync(&total, off + n, sizeof(int64_t),
                                      hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_fail(c, e, "candidate count");
        if (needed) *needed = total;
        if (cand_idx) {
            if (total > cap) {
                c->err = "candidate capacity " + std::to_string(cap) +
                         " < needed " + std::to_string(total);
                return LP_E_CAPACITY;
            }
            if (n > 0)
                hipLaunchKernelGGL(k_candidates<true>, dim3(blocks_for(n, EXP_P)),
                                   dim3(BLOCK), 0, s, v, off, cand_idx);
        }
    }
    if ((sten_cnt || sten_idx || ghost_mask) && n > 0)
        hipLaunchKernelGGL(k_export_stencils, dim3(blocks_for(n, EXP_P)), dim3(BLOCK), 0,
                           s, v, sten_cnt, sten_idx, ghost_mask);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(c, e, "export launch");
    return LP_OK;
}

}  // namespace lp
