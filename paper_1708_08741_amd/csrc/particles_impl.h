// particles_impl.h -- device functions of the particle kernels: kinematics,
// obstacle mapping and the classification of the cells around a particle
// (arXiv:1708.08741, Sec. 3.2: a cell is an obstacle cell of a particle iff
// its centre lies inside it; uncovered cells are refilled with f^eq(rho0, u_s)
// by the sweep).  One workgroup per particle works on the particle's bounding
// box of cells.
//
// A level's map is kept twice: the owner of every obstacle cell (4 bytes per
// cell, kNone elsewhere), for the refill, the read-outs and the surface
// values, and the obstacle cells as one bit per cell, from which the
// classification forms its masks a row at a time.  Three levels are held
// (the previous, the current, and the next, which is mapped while the
// current one is streamed); a level's map is emptied once the level after it
// has been streamed.  The inside test uses the same FP64 operation sequence
// as a plain CPU evaluation (no contraction), so maps are bit-identical to
// it; shared cells go to the lowest particle index via an atomic minimum.
#pragma once
#include "lbmep_internal.h"

namespace lbmep {
namespace part {

__device__ __forceinline__ double min_image(double d, int len, int periodic) {
    if (periodic) {
        const double h = 0.5 * (double)len;
        if (d > h)
            d -= (double)len;
        else if (d < -h)
            d += (double)len;
    }
    return d;
}

// cell range [lo, lo+cnt) of a box on one axis, before wrapping
struct Box {
    int lo[3], cnt[3];
};

__device__ __forceinline__ void axis_range(double xmin, double xmax, int len, int periodic,
                                           int &lo, int &cnt) {
    // computed in FP64 so that huge radii cannot overflow the integer range
    double l = floor(xmin) - 1.0;
    double h = floor(xmax) + 1.0;
    if (periodic) {
        if (h - l + 1.0 >= (double)len) {
            l = 0.0;
            h = (double)len - 1.0;
        }
    } else {
        if (l < 0.0) l = 0.0;
        if (h > (double)len - 1.0) h = (double)len - 1.0;
    }
    lo = (int)l;
    cnt = h >= l ? (int)(h - l + 1.0) : 0;
}

__device__ __forceinline__ int box_size(const Box &b) {
    return (b.cnt[0] > 0 && b.cnt[1] > 0 && b.cnt[2] > 0) ? b.cnt[0] * b.cnt[1] * b.cnt[2] : 0;
}

// box around the ball of radius R at X (generous: every cell whose centre
// can be inside is in it)
__device__ __forceinline__ Box ball_box(const Grid &g, const double *X, double R) {
    Box b;
    const int len[3] = {g.nx, g.ny, g.nz};
    for (int k = 0; k < 3; ++k) axis_range(X[k] - R, X[k] + R, len[k], g.per[k], b.lo[k], b.cnt[k]);
    return b;
}

// floor(i / d) for i >= 0, d >= 1, with rd ~ 1 / d: the product in single
// precision is within a few units of the quotient, the integer corrections
// make it exact (an integer division is a long instruction sequence)
__device__ __forceinline__ int div_exact(int i, int d, float rd) {
    int q = (int)((float)i * rd);
    int r = i - q * d;
    while (r < 0) {
        --q;
        r += d;
    }
    while (r >= d) {
        ++q;
        r -= d;
    }
    return q;
}

// v wrapped into [0, len): box coordinates lie within one period of the
// grid, so one addition or subtraction does it (the remainder otherwise)
__device__ __forceinline__ int wrap_axis(int v, int len) {
    if (v < 0) v += len;
    else if (v >= len) v -= len;
    if (v < 0 || v >= len) v = ((v % len) + len) % len;
    return v;
}

// box-relative coordinates (ix, iy, iz) of the i-th cell of a box of
// cx x cy x ... cells (rcx, rcy: reciprocals of cx, cy)
__device__ __forceinline__ void box_split(int i, int cx, int cy, float rcx, float rcy, int &ix,
                                          int &iy, int &iz) {
    const int q = div_exact(i, cx, rcx);
    ix = i - q * cx;
    iz = div_exact(q, cy, rcy);
    iy = q - iz * cy;
}

// the i-th cell of a box (wrapped on periodic axes)
__device__ __forceinline__ void box_cell(const Grid &g, const Box &b, int i, int &x, int &y,
                                         int &z) {
    const int cx = b.cnt[0], cy = b.cnt[1];
    int ix, iy, iz;
    box_split(i, cx, cy, 1.0f / (float)cx, 1.0f / (float)cy, ix, iy, iz);
    x = b.lo[0] + ix;
    y = b.lo[1] + iy;
    z = b.lo[2] + iz;
    if (g.per[0]) x = wrap_axis(x, g.nx);
    if (g.per[1]) y = wrap_axis(y, g.ny);
    if (g.per[2]) z = wrap_axis(z, g.nz);
}

__device__ __forceinline__ size_t cell_of(const Grid &g, int x, int y, int z) {
    return (size_t)x + (size_t)g.nx * ((size_t)y + (size_t)g.ny * (size_t)z);
}

// inside test of Sec. 3.2 (closed ball, minimum image), FP64 without
// contraction, as a plain CPU evaluation orders it
__device__ __forceinline__ bool inside_ball(const Grid &g, int x, int y, int z, const double *Xp,
                                            double R) {
    const double r0 = min_image(((double)x + 0.5) - Xp[0], g.nx, g.per[0]);
    const double r1 = min_image(((double)y + 0.5) - Xp[1], g.ny, g.per[1]);
    const double r2 = min_image(((double)z + 0.5) - Xp[2], g.nz, g.per[2]);
    const double d2 = (r0 * r0 + r1 * r1) + r2 * r2;
    return d2 <= R * R;
}

// X_p(level) of the prescribed kinematics, component k, wrapped into [0, L)
// on periodic axes
__device__ __forceinline__ double position(const ParticleArgs &pa, int p, int k, int64_t level) {
    const int len[3] = {pa.g.nx, pa.g.ny, pa.g.nz};
    double x = pa.X0[3 * p + k];
    // prescribed kinematics X(n) = X(0) + n U, evaluated in this form; with
    // dynamics X0 already holds the level's position
    if (pa.moving && !pa.dynamic) x = pa.X0[3 * p + k] + (double)level * pa.U[3 * p + k];
    if (pa.g.per[k]) {
        x = x - (double)len[k] * floor(x / (double)len[k]);
        if (x >= (double)len[k]) x -= (double)len[k];
    }
    return x;
}

// The cells of the ball of radius R at Xp, row by row: fn(c0, x, n) for runs
// of n cells from column x of the row that starts at cell c0 (a row that
// crosses a periodic edge is given in two runs).  A thread (tid of nt) takes a
// row: along it the squared distance grows away from the centre, in floating point too
// (every operation of the test is monotonic, and neighbouring cells differ by
// far more than a rounding), so the cells inside are one run, whose ends are
// found by the test itself from an estimate.  A box as wide as its periodic x
// axis, where the nearest image changes along the row, is tested cell by cell.
// (The test of every cell of the box, 11^3 for R = 4, took 36 us at 512^3
// with 4096 particles in a launch of its own.)
template <typename F>
__device__ __forceinline__ void ball_rows(const Grid &g, const double *Xp, double R, int tid, int nt,
                                          F &&fn) {
    const Box b = ball_box(g, Xp, R);
    if (box_size(b) == 0) return;
    const bool whole = g.per[0] && b.cnt[0] >= g.nx;
    const int rows = b.cnt[1] * b.cnt[2];
    for (int r = tid; r < rows; r += nt) {
        int z = r / b.cnt[1], y = r - z * b.cnt[1];
        y += b.lo[1];
        z += b.lo[2];
        if (g.per[1]) y = wrap_axis(y, g.ny);
        if (g.per[2]) z = wrap_axis(z, g.nz);
        const size_t c0 = cell_of(g, 0, y, z);
        auto inside = [&](int x) {  // x: column before wrapping
            if (g.per[0]) x = wrap_axis(x, g.nx);
            return inside_ball(g, x, y, z, Xp, R);
        };
        if (whole) {
            for (int x = 0; x < g.nx; ++x)
                if (inside(x)) fn(c0, x, 1);
            continue;
        }
        const int first = b.lo[0], last = b.lo[0] + b.cnt[0] - 1;
        const double r1 = min_image(((double)y + 0.5) - Xp[1], g.ny, g.per[1]);
        const double r2 = min_image(((double)z + 0.5) - Xp[2], g.nz, g.per[2]);
        const double h2 = R * R - (r1 * r1 + r2 * r2);
        // (the sums of the test are monotonic in floating point too: where the
        // other two axes alone exceed the radius, no x is inside)
        if (h2 < -1.0) continue;
        const double h = h2 > 0.0 ? sqrt(h2) : 0.0;
        int l = max(first, min(last + 1, (int)ceil(Xp[0] - h - 0.5)));
        int e = min(last, max(l - 1, (int)floor(Xp[0] + h - 0.5)));
        while (l > first && inside(l - 1)) --l;
        while (l <= e && !inside(l)) ++l;
        if (l > e) e = l - 1;
        while (e < last && inside(e + 1)) ++e;
        while (e >= l && !inside(e)) --e;
        for (int x = l; x <= e;) {
            int xw = x, n = e - x + 1;
            if (g.per[0]) {
                xw = wrap_axis(x, g.nx);
                n = min(n, g.nx - xw);
            }
            fn(c0, xw, n);
            x += n;
        }
    }
}

// fn(w, m) for the words w and bit masks m of n bits from cell c on
template <typename F>
__device__ __forceinline__ void run_words(size_t c, int n, F &&fn) {
    while (n > 0) {
        const int s = (int)(c & 31u), k = min(n, 32 - s);
        fn(c >> 5, (k < 32 ? (1u << k) - 1u : ~0u) << s);
        c += (size_t)k;
        n -= k;
    }
}

// the cells particle p covers at m.X leave the map: every cell of a level's
// map lies in the ball of some particle, so this empties it (BITS: the map has
// bitmaps)
template <bool BITS = true>
__device__ __forceinline__ void map_clear(const ParticleArgs &pa, int p, const LevelMap &m) {
    ball_rows(pa.g, m.X + 3 * (size_t)p, pa.R[p], (int)threadIdx.x, (int)blockDim.x,
              [&](size_t c0, int x, int n) {
        const size_t c = c0 + (size_t)x;
        for (int k = 0; k < n; ++k) m.owner[c + (size_t)k] = kNone;
        // the other cells of the words leave the map as well
        if constexpr (BITS) run_words(c, n, [&](size_t w, uint32_t) { m.bits[w] = 0u; });
    });
}

// the cells particle p covers at Xp enter the (emptied) map
template <bool BITS>
__device__ __forceinline__ void map_set(const ParticleArgs &pa, int p, const double *Xp,
                                        const LevelMap &m, int tid, int nt) {
    ball_rows(pa.g, Xp, pa.R[p], tid, nt, [&](size_t c0, int x, int n) {
        if constexpr (!BITS) {
            for (size_t c = c0 + (size_t)x; c < c0 + (size_t)(x + n); ++c)
                if (!(pa.flag[c] & kWall)) atomicMin(&m.owner[c], (uint32_t)p);
            return;
        }
        run_words(c0 + (size_t)x, n, [&](size_t w, uint32_t mask) {
            if (pa.wallbits) mask &= ~pa.wallbits[w];
            if (!mask) return;
            atomicOr(&m.bits[w], mask);
            for (uint32_t k = mask; k; k &= k - 1u)
                atomicMin(&m.owner[32 * w + (size_t)(__ffs((int)k) - 1)], (uint32_t)p);
        });
    });
}

// particle p at `level`: its position into the level's map and its cells, by
// nt threads (tid: this one's number among them)
template <bool BITS = true>
__device__ __forceinline__ void advance_set(const ParticleArgs &pa, int p, int64_t level,
                                            const LevelMap &m, int tid, int nt) {
    const double Xp[3] = {position(pa, p, 0, level), position(pa, p, 1, level),
                          position(pa, p, 2, level)};
    if (tid < 3) m.X[3 * (size_t)p + (size_t)tid] = tid == 0 ? Xp[0] : tid == 1 ? Xp[1] : Xp[2];
    map_set<BITS>(pa, p, Xp, m, tid, nt);
}

// one cell's classification from the wall bits and the map (global reads):
// its flag; *wmask = directions whose neighbour is a wall cell; *pmask =
// directions whose neighbour is an obstacle cell of particle p (p != kNone);
// with owner_old, a fluid cell that was an obstacle cell is marked uncovered.
// WALLS: the wall directions of obstacle cells as well (a sphere may uncover
// them while the walls are as they are)
template <bool WALLS>
__device__ __forceinline__ uint8_t classify_cell(const Grid &g, int x, int y, int z,
                                                 const uint8_t *flag, const uint32_t *owner,
                                                 const uint32_t *owner_old, uint32_t p,
                                                 uint32_t *wmask, uint32_t *pmask) {
    const size_t c = cell_of(g, x, y, z);
    const uint8_t wall = flag[c] & kWall;
    const bool obst = !wall && owner && owner[c] != kNone;
    uint8_t f = wall;
    uint32_t mask = 0, wm = 0, pm = 0;
    if (!wall && (WALLS || !obst)) {
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            int sx = x + kCx[q], sy = y + kCy[q], sz = z + kCz[q];
            bool solid = false;
            if (sx < 0 || sx >= g.nx) {
                if (g.per[0]) sx = sx < 0 ? sx + g.nx : sx - g.nx; else solid = true;
            }
            if (sy < 0 || sy >= g.ny) {
                if (g.per[1]) sy = sy < 0 ? sy + g.ny : sy - g.ny; else solid = true;
            }
            if (sz < 0 || sz >= g.nz) {
                if (g.per[2]) sz = sz < 0 ? sz + g.nz : sz - g.nz; else solid = true;
            }
            if (!solid) {
                const size_t s = cell_of(g, sx, sy, sz);
                const bool w = flag[s] & kWall;
                const uint32_t o = owner ? owner[s] : kNone;
                solid = w || o != kNone;
                if (w) wm |= 1u << (q - 1);
                if (!w && o != kNone && o == p) pm |= 1u << (q - 1);
            }
            if (solid) mask |= 1u << (q - 1);
        }
        f = (mask ? kNear : 0) | ((mask & kFaceDirs) ? kNear7 : 0);
        if (owner_old && owner_old[c] != kNone) f |= kUncov;
    }
    if (obst) {
        f = kObst;
        pm = 0;
    }
    *wmask = wm;
    *pmask = pm;
    return f | wall;
}

// n <= 64 consecutive bits from cell c on
__device__ __forceinline__ uint64_t get_bits(const uint32_t *bits, size_t c, int n) {
    const size_t w = c >> 5;
    const int s = (int)(c & 31u);
    uint64_t v = (uint64_t)bits[w];
    if (s + n > 32) v |= (uint64_t)bits[w + 1] << 32;
    v >>= s;
    if (s + n > 64) v |= (uint64_t)bits[w + 2] << (64 - s);
    return n < 64 ? v & ((1ull << n) - 1ull) : v;
}

// bits of the cells x0 .. x0 + n - 1 (n <= 64) of the row that starts at cell
// c0, wrapped on a periodic axis, 0 beyond a non-periodic edge
__device__ __forceinline__ uint64_t row_bits(const uint32_t *bits, size_t c0, int x0, int n, int nx,
                                             int periodic) {
    if (x0 >= 0 && x0 + n <= nx) return get_bits(bits, c0 + (size_t)x0, n);
    uint64_t r = 0;
    for (int i = 0; i < n;) {
        int x = x0 + i;
        if (x < 0 || x >= nx) {
            if (!periodic) {
                ++i;
                continue;
            }
            x = wrap_axis(x, nx);
        }
        const int m = min(n - i, nx - x);
        r |= get_bits(bits, c0 + (size_t)x, m) << i;
        i += m;
    }
    return r;
}

// exclusive prefix of `mine` over the workgroup; the total in *total.  wsum:
// one word per wavefront, free again after the next barrier
__device__ __forceinline__ uint32_t block_prefix(uint32_t mine, uint32_t *wsum, uint32_t *total) {
    const int lane = (int)__lane_id(), wave = (int)threadIdx.x / 64, nw = (int)blockDim.x / 64;
    uint32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)incl, off);
        if (lane >= off) incl += t;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t pre = incl - mine, tot = 0;
    for (int w = 0; w < nw; ++w) {
        if (w < wave) pre += wsum[w];
        tot += wsum[w];
    }
    *total = tot;
    return pre;
}

// rows of a particle's box with a one-cell halo (one bit per cell, bit i the
// cell i of the halo row) kept in LDS for the classification
struct BoxRows {
    uint64_t *solid, *obst, *mine, *uncov, *near, *near7;
    uint32_t *wsum;
    uint32_t *cell;  // row_cells(threads) list entries in the making: row, column
};
__host__ __device__ constexpr uint32_t row_cells(int threads) { return 4u * (uint32_t)threads; }

// Classification around particle p (union of its boxes at the previous and
// the new position, grown by one cell): flags of the new level and the list
// of p's links, (cell, directions whose neighbour is an obstacle cell of p),
// for the bounce-back / exchange kernel, in box order.
//
// Boxes whose halo rows fit in 64 bits and whose rows fit in LDS (pa.box_rows;
// radii up to about 11) are formed from the bitmaps: a thread holds a row,
// the neighbour tests of a whole row are shifts and ORs of its nine rows, and
// only obstacle cells need their owner.  What it replaced staged the flag and
// the owner of every halo cell (5 bytes against 3 bits) and tested 18 LDS
// bytes per cell; both are bound by their chains of dependent round trips, so
// fewer trips and more threads are what counts.  Larger boxes are classified
// cell by cell from the maps.
__device__ __forceinline__ void classify(const ParticleArgs &pa, int p, const LevelMap &old,
                                         const LevelMap &now, const BoxRows &rows) {
    const Grid &g = pa.g;
    const double R = pa.R[p];
    Box b;
    const int len[3] = {g.nx, g.ny, g.nz};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double a0 = old.X[3 * (size_t)p + k], a1 = now.X[3 * (size_t)p + k];
        double mn = a0 < a1 ? a0 : a1, mx = a0 < a1 ? a1 : a0;
        // a particle that wrapped around a periodic axis: the way that it went
        // (box cells are wrapped; with the whole axis in the box instead, a
        // crossing sphere was the longest chain of a step: 600 spheres of radius 4
        // in 64^3 FP32 at up to 0.02 cells a step, 65 -> 45 us)
        if (g.per[k] && mx - mn > 0.5 * (double)len[k]) {
            const double t = mn + (double)len[k];
            mn = mx;
            mx = t;
        }
        // one more cell on each side for the NEAR ring and for the uncovered
        // marks of the previous level (motion < 1 cell/step)
        axis_range(mn - R - 1.0, mx + R + 1.0, len[k], g.per[k], b.lo[k], b.cnt[k]);
    }
    const int n = box_size(b);
    const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
    uint2 *plist = pa.plist + (size_t)p * pa.pcap;
    const int hx = b.cnt[0] + 2, hy = b.cnt[1] + 2, hz = b.cnt[2] + 2;
    const int hrows = hy * hz;
    uint32_t base = 0;
    if (n > 0 && hx <= 64 && hrows <= (int)pa.box_rows) {
        // the halo rows: solid (wall, obstacle, or beyond a non-periodic
        // edge), obstacle, uncovered (obstacle of the previous level only)
        const uint64_t all = hx < 64 ? (1ull << hx) - 1ull : ~0ull;
        uint64_t inx = all;  // columns inside the grid
        if (!g.per[0]) {
            const int l = b.lo[0] - 1 < 0 ? 1 : 0, r = b.lo[0] + b.cnt[0] >= g.nx ? 1 : 0;
            if (l) inx &= ~1ull;
            if (r) inx &= ~(1ull << (hx - 1));
        }
        for (int h = tid; h < hrows; h += nt) {
            int y = b.lo[1] - 1 + h % hy, z = b.lo[2] - 1 + h / hy;
            bool in = true;
            if (y < 0 || y >= g.ny) {
                if (g.per[1]) y = wrap_axis(y, g.ny); else in = false;
            }
            if (z < 0 || z >= g.nz) {
                if (g.per[2]) z = wrap_axis(z, g.nz); else in = false;
            }
            uint64_t o = 0, w = 0, u = 0;
            if (in) {
                const size_t c0 = cell_of(g, 0, y, z);
                o = row_bits(now.bits, c0, b.lo[0] - 1, hx, g.nx, g.per[0]);
                u = row_bits(old.bits, c0, b.lo[0] - 1, hx, g.nx, g.per[0]);
                if (pa.wallbits) w = row_bits(pa.wallbits, c0, b.lo[0] - 1, hx, g.nx, g.per[0]);
            }
            const uint64_t s = in ? (o | w | ~inx) & all : all;
            rows.obst[h] = o;
            rows.solid[h] = s;
            rows.uncov[h] = u & ~s;
            rows.mine[h] = 0ull;
        }
        __syncthreads();
        // p's own obstacle cells, of those with a neighbour that is not solid
        // (links lead to no others; four owners of a row in flight)
        for (int h = tid; h < hrows; h += nt) {
            uint64_t o = rows.obst[h], mine = 0;
            if (!o) continue;
            const int iy = h % hy, iz = h / hy;
            if (iy > 0 && iy < hy - 1 && iz > 0 && iz < hz - 1) {
                const uint64_t *S = rows.solid + h;
                const uint64_t face = S[-1] & S[1] & S[-hy] & S[hy], all5 = S[0] & face;
                // closed: all 18 neighbours solid; the end columns stay open
                const uint64_t closed = face & S[-1 - hy] & S[1 - hy] & S[-1 + hy] & S[1 + hy] &
                                        (all5 << 1) & (all5 >> 1);
                o &= ~closed;
            }
            int y = b.lo[1] - 1 + iy, z = b.lo[2] - 1 + iz;
            if (g.per[1]) y = wrap_axis(y, g.ny);
            if (g.per[2]) z = wrap_axis(z, g.nz);
            const uint32_t *ow = now.owner + cell_of(g, 0, y, z);
            while (o) {
                constexpr int U = 4;
                uint64_t bit[U];
                uint32_t who[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    bit[u] = o & (0ull - o);
                    who[u] = kNone;
                    if (o) {
                        int x = b.lo[0] - 1 + (__ffsll((unsigned long long)o) - 1);
                        if (g.per[0]) x = wrap_axis(x, g.nx);
                        who[u] = ow[x];
                    }
                    o &= o - 1ull;
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (who[u] == (uint32_t)p) mine |= bit[u];
            }
            rows.mine[h] = mine;
        }
        __syncthreads();
        // rows of the box: NEAR masks, and the list of links
        const uint64_t inbox = ((1ull << b.cnt[0]) - 1ull) << 1;
        const int brows = b.cnt[1] * b.cnt[2];
        for (int r0 = 0; r0 < brows; r0 += nt) {
            const int r = r0 + tid;
            const bool act = r < brows;
            const int iz = act ? r / b.cnt[1] : 0, iy = act ? r - iz * b.cnt[1] : 0;
            const int h = (iy + 1) + hy * (iz + 1);
            auto both = [](uint64_t v) { return (v << 1) | (v >> 1); };
            uint64_t ml = 0;
            if (act) {
                const uint64_t *S = rows.solid + h;
                const uint64_t ym = S[-1], yp = S[1], zm = S[-hy], zp = S[hy];
                const uint64_t n7 = both(S[0]) | ym | yp | zm | zp;
                const uint64_t nn = n7 | both(ym) | both(yp) | both(zm) | both(zp) | S[-1 - hy] |
                                    S[1 - hy] | S[-1 + hy] | S[1 + hy];
                const uint64_t fluid = ~S[0] & inbox;
                rows.near[h] = nn & fluid;
                rows.near7[h] = n7 & fluid;
                const uint64_t *M = rows.mine + h;
                ml = (both(M[0] | M[-1] | M[1] | M[-hy] | M[hy]) | M[-1] | M[1] | M[-hy] | M[hy] |
                      M[-1 - hy] | M[1 - hy] | M[-1 + hy] | M[1 + hy]) & fluid;
            }
            uint32_t total;
            uint32_t pos = base + block_prefix((uint32_t)__popcll(ml), rows.wsum, &total);
            base += total;
            // a row's cells are laid out in LDS, then taken one per thread: a
            // row thread that formed their masks itself held up the others
            // (14 cells of 18 directions)
            const uint32_t start = base - total, cells = row_cells(nt);
            for (uint32_t w0 = 0; w0 < total; w0 += cells) {
                for (; ml && pos - start - w0 < cells; ml &= ml - 1ull, ++pos)
                    rows.cell[pos - start - w0] =
                        (uint32_t)h << 6 | (uint32_t)(__ffsll((unsigned long long)ml) - 1);
                __syncthreads();
                const uint32_t m = min(cells, total - w0);
                for (uint32_t k = (uint32_t)tid; k < m; k += (uint32_t)nt) {
                    const uint32_t w = rows.cell[k];
                    const int ch = (int)(w >> 6), ix = (int)(w & 63u);
                    const int cz = ch / hy;
                    int x = b.lo[0] - 1 + ix, y = b.lo[1] - 1 + (ch - cz * hy), z = b.lo[2] - 1 + cz;
                    if (g.per[0]) x = wrap_axis(x, g.nx);
                    if (g.per[1]) y = wrap_axis(y, g.ny);
                    if (g.per[2]) z = wrap_axis(z, g.nz);
                    const uint64_t *M = rows.mine + ch;
                    uint32_t pm = 0;
#pragma unroll
                    for (int q = 1; q < Q; ++q)
                        pm |= (uint32_t)((M[kCy[q] + hy * kCz[q]] >> (ix + kCx[q])) & 1ull) << (q - 1);
                    if (start + w0 + k < pa.pcap)
                        plist[start + w0 + k] = make_uint2((uint32_t)cell_of(g, x, y, z), pm);
                }
                __syncthreads();
            }
            __syncthreads();  // wsum is reused; near rows are complete after the last pass
        }
        // the flags
        const float rcx = 1.0f / (float)b.cnt[0], rcy = 1.0f / (float)b.cnt[1];
        for (int i = tid; i < n; i += nt) {
            int ix, iy, iz;
            box_split(i, b.cnt[0], b.cnt[1], rcx, rcy, ix, iy, iz);
            int x = b.lo[0] + ix, y = b.lo[1] + iy, z = b.lo[2] + iz;
            if (g.per[0]) x = wrap_axis(x, g.nx);
            if (g.per[1]) y = wrap_axis(y, g.ny);
            if (g.per[2]) z = wrap_axis(z, g.nz);
            const int h = (iy + 1) + hy * (iz + 1), bit = ix + 1;
            uint32_t f;
            if ((rows.solid[h] >> bit) & 1ull)
                f = (rows.obst[h] >> bit) & 1ull ? kObst : kWall;
            else
                f = (((rows.near[h] >> bit) & 1ull) ? kNear : 0u) |
                    (((rows.near7[h] >> bit) & 1ull) ? kNear7 : 0u) |
                    (((rows.uncov[h] >> bit) & 1ull) ? kUncov : 0u);
            pa.flag[cell_of(g, x, y, z)] = (uint8_t)f;
        }
        __syncthreads();  // the rows may be used for another particle
    } else {
        for (int i0 = 0; i0 < n; i0 += nt) {
            const int i = i0 + tid;
            uint32_t pm = 0;
            size_t c = 0;
            if (i < n) {
                int x, y, z;
                box_cell(g, b, i, x, y, z);
                c = cell_of(g, x, y, z);
                uint32_t wm;
                uint8_t f = classify_cell<false>(g, x, y, z, pa.flag, now.owner, old.owner, (uint32_t)p, &wm, &pm);
                pa.flag[c] = f;
            }
            uint32_t total;
            const uint32_t pos = base + block_prefix(pm ? 1u : 0u, rows.wsum, &total);
            base += total;
            if (pm && pos < pa.pcap) plist[pos] = make_uint2((uint32_t)c, pm);
            __syncthreads();
        }
    }
    if (tid == 0) pa.pcount[p] = base < pa.pcap ? base : pa.pcap;
}

// LDS of classify for up to box_rows halo rows and workgroups of 8 wavefronts
constexpr int kRowArrays = 6;
__device__ __forceinline__ BoxRows box_rows(unsigned char *lds, uint32_t nrows) {
    uint64_t *w = reinterpret_cast<uint64_t *>(lds);
    BoxRows r;
    r.solid = w;
    r.obst = w + nrows;
    r.mine = w + 2 * (size_t)nrows;
    r.uncov = w + 3 * (size_t)nrows;
    r.near = w + 4 * (size_t)nrows;
    r.near7 = w + 5 * (size_t)nrows;
    r.wsum = reinterpret_cast<uint32_t *>(w + kRowArrays * (size_t)nrows);
    r.cell = r.wsum + 16;
    return r;
}

}  // namespace part
}  // namespace lbmep
