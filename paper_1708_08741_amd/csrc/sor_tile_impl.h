// sor_tile_impl.h -- K red-black SOR iterations of the Debye-Hueckel equation
// in one pass over psi (arXiv:1708.08741, Sec. "Solver for Linear Elliptic
// PDEs with Moving Boundaries"), for even nx with a row of one colour in at
// most four wavefronts (tile_pays: where it is the faster form).  Included by
// k_potential.hip.
//
// Buffer A holds iterate n and is only read, buffer B receives iterate n + K.
// A workgroup of 16 wavefronts holds `ns` consecutive rows (y) of one plane,
// one row in nwx = 16 / ns wavefronts, V consecutive entries of the
// colour-split psi per lane, and marches along z.  The 2K half-sweeps of the
// pass are stages of a pipeline: at step z stage j relaxes colour j & 1 of
// plane z + 2K - 1 - j from the output of stage j - 1 (stage 0: from A).  A
// lane keeps the last three planes of every stage's input for its own
// entries in registers; rows y -+ 1 come through LDS, where every stage
// leaves its new plane for the next step (double-buffered by step parity: one
// barrier per step).  Each stage is valid on one row less at either end, so
// ns - 2 (2K - 1) rows are written.  A half-sweep is order-free, so every
// value is formed from the operands of the in-place red-black sweep in the
// same order: the result is bitwise that sweep's.
//
// While a solve runs, psi is 0 in solid cells (their own values are kept
// aside, k_tile_solid / k_tile_prepare), and a boundary cell's row is held as
// its constant right-hand side (the Dirichlet faces' 2 b) and its diagonal.
// Every neighbour then enters the sum as its stored value -- a wall or
// obstacle cell as an exact 0, as does a neighbour beyond a non-periodic
// edge -- and one formula serves every cell; a solid cell's result is set to
// 0 whatever its neighbours hold (0 times an infinity or a NaN would not be 0,
// and would reach the other side of the wall).
//
// What bounds it: the vector unit (about 285 vector instructions per
// wavefront and step of 64 V entries in each of four stages, half of the
// time) and the step's chain of one barrier, four dependent stages and the
// loads of the next step, with one workgroup per CU; 2.0 GB move per pair of
// iterations at 512^3 FP32 (halo rows are re-read past L2) at 4.9 TB/s.  Why
// whole rows and 16 bytes of entries per lane: the x-neighbours of three of
// four entries are the lane's own, so a row costs one DPP rotate, one 16-byte
// load and store and two 16-byte LDS reads per 256 entries; the earlier
// one-entry-per-lane march (k_sor_march) needed about 68 vector instructions
// per cell and iteration and one pass over psi for each.  The (row block,
// plane) space is cut into one equal range per resident workgroup, so the
// last wave of workgroups is not nearly empty and small grids still use every
// CU.  Measured, a solve of 29 iterations with its set-up and boundaries:
// 512^3 FP32 with 4096 spheres 8.72 -> 6.47 ms, 64^3 FP32 1.57 -> 0.30 ms,
// 144^3 FP64 2.63 -> 0.75 ms, 256 x 200 x 300 FP64 3.34 -> 2.20 ms.  Two rows per wavefront (8 wavefronts,
// half the scalar work per row) took 7.45 ms, reading the next stage's LDS
// rows a stage early (spills) 6.73 ms.
#pragma once
#include <array>
#include <climits>
#include <type_traits>

#include "device_table.h"
#include "lbmep_internal.h"

namespace lbmep {
namespace {

template <typename CT, int V>
struct alignas(sizeof(CT) * V) Pack {
    using Ext = CT __attribute__((ext_vector_type(V)));  // one memory access
    CT v[V];
};

// the value is formed here: not moved behind a branch or a later wait
__device__ __forceinline__ void keep(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep(double &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep(uint32_t &v) { asm volatile("" : "+v"(v)); }
template <typename CT, int V>
__device__ __forceinline__ void keep(Pack<CT, V> &p) {
#pragma unroll
    for (int v = 0; v < V; ++v) keep(p.v[v]);
}

constexpr int kTileSlots = 16;          // rows of a workgroup, times the wavefronts of a row
constexpr int kTileWaves = 16;          // wavefronts of a workgroup, a row (or part of one) each
constexpr uint32_t kTileDiag0 = 6u;     // code of 6 + kappa^2; + Dirichlet - Neumann faces
constexpr uint32_t kTileSolid = 13u;    // code of a wall or obstacle cell

// entries per colour of the row arrays (rhs and diagonals of the boundary
// rows): N / 2 rounded up, so that a lane's V entries are aligned
__host__ __device__ inline size_t tile_stride(size_t N) { return (N / 2 + 15) / 16 * 16; }

// a / d for the launch-constant diagonal d, r = 1 / d: the product corrected
// by its exact remainder is the correctly rounded quotient when r is
// correctly rounded (Markstein, IBM J. Res. Dev. 34, 1990); tiny, huge and
// non-finite numerators, where the remainder may not be exact, are divided
__device__ __forceinline__ double quot_const(double a, double d, double r) {
    const double m = fabs(a);
    if (!(m > 0x1p-900 && m < 0x1p900)) return a / d;
    const double q = a * r;
    return __builtin_fma(__builtin_fma(-q, d, a), r, q);
}
__device__ __forceinline__ float quot_const(float a, float, float r) { return a * r; }

// a * b, and 0 where a factor is 0, whatever the other is (an infinity or a
// NaN too); else the ordinary product, subnormal ones as well (checked against
// it on 4 million pairs).  A comparison and a selection per entry instead made
// the pass 3.7 % slower among 4096 spheres.
__device__ __forceinline__ float mul_zero(float a, float b) {
    float r;
    asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// the constants of a boundary row for one lane: right-hand sides and, FP32,
// a code byte per entry (into the table of reciprocal diagonals), FP64, the
// diagonals
template <typename CT, int V>
struct RowCoef;
template <int V>
struct RowCoef<float, V> {
    Pack<float, V> rhs;
    uint32_t code;
};
template <int V>
struct RowCoef<double, V> {
    Pack<double, V> rhs, diag;
};

template <typename CT, int V, int K>
__global__ void __launch_bounds__(64 * kTileWaves)
    k_sor_tile(SorArgs a, const CT *A, CT *B, int nwx, int ns, uint32_t nyb, uint32_t planes,
               uint32_t cols) {
    constexpr int S = 2 * K;  // stages
    // (only a solve with a residual is ever done early)
    if (a.rf > 0.0 && a.ctl->done) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl->iters += K;
    extern __shared__ __align__(16) unsigned char tile_lds[];
    __shared__ float rd[16];  // FP32: reciprocal diagonals by code
    if (threadIdx.x < 16) rd[threadIdx.x] = threadIdx.x < 13 ? a.rdiag[threadIdx.x] : 0.0f;
    using P = Pack<CT, V>;
    const Grid &g = a.g;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int hx = nx >> 1;
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int slot = wave / nwx, seg = wave % nwx;  // row slot, part of the row
    const int rs = 64 * V * nwx;  // entries of an LDS row
    const int e0 = seg * 64 * V + lane * V;
    const bool act = e0 < hx;
    const int ec = act ? e0 : 0;
    // last lane of this wavefront that holds entries, and the entries beyond
    // the two ends of its part of the row (their places in the LDS row)
    const int lw = min(63, (hx - seg * 64 * V) / V - 1);
    const int eleft = seg == 0 ? hx - 1 : seg * 64 * V - 1;
    const int eright = (seg + 1) * 64 * V >= hx ? 0 : (seg + 1) * 64 * V;
    // uniform flags of the wavefront, tested bit by bit: the compiler would
    // keep each condition in a register pair of its own
    constexpr uint32_t kXl = 1, kXr = 2, kRot = 4, kYlo = 8, kYhi = 16, kMine = 32, kOuter = 64;
    uint32_t flags0 = 0;
    if (!g.per[0] && seg == 0) flags0 |= kXl;
    if (!g.per[0] && (seg + 1) * 64 * V >= hx) flags0 |= kXr;
    // one wavefront holds a whole periodic row in all its lanes: the rotate wraps
    if (g.per[0] && nwx == 1 && hx == 64 * V) flags0 |= kRot;
    // a stage's rows in LDS: the slots, and one row before and after them
    // (written for stage 0 only: the rows that the end slots need from A)
    const uint32_t rb = (uint32_t)(rs * (int)sizeof(CT));
    const uint32_t lo = (uint32_t)(slot + 1) * rb + (uint32_t)((seg * 64 * V + lane * V) * (int)sizeof(CT));
    const uint32_t bufb = (uint32_t)(ns + 2) * rb;
    auto lds = [&](int par, int j) -> unsigned char * { return tile_lds + (uint32_t)(par * S + j) * bufb; };
    const uint32_t el_o = (uint32_t)(slot + 1) * rb + (uint32_t)(eleft * (int)sizeof(CT));
    const uint32_t er_o = (uint32_t)(slot + 1) * rb + (uint32_t)(eright * (int)sizeof(CT));
    // end wavefronts bring the row beyond theirs from A for stage 0
    if (slot == 0 || slot == ns - 1) flags0 |= kOuter;
    const uint32_t lx = slot == 0 ? lo - rb : lo + rb;

    const size_t hxy = (size_t)hx * (size_t)ny, half = g.Ns >> 1, ts = tile_stride(g.N);
    // colour 1 (black) starts half32 entries after colour 0 (red)
    const uint32_t half32 = (uint32_t)half;
    const uint2 *mb = reinterpret_cast<const uint2 *>(a.ibits + 4 * sor_ibits_words_per_colour(g.N));
    const CT *rhs = static_cast<const CT *>(a.nrow);
    const uint8_t *code = reinterpret_cast<const uint8_t *>(a.codes);  // FP32
    const CT *dgs = rhs + 2 * ts;                                      // FP64
    const uint32_t io = (uint32_t)ec * (uint32_t)sizeof(CT);
    constexpr uint32_t full = (1u << V) - 1u;

    const CT om = (CT)a.omega, om1 = CT(1.0) - om;
    const CT diag0 = CT(6.0) + (CT)a.kappa2;
    CT rd0;
    if constexpr (sizeof(CT) == 4) rd0 = a.rdiag[kTileDiag0];
    else rd0 = CT(1.0) / diag0;

    auto ld = [&](const CT *row) -> P {
        const typename P::Ext t = *reinterpret_cast<GlobalPtr<const typename P::Ext>>(
            uniform_ptr(reinterpret_cast<const char *>(row)) + io);
        P r;
#pragma unroll
        for (int v = 0; v < V; ++v) r.v[v] = t[v];
        return r;
    };
    auto st = [&](CT *row, const P &v) {
        typename P::Ext t;
#pragma unroll
        for (int k = 0; k < V; ++k) t[k] = v.v[k];
        *reinterpret_cast<GlobalPtr<typename P::Ext>>(
            uniform_ptr(reinterpret_cast<char *>(row)) + io) = t;
    };
    auto zero = [](P &q) {
#pragma unroll
        for (int v = 0; v < V; ++v) q.v[v] = CT(0);
    };
    const uint32_t hxy32 = (uint32_t)hxy;
    const uint32_t total = nyb * (uint32_t)nz;
    const uint32_t wg = a.xcd_swizzle ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
    // this workgroup's planes of the row blocks laid end to end
    uint32_t t0 = wg * planes, t1 = min(total, t0 + planes);
    if (cols) {
        const uint32_t c = wg / cols;
        t0 = c * (uint32_t)nz + (wg - c * cols) * planes;
        t1 = min((c + 1) * (uint32_t)nz, t0 + planes);
    }
    while (t0 < t1) {
        const uint32_t yb = t0 / (uint32_t)nz;
        const int zs = (int)(t0 - yb * (uint32_t)nz);
        const int ze = min(nz, zs + (int)(t1 - t0));
        t0 += (uint32_t)(ze - zs);
        const int yu = (int)yb * (ns - 2 * (S - 1)) + slot - (S - 1);  // unwrapped row
        const int y = ((yu % ny) + ny) % ny;
        uint32_t fl = flags0;
        if (slot >= S - 1 && slot <= ns - S && yu < ny) fl |= kMine;
        if (!g.per[1] && y == 0) fl |= kYlo;
        if (!g.per[1] && y == ny - 1) fl |= kYhi;
        const uint32_t ro = (uint32_t)hx * (uint32_t)y;
        const uint32_t rx = (uint32_t)hx * (uint32_t)(slot == 0 ? (y == 0 ? ny - 1 : y - 1)
                                                                : (y == ny - 1 ? 0 : y + 1));
        // first entry of plane z (in 32 bits: N / 2 < 2^31)
        auto first = [&](int z) -> uint32_t { return hxy32 * (uint32_t)(((z % nz) + nz) % nz); };
        auto word = [&](uint32_t f) -> uint2 { return mb[(f + (uint32_t)ec) >> 5]; };
        auto nibbles = [&](uint32_t f, uint2 m) -> uint32_t {  // red low, black above
            const uint32_t b = (f + (uint32_t)ec) & 31u;
            return ((m.x >> b) & full) | (((m.y >> b) & full) << V);
        };
        // the row constants of colour c where the lane's bits are not all
        // interior (uniform: nothing where none of the wavefront's lanes has any)
        auto coef = [&](int c, uint32_t f, uint32_t nib, RowCoef<CT, V> &q) {
            const bool need = ((nib >> (c * V)) & full) != full;
            if (__ballot(need) == 0ull) return;
#pragma unroll
            for (int v = 0; v < V; ++v) q.rhs.v[v] = CT(0);
            if constexpr (sizeof(CT) == 4) {
                q.code = kTileDiag0 * 0x01010101u;
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v) q.diag.v[v] = diag0;
            }
            if (need) {
                const size_t e = (size_t)c * ts + f;
                q.rhs = ld(rhs + e);
                if constexpr (sizeof(CT) == 4) {
                    const GlobalPtr<const uint8_t> cp = uniform_ptr(code + e) + (uint32_t)ec;
                    if constexpr (V == 4) q.code = *reinterpret_cast<GlobalPtr<const uint32_t>>(cp);
                    else if constexpr (V == 2) q.code = *reinterpret_cast<GlobalPtr<const uint16_t>>(cp);
                    else q.code = *cp;
                } else {
                    q.diag = ld(dgs + e);
                }
            }
        };

        P G[S][3], Ro;
        uint32_t nib[S];
        RowCoef<CT, V> co[S];
        uint2 wn;
        const int P0 = zs - (S - 1);  // stage 0's first plane
        // entry offsets of planes p0 + 2, p0 + 1, ..., p0 - S + 1
        uint32_t fo[S + 2];
        int zn = ((P0 + 2) % nz + nz) % nz;  // plane p0 + 2, wrapped
#pragma unroll
        for (int j = 0; j < S + 2; ++j) fo[j] = first(P0 + 2 - j);
        __syncthreads();  // the previous range's reads of the rows in LDS
        {
            G[0][0] = ld(A + (half32 + fo[3] + ro));
            G[0][1] = ld(A + (half32 + fo[2] + ro));
            G[0][2] = ld(A + (half32 + fo[1] + ro));
            Ro = ld(A + (fo[2] + ro));
#pragma unroll
            for (int j = 0; j < S; ++j) {
                nib[j] = (1u << (2 * V)) - 1u;
                if (j > 0) {
                    zero(G[j][0]);
                    zero(G[j][1]);
                    zero(G[j][2]);
                }
            }
            nib[0] = nibbles(fo[2] + ro, word(fo[2] + ro));
            coef(0, fo[2] + ro, nib[0], co[0]);
            wn = word(fo[1] + ro);
            *reinterpret_cast<P *>(lds(0, 0) + lo) = G[0][1];
        }
        if (fl & kOuter) *reinterpret_cast<P *>(lds(0, 0) + lx) = ld(A + (half32 + fo[2] + rx));
        const int steps = ze - zs + 2 * (S - 1);
        const int zlo = g.per[2] ? INT_MIN : 0, zhi = g.per[2] ? INT_MIN : nz - 1;

        // step t; the windows rotate by name: a, b, c are planes -1, 0, +1
        auto step = [&](int t, auto ph) {
            constexpr int ia = decltype(ph)::value % 3, ib = (ia + 1) % 3, ic = (ia + 2) % 3;
            const int par = t & 1;
            const int p0 = P0 + t;  // stage 0's plane
            // the next step's operands
            P Gn, Rn, Xn;
            uint2 wt;
            uint32_t nib_n;
            {
                Gn = ld(A + (half32 + fo[0] + ro));
                Rn = ld(A + (fo[1] + ro));
                wt = word(fo[0] + ro);
                nib_n = nibbles(fo[1] + ro, wn);
            }
            Xn = Rn;
            if (fl & kOuter) Xn = ld(A + (half32 + fo[1] + rx));
            __syncthreads();
            P nw;
#pragma unroll
            for (int j = 0; j < S; ++j) {
                // before step 2 j a stage's operands are not complete and its
                // values are not used: it rests (a range of few planes spends
                // much of its time here: per iteration 64^3 FP32 9.3 -> 8.5
                // us, 320 x 300 x 280 FP32 54.5 -> 52.5, 192 x 160 x 128 FP64
                // 25.3 -> 24.2; 512^3 equal)
                if (t >= 2 * j) {
                const int pj = p0 - j;
                P up, dn;
                up = *reinterpret_cast<const P *>(lds(par, j) + lo - rb);
                dn = *reinterpret_cast<const P *>(lds(par, j) + lo + rb);
                {
                    if (fl & kYlo) zero(up);
                    if (fl & kYhi) zero(dn);
                    // planes beyond a non-periodic edge: 0 (nothing else uses them)
                    if (pj == zlo) zero(G[j][ia]);
                    if (pj == zhi) zero(G[j][ic]);
                }
                // x-neighbours: entry i itself and entry i + 1 (p = 1) or
                // i - 1 (p = 0); the cell of entry i is x = 2 i + p, and
                // (j & 1) + y + pj has the parity of y + p0 in every stage
                P s;
                auto right = [&] {
                    const P &c = G[j][ib];
                    CT nxt = lane_next(c.v[0]);
                    if (!(fl & kRot)) {
                        CT end = *reinterpret_cast<const CT *>(lds(par, j) + er_o);
                        if (fl & kXr) end = CT(0);
                        if (lane == lw) nxt = end;
                    }
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        s.v[v] = c.v[v] + (v + 1 < V ? c.v[v + 1 < V ? v + 1 : v] : nxt);
                    keep(s);
                };
                auto left = [&] {
                    const P &c = G[j][ib];
                    CT prv = lane_prev(c.v[V - 1]);
                    if (!(fl & kRot)) {
                        CT end = *reinterpret_cast<const CT *>(lds(par, j) + el_o);
                        if (fl & kXl) end = CT(0);
                        if (lane == 0) prv = end;
                    }
#pragma unroll
                    for (int v = 0; v < V; ++v) s.v[v] = (v > 0 ? c.v[v > 0 ? v - 1 : 0] : prv) + c.v[v];
                    keep(s);
                };
                if ((y + p0) & 1) {
                    right();
                } else {
                    left();
                }
                {
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        s.v[v] = (((s.v[v] + up.v[v]) + dn.v[v]) + G[j][ia].v[v]) +
                                    G[j][ic].v[v];
                }
                {
                    const P old = j == 0 ? Ro : G[j > 0 ? j - 1 : 0][ia];
                    const bool gen = __ballot(((nib[j] >> ((j & 1) * V)) & full) != full) != 0ull;
                    if (!gen) {
#pragma unroll
                        for (int v = 0; v < V; ++v)
                            nw.v[v] = om1 * old.v[v] + om * quot_const(s.v[v], diag0, rd0);
                    } else if constexpr (sizeof(CT) == 4) {
#pragma unroll
                        for (int v = 0; v < V; ++v) {
                            // (a solid cell holds 0: 0 from this product is its result)
                            const float r = rd[(co[j].code >> (8 * v)) & 15u];
                            nw.v[v] = om1 * old.v[v] + om * mul_zero(co[j].rhs.v[v] + s.v[v], r);
                        }
                    } else {
#pragma unroll
                        for (int v = 0; v < V; ++v) {
                            const double d = co[j].diag.v[v];  // a solid cell's is infinite
                            const double r = om1 * old.v[v] + om * ((co[j].rhs.v[v] + s.v[v]) / d);
                            nw.v[v] = (__double2hiint(d) & 0x7ff00000) == 0x7ff00000 ? 0.0 : r;
                        }
                    }
                    if (j + 1 < S) {
                        G[j + 1 < S ? j + 1 : j][ic] = nw;
                        *reinterpret_cast<P *>(lds(par ^ 1, j + 1) + lo) = nw;
                    }
                }
                }
                // the row constants of the next step, in the registers that
                // this stage is done with
                if (j < S - 2) coef(j & 1, fo[1 + j] + ro, j == 0 ? nib_n : nib[j > 0 ? j - 1 : 0], co[j]);
            }
            // the operands of the next step have to be here before the loads
            // and stores below are issued: their number varies, so a later
            // wait could not tell them apart
            keep(Gn);
            keep(Rn);
            keep(wt.x);
            keep(wt.y);
            if (fl & kOuter) *reinterpret_cast<P *>(lds(par ^ 1, 0) + lx) = Xn;
            coef((S - 2) & 1, fo[S - 1] + ro, S == 2 ? nib_n : nib[S > 2 ? S - 3 : 0], co[S - 2]);
            coef((S - 1) & 1, fo[S] + ro, nib[S - 2], co[S - 1]);
            {
                *reinterpret_cast<P *>(lds(par ^ 1, 0) + lo) = G[0][ic];
                if ((fl & kMine) && act) {
                    // black of plane p0 - S + 1 = z, red of plane z + 1
                    if (t >= 2 * (S - 1)) st(B + (half32 + fo[S + 1] + ro), nw);
                    if (t >= 2 * (S - 1) - 1 && t < steps - 1) st(B + (fo[S] + ro), G[S - 1][ic]);
                }
                // one plane up
#pragma unroll
                for (int j = S - 1; j > 0; --j) nib[j] = nib[j - 1];
                nib[0] = nib_n;
                G[0][ia] = Gn;  // plane p0 + 2
                Ro = Rn;
                wn = wt;
            }
#pragma unroll
            for (int j = S + 1; j > 0; --j) fo[j] = fo[j - 1];
            if (++zn == nz) {
                zn = 0;
                fo[0] = 0;
            } else {
                fo[0] += hxy32;
            }
        };
        for (int t = 0; t < steps; t += 3) {
            step(t, std::integral_constant<int, 0>{});
            if (t + 1 < steps) step(t + 1, std::integral_constant<int, 1>{});
            if (t + 2 < steps) step(t + 2, std::integral_constant<int, 2>{});
        }
    }
}

// once per solve, before the first pass: the rows of the boundary cells
// (rhs, and the diagonal as a code in FP32 and as a value in FP64, both
// formed as dha_row forms them), the solid cells' codes, and the solid
// cells' own values kept in save.  With surface potentials the right-hand
// sides do not read psi and the solid cells are zeroed here, otherwise by
// k_tile_solid afterwards.  A thread reads the flags of E entries of a row
// (2 E cells, one load); the cells of the groups with a boundary or solid
// cell are listed in LDS and taken one per lane (a thread per group that
// walked its cells took 426 us at 512^3 with 4096 spheres, bound by its chain
// of dependent loads).  E is a multiple of the V entries that a lane of the
// pass loads together: all of a group's rows are written.
template <int E>
__device__ __forceinline__ uint64_t pair_flags(const uint8_t *p) {
    if constexpr (E == 4) return *reinterpret_cast<const uint64_t *>(p);
    else if constexpr (E == 2) return *reinterpret_cast<const uint32_t *>(p);
    else return *reinterpret_cast<const uint16_t *>(p);
}
template <typename CT, int E>
__global__ void __launch_bounds__(256) k_tile_prepare(SorArgs a, CT *psi, CT *save) {
    const Grid &g = a.g;
    const int nx = g.nx, ny = g.ny, nz = g.nz, hx = nx >> 1;
    // the block's cells whose rows are written: cell of the block (thread
    // and cell of its group) | flag bits << 11, in no particular order
    __shared__ uint16_t list[256 * 2 * E];
    __shared__ uint32_t count;
    const int tid = (int)(threadIdx.y * blockDim.x + threadIdx.x);
    const int z = (int)blockIdx.z;
    if (tid == 0) count = 0;
    __syncthreads();
    {
        const int i0 = (int)(blockIdx.x * blockDim.x + threadIdx.x) * E;
        const int y = (int)(blockIdx.y * blockDim.y + threadIdx.y);
        if (i0 < hx && y < ny) {
            const size_t c0 = ((size_t)z * (size_t)ny + (size_t)y) * (size_t)nx + 2 * (size_t)i0;
            const uint64_t fw = pair_flags<E>(a.flag + c0);
            if (fw & (0x0101010101010101ull * (kWall | kObst | kNear7))) {
                const uint32_t at = atomicAdd(&count, 2u * E);
#pragma unroll
                for (int m = 0; m < 2 * E; ++m) {
                    const uint32_t fl = (uint32_t)(fw >> (8 * m)) & 0xFFu;
                    list[at + m] = (uint16_t)((tid * 2 * E + m) | (fl & kWall ? 1 << 11 : 0) |
                                              (fl & kObst ? 1 << 12 : 0) | (fl & kNear7 ? 1 << 13 : 0));
                }
            }
        }
    }
    __syncthreads();
    const uint32_t n = count;
    const size_t ts = tile_stride(g.N);
    CT *rhs = static_cast<CT *>(a.nrow);
    CT *dgs = rhs + 2 * ts;
    uint8_t *code = reinterpret_cast<uint8_t *>(a.codes);
    const size_t nxs = (size_t)nx, nxy = nxs * (size_t)ny;
    for (uint32_t i = (uint32_t)tid; i < n; i += 256u) {
        const uint32_t w = list[i];
        const int lc = (int)(w & 2047u), th = lc / (2 * E), m = lc - th * (2 * E);
        const int tx = th & ((int)blockDim.x - 1), ty = th / (int)blockDim.x;
        const int x = 2 * E * ((int)(blockIdx.x * blockDim.x) + tx) + m;
        const int y = (int)(blockIdx.y * blockDim.y) + ty;
        const size_t c = ((size_t)z * (size_t)ny + (size_t)y) * nxs + (size_t)x;
        const uint32_t col = (uint32_t)((x + y + z) & 1);
        const size_t e = (size_t)col * ts + (c >> 1);
        const size_t sl = (size_t)col * (g.Ns >> 1) + (c >> 1);
        if (w & (3u << 11)) {
            rhs[e] = CT(0);
            if constexpr (sizeof(CT) == 4) code[e] = (uint8_t)kTileSolid;
            else dgs[e] = (CT)__builtin_huge_val();
            save[sl] = psi[sl];
            if (a.zeta) psi[sl] = CT(0);
            continue;
        }
        if (!(w & (1u << 13))) {  // an interior cell in the lane of another's row
            rhs[e] = CT(0);
            if constexpr (sizeof(CT) == 4) code[e] = (uint8_t)kTileDiag0;
            else dgs[e] = CT(6.0) + (CT)a.kappa2;
            continue;
        }
        size_t s[6];
        bool edge[6];
        s[0] = x == 0 ? c + nxs - 1 : c - 1;
        s[1] = x == nx - 1 ? c + 1 - nxs : c + 1;
        s[2] = y == 0 ? c + nxy - nxs : c - nxs;
        s[3] = y == ny - 1 ? c + nxs - nxy : c + nxs;
        s[4] = z == 0 ? c + nxy * (size_t)(nz - 1) : c - nxy;
        s[5] = z == nz - 1 ? c - nxy * (size_t)(nz - 1) : c + nxy;
        edge[0] = x == 0 && !g.per[0];
        edge[1] = x == nx - 1 && !g.per[0];
        edge[2] = y == 0 && !g.per[1];
        edge[3] = y == ny - 1 && !g.per[1];
        edge[4] = z == 0 && !g.per[2];
        edge[5] = z == nz - 1 && !g.per[2];
        uint8_t fs[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) fs[k] = edge[k] ? (uint8_t)kWall : a.flag[s[k]];
        uint32_t po[6];
        CT bv[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const bool d = (fs[k] & kObst) && !(fs[k] & kWall);
            po[k] = kNone;
            bv[k] = CT(0);
            if (d && a.zeta) po[k] = a.owner[s[k]];
            if (d && !a.zeta) bv[k] = psi[(size_t)(col ^ 1u) * (g.Ns >> 1) + (s[k] >> 1)];
        }
#pragma unroll
        for (int k = 0; k < 6; ++k)
            if (po[k] != kNone) bv[k] = (CT)a.zeta[po[k]];
        CT diag = CT(6.0) + (CT)a.kappa2, r = CT(0);
        int nd = (int)kTileDiag0;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            if (fs[k] & kWall) {
                diag = diag - CT(1.0);
                --nd;
            } else if (fs[k] & kObst) {
                diag = diag + CT(1.0);
                ++nd;
                r = r + CT(2.0) * bv[k];
            }
        }
        rhs[e] = r;
        if constexpr (sizeof(CT) == 4) code[e] = (uint8_t)nd;
        else dgs[e] = diag;
    }
}

// the solid cells of one or two buffers: to 0 (save null), or back to the
// values kept in save
template <typename CT, int E>
__global__ void __launch_bounds__(256) k_tile_solid(SorArgs a, CT *p0, CT *p1, const CT *save) {
    const Grid &g = a.g;
    const int hx = g.nx >> 1;
    const int i0 = (int)(blockIdx.x * blockDim.x + threadIdx.x) * E;
    const int y = (int)(blockIdx.y * blockDim.y + threadIdx.y), z = (int)blockIdx.z;
    if (i0 >= hx || y >= g.ny) return;
    const size_t c0 = ((size_t)z * (size_t)g.ny + (size_t)y) * (size_t)g.nx + 2 * (size_t)i0;
    const uint64_t fw = pair_flags<E>(a.flag + c0);
    constexpr uint64_t ones = 0x0101010101010101ull;
    if (!(fw & (ones * (kWall | kObst)))) return;
#pragma unroll
    for (int m = 0; m < 2 * E; ++m) {
        if (!((fw >> (8 * m)) & (kWall | kObst))) continue;
        const uint32_t col = (uint32_t)((2 * i0 + m + y + z) & 1);
        const size_t sl = (size_t)col * (g.Ns >> 1) + ((c0 + (size_t)m) >> 1);
        const CT v = save ? save[sl] : CT(0);
        p0[sl] = v;
        if (p1) p1[sl] = v;
    }
}

// shape of a tile pass: entries per lane, wavefronts and row slots; V = 0
// when the rows do not fit
struct TileShape {
    int V = 0, nwx = 0, ns = 0;
};
// As many entries per lane as a 16-byte access holds, as long as the row
// does not fit in the wavefront's lanes with fewer (idle lanes cost as much
// as busy ones).  Rows of more than four wavefronts would leave fewer than
// four rows per workgroup, of which two are halo rows computed twice.
template <typename CT>
TileShape tile_shape(const Grid &g) {
    TileShape t;
    if (g.nx % 2) return t;
    const int hx = g.nx / 2;
    const int vmax = sizeof(CT) == 4 ? 4 : 2;
    int v = 1;
    while (v < vmax && hx % (2 * v) == 0 && hx > 64 * v) v *= 2;
    const int nwx = (hx + 64 * v - 1) / (64 * v);
    if (nwx > 4) return t;
    t.V = v;
    t.nwx = nwx == 3 ? 4 : nwx;  // whole rows of slots (a fourth wavefront idles)
    t.ns = kTileSlots / t.nwx;
    return t;
}

// Up to how many rows (ny nz) of a shape the tile pass is taken; larger grids
// take k_sor_march (even rows of up to 2048 cells).  The march has about 50 us
// per iteration (FP64 70-80) to fill the chip whatever the grid, and costs less
// per row than the tile pass where that computes many rows twice (two of four
// per workgroup with four wavefronts per row, six of eight kept with two) or
// holds one entry per lane.  March / tile pass, us per iteration, at 24.8 / 76.8
// / 256 thousand rows (nx):
//   FP32  V 1       32-128    53 / 19    54 / 36     63-71 / 88-90
//         V 2, 4    256, 512  55 / 22, 58 / 26   59 / 40, 93 / 61   152 / 122, 258 / 161
//         2 wavefronts, V 1   55 / 31    59 / 70     118-160 / 206-275
//                       V 2   57 / 36    62 / 84     185-196 / 301-304
//                       V 4   520: 60 / 42   130 / 125   341 / 361
//                             640-1024: 62-69 / 44-48    128-173 / 128-166
//         4 wavefronts        57-143 / 68-145        73-371 / 178-442
//                       (3.1 thousand rows: 52-54 / 15-18)
//   FP64  V 1       32-128    67-72 / 24-26   78 / 50-54   111-158 / 121-163
//         V 2       256, 512  78 / 31, 90 / 49   120 / 87, 221 / 162   280 / 235, 571 / 501
//         2 wavefronts, V 1   80 / 40    93-127 / 93-123   249-300 / 331-366
//         4 wavefronts, V 1   88-90 / 93-95   219-229 / 296-309
//                       V 2   516, 520: 94 / 103   305 / 318
//                             640-1024: 105-167 / 103-151   317-413 / 326-460
//                             (32 thousand: 125-168 / 148-180)
template <typename CT>
bool tile_pays(const Grid &g, const TileShape &t) {
    constexpr size_t any = ~size_t(0);
    const size_t rows = (size_t)g.ny * (size_t)g.nz;
    const int hx = g.nx / 2;
    size_t lim;
    if (sizeof(CT) == 4)
        lim = t.nwx == 1   ? (t.V == 1 ? 125000 : any)
              : t.nwx == 2 ? (t.V == 1 ? 50000 : t.V == 2 ? 46000 : hx <= 320 ? 150000 : any)
                           : 20000;
    else
        lim = t.nwx == 1   ? (t.V == 1 ? 200000 : any)
              : t.nwx == 2 ? (t.V == 1 ? 76000 : any)
                           : (t.V == 1 || hx < 320 ? 20000 : 28000);
    return t.V > 0 && rows <= lim;
}

// what a solve needs to know of its tile passes
struct TilePlan {
    TileShape shape;
    bool pairs = false;  // two iterations per pass
};
// Two iterations per pass halve the bytes of a solve; their 2 * 3 rows of
// halo need a workgroup of 16 rows (rows in one wavefront).  FP64 takes one:
// the operands of four stages do not fit in 128 registers, and of two rows of
// halo in 16 less is computed twice.  Per iteration in pairs and singly: FP64
// 64^3 13.6 / 11.5, 144^3 29.9 / 24.4, 200^3 45.6 / 37.1, 320 x 300 x 280 149 /
// 141, 512^3 539 / 536 us; FP32 144^3 17.9 / 19.3, 320 x 300 x 280 54 / 65,
// 512^3 196 / 277 us.
template <typename CT>
TilePlan tile_plan(const SorArgs &a, bool fused) {
    TilePlan t;
    if (!fused || !a.psi2 || !a.save || !a.codes) return t;
    t.shape = tile_shape<CT>(a.g);
    if (!tile_pays<CT>(a.g, t.shape)) t.shape = TileShape{};
    t.pairs = sizeof(CT) == 4 && t.shape.V > 0 && t.shape.nwx == 1;
    return t;
}

// one launch of K iterations: one workgroup per resident place, each with an
// equal range of the (row block, plane) space, or whole fractions of a
// column of planes where that takes fewer steps (a range that meets two
// columns fills its pipeline twice); a.mzc > 0 sets the planes
template <typename CT, int V, int K>
void launch_tile(const SorArgs &a, const TileShape &t, const CT *src, CT *dst, hipStream_t s) {
    auto lds_of = [](int nwx) {
        return 2u * 2u * K * (uint32_t)((kTileSlots / nwx + 2) * nwx) * 64u * V * (uint32_t)sizeof(CT);
    };
    // places of workgroups on the device by wavefronts per row (1, 2, 4)
    static DeviceTable<std::array<int, 3>> table;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    const std::array<int, 3> places = table.get(dev, [&] {
        int cu = 256;
        hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev);
        hipFuncSetAttribute(reinterpret_cast<const void *>(&k_sor_tile<CT, V, K>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_of(K == 2 ? 1 : 4));
        std::array<int, 3> r;
        for (int i = 0; i < 3; ++i) {
            int per = 1;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_sor_tile<CT, V, K>, 64 * kTileWaves,
                                                             lds_of(1 << i)) != hipSuccess || per < 1)
                per = 1;
            r[i] = cu * per;
        }
        (void)hipGetLastError();
        return r;
    });
    const uint32_t lds = lds_of(t.nwx);
    const int resident = places[t.nwx == 4 ? 2 : t.nwx - 1];
    const Grid &g = a.g;
    const int own = t.ns - 2 * (2 * K - 1), fill = 2 * (2 * K - 1);
    const uint32_t nyb = (uint32_t)((g.ny + own - 1) / own), nz = (uint32_t)g.nz;
    const uint32_t total = nyb * nz;
    uint32_t planes = (total + (uint32_t)resident - 1) / (uint32_t)resident, cols = 0;
    uint32_t cost = planes + (planes > 1 && nz % planes ? 2 : 1) * (uint32_t)fill;
    if ((uint32_t)resident >= nyb) {
        const uint32_t per = std::min(nz, (uint32_t)resident / nyb), pl = (nz + per - 1) / per;
        if (pl + (uint32_t)fill < cost) {
            planes = pl;
            cols = (nz + pl - 1) / pl;
        }
    }
    if (a.mzc > 0) {
        planes = std::min(nz, a.mzc);
        cols = (nz + planes - 1) / planes;
    }
    const uint32_t grid = cols ? cols * nyb : (total + planes - 1) / planes;
    hipLaunchKernelGGL((k_sor_tile<CT, V, K>), dim3(grid), dim3(64 * kTileWaves), lds, s, a, src,
                       dst, t.nwx, t.ns, nyb, planes, cols);
}

template <typename CT>
void launch_tile_pass(const SorArgs &a, const CT *src, CT *dst, int k, hipStream_t s) {
    const TileShape t = tile_shape<CT>(a.g);
    if constexpr (sizeof(CT) == 4) {
        if (k == 2) {
            if (t.V == 4) return launch_tile<CT, 4, 2>(a, t, src, dst, s);
            if (t.V == 2) return launch_tile<CT, 2, 2>(a, t, src, dst, s);
            return launch_tile<CT, 1, 2>(a, t, src, dst, s);
        }
        if (t.V == 4) return launch_tile<CT, 4, 1>(a, t, src, dst, s);
    }
    if (t.V == 2) return launch_tile<CT, 2, 1>(a, t, src, dst, s);
    return launch_tile<CT, 1, 1>(a, t, src, dst, s);
}

// launch shape of the passes over the flags: E entries (8 cells, whose flags
// are one aligned 8-byte load) per thread where the rows allow it
struct FlagGrid {
    dim3 grid, block;
    FlagGrid(const Grid &g, int e) {
        const int n = (g.nx / 2 + e - 1) / e;
        int tx = 64;
        while (tx > 8 && tx / 2 >= n) tx /= 2;
        const int ty = 256 / tx;
        block = dim3(tx, ty);
        grid = dim3((n + tx - 1) / tx, (g.ny + ty - 1) / ty, g.nz);
    }
};

template <typename CT>
void launch_tile_solid(const SorArgs &a, CT *p0, CT *p1, const CT *save, hipStream_t s) {
    if (a.g.nx % 8 == 0) {
        const FlagGrid f(a.g, 4);
        hipLaunchKernelGGL((k_tile_solid<CT, 4>), f.grid, f.block, 0, s, a, p0, p1, save);
    } else if (a.g.nx % 4 == 0) {
        const FlagGrid f(a.g, 2);
        hipLaunchKernelGGL((k_tile_solid<CT, 2>), f.grid, f.block, 0, s, a, p0, p1, save);
    } else {
        const FlagGrid f(a.g, 1);
        hipLaunchKernelGGL((k_tile_solid<CT, 1>), f.grid, f.block, 0, s, a, p0, p1, save);
    }
}

template <typename CT>
void launch_tile_prepare(const SorArgs &a, hipStream_t s) {
    CT *psi = static_cast<CT *>(a.psi), *save = static_cast<CT *>(a.save);
    if (a.g.nx % 8 == 0) {
        const FlagGrid f(a.g, 4);
        hipLaunchKernelGGL((k_tile_prepare<CT, 4>), f.grid, f.block, 0, s, a, psi, save);
    } else if (a.g.nx % 4 == 0) {
        const FlagGrid f(a.g, 2);
        hipLaunchKernelGGL((k_tile_prepare<CT, 2>), f.grid, f.block, 0, s, a, psi, save);
    } else {
        const FlagGrid f(a.g, 1);
        hipLaunchKernelGGL((k_tile_prepare<CT, 1>), f.grid, f.block, 0, s, a, psi, save);
    }
    if (!a.zeta && a.solids)
        launch_tile_solid<CT>(a, psi, static_cast<CT *>(nullptr), static_cast<const CT *>(nullptr), s);
}

}  // namespace
}  // namespace lbmep
