// near_impl.h -- velocity bounce-back and momentum exchange at the fluid
// cells next to solid cells (arXiv:1708.08741, Sec. 3.2: Eq. LBMMovWall and
// Eq. LBMhydrodynForce with the torque about the particle centre).
//
// Runs after the sweep on the post-collision state f* it wrote.  For every
// blocked link (fluid cell x, direction q, solid neighbour s = x + e_q) the
// value that returns to x as population q-bar at the next gather,
//     f*_q(x) - 2 w_q rho0 c_q.u_s / c_s^2,
// is written into slot q-bar of s (solid cells are not updated, so their
// slots are free); a link to an obstacle cell of particle p adds
// [2 f*_q - 2 w_q rho0 c_q.u_s / c_s^2] c_q to F_p and r x (that) to M_p.
//
// Work distribution: one workgroup per particle walks the particle's link
// list (written by the classification: the fluid cells next to the particle
// with the directions that hit it), one link per lane, so the particle's
// position and velocities are uniform, no owner
// look-up is needed, and force and torque are summed over each wavefront in
// a fixed order (DPP row butterflies), the wavefronts' sums are combined in
// wavefront order through LDS after one barrier, and the result is stored
// without atomics.  Links to wall cells come from a list built when the
// walls are set.
#pragma once
#include "particles_impl.h"
#include "sweep_impl.h"

namespace lbmep {
namespace sweep {

// per-particle sums: F_dev[3], M_dev[3], K[3], T[3]
constexpr int kAcc = 12;

// v of the lane selected by a DPP control inside each row of 16 lanes (the
// two 32-bit halves moved separately)
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)(uint32_t)hi << 32) |
                                            (unsigned long long)(uint32_t)lo));
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// sum of v over the wavefront (all 64 lanes active): butterfly inside each
// row of 16 by DPP (xor 1 and 2 by quad permutes, then the half-row and row
// mirrors), then the four row sums read from lanes 0, 16, 32, 48
__device__ __forceinline__ double wave_sum_f64(double v) {
    v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);  // row_half_mirror
    v += dpp_f64<0x140>(v);  // row_mirror
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// the D3Q19 velocity components as 2-bit fields (value + 1), for directions
// known only at run time
constexpr uint64_t pack_dir(const int (&v)[Q]) {
    uint64_t r = 0;
    for (int q = 0; q < Q; ++q) r |= (uint64_t)(v[q] + 1) << (2 * q);
    return r;
}
constexpr uint64_t kPackCx = pack_dir(kCx), kPackCy = pack_dir(kCy), kPackCz = pack_dir(kCz);

__device__ __forceinline__ int dir_comp(uint64_t packed, int q) {
    return (int)((packed >> (2 * q)) & 3u) - 1;
}

// wrap one coordinate of a neighbour on a periodic axis; false beyond the
// edge of a non-periodic axis
__device__ __forceinline__ bool wrap_axis(int &v, int len, int periodic) {
    if (v < 0 || v >= len) {
        if (!periodic) return false;
        v = v < 0 ? v + len : v - len;
    }
    return true;
}

// the value bounced into slot opp(q) of the solid neighbour s
template <typename ST, typename OFF>
__device__ __forceinline__ void store_slot(const SweepArgs &a, int q, OFF s,
                                           typename Storage<ST>::CT fq, double mw) {
    using T = Storage<ST>;
    using CT = typename T::CT;
    // population base in 64 bits (q Ns can exceed 4 GiB), cell offset in OFF
    void *slot_base = static_cast<char *>(a.dst) + (size_t)opp(q) * a.g.Ns * sizeof(ST);
    ST *slot = at<ST>(slot_base, s * (OFF)sizeof(ST));
    if constexpr (sizeof(CT) == 8) {
        T::store(slot, fq - mw);
    } else {
        T::store(slot, (CT)((double)fq - mw));
    }
}

// post-collision value of population q of cell c
template <typename ST, typename OFF>
__device__ __forceinline__ typename Storage<ST>::CT load_fstar(const SweepArgs &a, int q,
                                                               uint32_t c) {
    const void *base = static_cast<const char *>(a.dst) + (size_t)q * a.g.Ns * sizeof(ST);
    return Storage<ST>::load(at<ST>(base, (OFF)c * (OFF)sizeof(ST)));
}

// One link of particle p from cell (x, y, z) in direction q (1..18, known at
// run time) with the post-collision value fq: the bounce-back slot and the momentum exchange
// into the lane's sums.
template <typename ST, typename OFF>
__device__ __forceinline__ void particle_link(const SweepArgs &a, int x, int y, int z, int q,
                                              typename Storage<ST>::CT fq, const double Xp[3], const double Up[3],
                                              const double Wp[3], double acc[kAcc]) {
    using T = Storage<ST>;
    const Grid &g = a.g;
    const int cx = dir_comp(kPackCx, q), cy = dir_comp(kPackCy, q), cz = dir_comp(kPackCz, q);
    int sx = x + cx, sy = y + cy, sz = z + cz;
    wrap_axis(sx, g.nx, g.per[0]);  // an obstacle cell: always inside
    wrap_axis(sy, g.ny, g.per[1]);
    wrap_axis(sz, g.nz, g.per[2]);
    // lever arm r = x_s - x_C (minimum image) and u_s = U + W x r
    const double r0 = min_image(((double)sx + 0.5) - Xp[0], g.nx, g.per[0]);
    const double r1 = min_image(((double)sy + 0.5) - Xp[1], g.ny, g.per[1]);
    const double r2 = min_image(((double)sz + 0.5) - Xp[2], g.nz, g.per[2]);
    const double us0 = Up[0] + (Wp[1] * r2 - Wp[2] * r1);
    const double us1 = Up[1] + (Wp[2] * r0 - Wp[0] * r2);
    const double us2 = Up[2] + (Wp[0] * r1 - Wp[1] * r0);
    // c_q . u_s with unit components: the zero terms add exact zeros
    const double cus = ((double)cx * us0 + (double)cy * us1) + (double)cz * us2;
    const double w = q <= 6 ? wq(1) : wq(7);
    // 2 (w_q / c_s^2) rho0 c_q . u_s (Eq. LBMMovWall)
    const double mw = 2.0 * w * 3.0 * cus;
    // [2 f*_q - 2 (w_q/c_s^2) rho0 c_q . u_s] c_q (Eq. LBMhydrodynForce),
    // summed as [2 (f*_q - w_q) - ...] c_q plus the rest-weight part
    // 2 w_q c_q = (k/18) c_q (k = 2 axis, 1 diagonal), whose sum cancels
    // over a closed body and is accumulated exactly as integers:
    // K = sum k c_q, T = sum k x_s x c_q (x_s the exact half-integer image
    // of the cell centre)
    const double gm = 2.0 * T::devval(fq, q) - mw;
    const double g0 = cx == 0 ? 0.0 : (cx > 0 ? gm : -gm);
    const double g1 = cy == 0 ? 0.0 : (cy > 0 ? gm : -gm);
    const double g2 = cz == 0 ? 0.0 : (cz > 0 ? gm : -gm);
    const double k = q <= 6 ? 2.0 : 1.0;
    const double xs0 = image_coord((double)sx + 0.5, Xp[0], g.nx, g.per[0]);
    const double xs1 = image_coord((double)sy + 0.5, Xp[1], g.ny, g.per[1]);
    const double xs2 = image_coord((double)sz + 0.5, Xp[2], g.nz, g.per[2]);
    acc[0] += g0;
    acc[1] += g1;
    acc[2] += g2;
    acc[3] += r1 * g2 - r2 * g1;
    acc[4] += r2 * g0 - r0 * g2;
    acc[5] += r0 * g1 - r1 * g0;
    acc[6] += k * (double)cx;
    acc[7] += k * (double)cy;
    acc[8] += k * (double)cz;
    acc[9] += k * (xs1 * (double)cz - xs2 * (double)cy);
    acc[10] += k * (xs2 * (double)cx - xs0 * (double)cz);
    acc[11] += k * (xs0 * (double)cy - xs1 * (double)cx);
    const OFF s = (OFF)sx + (OFF)g.nx * ((OFF)sy + (OFF)g.ny * (OFF)sz);
    store_slot<ST, OFF>(a, q, s, fq, mw);
}

// LDS of near_particle by NT threads: per pass the cells of NT list entries and
// their links (at most 18 each) as entry | direction, then the sums
constexpr uint32_t near_lds_of(int nt) {
    return (uint32_t)(nt * 12 + nt * (Q - 1) * 2 + (nt / 64 + 1) * kAcc * 8 + 64);
}

// All links of particle p (its list from the classification: cells with the
// directions whose neighbour is an obstacle cell of p), one workgroup: the
// bounce-back slots and the momentum exchange, summed in a fixed order and
// stored (no atomics: the result does not depend on scheduling).  The
// workgroup takes one list entry per thread and pass and lays their links
// out one after the other, then works through them one link per lane, three
// per lane at a time with their loads issued together.  Bound by the chain
// of dependent round trips (list, links, values), so a particle of radius 4
// (about 300 entries, 1200 links) should fit one pass of one round: with 256
// threads and 128 entries per pass it took three passes of two rounds.
// Returns the 12 sums in LDS.
template <typename ST, typename OFF, int NT>
__device__ __forceinline__ const double *near_particle(const SweepArgs &a, uint32_t p,
                                                       unsigned char *lds) {
    using CT = typename Storage<ST>::CT;
    constexpr int NW = NT / 64;
    double *part = reinterpret_cast<double *>(lds);      // [NW + 1][kAcc]
    uint32_t *ecell = reinterpret_cast<uint32_t *>(part + (NW + 1) * kAcc);
    uint32_t *ex = ecell + NT, *eyz = ex + NT;  // its coordinates
    uint32_t *wsum = eyz + NT;
    uint16_t *link = reinterpret_cast<uint16_t *>(wsum + 16);
    const int tid = (int)threadIdx.x, lane = (int)__lane_id(), wave = tid / 64;
    const uint2 *list = a.plist + (size_t)p * a.pcap;
    const uint32_t n = a.pcount[p];
    const double Xp[3] = {a.Xc[3 * (size_t)p], a.Xc[3 * (size_t)p + 1], a.Xc[3 * (size_t)p + 2]};
    const double Up[3] = {a.U[3 * (size_t)p], a.U[3 * (size_t)p + 1], a.U[3 * (size_t)p + 2]};
    const double Wp[3] = {a.W[3 * (size_t)p], a.W[3 * (size_t)p + 1], a.W[3 * (size_t)p + 2]};
    double acc[kAcc];
#pragma unroll
    for (int j = 0; j < kAcc; ++j) acc[j] = 0.0;
    for (uint32_t i0 = 0; i0 < n; i0 += NT) {
        const uint32_t i = i0 + (uint32_t)tid;
        const uint2 e = i < n ? list[i] : make_uint2(0u, 0u);
        if (e.y) {  // one index decomposition per cell, not per link
            const uint32_t row = e.x / (uint32_t)a.g.nx, z = row / (uint32_t)a.g.ny;
            ecell[tid] = e.x;
            ex[tid] = e.x - row * (uint32_t)a.g.nx;
            eyz[tid] = (row - z * (uint32_t)a.g.ny) | z << 16;  // ny, nz <= 65535
        }
        uint32_t total;
        uint32_t pos = part::block_prefix((uint32_t)__popc(e.y), wsum, &total);
        for (uint32_t m = e.y; m; m &= m - 1u) link[pos++] = (uint16_t)(tid << 5 | __ffs((int)m));
        __syncthreads();
        constexpr int U = 3;
        for (uint32_t k0 = (uint32_t)tid; k0 < total; k0 += U * NT) {
            uint32_t en[U];
            int q[U];
            CT fq[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t k = k0 + (uint32_t)u * NT;
                const uint32_t l = link[k < total ? k : k0];
                en[u] = l >> 5;
                q[u] = (int)(l & 31u);
                fq[u] = load_fstar<ST, OFF>(a, q[u], ecell[en[u]]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + (uint32_t)u * NT < total) {
                    const uint32_t yz = eyz[en[u]];
                    particle_link<ST, OFF>(a, (int)ex[en[u]], (int)(yz & 0xFFFFu), (int)(yz >> 16), q[u],
                                           fq[u], Xp, Up, Wp, acc);
                }
        }
        __syncthreads();  // the links are rewritten by the next pass
    }
    // wave sums, then the waves' sums in wave order: a fixed order
#pragma unroll
    for (int k = 0; k < kAcc; ++k) {
        const double t = wave_sum_f64(acc[k]);
        if (lane == 0) part[wave * kAcc + k] = t;
    }
    __syncthreads();
    double *sum = part + NW * kAcc;
    if (tid < kAcc) {
        double t = part[tid];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += part[w * kAcc + tid];
        sum[tid] = t;
        if (a.FM) a.FM[kAcc * (size_t)p + tid] = t;
    }
    return sum;
}

// Newton-Euler update of particle p (Alg. "Electrophoresis Algorithm": the
// hydrodynamic force and torque of the step and the force q E of the
// applied field move the particle), one explicit step, velocities first:
//     U += (F_h + q E) / m,  W += M_h / I,  X(n+1) = X(n) + U,
// m = rho_p 4/3 pi R^3, I = 2/5 m R^2; F_h, M_h assembled from the 12 sums t
// as k_finalize_ft does, in the same order; one component per thread.  A
// component of one cell per step or more (an infinity and a NaN too) is
// reported and leaves the position as it is: the flags of a step are renewed
// around the positions of two levels, so after a longer way marks of the level
// before would stay whose owners the maps do not hold any more.
__device__ __forceinline__ void move_particle(const ParticleArgs &pa, const DynArgs &d, uint32_t p,
                                              const double *t, const double *Xp) {
    if (threadIdx.x >= 3) return;
    const int k = (int)threadIdx.x, k1 = (k + 1) % 3, k2 = (k + 2) % 3;
    const double F = t[k] + t[6 + k] / 18.0;
    const double M = t[3 + k] + (t[9 + k] - (Xp[k1] * t[6 + k2] - Xp[k2] * t[6 + k1])) / 18.0;
    const double R = pa.R[p];
    const double m = d.rho_p * (4.0 / 3.0) * 3.14159265358979323846 * R * R * R;
    const double I = 0.4 * m * R * R;
    const double qp = d.q ? d.q[p] : 0.0;
    const size_t i = 3 * (size_t)p + (size_t)k;
    const int len = k == 0 ? pa.g.nx : k == 1 ? pa.g.ny : pa.g.nz;
    const double u = d.U[i] + (F + qp * d.E[k]) / m;
    d.U[i] = u;
    d.W[i] = d.W[i] + M / I;
    const bool fast = !(fabs(u) < 1.0);
    double x = fast ? Xp[k] : Xp[k] + u;
    if (pa.g.per[k]) {
        x = x - (double)len * floor(x / (double)len);
        if (x >= (double)len) x -= (double)len;
    }
    d.X0[i] = x;
    if (fast) *d.too_fast = 1;
}

// Links to wall cells (a list fixed while the walls are): plain bounce-back
// from a resting wall, grid-stride over the listed cells with their
// wall-link masks.
template <typename ST, typename OFF>
__device__ __forceinline__ void near_walls(const SweepArgs &a, uint32_t blk, uint32_t nblk) {
    using CT = typename Storage<ST>::CT;
    const uint32_t n = *a.wcount;
    const Grid &g = a.g;
    const int nx = g.nx, ny = g.ny;
    for (uint32_t i = blk * blockDim.x + threadIdx.x; i < n; i += nblk * blockDim.x) {
        const uint32_t c = a.wlist[i];
        uint32_t mask = a.nearmask[c];
        const int x = (int)(c % (uint32_t)nx);
        const int y = (int)((c / (uint32_t)nx) % (uint32_t)ny);
        const int z = (int)(c / ((uint32_t)nx * (uint32_t)ny));
        while (mask) {
            const int q = __ffs((int)mask);
            mask &= mask - 1u;
            int sx = x + dir_comp(kPackCx, q), sy = y + dir_comp(kPackCy, q),
                sz = z + dir_comp(kPackCz, q);
            wrap_axis(sx, nx, g.per[0]);  // a wall cell: always inside
            wrap_axis(sy, ny, g.per[1]);
            wrap_axis(sz, g.nz, g.per[2]);
            const CT fq = load_fstar<ST, OFF>(a, q, c);
            const OFF s = (OFF)sx + (OFF)nx * ((OFF)sy + (OFF)ny * (OFF)sz);
            store_slot<ST, OFF>(a, q, s, fq, 0.0);
        }
    }
}

// LDS of a particle workgroup: the exchange or the classification
inline uint32_t parts_lds(int mode, uint32_t box_rows, int nt) {
    const uint32_t c = classify_lds(box_rows, nt), n = near_lds_of(nt);
    return mode != kPartsSplit && mode != kPartsOne ? n : c > n ? c : n;
}

// the particle workgroups of a step, blk of np (3 np when split, 2 np with the
// emptying beside the exchange) + wall blocks.  The classification of the next level reads that level's map
// (complete since the sweep's launch), the current one and the walls, and
// writes flags and the next level's link lists; the exchange reads the
// current lists and the post-collision state; nothing reads the previous
// level's map any more: they run side by side.  (DYN: lattices with dynamics
// may come; its run-time component index would keep the arguments that a
// packed launch loads in scratch memory.)
template <typename ST, typename OFF, bool DYN, int NT>
__device__ __forceinline__ void parts_block(const SweepArgs &a, const PartsArgs &q, uint32_t blk) {
    extern __shared__ __align__(16) unsigned char part_lds[];
    const uint32_t np = (uint32_t)a.np;
    constexpr bool kMany = NT == kManyThreads;  // the classification is elsewhere
    if (kMany ? q.mode == kPartsClear : q.mode == kPartsSplit) {
        if constexpr (!kMany) {
            if (blk < np) {  // first: these take longer
                part::classify(q.pa, (int)blk, q.cur, q.next, part::box_rows(part_lds, q.pa.box_rows));
                return;
            }
            blk -= np;
        }
        if (blk >= np + (uint32_t)q.wall_blocks) {
            part::map_clear(q.pa, (int)(blk - np - (uint32_t)q.wall_blocks), q.old);
            return;
        }
    }
    if (blk >= np) {
        near_walls<ST, OFF>(a, blk - np, (uint32_t)q.wall_blocks);
        return;
    }
    const double *sum = near_particle<ST, OFF, NT>(a, blk, part_lds);
    if (!kMany && q.mode == kPartsOne) {
        __syncthreads();  // part_lds is reused
        part::classify(q.pa, (int)blk, q.cur, q.next, part::box_rows(part_lds, q.pa.box_rows));
        part::map_clear(q.pa, (int)blk, q.old);
    } else if (DYN && (q.mode == kPartsDyn || q.mode == kPartsMove)) {
        __syncthreads();
        move_particle(q.pa, q.dyn, blk, sum, a.Xc + 3 * (size_t)blk);
        if (q.mode == kPartsMove) return;
        __syncthreads();  // X0 is read by every thread
        part::advance_set(q.pa, (int)blk, q.level, q.next, (int)threadIdx.x, (int)blockDim.x);
        part::map_clear(q.pa, (int)blk, q.old);
    }
}

template <typename ST, typename OFF, int NT>
__global__ void __launch_bounds__(NT, 4) k_parts(SweepArgs a, PartsArgs q) {
    const uint32_t blk = row_block();
    if (blk < q.blocks) parts_block<ST, OFF, true, NT>(a, q, blk);
}

// one workgroup per particle for several lattices in one dispatch
template <typename ST, int NT>
__global__ void __launch_bounds__(NT, 4) k_parts_packed(PackTable t) {
    const uint32_t gb = row_block();
    if (gb >= t.start[t.n]) return;
    const int e = pack_find(t, gb);
    const LatticeDev *d = t.d[e];
    const uint32_t st = t.state[e];
    const SweepArgs a = packed_args(&d->sweep[st]);
    const uint32_t c = st >> 1;
    PartsArgs q{};
    q.wall_blocks = load_uniform(&d->wall_blocks);
    q.pa = packed_args(&d->pa);
    const int split = load_uniform(&d->split);
    q.mode = !q.pa.moving || q.pa.np == 0 ? kPartsNear
             : NT == kManyThreads         ? kPartsClear
             : split                      ? kPartsSplit
                                          : kPartsOne;
    if (split) {
        q.pa.plist = as_global(load_uniform(&d->plist[st & 1u]));
        q.pa.pcount = as_global(load_uniform(&d->pcount[st & 1u]));
    }
    q.old = packed_args(&d->map[c == 0 ? 2 : c - 1]);
    q.cur = packed_args(&d->map[c]);
    q.next = packed_args(&d->map[c == 2 ? 0 : c + 1]);
    q.level = t.level[e];
    parts_block<ST, uint32_t, false, NT>(a, q, gb - t.start[e]);
}

// workgroups of the wall pass (0 without wall cells)
inline int near_wall_blocks(size_t N, bool walls, int threads) {
    if (!walls) return 0;
    size_t b = (N / 256 + 255) / 256;
    if (b > 1024) b = 1024;
    if (b < 1) b = 1;
    return (int)b * (kPartThreads / threads);
}

template <typename ST>
hipError_t launch_parts_packed_typed(const PackTable &t, int threads, uint32_t lds, hipStream_t s) {
    const uint32_t total = t.start[t.n];
    if (t.n == 0 || total == 0) return hipSuccess;
    if (threads == kPartThreads)
        hipLaunchKernelGGL((k_parts_packed<ST, kPartThreads>), row_grid(total), dim3(threads), lds, s, t);
    else
        hipLaunchKernelGGL((k_parts_packed<ST, kManyThreads>), row_grid(total), dim3(threads), lds, s, t);
    return hipGetLastError();
}

template <typename ST>
hipError_t launch_parts_typed(const SweepArgs &a, PartsArgs q, hipStream_t s) {
    q.blocks = parts_blocks(q.mode, a.np, q.wall_blocks);
    if (q.blocks == 0) return hipSuccess;
    const dim3 grid = row_grid(q.blocks);
    const int nt = q.pa.threads;
    const uint32_t lds = parts_lds(q.mode, q.pa.box_rows, nt);
    const bool small = 2 * a.g.Ns * sizeof(ST) < (size_t(1) << 32) && 4 * a.g.Ns < (size_t(1) << 32);
#define LBMEP_PARTS(OFF)                                                                          \
    do {                                                                                          \
        if (nt == kPartThreads)                                                                   \
            hipLaunchKernelGGL((k_parts<ST, OFF, kPartThreads>), grid, dim3(nt), lds, s, a, q);   \
        else                                                                                      \
            hipLaunchKernelGGL((k_parts<ST, OFF, kManyThreads>), grid, dim3(nt), lds, s, a, q);   \
    } while (0)
    if (small) LBMEP_PARTS(uint32_t);
    else LBMEP_PARTS(uint64_t);
#undef LBMEP_PARTS
    return hipGetLastError();
}

}  // namespace sweep
}  // namespace lbmep
