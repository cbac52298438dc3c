// sweep_impl.h -- fused gather-stream + collide sweep of the D3Q19 TRT lattice
// Boltzmann method with a body force and moving-obstacle bounce-back
// (arXiv:1708.08741, Sec. 3.1 Eq. LBMcollideStep / Eq. LBMstreamStep with
// Eq. LBE_forcetermLuo and Eq. modified_velocity; Sec. 3.2 Eq. LBMMovWall and
// Eq. LBMhydrodynForce).
//
// Pull scheme with post-collision storage.  The grid holds f*, the
// post-collision populations (with the forcing term) of the previous time
// level.  One thread per cell; a workgroup takes consecutive cells of the
// flat grid.  A thread gathers f*_q from x - e_q (reads shifted by at most
// one element along x; this completes the stream of Eq. LBMstreamStep),
// refills the cell if it has just been uncovered, collides, and writes its 19
// new values aligned to its own cell.
// Bounce-back needs no look-up at gather time: after the sweep, the kernel
// of near_impl.h writes the bounced value of every blocked link into a slot
// of the solid neighbour that the fluid cell gathers from at the next step.
// Only the edge of a non-periodic axis is resolved at gather time, from the
// cell coordinates.
//
// The template is instantiated in two translation units, k_stream_f64.hip
// (FP64) and k_stream_lp.hip (FP32 / FP16 deviation storage), both compiled
// without floating-point contraction: the FP64 sweep evaluates exactly the
// operation sequence of a plain CPU implementation; the FP32-compute sweep
// (FP32 and FP16 storage) uses the rearranged collision of collide_f32 with
// explicit FMAs; either way every sweep mode rounds identically.
// Byte offsets are 32-bit (global loads/stores with a scalar base) whenever a
// population array is smaller than 4 GiB.
#pragma once
#include "particles_impl.h"
#include "potential_impl.h"

namespace lbmep {
namespace sweep {

template <typename ST>
struct Storage;

// FP64: absolute populations
template <>
struct Storage<double> {
    using CT = double;
    static __device__ __forceinline__ double load(const double *p) { return *p; }
    static __device__ __forceinline__ void store(double *p, double v) { *p = v; }
    // streaming forms (non-temporal hint: each value is read or written once)
    static __device__ __forceinline__ double load_nt(const double *p) {
        return __builtin_nontemporal_load(p);
    }
    static __device__ __forceinline__ void store_nt(double *p, double v) {
        __builtin_nontemporal_store(v, p);
    }
    // deviation f - w_q of a computed population q, in FP64
    static __device__ __forceinline__ double devval(double v, int q) { return v - wq(q); }
    // f^eq(rho0 = 1, u) of population q (Eq. fequ_Incompr_SRT) as stored
    static __device__ __forceinline__ double feq(int q, double d) { return wq(q) * (1.0 + 1.0 * d); }
    // the sweep's compute units are the stored values themselves
    static __device__ __forceinline__ double lc(const double *p) { return load(p); }
    static __device__ __forceinline__ double lc_nt(const double *p) { return load_nt(p); }
    static __device__ __forceinline__ void sc(double *p, double v) { store(p, v); }
    static __device__ __forceinline__ void sc_nt(double *p, double v) { store_nt(p, v); }
    static __device__ __forceinline__ double feq_c(int q, double d) { return feq(q, d); }
};

// FP32: deviations f - w_q
template <>
struct Storage<float> {
    using CT = float;
    static __device__ __forceinline__ float load(const float *p) { return *p; }
    static __device__ __forceinline__ void store(float *p, float v) { *p = v; }
    static __device__ __forceinline__ float load_nt(const float *p) {
        return __builtin_nontemporal_load(p);
    }
    static __device__ __forceinline__ void store_nt(float *p, float v) {
        __builtin_nontemporal_store(v, p);
    }
    static __device__ __forceinline__ double devval(float v, int q) { return (double)v; }
    static __device__ __forceinline__ float feq(int q, double d) { return (float)(wq(q) * d); }
    // compute units: the deviations themselves
    static __device__ __forceinline__ float lc(const float *p) { return load(p); }
    static __device__ __forceinline__ float lc_nt(const float *p) { return load_nt(p); }
    static __device__ __forceinline__ void sc(float *p, float v) { store(p, v); }
    static __device__ __forceinline__ void sc_nt(float *p, float v) { store_nt(p, v); }
    static __device__ __forceinline__ float feq_c(int q, double d) { return feq(q, d); }
};

// FP16: deviations scaled by 2^22
template <>
struct Storage<__half> {
    using CT = float;
    static __device__ __forceinline__ float load(const __half *p) {
        return __half2float(*p) * kHalfInvScale;
    }
    static __device__ __forceinline__ void store(__half *p, float v) {
        *p = __float2half_rn(v * kHalfScale);
    }
    static __device__ __forceinline__ float load_nt(const __half *p) {
        const unsigned short b = __builtin_nontemporal_load(reinterpret_cast<const unsigned short *>(p));
        return __half2float(__ushort_as_half(b)) * kHalfInvScale;
    }
    static __device__ __forceinline__ void store_nt(__half *p, float v) {
        __builtin_nontemporal_store(__half_as_ushort(__float2half_rn(v * kHalfScale)),
                                    reinterpret_cast<unsigned short *>(p));
    }
    static __device__ __forceinline__ double devval(float v, int q) { return (double)v; }
    // rounded to the storage format, as a stored and re-loaded value would be
    static __device__ __forceinline__ float feq(int q, double d) {
        return __half2float(__float2half_rn((float)(wq(q) * d) * kHalfScale)) * kHalfInvScale;
    }
    // compute units: deviations times 2^22, the stored half values widened
    // (loads and stores convert only; the power-of-two scale is exact)
    static __device__ __forceinline__ float lc(const __half *p) { return __half2float(*p); }
    static __device__ __forceinline__ float lc_nt(const __half *p) {
        const unsigned short b = __builtin_nontemporal_load(reinterpret_cast<const unsigned short *>(p));
        return __half2float(__ushort_as_half(b));
    }
    static __device__ __forceinline__ void sc(__half *p, float v) { *p = __float2half_rn(v); }
    static __device__ __forceinline__ void sc_nt(__half *p, float v) {
        __builtin_nontemporal_store(__half_as_ushort(__float2half_rn(v)),
                                    reinterpret_cast<unsigned short *>(p));
    }
    static __device__ __forceinline__ float feq_c(int q, double d) {
        return __half2float(__float2half_rn((float)(wq(q) * d) * kHalfScale));
    }
};

// a . c_q for a lattice direction, with the zero terms of
// ((c_x a_x + c_y a_y) + c_z a_z) dropped (same value, same rounding)
template <int q, typename T>
__device__ __forceinline__ T cdot(T ax, T ay, T az) {
    constexpr int a = kCx[q], b = kCy[q], c = kCz[q];
    T r = T(0);
    if constexpr (a != 0 && b != 0) {
        r = (a > 0 ? ax : -ax) + (b > 0 ? ay : -ay);
    } else if constexpr (a != 0) {
        r = (a > 0 ? ax : -ax);
    } else if constexpr (b != 0) {
        r = (b > 0 ? ay : -ay);
    }
    if constexpr (c != 0) {
        if constexpr (a != 0 || b != 0)
            r = r + (c > 0 ? az : -az);
        else
            r = (c > 0 ? az : -az);
    }
    return r;
}

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

// nearest periodic image of the half-integer cell coordinate c to X (exact)
__device__ __forceinline__ double image_coord(double c, double X, int len, int periodic) {
    if (periodic) {
        const double d = c - X, h = 0.5 * (double)len;
        if (d > h)
            c -= (double)len;
        else if (d < -h)
            c += (double)len;
    }
    return c;
}

// address of element `off` (bytes) of the array starting at the uniform
// `base`; with OFF = uint32_t this becomes a global access with a scalar base
// register and a 32-bit vector offset
template <typename ST, typename OFF>
__device__ __forceinline__ ST *at(void *base, OFF off) {
    return reinterpret_cast<ST *>(static_cast<char *>(base) + off);
}
template <typename ST, typename OFF>
__device__ __forceinline__ const ST *at(const void *base, OFF off) {
    return reinterpret_cast<const ST *>(static_cast<const char *>(base) + off);
}

// sweep modes
enum { kPull = 0,     // gather f* of the previous level, refill, collide
       kLocal = 1,    // collide the post-stream state held in the grid
       kReadout = 2,  // gather and refill only: write the post-stream state
       kPullNT = 3,   // as kPull, loads and stores with streaming hints
       kPullNTS = 4   // as kPull, stores with streaming hints
};

// load / store of one stored population in compute units, with the
// streaming hint in kPullNT
template <int MODE, typename ST>
__device__ __forceinline__ typename Storage<ST>::CT pop_load(const ST *p) {
    if constexpr (MODE == kPullNT)
        return Storage<ST>::lc_nt(p);
    else
        return Storage<ST>::lc(p);
}
template <int MODE, typename ST>
__device__ __forceinline__ void pop_store(ST *p, typename Storage<ST>::CT v) {
    if constexpr (MODE == kPullNT || MODE == kPullNTS)
        Storage<ST>::sc_nt(p, v);
    else
        Storage<ST>::sc(p, v);
}

// the TRT collision of one opposite pair (q, q+1) with the forcing term
template <int q, typename CT>
__device__ __forceinline__ void collide_pair(CT (&v)[Q], CT rho, CT ux, CT uy, CT uz, CT uu,
                                             CT ufb, CT fb0, CT fb1, CT fb2, CT le, CT lo, CT ae,
                                             CT ao, bool forced) {
    constexpr int qb = q + 1;
    const CT w = (CT)wq(q);
    const CT cu = cdot<q>(ux, uy, uz);
    // equilibrium halves (Eq. EqPDF_TRT), rho0 = 1, 1/c_s^2 = 3, 1/c_s^4 = 9
    const CT feq_e = w * ((rho - uu * CT(1.5)) + (cu * cu) * CT(4.5));
    const CT feq_o = w * (CT(3.0) * cu);
    const CT fe = CT(0.5) * (v[q] + v[qb]);
    const CT fo = CT(0.5) * (v[q] - v[qb]);
    const CT A = le * (fe - feq_e);
    const CT B = lo * (fo - feq_o);
    CT fq = (v[q] + A) + B;
    CT fqb = (v[qb] + A) - B;
    if (forced) {
        // Luo term split into even / odd parts, weighted (1 + lambda/2)
        const CT cf = cdot<q>(fb0, fb1, fb2);
        const CT Fe = w * ((-ufb * CT(3.0)) + (cu * cf) * CT(9.0));
        const CT Fo = w * (cf * CT(3.0));
        fq = (fq + ae * Fe) + ao * Fo;
        fqb = (fqb + ae * Fe) - ao * Fo;
    }
    v[q] = fq;
    v[qb] = fqb;
}

// FP32 compute (FP32 and FP16 storage): the TRT collision with the Luo
// forcing term (Eq. LBMcollideStep with Eq. EqPDF_TRT, Eq. LBE_forcetermLuo
// and Eq. modified_velocity) rearranged to fewer operations.  With the pair
// sum s = f_q + f_qbar and difference d = f_q - f_qbar, the update of an
// opposite pair is f_q <- f_q + (E + O), f_qbar <- f_qbar + (E - O) with
//   E = le/2 s - G_k - (c.u)(9/2 le w (c.u) - 9 ae w (c.F))
//   O = le/2 d - 3 lo w (c.u) + 3 ao w (c.F)
//     = lo/6 (3 d - c.u) + ao/6 (c.F)      (axis, w = 1/18)
//     = lo/12 (6 d - c.u) + ao/12 (c.F)    (diagonal, w = 1/36)
// and G_k = le w (rho - 3/2 u.u) + 3 ae w u.F per weight class; the rest
// population becomes f_0 + (le f_0 - G_0).  The increments are added to the
// loaded values (the unit part of the update stays exact), and in the odd
// part d and c.u enter with exact integer weights, so the momentum the
// collision changes, lo (j - u) + ao F, has no bias from the rounding of the
// rates.  Algebraically the textbook form; the rounding differs (FMA,
// regrouped sums).  rho and j = sum c f come from the same pair sums and
// differences.  Values are in compute units (see TrtF32).
template <int q, bool FORCED>
__device__ __forceinline__ void trt_pair_f32(float (&v)[Q], const TrtF32 &t, float s, float d,
                                             float ux, float uy, float uz, float fx, float fy,
                                             float fz, float G) {
    constexpr int qb = q + 1;
    constexpr int k = q <= 6 ? 0 : 1;  // weight class: axis / diagonal
    const float cu = cdot<q>(ux, uy, uz);
    const float D = __builtin_fmaf(k == 0 ? 3.0f : 6.0f, d, -cu);
    float E, O;
    if constexpr (FORCED) {
        const float cf = cdot<q>(fx, fy, fz);
        const float h = __builtin_fmaf(t.k1[k], cu, -(t.k3[k] * cf));
        E = __builtin_fmaf(t.hle, s, -__builtin_fmaf(cu, h, G));
        O = __builtin_fmaf(t.hlo[k], D, t.k4[k] * cf);
    } else {
        E = __builtin_fmaf(t.hle, s, -__builtin_fmaf(cu, t.k1[k] * cu, G));
        O = t.hlo[k] * D;
    }
    v[q] = v[q] + (E + O);
    v[qb] = v[qb] + (E - O);
}

template <bool FORCED>
__device__ __forceinline__ void collide_f32(float (&v)[Q], const TrtF32 &t, float fx, float fy,
                                            float fz) {
    // directions 2p+1, 2p+2 are opposite; the first of each pair points
    // along +x for p = 0, 3, 4, 5, 6, along +y for p = 1, 3, 7, 8 and -y for
    // p = 4, along +z for p = 2, 5, 7 and -z for p = 6, 8
    static_assert(kCx[1] == 1 && kCx[7] == 1 && kCx[9] == 1 && kCx[11] == 1 && kCx[13] == 1 &&
                  kCx[3] == 0 && kCx[5] == 0 && kCx[15] == 0 && kCx[17] == 0, "x layout");
    static_assert(kCy[3] == 1 && kCy[7] == 1 && kCy[9] == -1 && kCy[15] == 1 && kCy[17] == 1 &&
                  kCy[1] == 0 && kCy[5] == 0 && kCy[11] == 0 && kCy[13] == 0, "y layout");
    static_assert(kCz[5] == 1 && kCz[11] == 1 && kCz[13] == -1 && kCz[15] == 1 && kCz[17] == -1 &&
                  kCz[1] == 0 && kCz[3] == 0 && kCz[7] == 0 && kCz[9] == 0, "z layout");
    static_assert(opp(1) == 2 && opp(7) == 8 && opp(17) == 18, "pairs");
    float s[9], d[9];
#pragma unroll
    for (int p = 0; p < 9; ++p) {
        s[p] = v[2 * p + 1] + v[2 * p + 2];
        d[p] = v[2 * p + 1] - v[2 * p + 2];
    }
    float rho = v[0];
#pragma unroll
    for (int p = 0; p < 9; ++p) rho += s[p];
    const float jx = (((d[0] + d[3]) + d[4]) + d[5]) + d[6];
    const float jy = (((d[1] + d[3]) - d[4]) + d[7]) + d[8];
    const float jz = (((d[2] + d[5]) - d[6]) + d[7]) - d[8];
    // Eq. modified_velocity: u = j + F/2 (rho0 = 1)
    const float ux = FORCED ? __builtin_fmaf(0.5f, fx, jx) : jx;
    const float uy = FORCED ? __builtin_fmaf(0.5f, fy, jy) : jy;
    const float uz = FORCED ? __builtin_fmaf(0.5f, fz, jz) : jz;
    const float uu = __builtin_fmaf(ux, ux, __builtin_fmaf(uy, uy, uz * uz));
    const float base = __builtin_fmaf(-t.b15, uu, rho);
    float G0, G1, G2;
    if constexpr (FORCED) {
        const float ufb = __builtin_fmaf(ux, fx, __builtin_fmaf(uy, fy, uz * fz));
        G0 = __builtin_fmaf(t.m0, ufb, t.lw0 * base);
        G1 = __builtin_fmaf(t.m[0], ufb, t.lw[0] * base);
        G2 = __builtin_fmaf(t.m[1], ufb, t.lw[1] * base);
    } else {
        G0 = t.lw0 * base;
        G1 = t.lw[0] * base;
        G2 = t.lw[1] * base;
    }
    v[0] = v[0] + __builtin_fmaf(t.le, v[0], -G0);
    trt_pair_f32<1, FORCED>(v, t, s[0], d[0], ux, uy, uz, fx, fy, fz, G1);
    trt_pair_f32<3, FORCED>(v, t, s[1], d[1], ux, uy, uz, fx, fy, fz, G1);
    trt_pair_f32<5, FORCED>(v, t, s[2], d[2], ux, uy, uz, fx, fy, fz, G1);
    trt_pair_f32<7, FORCED>(v, t, s[3], d[3], ux, uy, uz, fx, fy, fz, G2);
    trt_pair_f32<9, FORCED>(v, t, s[4], d[4], ux, uy, uz, fx, fy, fz, G2);
    trt_pair_f32<11, FORCED>(v, t, s[5], d[5], ux, uy, uz, fx, fy, fz, G2);
    trt_pair_f32<13, FORCED>(v, t, s[6], d[6], ux, uy, uz, fx, fy, fz, G2);
    trt_pair_f32<15, FORCED>(v, t, s[7], d[7], ux, uy, uz, fx, fy, fz, G2);
    trt_pair_f32<17, FORCED>(v, t, s[8], d[8], ux, uy, uz, fx, fy, fz, G2);
}

#define LBMEP_FOR_Q18(M) \
    M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15) M(16) M(17) M(18)

// where a cell's populations come from: byte offsets of the source cells
// x - e and whether they lie inside the grid (periodic axes wrapped), as the
// cell's own offset plus a step per axis (index e + 1)
template <typename OFF>
struct Sources {
    OFF cb, d[3][3];
    bool in[3][3];
    __device__ __forceinline__ Sources(const Grid &g, int x, int y, int z, OFF ci, OFF es) {
        cb = ci * es;
        const OFF str[3] = {es, (OFF)g.nx * es, (OFF)g.nx * (OFF)g.ny * es};
        const int pos[3] = {x, y, z}, len[3] = {g.nx, g.ny, g.nz};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const OFF wrap = str[a] * (OFF)(len[a] - 1);
            const bool first = pos[a] == 0, last = pos[a] == len[a] - 1;
            d[a][0] = last ? (OFF)0 - wrap : str[a];
            d[a][1] = 0;
            d[a][2] = first ? wrap : (OFF)0 - str[a];
            in[a][0] = !last || g.per[a];
            in[a][1] = true;
            in[a][2] = !first || g.per[a];
        }
    }
    __device__ __forceinline__ OFF at(int cx, int cy, int cz) const {
        return cb + d[0][cx + 1] + d[1][cy + 1] + d[2][cz + 1];
    }
    __device__ __forceinline__ bool ok(int cx, int cy, int cz) const {
        return in[0][cx + 1] && in[1][cy + 1] && in[2][cz + 1];
    }
};

// gather population q of the cell from x - e_q; beyond the edge of a
// non-periodic axis the population bounces at the (resting) edge: it is the
// cell's own opposite population
template <int q, typename ST, typename OFF, int MODE>
__device__ __forceinline__ typename Storage<ST>::CT gather(const void *src, OFF pst, OFF cb,
                                                           const Sources<OFF> &n) {
    constexpr int qb = opp(q);
    constexpr int lo = q < qb ? q : qb;
    const void *base = static_cast<const char *>(src) + (size_t)lo * pst;
    const OFF nb = (OFF)(q - lo) * pst + n.at(kCx[q], kCy[q], kCz[q]);
    const OFF own = (OFF)(qb - lo) * pst + cb;
    return pop_load<MODE, ST>(at<ST>(base, n.ok(kCx[q], kCy[q], kCz[q]) ? nb : own));
}

// Free-slip faces: a population that a face cell x gathers from beyond a
// free-slip face (direction q, source x - c_q outside along axis a) comes from
// the tangential neighbour s' (x - c_q with that component set back to x's) in
// the direction p = q mirrored across the face, unless s' was a wall or
// obstacle cell when the populations streamed (then the half-way bounce-back
// stands): the map of the level before decides, not that of the level they are
// gathered for, at which a sphere cut by the face may have moved on.  Along
// the normal, and
// where a diagonal crosses two faces at an edge, the reflection is the
// bounce-back that the gather has already taken.  So each face has four
// directions to take again, on the lanes at it: their slots lie in lines that
// the wavefront's gather reads anyway.  (A pass that swapped the slots of the
// pairs of such populations before every gather took 39 us beside a sweep of
// 375 us at 216 x 312 x 216 FP32, most of it on the x faces, a line per cell;
// 20 steps and a read-out there 9.72 -> 9.30 ms.)
template <int q, int ax, typename ST, typename OFF, int MODE>
__device__ __forceinline__ void slip_direction(const SweepArgs &a, const Sources<OFF> &n,
                                               typename Storage<ST>::CT &v) {
    constexpr int c[3] = {kCx[q], kCy[q], kCz[q]};
    constexpr int b = ax == 0 ? (c[1] != 0 ? 1 : 2) : ax == 1 ? (c[0] != 0 ? 0 : 2) : (c[0] != 0 ? 0 : 1);
    static_assert(c[ax] != 0 && c[b] != 0, "a diagonal");
    constexpr int p = mirror_dir(q, 1 << ax);
    if (!n.in[b][c[b] + 1]) return;  // an edge of two faces
    const OFF o = n.cb + n.d[b][c[b] + 1];
    const char *base = static_cast<const char *>(a.src) + (size_t)p * a.g.Ns * sizeof(ST);
    const uint8_t fs = a.flag[o / (OFF)sizeof(ST)];
    const typename Storage<ST>::CT t = pop_load<MODE, ST>(at<ST>(static_cast<const void *>(base), o));
    // kUncov: an obstacle cell of the level before; kObst: of this level, and of
    // that one if it had an owner there (a fixed map is both levels' map)
    bool fluid = !(fs & (kWall | kUncov));
    if (fluid && (fs & kObst)) fluid = a.owner_old[o / (OFF)sizeof(ST)] == kNone;
    if (fluid) v = t;
}

template <typename ST, typename OFF, int MODE>
__device__ __forceinline__ void slip_faces(const SweepArgs &a, const Sources<OFF> &n,
                                           typename Storage<ST>::CT (&v)[Q]) {
    // directions that come from beyond the low face of an axis have a
    // positive component along it, those from beyond the high face a negative
#define LBMEP_FACE(ax, side, q0, q1, q2, q3)                                       \
    if ((a.slip & (1 << (2 * ax + side))) && !n.in[ax][side ? 0 : 2]) {            \
        slip_direction<q0, ax, ST, OFF, MODE>(a, n, v[q0]);                        \
        slip_direction<q1, ax, ST, OFF, MODE>(a, n, v[q1]);                        \
        slip_direction<q2, ax, ST, OFF, MODE>(a, n, v[q2]);                        \
        slip_direction<q3, ax, ST, OFF, MODE>(a, n, v[q3]);                        \
    }
    LBMEP_FACE(0, 0, 7, 9, 11, 13)
    LBMEP_FACE(0, 1, 8, 10, 12, 14)
    LBMEP_FACE(1, 0, 7, 10, 15, 17)
    LBMEP_FACE(1, 1, 8, 9, 16, 18)
    LBMEP_FACE(2, 0, 11, 14, 15, 18)
    LBMEP_FACE(2, 1, 12, 13, 16, 17)
#undef LBMEP_FACE
    static_assert(kCx[7] == 1 && kCx[9] == 1 && kCx[11] == 1 && kCx[13] == 1, "low x face");
    static_assert(kCx[8] == -1 && kCx[10] == -1 && kCx[12] == -1 && kCx[14] == -1, "high x face");
    static_assert(kCy[7] == 1 && kCy[10] == 1 && kCy[15] == 1 && kCy[17] == 1, "low y face");
    static_assert(kCy[8] == -1 && kCy[9] == -1 && kCy[16] == -1 && kCy[18] == -1, "high y face");
    static_assert(kCz[11] == 1 && kCz[14] == 1 && kCz[15] == 1 && kCz[18] == 1, "low z face");
    static_assert(kCz[12] == -1 && kCz[13] == -1 && kCz[16] == -1 && kCz[17] == -1, "high z face");
}

// store population q of a cell at byte offset cb; addressed from the base of
// its opposite pair like the gather (a uniform base plus a 32-bit offset)
template <int q, int MODE, typename ST, typename OFF>
__device__ __forceinline__ void store_pop(void *dst, OFF pst, OFF cb, typename Storage<ST>::CT v) {
    constexpr int lo = q == 0 ? 0 : (q < opp(q) ? q : opp(q));
    char *base = static_cast<char *>(dst) + (size_t)lo * pst;
    pop_store<MODE, ST>(at<ST>(base, (OFF)(q - lo) * pst + cb), v);
}

// loaded inputs of one cell
template <typename CT, typename OFF>
struct CellIn {
    CT v[Q];
    CT fb0, fb1, fb2;
    OFF ci;      // cell index (in range also where not valid)
    bool valid;  // a cell of the grid
    uint8_t fl;
};

// issue every load of cell (x, y, z) (solid cells and cells beyond the grid
// load in-range values and drop them), so that the flag and the populations
// share one memory latency
template <typename ST, int FMODE, typename OFF, int MODE>
__device__ __forceinline__ void load_cell(const SweepArgs &a, int x, int y, int z, OFF ci,
                                          bool valid, CellIn<typename Storage<ST>::CT, OFF> &c) {
    using T = Storage<ST>;
    using CT = typename T::CT;
    const OFF es = (OFF)sizeof(ST);
    const OFF pst = (OFF)a.g.Ns * es;
    const OFF cb = ci * es;
    c.ci = ci;
    c.valid = valid;
    const uint8_t *flp = at<uint8_t>((const void *)a.flag, ci);
    uint8_t fl;
    if constexpr (MODE == kPullNT)
        fl = __builtin_nontemporal_load(flp);
    else
        fl = *flp;
    c.fl = valid ? fl : kWall;
    const Sources<OFF> n(a.g, x, y, z, ci, es);  // pull modes
    if constexpr (MODE == kLocal) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            c.v[q] = T::lc(at<ST>(static_cast<const char *>(a.src) + (size_t)q * pst, cb));
    } else {
        c.v[0] = pop_load<MODE, ST>(at<ST>(a.src, cb));
#define LBMEP_GATHER(q) c.v[q] = gather<q, ST, OFF, MODE>(a.src, pst, cb, n);
        LBMEP_FOR_Q18(LBMEP_GATHER)
#undef LBMEP_GATHER
        if (a.slip && valid && !(fl & (kWall | kObst))) slip_faces<ST, OFF, MODE>(a, n, c.v);
    }
    c.fb0 = c.fb1 = c.fb2 = CT(0);
    if constexpr (MODE != kReadout) {
        if constexpr (FMODE == kForceDense) {
            const OFF fo = ci * (OFF)sizeof(CT), fs = (OFF)a.g.Ns * (OFF)sizeof(CT);
            c.fb0 = *at<CT>(a.force, fo);
            c.fb1 = *at<CT>(a.force, fo + fs);
            c.fb2 = *at<CT>(a.force, fo + 2 * fs);
        } else if constexpr (FMODE == kForcePotential) {
            // colour-split psi (even nx) with even extents along the
            // periodic y and z axes, so a neighbour across a wrap keeps the
            // colour parity of its unwrapped place
            const bool split_even = psi_split(a.g) && (!a.g.per[1] || a.g.ny % 2 == 0) &&
                                    (!a.g.per[2] || a.g.nz % 2 == 0);
            if (MODE != kLocal && split_even && valid && !(fl & (kWall | kObst | kNear))) {
                // every neighbour a fluid cell inside the grid: the
                // stencil's slots from the gather's source cells (cell c' is
                // entry c' / 2, nx being even, the colour-1 half at Ns / 2);
                // the colour of the neighbour (x, y, z) + (dx, dy, dz) is the
                // cell's own xor the parity of dx + dy + dz
                const OFF half = (OFF)(a.g.Ns >> 1) * (OFF)sizeof(CT);
                const OFF cs = (OFF)(((x + y + z) & 1) ? half : 0), co = half - cs;
                auto val = [&](int dx, int dy, int dz) -> CT {
                    const OFF ob = n.at(-dx, -dy, -dz) / (2 * es) * (OFF)sizeof(CT) +
                                   (((dx + dy + dz) & 1) ? co : cs);
                    return *at<CT>(a.force, ob);
                };
                CT pc, g0, g1, g2;
                psi_grad_inner<CT>(val, pc, g0, g1, g2);
                edl_force<CT>(pc, g0, g1, g2, (CT)a.keps, (CT)a.E[0], (CT)a.E[1], (CT)a.E[2],
                              c.fb0, c.fb1, c.fb2);
            } else if (valid && !(fl & (kWall | kObst))) {
                potential_force<CT>(a.g, x, y, z, fl, static_cast<const CT *>(a.force), a.flag,
                                    a.owner, a.zeta, (CT)a.keps, (CT)a.E[0], (CT)a.E[1],
                                    (CT)a.E[2], c.fb0, c.fb1, c.fb2);
            }
        } else if constexpr (FMODE == kForceCharge) {
            const CT *rp = at<CT>(a.force, ci * (OFF)sizeof(CT));
            CT re;
            if constexpr (MODE == kPullNT)
                re = __builtin_nontemporal_load(rp);
            else
                re = *rp;
            if constexpr (sizeof(CT) == 4) {
                // the field in compute units (exact power-of-two scale)
                c.fb0 = re * a.tf.Ec[0];
                c.fb1 = re * a.tf.Ec[1];
                c.fb2 = re * a.tf.Ec[2];
            } else {
                c.fb0 = re * (CT)a.E[0];
                c.fb1 = re * (CT)a.E[1];
                c.fb2 = re * (CT)a.E[2];
            }
        }
        if constexpr (sizeof(ST) == 2 && (FMODE == kForceDense || FMODE == kForcePotential)) {
            c.fb0 *= a.tf.fscale;
            c.fb1 *= a.tf.fscale;
            c.fb2 *= a.tf.fscale;
        }
    }
}

// surface velocity u_s of particle p, centred at X, at cell (x, y, z)
__device__ __forceinline__ void surface_velocity(const SweepArgs &a, const double *X, uint32_t p,
                                                 int x, int y, int z, double (&u)[3]) {
    const double *Xp = X + 3 * (size_t)p;
    const double *U = a.U + 3 * (size_t)p;
    const double *W = a.W + 3 * (size_t)p;
    const double r0 = min_image(((double)x + 0.5) - Xp[0], a.g.nx, a.g.per[0]);
    const double r1 = min_image(((double)y + 0.5) - Xp[1], a.g.ny, a.g.per[1]);
    const double r2 = min_image(((double)z + 0.5) - Xp[2], a.g.nz, a.g.per[2]);
    u[0] = U[0] + (W[1] * r2 - W[2] * r1);
    u[1] = U[1] + (W[2] * r0 - W[0] * r2);
    u[2] = U[2] + (W[0] * r1 - W[1] * r0);
}

// f^eq(rho0, u) as stored, in compute units
template <typename ST>
__device__ __forceinline__ void equilibrium(const double (&u)[3], typename Storage<ST>::CT (&v)[Q]) {
    using T = Storage<ST>;
    const double uu = (u[0] * u[0] + u[1] * u[1]) + u[2] * u[2];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const double cu = ((double)kCx[q] * u[0] + (double)kCy[q] * u[1]) + (double)kCz[q] * u[2];
        v[q] = (typename T::CT)T::feq_c(q, (cu * 3.0 + (cu * cu) * 4.5) - uu * 1.5);
    }
}

// refill of a cell uncovered at this level: f^eq(rho0, u_s) with the surface
// velocity of its previous owner at its previous place (Sec. 3.2)
template <typename ST, typename OFF>
__device__ __forceinline__ void refill(const SweepArgs &a, int x, int y, int z,
                                       CellIn<typename Storage<ST>::CT, OFF> &c) {
    if ((c.fl & kUncov) && !(c.fl & (kWall | kObst))) {
        double u[3];
        surface_velocity(a, a.Xold, a.owner_old[c.ci], x, y, z, u);
        equilibrium<ST>(u, c.v);
    }
}

// refill (if uncovered), collide and store one loaded cell
template <typename ST, int FMODE, typename OFF, int MODE>
__device__ __forceinline__ void finish_cell(const SweepArgs &a, int x, int y, int z,
                                            CellIn<typename Storage<ST>::CT, OFF> &c) {
    using T = Storage<ST>;
    using CT = typename T::CT;
    const OFF es = (OFF)sizeof(ST);
    const OFF pst = (OFF)a.g.Ns * es;
    const bool act = !(c.fl & (kWall | kObst));  // not so beyond the grid
    const OFF ci = c.ci;
    const OFF cb = ci * es;
    CT(&v)[Q] = c.v;

    if constexpr (MODE != kLocal) refill<ST, OFF>(a, x, y, z, c);

    if constexpr (MODE == kReadout) {
        // solid cells get defined values: the rest state at walls and
        // f^eq(rho0, u_s) of the owning particle at obstacle cells
        if (!act && c.valid) {
            double u[3] = {0.0, 0.0, 0.0};
            if (!(c.fl & kWall)) surface_velocity(a, a.Xc, a.owner[ci], x, y, z, u);
            equilibrium<ST>(u, v);
        }
        if (c.valid) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
                T::sc(at<ST>(static_cast<char *>(a.dst) + (size_t)q * pst, cb), v[q]);
        }
    } else {
        // the collision runs on every lane
        if constexpr (sizeof(CT) == 4) {
            collide_f32<FMODE != kForceNone>(v, a.tf, c.fb0, c.fb1, c.fb2);
        } else {
        const CT fb0 = c.fb0, fb1 = c.fb1, fb2 = c.fb2;

        // moments (Eq. MacroscopVel), in q order
        CT rho = CT(0), jx = CT(0), jy = CT(0), jz = CT(0);
#pragma unroll
        for (int q = 0; q < Q; ++q) rho += v[q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (kCx[q] > 0) jx += v[q];
            if (kCx[q] < 0) jx -= v[q];
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (kCy[q] > 0) jy += v[q];
            if (kCy[q] < 0) jy -= v[q];
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (kCz[q] > 0) jz += v[q];
            if (kCz[q] < 0) jz -= v[q];
        }
        // Eq. modified_velocity: u = (sum c f + f_b / 2) / rho0
        const bool forced = FMODE != kForceNone;
        const CT ux = forced ? jx + CT(0.5) * fb0 : jx;
        const CT uy = forced ? jy + CT(0.5) * fb1 : jy;
        const CT uz = forced ? jz + CT(0.5) * fb2 : jz;
        const CT uu = (ux * ux + uy * uy) + uz * uz;
        const CT ufb = forced ? (ux * fb0 + uy * fb1) + uz * fb2 : CT(0);
        const CT le = (CT)a.le, lo = (CT)a.lo, ae = (CT)a.ae, ao = (CT)a.ao;

        // rest population
        {
            const CT w0 = (CT)wq(0);
            const CT feq_e = w0 * (rho - uu * CT(1.5));
            CT f0 = v[0] + le * (v[0] - feq_e);
            if (forced) f0 = f0 + ae * (w0 * (-ufb * CT(3.0)));
            v[0] = f0;
        }
        collide_pair<1>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        collide_pair<3>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        collide_pair<5>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        collide_pair<7>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        collide_pair<9>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        collide_pair<11>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        collide_pair<13>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        collide_pair<15>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        collide_pair<17>(v, rho, ux, uy, uz, uu, ufb, fb0, fb1, fb2, le, lo, ae, ao, forced);
        }

        // Aligned store of the post-collision state, also to the obstacle
        // cells beside fluid ones: the next gather reads there only the slots
        // that the exchange writes after the sweep, and whole lines cost less than
        // lines with holes (4096 spheres of radius 4, with the holes and
        // without: 512^3 FP32 3730 -> 3500 us, 512 x 384 x 320 FP16 1083 ->
        // 1001, 300 x 256^2 FP64 1230 -> 1126).  The slots of wall cells,
        // which a fixed list keeps up, stay untouched.
        if (__any(act) && c.valid && !(c.fl & kWall)) {
#define LBMEP_STORE(q) store_pop<q, MODE, ST, OFF>(a.dst, pst, cb, v[q]);
            LBMEP_STORE(0)
            LBMEP_FOR_Q18(LBMEP_STORE)
#undef LBMEP_STORE
        }
    }
}


// t / n for t < n + 2^11 (a segment or less past the axis), m = 2^31 / n + 1
// or one more: a single subtraction from n = 2^11 on, and below that the
// product's error, at most 2 t / 2^31 of a quotient step of 1 / n, is too small
__device__ __forceinline__ uint32_t quot(uint32_t t, int n, uint32_t m) {
    return n >= 2048 ? (uint32_t)(t >= (uint32_t)n) : __umulhi(2u * t, m);
}

// this lane's cell of segment lb; beyond the grid: not valid, cell 0
template <typename OFF>
struct Place {
    int x, y, z;
    OFF ci;
    bool valid;
    __device__ __forceinline__ Place(const SweepArgs &a, uint32_t lb) {
        const int nx = a.g.nx, ny = a.g.ny;
        // the segment's first cell in scalar registers: quotients by
        // multiplication with 2^63 / n + 1, exact while cell times extent is
        // below 2^63
        const OFF c0 = (OFF)lb * blockDim.x;
        const uint64_t row = __umul64hi(2u * (uint64_t)c0, a.mx);
        const uint64_t plane = __umul64hi(2u * row, a.my);
        const uint32_t x0 = (uint32_t)((uint64_t)c0 - row * (uint64_t)(uint32_t)nx);
        const uint32_t y0 = (uint32_t)(row - plane * (uint64_t)(uint32_t)ny);
        // this lane's, from there
        const uint32_t t = x0 + threadIdx.x;
        const uint32_t dy = quot(t, nx, (uint32_t)(a.mx >> 32) + 1u);
        const uint32_t ty = y0 + dy;
        const uint32_t dz = quot(ty, ny, (uint32_t)(a.my >> 32) + 1u);
        valid = (size_t)c0 + threadIdx.x < a.g.N;
        x = valid ? (int)(t - dy * (uint32_t)nx) : 0;
        y = valid ? (int)(ty - dz * (uint32_t)ny) : 0;
        z = valid ? (int)((uint32_t)plane + dz) : 0;
        ci = valid ? c0 + threadIdx.x : (OFF)0;
    }
};

// One workgroup's blockDim.x consecutive cells of the flat grid.  A sweep is
// bound by its memory traffic; with the cells dealt out across rows every
// lane has a cell and every store covers whole aligned lines, whatever nx is.
// (Segments of single rows, with y and z in scalar registers, left lanes idle
// at the rows' ends and split lines between workgroups.  Step of a lattice
// with a charge force, row segments and now, FP64 / FP32 / FP16:
//   101 x 67 x 83    39.7 -> 35.2   23.3 -> 18.7   16.5 -> 12.0 us
//   300 x 333 x 250  1722 -> 1411   1218 ->  696    690 ->  392 us
//   512^3            7614 -> 7068   3648 -> 3589   1883 -> 1818 us.)
template <typename ST, int FMODE, typename OFF, int MODE>
__device__ __forceinline__ void sweep_segment(const SweepArgs &a, uint32_t lb) {
    const Place<OFF> c(a, lb);
    CellIn<typename Storage<ST>::CT, OFF> in;
    load_cell<ST, FMODE, OFF, MODE>(a, c.x, c.y, c.z, c.ci, c.valid, in);
    finish_cell<ST, FMODE, OFF, MODE>(a, c.x, c.y, c.z, in);
}

// workgroup b of the next level's mapping: a particle per kMapThreads threads
// (the rows of a ball of radius 4 are 11^2; fewer workgroups with several
// particles take fewer of the sweep's places)
__device__ __forceinline__ void map_particles(const ParticleArgs &pa, uint32_t b, int64_t level,
                                              const LevelMap &m) {
    const uint32_t p = b * (blockDim.x / kMapThreads) + threadIdx.x / kMapThreads;
    if (p < (uint32_t)pa.np)
        part::advance_set(pa, (int)p, level, m, (int)(threadIdx.x % kMapThreads), kMapThreads);
}

// nseg segments; with ms.groups, the next level's mapping runs in the same
// launch: its workgroups come in groups of eight (so that a segment stays on
// its XCD) spread evenly among the sweep's, which hides their few dependent
// round trips behind the streaming (a launch of its own took 10 us at 128^3
// and 36-85 us at 512^3 with 4096 particles)
template <typename ST, int FMODE, typename OFF, int MODE>
__global__ void __launch_bounds__(512) k_sweep(SweepArgs a, MapSetArgs ms, uint32_t nseg) {
    uint32_t b = blockIdx.x;
    if (ms.groups) {
        const uint32_t g = b >> 3, m = g / ms.stride;
        if (g - m * ms.stride == 0 && m < ms.groups) {
            map_particles(ms.pa, 8u * m + (b & 7u), ms.level, ms.next);
            return;
        }
        b -= 8u * min(ms.groups, (g + ms.stride - 1u) / ms.stride);
        if (b >= nseg) return;
    }
    sweep_segment<ST, FMODE, OFF, MODE>(a, a.xcd_swizzle ? xcd_remap(b, nseg) : b);
}

// Density and velocity (Eq. MacroscopVel with the velocity of
// Eq. modified_velocity) as FP64 fields.  MODE kReadout gathers the
// populations from the post-collision state, as the next sweep will, and
// leaves that state as it is: one pass over the populations, bound by it (512^3
// FP32: 2.68 ms for 15.2 GB; 20 steps with 4096 spheres and a read-out took
// 86.3 ms with a gather into the spare grid, read again here and collided in
// place by the next step, and take 81.9 ms); kLocal reads the post-stream
// state in the grid.
template <typename ST, typename OFF, int MODE>
__global__ void __launch_bounds__(256) k_macro(SweepArgs a, int force_mode, double *rho, double *u) {
    using CT = typename Storage<ST>::CT;
    const Place<OFF> p(a, blockIdx.x);
    CellIn<CT, OFF> c;
    load_cell<ST, kForceNone, OFF, MODE>(a, p.x, p.y, p.z, p.ci, p.valid, c);
    const size_t N = a.g.N, i = (size_t)p.ci;
    double fb[3] = {0.0, 0.0, 0.0};
    if (force_mode == kForceDense) {
        const CT *f = static_cast<const CT *>(a.force) + i;
        for (int k = 0; k < 3; ++k) fb[k] = (double)f[(size_t)k * a.g.Ns];
    } else if (force_mode == kForceCharge) {
        const double re = (double)static_cast<const CT *>(a.force)[i];
        for (int k = 0; k < 3; ++k) fb[k] = re * a.E[k];
    } else if (force_mode == kForcePotential && !(c.fl & (kWall | kObst))) {
        // the force of the sweep, in its compute precision
        CT f0, f1, f2;
        potential_force<CT>(a.g, p.x, p.y, p.z, c.fl, static_cast<const CT *>(a.force), a.flag,
                            a.owner, a.zeta, (CT)a.keps, (CT)a.E[0], (CT)a.E[1], (CT)a.E[2], f0, f1,
                            f2);
        fb[0] = (double)f0;
        fb[1] = (double)f1;
        fb[2] = (double)f2;
    }
    if constexpr (MODE != kLocal) refill<ST, OFF>(a, p.x, p.y, p.z, c);
    if (!p.valid) return;
    double r = 1.0, v[3] = {0.0, 0.0, 0.0};
    if (c.fl & (kWall | kObst)) {
        if (!(c.fl & kWall)) surface_velocity(a, a.Xc, a.owner[i], p.x, p.y, p.z, v);
    } else {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            // the stored value: compute units of FP16 are scaled deviations
            double f = (double)c.v[q];
            if constexpr (sizeof(ST) == 2) f = (double)((float)c.v[q] * kHalfInvScale);
            s += f;
            v[0] += (double)kCx[q] * f;
            v[1] += (double)kCy[q] * f;
            v[2] += (double)kCz[q] * f;
        }
        r = sizeof(ST) == 8 ? s : 1.0 + s;
        for (int k = 0; k < 3; ++k) v[k] = v[k] + 0.5 * fb[k];
    }
    __builtin_nontemporal_store(r, rho + i);
    for (int k = 0; k < 3; ++k) __builtin_nontemporal_store(v[k], u + (size_t)k * N + i);
}

// 32-bit byte offsets when two population arrays fit in 4 GiB (the gather
// addresses an opposite pair from one base)
template <typename ST>
bool small_grid(const Grid &g) {
    return 2 * g.Ns * sizeof(ST) < (size_t(1) << 32) && 4 * g.Ns < (size_t(1) << 32);
}

// read-out of the post-collision state in a.src (pull) or of the post-stream
// state there
template <typename ST>
hipError_t launch_macro_typed(int force_mode, const SweepArgs &a, bool pull, double *rho, double *u,
                              hipStream_t s) {
    const dim3 grid((unsigned)((a.g.N + 255) / 256)), block(256);
#define LBMEP_MACRO(OFF, MD) \
    hipLaunchKernelGGL((k_macro<ST, OFF, MD>), grid, block, 0, s, a, force_mode, rho, u)
    if (small_grid<ST>(a.g)) {
        if (pull) LBMEP_MACRO(uint32_t, kReadout);
        else LBMEP_MACRO(uint32_t, kLocal);
    } else {
        if (pull) LBMEP_MACRO(uint64_t, kReadout);
        else LBMEP_MACRO(uint64_t, kLocal);
    }
#undef LBMEP_MACRO
    return hipGetLastError();
}

// A packed launch reads its arguments from the lattice's descriptor.  Loaded
// through a plain pointer they would be vector values, and the pointers among
// them generic ones: the descriptor is constant during the launch and the
// entry the same for the workgroup, so they are read into scalar registers,
// and the pointers are to global memory (eight lattices of 64^3 to 128^3 cells
// with up to 56 spheres each: exchange and classification 71 -> 42 us, in
// which 296 bytes of arguments per thread had also lain in scratch memory).
template <typename T>
__device__ __forceinline__ T *as_global(T *p) {
    return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}
template <typename T>
__device__ __forceinline__ T load_uniform(const T *p) {
    T r;
    __builtin_memcpy(&r, (const T *)(const __attribute__((address_space(4))) T *)(uintptr_t)p, sizeof(T));
    return r;
}
__device__ __forceinline__ SweepArgs packed_args(const SweepArgs *p) {
    SweepArgs a = load_uniform(p);
    a.src = as_global(a.src);
    a.dst = as_global(a.dst);
    a.flag = as_global(a.flag);
    a.nearmask = as_global(a.nearmask);
    a.owner = as_global(a.owner);
    a.owner_old = as_global(a.owner_old);
    a.Xc = as_global(a.Xc);
    a.Xold = as_global(a.Xold);
    a.U = as_global(a.U);
    a.W = as_global(a.W);
    a.FM = as_global(a.FM);
    a.force = as_global(a.force);
    a.zeta = as_global(a.zeta);
    a.plist = as_global(a.plist);
    a.pcount = as_global(a.pcount);
    a.wlist = as_global(a.wlist);
    a.wcount = as_global(a.wcount);
    return a;
}
__device__ __forceinline__ ParticleArgs packed_args(const ParticleArgs *p) {
    ParticleArgs a = load_uniform(p);
    a.X0 = as_global(a.X0);
    a.R = as_global(a.R);
    a.U = as_global(a.U);
    a.W = as_global(a.W);
    a.flag = as_global(a.flag);
    a.wallbits = as_global(a.wallbits);
    a.plist = as_global(a.plist);
    a.pcount = as_global(a.pcount);
    return a;
}
__device__ __forceinline__ LevelMap packed_args(const LevelMap *p) {
    LevelMap m = load_uniform(p);
    m.owner = as_global(m.owner);
    m.bits = as_global(m.bits);
    m.X = as_global(m.X);
    return m;
}

// the gather sweep of several lattices in one dispatch
// (MODE: kPullNTS, or kPull where the lattices fit in the Infinity Cache)
template <typename ST, int FMODE, int MODE>
__global__ void __launch_bounds__(kPackBlockX) k_sweep_packed(PackTable t) {
    const uint32_t gb = t.xcd_swizzle ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
    const int e = pack_find(t, gb);
    const LatticeDev *d = t.d[e];
    uint32_t b = gb - t.start[e];
    // the entry's first workgroups map its next level
    const uint32_t map_blocks = load_uniform(&d->map_blocks);
    if (b < map_blocks) {
        const uint32_t c = t.state[e] >> 1;
        map_particles(packed_args(&d->pa), b, t.level[e], packed_args(&d->map[c == 2 ? 0 : c + 1]));
        return;
    }
    b -= map_blocks;
    const SweepArgs a = packed_args(&d->sweep[t.state[e]]);
    sweep_segment<ST, FMODE, uint32_t, MODE>(a, b);
}

template <typename ST>
hipError_t launch_sweep_packed_typed(int force_mode, const PackTable &t, hipStream_t s) {
    const uint32_t total = t.start[t.n];
    if (t.n == 0 || total == 0) return hipSuccess;
#define LBMEP_PACKED(FM)                                                                         \
    do {                                                                                         \
        if (t.cached)                                                                            \
            hipLaunchKernelGGL((k_sweep_packed<ST, FM, kPull>), dim3(total), dim3(kPackBlockX), 0, s, t); \
        else                                                                                     \
            hipLaunchKernelGGL((k_sweep_packed<ST, FM, kPullNTS>), dim3(total), dim3(kPackBlockX), 0, s, t); \
    } while (0)
    if (force_mode == kForceNone) LBMEP_PACKED(kForceNone);
    else if (force_mode == kForceDense) LBMEP_PACKED(kForceDense);
    else if (force_mode == kForceCharge) LBMEP_PACKED(kForceCharge);
    else return hipErrorInvalidValue;  // served requests carry no potential force
#undef LBMEP_PACKED
    return hipGetLastError();
}

// host launcher for one storage type
template <typename ST>
hipError_t launch_typed(int mode, int force_mode, SweepArgs a, int block_x,
                        const MapSetArgs *map, hipStream_t s) {
    const bool small = small_grid<ST>(a.g);
    // the workgroups-per-CU cap was measured on the 32-bit-offset kernel;
    // the 64-bit one runs faster without it (864 x 1248 x 864 FP32: 24.6
    // against 27.5 ms)
    if (!small) a.lds = 0;
    const size_t nblocks = (a.g.N + (size_t)block_x - 1) / (size_t)block_x;
    const dim3 block(block_x, 1, 1);
    MapSetArgs ms{};
    size_t total = nblocks;
    if (map && map->pa.np > 0) {
        ms = *map;
        const uint32_t per = 8u * (uint32_t)(block_x / kMapThreads);
        ms.groups = ((uint32_t)map->pa.np + per - 1u) / per;
        const size_t groups = (nblocks + 7) / 8 + ms.groups;
        ms.stride = (uint32_t)(groups / ms.groups);
        total = 8 * groups;
    }
    const dim3 grid((unsigned)total, 1, 1);
    const uint32_t nseg = (uint32_t)nblocks;
#define LBMEP_LAUNCH(MD, FM, OFF) \
    hipLaunchKernelGGL((k_sweep<ST, FM, OFF, MD>), grid, block, a.lds, s, a, ms, nseg)
#define LBMEP_BY_FORCE(MD, OFF)                                           \
    do {                                                                  \
        if (force_mode == kForceNone) LBMEP_LAUNCH(MD, kForceNone, OFF);        \
        else if (force_mode == kForceDense) LBMEP_LAUNCH(MD, kForceDense, OFF); \
        else if (force_mode == kForceCharge) LBMEP_LAUNCH(MD, kForceCharge, OFF); \
        else LBMEP_LAUNCH(MD, kForcePotential, OFF);                            \
    } while (0)
    if (small) {
        if (mode == kPull) LBMEP_BY_FORCE(kPull, uint32_t);
        else if (mode == kPullNT) LBMEP_BY_FORCE(kPullNT, uint32_t);
        else if (mode == kPullNTS) LBMEP_BY_FORCE(kPullNTS, uint32_t);
        else if (mode == kLocal) LBMEP_BY_FORCE(kLocal, uint32_t);
        else LBMEP_LAUNCH(kReadout, kForceNone, uint32_t);
    } else {
        if (mode == kPull || mode == kPullNT || mode == kPullNTS) LBMEP_BY_FORCE(kPull, uint64_t);
        else if (mode == kLocal) LBMEP_BY_FORCE(kLocal, uint64_t);
        else LBMEP_LAUNCH(kReadout, kForceNone, uint64_t);
    }
#undef LBMEP_BY_FORCE
#undef LBMEP_LAUNCH
    return hipGetLastError();
}

}  // namespace sweep
}  // namespace lbmep
