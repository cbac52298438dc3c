// lbmep_api.hip -- host runtime behind the C ABI of include/lbmep.h: lattice
// object, argument checks, device memory, the per-step launch sequence and
// checkpointing.  Every step of the method runs in the device kernels of
// k_stream.hip, k_particles.hip and k_fields.hip.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "lattice.h"

using namespace lbmep;
using namespace lbmep::rt;

namespace {
thread_local std::string g_err;
}  // namespace

namespace lbmep {
namespace rt {

int fail(int code, const std::string &msg) {
    g_err = msg;
    return code;
}

#define HIP_TRY(expr) LBMEP_HIP_TRY(expr)

size_t round_up(size_t n, size_t m) { return (n + m - 1) / m * m; }

size_t storage_bytes(int precision) {
    return precision == LBMEP_FP64 ? 8 : (precision == LBMEP_FP32DEV ? 4 : 2);
}

// With a stride of exactly N = 2^k elements, the 19 source and 19
// destination streams of the sweep start at the same offset modulo every
// power of two, so the same cell of every population maps to the same HBM
// channel and bank; at 512^3 the pull pattern then moves ~7 % less data per
// second than with the arrays staggered.  The pad (in elements, a multiple
// of 128 so that the colour-split potential's halves stay aligned) is the
// best of a measured sweep per storage size (LBMEP_POP_PAD overrides it).
size_t population_stride(size_t N, int precision) {
    size_t pad = precision == LBMEP_FP64 ? 256 : 2048;
    if (const char *e = std::getenv("LBMEP_POP_PAD")) {
        const long v = std::atol(e);
        if (v >= 0) pad = round_up((size_t)v, 128);
    }
    return round_up(N, 128) + pad;
}

size_t compute_bytes(int precision) { return precision == LBMEP_FP64 ? 8 : 4; }

// the exponent of an infinity or NaN is all ones: adding one to it carries
// into the sign bit, and the or of the sums needs no branch per value, so the
// host's vector instructions do it
template <typename U, typename T>
bool finite_bits(const T *p, size_t n, U mask, U one) {
    for (size_t i = 0; i < n;) {
        const size_t e = std::min(n, i + 4096);
        U any = 0;
        for (; i < e; ++i) {
            U b;
            std::memcpy(&b, p + i, sizeof b);
            any |= (b & mask) + one;
        }
        if (any >> (8 * sizeof(U) - 1)) return false;
    }
    return true;
}
bool finite_all(const double *p, size_t n) {
    return finite_bits<uint64_t>(p, n, uint64_t(0x7ff) << 52, uint64_t(1) << 52);
}
bool finite_all(const float *p, size_t n) {
    return finite_bits<uint32_t>(p, n, uint32_t(0xff) << 23, uint32_t(1) << 23);
}

hipError_t dev_alloc(lbmep_lattice *L, void **p, size_t bytes) {
    if (!L->heap) {
        const hipError_t e = hipMalloc(p, bytes);
        if (e != hipSuccess) {
            *p = nullptr;
            (void)hipGetLastError();  // the next launch's check is not to find it
        }
        return e;
    }
    *p = L->heap->alloc(bytes);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}

void dev_free(lbmep_lattice *L, void *p) {
    if (!p) return;
    if (!L->heap)
        hipFree(p);
    else
        L->heap->release(p);
}

}  // namespace rt
}  // namespace lbmep


namespace lbmep {
namespace rt {

int set_device(lbmep_lattice *L) {
    HIP_TRY(hipSetDevice(L->cfg.device));
    return LBMEP_OK;
}

ParticleArgs particle_args(const lbmep_lattice *L) {
    ParticleArgs pa;
    pa.g = L->g;
    pa.np = L->np;
    pa.moving = L->cfg.move_particles;
    pa.dynamic = L->dynamic ? 1 : 0;
    pa.X0 = L->X0;
    pa.R = L->R;
    pa.U = L->U;
    pa.W = L->W;
    pa.flag = L->flag;
    pa.wallbits = L->has_walls ? L->wallbits : nullptr;
    pa.plist = L->plist_buf[L->lcur];
    pa.pcount = L->pcount_buf[L->lcur];
    pa.pcap = L->pcap;
    pa.box_rows = L->box_rows;
    pa.threads = L->part_threads;
    pa.box_threads = L->box_threads;
    return pa;
}

// map the particles at `level` into every owner buffer, classify the grid,
// list the cells with wall links, and write the particles' link lists
int remap_all(lbmep_lattice *L) {
    hipStream_t s = L->stream;
    L->lcur = 0;
    const ParticleArgs pa = particle_args(L);
    if (L->np > 0) {
        // the next level's map to its place; it is empty after a step
        const LevelMap m[3] = {L->map[L->cur_owner], L->map[next_map(L, L->cur_owner)],
                               L->map[old_map(L, L->cur_owner)]};
        for (int b = 0; b < 3 && !L->tight; ++b) L->map[b] = m[b];
        for (int b = 0; b < 3; ++b) {
            if (!L->map[b].owner || (b == 1 && L->next_empty)) continue;
            HIP_TRY(launch_fill_u32(L->map[b].owner, kNone, L->g.N, s));
            if (L->map[b].bits) HIP_TRY(launch_fill_u32(L->map[b].bits, 0u, map_words(L->g.N), s));
        }
        // the current and the previous level; the next one's stays empty
        if (L->has_walls && L->wallbits) HIP_TRY(launch_wall_bits(L->g, L->flag, L->wallbits, s));
        HIP_TRY(launch_map_set(pa, L->level, L->map[0], s));
        HIP_TRY(launch_map_set(pa, L->level, L->map[2], s));
        L->cur_owner = 0;
        L->ft_buf = 0;
        L->next_empty = L->map[1].owner != nullptr;
        HIP_TRY(launch_fill_f64(L->FM, 0.0, 18 * (size_t)L->np, s));
    }
    HIP_TRY(launch_classify_all(L->g, L->flag, L->wallmask, L->np > 0 ? L->map[0].owner : nullptr, s));
    HIP_TRY(launch_wall_list(L->g, L->wallmask, L->wall_list, L->wall_count, L->wall_scratch, s));
    if (L->np > 0) HIP_TRY(launch_classify_boxes(pa, L->map[0], L->map[0], s));
    return LBMEP_OK;
}

// constants of the FP32-compute collision (see TrtF32), rounded once from
// FP64 products
TrtF32 trt_f32_constants(const lbmep_lattice *L) {
    const double kc = L->precision == LBMEP_FP16DEV ? (double)kHalfScale : 1.0;
    const double le = L->le, lo = L->lo, ae = L->ae, ao = L->ao;
    const double w0 = 1.0 / 3.0, wk[2] = {1.0 / 18.0, 1.0 / 36.0};
    TrtF32 t;
    t.hle = (float)(0.5 * le);
    t.le = (float)le;
    t.b15 = (float)(1.5 / kc);
    t.lw0 = (float)(le * w0);
    t.m0 = (float)(3.0 * ae * w0 / kc);
    for (int k = 0; k < 2; ++k) {
        t.lw[k] = (float)(le * wk[k]);
        t.m[k] = (float)(3.0 * ae * wk[k] / kc);
        t.k1[k] = (float)(4.5 * le * wk[k] / kc);
        t.k3[k] = (float)(9.0 * ae * wk[k] / kc);
        t.hlo[k] = (float)(lo * 3.0 * wk[k]);
        t.k4[k] = (float)(3.0 * ao * wk[k]);
    }
    t.fscale = (float)kc;
    for (int k = 0; k < 3; ++k) t.Ec[k] = (float)L->E[k] * (float)kc;
    return t;
}

SweepArgs sweep_args_state(const lbmep_lattice *L, int cur, int co) {
    SweepArgs a;
    a.g = L->g;
    a.src = L->f[cur];
    a.dst = L->f[1 - cur];
    a.flag = L->flag;
    a.nearmask = L->wallmask;
    const bool parts = L->np > 0;
    a.owner = parts ? L->map[co].owner : nullptr;
    a.owner_old = parts ? L->map[old_map(L, co)].owner : nullptr;
    a.Xc = parts ? L->map[co].X : nullptr;
    a.Xold = parts ? L->map[old_map(L, co)].X : nullptr;
    a.U = L->U;
    a.W = L->W;
    a.FM = parts ? L->FM : nullptr;
    a.force = L->force;
    for (int k = 0; k < 3; ++k) a.E[k] = L->E[k];
    a.le = L->le;
    a.lo = L->lo;
    a.ae = L->ae;
    a.ao = L->ao;
    a.tf = trt_f32_constants(L);
    a.mx = (uint64_t(1) << 63) / (uint64_t)L->g.nx + 1;
    a.my = (uint64_t(1) << 63) / (uint64_t)L->g.ny + 1;
    a.xcd_swizzle = L->xcd_swizzle;
    a.slip = L->slip;
    // measured at 512^3 (4096 moving spheres, two repeats): a cap of 4
    // workgroups per CU is fastest for FP32 (3.56-3.71 ms; 3: 4.1-4.5, none:
    // 3.56-3.84) and FP64 (7.03-7.21 ms; none: 7.19-8.06) with a charge or
    // dense force; FP16 and the force from the potential (its neighbour
    // reads of psi want every wave: 4.4-4.6 ms uncapped, 5.8-6.2 with 4) run
    // best uncapped
    int wgcu = L->sweep_wgcu;
    if (wgcu < 0)
        wgcu = L->force_mode == kForcePotential || L->precision == LBMEP_FP16DEV ? 0 : 4;
    a.lds = wgcu > 0 ? (uint32_t)((160 * 1024) / wgcu / 16 * 16) : 0u;
    a.keps = L->keps;
    a.zeta = L->force_mode == kForcePotential ? L->zeta : nullptr;
    a.np = L->np;
    a.pcap = L->pcap;
    a.plist = L->plist_buf[L->lcur];
    a.pcount = L->pcount_buf[L->lcur];
    a.wlist = L->wall_list;
    a.wcount = L->wall_count;
    return a;
}

SweepArgs sweep_args(const lbmep_lattice *L) { return sweep_args_state(L, L->cur, L->cur_owner); }

void advance_state(lbmep_lattice *L) {
    L->ft_buf = L->cur_owner;
    L->cur = 1 - L->cur;
    L->pmode = true;
    if (L->np > 0 && L->cfg.move_particles) {
        L->cur_owner = next_map(L, L->cur_owner);
        // with dynamics the classification follows the exchange and may
        // rewrite the lists in place
        if (L->overlap && !L->dynamic) L->lcur ^= 1;
    }
    L->level += 1;
}

// bring the grid to the post-stream state of the current level (gather from
// the post-collision state), so that it can be read or modified in place
int materialize(lbmep_lattice *L) {
    if (!L->pmode) return LBMEP_OK;
    SweepArgs a = sweep_args(L);
    a.FM = nullptr;
    HIP_TRY(launch_sweep(L->precision, kSweepReadout, kForceNone, a, L->block_x, nullptr, L->stream));
    L->cur = 1 - L->cur;
    L->pmode = false;
    return LBMEP_OK;
}

void free_particles(lbmep_lattice *L) {
    dev_free(L, L->X0);
    dev_free(L, L->R);
    dev_free(L, L->U);
    dev_free(L, L->W);
    dev_free(L, L->FM);
    for (int b = 0; b < 3; ++b) {
        dev_free(L, L->map[b].X);
        L->map[b].X = nullptr;
    }
    for (int b = 0; b < 2; ++b) {
        dev_free(L, L->pcount_buf[b]);
        L->pcount_buf[b] = nullptr;
    }
    L->X0 = L->R = L->U = L->W = L->FM = nullptr;
    L->np_cap = 0;
}

// maps of the current (0) and the previous level (2), with moving particles
// of the next (1), their bitmaps and the walls'
bool alloc_maps(lbmep_lattice *L) {
    const size_t words = map_words(L->g.N);
    const bool third = L->cfg.move_particles && !L->tight;
    for (int b = 0; b < 3; ++b) {
        LevelMap &m = L->map[b];
        if (m.owner || (b == 1 && !third)) continue;
        if (dev_alloc(L, (void **)&m.owner, 4 * L->g.N) != hipSuccess) return false;
        L->next_empty = false;
    }
    if (L->tight || L->bitmaps) return true;
    // one buffer for the bitmaps (freeing one waits for the device)
    if (dev_alloc(L, (void **)&L->bitmaps, (third ? 4 : 3) * 4 * words) != hipSuccess) return false;
    L->wallbits = L->bitmaps;
    uint32_t *next = L->bitmaps + words;
    for (int b = 0; b < 3; ++b)
        if (L->map[b].owner) {
            L->map[b].bits = next;
            next += words;
        }
    return true;
}

// the particle table for n particles
bool alloc_tables(lbmep_lattice *L, size_t n) {
    if (n <= L->np_cap) return true;
    free_particles(L);
    const size_t b = 3 * n * sizeof(double);
    bool ok = dev_alloc(L, (void **)&L->X0, b) == hipSuccess && dev_alloc(L, (void **)&L->U, b) == hipSuccess &&
              dev_alloc(L, (void **)&L->W, b) == hipSuccess && dev_alloc(L, (void **)&L->R, b / 3) == hipSuccess &&
              dev_alloc(L, (void **)&L->FM, 6 * b) == hipSuccess;
    for (int r = 0; r < 3 && ok; ++r)
        if (L->map[r].owner) ok = dev_alloc(L, (void **)&L->map[r].X, b) == hipSuccess;
    for (int r = 0; r < (L->overlap ? 2 : 1) && ok; ++r)
        ok = dev_alloc(L, (void **)&L->pcount_buf[r], 4 * n) == hipSuccess;
    if (ok) L->np_cap = n;
    return ok;
}

// the link lists of `entries` entries altogether
bool alloc_lists(lbmep_lattice *L, size_t entries) {
    if (entries <= L->plist_entries) return true;
    L->plist_entries = 0;
    for (int r = 0; r < 2; ++r) {
        dev_free(L, L->plist_buf[r]);
        L->plist_buf[r] = nullptr;
    }
    for (int r = 0; r < (L->overlap ? 2 : 1); ++r)
        if (dev_alloc(L, (void **)&L->plist_buf[r], entries * sizeof(uint2)) != hipSuccess) return false;
    L->plist_entries = entries;
    return true;
}

// the form with two maps, one set of link lists and no bitmaps, from a new
// lattice's or before the particles are set anew (their tables go too)
void make_tight(lbmep_lattice *L) {
    free_particles(L);
    for (int b = 0; b < 3; ++b) L->map[b].bits = nullptr;
    dev_free(L, L->bitmaps);
    L->bitmaps = L->wallbits = nullptr;
    dev_free(L, L->map[1].owner);
    L->map[1].owner = nullptr;
    for (int r = 0; r < 2; ++r) {
        dev_free(L, L->plist_buf[r]);
        L->plist_buf[r] = nullptr;
    }
    L->plist_entries = 0;
    L->tight = true;
    L->overlap = false;
}

size_t lattice_bytes(const lbmep_config *cfg, int32_t n_particles, double r_max,
                     int force_mode, bool tight) {
    const size_t N = (size_t)cfg->nx * cfg->ny * cfg->nz;
    const size_t Ns = population_stride(N, cfg->precision);
    size_t b = 2 * (size_t)Q * Ns * storage_bytes(cfg->precision);  // two population grids
    b += round_up(N, 4096) + 4 * round_up(N, 4096) + 4 * N;      // flags, wall masks, wall list
    if (n_particles > 0) {
        const bool third = cfg->move_particles && !tight;
        const size_t maps = third ? 3 : 2, lists = third ? 2 : 1;
        b += maps * 4 * N;                                   // owners by level
        if (!tight) b += (maps + 1) * 4 * map_words(N);      // bits by level, wall bits
        b += (size_t)n_particles * (16 + (4 + maps) * 3) * 8;  // particle table
        // link lists; with overlapped stepping the next level's too
        b += lists * (size_t)n_particles * (8 * (size_t)link_capacity(r_max) + 4);
    }
    if (force_mode == kForceDense) b += 3 * Ns * compute_bytes(cfg->precision);
    if (force_mode == kForceCharge || force_mode == kForcePotential)
        b += Ns * compute_bytes(cfg->precision);
    if (force_mode == kForcePotential) b += 8 * (size_t)n_particles;
    Grid g{};
    g.nx = cfg->nx;
    g.ny = cfg->ny;
    g.nz = cfg->nz;
    g.N = N;
    g.Ns = Ns;
    b += 4 * wall_list_scratch(g) + 256;                          // list scan, list length
    b += (5 * (size_t)invariants_blocks(g) + 4) * sizeof(double);  // reductions
    return b;
}

int check_config(const lbmep_config *cfg) {
    if (!cfg) return fail(LBMEP_EINVAL, "null config");
    if (cfg->nx <= 0 || cfg->ny <= 0 || cfg->nz <= 0)
        return fail(LBMEP_EINVAL, "grid sizes must be positive");
    if ((double)cfg->nx * cfg->ny * cfg->nz > 4.0e9)
        return fail(LBMEP_EINVAL, "grid larger than 4e9 cells");
    if (cfg->nx > (1 << 20) || cfg->ny > 65535 || cfg->nz > 65535)
        return fail(LBMEP_EINVAL, "ny and nz must be <= 65535");
    if (!(std::isfinite(cfg->nu) && cfg->nu > 0.0)) return fail(LBMEP_EINVAL, "nu must be > 0");
    if (!(std::isfinite(cfg->magic) && cfg->magic > 0.0))
        return fail(LBMEP_EINVAL, "magic parameter must be > 0");
    if (cfg->precision < LBMEP_FP64 || cfg->precision > LBMEP_FP16DEV)
        return fail(LBMEP_EINVAL, "unknown precision");
    if (cfg->reserved != 0) return fail(LBMEP_EINVAL, "reserved must be 0");
    return LBMEP_OK;
}

}  // namespace rt
}  // namespace lbmep

extern "C" {

const char *lbmep_last_error(void) { return g_err.c_str(); }

int lbmep_footprint(const lbmep_config *cfg, int32_t n_particles, double r_max, int with_charge,
                    size_t *bytes) {
    int rc = check_config(cfg);
    if (rc) return rc;
    if (!bytes || n_particles < 0 || !(r_max >= 0.0) || !std::isfinite(r_max))
        return fail(LBMEP_EINVAL, "bad footprint arguments");
    *bytes = lattice_bytes(cfg, n_particles, r_max, with_charge ? kForceCharge : kForceNone, false);
    // (fixed particles, which do without the next level's map, are given as
    // much, so that a configuration differs from its moving one by the lists)
    if (n_particles > 0 && !cfg->move_particles)
        *bytes += 4 * ((size_t)cfg->nx * cfg->ny * cfg->nz + map_words((size_t)cfg->nx * cfg->ny * cfg->nz)) +
                  24 * (size_t)n_particles;
    return LBMEP_OK;
}

int lbmep_copy_reference(void *dst, const void *src, size_t bytes, void *stream) {
    if (!dst || !src) return fail(LBMEP_EINVAL, "null pointer");
    if ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src) | bytes) & 15u)
        return fail(LBMEP_EINVAL, "pointers and size must be multiples of 16 bytes");
    HIP_TRY(launch_copy16(src, dst, bytes, (hipStream_t)stream));
    return LBMEP_OK;
}

int lbmep_destroy(lbmep_lattice *L) { return destroy_lattice(L, true); }

int lbmep_create(const lbmep_config *cfg, lbmep_lattice **out) {
    return create_lattice(cfg, nullptr, out);
}

}  // extern "C"

namespace lbmep {
namespace rt {

int destroy_lattice(lbmep_lattice *L, bool sync) {
    if (!L) return LBMEP_OK;
    hipSetDevice(L->cfg.device);
    if (sync) hipStreamSynchronize(L->stream);
    dev_free(L, L->f[0]);
    dev_free(L, L->f[1]);
    dev_free(L, L->flag);
    dev_free(L, L->wallmask);
    dev_free(L, L->wall_list);
    dev_free(L, L->wall_count);
    dev_free(L, L->wall_scratch);
    for (int b = 0; b < 2; ++b) dev_free(L, L->plist_buf[b]);
    for (int b = 0; b < 3; ++b) dev_free(L, L->map[b].owner);
    dev_free(L, L->bitmaps);
    dev_free(L, L->force);
    dev_free(L, L->red);
    dev_free(L, L->zeta);
    dev_free(L, L->q);
    dev_free(L, L->too_fast);
    dev_free(L, L->sor_ctl);
    dev_free(L, L->sor_partial);
    dev_free(L, L->sor_nlist);
    dev_free(L, L->sor_nscratch);
    dev_free(L, L->sor_nrow);
    dev_free(L, L->sor_nmask);
    dev_free(L, L->sor_ibits);
    dev_free(L, L->psi2);
    dev_free(L, L->sor_save);
    dev_free(L, L->sor_codes);
    free_particles(L);
    for (hipEvent_t e : L->ev) hipEventDestroy(e);
    delete L;
    return LBMEP_OK;
}

size_t population_bytes(const Grid &g, int precision) {
    return 2 * (size_t)Q * g.Ns * storage_bytes(precision);
}
bool cache_resident(const Grid &g, int precision) {
    return population_bytes(g, precision) < kInfinityCache;
}

int create_lattice(const lbmep_config *cfg, DevHeap *heap, lbmep_lattice **out) {
    int rc = check_config(cfg);
    if (rc) return rc;
    if (!out) return fail(LBMEP_EINVAL, "null output pointer");
    *out = nullptr;
    int ndev = 0;
    HIP_TRY(hipGetDeviceCount(&ndev));
    if (cfg->device < 0 || cfg->device >= ndev) return fail(LBMEP_EINVAL, "no such device");
    HIP_TRY(hipSetDevice(cfg->device));
    lbmep_lattice *L = new lbmep_lattice();
    L->heap = heap;
    L->cfg = *cfg;
    L->stream = (hipStream_t)cfg->stream;
    // overlapped stepping for a lattice of its own with moving particles
    // (LBMEP_STEP_OVERLAP=0: the classification after the exchange, in the
    // same workgroups, for comparisons)
    L->overlap = cfg->move_particles != 0;
    if (const char *e = std::getenv("LBMEP_STEP_OVERLAP")) L->overlap = L->overlap && std::atoi(e) != 0;
    // (LBMEP_STEP_TIGHT=1: the form for lattices that the memory has no room
    // for otherwise, for comparisons)
    if (const char *e = std::getenv("LBMEP_STEP_TIGHT"))
        if (std::atoi(e) != 0) make_tight(L);
    L->precision = cfg->precision;
    Grid &g = L->g;
    g.nx = cfg->nx;
    g.ny = cfg->ny;
    g.nz = cfg->nz;
    for (int k = 0; k < 3; ++k) g.per[k] = cfg->periodic[k] ? 1 : 0;
    g.N = (size_t)g.nx * g.ny * g.nz;
    g.Ns = population_stride(g.N, cfg->precision);
    // Eq. kinVisc: nu = (tau - 1/2) c_s^2; lambda_e = -1/tau (Sec. 3.1); the
    // odd rate from Lambda = (1/s_e - 1/2)(1/s_o - 1/2), s = -lambda
    L->tau = cfg->nu * 3.0 + 0.5;
    L->le = -1.0 / L->tau;
    L->lo = -1.0 / (0.5 + cfg->magic / (L->tau - 0.5));
    L->ae = 1.0 + 0.5 * L->le;
    L->ao = 1.0 + 0.5 * L->lo;
    if (!(L->lo > -2.0 && L->lo < 0.0)) {
        delete L;
        return fail(LBMEP_EINVAL, "odd relaxation rate outside ]-2,0[");
    }
    // launch shape of the sweep: segments of block_x consecutive cells (whole
    // wavefronts), streaming (non-temporal) hints on its stores;
    // LBMEP_BLOCK_X, LBMEP_XCD_SWIZZLE and LBMEP_SWEEP_NT override the
    // defaults for launch-shape sweeps.
    // Measured with a charge force, segments of 64 / 128 / 256 / 512 cells:
    //   216 x 312 x 216  FP64 881 / 849 / 857 / 863, FP32 527 / 405 / 402 /
    //                    421, FP16 246 / 222 / 206 / 208 us
    //   512^3            FP64 7.7 / 7.5 / 7.1 / 7.6, FP32 4.69 / 3.44 / 3.44 /
    //                    3.55, FP16 2.31 / 2.05 / 1.86 / 1.78 ms
    //   32^3             FP64 4.9 / 4.9 / 5.4 / 6.1, FP32 4.1 / 4.0 / 4.4 /
    //                    4.6, FP16 3.9 / 3.8 / 4.1 / 4.4 us
    // Lattices whose two population grids fit in the 256 MB Infinity Cache
    // keep them there: no streaming hints, and segments dealt onto XCDs in
    // contiguous runs, so that most neighbours come from the XCD's own L2;
    // larger ones stream in the hardware's order (every XCD on the same
    // planes).  With hints and hardware order / without and in runs:
    //   48^3             FP64 9.5 / 7.2, FP32 6.0 / 5.0, FP16 4.9 / 4.3 us
    //   101 x 67 x 83    FP64 35.1 / 28.6, FP32 18.7 / 14.8, FP16 11.8 / 9.2
    //   128 x 96^2       FP64 (359 MB) 69.3 / 77.7, FP32 (179 MB) 40.2 / 28.7
    //   150^3            FP32 (513 MB) 93.9 / 105, FP16 (256 MB) 49.9 / 54.7
    //   216^3            FP64 550 / 612, FP32 283 / 312, FP16 149 / 162
    const bool cached = cache_resident(g, L->precision);
    L->block_x = L->precision == LBMEP_FP64 ? 128 : L->precision == LBMEP_FP16DEV ? 512 : 256;
    L->xcd_swizzle = cached;
    // SOR tiles: 8 rows per thread and 8-plane chunks for FP32 psi; FP64 psi
    // needs twice the registers per row, so 4 and 4 (measured best of each)
    L->sor_rows = L->precision == LBMEP_FP64 ? 4 : 8;
    L->sor_zc = L->precision == LBMEP_FP64 ? 4 : 8;
    if (const char *e = std::getenv("LBMEP_SOR_ZC")) {
        const int c = std::atoi(e);
        if (c >= 1 && c <= 1024) L->sor_zc = c;
    }
    if (const char *e = std::getenv("LBMEP_SOR_WX")) {
        const int c = std::atoi(e);
        if (c == 1 || c == 2 || c == 4) L->sor_wx = c;
    }
    if (const char *e = std::getenv("LBMEP_SOR_XCD")) L->sor_xcd = std::atoi(e) != 0;
    if (const char *e = std::getenv("LBMEP_SOR_NEARBLK")) {
        const int c = std::atoi(e);
        if (c >= 8 && c <= 65536 && c % 8 == 0) L->sor_near_blocks = c;
    }
    // one-pass SOR iteration: rows per thread and planes per workgroup
    L->sor_mrw = 4;
    if (const char *e = std::getenv("LBMEP_SOR_MRW")) {
        const int c = std::atoi(e);
        if (c == 1 || c == 2 || c == 4 || c == 8) L->sor_mrw = c;
    }
    if (const char *e = std::getenv("LBMEP_SOR_MZC")) {
        const int c = std::atoi(e);
        if (c >= 1 && c <= 1024) L->sor_mzc = c;
    }
    if (const char *e = std::getenv("LBMEP_SOR_ROWS")) {
        const int c = std::atoi(e);
        if (c == 4 || c == 8) L->sor_rows = c;
    }
    if (const char *e = std::getenv("LBMEP_BLOCK_X")) {
        const int b = std::atoi(e);
        if (b >= 64 && b <= 512 && b % 64 == 0) L->block_x = b;
    }
    if (const char *e = std::getenv("LBMEP_XCD_SWIZZLE")) L->xcd_swizzle = std::atoi(e) != 0;
    // measured at 512^3: hints on the stores only are fastest for every
    // storage type (the loads' one-element overlaps along x then hit L2;
    // FP16 with 512-cell segments: 1.99 against 2.02-2.06 ms with hints on
    // the loads too)
    // workgroups per CU of the sweep capped by a dynamic LDS allocation per
    // workgroup (the kernel uses none of it; 160 KiB of LDS per CU), set per
    // force mode in sweep_args_state; LBMEP_SWEEP_WGCU (workgroups per CU, 0:
    // no cap) overrides it
    L->sweep_wgcu = -1;
    if (const char *e = std::getenv("LBMEP_SWEEP_WGCU")) {
        const int w = std::atoi(e);
        if (w >= 0 && w <= 32) L->sweep_wgcu = w;
    }
    L->sweep_nt = cached ? 0 : 2;
    if (const char *e = std::getenv("LBMEP_SWEEP_NT")) {
        const int v = std::atoi(e);
        if (v >= 0 && v <= 2) L->sweep_nt = v;
    }
    const size_t es = storage_bytes(L->precision);
    bool ok = true;
    ok = ok && dev_alloc(L, (void **)&L->f[0], Q * g.Ns * es) == hipSuccess;
    ok = ok && dev_alloc(L, (void **)&L->f[1], Q * g.Ns * es) == hipSuccess;
    // flags padded for the 16-byte reads of the NEAR-list compaction
    ok = ok && dev_alloc(L, (void **)&L->flag, round_up(g.N, 4096)) == hipSuccess;
    // wall masks padded for the 16-byte reads of the list compaction
    ok = ok && dev_alloc(L, (void **)&L->wallmask, 4 * round_up(g.N, 4096)) == hipSuccess;
    ok = ok && dev_alloc(L, (void **)&L->wall_list, 4 * g.N) == hipSuccess;
    ok = ok && dev_alloc(L, (void **)&L->wall_count, 256) == hipSuccess;
    ok = ok && dev_alloc(L, (void **)&L->wall_scratch, 4 * wall_list_scratch(g)) == hipSuccess;
    L->red_blocks = invariants_blocks(g);
    ok = ok && dev_alloc(L, (void **)&L->red, (5 * (size_t)L->red_blocks + 4) * sizeof(double)) == hipSuccess;
    if (!ok) {
        destroy_lattice(L, true);
        return fail(LBMEP_ENOMEM, "device allocation failed");
    }
    hipStream_t s = L->stream;
    hipError_t e = hipMemsetAsync(L->flag, 0, round_up(g.N, 4096), s);
    if (e == hipSuccess) e = hipMemsetAsync(L->wallmask, 0, 4 * round_up(g.N, 4096), s);
    if (e == hipSuccess) e = launch_classify_all(g, L->flag, L->wallmask, nullptr, s);
    if (e == hipSuccess)
        e = launch_wall_list(g, L->wallmask, L->wall_list, L->wall_count, L->wall_scratch, s);
    const double u0[3] = {0, 0, 0};
    if (e == hipSuccess) e = launch_init_equilibrium(L->precision, g, L->f[0], 1.0, u0, s);
    if (e == hipSuccess) e = launch_init_equilibrium(L->precision, g, L->f[1], 1.0, u0, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        destroy_lattice(L, true);
        return fail(LBMEP_EDEVICE, std::string("initialisation: ") + hipGetErrorString(e));
    }
    *out = L;
    return LBMEP_OK;
}

}  // namespace rt
}  // namespace lbmep

extern "C" {

int lbmep_set_flags(lbmep_lattice *L, const uint8_t *flags, int on_device) {
    if (!L || !flags) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    const size_t N = L->g.N;
    if (!on_device) {
        for (size_t i = 0; i < N; ++i)
            if (flags[i] != LBMEP_FLUID && flags[i] != LBMEP_WALL)
                return fail(LBMEP_EINVAL, "flag values must be LBMEP_FLUID or LBMEP_WALL");
    }
    rc = materialize(L);
    if (rc) return rc;
    uint8_t *tmp = nullptr;
    const uint8_t *src = flags;
    if (!on_device) {
        HIP_TRY(dev_alloc(L, (void **)&tmp, N));
        hipError_t e = hipMemcpyAsync(tmp, flags, N, hipMemcpyHostToDevice, L->stream);
        if (e != hipSuccess) {
            dev_free(L, tmp);
            return fail(LBMEP_EDEVICE, hipGetErrorString(e));
        }
        src = tmp;
    }
    hipError_t e = launch_import_flags(L->g, src, L->flag, L->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
    dev_free(L, tmp);
    if (e != hipSuccess) return fail(LBMEP_EDEVICE, hipGetErrorString(e));
    // the wall pass of the exchange kernel is launched only with wall cells
    // (device flags are not inspected on the host: assume some)
    L->has_walls = true;
    if (!on_device) {
        L->has_walls = false;
        for (size_t i = 0; i < N && !L->has_walls; ++i) L->has_walls = flags[i] == LBMEP_WALL;
    }
    return remap_all(L);
}

int lbmep_set_particles(lbmep_lattice *L, int32_t n, const double *X, const double *R,
                        const double *U, const double *W) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    if (n < 0) return fail(LBMEP_EINVAL, "negative particle count");
    if (n > 0 && (!X || !R || !U)) return fail(LBMEP_EINVAL, "null particle array");
    if (n > 0) {
        if (!finite_all(X, 3 * (size_t)n) || !finite_all(R, n) || !finite_all(U, 3 * (size_t)n) ||
            (W && !finite_all(W, 3 * (size_t)n)))
            return fail(LBMEP_EINVAL, "non-finite particle data");
        for (int i = 0; i < n; ++i)
            if (!(R[i] > 0.0)) return fail(LBMEP_EINVAL, "radii must be > 0");
        // the re-mapping of a step covers the boxes of two consecutive
        // positions grown by one cell: a body may move less than one cell
        if (L->cfg.move_particles)
            for (size_t i = 0; i < 3 * (size_t)n; ++i)
                if (!(std::fabs(U[i]) < 1.0))
                    return fail(LBMEP_EINVAL, "particles must move less than one cell per step");
    }
    int rc = set_device(L);
    if (rc) return rc;
    rc = materialize(L);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(L->stream));
    // capacity of the link lists per particle, from the largest radius
    double rmax = 0.0;
    for (int i = 0; i < n; ++i) rmax = R[i] > rmax ? R[i] : rmax;
    const uint32_t pcap = n > 0 ? link_capacity(rmax) : 0;
    // the maps, the tables and the lists, in the tight form where the memory
    // has no room for the other (a lattice of a server keeps the form that it
    // was admitted in)
    bool ok = n == 0 || (alloc_maps(L) && alloc_tables(L, n) && alloc_lists(L, (size_t)n * pcap));
    if (!ok && !L->heap && !L->tight) {
        make_tight(L);
        ok = alloc_maps(L) && alloc_tables(L, n) && alloc_lists(L, (size_t)n * pcap);
    }
    if (!ok) {  // the lattice is left without particles, their flags with them
        free_particles(L);
        L->np = 0;
        rc = remap_all(L);
        return rc ? rc : fail(LBMEP_ENOMEM, "particle map, table or link list allocation failed");
    }
    L->pcap = pcap;
    // (without bitmaps every box is classified cell by cell)
    L->box_rows = n > 0 && !L->tight ? box_row_capacity(rmax) : 0;
    L->part_threads = part_threads((size_t)n);
    L->box_threads = box_threads((size_t)n, rmax);
    // boundary values of the potential and the dynamics belong to the
    // particle table they were given with
    dev_free(L, L->zeta);
    L->zeta = nullptr;
    L->hzeta.clear();
    dev_free(L, L->q);
    L->q = nullptr;
    L->hq.clear();
    L->dynamic = false;
    if (L->too_fast) HIP_TRY(hipMemset(L->too_fast, 0, 64));  // of the table before
    L->np = n;
    L->hX0.assign(X, X + 3 * (size_t)n);
    L->hR.assign(R, R + n);
    L->hU.assign(U, U + 3 * (size_t)n);
    if (W)
        L->hW.assign(W, W + 3 * (size_t)n);
    else
        L->hW.assign(3 * (size_t)n, 0.0);
    if (n > 0) {
        const size_t b = 3 * (size_t)n * sizeof(double);
        HIP_TRY(hipMemcpy(L->X0, L->hX0.data(), b, hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(L->R, L->hR.data(), b / 3, hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(L->U, L->hU.data(), b, hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(L->W, L->hW.data(), b, hipMemcpyHostToDevice));
    }
    L->level = 0;
    rc = remap_all(L);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(L->stream));
    return LBMEP_OK;
}

static int set_force_common(lbmep_lattice *L, const void *in, int dtype, int on_device,
                            int ncomp, int mode) {
    if (!L || !in) return fail(LBMEP_EINVAL, "null argument");
    if (dtype != LBMEP_DTYPE_F64 && dtype != LBMEP_DTYPE_F32)
        return fail(LBMEP_EINVAL, "unknown dtype");
    int rc = set_device(L);
    if (rc) return rc;
    const size_t N = L->g.N, Ns = L->g.Ns;
    const size_t ib = dtype == LBMEP_DTYPE_F64 ? 8 : 4;
    if (!on_device && !(dtype == LBMEP_DTYPE_F64 ? finite_all((const double *)in, (size_t)ncomp * N)
                                                 : finite_all((const float *)in, (size_t)ncomp * N)))
        return fail(LBMEP_EINVAL, "non-finite force value");
    HIP_TRY(hipStreamSynchronize(L->stream));
    const size_t need = (size_t)ncomp * Ns * compute_bytes(L->precision);
    if (L->force_bytes < need) {
        dev_free(L, L->force);
        L->force = nullptr;
        L->force_bytes = 0;
        if (dev_alloc(L, (void **)&L->force, need) != hipSuccess) {
            L->force_mode = kForceNone;
            return fail(LBMEP_ENOMEM, "force field allocation failed");
        }
        L->force_bytes = need;
    }
    const void *src = in;
    void *tmp = nullptr;
    if (!on_device) {
        HIP_TRY(dev_alloc(L, (void **)&tmp, (size_t)ncomp * N * ib));
        hipError_t e = hipMemcpy(tmp, in, (size_t)ncomp * N * ib, hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            dev_free(L, tmp);
            return fail(LBMEP_EDEVICE, hipGetErrorString(e));
        }
        src = tmp;
    }
    // psi goes into its storage order (colour-split for even nx)
    hipError_t e = mode == kForcePotential
                       ? launch_potential_pack(L->precision, L->g, src, dtype, L->force, L->stream)
                       : launch_convert_force(L->precision, src, dtype, L->force, N, N, Ns, ncomp,
                                              L->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
    dev_free(L, tmp);
    if (e != hipSuccess) return fail(LBMEP_EDEVICE, hipGetErrorString(e));
    L->force_mode = mode;
    return LBMEP_OK;
}

int lbmep_set_force(lbmep_lattice *L, const void *fb, int dtype, int on_device) {
    int rc = set_force_common(L, fb, dtype, on_device, 3, kForceDense);
    if (rc == LBMEP_OK) L->E[0] = L->E[1] = L->E[2] = 0.0;
    return rc;
}

int lbmep_set_charge_force(lbmep_lattice *L, const void *rho_e, int dtype, const double E[3],
                           int on_device) {
    if (!E || !finite_all(E, 3)) return fail(LBMEP_EINVAL, "bad field E");
    int rc = set_force_common(L, rho_e, dtype, on_device, 1, kForceCharge);
    if (rc == LBMEP_OK) {
        L->E[0] = E[0];
        L->E[1] = E[1];
        L->E[2] = E[2];
    }
    return rc;
}

int lbmep_set_potential_force(lbmep_lattice *L, const void *psi, int dtype, double kappa2_eps,
                              const double E[3], const double *zeta, int on_device) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    if (!E || !finite_all(E, 3)) return fail(LBMEP_EINVAL, "bad field E");
    if (!std::isfinite(kappa2_eps)) return fail(LBMEP_EINVAL, "non-finite kappa^2 eps");
    if (zeta && !finite_all(zeta, (size_t)L->np)) return fail(LBMEP_EINVAL, "non-finite zeta");
    int rc = set_device(L);
    if (rc) return rc;
    double *dz = nullptr;
    if (zeta && L->np > 0) {
        if (dev_alloc(L, (void **)&dz, 8 * (size_t)L->np) != hipSuccess)
            return fail(LBMEP_ENOMEM, "zeta allocation failed");
    }
    rc = set_force_common(L, psi, dtype, on_device, 1, kForcePotential);
    if (rc) {
        dev_free(L, dz);
        return rc;
    }
    dev_free(L, L->zeta);
    L->zeta = dz;
    L->hzeta.clear();
    if (dz) {
        L->hzeta.assign(zeta, zeta + L->np);
        HIP_TRY(hipMemcpy(dz, zeta, 8 * (size_t)L->np, hipMemcpyHostToDevice));
    }
    L->keps = kappa2_eps;
    for (int k = 0; k < 3; ++k) L->E[k] = E[k];
    return LBMEP_OK;
}

static SorArgs sor_args(const lbmep_lattice *L) {
    SorArgs a;
    a.g = L->g;
    a.psi = L->force;
    a.psi2 = L->psi2;
    a.flag = L->flag;
    a.owner = L->np > 0 ? L->map[L->cur_owner].owner : nullptr;
    a.zeta = L->zeta;
    a.kappa2 = L->sor_kappa2;
    a.omega = L->sor_omega;
    a.rf = L->sor_rf;
    a.ctl = L->sor_ctl;
    a.partial = L->sor_partial;
    a.nlist = L->sor_nlist;
    a.nscratch = L->sor_nscratch;
    a.nrow = L->sor_nrow;
    a.nmask = L->sor_nmask;
    a.ibits = L->sor_ibits;
    a.xcd_swizzle = (uint32_t)L->sor_xcd;
    a.zc = (uint32_t)L->sor_zc;
    a.wx = (uint32_t)L->sor_wx;
    a.rows = (uint32_t)L->sor_rows;
    a.near_blocks = (uint32_t)L->sor_near_blocks;
    a.codes = L->sor_codes;
    a.save = L->sor_save;
    a.mzc = (uint32_t)L->sor_mzc;
    a.mrw = (uint32_t)L->sor_mrw;
    a.solids = L->np > 0 || L->has_walls;
    return a;
}

// one solve as configured; the fused iteration may leave the result in the
// second buffer, which then becomes psi
static int run_solve(lbmep_lattice *L, hipStream_t s) {
    int swapped = 0;
    HIP_TRY(launch_sor_solve(L->precision, sor_args(L), L->sor_iters, L->sor_check,
                             L->sor_fused, s, &swapped));
    if (swapped) {
        std::swap(L->force, L->psi2);
        std::swap(L->force_bytes, L->psi2_bytes);
    }
    return LBMEP_OK;
}

int lbmep_set_potential_solver(lbmep_lattice *L, double kappa2, double omega, int32_t max_iter,
                               double rf, int32_t check_every) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    if (L->force_mode != kForcePotential) return fail(LBMEP_EINVAL, "no potential set");
    if (!(std::isfinite(kappa2) && kappa2 > 0.0)) return fail(LBMEP_EINVAL, "kappa^2 must be > 0");
    if (!(omega > 0.0 && omega < 2.0)) return fail(LBMEP_EINVAL, "omega outside (0, 2)");
    if (max_iter < 0 || check_every < 1 || !std::isfinite(rf))
        return fail(LBMEP_EINVAL, "bad iteration parameters");
    const int len[3] = {L->g.nx, L->g.ny, L->g.nz};
    for (int k = 0; k < 3; ++k)
        if (L->g.per[k] && (len[k] & 1))
            return fail(LBMEP_EINVAL, "red-black ordering needs even periodic extents");
    if (L->g.N + 2 >= ((size_t)1 << 32))
        return fail(LBMEP_EINVAL, "the solver lists cells with 32-bit indices (N < 2^32 - 2)");
    int rc = set_device(L);
    if (rc) return rc;
    if (!L->sor_ctl) {
        if (dev_alloc(L, (void **)&L->sor_ctl, sizeof(SorCtl)) != hipSuccess)
            return fail(LBMEP_ENOMEM, "solver control block");
        if (dev_alloc(L, (void **)&L->sor_partial, sizeof(double) * kSorPartials) != hipSuccess)
            return fail(LBMEP_ENOMEM, "solver partial sums");
        if (dev_alloc(L, (void **)&L->sor_nlist, 4 * sor_nlist_entries(L->g.N)) != hipSuccess)
            return fail(LBMEP_ENOMEM, "solver boundary list");
        if (dev_alloc(L, (void **)&L->sor_nscratch, 4 * sor_nscratch_entries(L->g.N)) != hipSuccess)
            return fail(LBMEP_ENOMEM, "solver list scratch");
        if (dev_alloc(L, &L->sor_nrow, 2 * compute_bytes(L->precision) *
                                           sor_nrow_entries(L->g.N)) != hipSuccess ||
            dev_alloc(L, (void **)&L->sor_nmask, sor_nlist_entries(L->g.N)) != hipSuccess ||
            dev_alloc(L, (void **)&L->sor_ibits, 6 * 4 * sor_ibits_words_per_colour(L->g.N)) !=
                hipSuccess)
            return fail(LBMEP_ENOMEM, "solver boundary rows");
        SorCtl c{};
        c.res0 = c.res = -1.0;
        HIP_TRY(hipMemcpy(L->sor_ctl, &c, sizeof c, hipMemcpyHostToDevice));
    }
    // one pass per iteration where it applies (even nx, rows of up to 2048
    // cells), else one launch per colour; LBMEP_SOR_FUSED=0 forces the latter
    L->sor_fused = L->g.nx % 2 == 0 && L->g.nx <= 2048;
    if (const char *e = std::getenv("LBMEP_SOR_FUSED")) L->sor_fused = L->sor_fused && std::atoi(e) != 0;
    const size_t need = L->g.Ns * compute_bytes(L->precision);
    if (L->sor_fused && L->psi2_bytes < need) {
        dev_free(L, L->psi2);
        dev_free(L, L->sor_save);
        L->psi2 = L->sor_save = nullptr;
        L->psi2_bytes = 0;
        if (dev_alloc(L, &L->psi2, need) != hipSuccess || dev_alloc(L, &L->sor_save, need) != hipSuccess)
            return fail(LBMEP_ENOMEM, "second potential buffer");
        L->psi2_bytes = need;
    }
    if (L->sor_fused && !L->sor_codes &&
        dev_alloc(L, (void **)&L->sor_codes, 4 * (L->g.N / 2 + 16)) != hipSuccess)
        return fail(LBMEP_ENOMEM, "solver row codes");
    L->sor_kappa2 = kappa2;
    L->sor_omega = omega;
    L->sor_iters = max_iter;
    L->sor_rf = rf;
    L->sor_check = check_every;
    L->sor_set = true;
    return LBMEP_OK;
}

int lbmep_solve_potential(lbmep_lattice *L, int32_t *iters, double res[2]) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    if (L->force_mode != kForcePotential || !L->sor_set)
        return fail(LBMEP_EINVAL, "no potential solver configured");
    int rc = set_device(L);
    if (rc) return rc;
    rc = run_solve(L, L->stream);
    if (rc) return rc;
    if (iters || res) {
        SorCtl c;
        HIP_TRY(hipMemcpyAsync(&c, L->sor_ctl, sizeof c, hipMemcpyDeviceToHost, L->stream));
        HIP_TRY(hipStreamSynchronize(L->stream));
        if (iters) *iters = c.iters;
        if (res) {
            res[0] = c.res0;
            res[1] = c.res;
        }
    }
    return LBMEP_OK;
}

int lbmep_get_solver_stats(lbmep_lattice *L, int32_t *iters, double res[2]) {
    if (!L || !iters || !res) return fail(LBMEP_EINVAL, "null argument");
    if (!L->sor_ctl) return fail(LBMEP_EINVAL, "no potential solver configured");
    int rc = set_device(L);
    if (rc) return rc;
    SorCtl c;
    HIP_TRY(hipMemcpyAsync(&c, L->sor_ctl, sizeof c, hipMemcpyDeviceToHost, L->stream));
    HIP_TRY(hipStreamSynchronize(L->stream));
    *iters = c.iters;
    res[0] = c.res0;
    res[1] = c.res;
    return LBMEP_OK;
}

int lbmep_get_solver_shape(const lbmep_lattice *L, int32_t shape[4]) {
    if (!L || !shape) return fail(LBMEP_EINVAL, "null argument");
    if (!L->sor_set) return fail(LBMEP_EINVAL, "no potential solver configured");
    const bool one = L->sor_fused && L->g.nx % 2 == 0 && L->g.nx <= 2048;
    if (one && sor_tile_shape(L->precision, L->g, (uint32_t)L->sor_mzc, shape + 1)) {
        shape[0] = 1;
    } else if (one) {
        int rw = L->sor_mrw >= 4 ? 4 : (L->sor_mrw >= 2 ? 2 : 1);  // as the solve picks it
        while (L->g.ny % rw) rw >>= 1;
        shape[0] = 1;
        shape[1] = rw;
        shape[2] = L->sor_mzc > 0 ? L->sor_mzc : 16;
        shape[3] = (L->g.nx / 2 + 63) / 64;
    } else {
        shape[0] = 0;
        shape[1] = L->g.nx % 2 == 0 ? L->sor_rows : 4;
        shape[2] = L->g.nx % 2 == 0 ? L->sor_zc : 1;
        shape[3] = L->g.nx % 2 == 0 ? L->sor_wx : 1;
    }
    return LBMEP_OK;
}

int lbmep_get_potential(lbmep_lattice *L, double *psi, int on_device) {
    if (!L || !psi) return fail(LBMEP_EINVAL, "null argument");
    if (L->force_mode != kForcePotential) return fail(LBMEP_EINVAL, "no potential set");
    int rc = set_device(L);
    if (rc) return rc;
    const size_t N = L->g.N;
    double *d = psi;
    if (!on_device && dev_alloc(L, (void **)&d, N * sizeof(double)) != hipSuccess)
        return fail(LBMEP_ENOMEM, "temp");
    hipError_t e = launch_potential_to_f64(L->precision, L->g, L->force, d, L->stream);
    if (e == hipSuccess && !on_device)
        e = hipMemcpyAsync(psi, d, N * sizeof(double), hipMemcpyDeviceToHost, L->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
    if (!on_device) dev_free(L, d);
    if (e != hipSuccess) return fail(LBMEP_EDEVICE, hipGetErrorString(e));
    return LBMEP_OK;
}

int lbmep_set_dynamics(lbmep_lattice *L, double rho_p, const double *q, const double E[3]) {
    if (!L || !E) return fail(LBMEP_EINVAL, "null argument");
    if (!L->cfg.move_particles) return fail(LBMEP_EINVAL, "dynamics need move_particles = 1");
    if (!(std::isfinite(rho_p) && rho_p > 0.0)) return fail(LBMEP_EINVAL, "rho_p must be > 0");
    if (!finite_all(E, 3) || (q && !finite_all(q, (size_t)L->np)))
        return fail(LBMEP_EINVAL, "non-finite E or charge");
    int rc = set_device(L);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(L->stream));
    if (!L->too_fast) {
        if (dev_alloc(L, (void **)&L->too_fast, 64) != hipSuccess) return fail(LBMEP_ENOMEM, "flag");
        HIP_TRY(hipMemset(L->too_fast, 0, 64));
    }
    dev_free(L, L->q);
    L->q = nullptr;
    L->hq.clear();
    if (q && L->np > 0) {
        if (dev_alloc(L, (void **)&L->q, 8 * (size_t)L->np) != hipSuccess)
            return fail(LBMEP_ENOMEM, "charges");
        L->hq.assign(q, q + L->np);
        HIP_TRY(hipMemcpy(L->q, q, 8 * (size_t)L->np, hipMemcpyHostToDevice));
    }
    if (L->np > 0 && !L->dynamic) {
        // from now on X0 holds the current level's positions
        const ParticleArgs pa = particle_args(L);
        HIP_TRY(launch_positions(pa, L->level, L->X0, L->stream));
        HIP_TRY(hipStreamSynchronize(L->stream));
    }
    L->rho_p = rho_p;
    for (int k = 0; k < 3; ++k) L->Edyn[k] = E[k];
    L->dynamic = true;
    return LBMEP_OK;
}

int lbmep_get_particles(lbmep_lattice *L, double *X, double *U, double *W) {
    if (!L || (L->np > 0 && (!X || !U || !W))) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    if (L->np == 0) return LBMEP_OK;
    const size_t b = 3 * (size_t)L->np * sizeof(double);
    HIP_TRY(hipMemcpyAsync(X, L->map[L->cur_owner].X, b, hipMemcpyDeviceToHost, L->stream));
    HIP_TRY(hipMemcpyAsync(U, L->U, b, hipMemcpyDeviceToHost, L->stream));
    HIP_TRY(hipMemcpyAsync(W, L->W, b, hipMemcpyDeviceToHost, L->stream));
    int32_t fast = 0;
    if (L->too_fast)
        HIP_TRY(hipMemcpyAsync(&fast, L->too_fast, 4, hipMemcpyDeviceToHost, L->stream));
    HIP_TRY(hipStreamSynchronize(L->stream));
    if (fast) return fail(LBMEP_EINVAL, "a particle reached one cell per step: the mapping is not valid");
    return LBMEP_OK;
}

int lbmep_set_free_slip(lbmep_lattice *L, const int32_t faces[6]) {
    if (!L || !faces) return fail(LBMEP_EINVAL, "null argument");
    int bits = 0;
    for (int k = 0; k < 6; ++k) {
        if (faces[k] != 0 && faces[k] != 1) return fail(LBMEP_EINVAL, "face value not 0 / 1");
        if (faces[k] && L->g.per[k / 2]) return fail(LBMEP_EINVAL, "free-slip face on a periodic axis");
        if (faces[k]) bits |= 1 << k;
    }
    int rc = set_device(L);
    if (rc) return rc;
    // the stored state is the post-stream state of its level under the old
    // faces; bring it there before the faces change
    rc = materialize(L);
    if (rc) return rc;
    L->slip = bits;
    return LBMEP_OK;
}

int lbmep_get_particle_count(const lbmep_lattice *L, int32_t *n) {
    if (!L || !n) return fail(LBMEP_EINVAL, "null argument");
    *n = L->np;
    return LBMEP_OK;
}

int lbmep_init_equilibrium(lbmep_lattice *L, double rho, const double u[3]) {
    if (!L || !u) return fail(LBMEP_EINVAL, "null argument");
    if (!std::isfinite(rho) || !finite_all(u, 3)) return fail(LBMEP_EINVAL, "non-finite state");
    int rc = set_device(L);
    if (rc) return rc;
    HIP_TRY(launch_init_equilibrium(L->precision, L->g, L->f[L->cur], rho, u, L->stream));
    HIP_TRY(hipStreamSynchronize(L->stream));
    L->pmode = false;
    return LBMEP_OK;
}

int lbmep_set_pdfs(lbmep_lattice *L, const double *f, int on_device) {
    if (!L || !f) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    const size_t N = L->g.N;
    if (!on_device && !finite_all(f, Q * N)) return fail(LBMEP_EINVAL, "non-finite populations");
    double *tmp = nullptr;
    if (!on_device) HIP_TRY(dev_alloc(L, (void **)&tmp, N * sizeof(double)));
    hipError_t e = hipSuccess;
    for (int q = 0; q < Q && e == hipSuccess; ++q) {
        const double *src = f + (size_t)q * N;
        if (!on_device) {
            e = hipMemcpyAsync(tmp, src, N * sizeof(double), hipMemcpyHostToDevice, L->stream);
            src = tmp;
        }
        if (e == hipSuccess) e = launch_pdfs_from_f64(L->precision, L->g, q, src, L->f[L->cur], L->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
    }
    dev_free(L, tmp);
    if (e != hipSuccess) return fail(LBMEP_EDEVICE, hipGetErrorString(e));
    L->pmode = false;
    return LBMEP_OK;
}

int lbmep_get_pdfs(lbmep_lattice *L, double *f, int on_device) {
    if (!L || !f) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    rc = materialize(L);
    if (rc) return rc;
    const size_t N = L->g.N;
    double *tmp = nullptr;
    if (!on_device) HIP_TRY(dev_alloc(L, (void **)&tmp, N * sizeof(double)));
    hipError_t e = hipSuccess;
    for (int q = 0; q < Q && e == hipSuccess; ++q) {
        double *dst = on_device ? f + (size_t)q * N : tmp;
        e = launch_pdfs_to_f64(L->precision, L->g, q, L->f[L->cur], dst, L->stream);
        if (e == hipSuccess && !on_device)
            e = hipMemcpyAsync(f + (size_t)q * N, tmp, N * sizeof(double), hipMemcpyDeviceToHost,
                               L->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
    }
    dev_free(L, tmp);
    if (e != hipSuccess) return fail(LBMEP_EDEVICE, hipGetErrorString(e));
    return LBMEP_OK;
}

int lbmep_step(lbmep_lattice *L, int32_t nsteps) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    if (nsteps < 0) return fail(LBMEP_EINVAL, "negative step count");
    int rc = set_device(L);
    if (rc) return rc;
    hipStream_t s = L->stream;
    const bool solve = L->force_mode == kForcePotential && L->sor_set && L->sor_iters > 0;
    // the next level's map: with prescribed kinematics it is set in the
    // sweep's launch and classified beside the exchange; with dynamics its
    // positions follow from the exchange
    const bool moving = L->np > 0 && L->cfg.move_particles;
    const bool dyn = moving && L->dynamic;
    for (int32_t it = 0; it < nsteps; ++it) {
        // the EDL potential of this level's map, before the collision that
        // uses its force
        if (solve) {
            rc = run_solve(L, s);
            if (rc) return rc;
        }
        const SweepArgs a = sweep_args(L);
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (L->timing) {
            while (L->ev.size() < L->ev_used + 2) {
                hipEvent_t e;
                HIP_TRY(hipEventCreate(&e));
                L->ev.push_back(e);
            }
            e0 = L->ev[L->ev_used];
            e1 = L->ev[L->ev_used + 1];
            L->ev_used += 2;
            HIP_TRY(hipEventRecord(e0, s));
        }
        // gather + refill + collide + bounce-back slots (or, right after the
        // state was set, collide the stored post-stream state in place)
        const int mode = !L->pmode ? kSweepLocal
                         : L->sweep_nt == 1 ? kSweepPullNT
                         : L->sweep_nt == 2 ? kSweepPullNTS
                                            : kSweepPull;
        const int c = L->cur_owner;
        PartsArgs q{};
        q.wall_blocks = near_wall_blocks(L->g, L->has_walls, L->part_threads);
        q.pa = particle_args(L);
        MapSetArgs ms{};
        // the classification in a launch of its own, after the particles'
        const bool apart = moving && (dyn || L->tight || L->part_threads == kManyThreads);
        if (moving) {
            const bool split = L->overlap && !dyn;
            q.mode = L->tight ? (dyn ? kPartsMove : kPartsNear)
                     : dyn    ? kPartsDyn
                     : apart  ? kPartsClear
                     : split  ? kPartsSplit
                              : kPartsOne;
            // the next level's link lists
            q.pa.plist = L->plist_buf[split ? L->lcur ^ 1 : L->lcur];
            q.pa.pcount = L->pcount_buf[split ? L->lcur ^ 1 : L->lcur];
            q.old = L->map[old_map(L, c)];
            q.cur = L->map[c];
            q.next = L->map[next_map(L, c)];
            q.level = L->level + 1;
            if (dyn) {
                // the particles move under this step's force and torque
                q.dyn.q = L->q;
                q.dyn.U = L->U;
                q.dyn.W = L->W;
                q.dyn.X0 = L->X0;
                q.dyn.rho_p = L->rho_p;
                for (int k = 0; k < 3; ++k) q.dyn.E[k] = L->Edyn[k];
                q.dyn.too_fast = L->too_fast;
            } else {
                ms.pa = q.pa;
                ms.next = q.next;
                ms.level = q.level;
            }
        }
        L->next_empty = false;  // until the step is launched
        HIP_TRY(launch_sweep(L->precision, mode, L->force_mode, a, L->block_x,
                             moving && !dyn && !L->tight ? &ms : nullptr, s));
        if (L->timing) HIP_TRY(hipEventRecord(e1, s));
        // bounce-back slots and momentum exchange next to solid cells, and the
        // next level's flags and link lists
        HIP_TRY(launch_parts(L->precision, a, q, s));
        if (moving && L->tight) {
            // (the next level takes the previous one's map)
            HIP_TRY(launch_map_clear(q.pa, q.next, s));
            HIP_TRY(launch_map_set(q.pa, q.level, q.next, s));
        }
        if (apart) HIP_TRY(launch_classify_boxes(q.pa, q.cur, q.next, s));
        L->next_empty = moving && !L->tight;
        advance_state(L);
    }
    return LBMEP_OK;
}

int lbmep_sync(lbmep_lattice *L) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    int rc = set_device(L);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(L->stream));
    return LBMEP_OK;
}

int lbmep_get_macro(lbmep_lattice *L, double *rho, double *u, int on_device) {
    if (!L || !rho || !u) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    const size_t N = L->g.N;
    double *drho = rho, *du = u;
    if (!on_device) {
        if (dev_alloc(L, (void **)&drho, N * sizeof(double)) != hipSuccess) return fail(LBMEP_ENOMEM, "temp");
        if (dev_alloc(L, (void **)&du, 3 * N * sizeof(double)) != hipSuccess) {
            dev_free(L, drho);
            return fail(LBMEP_ENOMEM, "temp");
        }
    }
    hipError_t e = launch_macro(L->precision, L->force_mode, sweep_args(L), L->pmode, drho, du,
                                L->stream);
    if (e == hipSuccess && !on_device) {
        e = hipMemcpyAsync(rho, drho, N * sizeof(double), hipMemcpyDeviceToHost, L->stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(u, du, 3 * N * sizeof(double), hipMemcpyDeviceToHost, L->stream);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
    if (!on_device) {
        dev_free(L, drho);
        dev_free(L, du);
    }
    if (e != hipSuccess) return fail(LBMEP_EDEVICE, hipGetErrorString(e));
    return LBMEP_OK;
}

int lbmep_get_particle_ft(lbmep_lattice *L, double *F, double *M) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    if (L->np == 0) return LBMEP_OK;
    if (!F || !M) return fail(LBMEP_EINVAL, "null output");
    int rc = set_device(L);
    if (rc) return rc;
    std::vector<double> h(6 * (size_t)L->np);
    double *out = L->FM + 12 * (size_t)L->np;
    HIP_TRY(launch_finalize_ft(L->np, L->FM, L->map[L->ft_buf].X, out, L->stream));
    HIP_TRY(hipMemcpyAsync(h.data(), out, h.size() * sizeof(double), hipMemcpyDeviceToHost,
                           L->stream));
    HIP_TRY(hipStreamSynchronize(L->stream));
    for (int p = 0; p < L->np; ++p)
        for (int k = 0; k < 3; ++k) {
            F[3 * p + k] = h[6 * (size_t)p + k];
            M[3 * p + k] = h[6 * (size_t)p + 3 + k];
        }
    return LBMEP_OK;
}

int lbmep_get_map(lbmep_lattice *L, uint8_t *flags, int32_t *owner) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    int rc = set_device(L);
    if (rc) return rc;
    const size_t N = L->g.N;
    if (flags) {
        uint8_t *tmp = nullptr;
        HIP_TRY(dev_alloc(L, (void **)&tmp, N));
        hipError_t e = launch_export_flags(L->g, L->flag, tmp, L->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(flags, tmp, N, hipMemcpyDeviceToHost, L->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
        dev_free(L, tmp);
        if (e != hipSuccess) return fail(LBMEP_EDEVICE, hipGetErrorString(e));
    }
    if (owner) {
        if (L->np > 0) {
            HIP_TRY(hipMemcpyAsync(owner, L->map[L->cur_owner].owner, 4 * N, hipMemcpyDeviceToHost,
                                   L->stream));
            HIP_TRY(hipStreamSynchronize(L->stream));
        } else {
            for (size_t i = 0; i < N; ++i) owner[i] = -1;
        }
    }
    return LBMEP_OK;
}

int lbmep_get_invariants(lbmep_lattice *L, double out[4]) {
    if (!L || !out) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    rc = materialize(L);
    if (rc) return rc;
    double *dout = L->red + 5 * (size_t)L->red_blocks;
    HIP_TRY(launch_invariants(L->precision, L->g, L->f[L->cur], L->flag, L->red, L->red_blocks,
                              dout, L->stream));
    HIP_TRY(hipMemcpyAsync(out, dout, 4 * sizeof(double), hipMemcpyDeviceToHost, L->stream));
    HIP_TRY(hipStreamSynchronize(L->stream));
    if (!finite_all(out, 4)) return fail(LBMEP_ENONFINITE, "non-finite mass or momentum");
    return LBMEP_OK;
}

int lbmep_get_time(lbmep_lattice *L, int64_t *step) {
    if (!L || !step) return fail(LBMEP_EINVAL, "null argument");
    *step = L->level;
    return LBMEP_OK;
}

int lbmep_set_timing(lbmep_lattice *L, int enable) {
    if (!L) return fail(LBMEP_EINVAL, "null lattice");
    L->timing = enable != 0;
    return LBMEP_OK;
}

int lbmep_get_timing(lbmep_lattice *L, double *total_ms, int64_t *launches) {
    if (!L || !total_ms || !launches) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(L->stream));
    double tot = 0.0;
    for (size_t i = 0; i + 1 < L->ev_used; i += 2) {
        float ms = 0.0f;
        HIP_TRY(hipEventElapsedTime(&ms, L->ev[i], L->ev[i + 1]));
        tot += ms;
    }
    *total_ms = tot;
    *launches = (int64_t)(L->ev_used / 2);
    L->ev_used = 0;
    return LBMEP_OK;
}

// ---------------------------------------------------------------------------
// checkpoint
// ---------------------------------------------------------------------------

namespace {
const char kMagic[8] = {'L', 'B', 'M', 'E', 'P', 'c', 'k', '4'};  // 4: psi in cell order, FP64

struct Header {
    char magic[8];
    int32_t nx, ny, nz, per[3], precision, move;
    double nu, magic_param;
    int64_t level;
    int32_t np, force_mode;
    double E[3];
    double keps;       // potential force: kappa^2 eps_e
    int32_t nzeta, pad; // potential force: boundary values that follow the particles
    // red-black SOR of the potential (sor_set = 0: not configured)
    double sor_kappa2, sor_omega, sor_rf;
    int32_t sor_iters, sor_check, sor_set, pad2;
    // particle dynamics (dyn = 0: prescribed); with dynamics the particle
    // table holds the current positions and velocities
    double rho_p, Edyn[3];
    int32_t dyn, nq;
    int32_t slip, pad3;  // free-slip faces
};
}  // namespace

int lbmep_save_state(lbmep_lattice *L, const char *path) {
    if (!L || !path) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    rc = materialize(L);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(L->stream));
    FILE *fp = std::fopen(path, "wb");
    if (!fp) return fail(LBMEP_EINVAL, std::string("cannot open ") + path);
    Header h{};
    std::memcpy(h.magic, kMagic, 8);
    h.nx = L->g.nx;
    h.ny = L->g.ny;
    h.nz = L->g.nz;
    for (int k = 0; k < 3; ++k) h.per[k] = L->g.per[k];
    h.precision = L->precision;
    h.move = L->cfg.move_particles;
    h.nu = L->cfg.nu;
    h.magic_param = L->cfg.magic;
    h.level = L->level;
    h.np = L->np;
    h.force_mode = L->force_mode;
    for (int k = 0; k < 3; ++k) h.E[k] = L->E[k];
    h.keps = L->keps;
    h.nzeta = (int32_t)L->hzeta.size();
    h.sor_kappa2 = L->sor_kappa2;
    h.sor_omega = L->sor_omega;
    h.sor_rf = L->sor_rf;
    h.sor_iters = L->sor_iters;
    h.sor_check = L->sor_check;
    h.sor_set = L->sor_set ? 1 : 0;
    h.dyn = L->dynamic ? 1 : 0;
    h.rho_p = L->rho_p;
    for (int k = 0; k < 3; ++k) h.Edyn[k] = L->Edyn[k];
    h.nq = (int32_t)L->hq.size();
    h.slip = L->slip;
    // with dynamics the table's positions and velocities are the device state
    std::vector<double> pX = L->hX0, pU = L->hU, pW = L->hW;
    if (L->dynamic && L->np > 0) {
        const size_t b = 3 * (size_t)L->np * sizeof(double);
        if (hipMemcpy(pX.data(), L->X0, b, hipMemcpyDeviceToHost) != hipSuccess ||
            hipMemcpy(pU.data(), L->U, b, hipMemcpyDeviceToHost) != hipSuccess ||
            hipMemcpy(pW.data(), L->W, b, hipMemcpyDeviceToHost) != hipSuccess) {
            std::fclose(fp);
            return fail(LBMEP_EDEVICE, "particle state read-back failed");
        }
    }
    bool ok = std::fwrite(&h, sizeof h, 1, fp) == 1;
    const size_t N = L->g.N, Ns = L->g.Ns;
    if (ok && L->np > 0) {
        ok = std::fwrite(pX.data(), 8, pX.size(), fp) == pX.size() &&
             std::fwrite(L->hR.data(), 8, L->hR.size(), fp) == L->hR.size() &&
             std::fwrite(pU.data(), 8, pU.size(), fp) == pU.size() &&
             std::fwrite(pW.data(), 8, pW.size(), fp) == pW.size();
    }
    if (ok && h.nzeta > 0) ok = std::fwrite(L->hzeta.data(), 8, L->hzeta.size(), fp) == L->hzeta.size();
    if (ok && h.nq > 0) ok = std::fwrite(L->hq.data(), 8, L->hq.size(), fp) == L->hq.size();
    // user wall flags
    std::vector<uint8_t> fl(N);
    if (ok) {
        if (hipMemcpy(fl.data(), L->flag, N, hipMemcpyDeviceToHost) != hipSuccess) ok = false;
        for (size_t i = 0; i < N; ++i) fl[i] = (fl[i] & kWall) ? LBMEP_WALL : LBMEP_FLUID;
        ok = ok && std::fwrite(fl.data(), 1, N, fp) == N;
    }
    // force (compute precision); the potential psi in cell order as FP64
    // (its storage order, colour-split for even nx, spans Ns/2 + N/2 slots
    // of a colour, not the first N)
    if (ok && L->force_mode == kForcePotential) {
        double *d = nullptr;
        std::vector<double> buf(N);
        ok = dev_alloc(L, (void **)&d, N * sizeof(double)) == hipSuccess;
        ok = ok && launch_potential_to_f64(L->precision, L->g, L->force, d, L->stream) == hipSuccess &&
             hipMemcpyAsync(buf.data(), d, N * sizeof(double), hipMemcpyDeviceToHost, L->stream) ==
                 hipSuccess &&
             hipStreamSynchronize(L->stream) == hipSuccess;
        if (d) dev_free(L, d);
        ok = ok && std::fwrite(buf.data(), 8, N, fp) == N;
    } else if (ok && L->force_mode != kForceNone) {
        const int nc = L->force_mode == kForceDense ? 3 : 1;
        std::vector<char> buf(N * compute_bytes(L->precision));
        for (int k = 0; k < nc && ok; ++k) {
            ok = hipMemcpy(buf.data(), (char *)L->force + k * Ns * compute_bytes(L->precision),
                           buf.size(), hipMemcpyDeviceToHost) == hipSuccess &&
                 std::fwrite(buf.data(), 1, buf.size(), fp) == buf.size();
        }
    }
    // populations, raw storage format
    if (ok) {
        const size_t es = storage_bytes(L->precision);
        std::vector<char> buf(N * es);
        for (int q = 0; q < Q && ok; ++q) {
            ok = hipMemcpy(buf.data(), (char *)L->f[L->cur] + q * Ns * es, buf.size(),
                           hipMemcpyDeviceToHost) == hipSuccess &&
                 std::fwrite(buf.data(), 1, buf.size(), fp) == buf.size();
        }
    }
    ok = (std::fclose(fp) == 0) && ok;
    if (!ok) return fail(LBMEP_EDEVICE, "checkpoint write failed");
    return LBMEP_OK;
}

int lbmep_load_state(lbmep_lattice *L, const char *path) {
    if (!L || !path) return fail(LBMEP_EINVAL, "null argument");
    int rc = set_device(L);
    if (rc) return rc;
    FILE *fp = std::fopen(path, "rb");
    if (!fp) return fail(LBMEP_EINVAL, std::string("cannot open ") + path);
    Header h{};
    bool ok = std::fread(&h, sizeof h, 1, fp) == 1 && std::memcmp(h.magic, kMagic, 8) == 0 &&
              h.nx == L->g.nx && h.ny == L->g.ny && h.nz == L->g.nz && h.per[0] == L->g.per[0] &&
              h.per[1] == L->g.per[1] && h.per[2] == L->g.per[2] &&
              h.precision == L->precision && h.move == L->cfg.move_particles &&
              h.nu == L->cfg.nu && h.magic_param == L->cfg.magic && h.np >= 0 && h.level >= 0 &&
              (h.nzeta == 0 || h.nzeta == h.np) && (h.nq == 0 || h.nq == h.np) &&
              (h.dyn == 0 || (h.dyn == 1 && h.move)) && (h.slip & ~63) == 0 &&
              h.force_mode >= kForceNone &&
              h.force_mode <= kForcePotential;
    if (!ok) {
        std::fclose(fp);
        return fail(LBMEP_EINVAL, "checkpoint does not match this lattice");
    }
    const size_t N = L->g.N, Ns = L->g.Ns;
    std::vector<double> X(3 * (size_t)h.np), R(h.np), U(3 * (size_t)h.np), W(3 * (size_t)h.np);
    if (h.np > 0)
        ok = std::fread(X.data(), 8, X.size(), fp) == X.size() &&
             std::fread(R.data(), 8, R.size(), fp) == R.size() &&
             std::fread(U.data(), 8, U.size(), fp) == U.size() &&
             std::fread(W.data(), 8, W.size(), fp) == W.size();
    std::vector<double> zeta(h.nzeta);
    if (h.nzeta > 0) ok = ok && std::fread(zeta.data(), 8, zeta.size(), fp) == zeta.size();
    std::vector<double> qv(h.nq);
    if (h.nq > 0) ok = ok && std::fread(qv.data(), 8, qv.size(), fp) == qv.size();
    std::vector<uint8_t> fl(N);
    ok = ok && std::fread(fl.data(), 1, N, fp) == N;
    const int nc = h.force_mode == kForceDense ? 3 : (h.force_mode == kForceNone ? 0 : 1);
    const size_t fbytes = h.force_mode == kForcePotential ? 8 : compute_bytes(L->precision);
    std::vector<char> force(nc * N * fbytes);
    ok = ok && std::fread(force.data(), 1, force.size(), fp) == force.size();
    const size_t es = storage_bytes(L->precision);
    std::vector<char> pdf(Q * N * es);
    ok = ok && std::fread(pdf.data(), 1, pdf.size(), fp) == pdf.size();
    std::fclose(fp);
    if (!ok) return fail(LBMEP_EINVAL, "truncated checkpoint");
    // walls, particles (time level 0 map), then the saved time level
    rc = lbmep_set_flags(L, fl.data(), 0);
    if (rc) return rc;
    L->slip = h.slip;
    rc = lbmep_set_particles(L, h.np, X.data(), R.data(), U.data(), W.data());
    if (rc) return rc;
    if (h.dyn) {
        // the table holds the saved level's positions and velocities
        rc = lbmep_set_dynamics(L, h.rho_p, h.nq > 0 ? qv.data() : nullptr, h.Edyn);
        if (rc) return rc;
    }
    L->level = h.level;
    rc = remap_all(L);
    if (rc) return rc;
    if (nc > 0) {
        const size_t need = nc * Ns * compute_bytes(L->precision);
        if (L->force_bytes < need) {
            dev_free(L, L->force);
            L->force = nullptr;
            L->force_bytes = 0;
            if (dev_alloc(L, (void **)&L->force, need) != hipSuccess) return fail(LBMEP_ENOMEM, "force");
            L->force_bytes = need;
        }
        if (h.force_mode == kForcePotential) {
            // psi from cell order into its storage order
            double *d = nullptr;
            if (dev_alloc(L, (void **)&d, N * sizeof(double)) != hipSuccess)
                return fail(LBMEP_ENOMEM, "psi staging");
            hipError_t e = hipMemcpy(d, force.data(), N * sizeof(double), hipMemcpyHostToDevice);
            if (e == hipSuccess)
                e = launch_potential_pack(L->precision, L->g, d, LBMEP_DTYPE_F64, L->force, L->stream);
            if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
            dev_free(L, d);
            if (e != hipSuccess) return fail(LBMEP_EDEVICE, hipGetErrorString(e));
        } else {
            const size_t cb = N * compute_bytes(L->precision);
            for (int k = 0; k < nc; ++k)
                HIP_TRY(hipMemcpy((char *)L->force + k * Ns * compute_bytes(L->precision),
                                  force.data() + k * cb, cb, hipMemcpyHostToDevice));
        }
    }
    L->force_mode = h.force_mode;
    for (int k = 0; k < 3; ++k) L->E[k] = h.E[k];
    L->keps = h.keps;
    dev_free(L, L->zeta);
    L->zeta = nullptr;
    L->hzeta.clear();
    if (h.nzeta > 0) {
        if (dev_alloc(L, (void **)&L->zeta, 8 * (size_t)h.nzeta) != hipSuccess)
            return fail(LBMEP_ENOMEM, "zeta");
        L->hzeta = zeta;
        HIP_TRY(hipMemcpy(L->zeta, zeta.data(), 8 * (size_t)h.nzeta, hipMemcpyHostToDevice));
    }
    for (int q = 0; q < Q; ++q)
        HIP_TRY(hipMemcpy((char *)L->f[L->cur] + q * Ns * es, pdf.data() + q * N * es, N * es,
                          hipMemcpyHostToDevice));
    HIP_TRY(hipStreamSynchronize(L->stream));
    L->sor_set = false;
    if (h.sor_set) {
        rc = lbmep_set_potential_solver(L, h.sor_kappa2, h.sor_omega, h.sor_iters, h.sor_rf,
                                        h.sor_check);
        if (rc) return rc;
    }
    L->pmode = false;
    return LBMEP_OK;
}

}  // extern "C"
