// k_particles.hip -- the particle kernels outside a step (positions, the map
// and the classification when flags or particles are set, the wall lists) and
// the force read-out; the per-particle device functions are in
// particles_impl.h, the kernels of a step in near_impl.h and sweep_impl.h.
#include <cmath>

#include "particles_impl.h"

namespace lbmep {
namespace {

using namespace part;

constexpr int kBoxThreads = 256;

__global__ void k_positions(ParticleArgs pa, int64_t level, double *X) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= pa.np) return;
    for (int k = 0; k < 3; ++k) X[3 * p + k] = position(pa, p, k, level);
}

// map every particle at `level` (into an emptied map)
template <bool BITS>
__global__ void __launch_bounds__(kBoxThreads) k_map_set(ParticleArgs pa, int64_t level, LevelMap m) {
    const uint32_t p = row_block();
    if (p < (uint32_t)pa.np)
        advance_set<BITS>(pa, (int)p, level, m, (int)threadIdx.x, (int)blockDim.x);
}

// the previous level's cells leave a map without bitmaps (with them the step's
// own launches do it)
__global__ void __launch_bounds__(kBoxThreads) k_map_clear(ParticleArgs pa, LevelMap m) {
    const uint32_t p = row_block();
    if (p < (uint32_t)pa.np) map_clear<false>(pa, (int)p, m);
}

__global__ void __launch_bounds__(kPartThreads)
    k_classify_boxes(ParticleArgs pa, LevelMap old, LevelMap now) {
    extern __shared__ __align__(16) unsigned char part_lds[];
    const uint32_t p = row_block();
    if (p < (uint32_t)pa.np) classify(pa, (int)p, old, now, box_rows(part_lds, pa.box_rows));
}

// wall cells as one bit per cell; one word per thread
__global__ void __launch_bounds__(256) k_wall_bits(Grid g, const uint8_t *flag, uint32_t *bits) {
    const size_t w = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (w >= map_words(g.N)) return;
    uint32_t v = 0;
    for (int k = 0; k < 32; ++k) {
        const size_t c = 32 * w + (size_t)k;
        if (c < g.N && (flag[c] & kWall)) v |= 1u << k;
    }
    bits[w] = v;
}

// exclusive prefix of `mine` over the workgroup (256 threads); returns the
// workgroup total in *total
__device__ __forceinline__ uint32_t block_scan(uint32_t mine, uint32_t *wsum, uint32_t *total) {
    const int tid = threadIdx.x, lane = (int)__lane_id(), wave = tid / 64;
    uint32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)incl, off);
        if (lane >= off) incl += t;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t pre = incl - mine;
    for (int w = 0; w < wave; ++w) pre += wsum[w];
    *total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    return pre;
}

// the whole grid (after the flags or the particle table changed): flags and
// the wall-link masks of every cell.  An obstacle cell's wall links are listed
// too: the slot of a wall cell is read by the cell it was bounced from alone,
// so they do no harm until a sphere uncovers the cell.
__global__ void k_classify_all(Grid g, uint8_t *flag, uint32_t *wallmask, const uint32_t *owner) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= g.nx) return;
    const int y = blockIdx.y, z = blockIdx.z;
    uint32_t wm, pm;
    const uint8_t f = classify_cell<true>(g, x, y, z, flag, owner, nullptr, kNone, &wm, &pm);
    const size_t c = cell_of(g, x, y, z);
    flag[c] = f;
    wallmask[c] = wm;
}

// compact list, in cell order, of the cells with a wall link (wall-link mask
// != 0), by a three-kernel scan (no contended atomics): per-block counts, a
// scan of the counts in tiles of 1024, then each block writing its cells
// from its offset.  A thread reads the masks of 16 consecutive cells as four
// 16-byte loads (the mask array is padded to a multiple of kListChunk).
// Built when the walls or the particle table are set, not per step.
constexpr int kListCells = 16;
constexpr int kListChunk = 256 * kListCells;

__device__ __forceinline__ uint32_t wall_bits(const Grid &g, const uint32_t *wallmask, size_t c0) {
    const uint4 *v = reinterpret_cast<const uint4 *>(wallmask + c0);
    uint32_t take = 0;  // bit k: cell c0 + k has a wall link
#pragma unroll
    for (int j = 0; j < kListCells / 4; ++j) {
        const uint4 m = v[j];
        const uint32_t w[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (w[i] && c0 + 4 * j + i < g.N) take |= 1u << (4 * j + i);
    }
    return take;
}

__global__ void __launch_bounds__(256) k_wall_count(Grid g, const uint32_t *wallmask,
                                                    uint32_t *bcount) {
    __shared__ uint32_t wsum[4];
    const size_t c0 = (size_t)blockIdx.x * kListChunk + (size_t)threadIdx.x * kListCells;
    uint32_t total;
    block_scan((uint32_t)__popc(wall_bits(g, wallmask, c0)), wsum, &total);
    if (threadIdx.x == 0) bcount[blockIdx.x] = total;
}

// second level of the scan: workgroup t turns the counts of list blocks
// [1024 t, 1024 t + 1024) into exclusive prefixes within that tile (one
// coalesced load per thread) and stores the tile total after the counts
constexpr int kTile = 1024;

__global__ void __launch_bounds__(kTile) k_wall_tiles(uint32_t *bcount, int nb) {
    const uint32_t tile = blockIdx.x;
    __shared__ uint32_t wsum[kTile / 64];
    const int tid = threadIdx.x, lane = (int)__lane_id(), wave = tid / 64;
    const size_t i = (size_t)tile * kTile + tid;
    const uint32_t mine = i < (size_t)nb ? bcount[i] : 0u;
    uint32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)incl, off);
        if (lane >= off) incl += t;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t pre = incl - mine;
    for (int w = 0; w < wave; ++w) pre += wsum[w];
    if (i < (size_t)nb) bcount[i] = pre;
    if (tid == kTile - 1) {
        uint32_t tot = 0;
        for (int w = 0; w < kTile / 64; ++w) tot += wsum[w];
        bcount[nb + tile] = tot;
    }
}

// list block blk writes its cells from its offset: the exclusive prefix
// within its tile plus the totals of the earlier tiles; the last block also
// stores the list length
__global__ void __launch_bounds__(256) k_wall_write(Grid g, const uint32_t *wallmask,
                                                    const uint32_t *bcount, int nb,
                                                    uint32_t *list, uint32_t *count) {
    __shared__ uint32_t wsum[4];
    const uint32_t blk = blockIdx.x;
    const size_t c0 = (size_t)blk * kListChunk + (size_t)threadIdx.x * kListCells;
    const uint32_t take = wall_bits(g, wallmask, c0);
    uint32_t off = bcount[blk];
    const uint32_t *tsum = bcount + nb;
    for (uint32_t t = 0; t < blk / kTile; ++t) off += tsum[t];
    uint32_t total;
    uint32_t pos = off + block_scan((uint32_t)__popc(take), wsum, &total);
#pragma unroll
    for (int k = 0; k < kListCells; ++k)
        if (take & (1u << k)) list[pos++] = (uint32_t)(c0 + k);
    if (blk == (uint32_t)nb - 1 && threadIdx.x == 0) *count = off + total;
}

// F = F_dev + K/18 and M = M_dev + (T - X x K)/18 from the per-particle
// accumulators F_dev[3], M_dev[3], K[3], T[3] of the sweep
__global__ void k_finalize_ft(int np, const double *acc, const double *X, double *out) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const double *t = acc + 12 * (size_t)p;
    const double *Xp = X + 3 * (size_t)p;
    out[6 * (size_t)p + 0] = t[0] + t[6] / 18.0;
    out[6 * (size_t)p + 1] = t[1] + t[7] / 18.0;
    out[6 * (size_t)p + 2] = t[2] + t[8] / 18.0;
    out[6 * (size_t)p + 3] = t[3] + (t[9] - (Xp[1] * t[8] - Xp[2] * t[7])) / 18.0;
    out[6 * (size_t)p + 4] = t[4] + (t[10] - (Xp[2] * t[6] - Xp[0] * t[8])) / 18.0;
    out[6 * (size_t)p + 5] = t[5] + (t[11] - (Xp[0] * t[7] - Xp[1] * t[6])) / 18.0;
}

}  // namespace

int wall_list_blocks(const Grid &g) { return (int)((g.N + kListChunk - 1) / kListChunk); }
int wall_list_tiles(const Grid &g) { return (wall_list_blocks(g) + kTile - 1) / kTile; }
size_t wall_list_scratch(const Grid &g) {
    return (size_t)wall_list_blocks(g) + (size_t)wall_list_tiles(g) + 64;
}

// halo rows of the largest particle's box when it moves less than one cell,
// (2 ceil(R) + 9)^2, if the classification keeps them in LDS (at most 1024
// rows, 48 KiB: larger boxes would leave one workgroup per CU)
uint32_t box_row_capacity(double r_max) {
    const double e = 2.0 * std::ceil(r_max) + 9.0;
    return e * e <= 1024.0 ? (uint32_t)(e * e) : 1024u;
}
uint32_t classify_lds(uint32_t box_rows, int threads) {
    return box_rows * 8u * kRowArrays + 64u + 4u * row_cells(threads);
}

uint32_t link_capacity(double r_max) {
    const double e = 2.0 * std::ceil(r_max) + 3.0;
    return (uint32_t)(e * e * e);
}

hipError_t launch_wall_list(const Grid &g, const uint32_t *wallmask, uint32_t *list,
                            uint32_t *count, uint32_t *scratch, hipStream_t s) {
    const int nb = wall_list_blocks(g);
    hipLaunchKernelGGL(k_wall_count, dim3(nb), dim3(256), 0, s, g, wallmask, scratch);
    hipLaunchKernelGGL(k_wall_tiles, dim3(wall_list_tiles(g)), dim3(kTile), 0, s, scratch, nb);
    hipLaunchKernelGGL(k_wall_write, dim3(nb), dim3(256), 0, s, g, wallmask, scratch, nb, list,
                       count);
    return hipGetLastError();
}

hipError_t launch_finalize_ft(int np, const double *acc, const double *X, double *out,
                              hipStream_t s) {
    if (np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_finalize_ft, dim3((np + 127) / 128), dim3(128), 0, s, np, acc, X, out);
    return hipGetLastError();
}

hipError_t launch_positions(const ParticleArgs &pa, int64_t level, double *X, hipStream_t s) {
    if (pa.np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_positions, dim3((pa.np + 127) / 128), dim3(128), 0, s, pa, level, X);
    return hipGetLastError();
}

hipError_t launch_map_set(const ParticleArgs &pa, int64_t level, const LevelMap &m, hipStream_t s) {
    if (pa.np == 0) return hipSuccess;
    const dim3 grid = row_grid((size_t)pa.np), block(kBoxThreads);
    if (m.bits)
        hipLaunchKernelGGL(k_map_set<true>, grid, block, 0, s, pa, level, m);
    else
        hipLaunchKernelGGL(k_map_set<false>, grid, block, 0, s, pa, level, m);
    return hipGetLastError();
}

hipError_t launch_map_clear(const ParticleArgs &pa, const LevelMap &m, hipStream_t s) {
    if (pa.np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_map_clear, row_grid((size_t)pa.np), dim3(kBoxThreads), 0, s, pa, m);
    return hipGetLastError();
}

hipError_t launch_wall_bits(const Grid &g, const uint8_t *flag, uint32_t *bits, hipStream_t s) {
    hipLaunchKernelGGL(k_wall_bits, dim3((unsigned)((map_words(g.N) + 255) / 256)), dim3(256), 0, s, g,
                       flag, bits);
    return hipGetLastError();
}

hipError_t launch_classify_all(const Grid &g, uint8_t *flag, uint32_t *wallmask,
                               const uint32_t *owner, hipStream_t s) {
    const int bx = 64;
    hipLaunchKernelGGL(k_classify_all, dim3((g.nx + bx - 1) / bx, g.ny, g.nz), dim3(bx), 0, s, g,
                       flag, wallmask, owner);
    return hipGetLastError();
}

hipError_t launch_classify_boxes(const ParticleArgs &pa, const LevelMap &old, const LevelMap &now,
                                 hipStream_t s) {
    if (pa.np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_classify_boxes, row_grid((size_t)pa.np), dim3(pa.box_threads),
                       classify_lds(pa.box_rows, pa.box_threads), s, pa, old, now);
    return hipGetLastError();
}

}  // namespace lbmep
