// Interpolation (eq. 6) and conservative spreading (eq. 7-8).
//
// Interpolation: one lane per marker gathers the 27 support values of each
// component and contracts them with its shape function (SoA loads).
//
// Spreading is deterministic without floating-point atomics:
//   1. every marker is binned into the tiles of the forcing grid that its
//      supports touch (a counting sort: count, exclusive scan, fill);
//   2. one workgroup owns a tile: it accumulates all contributions landing in
//      the tile in LDS as 64-bit fixed-point integers (integer addition is
//      associative, so the sum does not depend on the order in which lanes or
//      markers arrive) and finally adds the tile, converted back to FP32, into
//      the caller's field.  Each node belongs to exactly one tile, so the
//      global update is a plain read-modify-write.
// The fixed-point scale of a tile is a power of two chosen from the largest
// |c_l F_l| (eq. 8) among the tile's markers, so that no sum can overflow and
// the quantum follows the tile's own forces.
#include <cmath>
#include <mutex>

#include "mls_exact.h"

namespace mls {

namespace {

constexpr int kBlock = 256;
constexpr int kSpreadBlock = 256;   // most threads of a spreading tile workgroup

__global__ void __launch_bounds__(kBlock)
k_interp(const Grid *__restrict__ gp, int64_t n, const uint32_t *__restrict__ home, const float *__restrict__ phi,
         const float *__restrict__ u, const float *__restrict__ v, const float *__restrict__ w,
         float *__restrict__ U, float *__restrict__ V, float *__restrict__ W, ErrWord *err)
{
    const Grid &g = *gp;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t l = xcd_block() * blockDim.x + threadIdx.x; l < n; l += stride) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float *q = c == 0 ? u : (c == 1 ? v : w);
            const uint32_t h = home[home_at(l, c)];
            int i, j, k;
            unpack_home(h, i, j, k);
            float *out = c == 0 ? U : (c == 1 ? V : W);
            if (!home_ok(g, c, i, j, k)) {
                raise_error(err, l, MLS_E_SUPPORT);
                out[l] = __builtin_nanf("");
                continue;
            }
            uint32_t oy[3], oz[3];
            support_rows(j, k, g.dims[c][0], g.dims[c][1], g.dims[c][2], oy, oz);
            float qv[kNe];
            load_rows(q, i, g.dims[c][0], oy, oz, qv);
            const float *p = phi + phi_at(l, c);
            float ph[kNe];
#pragma unroll
            for (int kk = 0; kk < kNe; ++kk) ph[kk] = p[kk * kLanes];
            wrap_rows(q, i, j, k, g.dims[c][0], g.dims[c][1], g.dims[c][2], qv);
            float acc = 0.f;
#pragma unroll
            for (int kk = 0; kk < kNe; ++kk) acc += ph[kk] * qv[kk];
            out[l] = acc;
        }
    }
}

// ---- spreading: tile binning -------------------------------------------------
//
// Every marker belongs to exactly one tile of the grid: the tile holding its
// cell (the home of a centre-staggered component on each axis).  A tile's
// markers spread into an LDS box that covers the tile plus the one-node halo
// of their supports (tile + 3 nodes per axis).  Tiles are coloured by the
// parity of their index per axis (a third colour for the last tile of a
// periodic axis with an odd tile count); boxes of tiles of one colour never
// overlap, so a colour's tiles add their boxes into the field with plain
// read-modify-writes, and the colours run one after another.  Each node thus
// receives its additions in the fixed colour order, and inside a box the
// contributions are summed in 64-bit fixed point, whose sum does not depend on
// the order of the markers: the result is bitwise reproducible.


__device__ __forceinline__ int64_t marker_tile(const Grid &g, const uint32_t *__restrict__ home, int64_t l,
                                               bool &valid)
{
    int hc[3][3];
    valid = true;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        unpack_home(home[home_at(l, c)], hc[c][0], hc[c][1], hc[c][2]);
        valid = valid && home_ok(g, c, hc[c][0], hc[c][1], hc[c][2]);
    }
    // the cell on axis d is the home of component (d + 1) % 3 (centre-staggered on d)
    const int tx = tile_of(hc[1][0], g.ax[0].inv_tile);
    const int ty = tile_of(hc[2][1], g.ax[1].inv_tile);
    const int tz = tile_of(hc[0][2], g.ax[2].inv_tile);
    return ((int64_t)tz * g.ntile[1] + ty) * g.ntile[0] + tx;
}

// Lanes of a wavefront that hit the same tile are combined into one atomic:
// the leader adds the count and the others take consecutive slots in lane
// order, so a tile's marker list is made of runs of consecutive markers.
// The counting pass also records each marker's tile (ntiles for a marker
// without a usable support) for the per-tile force maxima.
// Counting sort step of one wavefront (all lanes active): lanes with tile
// t >= 0 are grouped by tile; the counting pass adds each group's size to
// count[t], the filling pass reserves a range of cursor[t] per group and
// writes the group's markers there in lane order.  The groups are found with
// ballots first, then every group leader issues its atomic in one
// instruction, so the wavefront waits for one round trip, not one per tile.
template <bool FILL>
__device__ __forceinline__ void wave_bin(int64_t t, int lane, uint32_t *count, uint32_t *cursor, uint32_t *entries,
                                         uint32_t marker)
{
    unsigned long long pending = __ballot(t >= 0);
    unsigned long long group = 0;   // lanes of this lane's tile
    int leader = 0;
    while (pending) {
        const int lead = __ffsll((long long)pending) - 1;
        const int64_t tl = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)((uint64_t)t >> 32), lead)
                                      << 32) |
                                     (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)t, lead));
        const unsigned long long mask = __ballot(t == tl) & pending;
        if (t == tl) { group = mask; leader = lead; }
        pending &= ~mask;
    }
    if (t < 0) return;
    const uint32_t cnt = (uint32_t)__popcll(group);
    if (!FILL) {
        if (lane == leader) atomicAdd(&count[t], cnt);
    } else {
        uint32_t pos = 0;
        if (lane == leader) pos = atomicAdd(&cursor[t], cnt);
        pos = __shfl(pos, leader);
        entries[pos + __popcll(group & ((1ull << lane) - 1ull))] = marker;
    }
}

template <bool FILL>
__global__ void __launch_bounds__(kBlock)
k_bin(const Grid *__restrict__ gp, int64_t n, const uint32_t *__restrict__ home, uint32_t *__restrict__ count,
      uint32_t *__restrict__ cursor, uint32_t *__restrict__ entries, uint32_t *__restrict__ tile_of_marker,
      ErrWord *err)
{
    const Grid &g = *gp;
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    // the loop bound is wave-uniform so that the ballots see the whole wave
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63); base < n; base += stride) {
        const int64_t l = base + lane;
        int64_t t = -1;
        if (l < n) {
            bool valid;
            const int64_t tt = marker_tile(g, home, l, valid);
            if (valid) t = tt;
            else if (!FILL) raise_error(err, l, MLS_E_SUPPORT);   // contributes nothing
            if (!FILL) tile_of_marker[l] = valid ? (uint32_t)tt : (uint32_t)g.ntiles;
        }
        wave_bin<FILL>(t, lane, count, cursor, entries, (uint32_t)l);
    }
}

// Binning straight from the marker positions (the exact time step): the
// tile of the cell that holds the marker (centre-staggered home on each
// axis); a marker whose cell support leaves a wall axis, or whose position is
// not finite, goes to the extra bucket ntiles, after all tiles.  The counting
// pass locates the markers and records each one's tile in tiles[]; the
// filling pass reads it back.  With jitter (amp2 > 0) the counting pass reads
// the rest positions x, y, z, jitters them (the time step's generator) and
// stores the result in jx, jy, jz, which it then locates.  The filling pass of
// a time step, the counter's last reader behind it, advances the step counter
// (step_ctr non-NULL).
template <bool FILL>
__global__ void __launch_bounds__(kBlock)
k_bin_pos(const Grid *__restrict__ gp, int64_t n, const float *__restrict__ x, const float *__restrict__ y,
          const float *__restrict__ z, uint32_t *__restrict__ count, uint32_t *__restrict__ cursor,
          uint32_t *__restrict__ entries, uint32_t *__restrict__ tiles, float *__restrict__ jx,
          float *__restrict__ jy, float *__restrict__ jz, float amp2, uint64_t seed, unsigned long long *step_ctr)
{
    const Grid &g = *gp;
    const uint64_t step = (!FILL && amp2 > 0.0f) ? *step_ctr : 0ull;
    if (FILL && step_ctr && blockIdx.x == 0 && threadIdx.x == 0) *step_ctr += 1ull;
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const float itx = g.ax[0].inv_tile, ity = g.ax[1].inv_tile, itz = g.ax[2].inv_tile;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63); base < n; base += stride) {
        const int64_t l = base + lane;
        int64_t t = -1;
        if (l < n) {
            if (FILL) {
                t = tiles[l];
            } else {
                float px = x[l], py = y[l], pz = z[l];
                if (amp2 > 0.0f) {
                    jitter_marker(seed, step, n, l, amp2, px, py, pz, px, py, pz);
                    jx[l] = px;
                    jy[l] = py;
                    jz[l] = pz;
                }
                const float p[3] = {px, py, pz};
                int cell[3] = {0, 0, 0};
                bool ok = true;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    // the cell is the centre-staggered home; both its
                    // neighbours must exist on a wall axis
                    ok = ok && cell_axis_f(g.ax[d], p[d], cell[d]);
                    ok = ok && (g.ax[d].periodic || (cell[d] >= 1 && cell[d] + 1 < g.ax[d].n));
                }
                t = ok ? ((int64_t)tile_of(cell[2], itz) * g.ntile[1] + tile_of(cell[1], ity)) * g.ntile[0] +
                             tile_of(cell[0], itx)
                       : g.ntiles;
                tiles[l] = (uint32_t)t;
            }
        }
        wave_bin<FILL>(t, lane, count, cursor, entries, (uint32_t)l);
    }
}

// Clears what a spreading call counts in: the n tile counts, the colour-list
// sizes and claim cursors, and (compact step) the count of the FP64 queue.
__global__ void k_clear(uint32_t *__restrict__ count, int64_t n, uint32_t *__restrict__ work,
                        uint32_t *__restrict__ queue)
{
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 == 0 && queue) queue[0] = 0u;
    for (int64_t i = i0; i < n + kWorkWords; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < kWorkWords) work[i] = 0u;
        else count[i - kWorkWords] = 0u;
    }
}

// Zeroes n words (a kernel rather than a memset node, for graph capture).
__global__ void k_clear_words(uint32_t *p, int64_t n)
{
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

// Exclusive scan of the tile counts, off[ntiles] = total: every block scans
// its chunk from the sum of the chunks before it (ScanFrom).  A launch costs
// about 4.3 us however little it does, so the fewer the chunks, the fewer the
// launches: up to kScanDirect chunks a block adds up the counts before its
// chunk itself; up to kScanAdd chunks it adds up the chunks' sums (one launch
// more); beyond that one workgroup scans the sums first (two more).  On one
// sphere in 64^3 (one chunk) the step's binning went from seven launches to
// four and its total from 30 to 18 us; a block of the last kernel reads at
// most 64 KB of counts, or 16 KB of sums.
constexpr int kScanChunk = 2048;   // elements per block (256 threads x 8)
constexpr int kScanDirect = 8, kScanAdd = 4096;
enum class ScanFrom { Counts, Sums, Scanned };

__global__ void __launch_bounds__(kBlock) k_scan_partials(const uint32_t *__restrict__ count, int64_t nt,
                                                          uint32_t *__restrict__ partial)
{
    __shared__ uint32_t sh[4];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk;
    uint32_t s = 0;
    for (int q = 0; q < kScanChunk / kBlock; ++q) {
        const int64_t i = base + (int64_t)q * kBlock + threadIdx.x;
        if (i < nt) s += count[i];
    }
    uint32_t total;
    block_exclusive_scan(s, sh, total);
    if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kBlock) k_scan_top(uint32_t *__restrict__ partial, int64_t nb)
{
    __shared__ uint32_t sh[4];
    uint32_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kBlock) {
        const int64_t i = b0 + threadIdx.x;
        const uint32_t v = i < nb ? partial[i] : 0u;
        uint32_t total;
        const uint32_t ex = block_exclusive_scan(v, sh, total);
        if (i < nb) partial[i] = carry + ex;
        carry += total;
        __syncthreads();
    }
}

__device__ __forceinline__ int axis_colour(const Grid &g, int d, int t)
{
    const int k = g.ncol[d];
    return k == 1 ? 0 : ((k == 3 && t == g.ntile[d] - 1) ? 2 : (t & 1));
}

// One past the last slot of colour col in the active-tile list (the colours
// in use are 0 .. ncol_x ncol_y ncol_z - 1, their slots consecutive).
__device__ __forceinline__ int64_t colour_end(const Grid &g, int col)
{
    const int used = g.ncol[0] * g.ncol[1] * g.ncol[2];
    return col + 1 < used ? g.colour_base[col + 1] : g.ntiles;
}

// Offsets of a chunk's tiles, and what else follows from its counts: the
// per-tile force maxima tmax[3][tstride] are cleared, ahead of the kernels
// that write c_l F_l, and the non-empty tiles are listed per colour
// (work[col] counts them, active[colour_base[col] + i] lists them; a block
// gathers its tiles in LDS and takes its slots with one atomic per colour;
// tile_slot, if given, receives a tile's place in its list).
// Each thread scans 8 consecutive counts; the counts come in and the offsets
// go out through LDS so that every global access of a wavefront is one
// contiguous run (8-element strided stores leave partial lines that reach
// memory several times over).
__global__ void __launch_bounds__(kBlock)
k_scan_final(const Grid *__restrict__ gp, const uint32_t *__restrict__ count, int64_t nt,
             const uint32_t *__restrict__ partial, ScanFrom from, uint32_t *__restrict__ off,
             uint32_t *__restrict__ cursor, uint32_t *__restrict__ work, uint32_t *__restrict__ active,
             uint32_t *__restrict__ tile_slot, uint32_t *__restrict__ tmax, int64_t tstride)
{
    __shared__ uint32_t sh[4];
    __shared__ uint32_t buf[kScanChunk];
    __shared__ uint32_t lcount[27], lbase[27];
    const Grid &g = *gp;
    const int64_t base = (int64_t)blockIdx.x * kScanChunk;
    constexpr int per = kScanChunk / kBlock;
    if (threadIdx.x < 27) lcount[threadIdx.x] = 0u;
    uint32_t before = 0;
    if (from == ScanFrom::Scanned) {
        before = partial[blockIdx.x];
    } else {
        uint32_t s = 0;
        if (from == ScanFrom::Counts)
            for (int64_t i = threadIdx.x; i < base; i += kBlock) s += count[i];
        else
            for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kBlock) s += partial[i];
        block_exclusive_scan(s, sh, before);
    }
    for (int q = 0; q < per; ++q) {
        const int64_t i = base + q * kBlock + threadIdx.x;
        buf[q * kBlock + threadIdx.x] = i < nt ? count[i] : 0u;
    }
    __syncthreads();
    const int64_t first = base + (int64_t)threadIdx.x * per;
    uint32_t vals[per];
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < per; ++q) {
        vals[q] = buf[threadIdx.x * per + q];
        s += vals[q];
    }
    int col[per];
    uint32_t pos[per];
#pragma unroll
    for (int q = 0; q < per; ++q) {
        const int64_t t = first + q;
        col[q] = -1;
        if (vals[q] && t < g.ntiles) {
            const uint32_t tu = (uint32_t)t, nx = (uint32_t)g.ntile[0], ny = (uint32_t)g.ntile[1];
            const uint32_t row = tu / nx;
            const int tx = (int)(tu - row * nx), ty = (int)(row % ny), tz = (int)(row / ny);
            col[q] = axis_colour(g, 0, tx) + g.ncol[0] * (axis_colour(g, 1, ty) + g.ncol[1] * axis_colour(g, 2, tz));
            pos[q] = atomicAdd(&lcount[col[q]], 1u);
        }
    }
    uint32_t total;
    uint32_t run = before + block_exclusive_scan(s, sh, total);
#pragma unroll
    for (int q = 0; q < per; ++q) {
        buf[threadIdx.x * per + q] = run;
        run += vals[q];
    }
    // the owner of the last tile also writes off[nt] = total
    if (first <= nt - 1 && nt - 1 < first + per) off[nt] = run;
    if (threadIdx.x < 27)
        lbase[threadIdx.x] = lcount[threadIdx.x] ? atomicAdd(&work[threadIdx.x], lcount[threadIdx.x]) : 0u;
    __syncthreads();
    for (int q = 0; q < per; ++q) {
        const int64_t i = base + q * kBlock + threadIdx.x;
        if (i < nt) {
            const uint32_t o = buf[q * kBlock + threadIdx.x];
            off[i] = o;
            cursor[i] = o;
            tmax[i] = 0u;
            tmax[tstride + i] = 0u;
            tmax[2 * tstride + i] = 0u;
        }
    }
#pragma unroll
    for (int q = 0; q < per; ++q)
        if (col[q] >= 0) {
            const int64_t slot = g.colour_base[col[q]] + lbase[col[q]] + pos[q];
            if (slot < colour_end(g, col[q])) active[slot] = (uint32_t)(first + q);
            if (tile_slot) tile_slot[first + q] = lbase[col[q]] + pos[q];
        }
}

// ---- spreading: per-tile fixed-point accumulation ------------------------------

// Box-local index of node i (wrapped) on axis a for a box starting at node b0.
__device__ __forceinline__ int box_local(const Axis &a, int ntile, int nodes, int b0, int i)
{
    if (a.periodic && ntile == 1) return i;            // the box is the whole (short) axis
    int l = i - b0;
    if (a.periodic) l = l < 0 ? l + nodes : (l >= nodes ? l - nodes : l);
    return l;
}

// Workgroup barrier for LDS only.  The phases of a tile share data through
// LDS alone: each field node is flushed by one thread and same-colour tiles
// never overlap, so no thread needs another's global stores.  A full
// __syncthreads would also wait for every outstanding global store (the
// flush of the previous component) before the next phase could start.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): this thread's LDS operations are done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Adds a tile's box (64-bit fixed point, scale qscale) into the FP32 field f
// and returns its nodes to zero.  Consecutive threads take consecutive box
// nodes (their field accesses coalesce along x rows), kFlush per thread at a
// time: the kFlush sums are read from LDS together, then the nonzero ones are
// decoded into box coordinates, their field values loaded together and
// written back.  Box coordinates come from the compile-time row length BX
// (BX > 0) or FP32 reciprocals of the box edges (exact below 2^22 nodes).
// INSIDE: the box lies inside the grid, so a node's index is the origin's
// plus an affine offset; otherwise periodic axes wrap and nodes past a wall
// are skipped.
template <bool INSIDE, int BX>
__device__ __forceinline__ void flush_box(const Grid &g, int c, unsigned long long *acc, int bnodes, int bx_rt,
                                          int by, int b0x, int b0y, int b0z, int nxc, int nyc, int nzc, float inv_bx,
                                          float inv_by, float inv_bxy, double qscale, float *__restrict__ f)
{
    constexpr int kFlush = 8;
    const int bx = BX > 0 ? BX : bx_rt;
    const Axis &AX = g.ax[0], &AY = g.ax[1], &AZ = g.ax[2];
    float *const fo = INSIDE ? f + field_index(g, c, b0x, b0y, b0z) : f;
    const int sz = nxc * nyc;
    for (int q0 = threadIdx.x; q0 < bnodes; q0 += kFlush * blockDim.x) {
        long long sv[kFlush];
#pragma unroll
        for (int u = 0; u < kFlush; ++u) {
            const int q = q0 + u * (int)blockDim.x;
            sv[u] = q < bnodes ? (long long)acc[q] : 0;
        }
        float *dst[kFlush];
        float add[kFlush];
        float old[kFlush];
#pragma unroll
        for (int u = 0; u < kFlush; ++u) {
            dst[u] = nullptr;
            add[u] = 0.f;
            const int q = q0 + u * (int)blockDim.x;
            if (sv[u] == 0) continue;
            acc[q] = 0ull;
            int lx, ly, lz;
            if constexpr (BX > 0) {
                const int rq = q / BX;
                lx = q - rq * BX;
                lz = (int)(((float)rq + 0.5f) * inv_by);
                ly = rq - lz * by;
            } else {
                lz = (int)(((float)q + 0.5f) * inv_bxy);
                const int rq = q - lz * (bx * by);
                ly = (int)(((float)rq + 0.5f) * inv_bx);
                lx = rq - ly * bx;
            }
            if constexpr (INSIDE) {
                dst[u] = fo + (lz * sz + ly * nxc + lx);
            } else {
                int gx = b0x + lx, gy = b0y + ly, gz = b0z + lz;
                if (AX.periodic) gx = gx < 0 ? gx + nxc : (gx >= nxc ? gx - nxc : gx);
                if (AY.periodic) gy = gy < 0 ? gy + nyc : (gy >= nyc ? gy - nyc : gy);
                if (AZ.periodic) gz = gz < 0 ? gz + nzc : (gz >= nzc ? gz - nzc : gz);
                if ((unsigned)gx >= (unsigned)nxc || (unsigned)gy >= (unsigned)nyc || (unsigned)gz >= (unsigned)nzc)
                    continue;
                dst[u] = f + field_index(g, c, gx, gy, gz);
            }
            add[u] = (float)((double)sv[u] * qscale);
        }
#pragma unroll
        for (int u = 0; u < kFlush; ++u) old[u] = dst[u] ? *dst[u] : 0.f;
#pragma unroll
        for (int u = 0; u < kFlush; ++u)
            if (dst[u]) *dst[u] = old[u] + add[u];
    }
}

// Fixed-point scale of a tile and component from the largest finite |c_l F_l|
// of its rows (written with c_l F_l by the build, or k_spread_coef): with
// |phi_k| <= 4 every scaled contribution stays below 2^30 (converted to int32,
// summed in int64), |c_l F_l| is scaled below 2^28, and the quantum is 2^-30
// of 4 max |c_l F_l| over the tile.  A non-finite c_l F_l is left out of the
// maximum and fails the range test of accumulate_rows.
struct TileScale {
    float scale;
    double quantum;
};
__device__ __forceinline__ TileScale tile_scale(uint32_t tmax_bits)
{
    const float fm = __uint_as_float(tmax_bits);
    int ebits = 0;
    frexpf(fm, &ebits);                    // fm < 2^ebits
    const int S = min(28 - ebits, 126);
    return {fm > 0.f ? ldexpf(1.0f, S) : 0.0f, ldexp(1.0, -S)};
}

// Adds the contributions of component c of the rows beg .. end of a tile into
// its box acc (64-bit fixed point), whose first node is (b0x, b0y, b0z); all
// threads of the workgroup take part.
template <bool SORTED, int NF, int BX>
__device__ __forceinline__ void
accumulate_rows(const Grid &g, int c, uint32_t beg, uint32_t end, int by, int bz, int b0x, int b0y, int b0z,
                float scale_f,
                const uint32_t *__restrict__ home, const float *__restrict__ phi, const float *__restrict__ cf,
                int64_t cf_stride, const uint32_t *__restrict__ entries, const float *__restrict__ coef,
                const Weight &W, unsigned long long *acc, ErrWord *err)
{
    const Axis &AX = g.ax[0], &AY = g.ax[1], &AZ = g.ax[2];
    const int bx = BX > 0 ? BX : g.box[0];
    const int nxc = g.dims[c][0], nyc = g.dims[c][1], nzc = g.dims[c][2];
    const float lim = 1073741824.0f;       // 2^30
    // Neighbouring rows mostly come from neighbouring markers, whose supports
    // share nodes: with 64 consecutive rows in a wavefront its atomics meet on
    // the same addresses, which LDS serves one after another (18 cycles an
    // instruction where distinct banks take 9 to 13).  Compact rows are
    // therefore dealt out in turn to the groups of 16 lanes that LDS takes
    // together.  Whole steps, consecutive / dealt out to the wavefronts / to
    // groups of 16: 1000 ellipsoids in 512^3 436 / 423 / 416 us, 2000 spheres in
    // the 512 x 512 x 768 channel 901 / 876 / 864, 22.4e6 markers in 1024^3
    // 4634 / 4563 / 4525.  Full rows are read as 27 words of 64 consecutive
    // rows, of which every wavefront would then use a part of each line: they
    // stay consecutive (509 us, dealt out 522 to 582, permuted within a
    // wavefront no change).
    const uint32_t e0 = NF > 0 ? (threadIdx.x & 15u) * (blockDim.x >> 4) + (threadIdx.x >> 4) : threadIdx.x;
    for (uint32_t e = beg + e0; e < end; e += blockDim.x) {
        // tile order: the row is the entry, so no load waits for the
        // marker index (read on the error path only)
        const int64_t row = SORTED ? (int64_t)e : (int64_t)entries[e];
        int hi, hj, hk;
        unpack_home(home[home_at(row, c)], hi, hj, hk);
        float cfv;
        float ph[kNe];
        if constexpr (NF == 0) {
            cfv = cf[c * cf_stride + row];
            const float *p = phi + phi_at(row, c);
    #pragma unroll
            for (int k = 0; k < kNe; ++k) ph[k] = p[k * kLanes];
        } else {
            // the compact row and c_l F_l in two or four 16-byte loads
            float cfr[kCoefStride<NF>];
    #pragma unroll
            for (int q = 0; q < kCoefStride<NF> / 4; ++q) {
                const f32x4 t =
                    *reinterpret_cast<const f32x4 *>(coef + coef_word(row, c, kCoefStride<NF>, q));
                cfr[4 * q] = t.x; cfr[4 * q + 1] = t.y; cfr[4 * q + 2] = t.z; cfr[4 * q + 3] = t.w;
            }
            cfv = cfr[NF];
            // evaluated for every row (all loads issue at once); a row the
            // build solved in FP64 has a NaN gamma_0 and its stored phi is
            // read instead, under a wavefront-wide test
            float sv[3][3], wv[3][3];
    #pragma unroll
            for (int d = 0; d < 3; ++d) {
                if constexpr (NF == 7) {
                    sv[d][1] = cfr[4 + d];
                    sv[d][0] = sv[d][1] - 1.0f;
                    sv[d][2] = sv[d][1] + 1.0f;
                } else {
    #pragma unroll
                    for (int a = 0; a < 3; ++a) sv[d][a] = cfr[4 + 3 * d + a];
                }
    #pragma unroll
                for (int a = 0; a < 3; ++a) wv[d][a] = weight1(W, sv[d][a]);
            }
            phi_from_gamma(wv, sv, cfr, ph);
            const bool stored = cfr[0] != cfr[0];
            if (__any(stored)) {
                if (stored) {
                    const float *p = phi + phi_at(row, c);
    #pragma unroll
                    for (int k = 0; k < kNe; ++k) ph[k] = p[k * kLanes];
                }
            }
        }
        int ix[3], iy[3], iz[3];
        bool inbox = true;
        if constexpr (BX > 0) {
            // the support's first node on each axis; the others follow it
            ix[0] = box_local(AX, g.ntile[0], nxc, b0x, nb_index(hi, -1, nxc, AX.periodic));
            iy[0] = box_local(AY, g.ntile[1], nyc, b0y, nb_index(hj, -1, nyc, AY.periodic));
            iz[0] = box_local(AZ, g.ntile[2], nzc, b0z, nb_index(hk, -1, nzc, AZ.periodic));
            inbox = (unsigned)ix[0] <= (unsigned)(BX - 3) && (unsigned)iy[0] <= (unsigned)(by - 3) &&
                    (unsigned)iz[0] <= (unsigned)(bz - 3);
        } else {
    #pragma unroll
            for (int a = 0; a < 3; ++a) {
                ix[a] = box_local(AX, g.ntile[0], nxc, b0x, nb_index(hi, a - 1, nxc, AX.periodic));
                iy[a] = box_local(AY, g.ntile[1], nyc, b0y, nb_index(hj, a - 1, nyc, AY.periodic));
                iz[a] = box_local(AZ, g.ntile[2], nzc, b0z, nb_index(hk, a - 1, nzc, AZ.periodic));
                inbox = inbox && (unsigned)ix[a] < (unsigned)bx && (unsigned)iy[a] < (unsigned)by &&
                        (unsigned)iz[a] < (unsigned)bz;
            }
        }
        if (!inbox) {           // cannot happen for a home written by the build
            raise_error(err, SORTED ? (int64_t)entries[e] : row, MLS_E_RANGE);
            continue;
        }
        // c_l F_l (eq. 8), pre-scaled
        const float vsc = cfv * scale_f;
        // Rounding is monotonic, so |phi_k vsc| <= max_k |phi_k| |vsc| for
        // every k, with equality at the largest: one comparison bounds all
        // 27 scaled contributions.  A NaN or infinity in the force or the
        // coefficient reaches vsc and fails it too.  Sorted rows hold the
        // library's own shape functions (finite for a usable support);
        // a caller's phi is checked here.
        float pm = 0.f;
    #pragma unroll
        for (int k = 0; k < kNe; ++k) pm = fmaxf(pm, fabsf(ph[k]));
        if constexpr (!SORTED) {
            // caller-provided phi: a NaN or infinite value fails through
            // the sum (fmaxf above ignores a NaN operand); c_l of a grid
            // with equal widths does not depend on phi
            float ps = 0.f;
    #pragma unroll
            for (int k = 0; k < kNe; ++k) ps += ph[k];
            if (!(fabsf(ps) <= 3.0e38f)) pm = __builtin_inff();
        }
        if (!(fabsf(vsc) * pm < lim)) {
            raise_error(err, SORTED ? (int64_t)entries[e] : row, MLS_E_RANGE);
            continue;
        }
        // truncation toward zero: within one quantum, the same on every run
        if constexpr (BX > 0) {
            // byte address of the first node per z layer; node (a, b) of a
            // layer sits (b BX + a) nodes further
            char *const a0 = reinterpret_cast<char *>(acc) +
                             (uint32_t)__umul24(__umul24(iz[0], by) + iy[0], BX) * 8u + (uint32_t)ix[0] * 8u;
            const uint32_t zs = (uint32_t)(by * BX) * 8u;
    #pragma unroll
            for (int k = 0; k < kNe; ++k) {
                const long long qv = (long long)(int)(ph[k] * vsc);
                char *const p = a0 + (k / 9) * zs + (((k / 3) % 3) * BX + (k % 3)) * 8;
                atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)qv);
            }
        } else {
            // byte offsets of the box rows (b, cz) and columns a
            uint32_t rowo[9], colo[3];
    #pragma unroll
            for (int a = 0; a < 3; ++a) colo[a] = (uint32_t)ix[a] * 8u;
    #pragma unroll
            for (int r = 0; r < 9; ++r) rowo[r] = (uint32_t)((iz[r / 3] * by + iy[r % 3]) * bx) * 8u;
    #pragma unroll
            for (int k = 0; k < kNe; ++k) {
                const long long qv = (long long)(int)(ph[k] * vsc);
                atomicAdd(reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(acc) +
                                                                 rowo[k / 3] + colo[k % 3]),
                          (unsigned long long)qv);
            }
        }
    }
}

// NF > 0 (sorted rows of a compact exact step): phi is evaluated from the
// row's compact transfer function (gamma and the support offsets, NF = 7 or
// 13 floats, see k_build_interp) with the build's own arithmetic, or read
// from phi for a row the build solved in FP64 (NaN gamma_0).
// c_l F_l of eq. 8 per component comes with a compact row (NF > 0), or from
// cf: by row in tile order (SORTED with full rows, the time step's fused
// builds write them) or by marker (a standalone call: k_spread_coef).  Per tile, the largest finite |c_l F_l|
// of its rows sets the fixed-point scale of each component.
// Workgroups of 128, 192 or 256 threads (tuned, at most kSpreadBlock).  A tile
// holds some 200 rows: fewer threads leave fewer lanes idle, pay cheaper
// barriers and keep more tiles in flight per compute unit; more finish a tile
// sooner when a colour has only a tile or two per workgroup.
// BX > 0: every axis has more than one tile and the box rows hold BX nodes.
// Then the 27 support nodes of a row are three consecutive nodes on each box
// axis, so one box address per row serves all 27 atomics (the others are
// immediate offsets) and the flush decodes box coordinates with it.
// BX = 0: any tiling (a short periodic axis kept whole wraps inside its box).
template <bool SORTED, int NF, int BX>
__global__ void __launch_bounds__(kSpreadBlock) __attribute__((amdgpu_waves_per_eu(SORTED ? 6 : 5)))
k_spread_colour(const Grid *__restrict__ gp, int colour, const uint32_t *__restrict__ home,
                const float *__restrict__ phi, const float *__restrict__ cf, int64_t cf_stride,
                float *__restrict__ fx, float *__restrict__ fy, float *__restrict__ fz,
                const uint32_t *__restrict__ off, const uint32_t *__restrict__ entries,
                const uint32_t *__restrict__ active, uint32_t *work, const float *__restrict__ coef, const Weight W,
                const uint32_t *__restrict__ tmax, int64_t tstride, ErrWord *err)
{
    const Grid &g = *gp;
    extern __shared__ unsigned long long acc[];     // the box of one component
    const Axis &AX = g.ax[0], &AY = g.ax[1], &AZ = g.ax[2];
    const int bx = BX > 0 ? BX : g.box[0];
    const float inv_bx = 1.0f / (float)bx;
    const int64_t abase = g.colour_base[colour];
    const uint32_t nact = (uint32_t)min((int64_t)work[colour], colour_end(g, colour) - abase);
    __shared__ int64_t unit_sh;
    // Work units of a launch: a colour with up to three tiles a workgroup is cut
    // into its (tile, component) pairs, so that a tile's three components run
    // side by side and the last round is short (2000 spheres in the channel,
    // 1.1 tiles a workgroup: 840 us a step, whole tiles 946); else a unit is a
    // whole tile (cut up to eight tiles a workgroup: 862).
    const uint32_t G = gridDim.x;
    const bool split = nact <= 3u * G;
    const uint32_t units = split ? 3u * nact : nact;
    // Workgroup b starts with unit b and ends there if the first round covers
    // all units; further units are claimed.  Atomics on one address are served
    // one after another (about 12 ns each), so with a single counter the
    // claims of 4096 workgroups alone took 60 us a launch: workgroups claim
    // from one of kShards counters on lines of their own, counter r handing
    // out the units G + r, G + r + kShards, ...
    uint32_t unit = blockIdx.x;
    if (unit >= units) return;
    // The box is cleared once here; afterwards every flush returns the nodes
    // it reads to zero, so each component and tile starts from a clear box.
    for (int q = threadIdx.x; q < bx * g.box[1] * g.box[2]; q += blockDim.x) acc[q] = 0ull;
    for (bool first = true;; first = false) {
        if (!first) {
            if (units <= G) break;
            lds_barrier();   // every thread has read unit_sh of the round before
            if (threadIdx.x == 0) {
                const uint32_t r = blockIdx.x % kShards;
                unit_sh = (int64_t)G + r + (int64_t)kShards * atomicAdd(&work[kCursor(colour, r)], 1u);
            }
            lds_barrier();
            if (unit_sh >= units) break;
            unit = (uint32_t)unit_sh;
        }
        const uint32_t slot = split ? unit / 3u : unit;
        const int c_beg = split ? (int)(unit - 3u * slot) : 0, c_end = split ? c_beg + 1 : 3;
        const int64_t t = active[abase + slot];
        if (t >= g.ntiles) break;
        const uint32_t beg = off[t], end = off[t + 1];
        const int tx = (int)(t % g.ntile[0]);
        const int ty = (int)((t / g.ntile[0]) % g.ntile[1]);
        const int tz = (int)(t / ((int64_t)g.ntile[0] * g.ntile[1]));
        // box origin: one node below the tile (a single-tile periodic axis keeps the whole axis)
        const int b0x = (AX.periodic && g.ntile[0] == 1) ? 0 : tx * AX.tile - 1;
        const int b0y = (AY.periodic && g.ntile[1] == 1) ? 0 : ty * AY.tile - 1;
        const int b0z = (AZ.periodic && g.ntile[2] == 1) ? 0 : tz * AZ.tile - 1;
        // one component at a time: a third of the LDS per workgroup, so more
        // workgroups fit a compute unit and tiles can be larger
#pragma unroll 1
        for (int c = c_beg; c < c_end; ++c) {
            lds_barrier();
            const TileScale ts = tile_scale(tmax[c * tstride + t]);
            const int nxc = g.dims[c][0], nyc = g.dims[c][1], nzc = g.dims[c][2];
            // The box of a component reaches tile + 3 nodes on the axis it is
            // face-staggered on and tile + 2 on the others (its homes are the
            // tile's cells there), so with homes of the build the last layer
            // of y or z is left out of the box, and the flush scans 1100 or
            // 1210 nodes instead of 1331 (tile edge 8).  Steps: fast-MLS of 1000
            // ellipsoids in 512^3 516 -> 501 us, spheres in the channel, exact
            // 864 -> 852 and learned 2317 -> 2270.  Homes from a caller may
            // reach further and keep the whole box.
            constexpr bool trim = SORTED && BX > 0;
            const int by = g.box[1] - (trim && c != 1 ? 1 : 0), bz = g.box[2] - (trim && c != 2 ? 1 : 0);
            const int bnodes = bx * by * bz;
            // box-local coordinates of a node index without integer division: with
            // fewer than 2^22 nodes, (q + 1/2) times the FP32 reciprocal of the divisor
            // stays within 1/2 of a quotient's interval from its floor
            const float inv_by = 1.0f / (float)by, inv_bxy = 1.0f / (float)(bx * by);
            accumulate_rows<SORTED, NF, BX>(g, c, beg, end, by, bz, b0x, b0y, b0z, ts.scale, home, phi, cf, cf_stride,
                                            entries, coef, W, acc, err);
            lds_barrier();
            // flush: the box nodes of a thread are read in batches of kFlush
            // before any is written back, so their loads overlap
            float *f = c == 0 ? fx : (c == 1 ? fy : fz);
            const double qscale = ts.quantum;
            // a box inside the component's grid on every axis (no wrap, no node
            // past a wall) addresses its nodes as offsets from its origin
            const bool inside = b0x >= 0 && b0y >= 0 && b0z >= 0 && b0x + bx <= nxc && b0y + by <= nyc &&
                                b0z + bz <= nzc;
            if (inside)
                flush_box<true, BX>(g, c, acc, bnodes, bx, by, b0x, b0y, b0z, nxc, nyc, nzc, inv_bx, inv_by, inv_bxy,
                                    qscale, f);
            else
                flush_box<false, BX>(g, c, acc, bnodes, bx, by, b0x, b0y, b0z, nxc, nyc, nzc, inv_bx, inv_by, inv_bxy,
                                     qscale, f);
        }
    }
}

// ---- spreading in two launches --------------------------------------------------
//
// With few tiles the 8 to 27 colour launches cost more than the work in them
// (a launch about 4.3 us, and each waits for its slowest tile).  Where
// spread_staged says so, every (tile, component) pair accumulates its box at once
// and stores it in the staging buffer, converted to FP32 as the flush converts it (k_spread_stage); then every node
// takes its additions from the up to eight boxes that hold it, one after
// another in the order of the tiles' colours (k_spread_merge): the same
// additions in the same order as with one launch per colour, bit for bit.
// Measured: spreading one sphere in 64^3 (8 colours) 83 -> 18 us, the whole
// step of 320 markers in 96 x 72 x 45 (18 colours) 96 -> 40 us.

// The non-empty tile of dense slot `slot` of all colour lists, in colour
// order; -1 past the last.  prefix (27 words of LDS) receives the number of
// tiles before each colour.  Every thread of the workgroup calls it.
__device__ __forceinline__ int64_t slot_tile(const Grid &g, uint32_t slot, const uint32_t *__restrict__ active,
                                             const uint32_t *__restrict__ work, uint32_t *prefix)
{
    const int lane = threadIdx.x & 63;
    const int used = g.ncol[0] * g.ncol[1] * g.ncol[2];
    const uint32_t v = lane < used ? (uint32_t)min((int64_t)work[lane], colour_end(g, lane) - g.colour_base[lane]) : 0u;
    uint32_t x = v;
    for (int o = 1; o < 32; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (threadIdx.x < 27) prefix[threadIdx.x] = x - v;
    const unsigned long long after = __ballot(lane < used && slot < x);
    if (!after) return -1;
    const int col = __ffsll((long long)after) - 1;
    const uint32_t before = __shfl(x - v, col);
    const int64_t t = active[g.colour_base[col] + (slot - before)];
    return t < g.ntiles ? t : -1;
}

struct TilePos {
    int x, y, z;
};
__device__ __forceinline__ TilePos tile_pos_of(const Grid &g, int64_t t)
{
    const uint32_t tu = (uint32_t)t, nx = (uint32_t)g.ntile[0], ny = (uint32_t)g.ntile[1];
    const uint32_t row = tu / nx;
    return {(int)(tu - row * nx), (int)(row % ny), (int)(row / ny)};
}

// First node of a tile's box along axis d: one below the tile (a single-tile
// periodic axis keeps the whole axis).
__device__ __forceinline__ int box_origin(const Grid &g, int d, int t)
{
    return (g.ax[d].periodic && g.ntile[d] == 1) ? 0 : t * g.ax[d].tile - 1;
}

template <bool SORTED, int NF, int BX>
__global__ void __launch_bounds__(kSpreadBlock)
k_spread_stage(const Grid *__restrict__ gp, const uint32_t *__restrict__ home, const float *__restrict__ phi,
               const float *__restrict__ cf, int64_t cf_stride, const uint32_t *__restrict__ off,
               const uint32_t *__restrict__ entries, const uint32_t *__restrict__ active,
               const uint32_t *__restrict__ work, const float *__restrict__ coef, const Weight W,
               const uint32_t *__restrict__ tmax, int64_t tstride, float *__restrict__ stage, ErrWord *err)
{
    const Grid &g = *gp;
    extern __shared__ unsigned long long acc[];
    __shared__ uint32_t prefix[27];
    const int bnodes = (BX > 0 ? BX : g.box[0]) * g.box[1] * g.box[2];
    const int c = (int)(blockIdx.x % 3u);
    const int64_t t = slot_tile(g, blockIdx.x / 3u, active, work, prefix);
    if (t < 0) return;
    const TilePos p = tile_pos_of(g, t);
    const uint32_t beg = off[t], end = off[t + 1];
    const TileScale ts = tile_scale(tmax[c * tstride + t]);
    for (int q = threadIdx.x; q < bnodes; q += blockDim.x) acc[q] = 0ull;
    __syncthreads();
    accumulate_rows<SORTED, NF, BX>(g, c, beg, end, g.box[1], g.box[2], box_origin(g, 0, p.x), box_origin(g, 1, p.y),
                                    box_origin(g, 2, p.z), ts.scale, home, phi, cf, cf_stride, entries, coef, W, acc,
                                    err);
    __syncthreads();
    float *out = stage + (int64_t)blockIdx.x * bnodes;
    for (int q = threadIdx.x; q < bnodes; q += blockDim.x)
        out[q] = (float)((double)(long long)acc[q] * ts.quantum);
}

// Neighbour of tile index i along axis d in direction s (-1, +1) whose box
// shares nodes with it; -1 if there is none.
__device__ __forceinline__ int tile_neighbour(const Grid &g, int d, int i, int s)
{
    const int m = g.ntile[d];
    if (m == 1) return -1;
    const int j = i + s;
    if (g.ax[d].periodic) return j < 0 ? m - 1 : (j >= m ? 0 : j);
    return j >= 0 && j < m ? j : -1;
}

// A workgroup of 1024 threads takes a box of eight-cell tiles in two rounds (of
// 256: six, 23 us on one sphere instead of 10).
constexpr int kMergeBlock = 1024;
__global__ void __launch_bounds__(kMergeBlock)
k_spread_merge(const Grid *__restrict__ gp, const uint32_t *__restrict__ off, const uint32_t *__restrict__ active,
               const uint32_t *__restrict__ work, const uint32_t *__restrict__ tile_slot,
               const float *__restrict__ stage, float *__restrict__ fx, float *__restrict__ fy,
               float *__restrict__ fz)
{
    const Grid &g = *gp;
    __shared__ uint32_t prefix[27];
    __shared__ int64_t nb_base[27];   // staged box of each neighbour (dx, dy, dz), -1: no markers there
    const int bx = g.box[0], by = g.box[1], bz = g.box[2], bnodes = bx * by * bz;
    const int c = (int)(blockIdx.x % 3u);
    const int64_t t = slot_tile(g, blockIdx.x / 3u, active, work, prefix);
    if (t < 0) return;
    const TilePos tp = tile_pos_of(g, t);
    const int ti[3] = {tp.x, tp.y, tp.z};
    __syncthreads();
    if (threadIdx.x < 27) {
        const int dd[3] = {(int)threadIdx.x % 3 - 1, (int)threadIdx.x / 3 % 3 - 1, (int)threadIdx.x / 9 - 1};
        int q[3];
        bool there = true;
        for (int d = 0; d < 3; ++d) {
            q[d] = dd[d] ? tile_neighbour(g, d, ti[d], dd[d]) : ti[d];
            there = there && q[d] >= 0;
        }
        int64_t base = -1;
        if (there) {
            const int64_t u = ((int64_t)q[2] * g.ntile[1] + q[1]) * g.ntile[0] + q[0];
            if (off[u + 1] > off[u]) {
                const int col = axis_colour(g, 0, q[0]) +
                                g.ncol[0] * (axis_colour(g, 1, q[1]) + g.ncol[1] * axis_colour(g, 2, q[2]));
                base = ((int64_t)(prefix[col] + tile_slot[u]) * 3 + c) * bnodes;
            }
        }
        nb_base[threadIdx.x] = base;
    }
    __syncthreads();
    // per axis: which neighbours exist, and whether their colour comes first
    bool left[3], right[3], left_first[3], right_first[3];
    int b0[3], nn[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int l = tile_neighbour(g, d, ti[d], -1), r = tile_neighbour(g, d, ti[d], 1);
        left[d] = l >= 0;
        right[d] = r >= 0;
        left_first[d] = left[d] && axis_colour(g, d, l) < axis_colour(g, d, ti[d]);
        right_first[d] = right[d] && axis_colour(g, d, r) < axis_colour(g, d, ti[d]);
        b0[d] = box_origin(g, d, ti[d]);
        nn[d] = g.dims[c][d];
    }
    float *const f = c == 0 ? fx : (c == 1 ? fy : fz);
    const float inv_bx = 1.0f / (float)bx, inv_bxy = 1.0f / (float)(bx * by);   // as in flush_box
    for (int q = threadIdx.x; q < bnodes; q += blockDim.x) {
        const int lz = (int)(((float)q + 0.5f) * inv_bxy);
        const int rq = q - lz * (bx * by);
        const int ly = (int)(((float)rq + 0.5f) * inv_bx);
        const int lx = rq - ly * bx;
        const int l3[3] = {lx, ly, lz};
        // the neighbour along each axis whose box holds this node too (0:
        // none), the colour order of the two, and the node's index there
        int first[3], second[3], gi[3];
        bool in = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int zone = left[d] && l3[d] < 3 ? -1 : (right[d] && l3[d] >= g.ax[d].tile ? 1 : 0);
            const bool before = zone < 0 ? left_first[d] : (zone > 0 && right_first[d]);
            first[d] = before ? zone : 0;
            second[d] = before ? 0 : zone;
            int i = b0[d] + l3[d];
            if (g.ax[d].periodic) i = i < 0 ? i + nn[d] : (i >= nn[d] ? i - nn[d] : i);
            in = in && (unsigned)i < (unsigned)nn[d];
            gi[d] = i;
        }
        if (!in) continue;
        // The box of the first colour that holds the node adds for all: its
        // loads from the (up to eight) boxes are issued together.
        int64_t at[8];
        bool mine = true, found = false;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int dx = k & 1 ? second[0] : first[0], dy = k & 2 ? second[1] : first[1],
                      dz = k & 4 ? second[2] : first[2];
            // a node with no neighbour along an axis is visited once
            const bool twice = ((k & 1) && !(first[0] | second[0])) || ((k & 2) && !(first[1] | second[1])) ||
                               ((k & 4) && !(first[2] | second[2]));
            const int64_t base = twice ? -1 : nb_base[(dz + 1) * 9 + (dy + 1) * 3 + dx + 1];
            if (!found && base >= 0) {
                mine = (dx | dy | dz) == 0;
                found = true;
            }
            at[k] = base < 0 ? -1 : base + ((lz - dz * g.ax[2].tile) * by + ly - dy * g.ax[1].tile) * bx + lx -
                                        dx * g.ax[0].tile;
        }
        if (!mine) continue;
        float v[8];
        bool any = false;
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = at[k] >= 0 ? stage[at[k]] : 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) any = any || v[k] != 0.f;
        if (!any) continue;
        float *dst = f + field_index(g, c, gi[0], gi[1], gi[2]);
        float sum = *dst;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (v[k] != 0.f) sum += v[k];
        *dst = sum;
    }
}

// c_l F_l (eq. 8) by marker for a standalone spreading call, from the stored
// shape functions, homes, areas and forces.  A marker whose homes are not
// usable gets 0 (the binning leaves it out).
// It also records the largest finite |c_l F_l| per tile (marker_tile from
// the binning) and component in tmax.
__global__ void __launch_bounds__(kBlock)
k_spread_coef(const Grid *__restrict__ gp, int64_t n, const uint32_t *__restrict__ home,
              const float *__restrict__ phi, const float *__restrict__ area, const float *__restrict__ Fx,
              const float *__restrict__ Fy, const float *__restrict__ Fz, float *__restrict__ cf, int64_t cf_stride,
              const uint32_t *__restrict__ marker_tile, uint32_t *__restrict__ tmax, int64_t tstride)
{
    const Grid &g = *gp;
    // wave-uniform loop bound: every lane takes part in the per-tile maxima
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t base = xcd_block() * blockDim.x + (threadIdx.x & ~63); base < n; base += stride) {
        const int64_t l = base + (threadIdx.x & 63);
        const bool in = l < n;
        const float a = in ? area[l] : 0.f;
        const uint32_t tl = in ? marker_tile[l] : (uint32_t)g.ntiles;
        const int64_t key = tl < (uint32_t)g.ntiles ? (int64_t)tl : -1;
#pragma unroll 1
        for (int c = 0; c < 3; ++c) {
            int hi = 0, hj = 0, hk = 0;
            if (in) unpack_home(home[home_at(l, c)], hi, hj, hk);
            float v = 0.0f;
            if (in && home_ok(g, c, hi, hj, hk)) {
                const float Fc = c == 0 ? Fx[l] : (c == 1 ? Fy[l] : Fz[l]);
                if (g.inv_cw2 > 0.f) {
                    // equal control-volume widths w: c_l = A_l / w^2 whatever
                    // the shape functions (a non-finite phi is caught by the
                    // tile kernel, which reads phi anyway)
                    v = a * Fc * g.inv_cw2;
                } else {
                    const float *p = phi + phi_at(l, c);
                    float ph[kNe];
#pragma unroll
                    for (int k = 0; k < kNe; ++k) ph[k] = p[k * kLanes];
                    v = eq8_coef(g, c, hi, hj, hk, ph, a * Fc);
                }
            }
            if (in) cf[c * cf_stride + l] = v;
            wave_key_max(tmax + c * tstride, key, finite_abs(v));
        }
    }
}

int grid_for(int64_t work, int cu)
{
    int64_t b = (work + kBlock - 1) / kBlock;
    const int64_t cap = (int64_t)cu * 32;
    if (b > cap) b = cap;
    return (int)(b < 1 ? 1 : b);
}

}  // namespace

size_t spread_lds_bytes(const Ctx &c)
{
    return (size_t)c.g.box[0] * c.g.box[1] * c.g.box[2] * sizeof(unsigned long long);
}

// Floats of the staged boxes of `tiles` tiles, three components each.
int64_t stage_floats(const Grid &g, int64_t tiles)
{
    return tiles * 3 * g.box[0] * g.box[1] * g.box[2];
}

// Whether n markers are spread in two launches through the staging buffer
// rather than in one per colour.  The boxes of all tiles that can hold markers
// have to fit it.  Then a colour launch costs about 10 us, whatever is in it;
// the staged route costs 0.08 us a tile with markers (its three boxes go through
// memory) and 4.4 ns a tile that could have some (its workgroups start and find
// none), so the line lies at 150 tiles a colour, 18 of the latter for one.  How
// many tiles hold markers the host does not know; it takes 96 markers a tile of
// 8^3 cells and 1.5 times the 2/3 power of the cells in general, as for closed
// surfaces of markers 0.8 cells apart (70 for the smallest particles, 150 for
// large ones).  Whole exact steps, staged / colours, us: 8 colours, particles of
// 320 markers in 128^3, 32000 markers 97 / 108, 64000 121 / 113, 128000
// 164 / 127; of 1280 64000 106 / 117, 128000 139 / 136; of 5120 102400 127 / 126;
// packed, all 1728 tiles of 96^3 186 / 142, all 4096 of 128^3 378 / 207; 12
// colours, 141440 markers 152 / 170; 27 colours, 134400 140 / 272.  4-cell tiles
// in 96^3: 4000 markers 76 / 96, 16000 148 / 96.  (Markers scattered singly over
// the box fill more tiles than that: 16000 in 128^3 320 / 139.)
bool spread_staged(const Grid &g, int64_t n)
{
    const int colours = g.ncol[0] * g.ncol[1] * g.ncol[2];
    const int64_t most = std::min(g.ntiles, n);
    if (colours <= 2 || stage_floats(g, most) > kStageBytes / (int64_t)sizeof(float)) return false;
    const double cells = (double)g.ax[0].tile * g.ax[1].tile * g.ax[2].tile;
    const double full = std::min((double)most, (double)n / (1.5 * std::cbrt(cells * cells)));
    return full + (double)most / 18.0 <= 150.0 * colours;
}

// Device buffers of one spreading call: the context's own (mls_spread, the
// time step) or carved out of the library's fixed array (mls_spread_noalloc).
struct SpreadScratch {
    uint32_t *tile_count, *tile_off, *tile_cursor, *tile_active, *block_sums, *work, *tile_fmax, *marker_tile,
        *entries;
    float *cf;
    int64_t cf_stride;
    uint32_t *tile_slot;   // NULL: no staging (mls_spread_noalloc)
    float *stage;
    int64_t stage_floats;
};

static SpreadScratch ctx_scratch(Ctx &c)
{
    return {c.tile_count, c.tile_off, c.tile_cursor, c.tile_active, c.block_sums, c.work, c.tile_fmax,
            c.marker_tile, c.entries, c.cf_rows, c.cf_stride, c.tile_slot, c.stage, c.stage_floats};
}

template <bool SORTED, int NF, int BX>
static hipError_t launch_tiles_bx(Ctx &c, const SpreadScratch &sc, int64_t n, const uint32_t *home,
                                  const float *phi, float *fx, float *fy, float *fz, hipStream_t s, bool timed)
{
    const size_t lds = spread_lds_bytes(c);
    const int64_t tiles = std::min(c.g.ntiles, n);
    const bool staged = sc.tile_slot && spread_staged(c.g, n) && stage_floats(c.g, tiles) <= sc.stage_floats;
    if (lds > 64 * 1024) {
        const void *k = staged ? (const void *)k_spread_stage<SORTED, NF, BX>
                               : (const void *)k_spread_colour<SORTED, NF, BX>;
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    TimedLaunch tt(c, timed ? MLS_K_SPREAD_TILES : -1, s);
    if (staged) {
        const dim3 grid((unsigned)(3 * tiles));
        hipLaunchKernelGGL((k_spread_stage<SORTED, NF, BX>), grid, dim3(kSpreadBlock), lds, s, c.d_grid, home, phi,
                           sc.cf, sc.cf_stride, sc.tile_off, sc.entries, sc.tile_active, sc.work,
                           NF ? c.coef_rows : nullptr, c.w, sc.tile_fmax, c.g.ntiles + 1, sc.stage, c.err);
        hipLaunchKernelGGL(k_spread_merge, grid, dim3(kMergeBlock), 0, s, c.d_grid, sc.tile_off, sc.tile_active, sc.work,
                           sc.tile_slot, sc.stage, fx, fy, fz);
        return hipGetLastError();
    }
    for (int col = 0; col < 27; ++col) {
        if (c.colour_tiles[col] == 0) continue;
        // at most one workgroup per (tile, component) pair
        const int64_t most = 3 * std::min(c.colour_tiles[col], n);
        const unsigned persist = (unsigned)std::min((int64_t)c.cu_count * c.spread_blocks_per_cu, most);
        hipLaunchKernelGGL((k_spread_colour<SORTED, NF, BX>), dim3(persist), dim3(c.spread_threads), lds, s, c.d_grid,
                           col, home, phi, sc.cf, sc.cf_stride, fx, fy, fz, sc.tile_off, sc.entries, sc.tile_active,
                           sc.work, NF ? c.coef_rows : nullptr, c.w, sc.tile_fmax, c.g.ntiles + 1, c.err);
    }
    return hipGetLastError();
}

// The box-row length the tile kernels are specialised for: the boxes of tile
// edges 4, 6, 8, 10, 12 and 16 on grids whose every axis has several tiles;
// 0 (the general kernel) otherwise.
static int box_row_template(const Ctx &c)
{
    const Grid &g = c.g;
    if (g.ntile[0] < 2 || g.ntile[1] < 2 || g.ntile[2] < 2) return 0;
    switch (g.box[0]) {
    case 7: case 9: case 11: case 13: case 15: case 19: return g.box[0];
    default: return 0;
    }
}

template <bool SORTED, int NF>
static hipError_t launch_tiles(Ctx &c, const SpreadScratch &sc, int64_t n, const uint32_t *home, const float *phi,
                               float *fx, float *fy, float *fz, hipStream_t s, bool timed = true)
{
    switch (box_row_template(c)) {
    case 7: return launch_tiles_bx<SORTED, NF, 7>(c, sc, n, home, phi, fx, fy, fz, s, timed);
    case 9: return launch_tiles_bx<SORTED, NF, 9>(c, sc, n, home, phi, fx, fy, fz, s, timed);
    case 11: return launch_tiles_bx<SORTED, NF, 11>(c, sc, n, home, phi, fx, fy, fz, s, timed);
    case 13: return launch_tiles_bx<SORTED, NF, 13>(c, sc, n, home, phi, fx, fy, fz, s, timed);
    case 15: return launch_tiles_bx<SORTED, NF, 15>(c, sc, n, home, phi, fx, fy, fz, s, timed);
    case 19: return launch_tiles_bx<SORTED, NF, 19>(c, sc, n, home, phi, fx, fy, fz, s, timed);
    default: return launch_tiles_bx<SORTED, NF, 0>(c, sc, n, home, phi, fx, fy, fz, s, timed);
    }
}

hipError_t launch_interp(const Ctx &c, int64_t n, const uint32_t *home, const float *phi,
                         const float *u, const float *v, const float *w,
                         float *U, float *V, float *W, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    int64_t blocks = (n + kBlock - 1) / kBlock;
    blocks = round_up8(std::min(blocks, (int64_t)c.cu_count * c.interp_blocks_per_cu));
    hipLaunchKernelGGL(k_interp, dim3((unsigned)blocks), dim3(kBlock), 0, s, c.d_grid, n, home, phi,
                       u, v, w, U, V, W, c.err);
    return hipGetLastError();
}

// Clears the nt tile counts and the colour lists of a call (and the count of
// the FP64 queue, if given).
static void launch_clear(const Ctx &c, const SpreadScratch &sc, int64_t nt, uint32_t *queue, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear, dim3(grid_for(nt + kWorkWords, c.cu_count)), dim3(kBlock), 0, s, sc.tile_count, nt,
                       sc.work, queue);
}

// Offsets of nt tiles from their counts, with the colour lists (k_scan_final).
static void launch_scan(const Ctx &c, const SpreadScratch &sc, int64_t nt, hipStream_t s)
{
    const int64_t nb = (nt + kScanChunk - 1) / kScanChunk;
    ScanFrom from = ScanFrom::Counts;
    if (nb > kScanDirect) {
        hipLaunchKernelGGL(k_scan_partials, dim3((unsigned)nb), dim3(kBlock), 0, s, sc.tile_count, nt, sc.block_sums);
        from = ScanFrom::Sums;
    }
    if (nb > kScanAdd) {
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kBlock), 0, s, sc.block_sums, nb);
        from = ScanFrom::Scanned;
    }
    hipLaunchKernelGGL(k_scan_final, dim3((unsigned)nb), dim3(kBlock), 0, s, c.d_grid, sc.tile_count, nt,
                       sc.block_sums, from, sc.tile_off, sc.tile_cursor, sc.work, sc.tile_active, sc.tile_slot,
                       sc.tile_fmax, c.g.ntiles + 1);
}

// The standalone spreading on the buffers sc: binning from the homes, c_l F_l
// and the per-tile maxima by marker, then the coloured tile launches.  timed:
// per-kernel timing marks (they may create HIP events).
static hipError_t launch_spread_with(Ctx &c, const SpreadScratch &sc, int64_t n, const uint32_t *home,
                                     const float *phi, const float *area, const float *Fx, const float *Fy,
                                     const float *Fz, float *fx, float *fy, float *fz, hipStream_t s, bool timed)
{
    if (n == 0) return hipSuccess;
    const int64_t nt = c.g.ntiles;
    {
        TimedLaunch tb(c, timed ? MLS_K_SPREAD_BIN : -1, s);
        launch_clear(c, sc, nt, nullptr, s);
        const int gbin = grid_for(n, c.cu_count);
        hipLaunchKernelGGL(k_bin<false>, dim3(gbin), dim3(kBlock), 0, s, c.d_grid, n, home, sc.tile_count,
                           sc.tile_cursor, sc.entries, sc.marker_tile, c.err);
        launch_scan(c, sc, nt, s);
        hipLaunchKernelGGL(k_bin<true>, dim3(gbin), dim3(kBlock), 0, s, c.d_grid, n, home, sc.tile_count,
                           sc.tile_cursor, sc.entries, sc.marker_tile, c.err);
        hipLaunchKernelGGL(k_spread_coef, dim3((unsigned)round_up8(grid_for(n, c.cu_count))), dim3(kBlock), 0, s,
                           c.d_grid, n, home, phi, area, Fx, Fy, Fz, sc.cf, sc.cf_stride, sc.marker_tile,
                           sc.tile_fmax, nt + 1);
    }
    return launch_tiles<false, 0>(c, sc, n, home, phi, fx, fy, fz, s, timed);
}

hipError_t launch_spread(Ctx &c, int64_t n, const uint32_t *home, const float *phi,
                         const float *area, const float *Fx, const float *Fy, const float *Fz,
                         float *fx, float *fy, float *fz, hipStream_t s)
{
    return launch_spread_with(c, ctx_scratch(c), n, home, phi, area, Fx, Fy, Fz, fx, fy, fz, s, true);
}

hipError_t launch_sort_positions(Ctx &c, int64_t n, const float *x, const float *y, const float *z, hipStream_t s,
                                 float *jx, float *jy, float *jz, float jitter, uint64_t seed, bool advance)
{
    const float amp2 = jx ? 2.0f * jitter : 0.0f;
    if (n == 0) return hipSuccess;
    const int64_t nt = c.g.ntiles + 1;   // tiles and the bucket of markers without a valid support
    const SpreadScratch sc = ctx_scratch(c);
    TimedLaunch tb(c, MLS_K_SPREAD_BIN, s);
    launch_clear(c, sc, nt, c.step_nf ? c.route_queue : nullptr, s);
    hipLaunchKernelGGL(k_bin_pos<false>, dim3(grid_for(n, c.cu_count)), dim3(kBlock), 0, s, c.d_grid, n, x, y, z,
                       c.tile_count, c.tile_cursor, c.entries, c.marker_tile, jx, jy, jz, amp2, seed, c.step_ctr);
    launch_scan(c, sc, nt, s);
    hipLaunchKernelGGL(k_bin_pos<true>, dim3(grid_for(n, c.cu_count)), dim3(kBlock), 0, s, c.d_grid, n, x, y, z,
                       c.tile_count, c.tile_cursor, c.entries, c.marker_tile, nullptr, nullptr, nullptr, 0.0f,
                       (uint64_t)0, advance ? c.step_ctr : nullptr);
    return hipGetLastError();
}

hipError_t launch_spread_sorted(Ctx &c, int64_t n, const uint32_t *home, const float *phi, float *fx, float *fy,
                                float *fz, hipStream_t s, bool again)
{
    if (n == 0) return hipSuccess;
    const SpreadScratch sc = ctx_scratch(c);
    // the sort clears the claim cursors; a further spreading of it clears them here
    if (again)
        hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(kBlock), 0, s, sc.work + kCursor(0, 0),
                           (int64_t)(kWorkWords - kCursor(0, 0)));
    if (c.step_nf == 7) return launch_tiles<true, 7>(c, sc, n, home, phi, fx, fy, fz, s);
    if (c.step_nf == 13) return launch_tiles<true, 13>(c, sc, n, home, phi, fx, fy, fz, s);
    return launch_tiles<true, 0>(c, sc, n, home, phi, fx, fy, fz, s);
}


// ---- allocation-free spreading --------------------------------------------
//
// The scratch of mls_spread_noalloc lives in one fixed array in the library's
// code object.  Each GPU the library runs on holds its own copy, allocated
// when the code object is loaded on that device and kept until the process
// ends.  In host code the array's name only stands for the symbol: its
// address on a device comes from hipGetSymbolAddress, taken once per device
// by noalloc_setup (called from mls_ctx_create, with that device current) and
// kept in noalloc_ptr[]; every use on the host goes through that pointer.

static __device__ __align__(256) unsigned char scratch[MLS_SPREAD_NOALLOC_BYTES + kWorkWords * 4];

namespace {
constexpr int kMaxDevices = 64;
void *noalloc_ptr[kMaxDevices] = {};
std::mutex noalloc_mu;

// Carves the buffers of a standalone spreading of n markers over nt tiles out
// of base (or only measures them when base is NULL); returns the bytes needed.
size_t carve(int64_t nt, int64_t n, unsigned char *base, SpreadScratch &sc)
{
    size_t off = 0;
    auto take = [&](size_t bytes) -> void * {
        void *p = base ? base + off : nullptr;
        off += (bytes + 255) & ~(size_t)255;
        return p;
    };
    const int64_t nb = (nt + 1 + kScanChunk - 1) / kScanChunk;
    const int64_t stride = (n + 63) / 64 * 64;
    sc.tile_count = (uint32_t *)take((size_t)(nt + 1) * 4);
    sc.tile_off = (uint32_t *)take((size_t)(nt + 2) * 4);
    sc.tile_cursor = (uint32_t *)take((size_t)(nt + 1) * 4);
    sc.tile_active = (uint32_t *)take((size_t)nt * 4);
    sc.block_sums = (uint32_t *)take((size_t)(nb + 1) * 4);
    take(128 * 4);   // part of the documented size; the list sizes and cursors lie behind it
    sc.work = base ? (uint32_t *)(base + MLS_SPREAD_NOALLOC_BYTES) : nullptr;
    sc.tile_fmax = (uint32_t *)take((size_t)3 * (nt + 1) * 4);
    sc.marker_tile = (uint32_t *)take((size_t)n * 4);
    sc.entries = (uint32_t *)take((size_t)n * 4);
    sc.cf = (float *)take((size_t)3 * stride * 4);
    sc.cf_stride = stride;
    return off;
}
}  // namespace

hipError_t noalloc_setup(int device)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(noalloc_mu);
    if (noalloc_ptr[device]) return hipSuccess;
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    noalloc_ptr[device] = p;
    return hipSuccess;
}

size_t noalloc_bytes(const Ctx &c, int64_t n)
{
    SpreadScratch sc = {};
    return carve(c.g.ntiles, n, nullptr, sc);
}

hipError_t launch_spread_noalloc(Ctx &c, int64_t n, const uint32_t *home, const float *phi, const float *area,
                                 const float *Fx, const float *Fy, const float *Fz, float *fx, float *fy, float *fz,
                                 hipStream_t s)
{
    void *base = nullptr;
    {
        std::lock_guard<std::mutex> lock(noalloc_mu);
        if (c.device >= 0 && c.device < kMaxDevices) base = noalloc_ptr[c.device];
    }
    if (!base) return hipErrorInvalidDevicePointer;
    SpreadScratch sc = {};
    carve(c.g.ntiles, n, static_cast<unsigned char *>(base), sc);
    return launch_spread_with(c, sc, n, home, phi, area, Fx, Fy, Fz, fx, fy, fz, s, false);
}

}  // namespace mls
