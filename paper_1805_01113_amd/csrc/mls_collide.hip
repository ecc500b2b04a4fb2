// Coarse-grained collision detection (Sec. 4): an integer array over the
// Eulerian cells records, per cell, whether no marker, the markers of one
// body, or markers of several bodies lie in it; markers in a cell of the last
// kind are flagged for a collision force.
//
// The paper fills the array in one sequential sweep (an empty cell takes the
// body id, a cell holding another id becomes -1).  Its final state does not
// depend on the order of the sweep: -1 exactly where two or more bodies meet,
// else the one body's id.  So markers enter their ids in parallel: a
// compare-and-swap puts the id into an empty cell, and where it finds another
// body's id, -1 replaces it.  The result is the same bit for bit on any schedule.
// (Plain stores, settled by a second pass, lose ids now and then: a cell that
// markers on two XCDs write at once can look different to each of them even in
// the next launch.)
//
// Entering is bound by the compare-and-swaps, which the memory side executes:
// 0.56 ms for 22.4 M markers in 1024^3 beyond the pass over them when every
// marker made one whose cell did not yet show its id.  About two thirds of the
// markers share a cell with another of their body that the same workgroup
// handles, so the workgroup keeps the (cell, body) pairs it has entered in LDS
// and makes one per cell: 0.75 -> 0.26 ms.  Marking (0.16 ms) and clearing
// (0.17 ms) read 12 B per marker and about 19 B of its cells' 128-byte lines
// (surfaces fill them sparsely), 4 to 5 TB/s.
#include "mls_device.h"

namespace mls {

namespace {

constexpr int kCollBlock = 256;
// 2^kEnteredBits pairs (8 KB); 2^9 to 2^11 take the same time, 2^12 leaves too
// few workgroups per compute unit (collide and clear 0.59 -> 0.73 ms).
constexpr int kEnteredBits = 10;

// Linear index [z][y][x] of the cell of marker l, or -1 (error raised, if err is given).
__device__ __forceinline__ int64_t marker_cell(const Grid &g, int64_t l, const float *x, const float *y,
                                               const float *z, ErrWord *err)
{
    int i, j, k;
    if (!cell_axis_f(g.ax[0], x[l], i) || !cell_axis_f(g.ax[1], y[l], j) || !cell_axis_f(g.ax[2], z[l], k)) {
        if (err) raise_error(err, l, MLS_E_SUPPORT);
        return -1;
    }
    return ((int64_t)k * g.ax[1].n + j) * g.ax[0].n + i;
}

// Ids into the cells.  A body id out of range is left out (reported here).
// entered holds (cell, body) pairs that the workgroup has entered, by a hash of
// the cell, the newest in its place: a marker that finds its own pair there is
// done.  One that finds another body's pair of its cell looks at the cell before
// it swaps, and so does a wavefront of whose markers less than half are done
// (markers next to each other in the array, but not in space): a cell only moves
// 0 -> id -> -1, so a plain read that shows the marker's id or -1, possibly an
// earlier state, spares the swap.  Collision, flags and clearing, never looking
// / so / always looking, us: 22.4 M markers body after body 590 / 593 / 619,
// shuffled 1918 / 1636 / -; 4 M markers of 1000 bodies at random in 64^3 245 /
// 163 / -, in 40 cells of it 1243 / 267 / -.
__global__ void __launch_bounds__(kCollBlock)
k_coll_enter(const Grid *__restrict__ gp, int64_t n, const float *__restrict__ x, const float *__restrict__ y,
             const float *__restrict__ z, const int32_t *__restrict__ body, int32_t *__restrict__ coll,
             ErrWord *err)
{
    __shared__ unsigned long long entered[1 << kEnteredBits];
    const Grid &g = *gp;
    for (int q = threadIdx.x; q < 1 << kEnteredBits; q += kCollBlock) entered[q] = ~0ull;   // no body has id -1
    __syncthreads();
    // the workgroup's markers: a contiguous range
    const int64_t per = ((n + gridDim.x - 1) / gridDim.x + 63) & ~(int64_t)63;
    const int64_t first = xcd_block() * per, last = min(first + per, n);
    int met = 0, known = 0;   // markers of this wavefront, and those whose pair was in the table
    for (int64_t l = first + threadIdx.x; l < last; l += kCollBlock) {
        int64_t cell = marker_cell(g, l, x, y, z, err);
        const int32_t b = body[l];
        if (cell >= 0 && (b < 0 || b > 2147483646)) {
            raise_error(err, l, MLS_E_ARG);
            cell = -1;
        }
        bool done = cell < 0, look = false;
        if (!done) {
            const unsigned long long pair = (unsigned long long)(uint32_t)cell << 32 | (uint32_t)b;
            const unsigned long long was =
                atomicExch(&entered[((uint32_t)cell * 2654435761u) >> (32 - kEnteredBits)], pair);
            done = was == pair;
            look = (was ^ pair) >> 32 == 0;
        }
        met += __popcll(__ballot(1));
        known += __popcll(__ballot(done));
        if (!done && (look || 2 * known < met)) {
            const int32_t now = coll[cell];
            done = now == b + 1 || now == -1;
        }
        if (!done) {
            const int32_t old = atomicCAS(&coll[cell], 0, b + 1);
            if (old != 0 && old != b + 1 && old != -1) atomicExch(&coll[cell], -1);
        }
    }
}

// flags[l] = 1 where the cell of marker l holds -1 (markers of several bodies).
__global__ void __launch_bounds__(kCollBlock)
k_coll_mark(const Grid *__restrict__ gp, int64_t n, const float *__restrict__ x, const float *__restrict__ y,
            const float *__restrict__ z, const int32_t *__restrict__ coll, uint8_t *__restrict__ flags)
{
    const Grid &g = *gp;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t l = xcd_block() * blockDim.x + threadIdx.x; l < n; l += stride) {
        const int64_t cell = marker_cell(g, l, x, y, z, nullptr);
        flags[l] = cell >= 0 && coll[cell] == -1 ? 1 : 0;
    }
}

// Returns the cells of the markers to 0 (plain stores of one value: any order).
__global__ void __launch_bounds__(kCollBlock)
k_coll_clear(const Grid *__restrict__ gp, int64_t n, const float *__restrict__ x, const float *__restrict__ y,
             const float *__restrict__ z, int32_t *__restrict__ coll)
{
    const Grid &g = *gp;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t l = xcd_block() * blockDim.x + threadIdx.x; l < n; l += stride) {
        const int64_t cell = marker_cell(g, l, x, y, z, nullptr);
        if (cell >= 0) coll[cell] = 0;
    }
}

unsigned coll_blocks(const Ctx &c, int64_t n)
{
    int64_t b = (n + kCollBlock - 1) / kCollBlock;
    b = std::min(b, (int64_t)c.cu_count * 16);
    return (unsigned)round_up8(std::max<int64_t>(b, 1));
}

}  // namespace

hipError_t launch_collide(const Ctx &c, int64_t n, const float *x, const float *y, const float *z,
                          const int32_t *body, int32_t *coll, uint8_t *flags, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const unsigned nb = coll_blocks(c, n);
    hipLaunchKernelGGL(k_coll_enter, dim3(nb), dim3(kCollBlock), 0, s, c.d_grid, n, x, y, z, body, coll, c.err);
    if (flags) hipLaunchKernelGGL(k_coll_mark, dim3(nb), dim3(kCollBlock), 0, s, c.d_grid, n, x, y, z, coll, flags);
    return hipGetLastError();
}

hipError_t launch_collide_clear(const Ctx &c, int64_t n, const float *x, const float *y, const float *z,
                                int32_t *coll, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_coll_clear, dim3(coll_blocks(c, n)), dim3(kCollBlock), 0, s, c.d_grid, n, x, y, z, coll);
    return hipGetLastError();
}

}  // namespace mls
