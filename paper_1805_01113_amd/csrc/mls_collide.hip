// Coarse-grained collision detection (Sec. 4): an integer array over the
// Eulerian cells records, per cell, whether no marker, the markers of one
// body, or markers of several bodies lie in it; markers in a cell of the last
// kind are flagged for a collision force.
//
// The paper fills the array in one sequential sweep (an empty cell takes the
// body id, a cell holding another id becomes -1).  Its final state does not
// depend on the order of the sweep: -1 exactly where two or more bodies meet,
// else the one body's id.  Here that state is reached without an atomic, in two
// launches: in the first every marker of an empty cell stores its id, and one
// that sees another body's id stores -1; whichever store lasts, the cell then
// holds one of its bodies' ids or -1.  In the second every marker whose cell
// holds neither its own id nor -1 stores -1, the only value stored there, so a
// cell of several bodies ends at -1 (all but one body see a foreign id) and a
// cell of one body keeps its id, bit for bit on any schedule.
//
// Bound by memory: a pass reads 12-16 B per marker and about 19 B of its cells'
// 128-byte lines (surfaces fill them sparsely), the first also writes those.
// 22.4 M markers in 1024^3: 0.24 and 0.19 ms for the two launches, 5 TB/s;
// entering with a compare-and-swap per marker, which the memory side executes,
// took 0.75 ms.  Four markers a thread at a time change nothing.
#include "mls_device.h"

namespace mls {

namespace {

constexpr int kCollBlock = 256;

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

// First launch: ids into empty cells, -1 where another body's id is seen.  A
// body id out of range is left out (reported here).
__global__ void __launch_bounds__(kCollBlock)
k_coll_enter(const Grid *__restrict__ gp, int64_t n, const float *__restrict__ x, const float *__restrict__ y,
             const float *__restrict__ z, const int32_t *__restrict__ body, int32_t *__restrict__ coll,
             ErrWord *err)
{
    const Grid &g = *gp;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t l = xcd_block() * blockDim.x + threadIdx.x; l < n; l += stride) {
        const int64_t cell = marker_cell(g, l, x, y, z, err);
        if (cell < 0) continue;
        const int32_t b = body[l];
        if (b < 0 || b > 2147483646) {
            raise_error(err, l, MLS_E_ARG);
            continue;
        }
        const int32_t seen = coll[cell];
        if (seen == b + 1 || seen == -1) continue;
        coll[cell] = seen == 0 ? b + 1 : -1;
    }
}

// Second launch: -1 where a marker's cell kept another body's id.
__global__ void __launch_bounds__(kCollBlock)
k_coll_settle(const Grid *__restrict__ gp, int64_t n, const float *__restrict__ x, const float *__restrict__ y,
              const float *__restrict__ z, const int32_t *__restrict__ body, int32_t *__restrict__ coll)
{
    const Grid &g = *gp;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t l = xcd_block() * blockDim.x + threadIdx.x; l < n; l += stride) {
        const int64_t cell = marker_cell(g, l, x, y, z, nullptr);
        const int32_t b = body[l];
        if (cell < 0 || b < 0 || b > 2147483646) continue;
        const int32_t seen = coll[cell];
        if (seen != b + 1 && seen != -1) coll[cell] = -1;
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
    hipLaunchKernelGGL(k_coll_settle, dim3(nb), dim3(kCollBlock), 0, s, c.d_grid, n, x, y, z, body, coll);
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
