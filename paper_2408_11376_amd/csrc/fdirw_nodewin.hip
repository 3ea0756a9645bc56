// fdirw_nodewin.hip -- node windows of the coarse build by cells (gfx950): the
// column of every group J is the explicit FD of unit mass on J's grouped cells,
// on the blocks within K of J's block (walls at the window's faces).
//
// Many windows cover the same cell, with the same face coefficients and the
// same neighbours, so the state is kept as rows: row c holds the value of
// active cell c in the windows of 64 nodes, one lane each.  Only cells that can
// ever hold something have a row: those that are grouped or have a nonzero face
// (far-field cells, held at 0, share one row of zeros).  A wave takes a cell:
// its coefficients and neighbour rows are scalars, every access to the state is
// one contiguous row, and a window's wall is a lane whose node is K blocks away
// from the cell's block on a face that leaves the block.  Per cell and sub-step
// the terms and their order are those of nodewin_substep_kernel, so the values
// are the same bit for bit.
// Bound by the L2 traffic of the rows (seven reads and one write per lane): a
// particle of radius 16 in 64^3 cells (r = 20, blocks of 5, 420 nodes) takes 33
// us per sub-step, 353 G lanes/s, against 192 us over whole windows.  More
// loads in flight or other rows per wave (2, 8) changed nothing or cost 8 %.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fdirw_device.h"
#include "fdirw_launch.h"

namespace fdirw {

namespace {

constexpr int NW_NT = 256;            // threads per workgroup
constexpr int NW_CPW = 4;             // rows per wave and sub-step launch

template <typename St> struct NwCell {
    St l[6];                          // face coefficients: -x, +x, -y, +y, -z, +z
    int nb[6];                        // their cells' rows
    int bx, by, bz;                   // block of the cell
    int flags;                        // bit f: face f leaves the block; bit 6: grouped
};

// Whether cell i has a row.
template <typename St>
__device__ __forceinline__ bool nw_active(const NodeWinArgs &a, int64_t i)
{
    const int nd = a.node[i];
    if (a.sink && nd == COARSE_RESERVOIR) return false;
    if (nd >= 0) return true;
    const St *lx = (const St *)a.lx, *ly = lx + a.n, *lz = ly + a.n;
    const int x = (int)(i % a.nx), y = (int)((i / a.nx) % a.ny);
    const int64_t sy = a.nx, sz = (int64_t)a.nx * a.ny;
    return lx[i] > St(0) || ly[i] > St(0) || lz[i] > St(0) || (x > 0 && lx[i - 1] > St(0)) ||
           (y > 0 && ly[i - sy] > St(0)) || (i >= sz && lz[i - sz] > St(0));
}

// Cell number v of block (bx, by, bz), in z, y, x order; -1 past the domain.
__device__ __forceinline__ int64_t nw_block_cell(const NodeWinArgs &a, int bx, int by, int bz, int v)
{
    const int x = bx * a.B + v % a.B, y = by * a.B + (v / a.B) % a.B, z = bz * a.B + v / (a.B * a.B);
    return x < a.nx && y < a.ny && z < a.nz ? ((int64_t)z * a.ny + y) * a.nx + x : -1;
}

// block[I] = active cells of block I.
template <typename St>
__global__ void __launch_bounds__(NW_NT) nw_count_kernel(NodeWinArgs a, int *__restrict__ block)
{
    __shared__ int total;
    const int I = blockIdx.x;
    const int bx = I % a.ncx, by = (I / a.ncx) % a.ncy, bz = I / (a.ncx * a.ncy);
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    int mine = 0;
    for (int v = threadIdx.x; v < a.B * a.B * a.B; v += NW_NT) {
        const int64_t i = nw_block_cell(a, bx, by, bz, v);
        if (i >= 0 && nw_active<St>(a, i)) ++mine;
    }
    if (mine) atomicAdd(&total, mine);
    __syncthreads();
    if (threadIdx.x == 0) block[I] = total;
}

// Exclusive scan of the block counts by one workgroup (thread t a contiguous
// piece); run[n_run] receives the total.
__global__ void __launch_bounds__(1024) nw_scan_kernel(int *__restrict__ run, int n_run)
{
    __shared__ int sums[1024];
    const int per = (n_run + 1023) / 1024;
    const int b = threadIdx.x * per, e = min(n_run, b + per);
    int s = 0;
    for (int k = b; k < e; ++k) s += run[k];
    sums[threadIdx.x] = s;
    __syncthreads();
    for (int w = 1; w < 1024; w <<= 1) {
        const int v = (int)threadIdx.x >= w ? sums[threadIdx.x - w] : 0;
        __syncthreads();
        sums[threadIdx.x] += v;
        __syncthreads();
    }
    int at = threadIdx.x > 0 ? sums[threadIdx.x - 1] : 0;
    for (int k = b; k < e; ++k) {
        const int v = run[k];
        run[k] = at;
        at += v;
    }
    if (threadIdx.x == 1023) run[n_run] = sums[1023];
}

// row[i] = the row of cell i (block by block, in z, y, x order within one), or
// -1.
template <typename St>
__global__ void __launch_bounds__(NW_NT) nw_number_kernel(NodeWinArgs a, const int *__restrict__ start,
                                                          int *__restrict__ row)
{
    __shared__ int wsum[NW_NT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int I = blockIdx.x;
    const int bx = I % a.ncx, by = (I / a.ncx) % a.ncy, bz = I / (a.ncx * a.ncy);
    const int n = a.B * a.B * a.B;
    int at = start[I];
    for (int v0 = 0; v0 < n; v0 += NW_NT) {
        const int v = v0 + threadIdx.x;
        const int64_t i = v < n ? nw_block_cell(a, bx, by, bz, v) : -1;
        const bool act = i >= 0 && nw_active<St>(a, i);
        const unsigned long long bal = __ballot(act);
        if (lane == 0) wsum[wave] = __popcll(bal);
        __syncthreads();
        int before = at + __popcll(bal & ((1ull << lane) - 1));
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (i >= 0) row[i] = act ? before : -1;
        for (int w = 0; w < NW_NT / 64; ++w) at += wsum[w];
        __syncthreads();
    }
}

template <typename St>
__global__ void nw_cells_kernel(NodeWinArgs a, const int *__restrict__ row, int n_act, NwCell<St> *__restrict__ cells)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= a.n || row[i] < 0) return;
    const St *lx = (const St *)a.lx, *ly = lx + a.n, *lz = ly + a.n;
    const int x = (int)(i % a.nx), y = (int)((i / a.nx) % a.ny), z = (int)(i / ((int64_t)a.nx * a.ny));
    const int64_t sy = a.nx, sz = (int64_t)a.nx * a.ny;
    NwCell<St> c;
    c.bx = x / a.B; c.by = y / a.B; c.bz = z / a.B;
    c.flags = a.node[i] >= 0 ? 64 : 0;
    const bool has[6] = {x > 0, x < a.nx - 1, y > 0, y < a.ny - 1, z > 0, z < a.nz - 1};
    const int64_t step[6] = {-1, 1, -sy, sy, -sz, sz};
    const int pos[6] = {x, x, y, y, z, z};
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const St *l = f < 2 ? lx : f < 4 ? ly : lz;
        c.l[f] = has[f] ? l[f % 2 ? i : i + step[f]] : St(0);
        const int r = has[f] ? row[i + step[f]] : -1;
        c.nb[f] = r >= 0 ? r : n_act;                          // the row of zeros
        if (f % 2 ? (pos[f] + 1) % a.B == 0 : pos[f] % a.B == 0) c.flags |= 1 << f;
    }
    cells[row[i]] = c;
}

struct NwState {
    int n_act, K;
    int ncx, ncy;
    const int *lanes;                 // [chunks][64] node ids, -1: none
};

struct NwLane {
    int x, y, z;                      // block of the lane's node
};

__device__ __forceinline__ NwLane nw_lane(const NwState &s, int chunk)
{
    const int J = s.lanes[chunk * 64 + (threadIdx.x & 63)];
    NwLane n;
    n.x = J < 0 ? -(1 << 24) : J % s.ncx;
    n.y = J < 0 ? 0 : (J / s.ncx) % s.ncy;
    n.z = J < 0 ? 0 : J / (s.ncx * s.ncy);
    return n;
}

__device__ __forceinline__ bool nw_inside(int dx, int dy, int dz, int K)
{
    return dx >= -K && dx <= K && dy >= -K && dy <= K && dz >= -K && dz <= K;
}

// Rows of the chunk: 1 in the lane of the cell's own group, else 0; the last
// row (far-field cells) 0 in both buffers.
template <typename St>
__global__ void __launch_bounds__(NW_NT) nw_init_kernel(NwState s, const NwCell<St> *__restrict__ cells,
                                                        St *__restrict__ g0, St *__restrict__ g1)
{
    const int lane = threadIdx.x & 63;
    const NwLane n = nw_lane(s, blockIdx.y);
    const int c = blockIdx.x * (NW_NT / 64) + (threadIdx.x >> 6);
    if (c > s.n_act) return;
    const int64_t at = ((int64_t)blockIdx.y * (s.n_act + 1) + c) * 64 + lane;
    if (c == s.n_act) {
        g0[at] = g1[at] = St(0);
        return;
    }
    const NwCell<St> &k = cells[c];
    g0[at] = (k.flags & 64) && k.bx == n.x && k.by == n.y && k.bz == n.z ? St(1) : St(0);
}

// One sub-step of the rows [unit.row, unit.end) (of one block) in the windows
// of chunk unit.chunk; a.units lists every block within reach of a chunk.
template <typename St>
__global__ void __launch_bounds__(NW_NT) nw_substep_kernel(NwState s, const NodeWinUnit *__restrict__ units,
                                                           const NwCell<St> *__restrict__ cells,
                                                           const St *__restrict__ in, St *__restrict__ out)
{
    const NodeWinUnit unit = units[xcd_remap((int)blockIdx.x, (int)gridDim.x)];   // neighbouring blocks on one XCD
    const int c0 = __builtin_amdgcn_readfirstlane(unit.row + (int)(threadIdx.x >> 6) * NW_CPW);
    if (c0 >= unit.end) return;                                // uniform per wave
    const NwLane n = nw_lane(s, unit.chunk);
    const int64_t base = (int64_t)unit.chunk * (s.n_act + 1) * 64 + (threadIdx.x & 63);
    in += base;
    out += base;
    const int d[3] = {unit.bx - n.x, unit.by - n.y, unit.bz - n.z};
    if (!nw_inside(d[0], d[1], d[2], s.K)) return;              // half a row that no window holds costs nothing
    // every load of the wave's rows before the first is used (the last row in
    // the place of rows past the unit)
    St gv[NW_CPW], v[NW_CPW][6];
    int row[NW_CPW];
#pragma unroll
    for (int u = 0; u < NW_CPW; ++u) {
        row[u] = min(c0 + u, unit.end - 1);
        const NwCell<St> &k = cells[row[u]];
        gv[u] = in[(int64_t)row[u] * 64];
#pragma unroll
        for (int f = 0; f < 6; ++f) v[u][f] = in[(int64_t)k.nb[f] * 64];
    }
#pragma unroll
    for (int u = 0; u < NW_CPW; ++u) {
        const NwCell<St> &k = cells[row[u]];
        St acc = gv[u];
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const St t = __builtin_elementwise_fma(k.l[f], v[u][f] - gv[u], acc);
            const bool wall = ((k.flags >> f) & 1) && d[f / 2] == (f % 2 ? s.K : -s.K);
            acc = wall ? acc : t;
        }
        out[(int64_t)row[u] * 64] = acc;                        // a repeated row: the same value
    }
}

// S[o][I] = the sum over block I's grouped cells (in z, y, x order) of the
// lane's window, for the blocks I within K of the lane's node.  One wave per
// (block, chunk); nx, ny, nz, B, node as in NodeWinArgs.
template <typename St>
__global__ void __launch_bounds__(64) nw_bin_kernel(NodeWinArgs a, NwState s, const int *__restrict__ row,
                                                    const St *__restrict__ g, double *__restrict__ S)
{
    const int lane = threadIdx.x;
    const int64_t I = blockIdx.x;
    const NwLane n = nw_lane(s, blockIdx.y);
    const int bx = (int)(I % a.ncx), by = (int)((I / a.ncx) % a.ncy), bz = (int)(I / ((int64_t)a.ncx * a.ncy));
    const int dx = bx - n.x, dy = by - n.y, dz = bz - n.z;
    const bool inside = nw_inside(dx, dy, dz, s.K);
    if (!__any(inside)) return;
    const St *gl = g + (int64_t)blockIdx.y * (s.n_act + 1) * 64 + lane;
    double sum = 0.0;
    for (int z = bz * a.B; z < min(a.nz, (bz + 1) * a.B); ++z)
        for (int y = by * a.B; y < min(a.ny, (by + 1) * a.B); ++y)
            for (int x = bx * a.B; x < min(a.nx, (bx + 1) * a.B); ++x) {
                const int64_t i = ((int64_t)z * a.ny + y) * a.nx + x;
                if (a.node[i] >= 0) sum += (double)gl[(int64_t)row[i] * 64];
            }
    if (inside) {
        const int KW = 2 * a.K + 1;
        const int o = ((dz + a.K) * KW + dy + a.K) * KW + dx + a.K;
        S[(int64_t)o * a.n_nodes + I] = sum;
    }
}

// Scales the column of every listed node to N_J over its bins (one wave per
// node: lanes over the offsets, a fixed butterfly).
__global__ void __launch_bounds__(64) nw_scale_kernel(NodeWinArgs a, const int *__restrict__ lanes,
                                                      const double *__restrict__ count, double *__restrict__ S)
{
    const int J = lanes[blockIdx.x];
    if (J < 0) return;
    const int KW = 2 * a.K + 1, nb = KW * KW * KW;
    const int jx = J % a.ncx, jy = (J / a.ncx) % a.ncy, jz = J / (a.ncx * a.ncy);
    auto entry = [&](int o) -> int64_t {
        const int x = jx + o % KW - a.K, y = jy + (o / KW) % KW - a.K, z = jz + o / (KW * KW) - a.K;
        if (x < 0 || x >= a.ncx || y < 0 || y >= a.ncy || z < 0 || z >= a.ncz) return -1;
        return (int64_t)o * a.n_nodes + ((int64_t)z * a.ncy + y) * a.ncx + x;
    };
    double tot = 0.0;
    for (int o = threadIdx.x; o < nb; o += 64) {
        const int64_t e = entry(o);
        if (e >= 0) tot += S[e];
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) tot += __shfl_xor(tot, m, 64);
    const double scale = tot > 0.0 ? count[J] / tot : 0.0;
    for (int o = threadIdx.x; o < nb; o += 64) {
        const int64_t e = entry(o);
        if (e >= 0) S[e] *= scale;
    }
}

template <typename St>
hipError_t number_cells(const NodeWinArgs &a, int *block, int *start, int *row, hipStream_t st)
{
    hipLaunchKernelGGL(nw_count_kernel<St>, dim3((unsigned)a.n_nodes), dim3(NW_NT), 0, st, a, block);
    hipError_t e = hipMemcpyAsync(start, block, (size_t)a.n_nodes * sizeof(int), hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(nw_scan_kernel, dim3(1), dim3(1024), 0, st, start, (int)a.n_nodes);
    hipLaunchKernelGGL(nw_number_kernel<St>, dim3((unsigned)a.n_nodes), dim3(NW_NT), 0, st, a, start, row);
    return hipGetLastError();
}

template <typename St>
hipError_t build(const NodeWinArgs &a, int n_sub, const int *row, int n_act, void *cells, const int *lanes,
                 int n_chunk, const NodeWinUnit *units, int n_unit, void *ga, void *gb, const double *count, double *S,
                 hipStream_t st)
{
    NwCell<St> *cell = (NwCell<St> *)cells;
    const NwState s{n_act, a.K, a.ncx, a.ncy, lanes};
    const int per = NW_NT / 64;
    hipLaunchKernelGGL(nw_init_kernel<St>, dim3((n_act + per) / per, n_chunk), dim3(NW_NT), 0, st, s, cell, (St *)ga,
                       (St *)gb);
    hipError_t e = hipGetLastError();
    St *in = (St *)ga, *out = (St *)gb;
    for (int k = 0; k < n_sub && e == hipSuccess && n_unit > 0; ++k) {
        hipLaunchKernelGGL(nw_substep_kernel<St>, dim3(n_unit), dim3(NW_NT), 0, st, s, units, cell, in, out);
        e = hipGetLastError();
        St *t = in; in = out; out = t;
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(nw_bin_kernel<St>, dim3((unsigned)a.n_nodes, n_chunk), dim3(64), 0, st, a, s, row, in, S);
    if (!a.sink) hipLaunchKernelGGL(nw_scale_kernel, dim3(64 * n_chunk), dim3(64), 0, st, a, lanes, count, S);
    return hipGetLastError();
}

}  // namespace

size_t nodewin_cell_bytes(int fp64) { return fp64 ? sizeof(NwCell<double>) : sizeof(NwCell<float>); }

int nodewin_unit_rows() { return NW_NT / 64 * NW_CPW; }

hipError_t launch_nodewin_number(int fp64, const NodeWinArgs &a, int *block, int *start, int *row, hipStream_t st)
{
    return fp64 ? number_cells<double>(a, block, start, row, st) : number_cells<float>(a, block, start, row, st);
}

hipError_t launch_nodewin_cells(int fp64, const NodeWinArgs &a, const int *row, int n_act, void *cells, hipStream_t st)
{
    const dim3 g((unsigned)((a.n + NW_NT - 1) / NW_NT));
    if (fp64) hipLaunchKernelGGL(nw_cells_kernel<double>, g, dim3(NW_NT), 0, st, a, row, n_act, (NwCell<double> *)cells);
    else hipLaunchKernelGGL(nw_cells_kernel<float>, g, dim3(NW_NT), 0, st, a, row, n_act, (NwCell<float> *)cells);
    return hipGetLastError();
}

hipError_t launch_nodewin_rows(int fp64, const NodeWinArgs &a, int n_sub, const int *row, int n_act, void *cells,
                               const int *lanes, int n_chunk, const NodeWinUnit *units, int n_unit, void *ga, void *gb,
                               const double *count, double *S, hipStream_t st)
{
    if (n_chunk <= 0 || n_act <= 0) return hipSuccess;
    if (n_chunk > 65535 || 2 * a.K + 1 > 17) return hipErrorInvalidValue;
    return fp64 ? build<double>(a, n_sub, row, n_act, cells, lanes, n_chunk, units, n_unit, ga, gb, count, S, st)
                : build<float>(a, n_sub, row, n_act, cells, lanes, n_chunk, units, n_unit, ga, gb, count, S, st);
}

}  // namespace fdirw
