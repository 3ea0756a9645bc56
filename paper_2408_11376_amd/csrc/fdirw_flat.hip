// fdirw_flat.hip -- the fused FDiRW big step with a flat window layout
// (gfx950, FP32 or FP64 state).
//
// Same computation as line_kernel (the column form of Eq. 8 of arXiv
// 2408.11376: every source's window kernel of Sec. 3.1 is generated by the
// explicit 7-point FD and added, times c(s), into the output), organised in
// FP32 for a 256-thread workgroup of four waves, one per SIMD, that runs one
// source line (r = 7, 8), two (r = 5, 6) or four (r = 4) side by side, and in
// FP64 for a workgroup of 64 to 576 threads per line (r = 3..8):
//   * the W^3 window cells are numbered flat, i = cy PY + cx W + z (z fastest;
//     PY is W^2 rounded up to whole 16-byte chunks, the cells between are
//     unused), and thread t of a line's SG threads owns the RUN consecutive
//     cells [RUN t, RUN t + RUN) in registers (FP32, r = 8: RUN = 20, 249 of 256
//     lanes busy; an odd number of chunks, so the exchange accesses of 16
//     consecutive lanes meet no LDS bank twice);
//   * the z neighbours of a cell are its run neighbours (registers), except
//     at the two run ends (from LDS); a run crossing a column boundary meets
//     a window wall there (coefficient 0);
//   * the y neighbours are the runs at offsets +-PY, read from the LDS copy of
//     the window as aligned 128-bit loads.  The runs at +-W (x) overlap the own
//     run where RUN > W (FP32, every radius 4..8): only the W cells
//     before and after it are read (aligned, ceil(W / 4) loads each, which
//     also hold the two run-end z neighbours), the rest come from registers;
//   * double-buffered exchange, one barrier per sub-step;
//   * the superposition ring is a shift register of RUN FP64 accumulators
//     per thread instead of W planes in LDS: after source sz the cells of
//     window plane z = 0 hold the finished plane sz - R, which is added to
//     c_out with one atomic per window column; then every accumulator moves
//     down one cell (cell i takes cell i + 1, the run's top cell takes the
//     next thread's bottom cell), which is the window of source sz + 1.
// What bounds a sub-step is the LDS pipe.  FP32: a 128-bit write of a wave takes
// 13.6 clocks of it and a read 5.2 (measured alone), 5 + 20 of them per wave at
// r = 8, i.e. 690 clocks per window and sub-step against 560 of FP32 FMAs.  The
// pitch PY saves two reads per wave and sub-step (the offset W^2 is odd, and a
// misaligned run spans RUN / 4 + 1 loads).  LDS (<= 53 KB) and 168 registers
// let three workgroups share a CU and fill each other's barrier and LDS waits;
// at that budget the compiler keeps the ring in private memory across the
// sub-step loop, which itself holds no spills.  96^3 steps, 3 workgroups of
// pitch PY against 2 of pitch W^2: r = 4 (50 sub-steps) 12.3 -> 8.9 ms, r = 5
// (78) 31.1 -> 24.8 ms, r = 6 (113) 68.6 -> 63.0 ms, r = 7 (153) 174 -> 163 ms,
// r = 8 (200) 233 -> 222 ms.
// FP64 moves twice the bytes: at r = 8 its 8 waves take 5 + 22 accesses of 16
// bytes and two of 8 per wave and sub-step, ~1,520 clocks of the LDS pipe, where
// line_kernel's columns of 9 cells take ~1,750 (top and first cells of a segment
// go through LDS twice more) and spill in the loop.  The registers let only one
// workgroup per CU run, so its barriers are not filled by another.  61 x 57 x 60
// cells, line_kernel / this (ms): r = 3 (28 sub-steps) 1.68 / 1.46, r = 4 7.1 /
// 4.4, r = 5 16.1 / 13.4, r = 6 59.0 / 32.1, r = 7 97.3 / 70.8, r = 8 160 / 119.
// Per cell and sub-step the arithmetic is that of one_substep (same terms,
// same order), so the kernels equal line_kernel's bit for bit.
#include "fdirw_flat.h"
#include "fdirw_launch.h"

namespace fdirw {

// One source line of one domain for the flat layout; the face coefficients
// come from the accessor f (FaceArrays over [3][n] owned-face coefficients, or
// FaceLabels over a phase-pair table).  part (the
// deterministic form): completed planes go to the partial slots part[(col
// part_planes + Z - part_z0) nxy + Y nx + X] as plain stores instead of FP64
// atomics into c_out.
template <typename Faces> struct FlatLine {
    int nx, ny, nz;
    int64_t n;
    int n_sub;
    Faces f;
    const double *c_in;
    double *c_out;
    double *part;
    int part_z0, part_planes;
};

// Adds plane Z (when inside the domain) of the window of line (sx, sy) to
// c_out: column col of the window, held at pl[col], goes to cell (Z,
// sy - R + col / W, sx - R + col % W); thread tg of the window's SG threads
// takes columns tg, tg + SG, ... (consecutive lanes, consecutive x:
// coalesced FP64 atomics).  In the deterministic form (DET, a.part) every
// in-domain column is stored to its own partial slot, zeros too, so that
// each slot the reduction reads is written.
template <int R, int SG, bool DET, typename Line>
__device__ __forceinline__ void flush_plane(const Line &a, const double *pl, int sx, int sy, int Z, int tg)
{
    constexpr int W = 2 * R + 1, W2 = W * W;
    if (Z < 0 || Z >= a.nz) return;                          // uniform per block
    const int64_t nxy = (int64_t)a.nx * a.ny;
    for (int col = tg; col < W2; col += SG) {
        const int X = sx - R + col % W, Y = sy - R + col / W;
        const double v = pl[col];
        if (X < 0 || X >= a.nx || Y < 0 || Y >= a.ny) continue;
        if constexpr (DET)
            a.part[((int64_t)col * a.part_planes + (Z - a.part_z0)) * nxy + (int64_t)Y * a.nx + X] = v;
        else if (v != 0.0)
            unsafeAtomicAdd(&a.c_out[(int64_t)Z * nxy + (int64_t)Y * a.nx + X], v);
    }
}

// Plane Z of a line whose ring is empty: nothing to add, and in the
// deterministic form zeros in its slots.
template <int R, int SG, bool DET, typename Line>
__device__ __forceinline__ void flush_empty(const Line &a, int sx, int sy, int Z, int tg)
{
    constexpr int W = 2 * R + 1, W2 = W * W;
    if (!DET || Z < 0 || Z >= a.nz) return;
    const int64_t nxy = (int64_t)a.nx * a.ny;
    for (int col = tg; col < W2; col += SG) {
        const int X = sx - R + col % W, Y = sy - R + col / W;
        if (X >= 0 && X < a.nx && Y >= 0 && Y < a.ny)
            a.part[((int64_t)col * a.part_planes + (Z - a.part_z0)) * nxy + (int64_t)Y * a.nx + X] = 0.0;
    }
}

constexpr int FLAT_CS = 32;        // sources of a line read at a time

// LDS of one workgroup at radius R: exchange floats (two buffers per line) and
// output-plane doubles (one per line and parity); _MAX over the radii 0..8.
template <int R> constexpr int FLAT_XB = 2 * Flat<R>::LPW * Flat<R>::XLEN;
template <int R> constexpr int FLAT_PLANE = 2 * Flat<R>::LPW * Flat<R>::W2;
constexpr int flat_max(int a, int b) { return a > b ? a : b; }
template <int R> constexpr int flat_xb_max()
{
    if constexpr (R == 0) return FLAT_XB<0>;
    else return flat_max(FLAT_XB<R>, flat_xb_max<R - 1>());
}
template <int R> constexpr int flat_plane_max()
{
    if constexpr (R == 0) return FLAT_PLANE<0>;
    else return flat_max(FLAT_PLANE<R>, flat_plane_max<R - 1>());
}

// The sources (sx, sy, z0 .. z1 - 1) of the lines line0 .. line0 + nlines - 1
// (line = sy nx + sx; 1 <= nlines <= F::LPW) by a workgroup of F::NT
// threads, F::SG threads per line, the lines side by side in lockstep
// (their sub-steps share the barriers): kernels generated and superposed into
// a.c_out (FP64 atomics).  xb: 2 LPW XLEN cells of LDS (16-byte aligned),
// red: NT / 64 doubles, edge: EDGE doubles, plane: 2 LPW W2 doubles, csrc: LPW
// FLAT_CS doubles.  Every thread of the block calls it; the first thread of line
// g leaves the line's smallest and largest kernel mass and its number of kernels
// in fig[3 g .. 3 g + 2] (LDS; kept there and not in registers, which the
// sub-step loop needs all).  A window group
// past nlines runs on zero coefficients and writes nothing.  DET:
// the deterministic form (partial slots, a.part).
template <typename F, bool DET, typename Faces>
__device__ __forceinline__ void flat_line(const FlatLine<Faces> &a, int line0, int nlines, int z0, int z1,
                                          typename F::S *xb, double *red, double *edge, double *plane, double *fig,
                                          double *csrc)
{
    using S = typename F::S;
    constexpr int R = F::R, FLAT_EDGE = F::EDGE;
    constexpr bool RENORM = sizeof(S) == 4;                   // FP64 kernels are taken as they are
    constexpr int W = F::W, W2 = F::W2, RUN = F::RUN, PAD = F::PAD, XLEN = F::XLEN;
    constexpr int SG = F::SG, LPW = F::LPW;

    const int t = threadIdx.x;
    const int g = LPW == 1 ? 0 : t / SG;                      // the thread's line in the workgroup
    const int tg = t - g * SG;                               // its index among the line's threads
    const int s0 = tg * RUN;                                 // first cell of the run
    const bool act = tg < F::NACT;
    // a group past the last line flushes nothing (with one line per
    // workgroup, nlines is 1)
    const bool live = LPW == 1 || g < nlines;
    const int ln = line0 + (live ? g : 0);
    const int sy = ln / a.nx, sx = ln - sy * a.nx;
    S *const xg = xb + g * XLEN;                         // the line's first exchange buffer
    __syncthreads();                                        // LDS of a previous line is no longer read
    for (int i = t; i < 2 * LPW * XLEN; i += F::NT) xb[i] = S(0);
    if (t < FLAT_EDGE) edge[t] = 0.0;
    if (tg == 0) { fig[3 * g] = INFINITY; fig[3 * g + 1] = -INFINITY; fig[3 * g + 2] = 0.0; }
    __syncthreads();
    const int64_t nxy = (int64_t)a.nx * a.ny;

    // s0v: the run start laundered per source, so that the cell positions are
    // recomputed where they are used instead of being kept in registers
    // across the sub-step loop (idle threads get a start past the window)
    const int own = PAD + s0;                                // exchange index of the run's first cell

    double acc[RUN];
#pragma unroll
    for (int k = 0; k < RUN; ++k) acc[k] = 0.0;
    int par = 0;
    int last = z0 - W;                                       // the last source with a kernel: the ring holds planes up to last + R

    // FLAT_CS sources of every line at a time, into LDS: the memory's latency is
    // met once for all of them, which is what lines without sources wait for
    // (61 x 57 x 60 cells, one nonzero source, ms with a load per source / so: FP64
    // r = 7 1.14 / 0.20, r = 8 1.44 / 0.18, FP32 r = 8 1.03 / 0.11; 10 % nonzero,
    // FP64 r = 6, 8 sub-steps 1.18 / 0.96).  Bit k of some: a line has a nonzero
    // source at the k-th one from sz on.
    unsigned some = 0;
    for (int sz = z0; sz < z1; ++sz, some >>= 1) {
        if (((sz - z0) & (FLAT_CS - 1)) == 0) {
            const int z = sz + (t & (FLAT_CS - 1));
            bool nz = false;
#pragma unroll
            for (int h = 0; h < LPW; ++h) {
                const double c = h < nlines && z < z1 ? a.c_in[(int64_t)z * nxy + line0 + h] : 0.0;
                nz = nz || c != 0.0;
                if (t / FLAT_CS == h) csrc[t] = c;               // read after the next barrier, written after the last read's
            }
            some = (unsigned)__ballot(nz);
        }
        // a kernel is generated for every line when one of them has a nonzero
        // source; past the window of the last one the ring is empty and stays
        // so.  Uniform per block.
        const bool any = some & 1u;
        if (!any && sz - last >= W) {
            if (live) flush_empty<R, SG, DET>(a, sx, sy, sz - R, tg);
            continue;
        }
        int s0v = act ? s0 : F::NCELL;
        asm volatile("" : "+v"(s0v));
        if (any) {
            last = sz;
            FlatSeg<F> c;
            flat_load<F>(c, a.f, a.nx, a.ny, a.nz, sx, sy, sz, s0v);
            S Gs[RUN];
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                const FlatCell<F> p(s0v + k);
                Gs[k] = (p.ok && p.cx == R && p.cy == R && p.z == R) ? S(1) : S(0);
            }
            flat_substeps<F, false>(Gs, c, xg, xg + LPW * XLEN, own, a.n_sub, 0u);
            // kernel mass: per thread in cell order, then over the line's threads
            double ms = 0.0;
            if (act) {
#pragma unroll
                for (int k = 0; k < RUN; ++k) ms += (double)Gs[k];
            }
            const double m = flat_window_sum<F>(ms, red, g);
            const double cs = csrc[g * FLAT_CS + ((sz - z0) & (FLAT_CS - 1))];   // 0 past the last line
            if (tg == 0 && cs != 0.0) {
                fig[3 * g] = fmin(fig[3 * g], m);
                fig[3 * g + 1] = fmax(fig[3 * g + 1], m);
                fig[3 * g + 2] += 1.0;
            }
            const double scale = cs != 0.0 ? (RENORM ? cs / m : cs) : 0.0;
#pragma unroll
            for (int k = 0; k < RUN; ++k) acc[k] = __builtin_fma(scale, (double)Gs[k], acc[k]);
        }
        s0v = act ? s0 : F::NCELL;
        asm volatile("" : "+v"(s0v));
        // window plane z = 0 is plane sz - R of the output, complete for this
        // line: its cells go to the LDS plane by column, so that the flush
        // below gives consecutive lanes consecutive columns (coalesced atomics)
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            const FlatCell<F> p(s0v + k);
            if (p.z == 0) {
                if (p.ok) plane[(par * LPW + g) * W2 + p.col] = acc[k];
                acc[k] = 0.0;
            }
        }
        // shift by one cell: the window of source sz + 1.  The run's top cell
        // takes the next thread's bottom cell (the next lane's, or through
        // LDS the next wave's first; a line's last thread takes 0)
        const double bottom = act ? acc[0] : 0.0;
        double *const ed = edge + par * (FLAT_EDGE / 2);
        if ((t & 63) == 0) ed[t >> 6] = bottom;
        __syncthreads();
        if (live) flush_plane<R, SG, DET>(a, plane + (par * LPW + g) * W2, sx, sy, sz - R, tg);
        double top = __shfl_down(bottom, 1, 64);
        if ((t & 63) == 63) top = ed[(t >> 6) + 1];
        if (tg + 1 == SG) top = 0.0;
#pragma unroll
        for (int k = 0; k < RUN - 1; ++k) acc[k] = acc[k + 1];
        acc[RUN - 1] = top;
        par ^= 1;
    }
    // the planes still held: after the last shift cell (col, z) holds plane
    // z1 - R + z (z = W - 1 holds the plane no source reached yet: zeros), up to
    // plane last + R
    const int s0v = act ? s0 : F::NCELL;
    const int zp_end = max(0, min(W - 1, last + W - z1));
    for (int zp = 0; zp < zp_end; ++zp) {
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            const FlatCell<F> p(s0v + k);
            if (p.ok && p.z == zp) plane[(par * LPW + g) * W2 + p.col] = acc[k];
        }
        __syncthreads();
        if (live) flush_plane<R, SG, DET>(a, plane + (par * LPW + g) * W2, sx, sy, z1 - R + zp, tg);
        par ^= 1;
    }
    for (int zp = zp_end; DET && zp < W - 1; ++zp)
        if (live) flush_empty<R, SG, DET>(a, sx, sy, z1 - R + zp, tg);
}

template <typename F, bool LAB, bool DET>
__global__ void __launch_bounds__(F::NT) __attribute__((amdgpu_waves_per_eu(F::WPE)))
flat_line_kernel(LineArgs a)
{
    using S = typename F::S;
    __shared__ __align__(16) S xb[2 * F::LPW * F::XLEN];
    __shared__ double red[F::NT / 64];
    __shared__ double edge[F::EDGE];
    __shared__ double plane[2 * F::LPW * F::W2];
    // block b: lines LPW lg .. + LPW - 1 (those inside the domain), segment sgi
    const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int lg = b / a.n_seg, sgi = b - lg * a.n_seg;
    const int line0 = lg * F::LPW, nlines = min(F::LPW, a.nx * a.ny - line0);
    const int z0 = a.z_begin + sgi * a.seg_len;
    const int z1 = min(a.z_end, z0 + a.seg_len);
    if (z0 >= z1) return;                                   // uniform per block
    __shared__ double fig[3 * F::LPW];
    __shared__ double csrc[F::LPW * FLAT_CS];
    if constexpr (LAB) {
        const FaceLabels<S> f{a.label, (const S *)a.lam_tab, a.n_phase, a.nx, a.ny, a.nz};
        const FlatLine<FaceLabels<S>> fl{a.nx,   a.ny,    a.nz,   a.n,         a.n_sub, f,
                                         a.c_in, a.c_out, a.part, a.part_z0, a.part_planes};
        flat_line<F, DET>(fl, line0, nlines, z0, z1, xb, red, edge, plane, fig, csrc);
    } else {
        const S *lx = (const S *)a.lx;
        const FlatLine<FaceArrays<S>> fl{a.nx,   a.ny,    a.nz,   a.n,         a.n_sub, {lx, lx + a.n, lx + 2 * a.n},
                                         a.c_in, a.c_out, a.part, a.part_z0, a.part_planes};
        flat_line<F, DET>(fl, line0, nlines, z0, z1, xb, red, edge, plane, fig, csrc);
    }
    // per line and segment: entry line n_seg + sgi of the kernel-mass range
    const int g = (int)threadIdx.x / F::SG;
    if ((int)threadIdx.x == g * F::SG && g < nlines) {
        const int64_t e = (int64_t)(line0 + g) * a.n_seg + sgi;
        if (a.wg_kmass) { a.wg_kmass[2 * e] = fig[3 * g]; a.wg_kmass[2 * e + 1] = fig[3 * g + 1]; }
        if (a.n_used && fig[3 * g + 2] > 0.0) atomicAdd(a.n_used, (unsigned long long)fig[3 * g + 2]);
    }
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T> __device__ __forceinline__ T *uniform(T *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = (uint32_t)uniform((int)(uint32_t)v), hi = (uint32_t)uniform((int)(uint32_t)(v >> 32));
    return (T *)((uint64_t)hi << 32 | lo);
}

// The lines of one batched item as a separate function per radius (the
// persistent kernel's switch over nine inlined bodies would share one
// register allocation).  The kernel-mass range and source count of the item
// (all its lines) come back in thread 0's km and used.
template <int R>
__device__ __attribute__((noinline)) void flat_line_item(const FlatLine<FaceArrays<float>> &a, int line0, int nlines,
                                                          int z0, int z1, float *xb, double *red,
                                                          double *edge, double *plane, double *fig, double *csrc, double *km,
                                                          int *used)
{
    // arguments of a function arrive in vector registers: without this the
    // sub-step loop counts per lane, and its registers are copied every trip
    const int nx = uniform(a.nx), ny = uniform(a.ny), nz = uniform(a.nz);
    const int64_t n = (int64_t)nx * ny * nz;
    const float *lx = uniform(a.f.lx);
    const FlatLine<FaceArrays<float>> u{nx, ny, nz, n, uniform(a.n_sub), {lx, lx + n, lx + 2 * n},
                                        uniform(a.c_in), uniform(a.c_out), nullptr, 0, 0};
    nlines = uniform(nlines);
    flat_line<Flat<R>, false>(u, uniform(line0), nlines, uniform(z0), uniform(z1), xb, red, edge, plane, fig, csrc);
    const int t = threadIdx.x;
    __syncthreads();                                         // every line's figures are there
    if (t == 0) {
        double lo = INFINITY, hi = -INFINITY, n = 0.0;
        for (int h = 0; h < nlines; ++h) {
            lo = fmin(lo, fig[3 * h]);
            hi = fmax(hi, fig[3 * h + 1]);
            n += fig[3 * h + 2];
        }
        km[0] = lo;
        km[1] = hi;
        *used = (int)n;
    }
}

// Many domains in one persistent launch with the flat layout (FP32): each
// workgroup pulls items (domain, a run of source lines, plane range) from the
// atomic counter and runs flat_line for the domain's radius.  An item holds
// up to Flat<r>::LPW consecutive lines of its domain (flat_lines_per_group).
__global__ void __launch_bounds__(FLAT_NT) __attribute__((amdgpu_waves_per_eu(3)))
flat_batched_kernel(BatchArgs a)
{
    __shared__ __align__(16) float xb[flat_xb_max<8>()];
    __shared__ double red[4];
    __shared__ double edge[Flat<8>::EDGE];
    __shared__ double plane[flat_plane_max<8>()];
    __shared__ double fig[3 * (FLAT_NT / 64)];
    __shared__ double csrc[FLAT_NT / 64 * FLAT_CS];
    __shared__ int s_item;
    for (;;) {
        if (threadIdx.x == 0) s_item = (int)atomicAdd(a.head, 1u);
        __syncthreads();
        const int it = s_item;
        __syncthreads();
        if (it >= a.n_items) break;                         // uniform: every wave leaves
        const BatchItem item = a.items[it];
        const BatchDom d = a.doms[item.dom];
        const float *lx = (const float *)d.lam;
        const FlatLine<FaceArrays<float>> fl{d.nx,   d.ny,    d.nz,    d.n, d.n_sub, {lx, lx + d.n, lx + 2 * d.n},
                                             d.c_in, d.c_out, nullptr, 0,   0};
        double km[2];
        int used = 0;
        switch (d.r) {
        case 0: flat_line_item<0>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        case 1: flat_line_item<1>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        case 2: flat_line_item<2>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        case 3: flat_line_item<3>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        case 4: flat_line_item<4>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        case 5: flat_line_item<5>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        case 6: flat_line_item<6>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        case 7: flat_line_item<7>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        default: flat_line_item<8>(fl, item.line0, item.nlines, item.z0, item.z1, xb, red, edge, plane, fig, csrc, km, &used); break;
        }
        if (threadIdx.x == 0) {
            if (a.item_kmass) { a.item_kmass[2 * it] = km[0]; a.item_kmass[2 * it + 1] = km[1]; }
            if (used && d.n_used) atomicAdd(d.n_used, (unsigned long long)used);
        }
    }
}

hipError_t launch_batched_flat(const BatchArgs &a, int grid, hipStream_t st)
{
    hipLaunchKernelGGL(flat_batched_kernel, dim3(grid), dim3(FLAT_NT), 0, st, a);
    return hipGetLastError();
}

hipError_t batched_flat_occupancy(int *blocks)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, flat_batched_kernel, FLAT_NT, 0);
}

int flat_lines_per_group(int r)
{
    return r >= 0 && r <= 8 ? FLAT_NT / line_threads(r) : 1;
}

template <typename F, bool LAB, bool DET>
static hipError_t launch_flat_f(const LineArgs &a, hipStream_t st)
{
    const int64_t groups = ((int64_t)a.nx * a.ny + F::LPW - 1) / F::LPW;
    hipLaunchKernelGGL((flat_line_kernel<F, LAB, DET>), dim3((unsigned)(groups * a.n_seg)), dim3(F::NT), 0, st, a);
    return hipGetLastError();
}

// FP32: three waves per SIMD, or two where the registers count for more than the
// sub-steps.  r = 6: at three, part of a source's coefficients is spilled while
// they are loaded.  Measured (two / three, ms): 61 x 57 x 60 cells, 10 sub-steps
// 3.94 / 5.08, 40 7.32 / 7.38, 112 16.4 / 15.7; 96 x 40 x 40, 40 5.48 / 5.89, 90
// 10.2 / 10.5, 150 15.9 / 16.2; 80^3, 56 23.0 / 23.1, 112 40.9 / 39.6.
// Deterministic form: a launch holds a slab of planes only, and lines that short
// meet the spills around their ends more often; a large grid makes up for it.  40^3
// cells, 100 sub-steps: r = 6 5.79 / 7.41 ms, r = 7 10.3 / 10.7, r = 8 10.9 / 11.7;
// 64^3, r = 8, 200 sub-steps 66.5 / 70.1; 96^3 225 / 225; 192^3 1800 / 1751; 128^3,
// 60 sub-steps 206 / 210.
constexpr int FLAT_THREE_WAVES_SUB = 96;
constexpr int64_t FLAT_DET_THREE_WAVES_LINES = 128 * 128;

static bool flat_three_waves(int r, const LineArgs &a)
{
    const bool subs = a.n_sub >= FLAT_THREE_WAVES_SUB;
    if (a.part) return r < 6 || (subs && (int64_t)a.nx * a.ny >= FLAT_DET_THREE_WAVES_LINES);
    return r != 6 || subs;
}

template <int R, bool LAB, bool DET>
static hipError_t launch_flat_rd(int mode, const LineArgs &a, hipStream_t st)
{
    if (mode == M_FP64) return launch_flat_f<Flat64<R>, LAB, DET>(a, st);
    if constexpr (R >= 4) {
        if constexpr (R == 6 || (DET && R > 6))
            if (!flat_three_waves(R, a)) return launch_flat_f<Flat<R, 2>, LAB, DET>(a, st);
        return launch_flat_f<Flat<R>, LAB, DET>(a, st);
    }
    return hipErrorInvalidValue;
}

template <int R, bool LAB>
static hipError_t launch_flat_r(int mode, const LineArgs &a, hipStream_t st)
{
    return a.part ? launch_flat_rd<R, LAB, true>(mode, a, st) : launch_flat_rd<R, LAB, false>(mode, a, st);
}

template <bool LAB>
static hipError_t launch_flat(int mode, int r, const LineArgs &a, hipStream_t st)
{
    // the deterministic form needs whole lines (one plane range per line, so
    // that each partial slot has one writer)
    if ((mode != M_FP32 && mode != M_FP64) || (a.part && a.n_seg != 1)) return hipErrorInvalidValue;
    switch (r) {
    case 3: return launch_flat_r<3, LAB>(mode, a, st);
    case 4: return launch_flat_r<4, LAB>(mode, a, st);
    case 5: return launch_flat_r<5, LAB>(mode, a, st);
    case 6: return launch_flat_r<6, LAB>(mode, a, st);
    case 7: return launch_flat_r<7, LAB>(mode, a, st);
    case 8: return launch_flat_r<8, LAB>(mode, a, st);
    default: return hipErrorInvalidValue;
    }
}

// The flat-layout fused step: FP32 mode, radii 4..8, and FP64, 3..8, atomic superposition or,
// with a.part and one segment per line, the partial slots of the
// deterministic form.  Returns hipErrorInvalidValue for other requests.
hipError_t launch_line_flat(int mode, int r, const LineArgs &a, hipStream_t st)
{
    return launch_flat<false>(mode, r, a, st);
}

// The same with the coefficients looked up per phase pair (a.label,
// a.lam_tab, a.n_phase).
hipError_t launch_line_flat_labels(int mode, int r, const LineArgs &a, hipStream_t st)
{
    return launch_flat<true>(mode, r, a, st);
}

}  // namespace fdirw
