// fdirw_flatwin.hip -- window kernels in the flat layout (gfx950, FP32 state, r
// = 4..8): the kernels of a source list (fdirw_kernels, the stored bank, the
// surrogate's targets and audit), the coarse build's kernels binned per block,
// and the kernels with a steady flow.  Per cell and sub-step the arithmetic is
// that of the fused step, so a source's kernel is the same bit for bit.
#include "fdirw_flat.h"
#include "fdirw_launch.h"

namespace fdirw {

// Window kernels of a source list (Sec. 3.1 of arXiv 2408.11376: the columns
// of P), Flat<R>::LPW sources per workgroup side by side.  M: FP32, or the
// 16-bit bank modes (FP32 state, the finished kernel rounded once).
// Bound by the LDS exchange like the fused step: 645 clocks per CU, window and
// sub-step at r = 8 (4.6 T cell-sub-steps/s; the segment layout 1,340), 89 at
// r = 4.  The bank of a 56 x 48 x 52 grid (r = 8, 200 sub-steps, FP16) is built
// in 35.5 ms, 57.9 ms in the segment layout; with few sub-steps the coefficient
// loads bound it and the segment layout is the faster one (flat_window_min_sub).
template <int M, int R>
__global__ void __launch_bounds__(FLAT_NT) __attribute__((amdgpu_waves_per_eu(3)))
flat_window_kernel(WindowArgs a)
{
    using F = Flat<R>;
    using T = Traits<M>;
    using B = typename T::B;
    constexpr int W = F::W, W2 = F::W2, W3 = F::W3, RUN = F::RUN, PAD = F::PAD, XLEN = F::XLEN;
    constexpr int SG = F::SG, LPW = F::LPW;
    __shared__ __align__(16) float xb[2 * LPW * XLEN];
    __shared__ double red[4];
    const int t = threadIdx.x;
    const int g = LPW == 1 ? 0 : t / SG;                      // the thread's window in the workgroup
    const int tg = t - g * SG;
    const int s0 = tg * RUN;
    float *const xg = xb + g * XLEN;                         // the window's first exchange buffer
    float *const xg1 = xg + LPW * XLEN;
    const float *lx = (const float *)a.lx;
    const FaceArrays<float> f{lx, lx + a.n, lx + 2 * a.n};
    const int64_t nxy = (int64_t)a.nx * a.ny;
    for (int i = t; i < 2 * LPW * XLEN; i += FLAT_NT) xb[i] = 0.0f;

    const int64_t b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    for (int64_t q0 = b * LPW; q0 < a.n_src; q0 += (int64_t)gridDim.x * LPW) {
        const int64_t q = q0 + g;
        const bool live = q < a.n_src;                         // a window past the list runs on zeros
        const int64_t s = !live ? 0 : a.src ? a.src[q] : q;
        const int sx = (int)(s % a.nx), sy = (int)((s / a.nx) % a.ny), sz = (int)(s / nxy);
        int s0v = live && tg < F::NACT ? s0 : F::NCELL;
        // the cell positions are recomputed where they are used instead of
        // being kept in registers across the sub-step loop
        asm volatile("" : "+v"(s0v));
        __syncthreads();                                       // LDS of the previous sources is no longer read
        FlatSeg<F> c;
        flat_load<F>(c, f, a.nx, a.ny, a.nz, sx, sy, sz, s0v);
        float Gs[RUN];
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            const FlatCell<F> p(s0v + k);
            Gs[k] = (p.ok && p.cx == R && p.cy == R && p.z == R) ? 1.0f : 0.0f;
        }
        flat_substeps<F, false>(Gs, c, xg, xg1, PAD + s0, a.n_sub, 0u);
        double ms = 0.0;
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            if constexpr (T::bank) Gs[k] = round_to<B>(Gs[k]);
            ms += (double)Gs[k];                               // cells past the window hold 0
        }
        const double m = flat_window_sum<F>(ms, red, g);
        if (tg == 0 && live && a.mass) a.mass[q] = m;
        const bool norm = !T::bank && a.normalize;
        const double inv = norm ? 1.0 / m : 1.0;
        asm volatile("" : "+v"(s0v));
        if (a.offset_major) {
            // bank layout [offset][z / zb][y][x][z % zb] (zb = 16 B /
            // element): the value at cell x = s + o is P[o][x]; cells outside
            // the domain are walls (0) and are not stored
            const int zb = T::bank && a.out_lp ? 8 : 4;
            const int64_t plane = (int64_t)((a.nz + zb - 1) / zb) * nxy * zb;
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                const FlatCell<F> p(s0v + k);
                const int X = sx - R + p.cx, Y = sy - R + p.cy, Z = sz - R + p.z;
                if (!p.ok || X < 0 || X >= a.nx || Y < 0 || Y >= a.ny || Z < 0 || Z >= a.nz) continue;
                const int64_t o = (int64_t)(p.z * W2 + p.col) * plane +
                                  ((int64_t)(Z / zb) * nxy + (int64_t)Y * a.nx + X) * zb + Z % zb;
                const float v = norm ? (float)((double)Gs[k] * inv) : Gs[k];
                if (T::bank && a.out_lp) ((B *)a.G)[o] = (B)v;
                else ((float *)a.G)[o] = v;
            }
        } else {
            // the kernel in (z, y, x) window order through the run region of
            // the second buffer (rewritten by every sub-step before a read),
            // so that the stores are coalesced
            float *stage = xg1 + PAD;
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                const FlatCell<F> p(s0v + k);
                if (p.ok) stage[p.z * W2 + p.col] = norm ? (float)((double)Gs[k] * inv) : Gs[k];
            }
            __syncthreads();
            if (live) {
                const int64_t o = q * (int64_t)W3;
                for (int w = tg; w < W3; w += SG) {
                    if (T::bank && a.out_lp) ((B *)a.G)[o + w] = (B)stage[w];
                    else ((float *)a.G)[o + w] = stage[w];
                }
            }
        }
    }
}

// The kernels of the coarse build: Flat<R>::LPW grouped sources per workgroup,
// each kernel's grouped cells summed per destination block into S[offset][I]
// (offset = I - J + K per axis, J the source's block).  Without a far field
// the kernel is renormalised to unit mass over the grouped cells; with one
// (SINK) the far-field cells absorb and the kernel keeps the mass that is
// left.  The bins of a window live in its exchange buffers, which are free
// after the sub-steps; consecutive cells of a run mostly fall in one bin and
// are added up in a register first.  An 80 x 64 x 72 build (porous medium, r = 8,
// 200 sub-steps) takes 64 ms, 117 ms in the segment layout.
template <int R, bool SINK>
__global__ void __launch_bounds__(FLAT_NT) __attribute__((amdgpu_waves_per_eu(3)))
flat_coarse_kernel(CoarseGenArgs a)
{
    using F = Flat<R>;
    constexpr int W = F::W, W3 = F::W3, RUN = F::RUN, PAD = F::PAD, XLEN = F::XLEN;
    constexpr int SG = F::SG, LPW = F::LPW;
    static_assert(RUN <= 32 && 3 * W <= SG && 2 * XLEN * sizeof(float) >= W3 * sizeof(double), "flags, tables, bins");
    __shared__ __align__(16) float xb[2 * LPW * XLEN];
    __shared__ double red[4];
    __shared__ int dest[LPW][3][W];                           // destination block of window row x / y / z, 0 .. 2K
    const int t = threadIdx.x;
    const int g = LPW == 1 ? 0 : t / SG;
    const int tg = t - g * SG;
    const int s0 = tg * RUN;
    float *const xg = xb + g * XLEN;
    double *const bins = (double *)(xb + g * 2 * XLEN);
    const float *lx = (const float *)a.lx;
    const FaceArrays<float> f{lx, lx + a.n, lx + 2 * a.n};
    const int64_t nxy = (int64_t)a.nx * a.ny;
    const int B = a.block, K = a.K, KW = 2 * K + 1, nb = KW * KW * KW;
    for (int i = t; i < 2 * LPW * XLEN; i += FLAT_NT) xb[i] = 0.0f;

    // runs of 128 groups of cells per XCD, the runs in turn: neighbours share
    // their coefficients in one L2, and clumps of grouped cells are spread over the
    // XCDs.  One range per XCD / groups one by one / runs of 32, 128, 512 (ms):
    // particle of radius 50 in 192^3 cells 112.6 / 137.9 / 108.8, 106.4, 111.9; 56^3
    // cells, r = 8, 5 % grouped in clumps 5.3 / 3.5 / 3.3, 3.5, 3.4, all grouped 44
    // each; 80 x 64 x 72 72.3 / 65.7 / 62.3, 63.4, 63.1
    const int b = xcd_runs((int)blockIdx.x, (int)gridDim.x, 128);
    for (int64_t q0 = (int64_t)b * LPW; q0 < a.n; q0 += (int64_t)gridDim.x * LPW) {
        // sources outside every group are skipped (when all of the
        // workgroup's are, the whole trip: uniform per block)
        bool any = false, live = false;
#pragma unroll
        for (int h = 0; h < LPW; ++h) {
            const bool lh = q0 + h < a.n && a.node[q0 + h] >= 0;
            any = any || lh;
            if (h == g) live = lh;
        }
        if (!any) continue;
        const int64_t s = q0 + g < a.n ? q0 + g : 0;
        const int sx = (int)(s % a.nx), sy = (int)((s / a.nx) % a.ny), sz = (int)(s / nxy);
        const int jx = sx / B, jy = sy / B, jz = sz / B;
        int s0v = live && tg < F::NACT ? s0 : F::NCELL;
        asm volatile("" : "+v"(s0v));
        __syncthreads();                                       // LDS of the previous sources is no longer read
        if (tg < 3 * W) {
            const int ax = tg / W, j = tg - ax * W;
            const int at = (ax == 0 ? sx : ax == 1 ? sy : sz) - R + j;
            dest[g][ax][j] = (at < 0 ? 0 : at / B) - (ax == 0 ? jx : ax == 1 ? jy : jz) + K;
        }
        // which cells of the run are grouped / far-field cells, read in grid
        // order and changed to the run order in LDS: 1 grouped, 2 far field, 0
        // else (the coefficients come straight from memory, see flat_load)
        int at = tg;
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int j = 0; j < (W3 + SG - 1) / SG; ++j) {
            const int w = at + j * SG;
            const int row = w / W, cx = w - row * W, zw = row / W, cy = row - zw * W;
            const int X = sx - R + cx, Y = sy - R + cy, Z = sz - R + zw;
            float v = 0.0f;
            if (live && w < W3 && X >= 0 && X < a.nx && Y >= 0 && Y < a.ny && Z >= 0 && Z < a.nz) {
                const int nd = a.node[(int64_t)Z * nxy + (int64_t)Y * a.nx + X];
                v = nd >= 0 ? 1.0f : nd == COARSE_RESERVOIR ? 2.0f : 0.0f;
            }
            if (w < W3) xg[PAD + cy * F::PY + cx * W + zw] = v;
        }
        __syncthreads();
        unsigned grp = 0u, sink = 0u;
        {
            float v[RUN];
            read_run<RUN, 0>(xg, PAD + s0, v);             // unused cells hold 0
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                grp |= v[k] == 1.0f ? 1u << k : 0u;
                if constexpr (SINK) sink |= v[k] == 2.0f ? 1u << k : 0u;
            }
        }
        FlatSeg<F> c;
        flat_load<F>(c, f, a.nx, a.ny, a.nz, sx, sy, sz, s0v);
        float Gs[RUN];
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            const FlatCell<F> p(s0v + k);
            Gs[k] = (p.ok && p.cx == R && p.cy == R && p.z == R) ? 1.0f : 0.0f;
        }
        flat_substeps<F, SINK>(Gs, c, xg, xg + LPW * XLEN, PAD + s0, a.n_sub, sink);
        double part = 0.0;
#pragma unroll
        for (int k = 0; k < RUN; ++k) part += (grp >> k) & 1u ? (double)Gs[k] : 0.0;
        const double m = flat_window_sum<F>(part, red, g);
        const double inv = SINK ? 1.0 : 1.0 / m;
        for (int o = tg; o < nb; o += SG) bins[o] = 0.0;
        __syncthreads();
        asm volatile("" : "+v"(s0v));
        int cur = -1;
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            if ((grp >> k) & 1u && Gs[k] != 0.0f) {
                const FlatCell<F> p(s0v + k);
                const int o = (dest[g][2][p.z] * KW + dest[g][1][p.cy]) * KW + dest[g][0][p.cx];
                if (o != cur) {
                    if (cur >= 0) atomicAdd(&bins[cur], sum);
                    cur = o;
                    sum = 0.0;
                }
                sum += (double)Gs[k] * inv;
            }
        }
        if (cur >= 0) atomicAdd(&bins[cur], sum);
        __syncthreads();
        // the nonzero bins leave; all are 0 again (the exchange padding has to be)
        for (int o = tg; o < nb; o += SG) {
            const double v = bins[o];
            if (v != 0.0) {
                const int oz = o / (KW * KW), oy = (o / KW) % KW, ox = o % KW;
                const int64_t I = ((int64_t)(jz + oz - K) * a.ncy + (jy + oy - K)) * a.ncx + (jx + ox - K);
                atomicAdd(&a.S[(int64_t)o * a.n_nodes + I], v);
                bins[o] = 0.0;
            }
        }
    }
}

// Window kernels with a steady flow (the flow_window_kernel update: diffusion
// plus first-order upwind advection through every face, far-field cells held
// at 0) in the flat layout, FP32: Flat<R>::LPW sources per workgroup side by
// side (as many as flat_line runs lines), the seven update coefficients of a
// thread's RUN cells in registers, the same neighbour reads as flat_line and
// the same FMA sequence per cell as flow_window_kernel (diagonal, then x-,
// x+, y-, y+, z-, z+).  G leaves in the window's (z, y, x) order through the
// LDS run region of the window's second exchange buffer (coalesced stores).
// A window group past the list, or on a source outside every group, runs on
// zeros and writes nothing.
template <int R>
__global__ void __launch_bounds__(FLAT_NT) __attribute__((amdgpu_waves_per_eu(2)))
flat_flow_kernel(FlowArgs a)
{
    using F = Flat<R>;
    constexpr int W = F::W, W2 = F::W2, W3 = F::W3, RUN = F::RUN, PAD = F::PAD, XLEN = F::XLEN;
    constexpr int SG = F::SG, LPW = F::LPW;
    static_assert(RUN <= 32, "sink flags in one word");
    __shared__ __align__(16) float xb[2 * LPW * XLEN];
    __shared__ double red[4];
    const int t = threadIdx.x;
    const int g = LPW == 1 ? 0 : t / SG;                      // the thread's window in the workgroup
    const int tg = t - g * SG;
    const int s0 = tg * RUN;
    const bool act = tg < F::NACT;
    const int own = PAD + s0;
    float *const xg = xb + g * XLEN;                         // the window's first exchange buffer
    const float *lx = (const float *)a.lam, *ly = lx + a.n, *lz = ly + a.n;
    const double *ux = a.u, *uy = ux + a.n, *uz = uy + a.n;
    const double cour = a.dt / a.h;
    const int64_t nxy = (int64_t)a.nx * a.ny;
    for (int i = t; i < 2 * LPW * XLEN; i += F::NT) xb[i] = 0.0f;

    for (int64_t q0 = (int64_t)blockIdx.x * LPW; q0 < a.n_src; q0 += (int64_t)gridDim.x * LPW) {
        // the sources of the workgroup's windows: those outside every group
        // are skipped (when all are, the whole step: uniform per block)
        bool any = false, live = false;
        int64_t src = 0;
#pragma unroll
        for (int h = 0; h < LPW; ++h) {
            if (q0 + h < a.n_src) {
                const int64_t sh = a.src ? a.src[q0 + h] : a.src_base + q0 + h;
                const bool lh = !(a.node && a.node[sh] < 0);
                any = any || lh;
                if (h == g) { live = lh; src = sh; }
            }
        }
        if (!any) continue;
        const int64_t q = q0 + g;
        __syncthreads();                                       // LDS of the previous sources is no longer read
        const int sx = (int)(src % a.nx), sy = (int)((src / a.nx) % a.ny), sz = (int)(src / nxy);
        int s0v = act ? s0 : F::NCELL;
        asm volatile("" : "+v"(s0v));
        float c0[RUN], cxm[RUN], cxp[RUN], cym[RUN], cyp[RUN], czm[RUN], czp[RUN];
        unsigned sink = 0;
        float Gs[RUN];
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            const FlatCell<F> p(s0v + k);
            const int cx = p.cx, cy = p.cy, zw = p.z;
            const int X = sx - R + cx, Y = sy - R + cy, Z = sz - R + zw;
            const bool in = live && p.ok && X >= 0 && X < a.nx && Y >= 0 && Y < a.ny && Z >= 0 && Z < a.nz;
            // per face: lambda (diffusion) and the Courant number of the flow
            // (through the -x, +x, -y, +y, -z, +z faces); the inflow adds to
            // the neighbour's coefficient, the outflow leaves the diagonal
            float fl[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, vl[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (in) {
                const int64_t c = (int64_t)Z * nxy + (int64_t)Y * a.nx + X;
                if (cx > 0 && X > 0) { fl[0] = lx[c - 1]; vl[0] = (float)(ux[c - 1] * cour); }
                if (cx < W - 1 && X < a.nx - 1) { fl[1] = lx[c]; vl[1] = (float)(ux[c] * cour); }
                if (cy > 0 && Y > 0) { fl[2] = ly[c - a.nx]; vl[2] = (float)(uy[c - a.nx] * cour); }
                if (cy < W - 1 && Y < a.ny - 1) { fl[3] = ly[c]; vl[3] = (float)(uy[c] * cour); }
                if (zw > 0 && Z > 0) { fl[4] = lz[c - nxy]; vl[4] = (float)(uz[c - nxy] * cour); }
                if (zw < W - 1 && Z < a.nz - 1) { fl[5] = lz[c]; vl[5] = (float)(uz[c] * cour); }
                if (a.node && a.node[c] == COARSE_RESERVOIR) sink |= 1u << k;
            }
            double out = 0.0, lam = 0.0;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                lam += (double)fl[2 * ax] + (double)fl[2 * ax + 1];
                out += (vl[2 * ax] < 0.f ? -(double)vl[2 * ax] : 0.0) + (vl[2 * ax + 1] > 0.f ? (double)vl[2 * ax + 1] : 0.0);
            }
            c0[k] = (float)(1.0 - lam - out);
            cxm[k] = fl[0] + (vl[0] > 0.f ? vl[0] : 0.f);
            cxp[k] = fl[1] + (vl[1] < 0.f ? -vl[1] : 0.f);
            cym[k] = fl[2] + (vl[2] > 0.f ? vl[2] : 0.f);
            cyp[k] = fl[3] + (vl[3] < 0.f ? -vl[3] : 0.f);
            czm[k] = fl[4] + (vl[4] > 0.f ? vl[4] : 0.f);
            czp[k] = fl[5] + (vl[5] < 0.f ? -vl[5] : 0.f);
            Gs[k] = (live && p.ok && cx == R && cy == R && zw == R) ? 1.0f : 0.0f;
        }
        auto substep = [&](float *buf) {
            // (raising the wave priority after the barrier, as flat_line
            // does, measured 6 % slower here)
#pragma unroll
            for (int qd = 0; qd < RUN / 4; ++qd)
                *(float4 *)(buf + own + 4 * qd) = make_float4(Gs[4 * qd], Gs[4 * qd + 1], Gs[4 * qd + 2], Gs[4 * qd + 3]);
            __syncthreads();
            float zlo, zhi;
            float v0[RUN], v1[RUN];
            read_x_runs<RUN, W>(buf, own, Gs, v0, v1, zlo, zhi);
            float acc2[RUN];
#pragma unroll
            for (int k = 0; k < RUN; ++k) acc2[k] = __builtin_fmaf(cxm[k], v0[k], c0[k] * Gs[k]);
            read_run<RUN, -F::PY>(buf, own, v0);
#pragma unroll
            for (int k = 0; k < RUN; ++k) acc2[k] = __builtin_fmaf(cxp[k], v1[k], acc2[k]);
            read_run<RUN, F::PY>(buf, own, v1);
#pragma unroll
            for (int k = 0; k < RUN; ++k) acc2[k] = __builtin_fmaf(cym[k], v0[k], acc2[k]);
#pragma unroll
            for (int k = 0; k < RUN; ++k) acc2[k] = __builtin_fmaf(cyp[k], v1[k], acc2[k]);
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                float v = __builtin_fmaf(czm[k], k > 0 ? Gs[k - 1] : zlo, acc2[k]);
                v = __builtin_fmaf(czp[k], k < RUN - 1 ? Gs[k + 1] : zhi, v);
                acc2[k] = v;
            }
#pragma unroll
            for (int k = 0; k < RUN; ++k) Gs[k] = (sink >> k) & 1u ? 0.0f : acc2[k];
        };
        int step = 0;
        for (; step + 1 < a.n_sub; step += 2) {
            substep(xg);
            substep(xg + LPW * XLEN);
        }
        if (step < a.n_sub) substep(xg);
        // mass: per thread in cell order, xor butterfly per wave, the
        // window's waves in order
        double ms = 0.0;
        if (act) {
#pragma unroll
            for (int k = 0; k < RUN; ++k) ms += (double)Gs[k];
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) ms += __shfl_xor(ms, off, 64);
        __syncthreads();                                       // every exchange read is done
        if ((t & 63) == 0) red[t >> 6] = ms;
        if (a.G && live) {
            // the kernel in (z, y, x) window order into the run region of
            // the second buffer (rewritten by every sub-step before a read)
            float *stage = xg + LPW * XLEN + PAD;
            // positions recomputed, not kept across the sub-steps: at 20 cells per
            // thread they were spilled (16,000 sources, ms: r = 6, 113 sub-steps
            // 2.60 -> 2.12, r = 7, 153 5.64 -> 4.86, r = 8, 200 6.60 -> 5.96)
            asm volatile("" : "+v"(s0v));
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                const FlatCell<F> p(s0v + k);
                if (p.ok) stage[p.z * W2 + p.col] = Gs[k];
            }
        }
        __syncthreads();
        if (tg == 0 && live && a.mass) {
            double m;
            if constexpr (SG == 256) m = ((red[0] + red[1]) + red[2]) + red[3];
            else if constexpr (SG == 128) m = red[2 * g] + red[2 * g + 1];
            else m = red[g];
            a.mass[q] = m;
        }
        if (a.G && live) {
            const float *stage = xg + LPW * XLEN + PAD;
            float *go = (float *)a.G + q * (int64_t)W3;
            for (int w = tg; w < W3; w += SG) go[w] = stage[w];
        }
    }
}

template <int R>
static hipError_t launch_flow_flat_r(const FlowArgs &a, hipStream_t st)
{
    const int64_t groups = (a.n_src + Flat<R>::LPW - 1) / Flat<R>::LPW;
    const int64_t nblk = groups < 65536 * 16 ? groups : 65536 * 16;
    if (nblk <= 0) return hipSuccess;
    hipLaunchKernelGGL((flat_flow_kernel<R>), dim3((unsigned)nblk), dim3(FLAT_NT), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_flow_flat(int r, const FlowArgs &a, hipStream_t st)
{
    switch (r) {
    case 4: return launch_flow_flat_r<4>(a, st);
    case 5: return launch_flow_flat_r<5>(a, st);
    case 6: return launch_flow_flat_r<6>(a, st);
    case 7: return launch_flow_flat_r<7>(a, st);
    case 8: return launch_flow_flat_r<8>(a, st);
    default: return hipErrorInvalidValue;
    }
}

// Workgroups of a launch over `groups` groups of sources (grid-stride beyond).
static unsigned flat_grid(int64_t groups)
{
    return (unsigned)(groups < 65536 * 16 ? groups : 65536 * 16);
}

template <int M, int R> static hipError_t launch_window_flat_mr(const WindowArgs &a, hipStream_t st)
{
    const int64_t groups = (a.n_src + Flat<R>::LPW - 1) / Flat<R>::LPW;
    if (groups <= 0) return hipSuccess;
    hipLaunchKernelGGL((flat_window_kernel<M, R>), dim3(flat_grid(groups)), dim3(FLAT_NT), 0, st, a);
    return hipGetLastError();
}

template <int M> static hipError_t launch_window_flat_m(int r, const WindowArgs &a, hipStream_t st)
{
    switch (r) {
    case 4: return launch_window_flat_mr<M, 4>(a, st);
    case 5: return launch_window_flat_mr<M, 5>(a, st);
    case 6: return launch_window_flat_mr<M, 6>(a, st);
    case 7: return launch_window_flat_mr<M, 7>(a, st);
    case 8: return launch_window_flat_mr<M, 8>(a, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_window_flat(int mode, int r, const WindowArgs &a, hipStream_t st)
{
    switch (mode) {
    case M_FP32: return launch_window_flat_m<M_FP32>(r, a, st);
    case M_F16BANK: return launch_window_flat_m<M_F16BANK>(r, a, st);
    case M_BF16BANK: return launch_window_flat_m<M_BF16BANK>(r, a, st);
    default: return hipErrorInvalidValue;
    }
}

template <int R, bool SINK> static hipError_t launch_coarse_flat_r(const CoarseGenArgs &a, hipStream_t st)
{
    const int64_t groups = (a.n + Flat<R>::LPW - 1) / Flat<R>::LPW;
    if (groups <= 0) return hipSuccess;
    hipLaunchKernelGGL((flat_coarse_kernel<R, SINK>), dim3(flat_grid(groups)), dim3(FLAT_NT), 0, st, a);
    return hipGetLastError();
}

template <bool SINK> static hipError_t launch_coarse_flat_s(int r, const CoarseGenArgs &a, hipStream_t st)
{
    switch (r) {
    case 4: return launch_coarse_flat_r<4, SINK>(a, st);
    case 5: return launch_coarse_flat_r<5, SINK>(a, st);
    case 6: return launch_coarse_flat_r<6, SINK>(a, st);
    case 7: return launch_coarse_flat_r<7, SINK>(a, st);
    case 8: return launch_coarse_flat_r<8, SINK>(a, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_coarse_flat(int sink, int r, const CoarseGenArgs &a, hipStream_t st)
{
    return sink ? launch_coarse_flat_s<true>(r, a, st) : launch_coarse_flat_s<false>(r, a, st);
}

}  // namespace fdirw
