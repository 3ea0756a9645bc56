// fdirw_flat.h -- device-side building blocks of the flat window layout (gfx950,
// FP32 state), shared by the fused step (fdirw_flat.hip) and the window kernels
// (fdirw_flatwin.hip).
//
// A workgroup of 256 threads holds one window (r = 7, 8), two (r = 5, 6) or
// four (r = 4) side by side.  The W^3 cells of a window are numbered flat, i =
// cy PY + cx W + z (z fastest), and thread t of its SG threads owns the RUN
// consecutive cells [RUN t, RUN t + RUN) in registers; neighbours outside the
// run come from an LDS copy of the window (double-buffered, one barrier per
// sub-step).  fdirw_flat.hip describes the layout in full.
#pragma once
#include "fdirw_device.h"

namespace fdirw {

constexpr int FLAT_NT = 256;

// Cells per thread when sg threads share a window of w3 cells: a multiple of
// 4 whose quarter is odd, so that the 16-byte run starts of 16 consecutive
// lanes fall on 16 distinct groups of four LDS banks (a quarter of 2 or 4
// would put two or four lanes on one group: 2- or 4-way conflicts on every
// exchange access).
constexpr int odd_run(int need)
{
    int q = (need + 3) / 4;
    if (q % 2 == 0) ++q;
    return 4 * q;
}
// Flat cells of a window of radius R: W planes of W^2 cells at a pitch that is
// a multiple of 4 (the last plane without its unused cells).
constexpr int flat_cells(int R)
{
    const int w = 2 * R + 1, w2 = w * w;
    return (w - 1) * ru(w2, 4) + w2;
}
constexpr int run_for(int w3, int sg) { return odd_run((w3 + sg - 1) / sg); }

// Threads per source line of the fused step at radius R: 64, 128 or 256,
// whichever leaves the fewest of a 256-thread workgroup's lanes idle with at
// most 20 cells per thread (the register budget of three waves per SIMD); the
// workgroup runs 256 / that many lines side by side.  r = 4: 4 lines of 64
// threads x 12 cells (63 busy); r = 5, 6: 2 lines of 128 x 12 / 20 (114 /
// 112 busy); r = 7, 8: one line of 256 x 20 (171 / 249 busy).
constexpr int line_threads(int R)
{
    const int w3 = flat_cells(R);
    int best = 256, best_busy = -1;
    for (int sg = 256; sg >= 64; sg /= 2) {
        const int run = run_for(w3, sg);
        if (run > 20) continue;
        const int busy = (w3 + run - 1) / run * (256 / sg);
        if (busy > best_busy) { best_busy = busy; best = sg; }
    }
    return best;
}

template <int R, int SG_ = line_threads(R)> struct Flat {
    static constexpr int W = 2 * R + 1;
    static constexpr int W2 = W * W;
    static constexpr int W3 = W2 * W;
    static constexpr int PY = ru(W2, 4);                       // pitch of a window y plane: its W^2 cells, then unused ones
    static constexpr int NCELL = (W - 1) * PY + W2;            // flat cells, the unused ones included
    static constexpr int NT = 256;                             // threads per workgroup
    static constexpr int SG = SG_;                             // threads per window
    static constexpr int LPW = NT / SG;                        // windows per workgroup
    static constexpr int RUN = run_for(NCELL, SG);             // cells per thread
    static constexpr int NACT = (NCELL + RUN - 1) / RUN;       // threads of a window that own cells
    static constexpr int PAD = ru(PY + 4, 4);                  // zero cells before and after
    // one exchange buffer of one window: its threads past the window (index
    // >= NACT) run the sub-steps too, on zero values and coefficients,
    // writing zeros after it
    static constexpr int XLEN = ru(PAD + SG * RUN + PY + 8, 4);
    static_assert(NT % SG == 0 && NACT <= SG, "window does not fit its threads");
};

typedef float v4f __attribute__((ext_vector_type(4)));

// Misalignment m in [0, 4) of a neighbour run at offset d from an aligned start.
constexpr int mis(int d) { return ((d % 4) + 4) % 4; }

// Reads the RUN values at buf[base + d .. + RUN) (base 4-aligned) as aligned
// 128-bit loads into v[0 .. RUN).
template <int RUN, int D>
__device__ __forceinline__ void read_run(const float *__restrict__ buf, int base, float (&v)[RUN])
{
    constexpr int M = mis(D);
    constexpr int NC = (RUN + M + 3) / 4;
    const v4f *p = (const v4f *)(buf + base + D - M);
    float t[4 * NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        v4f q = p[c];
        // keep the whole 16-byte load (otherwise the unused lanes of the
        // first / last chunk let the compiler split it into 32-bit loads)
        asm("" : "+v"(q));
        t[4 * c] = q.x; t[4 * c + 1] = q.y; t[4 * c + 2] = q.z; t[4 * c + 3] = q.w;
    }
#pragma unroll
    for (int k = 0; k < RUN; ++k) v[k] = t[k + M];
}

// Reads the 4 NC values at buf[base + OFF .. + 4 NC) (base + OFF 4-aligned) as
// aligned 128-bit loads into t.
template <int NC, int OFF>
__device__ __forceinline__ void read_chunks(const float *__restrict__ buf, int base, float (&t)[4 * NC])
{
    const v4f *p = (const v4f *)(buf + base + OFF);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        v4f q = p[c];
        asm("" : "+v"(q));
        t[4 * c] = q.x; t[4 * c + 1] = q.y; t[4 * c + 2] = q.z; t[4 * c + 3] = q.w;
    }
}

// The runs at -W and +W (v0, v1) and the cells next to the run's ends (zlo,
// zhi) for the run of g at buf[base .. + RUN).  Where RUN > W they are the W
// cells before the run (previous thread) and after it (next thread) plus
// RUN - W cells of the own run (registers); else the aligned spans of read_run.
template <int RUN, int W>
__device__ __forceinline__ void read_x_runs(const float *__restrict__ buf, int base, const float (&g)[RUN],
                                            float (&v0)[RUN], float (&v1)[RUN], float &zlo, float &zhi)
{
    if constexpr (RUN > W) {
        constexpr int NC = (W + 3) / 4;
        float tp[4 * NC], tn[4 * NC];
        read_chunks<NC, -4 * NC>(buf, base, tp);
        read_chunks<NC, RUN>(buf, base, tn);
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            v0[k] = k < W ? tp[4 * NC - W + k] : g[k < W ? 0 : k - W];
            v1[k] = k < RUN - W ? g[k < RUN - W ? k + W : 0] : tn[k + W - RUN];
        }
        zlo = tp[4 * NC - 1];
        zhi = tn[0];
    } else {
        zlo = buf[base - 1];
        zhi = buf[base + RUN];
        read_run<RUN, -W>(buf, base, v0);
        read_run<RUN, W>(buf, base, v1);
    }
}

template <int R> struct FlatSeg {
    static constexpr int RUN = Flat<R>::RUN;
    float xm[RUN], xp[RUN], ym[RUN], yp[RUN];
    float zf[RUN + 1];        // zf[k]: face between run cells k - 1 and k
    float diag[RUN];
};

// Window position of flat cell i = cy PY + cx W + z (any i >= 0): column col =
// cy W + cx, height z; ok: the cell exists (unused cells of a plane's pitch
// have coefficients 0 and hold 0).
template <int R> struct FlatCell {
    int col, cx, cy, z;
    bool ok;
    __device__ __forceinline__ explicit FlatCell(int i)
    {
        using F = Flat<R>;
        cy = i / F::PY;
        const int rem = i - cy * F::PY;
        cx = rem / F::W;
        z = rem - cx * F::W;
        col = cy * F::W + cx;
        ok = i < F::NCELL && rem < F::W2;
    }
};

// Coefficients of the run that starts at cell s0v (Flat<R>::NCELL: no cells,
// all 0) of the window of (sx, sy, sz), through the owned-face accessor f.
// (A lane's run touches its own cache lines, so these loads take 25,600 line
// accesses per source at r = 8.  Reading the faces in grid order and changing
// to the run order in LDS takes a third of their time, but its LDS accesses
// delay the other workgroups' sub-steps, under which these loads mostly
// disappear: 239 against 222 ms per 96^3 step at r = 8.)
template <int R, typename Faces>
__device__ __forceinline__ void flat_load(FlatSeg<R> &c, const Faces &f, int nx, int ny, int nz, int sx, int sy,
                                          int sz, int s0v)
{
    using F = Flat<R>;
    constexpr int W = F::W, RUN = F::RUN;
    const int64_t nxy = (int64_t)nx * ny;
#pragma unroll
    for (int k = 0; k < RUN; ++k) {
        const FlatCell<R> p(s0v + k);
        const int X = sx - R + p.cx, Y = sy - R + p.cy, Z = sz - R + p.z;
        const bool in = p.ok && X >= 0 && X < nx && Y >= 0 && Y < ny && Z >= 0 && Z < nz;
        float xm = 0.f, xp = 0.f, ym = 0.f, yp = 0.f, zf = 0.f;
        if (in) {
            const int64_t i = (int64_t)Z * nxy + (int64_t)Y * nx + X;
            if (p.cx < W - 1) xp = f.x(i, X);
            if (p.cx > 0 && X > 0) xm = f.x(i - 1, X - 1);
            if (p.cy < W - 1) yp = f.y(i, Y);
            if (p.cy > 0 && Y > 0) ym = f.y(i - nx, Y - 1);
            if (p.z > 0 && Z > 0) zf = f.z(i - nxy, Z - 1);
        }
        c.xm[k] = xm; c.xp[k] = xp; c.ym[k] = ym; c.yp[k] = yp; c.zf[k] = zf;
    }
    {
        // face above the run's top cell: the face below cell s0v + RUN
        const FlatCell<R> p(s0v + RUN);
        const int X = sx - R + p.cx, Y = sy - R + p.cy, Z = sz - R + p.z;
        float zf = 0.f;
        if (p.ok && p.z > 0 && X >= 0 && X < nx && Y >= 0 && Y < ny && Z > 0 && Z < nz)
            zf = f.z((int64_t)(Z - 1) * nxy + (int64_t)Y * nx + X, Z - 1);
        c.zf[RUN] = zf;
    }
#pragma unroll
    for (int k = 0; k < RUN; ++k) {
        float s = c.xm[k] + c.xp[k];
        s = s + c.ym[k];
        s = s + c.yp[k];
        s = s + c.zf[k];
        s = s + c.zf[k + 1];
        c.diag[k] = 1.0f - s;
    }
}

// n_sub explicit sub-steps of the run G, exchange buffers buf0 and buf1
// alternating; own: the run's first cell in them.  Every thread of the
// workgroup runs them without a branch (an idle thread's run is zeros: its
// writes land in the zero band after the window), so that the new values need
// not be merged with the old ones of idle threads; two sub-steps per trip let
// the registers of G and of the new values alternate instead of being copied
// back.  SINK: the cells of the run whose bit is set in sink are held at 0
// after every sub-step.
template <int R, bool SINK>
__device__ __forceinline__ void flat_substeps(float (&Gs)[Flat<R>::RUN], const FlatSeg<R> &c, float *buf0,
                                              float *buf1, int own, int n_sub, unsigned sink)
{
    using F = Flat<R>;
    constexpr int W = F::W, PY = F::PY, RUN = F::RUN;
    auto substep = [&](float *buf) {
        // a wave that has passed the barrier issues ahead of the
        // other workgroup's wave on its SIMD until its next write
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int q = 0; q < RUN / 4; ++q)
            *(float4 *)(buf + own + 4 * q) = make_float4(Gs[4 * q], Gs[4 * q + 1], Gs[4 * q + 2], Gs[4 * q + 3]);
        __syncthreads();
        __builtin_amdgcn_s_setprio(1);
        // the neighbour runs are requested two directions ahead
        // of their use (two buffers), so their LDS latency
        // overlaps the FMAs of the previous direction
        float zlo, zhi;
        float v0[RUN], v1[RUN];
        read_x_runs<RUN, W>(buf, own, Gs, v0, v1, zlo, zhi);
        float acc2[RUN];
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            float a2 = c.diag[k] * Gs[k];
            a2 = __builtin_fmaf(c.zf[k], k > 0 ? Gs[k - 1] : zlo, a2);
            acc2[k] = __builtin_fmaf(c.zf[k + 1], k < RUN - 1 ? Gs[k + 1] : zhi, a2);
        }
#pragma unroll
        for (int k = 0; k < RUN; ++k) acc2[k] = __builtin_fmaf(c.xm[k], v0[k], acc2[k]);
        read_run<RUN, -PY>(buf, own, v0);
#pragma unroll
        for (int k = 0; k < RUN; ++k) acc2[k] = __builtin_fmaf(c.xp[k], v1[k], acc2[k]);
        read_run<RUN, PY>(buf, own, v1);
#pragma unroll
        for (int k = 0; k < RUN; ++k) acc2[k] = __builtin_fmaf(c.ym[k], v0[k], acc2[k]);
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            Gs[k] = __builtin_fmaf(c.yp[k], v1[k], acc2[k]);
            if constexpr (SINK) Gs[k] = (sink >> k) & 1u ? 0.0f : Gs[k];
        }
    };
    int step = 0;
    for (; step + 1 < n_sub; step += 2) {
        substep(buf0);
        substep(buf1);
    }
    if (step < n_sub) substep(buf0);
}

// Sum of ms over the threads of window g of the workgroup (the same in each):
// xor butterfly per wave, the window's waves in order.  red: 4 doubles.
// Every thread calls it (two barriers; LDS reads before the call are done
// after it).
template <int R> __device__ __forceinline__ double flat_window_sum(double ms, double *red, int g)
{
    constexpr int SG = Flat<R>::SG;
    const int t = threadIdx.x;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ms += __shfl_xor(ms, off, 64);
    __syncthreads();
    if ((t & 63) == 0) red[t >> 6] = ms;
    __syncthreads();
    if constexpr (SG == 256) return ((red[0] + red[1]) + red[2]) + red[3];
    else if constexpr (SG == 128) return red[2 * g] + red[2 * g + 1];
    else return red[g];
}

}  // namespace fdirw
