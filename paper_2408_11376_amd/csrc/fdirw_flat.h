// fdirw_flat.h -- device-side building blocks of the flat window layout (gfx950,
// FP32 or FP64 state), shared by the fused step (fdirw_flat.hip) and the window
// kernels (fdirw_flatwin.hip).
//
// FP32: a workgroup of 256 threads holds one window (r = 7, 8), two (r = 5, 6)
// or four (r = 4) side by side; FP64: one window of 64 to 576 threads.  The W^3 cells of a window are numbered flat, i =
// cy PY + cx W + z (z fastest), and thread t of its SG threads owns the RUN
// consecutive cells [RUN t, RUN t + RUN) in registers; neighbours outside the
// run come from an LDS copy of the window (double-buffered, one barrier per
// sub-step).  fdirw_flat.hip describes the layout in full.
#pragma once
#include "fdirw_device.h"

namespace fdirw {

constexpr int FLAT_NT = 256;

// Cells per thread when sg threads share a window of w3 cells: a multiple of
// a 16-byte chunk's ch cells with an odd quotient, so that the 16-byte run
// starts of 16 consecutive lanes fall on 16 distinct groups of four LDS banks
// (an even quotient would put two or four lanes on one group: 2- or 4-way
// conflicts on every exchange access).
constexpr int odd_run(int need, int ch)
{
    int q = (need + ch - 1) / ch;
    if (q % 2 == 0) ++q;
    return ch * q;
}
// Flat cells of a window of radius R: W planes of W^2 cells at a pitch that is
// a multiple of the chunk's ch cells (the last plane without its unused cells).
constexpr int flat_cells(int R, int ch)
{
    const int w = 2 * R + 1, w2 = w * w;
    return (w - 1) * ru(w2, ch) + w2;
}
constexpr int run_for(int w3, int sg) { return odd_run((w3 + sg - 1) / sg, 4); }

// Threads per source line of the fused step at radius R: 64, 128 or 256,
// whichever leaves the fewest of a 256-thread workgroup's lanes idle with at
// most 20 cells per thread (the register budget of three waves per SIMD); the
// workgroup runs 256 / that many lines side by side.  r = 4: 4 lines of 64
// threads x 12 cells (63 busy); r = 5, 6: 2 lines of 128 x 12 / 20 (114 /
// 112 busy); r = 7, 8: one line of 256 x 20 (171 / 249 busy).
constexpr int line_threads(int R)
{
    const int w3 = flat_cells(R, 4);
    int best = 256, best_busy = -1;
    for (int sg = 256; sg >= 64; sg /= 2) {
        const int run = run_for(w3, sg);
        if (run > 20) continue;
        const int busy = (w3 + run - 1) / run * (256 / sg);
        if (busy > best_busy) { best_busy = busy; best = sg; }
    }
    return best;
}

// A window of radius R_ with state S_: SG_ threads of a workgroup of NT_, RUN_
// cells each.
template <typename S_, int R_, int NT_, int SG_, int RUN_, int WPE_> struct FlatGeo {
    using S = S_;
    static constexpr int R = R_;
    static constexpr int CH = 16 / (int)sizeof(S);             // cells of a 16-byte chunk
    static constexpr int W = 2 * R + 1;
    static constexpr int W2 = W * W;
    static constexpr int W3 = W2 * W;
    static constexpr int PY = ru(W2, CH);                      // pitch of a window y plane: its W^2 cells, then unused ones
    static constexpr int NCELL = (W - 1) * PY + W2;            // flat cells, the unused ones included
    static constexpr int NT = NT_;                             // threads per workgroup
    static constexpr int SG = SG_;                             // threads per window
    static constexpr int LPW = NT / SG;                        // windows per workgroup
    static constexpr int RUN = RUN_;                           // cells per thread
    static constexpr int NACT = (NCELL + RUN - 1) / RUN;       // threads of a window that own cells
    static constexpr int PAD = ru(PY + CH, CH);                // zero cells before and after
    // one exchange buffer of one window: its threads past the window (index
    // >= NACT) run the sub-steps too, on zero values and coefficients,
    // writing zeros after it
    static constexpr int XLEN = ru(PAD + SG * RUN + PY + 2 * CH, CH);
    static constexpr int WPE = WPE_;                           // waves per SIMD the registers are budgeted for
    static constexpr int EDGE = 2 * (NT / 64 + 1);             // one value per wave and parity, and a 0
    static_assert(NT % SG == 0 && SG % 64 == 0 && NACT <= SG, "window does not fit its threads");
    static_assert(RUN % CH == 0 && RUN / CH % 2 == 1, "run");
};

// FP32: see line_threads.
template <int R, int WPE = 3>
using Flat = FlatGeo<float, R, FLAT_NT, line_threads(R), run_for(flat_cells(R, 4), line_threads(R)), WPE>;

// FP64, one window per workgroup (r = 3..8): 10 cells per thread at r = 6 and 8
// (256 and 512 threads of two waves per SIMD: 221 and 493 busy), 6 at the others
// (three waves per SIMD; r = 3: 59 of 64 threads busy, 4: 123 of 128, 5: 224 of
// 256, 7: 565 of 576).  Measured (61 x 57 x 60 cells, ms per step): r = 4 6 cells
// 4.4, 10 6.6; r = 5 6 13.4, 10 19.7, 14 13.8; r = 6 6 43.1, 10 32.1; r = 7 6
// 70.8, 10 78.6; r = 8 6 126.7, 10 118.8; 14 spill in the loop at r = 6, 7.
constexpr int f64_run(int R) { return R == 6 || R == 8 ? 10 : 6; }
constexpr int f64_threads(int R) { return ru((flat_cells(R, 2) + f64_run(R) - 1) / f64_run(R), 64); }
template <int R> using Flat64 = FlatGeo<double, R, f64_threads(R), f64_threads(R), f64_run(R), f64_run(R) == 10 ? 2 : 3>;

// A 16-byte chunk of cells.
template <typename S> struct ChunkOf;
template <> struct ChunkOf<float> { typedef float T __attribute__((ext_vector_type(4))); };
template <> struct ChunkOf<double> { typedef double T __attribute__((ext_vector_type(2))); };

// Reads the CH NC values at buf[base + OFF .. + CH NC) (base + OFF a multiple
// of CH) as aligned 128-bit loads into t.
template <int NC, int OFF, typename S>
__device__ __forceinline__ void read_chunks(const S *__restrict__ buf, int base, S (&t)[16 / (int)sizeof(S) * NC])
{
    constexpr int CH = 16 / (int)sizeof(S);
    typedef typename ChunkOf<S>::T V;
    const V *p = (const V *)(buf + base + OFF);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        V q = p[c];
        // keep the whole 16-byte load (otherwise the unused lanes of the
        // first / last chunk let the compiler split it into smaller loads)
        asm("" : "+v"(q));
#pragma unroll
        for (int u = 0; u < CH; ++u) t[CH * c + u] = q[u];
    }
}

// Misalignment m in [0, ch) of a neighbour run at offset d from an aligned start.
constexpr int mis(int d, int ch) { return ((d % ch) + ch) % ch; }

// Reads the RUN values at buf[base + D .. + RUN) (base aligned to 16 bytes) as
// aligned 128-bit loads into v[0 .. RUN).
template <int RUN, int D, typename S>
__device__ __forceinline__ void read_run(const S *__restrict__ buf, int base, S (&v)[RUN])
{
    constexpr int CH = 16 / (int)sizeof(S), M = mis(D, CH);
    constexpr int NC = (RUN + M + CH - 1) / CH;
    S t[CH * NC];
    read_chunks<NC, D - M>(buf, base, t);
#pragma unroll
    for (int k = 0; k < RUN; ++k) v[k] = t[k + M];
}

// The runs at -W and +W (v0, v1) and the cells next to the run's ends (zlo,
// zhi) for the run of g at buf[base .. + RUN).  Where RUN > W they are the W
// cells before the run (previous thread) and after it (next thread) plus
// RUN - W cells of the own run (registers); else the aligned spans of read_run.
template <int RUN, int W, typename S>
__device__ __forceinline__ void read_x_runs(const S *__restrict__ buf, int base, const S (&g)[RUN], S (&v0)[RUN],
                                            S (&v1)[RUN], S &zlo, S &zhi)
{
    constexpr int CH = 16 / (int)sizeof(S);
    if constexpr (RUN > W) {
        constexpr int NC = (W + CH - 1) / CH;
        S tp[CH * NC], tn[CH * NC];
        read_chunks<NC, -CH * NC>(buf, base, tp);
        read_chunks<NC, RUN>(buf, base, tn);
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            v0[k] = k < W ? tp[CH * NC - W + k] : g[k < W ? 0 : k - W];
            v1[k] = k < RUN - W ? g[k < RUN - W ? k + W : 0] : tn[k + W - RUN];
        }
        zlo = tp[CH * NC - 1];
        zhi = tn[0];
    } else {
        zlo = buf[base - 1];
        zhi = buf[base + RUN];
        read_run<RUN, -W>(buf, base, v0);
        read_run<RUN, W>(buf, base, v1);
    }
}

template <typename F> struct FlatSeg {
    using S = typename F::S;
    static constexpr int RUN = F::RUN;
    S xm[RUN], xp[RUN], ym[RUN], yp[RUN];
    S zf[RUN + 1];            // zf[k]: face between run cells k - 1 and k
    S diag[RUN];
};

// Window position of flat cell i = cy PY + cx W + z (any i >= 0): column col =
// cy W + cx, height z; ok: the cell exists (unused cells of a plane's pitch
// have coefficients 0 and hold 0).
template <typename F> struct FlatCell {
    int col, cx, cy, z;
    bool ok;
    __device__ __forceinline__ explicit FlatCell(int i)
    {
        cy = i / F::PY;
        const int rem = i - cy * F::PY;
        cx = rem / F::W;
        z = rem - cx * F::W;
        col = cy * F::W + cx;
        ok = i < F::NCELL && rem < F::W2;
    }
};

// Coefficients of the run that starts at cell s0v (F::NCELL: no cells,
// all 0) of the window of (sx, sy, sz), through the owned-face accessor f.
// (A lane's run touches its own cache lines, so these loads take 25,600 line
// accesses per source at r = 8.  Reading the faces in grid order and changing
// to the run order in LDS takes a third of their time, but its LDS accesses
// delay the other workgroups' sub-steps, under which these loads mostly
// disappear: 239 against 222 ms per 96^3 step at r = 8.)
template <typename F, typename Faces>
__device__ __forceinline__ void flat_load(FlatSeg<F> &c, const Faces &f, int nx, int ny, int nz, int sx, int sy,
                                          int sz, int s0v)
{
    using S = typename F::S;
    constexpr int R = F::R, W = F::W, RUN = F::RUN;
    const int64_t nxy = (int64_t)nx * ny;
#pragma unroll
    for (int k = 0; k < RUN; ++k) {
        const FlatCell<F> p(s0v + k);
        const int X = sx - R + p.cx, Y = sy - R + p.cy, Z = sz - R + p.z;
        const bool in = p.ok && X >= 0 && X < nx && Y >= 0 && Y < ny && Z >= 0 && Z < nz;
        S xm = S(0), xp = S(0), ym = S(0), yp = S(0), zf = S(0);
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
        const FlatCell<F> p(s0v + RUN);
        const int X = sx - R + p.cx, Y = sy - R + p.cy, Z = sz - R + p.z;
        S zf = S(0);
        if (p.ok && p.z > 0 && X >= 0 && X < nx && Y >= 0 && Y < ny && Z > 0 && Z < nz)
            zf = f.z((int64_t)(Z - 1) * nxy + (int64_t)Y * nx + X, Z - 1);
        c.zf[RUN] = zf;
    }
#pragma unroll
    for (int k = 0; k < RUN; ++k) {
        S s = c.xm[k] + c.xp[k];
        s = s + c.ym[k];
        s = s + c.yp[k];
        s = s + c.zf[k];
        s = s + c.zf[k + 1];
        c.diag[k] = S(1) - s;
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
template <typename F, bool SINK>
__device__ __forceinline__ void flat_substeps(typename F::S (&Gs)[F::RUN], const FlatSeg<F> &c, typename F::S *buf0,
                                              typename F::S *buf1, int own, int n_sub, unsigned sink)
{
    using S = typename F::S;
    typedef typename ChunkOf<S>::T V;
    constexpr int CH = F::CH;
    constexpr int W = F::W, PY = F::PY, RUN = F::RUN;
    auto substep = [&](S *buf) {
        // a wave that has passed the barrier issues ahead of the
        // other workgroup's wave on its SIMD until its next write
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int q = 0; q < RUN / CH; ++q) {
            V v;
#pragma unroll
            for (int u = 0; u < CH; ++u) v[u] = Gs[CH * q + u];
            *(V *)(buf + own + CH * q) = v;
        }
        __syncthreads();
        __builtin_amdgcn_s_setprio(1);
        // the neighbour runs are requested two directions ahead
        // of their use (two buffers), so their LDS latency
        // overlaps the FMAs of the previous direction
        S zlo, zhi;
        S v0[RUN], v1[RUN];
        read_x_runs<RUN, W>(buf, own, Gs, v0, v1, zlo, zhi);
        S acc2[RUN];
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            S a2 = c.diag[k] * Gs[k];
            a2 = fmaT<S>(c.zf[k], k > 0 ? Gs[k - 1] : zlo, a2);
            acc2[k] = fmaT<S>(c.zf[k + 1], k < RUN - 1 ? Gs[k + 1] : zhi, a2);
        }
#pragma unroll
        for (int k = 0; k < RUN; ++k) acc2[k] = fmaT<S>(c.xm[k], v0[k], acc2[k]);
        read_run<RUN, -PY>(buf, own, v0);
#pragma unroll
        for (int k = 0; k < RUN; ++k) acc2[k] = fmaT<S>(c.xp[k], v1[k], acc2[k]);
        read_run<RUN, PY>(buf, own, v1);
#pragma unroll
        for (int k = 0; k < RUN; ++k) acc2[k] = fmaT<S>(c.ym[k], v0[k], acc2[k]);
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
            Gs[k] = fmaT<S>(c.yp[k], v1[k], acc2[k]);
            if constexpr (SINK) Gs[k] = (sink >> k) & 1u ? S(0) : Gs[k];
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
// xor butterfly per wave, the window's waves in order.  red: NT / 64 doubles.
// Every thread calls it (two barriers; LDS reads before the call are done
// after it).
template <typename F> __device__ __forceinline__ double flat_window_sum(double ms, double *red, int g)
{
    constexpr int NW = F::SG / 64;
    const int t = threadIdx.x;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ms += __shfl_xor(ms, off, 64);
    __syncthreads();
    if ((t & 63) == 0) red[t >> 6] = ms;
    __syncthreads();
    double s = red[NW * g];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[NW * g + w];
    return s;
}

}  // namespace fdirw
