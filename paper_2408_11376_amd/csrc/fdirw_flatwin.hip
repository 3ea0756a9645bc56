// fdirw_flatwin.hip -- window kernels in the flat layout (gfx950, FP32 state, r
// = 4..8): the kernels with a steady flow.
#include "fdirw_flat.h"
#include "fdirw_launch.h"

namespace fdirw {

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
            const FlatCell<R> p(s0v + k);
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
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                const FlatCell<R> p(s0v + k);
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

}  // namespace fdirw
