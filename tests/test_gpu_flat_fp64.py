"""GPU: the flat-layout fused step in FP64 (r = 3..8, from 2 to 28 sub-steps on).

Against the FP64 oracle (1e-13, the bar of the FP64 step), the deterministic
form (the same kernels, sums in another order: 1e-13 relative; repeats bitwise),
the step with coefficients by phase pair, and, for a one-hot field, the kernel
of fdirw_kernels (segment layout, the same arithmetic per cell): bit for bit.
Domains smaller than the window, ragged lines, zero sources between nonzero
ones, lines cut into segments, odd and even sub-step counts, and 15 sub-steps
at r = 7 (the segment layout)."""
import numpy as np
import pytest

import oracle
import synth
from helpers import place, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402


def _dev(d):
    return fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)


@pytest.mark.parametrize("shape,r,n_sub,tune", [
    ((9, 10, 11), 3, 28, 0), ((4, 3, 21), 3, 29, 3), ((12, 7, 13), 4, 31, 0), ((6, 15, 8), 5, 30, 2),
    ((10, 9, 11), 6, 29, 0), ((16, 14, 15), 7, 28, 0), ((19, 18, 20), 8, 29, 0), ((5, 6, 7), 8, 30, 5),
    ((23, 1, 4), 8, 31, 3), ((11, 12, 5), 7, 15, 0), ((7, 9, 17), 4, 2, 0), ((13, 5, 8), 6, 9, 0)])
def test_step(shape, r, n_sub, tune):
    d = synth.random_small(shape, 3, r=r, n_sub=n_sub, seed=940 + r + n_sub)
    c0 = d.c0.copy()
    c0.reshape(-1)[::3] = 0.0
    print(f"[flat fp64] shape={shape} r={r} n_sub={n_sub}", flush=True)
    dom = _dev(d)
    out, st = fd.fdirw_step(dom, to_dev(c0), prec=fd.FP64, tune=tune, stats=True)
    A = to_host(out)
    ref, used, (kmin, kmax) = oracle.Problem.from_domain(d).step(c0)
    assert np.max(np.abs(A - ref)) <= 1e-13
    assert st["n_sources"] == used
    assert st["kmass_min"] == pytest.approx(kmin, abs=1e-13) and st["kmass_max"] == pytest.approx(kmax, abs=1e-13)
    det = to_host(fd.fdirw_step(dom, to_dev(c0), prec=fd.FP64, deterministic=True))
    assert np.max(np.abs(A - det)) <= 1e-13 * np.abs(det).max()
    assert np.array_equal(det, to_host(fd.fdirw_step(dom, to_dev(c0), prec=fd.FP64, deterministic=True)))
    lab = to_host(fd.fdirw_step_noalloc(dom, to_dev(c0), torch.empty(shape, dtype=torch.float64, device="cuda"),
                                        prec=fd.FP64))
    assert np.max(np.abs(lab - ref)) <= 1e-12


@pytest.mark.parametrize("r", [3, 4, 5, 6, 7, 8])
def test_one_hot_is_the_placed_kernel(r):
    d = synth.random_small((14, 13, 15), 3, r=r, n_sub=28 + r, seed=960 + r)
    dom = _dev(d)
    nz, ny, nx = d.shape
    for (z, y, x) in [(0, 0, 0), (7, 6, 7), (13, 12, 14), (2, 12, 1)]:
        s = (z * ny + y) * nx + x
        e = np.zeros(d.shape)
        e[z, y, x] = 1.0
        out = to_host(fd.fdirw_step(dom, to_dev(e), prec=fd.FP64))
        G, _ = fd.fdirw_kernels(dom, to_dev(np.array([s], dtype=np.int64)), prec=fd.FP64)
        assert np.array_equal(out, place(d.shape, s, to_host(G)[0]))
