"""GPU: the fused step on both sides of the sub-step counts at which it changes its
layout (and, FP32, r = 6, its register budget), and with none or few sub-steps.

Against the oracle (FP64 1e-13, FP32 1e-5), the deterministic form and the step
with coefficients by phase pair (1e-13 relative)."""
import numpy as np
import pytest

import oracle
import synth
from helpers import to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402

LINES = {fd.FP64: {3: 24, 4: 2, 5: 28, 6: 8, 7: 28, 8: 24}, fd.FP32: {4: 12, 5: 15, 6: 5, 7: 48, 8: 26}}
CASES = [(p, r, n) for p, rs in LINES.items() for r, at in rs.items() for n in sorted({0, 1, at - 1, at})]
CASES += [(fd.FP32, 6, 95), (fd.FP32, 6, 96)]


@pytest.mark.parametrize("prec,r,n_sub", CASES)
def test_step(prec, r, n_sub):
    d = synth.random_small((11, 9, 10), 3, r=r, n_sub=n_sub, seed=300 + r)
    c0 = d.c0.copy()
    c0.reshape(-1)[::4] = 0.0
    print(f"[flat substeps] prec={prec} r={r} n_sub={n_sub}", flush=True)
    dom = fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)
    got = to_host(fd.fdirw_step(dom, to_dev(c0), prec=prec))
    ref, _, _ = oracle.Problem.from_domain(d).step(c0)
    assert np.max(np.abs(got - ref)) <= (1e-13 if prec == fd.FP64 else 1e-5)
    det = to_host(fd.fdirw_step(dom, to_dev(c0), prec=prec, deterministic=True))
    assert np.max(np.abs(got - det)) <= 1e-13 * np.abs(det).max()
    lab = to_host(fd.fdirw_step_noalloc(dom, to_dev(c0), torch.empty_like(to_dev(c0)), prec=prec))
    assert np.max(np.abs(lab - got)) <= 1e-13 * np.abs(got).max()


@pytest.mark.parametrize("r,n_sub", [(6, 95), (6, 96), (7, 96), (8, 95), (8, 96)])
def test_deterministic_step_of_many_lines(r, n_sub):
    # 128 x 128 lines, where the deterministic form changes its register budget;
    # few planes and sources
    d = synth.random_small((3, 128, 128), 3, r=r, n_sub=n_sub, seed=340 + r)
    c0 = d.c0.copy()
    c0[:, 24:, :] = 0.0
    c0[:, :, 20:] = 0.0
    dom = fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)
    det = to_host(fd.fdirw_step(dom, to_dev(c0), prec=fd.FP32, deterministic=True))
    ref, _, _ = oracle.Problem.from_domain(d).step(c0)
    assert np.max(np.abs(det - ref)) <= 1e-5
    assert np.array_equal(det, to_host(fd.fdirw_step(dom, to_dev(c0), prec=fd.FP32, deterministic=True)))
    got = to_host(fd.fdirw_step(dom, to_dev(c0), prec=fd.FP32))
    assert np.max(np.abs(got - det)) <= 1e-13 * np.abs(det).max()
