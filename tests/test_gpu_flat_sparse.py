"""GPU: the flat-layout fused step on fields with few nonzero sources.

A line's ring is empty once it has moved a window's height past its last nonzero
source, and the sources up to the next one are skipped; which sources are nonzero
is read 64 at a time.  Sources at both ends of a line, gaps of W - 1, W and W + 1,
at the 64-source steps, on one of several lines of a workgroup, in cut lines and
an empty field.  Bars of the fused step: FP64 1e-13, FP32 1e-5 against the oracle;
1e-13 relative against the deterministic form, which skips nothing."""
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

NZ, NY, NX = 139, 3, 2


def _field(kind, r, seed):
    c = np.zeros((NZ, NY, NX))
    w = 2 * r + 1
    rng = np.random.default_rng(seed)
    if kind == "gaps":
        z = 0
        for gap in (w - 1, w, w + 1, 2 * w):
            c[z, 0, 0] = rng.uniform(0.5, 1.5)
            z += gap
        c[NZ - 1, 2, 1] = 1.0
    elif kind == "steps":
        for z in (0, 63, 64, 127, 128):
            c[z, z % NY, z % NX] = rng.uniform(0.5, 1.5)
    elif kind == "first":
        c[0, 1, 1] = 1.0
    elif kind == "run":
        c[60:60 + r, 1, :] = rng.uniform(0.5, 1.5, (r, NX))
    return c


@pytest.mark.parametrize("prec", [fd.FP64, fd.FP32])
@pytest.mark.parametrize("r", [3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("kind,tune", [("gaps", 0), ("steps", 1), ("first", 0), ("run", 3), ("none", 0)])
def test_few_sources(prec, r, kind, tune):
    d = synth.random_small((NZ, NY, NX), 3, r=r, n_sub=49, seed=70 + r)
    c0 = _field(kind, r, r)
    print(f"[flat sparse] prec={prec} r={r} {kind}", flush=True)
    dom = fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)
    out, st = fd.fdirw_step(dom, to_dev(c0), prec=prec, tune=tune, stats=True)
    ref, used, _ = oracle.Problem.from_domain(d).step(c0)
    got = to_host(out)
    assert st["n_sources"] == used == np.count_nonzero(c0)
    assert np.max(np.abs(got - ref)) <= (1e-13 if prec == fd.FP64 else 1e-5)
    det = to_host(fd.fdirw_step(dom, to_dev(c0), prec=prec, deterministic=True))
    assert np.max(np.abs(got - det)) <= 1e-13 * max(np.abs(det).max(), 1e-300)
    lab = to_host(fd.fdirw_step_noalloc(dom, to_dev(c0), torch.empty_like(to_dev(c0)), prec=prec))
    assert np.max(np.abs(lab - got)) <= 1e-13 * max(np.abs(got).max(), 1e-300)
