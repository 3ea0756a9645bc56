"""GPU: node windows (coarse operator with r > 8) by rows of cells and by whole
windows, against the oracle's node windows.

Sizes where the rows can go wrong: several chunks of 64 nodes with a ragged last
one, windows clipped by the domain and walls inside it (K blocks shorter than
the grid), blocks with more rows than one unit, ungrouped permeable cells and
impermeable ones, far-field cells, odd, even and 0 sub-steps; and a large block
with few nodes, which takes whole windows.  FP64: 1e-13 as for the other coarse
matrices; FP32: every cell value within 8 n 2^-24 of the exact one (unit mass in
N_J <= B^3 cells), summed over a group and divided by its count."""
import numpy as np
import pytest

import oracle
import synth
from oracle import coarse

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402


@pytest.mark.parametrize("shape,B,r,n_sub,far,some,prec", [
    ((18, 16, 20), 2, 9, 7, False, False, "fp64"), ((18, 16, 20), 2, 9, 8, True, True, "fp64"),
    ((30, 11, 10), 2, 9, 5, False, True, "fp32"), ((9, 31, 12), 3, 9, 6, True, False, "fp32"),
    ((27, 22, 25), 5, 10, 6, False, True, "fp64"), ((12, 13, 40), 4, 12, 0, False, False, "fp64"),
    ((40, 21, 20), 10, 10, 4, False, False, "fp64"), ((40, 21, 20), 10, 10, 5, True, False, "fp32")])
def test_node_windows(shape, B, r, n_sub, far, some, prec):
    d = synth.random_small(shape, 4, r=r, n_sub=n_sub, seed=80 + B + n_sub)
    label = d.label.copy()
    dph = np.array(list(d.d_phase) + [1.0])
    grouped = [1, 0, 1, 0, 0] if some else None
    res = None
    if far:
        label[:, :, -2:] = 4
        res = [0, 0, 0, 0, 1]
    p = oracle.Problem(label, dph, r, n_sub, d.h, 0.1)
    P = coarse.coarse_matrix(p, B, grouped, res)
    cg = fd.Coarse(fd.Domain(label, dph, r, n_sub, d.h, 0.1), B, prec, grouped=grouped, reservoir=res)
    kw = 2 * cg.K + 1
    ncz, ncy, ncx = cg.coarse_shape
    got = cg.matrix()
    seen = np.zeros_like(P)
    I = np.arange(P.shape[0])
    iz, iy, ix = I // (ncy * ncx), I // ncx % ncy, I % ncx
    for o in range(kw ** 3):
        jz, jy, jx = iz - (o // kw ** 2 - cg.K), iy - (o // kw % kw - cg.K), ix - (o % kw - cg.K)
        ok = (jz >= 0) & (jz < ncz) & (jy >= 0) & (jy < ncy) & (jx >= 0) & (jx < ncx)
        seen[I[ok], ((jz * ncy + jy) * ncx + jx)[ok]] = got[o, I[ok]]
    tol = 1e-13 if prec == "fp64" else B ** 3 * 8 * max(1, n_sub) * 2.0 ** -24
    assert np.max(np.abs(seen - P)) <= tol
