"""GPU: the bank apply of a small grid, whose source rows are cut into parts,
against the apply in one part (a budget of exactly the bank, its masses and the
padded field leaves no room for the parts).  Sums of at most W^3 non-negative
terms in another grouping: W^3 2^-53 relative, per cell, per step.  Part counts
from 2 to W, ragged last parts, tiles ragged in x and z."""
import pytest

import synth
from helpers import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402


@pytest.mark.parametrize("shape,r,prec,esz", [
    ((5, 6, 7), 8, fd.FP16_BANK, 2), ((33, 20, 70), 8, fd.BF16_BANK, 2), ((35, 60, 66), 8, fd.FP16_BANK, 2),
    ((17, 31, 40), 5, fd.FP32, 4), ((9, 64, 65), 3, fd.FP64, 8), ((12, 10, 9), 1, fd.FP32, 4),
    ((3, 4, 5), 0, fd.FP32, 4), ((20, 129, 64), 2, fd.FP64, 8)])
def test_parts_equal_whole(shape, r, prec, esz):
    nz, ny, nx = shape
    d = synth.random_small(shape, 3, r=r, n_sub=3, seed=980 + r)
    dom = fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)
    zb = 16 // esz
    bank = (2 * r + 1) ** 3 * nx * ny * (-(-nz // zb) * zb) * esz
    own = bank + 8 * nx * ny * nz + 8 * (nx + 2 * r) * (ny + 2 * r) * (nz + 2 * r)
    n_steps = 2
    a, b = to_dev(d.c0), to_dev(d.c0)
    _, sa = fd.fdirw_run(dom, a, n_steps, prec=prec, bank_budget_bytes=own, stats=True)
    _, sb = fd.fdirw_run(dom, b, n_steps, prec=prec, bank_budget_bytes=8 << 30, stats=True)
    assert sa["bank_used"] == 1 and sb["bank_used"] == 1
    assert torch.all((a - b).abs() <= n_steps * (2 * r + 1) ** 3 * 2.0 ** -53 * a.abs())
