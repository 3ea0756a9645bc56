"""GPU: node windows by rows where memory is short.

The rows of 160^3 cells (half of them impermeable, r = 20, blocks of 5, FP64)
take 1 GB per 64 of the 32,768 nodes and buffer: with a limit above that of all
of them the allocation fails (537 GB), and the build takes whole windows. A limit
below one chunk takes whole windows without asking. Both give the same matrix.

A limit of a few chunks runs the rows in several launches, the last one ragged,
over buffers that hold the previous chunks' rows: the matrix is the same bit for
bit as from one launch, and from whole windows within the rounding of the scale
and the bins (FP64 sums of at most N_J W_b^3 terms in another order)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402
import synth  # noqa: E402


def test_failed_allocation_takes_whole_windows(monkeypatch):
    n = 160
    assert torch.cuda.get_device_properties(0).total_memory < 500e9
    label = np.random.default_rng(5).integers(0, 2, (n, n, n), dtype=np.uint8)
    dom = fd.Domain(label, np.array([1.0, 0.0]), 20, 1, 1.0, 0.1)

    def matrix(limit):
        monkeypatch.setenv("FDIRW_NODEWIN_BYTES", str(limit))
        op = fd.Coarse(dom, 5, "fp64")
        try:
            return op.matrix()
        finally:
            op.close()

    assert np.array_equal(matrix(1 << 50), matrix(1))


@pytest.mark.parametrize("shape,B,r,n_sub,far,prec", [
    ((18, 16, 20), 2, 9, 7, False, "fp64"), ((18, 16, 20), 2, 9, 8, True, "fp32"),
    ((40, 21, 35), 3, 9, 6, True, "fp64"), ((40, 21, 35), 3, 9, 5, False, "fp32"),
    ((27, 22, 25), 5, 10, 1, False, "fp64"), ((27, 22, 25), 5, 10, 0, True, "fp64")])
@pytest.mark.parametrize("chunks", [1, 2])
def test_several_launches_equal_one(monkeypatch, shape, B, r, n_sub, far, prec, chunks):
    d = synth.random_small(shape, 4, r=r, n_sub=n_sub, seed=90 + B + n_sub)
    label = d.label.copy()
    dph = np.array(list(d.d_phase) + [1.0])
    if far:
        label[:, :, -2:] = 4
    dom = fd.Domain(label, dph, r, n_sub, d.h, 0.1)

    def matrix(limit):
        monkeypatch.setenv("FDIRW_NODEWIN_BYTES", str(limit))
        op = fd.Coarse(dom, B, prec, reservoir=[0, 0, 0, 0, 1] if far else None)
        try:
            return op.matrix()
        finally:
            op.close()

    # a chunk of 64 nodes takes 64 values per cell with a row (at most all cells)
    # and buffer, and its units at most a tenth of that
    chunk = 64 * (label.size + 1) * (8 if prec == "fp64" else 4)
    one = matrix(1 << 36)
    assert np.array_equal(matrix(int(1.1 * chunks * chunk)), one)
    whole = matrix(1)
    assert np.max(np.abs(one - whole)) <= (1e-13 if prec == "fp64" else 2.0 ** -23)
