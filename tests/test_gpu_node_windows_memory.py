"""GPU: node windows by rows where memory is short.

The rows of 160^3 cells (half of them impermeable, r = 20, blocks of 5, FP64)
take 1 GB per 64 of the 32,768 nodes and buffer: with a limit above that of all
of them the allocation fails (537 GB), and the build takes whole windows. A limit
below one chunk takes whole windows without asking. Both give the same matrix."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402


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
