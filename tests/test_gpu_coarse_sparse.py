"""GPU: the coarse build's FP32 kernels where few cells are grouped.

Grouped cells at random and in a clump, on both sides of the shares at which r =
4 and 5 change between the layouts, down to one cell.  P from FP32 kernels against
P from FP64 kernels (pinned by the oracle): each kernel value is within 8 n 2^-24
of the exact one, an entry of P sums N_J <= B^3 of them per destination cell and
is rounded to FP32; the renormalisation over a share s of the cells scales the
error by at most 1 / m, m >= G(source) the kernel's mass on them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402

SHAPE, B, N_SUB = (14, 12, 13), 3, 6


def _labels(kind, share):
    n = int(np.prod(SHAPE))
    label = np.ones(n, np.uint8)
    if kind == "clump":
        label[n // 3:n // 3 + max(1, int(share * n))] = 0
    else:
        label[np.random.default_rng(7).permutation(n)[:max(1, int(share * n))]] = 0
    return label.reshape(SHAPE)


@pytest.mark.parametrize("r", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("kind,share", [("random", 0.0), ("random", 0.3), ("random", 0.36), ("random", 0.64),
                                        ("random", 0.7), ("clump", 0.1), ("clump", 0.6)])
def test_build_of_few_grouped_cells(r, kind, share):
    dom = fd.Domain(_labels(kind, share), np.array([1.0, 0.3]), r, N_SUB, 1.0, 0.1)
    got = fd.Coarse(dom, B, fd.FP32, grouped=[1, 0])
    want = fd.Coarse(dom, B, fd.FP64, grouped=[1, 0])
    # 6 dt D / h^2 = 0.6: a step keeps at least 0.4 of a cell's value
    m = 0.4 ** N_SUB
    assert np.max(np.abs(got.matrix() - want.matrix())) <= (B ** 3 * 8 * N_SUB * 2.0 ** -24) / m + 2.0 ** -24
