"""GPU: the window kernels in the flat layout (FP32 state, r = 4..8).

Calls with many sources run the flat layout, calls with few the segment layout,
with the same arithmetic per cell: the kernels must be equal bit for bit, the
masses up to the grouping of their FP64 sum (1e-14 relative).  The domain is
smaller than a window in places, its 1,716 cells are no multiple of the windows
per workgroup in the odd calls, and the sub-step counts are even, odd and 0."""
import numpy as np
import pytest

import synth
from helpers import to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402

SHAPE = (13, 12, 11)


def _dev(r, n_sub, seed):
    d = synth.random_small(SHAPE, 3, r=r, n_sub=n_sub, seed=seed)
    return d, fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)


@pytest.mark.parametrize("r,n_sub,prec", [(4, 11, fd.FP32), (5, 8, fd.FP32), (6, 7, fd.FP32), (7, 6, fd.FP32),
                                          (8, 9, fd.FP32), (8, 0, fd.FP32), (4, 6, fd.FP16_BANK),
                                          (8, 5, fd.FP16_BANK), (6, 5, fd.BF16_BANK)])
def test_many_sources_equal_few(r, n_sub, prec):
    d, dom = _dev(r, n_sub, 700 + r)
    n = d.label.size
    src = np.random.default_rng(r).permutation(np.arange(n, dtype=np.int64))
    src = np.concatenate([src, src[:23]])                    # 1,739 sources: a ragged last workgroup
    G, m = fd.fdirw_kernels(dom, to_dev(src), prec=prec)
    for at in range(0, len(src), 200):
        g, q = fd.fdirw_kernels(dom, to_dev(src[at:at + 200]), prec=prec)
        assert torch.equal(G[at:at + 200], g)
        assert torch.all((m[at:at + 200] - q).abs() <= 1e-14 * q)


@pytest.mark.parametrize("r,n_sub,prec", [(4, 7, "fp32"), (7, 4, "fp32"), (8, 6, "fp16_bank"), (5, 5, "bf16_bank")])
def test_bank_equals_fused_step(r, n_sub, prec):
    d, dom = _dev(r, n_sub, 720 + r)
    c = to_dev(d.c0)
    _, st = fd.fdirw_run(dom, c, 1, prec=prec, bank_budget_bytes=8 << 30, stats=True)
    assert st["bank_used"] == 1
    want = to_host(fd.fdirw_step(dom, to_dev(d.c0), prec=prec))
    assert np.max(np.abs(to_host(c) - want)) <= 1e-13 * np.abs(want).max()


@pytest.mark.parametrize("sink", [False, True])
@pytest.mark.parametrize("r,B", [(4, 1), (5, 2), (6, 3), (7, 5), (8, 2)])
def test_coarse_build(r, B, sink):
    # P from FP32 kernels against P from FP64 kernels (pinned by the oracle):
    # each kernel value is within 8 n 2^-24 of the exact one, an entry of P
    # sums N_J <= B^3 of them per destination cell and is rounded to FP32
    n_sub = 9
    d, dom = _dev(r, n_sub, 740 + r)
    res = [0, 1, 0] if sink else None
    got = fd.Coarse(dom, B, fd.FP32, reservoir=res)
    want = fd.Coarse(dom, B, fd.FP64, reservoir=res)
    assert np.max(np.abs(got.matrix() - want.matrix())) <= B ** 3 * 8 * n_sub * 2.0 ** -24 + 2.0 ** -24
