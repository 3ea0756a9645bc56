"""GPU: the FP32-state window kernels on both sides of the sub-step counts at which
calls with many sources change their layout.

Kernels of a source list: calls with many sources equal calls with few (the
segment layout) bit for bit, the masses within 1e-14 relative.  Bank: the run of
one step equals the fused step within 1e-13 relative.  Coarse build: P from FP32
kernels against P from FP64 ones, 8 n 2^-24 per kernel value, N_J <= B^3 of them
per entry, rounded to FP32."""
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


def _dev(r, n_sub):
    d = synth.random_small(SHAPE, 3, r=r, n_sub=n_sub, seed=400 + r)
    return d, fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)


@pytest.mark.parametrize("r,n_sub,prec", [(4, 9, fd.FP32), (4, 10, fd.FP32), (5, 19, fd.FP32), (5, 20, fd.FP32),
                                          (6, 21, fd.FP16_BANK), (6, 22, fd.FP32), (7, 1, fd.FP32), (7, 2, fd.FP32),
                                          (8, 13, fd.FP32), (8, 14, fd.FP32), (8, 15, fd.BF16_BANK)])
def test_many_sources_equal_few(r, n_sub, prec):
    d, dom = _dev(r, n_sub)
    src = np.random.default_rng(r).permutation(np.arange(d.label.size, dtype=np.int64))
    src = np.concatenate([src, src[:23]])
    G, m = fd.fdirw_kernels(dom, to_dev(src), prec=prec)
    for at in range(0, len(src), 200):
        g, q = fd.fdirw_kernels(dom, to_dev(src[at:at + 200]), prec=prec)
        assert torch.equal(G[at:at + 200], g)
        assert torch.all((m[at:at + 200] - q).abs() <= 1e-14 * q)


@pytest.mark.parametrize("r,n_sub,prec", [(4, 0, "fp32"), (5, 0, "fp16_bank"), (6, 13, "fp32"), (6, 14, "fp16_bank"),
                                          (7, 0, "fp32"), (8, 13, "bf16_bank"), (8, 14, "fp32")])
def test_bank_equals_fused_step(r, n_sub, prec):
    d, dom = _dev(r, n_sub)
    c = to_dev(d.c0)
    _, st = fd.fdirw_run(dom, c, 1, prec=prec, bank_budget_bytes=8 << 30, stats=True)
    assert st["bank_used"] == 1
    want = to_host(fd.fdirw_step(dom, to_dev(d.c0), prec=prec))
    assert np.max(np.abs(to_host(c) - want)) <= 1e-13 * np.abs(want).max()


@pytest.mark.parametrize("sink", [False, True])
@pytest.mark.parametrize("r,n_sub", [(4, 39), (4, 40), (5, 21), (5, 22), (6, 7), (6, 8), (7, 47), (7, 48), (8, 9),
                                     (8, 10)])
def test_coarse_build(r, n_sub, sink):
    B = 3
    _, dom = _dev(r, n_sub)
    res = [0, 1, 0] if sink else None
    got = fd.Coarse(dom, B, fd.FP32, reservoir=res)
    want = fd.Coarse(dom, B, fd.FP64, reservoir=res)
    assert np.max(np.abs(got.matrix() - want.matrix())) <= B ** 3 * 8 * n_sub * 2.0 ** -24 + 2.0 ** -24
