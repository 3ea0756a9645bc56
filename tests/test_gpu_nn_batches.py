"""GPU: the surrogate's gradient over batches that fill the weight-gradient
workgroups unevenly.

The gradient of a batch is the mean of its windows' gradients.  With a power of
two of windows the loss scale changes no BF16 rounding, so only the order of
the FP32 sums differs: at most about 1,000 additions per entry, 2^-24 sqrt(1000)
of the summed magnitudes, with room for a 50-fold cancellation 1e-4 of the
gradient's norm.  1 window is 6 slabs (most workgroups idle), 32 are 192 (one
each), 64 are 384 (one or two each)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402


@pytest.mark.parametrize("count", [1, 32, 64, 256])
def test_gradient_is_the_mean_of_the_windows(count):
    d = synth.random_small((20, 19, 21), 3, r=8, n_sub=12, seed=51)
    dom = fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)
    nn = fd.Surrogate(d.n_sub, seed=3)
    src = np.random.default_rng(count).integers(0, d.label.size, min(count, 64)).astype(np.int64)
    src = np.resize(src, count)
    (kl, l1), g = nn.backward(dom, torch.from_numpy(src).cuda(), grad=True)
    one = [nn.backward(dom, torch.from_numpy(src[i:i + 1]).cuda(), grad=True) for i in range(min(count, 64))]
    want = torch.stack([o[1].double() for o in one]).mean(dim=0)
    assert torch.linalg.vector_norm(g.double() - want) <= 1e-4 * torch.linalg.vector_norm(want)
    assert kl == pytest.approx(np.mean([o[0][0] for o in one]), rel=1e-9)
    assert l1 == pytest.approx(np.mean([o[0][1] for o in one]), rel=1e-9)
