"""GPU: mapping and remapping of the coarse step on grids of 5 2^20 cells and more
(the remapping by roles), and below (by node indices), with block edges of both
load rounds of the mapping (B^2 rows in rounds of 5 or 8).

With no sub-steps P is the identity: every grouped cell takes the mean of its
block's grouped cells, the others keep their value and far-field cells take the
boundary concentration.  The mean of at most B^3 values in [0, 1): B^3 2^-53 of
their sum's bound B^3, i.e. B^3 2^-53 after the division (times 2 for it)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402


@pytest.mark.parametrize("shape,B,far", [((181, 203, 229), 7, False), ((1, 40, 209716), 3, False),
                                         ((230, 1021, 41), 4, True), ((23, 31, 41), 5, False),
                                         ((220, 1000, 39), 2, False)])
def test_means_of_the_blocks(shape, B, far):
    rng = np.random.default_rng(B)
    label = rng.integers(0, 3 if far else 2, shape).astype(np.uint8)
    dom = fd.Domain(torch.from_numpy(label).cuda(), np.array([1.0, 0.5, 1.0])[:3 if far else 2], 1, 0)
    res = [0, 0, 1] if far else None
    cg = fd.Coarse(dom, B, fd.FP64, grouped=[1, 0, 0] if far else [1, 0], reservoir=res)
    c = rng.random(shape)
    dev = torch.from_numpy(c).cuda()
    if far:
        out, cff = cg.step_far_field(dev, 0.25, float(c.size), 1e9)
    else:
        out = cg.step(dev)
    lab = torch.from_numpy(label).cuda()
    i = [torch.arange(n, device="cuda") // B for n in shape]
    nc = [-(-n // B) for n in shape]
    block = (i[0][:, None, None] * nc[1] + i[1][None, :, None]) * nc[2] + i[2][None, None, :]
    g = lab == 0
    s = torch.zeros(nc[0] * nc[1] * nc[2], dtype=torch.float64, device="cuda").index_add_(0, block[g], dev[g])
    k = torch.zeros_like(s).index_add_(0, block[g], torch.ones_like(dev[g]))
    want = torch.where(g, (s / k.clamp(min=1.0))[block], dev)
    if far:
        want = torch.where(lab == 2, torch.full_like(want, cff), want)
    assert (out - want).abs().max().item() <= 2 * B ** 3 * 2.0 ** -53
    assert torch.equal(out[lab == 1], dev[lab == 1])
    cg.close()
