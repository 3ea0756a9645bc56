"""GPU: the forms of the ensemble coarse product agree bitwise.  Many members on
a large grid take several column tiles of 16 members per wave (K <= 2: the
plane-walking form from 8 column tiles and 40960 tiles x column tiles on; K = 3, 4:
from 7 and 6 column tiles and 8192), a few of them one: the same fragments summed
in the same order.  Ragged tiles, z-chunks and member counts, K = 0 .. 4, and
products just below the lines."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402


# 475 tiles at blocks of 2 (88 column tiles are above 40960, 86 below), 3330 at 1
@pytest.mark.parametrize("r,B,n_ens", [(0, 2, 1400), (2, 2, 1393), (3, 2, 1400), (3, 2, 1376),
                                       (3, 1, 112), (3, 1, 96), (4, 1, 90), (4, 1, 80)])
def test_members_of_a_large_ensemble(r, B, n_ens):
    d = synth.random_small((39, 33, 37), 2, r=r, n_sub=5, seed=90 + r, dt=0.125)
    cg = fd.Coarse(fd.Domain(d.label, np.asarray(d.d_phase), r, 5, d.h, d.dt), B, fd.FP16_BANK)
    K = {(0, 2): 0, (2, 2): 1, (3, 2): 2, (3, 1): 3, (4, 1): 4}[r, B]
    assert cg.K == K and cg.n_nodes == (20 * 17 * 19 if B == 2 else 39 * 33 * 37)
    C = torch.rand((n_ens, cg.n_nodes), dtype=torch.float64, device="cuda",
                   generator=torch.Generator("cuda").manual_seed(90 + r))
    C *= 10.0 ** (3.0 * (torch.arange(n_ens, device="cuda", dtype=torch.float64)[:, None] % 7) - 12.0)
    print(f"[ensemble] K={K} n_ens={n_ens}", flush=True)
    many = cg.apply_ensemble(C)
    for a, b in ((0, 16), (n_ens // 2, n_ens // 2 + 37), (n_ens - 19, n_ens)):
        few = cg.apply_ensemble(C[a:b].clone())
        assert torch.equal(few, many[a:b])
    cg.close()
