"""GPU: the far-field balance of Eq. 7 beside the next step's mapping.

Several steps in one call (balances beside the following mappings, the last one
in a launch of its own) against one step per call (each in its own launch): the
same sums in the same order, so field, c_ff and history agree bit for bit.  The
mapping by rows of blocks and the sparse one (a small particle in a large
box), blocks of 1 and 3, and several solid sub-steps (balance over the
active list)."""
import numpy as np
import pytest

import synth
from helpers import to_dev
from oracle import multiphysics as mp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402

ROLE = np.array([mp.ROLE_LIQUID, mp.ROLE_SOLID, mp.ROLE_FAR])


@pytest.mark.parametrize("n,r_p,B,n_sub_solid", [(16, 5.5, 1, 1), (16, 5.5, 3, 1), (44, 4.0, 3, 1), (44, 4.0, 2, 1),
                                                 (16, 5.5, 2, 3)])
def test_steps_of_one_call_equal_single_steps(n, r_p, B, n_sub_solid):
    label = synth.particle(n, r_p, shell=2.0, porosity=0.3, corr_len=1.5, seed=97)
    u = synth.uniform(98, label.size).reshape(label.shape)
    c0 = np.where(label == synth.PHASE_SOLID, 1e-4 * u, 0.2 + 0.05 * u)
    far = label == synth.PHASE_FAR_LIQUID
    c0[far] = 0.2
    m_total = c0[~far].sum() + 500.0 * 0.2
    s = fd.Multiphysics(fd.Domain(label, np.array([1.0, 0.02, 1.0]), 3, 6, 1.0, 0.5), ROLE, 0.3, 0.01, 1.0, 500.0,
                        a_over_rt=np.array([0.15, 0.5, 0.15]), n_sub_solid=n_sub_solid, block=B, prec=fd.FP64)
    a, b = to_dev(c0), to_dev(c0)
    cff, hist = s.step(a, 0.2, m_total, 5)
    one, rows = 0.2, []
    for _ in range(5):
        one, h = s.step(b, one, m_total, 1)
        rows.append(h[0])
    assert torch.equal(a, b)
    assert cff == one and np.array_equal(hist, np.array(rows))
    s.close()
