"""GPU: a training run repeats bit for bit, also from one version of the library to
the next: checksums of the gradient and the exact losses of every Adam step,
recorded from the weight gradient that adds the slabs of 128 windows in 512
partials (slab s in partial s mod 512), the partials in order, the groups of 128
in order, and from loss sums in the order of four waves.

The order of the FP32 sums is part of the result: another one gives gradients
equal to rounding at the first step, and other training runs after a few (BF16
weights, the sign in the L1 term).  Nothing is allowed to differ, so the values
are exact.  Batches of one window, of a part of a group, of whole and ragged
groups and of several micro-batches, computed and given targets."""
import zlib

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2408_11376_amd as fd  # noqa: E402

# windows, sub-steps, targets given, seed, (CRC-32 of the gradient, KL, L1) per step
RUNS = [
    (300, 12, False, 0, [
        (0xaa2f3a7e, "0x1.ebb46af014ff7p-1", "0x1.c044faacd47d7p-1"),
        (0x2bd40d0b, "0x1.dce2385c10046p-1", "0x1.ba11ad169c935p-1"),
        (0x3277fa38, "0x1.c7812bad51154p-1", "0x1.b0d472c09efd6p-1"),
        (0x5768b2ca, "0x1.a885e72209309p-1", "0x1.a2ec0945ff3a0p-1"),
        (0x09689102, "0x1.81596416da3bfp-1", "0x1.9033ab049d642p-1"),
        (0xf738cec6, "0x1.55823472f7040p-1", "0x1.79a0660e064e1p-1"),
        (0xc3f5d517, "0x1.288dcbdf05979p-1", "0x1.5ff270326fda1p-1"),
        (0x9361262a, "0x1.f6cebc95b236fp-2", "0x1.42aa7db08d743p-1"),
        (0x9c8d6714, "0x1.a4541a73bc0dcp-2", "0x1.22d9160db3dc9p-1"),
        (0xfd0888b0, "0x1.676627874b6c5p-2", "0x1.04b2c855cd081p-1")]),
    (256, 40, False, 1, [
        (0x0d38a0c4, "0x1.13ac9d964c115p-2", "0x1.ea3125a3cc31dp-2"),
        (0xdd9907bf, "0x1.0fd07b6e24391p-2", "0x1.e66294c55aa64p-2"),
        (0x0acec55a, "0x1.0a6d058a740acp-2", "0x1.e137a03830209p-2"),
        (0xd56bb83d, "0x1.00f64a1c0cef1p-2", "0x1.d83adc6da40ccp-2"),
        (0xdaca94f6, "0x1.e576899526415p-3", "0x1.ca63f2d727561p-2"),
        (0x6fe31cfb, "0x1.c7024a4879833p-3", "0x1.baac197cfd266p-2"),
        (0xa269b39c, "0x1.b6eb55173a833p-3", "0x1.b1098df0c9c3ep-2"),
        (0x733661f2, "0x1.9c2360310c99fp-3", "0x1.a0c9904f43c02p-2"),
        (0xa7440a6f, "0x1.815e87c2059efp-3", "0x1.8f797839fd88ap-2"),
        (0xa492e5f0, "0x1.7405025a7deb0p-3", "0x1.8500a6e06354cp-2")]),
    (150, 12, True, 2, [
        (0x01880856, "0x1.d6df591e65b02p-4", "0x1.fdd05d67b07bfp-1"),
        (0x3bb743ed, "0x1.140ff0a0b0169p-3", "0x1.0030c018d0f2dp+0"),
        (0xd9627c03, "0x1.4d5ceb45dbdaep-3", "0x1.01cde55e3f6acp+0")]),
    (1, 12, False, 3, [
        (0x2bc48da2, "0x1.902985e1c7b5fp-2", "0x1.7434b68f9ed33p-1"),
        (0x78036ac2, "0x1.6de8a43f54be0p-2", "0x1.61234e59a3f14p-1"),
        (0x3e8bf319, "0x1.42880dc0d12e4p-2", "0x1.47f1e8b688d64p-1")]),
    (90, 12, False, 4, [
        (0x24c283f1, "0x1.f017e0551ca95p+0", "0x1.2ca353013cd2fp+0"),
        (0x44f0a041, "0x1.e73d916fe7d84p+0", "0x1.2b7234dd01b82p+0"),
        (0x549ee594, "0x1.dadbff9215949p+0", "0x1.29ab6b012ecc1p+0")]),
    (513, 20, False, 5, [
        (0xe43c7cdf, "0x1.e8e9bdfdcf37ap+0", "0x1.1f73bc47d2320p+0"),
        (0x583caec3, "0x1.e626dc33f0a72p+0", "0x1.1efde70ccecdbp+0"),
        (0xf98e6b44, "0x1.e1b8e7b2b7dfbp+0", "0x1.1e2e4913b2bdap+0")]),
    (293, 12, True, 6, [
        (0xf2cb8ca1, "0x1.a87a88d1b3d16p-4", "0x1.fd690a7ad9462p-1"),
        (0x36c35a94, "0x1.f5fccf2874376p-4", "0x1.ffd6fc11c3060p-1"),
        (0x09fb5924, "0x1.32841494fa74bp-3", "0x1.0178ac7d56983p+0")]),
    (512, 9, True, 7, [
        (0x08b1cd79, "-0x1.10f9162756f2bp-5", "0x1.f33ad0b72b1e7p-1"),
        (0x43230dac, "-0x1.23cbf3426a4b4p-6", "0x1.f61425ad19093p-1")])
]


@pytest.mark.parametrize("count,n_sub,given,seed,want", RUNS, ids=[str(r[0]) for r in RUNS])
def test_training_run_repeats(count, n_sub, given, seed, want):
    d = synth.random_small((20, 19, 21), 3, r=8, n_sub=n_sub, seed=51 + seed)
    dom = fd.Domain(d.label, d.d_phase, d.r, d.n_sub, d.h, d.dt)
    nn = fd.Surrogate(d.n_sub, seed=3)
    src = torch.from_numpy(np.random.default_rng(60 + seed).integers(0, d.label.size, count)).cuda()
    target = None
    if given:
        q = np.random.default_rng(70 + seed).uniform(0.1, 1.0, (count, 17, 17, 17)).astype(np.float32)
        target = torch.from_numpy(q).cuda()
    got = []
    for _ in want:
        (kl, l1), g = nn.backward(dom, src, target, grad=True)
        got.append((zlib.crc32(g.cpu().numpy().tobytes()), float(kl).hex(), float(l1).hex()))
        nn.adam(1e-3)
    assert got == want
