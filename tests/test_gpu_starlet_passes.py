"""The starlet passes (several levels per launch) where they can go wrong: one level and the
most, grids under, at and above a tile, sides that no power of two divides, a filter wider than
the image's half, the change to FP32 tiles above 256 and at eight planes, three groups; and
PSF mode, whose launches carry the passes, with one group and with two.

Bars as in the parity suite: 2e-6 of the largest value for a transform, 1e-6 and 1e-4 (loss,
gradient per block) for PSF mode.
"""
import numpy as np
import pytest

from oracle import oracle as ora
from oracle import parity
from paper_2402_08725_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,J", [(2, 1), (3, 2), (9, 4), (15, 3), (16, 4), (17, 2), (33, 6), (47, 5), (65, 7),
                                 (129, 8), (250, 7), (256, 7), (257, 6), (259, 9), (512, 8), (520, 10)])
def test_transform_and_transpose(N, J):
    from paper_2402_08725_amd import starred as st
    print(f"N {N} J {J}", flush=True)
    rng = np.random.default_rng(N * 16 + J)
    plan = st.Plan(st.DECONV, [N], [3], 1, N, 0, J, 3.0)
    img = synth.f32(rng.standard_normal(N * N) * 10)
    got = plan.starlet_fwd(img).cpu().numpy().reshape(J, -1)
    ref = ora.starlet_fwd(N, J, img).reshape(J, -1)
    assert np.abs(got - ref).max() <= 2e-6 * np.abs(ref).max()
    z = synth.f32(rng.standard_normal(J * N * N))
    gota = plan.starlet_adj(z).cpu().numpy()
    refa = ora.starlet_adj(N, J, z)
    assert np.abs(gota - refa).max() <= 2e-6 * np.abs(refa).max()


@pytest.mark.parametrize("n,s,J", [(9, 1, 2), (23, 1, 4), (17, 2, 5), (33, 2, 6), (43, 3, 7), (65, 2, 8)])
def test_psf_mode(n, s, J):
    from paper_2402_08725_amd import starred as st
    print(f"n {n} s {s} J {J}", flush=True)
    prob = synth.make_psf(S=3, n=n, s=s, J=J)
    rng = np.random.default_rng(n)
    d, w = synth.add_noise(ora.psf_model(prob, prob.params_true), rng)
    plan = st.Plan.for_psf(prob)
    plan.set_frames(d, w, None, prob.W)
    p = synth.psf_eval_point(prob, "near", rng)
    loss, grad = plan.loss_grad(p)
    alone, _ = plan.loss_grad(p, want_grad=False)
    loss, alone, grad = loss.cpu().numpy(), alone.cpu().numpy(), grad.cpu().numpy().astype(np.float64)
    NN = prob.N * prob.N
    so, _ = parity.tie_override(prob.N, J, p[5:5 + NN], plan.starlet_fwd(p[5:5 + NN]).cpu().numpy())
    lo, go = ora.psf_loss_grad(prob, d, w, p, sgn_override=so)
    assert abs(loss[2] - lo[2]) <= 1e-6 * abs(lo[2]) and abs(alone[2] - lo[2]) <= 1e-6 * abs(lo[2])
    for k, v in parity.psf_blocks(prob, go).items():
        assert parity.rel_err(parity.psf_blocks(prob, grad)[k], v) <= 1e-4, k
