"""The operators on given scenes and residuals with few columns (all aliases of a column transformed
at once) and with many (one at a time), ragged frames among them.

Bar as in the parity suite: 2e-6 of the largest value."""
import numpy as np
import pytest

from oracle import oracle as ora
from paper_2402_08725_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("s", [1, 2, 3])
@pytest.mark.parametrize("E,n,K", [(1, 9, 4), (3, 64, 9), (5, 33, 80), (40, 33, 15), (130, 14, 9)])
def test_model_and_back_projection(s, E, n, K):
    from paper_2402_08725_amd import starred as st
    print(f"s {s} E {E} n {n} K {K}", flush=True)
    sides = [n] if E == 1 else [n, n - 4]
    prob = synth.make_small_deconv(s * E, E, sides, [K, K + 1] if E > 3 else K, s, s * n, 1, 1)
    rng = np.random.default_rng(s * E)
    scene = synth.f32(rng.standard_normal(int(np.sum((s * prob.n.astype(np.int64)) ** 2))))
    resid = synth.f32(rng.standard_normal(prob.data_size))
    plan = st.Plan.for_problem(prob, conv_algo=st.CONV_FFT)
    plan.set_frames(resid, np.ones_like(resid), prob.kernels, prob.W)
    for got, ref in ((plan.convolve_subsample(scene), ora.conv_sub(prob.n, prob.K, s, prob.kernels, scene)),
                     (plan.convolve_subsample_adj(resid), ora.conv_sub_adj(prob.n, prob.K, s, prob.kernels, resid))):
        assert np.abs(got.cpu().numpy() - ref).max() <= 2e-6 * np.abs(ref).max()
