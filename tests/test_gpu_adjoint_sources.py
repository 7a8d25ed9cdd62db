"""The frequency-domain adjoint with many sources: every count of sources a pass over the spectra
takes, the last pass full and partly filled, the last chunk of frames partly filled.

Bar as in the parity suite: gradient <= 1e-4 per block (relative, L2) against the FP64 oracle."""
import numpy as np
import pytest

from oracle import oracle as ora
from oracle import parity
from paper_2402_08725_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("s", [1, 2, 3])
@pytest.mark.parametrize("M", [9, 16, 17])
def test_chunks(s, M):
    from paper_2402_08725_amd import starred as st
    print(f"s {s} M {M}", flush=True)
    prob = synth.make_small_deconv(s * M, 5, [40, 28], [12 * s, 9], s, 40 * s, M, 1)
    rng = np.random.default_rng(s * M)
    d, w = synth.add_noise(rng.uniform(0, 300, prob.data_size), rng)
    p = synth.eval_point(prob, "near", rng)
    lo, go = ora.loss_grad(prob, d, w, p)
    plan = st.Plan.for_problem(prob, conv_algo=st.CONV_FFT)
    plan.set_frames(d, w, prob.kernels, prob.W)
    for frames in (1, 2, 4):
        for blocks in (512, 9):  # few rows per work group, and many
            plan.set_fft_shapes(adj_frames=frames, adj_blocks=blocks)
            _, grad = plan.loss_grad(p)
            grad = grad.cpu().numpy().astype(np.float64)
            for name, blk in parity.deconv_blocks(prob, grad).items():
                assert parity.rel_err(blk, parity.deconv_blocks(prob, go)[name]) <= 1e-4, (frames, blocks, name)
