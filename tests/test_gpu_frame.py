"""The one-launch forward at every transform length it has, against the oracle and
against the line passes, with one frame and with several frames per work group.

Bars as in the parity suite: loss <= 1e-6 and gradient <= 1e-4 (relative, L2) against the
FP64 oracle; 1e-5 between two FP32 evaluations (twice the rounding of transforms of
up to 540 points, a few 1e-7, with the same margin as between launch shapes).
"""
import numpy as np
import pytest

from oracle import oracle as ora
from oracle import parity
from paper_2402_08725_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = [18, 20, 24, 30, 32, 36, 40, 48, 50, 54, 60, 64, 72, 80, 90, 96, 100, 108, 120, 128, 144, 150, 160, 180]


def _problem(Q, s, E, M, seed):
    # frames of side n with a kernel that needs the whole length: s n + K/2 = s Q
    n = int(0.8 * Q) - (Q // 2) % 2  # odd sides too
    K = 2 * s * (Q - n) + (Q // 4) % 2
    prob = synth.make_small_deconv(seed, E, [n], K, s, s * n, M, 1)
    rng = np.random.default_rng(seed)
    d, w = synth.add_noise(rng.uniform(0, 300, prob.data_size), rng)
    return prob, d, w, synth.eval_point(prob, "near", rng)


def _plan(prob, d, w):
    from paper_2402_08725_amd import starred as st
    plan = st.Plan.for_problem(prob, conv_algo=st.CONV_FFT)
    plan.set_frames(d, w, prob.kernels, prob.W)
    return plan


def _eval(plan, p):
    loss, grad = plan.loss_grad(p)
    alone, _ = plan.loss_grad(p, want_grad=False)
    torch.cuda.synchronize()
    # the loss alone is the same launch, cut short: the same FP64 partials (a thousand at most
    # here), added by another final launch in another order
    assert abs(loss[2].item() - alone[2].item()) <= 1000 * 2.0 ** -53 * abs(loss[2].item())
    return loss.cpu().numpy(), grad.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("s", [1, 2, 3])
@pytest.mark.parametrize("Q", LENGTHS)
def test_length(Q, s):
    M = (0, 1, 3, 6)[(Q // 2 + s) % 4]
    if Q >= 150 and M > 1:
        M = 1  # (the tables of more sources fill the LDS: such frames take the line passes)
    print(f"Q {Q} s {s} M {M}", flush=True)
    prob, d, w, p = _problem(Q, s, 3, M, 7 * Q + s)
    plan = _plan(prob, d, w)
    ci = plan.classes()[0]
    assert ci["Q"] == Q and ci["fused"], ci
    loss, grad = _eval(plan, p)
    lo, go = ora.loss_grad(prob, d, w, p)
    assert abs(loss[2] - lo[2]) <= 1e-6 * abs(lo[2])
    for name, blk in parity.deconv_blocks(prob, grad).items():
        assert parity.rel_err(blk, parity.deconv_blocks(prob, go)[name]) <= 1e-4, name
    plan.set_fft_fused(False)
    _, lines = _eval(plan, p)
    assert parity.rel_err(grad, lines) <= 1e-5


@pytest.mark.parametrize("M", [1, 3, 6])
@pytest.mark.parametrize("Q", [q for q in LENGTHS if q <= 72] + [80, 90, 96, 100, 108, 128])
def test_several_frames_per_group(Q, M):
    """More frames than compute units: groups of four or two, the last one partly filled."""
    print(f"Q {Q} M {M}", flush=True)
    prob, d, w, p = _problem(Q, 2, torch.cuda.get_device_properties(0).multi_processor_count + 3, M, 11 * Q + M)
    plan = _plan(prob, d, w)
    assert plan.classes()[0]["Q"] == Q and plan.classes()[0]["fused"]
    loss, grad = _eval(plan, p)
    plan.set_fft_fused(False)
    ll, lines = _eval(plan, p)
    assert abs(loss[2] - ll[2]) <= 1e-6 * abs(ll[2])
    for name, blk in parity.deconv_blocks(prob, grad).items():
        assert parity.rel_err(blk, parity.deconv_blocks(prob, lines)[name]) <= 1e-5, name
