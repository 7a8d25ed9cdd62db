"""The one-launch forward where its work groups are fullest: the largest transforms with as many
sources as their tables leave room for, and a frame whose data are not finite beside others of
its work group.

Bars as in the parity suite: loss <= 1e-6 and gradient <= 1e-4 (relative, L2) against the FP64
oracle."""
import numpy as np
import pytest

from oracle import oracle as ora
from oracle import parity
from paper_2402_08725_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _problem(n, K, s, E, M, seed):
    prob = synth.make_small_deconv(seed, E, [n], K, s, s * n, M, 1)
    rng = np.random.default_rng(seed)
    d, w = synth.add_noise(rng.uniform(0, 300, prob.data_size), rng)
    return prob, d, w, synth.eval_point(prob, "near", rng)


def _plan(prob, d, w):
    from paper_2402_08725_amd import starred as st
    plan = st.Plan.for_problem(prob, conv_algo=st.CONV_FFT)
    plan.set_frames(d, w, prob.kernels, prob.W)
    return plan


@pytest.mark.parametrize("Q,s,M", [(150, 3, 3), (160, 2, 3), (160, 2, 4), (160, 2, 6), (180, 1, 6), (192, 1, 0)])
def test_sources_of_the_largest_transforms(Q, s, M):
    print(f"Q {Q} s {s} M {M}", flush=True)
    n = Q - 11
    prob, d, w, p = _problem(n, 2 * s * 11, s, 3, M, Q + M)
    plan = _plan(prob, d, w)
    ci = plan.classes()[0]
    assert ci["Q"] == Q and ci["fused"], ci
    loss, grad = plan.loss_grad(p)
    loss, grad = loss.cpu().numpy(), grad.cpu().numpy().astype(np.float64)
    lo, go = ora.loss_grad(prob, d, w, p)
    assert abs(loss[2] - lo[2]) <= 1e-6 * abs(lo[2])
    for name, blk in parity.deconv_blocks(prob, grad).items():
        assert parity.rel_err(blk, parity.deconv_blocks(prob, go)[name]) <= 1e-4, name


@pytest.mark.parametrize("s", [1, 2, 3])
@pytest.mark.parametrize("n,K,E", [(2, 3, 3), (8, 5, 3), (13, 3, 3), (16, 1, 3), (11, 9, 0)])
def test_the_shortest_transform(s, n, K, E):
    """Q = 16, for shorter needs too; E = 0: more frames than compute units."""
    print(f"n {n} K {K} s {s}", flush=True)
    E = E or torch.cuda.get_device_properties(0).multi_processor_count + 2
    prob, d, w, p = _problem(n, K, s, E, 1 if n == 2 else 3, n + s)
    plan = _plan(prob, d, w)
    ci = plan.classes()[0]
    assert ci["Q"] == 16 and ci["fused"], ci
    loss, grad = plan.loss_grad(p)
    loss, grad = loss.cpu().numpy(), grad.cpu().numpy().astype(np.float64)
    lo, go = ora.loss_grad(prob, d, w, p)
    assert abs(loss[2] - lo[2]) <= 1e-6 * abs(lo[2])
    for name, blk in parity.deconv_blocks(prob, grad).items():
        assert parity.rel_err(blk, parity.deconv_blocks(prob, go)[name]) <= 1e-4, name


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,K", [(12, 24), (40, 80)])  # groups of four frames, and of two
def test_a_frame_that_is_not_finite_leaves_the_others(n, K, bad):
    """The gradient of every other frame's background and amplitudes: the same bits."""
    print(f"n {n} {bad}", flush=True)
    E, M = torch.cuda.get_device_properties(0).multi_processor_count + 3, 2
    prob, d, w, p = _problem(n, K, 2, E, M, n)
    plan = _plan(prob, d, w)
    assert plan.classes()[0]["fused"]
    _, grad = plan.loss_grad(p)
    frame = 5
    poisoned = d.copy()
    poisoned[frame * n * n + 7] = bad
    plan.set_frames(poisoned, w, prob.kernels, prob.W)
    loss, got = plan.loss_grad(p)
    assert not np.isfinite(loss[2].item())
    NN = prob.N ** 2
    for ref, out in [(grad[NN:NN + E, None], got[NN:NN + E, None]),
                     (grad[NN + E:NN + E + E * M].reshape(E, M), got[NN + E:NN + E + E * M].reshape(E, M))]:
        keep = torch.arange(E) != frame
        assert torch.equal(ref[keep], out[keep])
        assert not torch.isfinite(out[frame]).any()
