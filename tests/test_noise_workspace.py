"""What a plan keeps for noise_weights between calls: the auxiliary plan with one frame's
kernel and the buffers of a batch."""
import numpy as np
import pytest

import fake_hip

SETUP = """
sides, ks, s, N, M, J = [16, 16, 12], [9, 9, 7], 2, 32, 1, 3
h = make_plan(sides, ks, s, N, M, J)
kern_at = np.cumsum([0] + [k * k for k in ks])
psf = f32(kern_at[-1], 1.0)
nd = sum(n * n for n in sides)
data, inv, w = f32(nd), f32(nd), f32(J)
def bind(k):
    assert L.starred_set_frames(h, ptr(data), ptr(inv), ptr(k), ptr(w)) == st.OK
def weights(frame, n_real=40):
    out = f32(J * N * N)
    return L.starred_noise_weights(h, frame, ptr(f32(sides[frame] ** 2, 1.0)), n_real, 1, None, 1, ptr(out))
def reads(k, frame):
    return hip.fake_copies_from(k.ctypes.data + 4 * int(kern_at[frame]))
bind(psf)
"""


def test_a_new_binding_is_read(tmp_path):
    """Weights asked for after other kernels are bound take those kernels."""
    fake_hip.run(tmp_path, SETUP + """
assert weights(0) == st.OK and reads(psf, 0) > 0
other = f32(kern_at[-1], 2.0)
bind(other)
assert weights(0) == st.OK and reads(other, 0) > 0
L.starred_plan_destroy(h)
""")


def test_a_loop_over_frames_holds_one_set_of_buffers(tmp_path):
    """Frames of another shape replace the buffers, those of the same shape use them."""
    fake_hip.run(tmp_path, SETUP + """
assert weights(2) == st.OK
small = hip.fake_live_bytes()
assert weights(0) == st.OK
held, mallocs = hip.fake_live_bytes(), hip.fake_mallocs()
assert weights(1) == st.OK and reads(psf, 1) > 0
assert weights(0, 20) == st.OK
assert (hip.fake_live_bytes(), hip.fake_mallocs()) == (held, mallocs)
for frame in (2, 0, 1, 2):
    assert weights(frame) == st.OK
    assert hip.fake_live_bytes() == (small if frame == 2 else held)
L.starred_plan_destroy(h)
assert hip.fake_live_count() == 0
""")


def test_out_of_memory_leaves_nothing_half_made(tmp_path):
    """Each allocation in turn fails, of a first call and of one that asks for a larger batch:
    the call says so, and the next one has every buffer."""
    fake_hip.run(tmp_path, SETUP + """
base = hip.fake_live_bytes()
for first in (0, 20):
    k = 0
    while True:
        L.starred_plan_destroy(h)
        h = make_plan(sides, ks, s, N, M, J)
        bind(psf)
        if first:
            assert weights(0, first) == st.OK
        k += 1
        m = hip.fake_mallocs()
        hip.fake_fail_malloc_in(k)
        rc = weights(0)
        hip.fake_fail_malloc_in(-1)
        if rc == st.OK:
            assert hip.fake_mallocs() - m < k  # (no allocation was left to fail)
            break
        assert rc in (st.ENOMEM, st.EHIP)
        assert hip.fake_live_bytes() == base
        m = hip.fake_mallocs()
        assert weights(0) == st.OK
        made, held = hip.fake_mallocs() - m, hip.fake_live_bytes()
        if k > 1:
            assert (made, held) == last
        last = (made, held)
    assert k > 12
L.starred_plan_destroy(h)
assert hip.fake_live_count() == 0
""")


@pytest.mark.gpu
def test_weights_after_a_new_binding_equal_a_fresh_plan():
    torch = pytest.importorskip("torch")
    from paper_2402_08725_amd import starred as st
    from paper_2402_08725_amd import synth
    prob = synth.make_small_deconv(3, 2, [12, 16], 9, 2, 32, 1, 3)
    rng = np.random.default_rng(3)
    d, w = synth.add_noise(rng.uniform(0, 300, prob.data_size), rng)
    other = synth.f32(prob.kernels * rng.uniform(0.5, 1.5, prob.kernels.size))
    sigma2 = synth.f32(rng.uniform(0.5, 2.0, prob.n[0] ** 2))

    def bound(plan, kernels):
        plan.set_frames(d, w, kernels, prob.W)
        return plan.noise_weights(sigma2, frame=0, n_real=70, seed=5)
    plan = st.Plan.for_problem(prob, conv_algo=st.CONV_FFT)
    first = bound(plan, prob.kernels)
    second = bound(plan, other)
    fresh = bound(st.Plan.for_problem(prob, conv_algo=st.CONV_FFT), other)
    assert torch.equal(second, fresh)  # (the same launches on the same inputs)
    assert not torch.equal(second, first)
