"""Transform lengths of the shape classes where the next 5-smooth length has no one-launch
forward: Q = 162 becomes 180 only where a class gains that forward by it."""
import numpy as np
import pytest

import fake_hip

# n, K, s, M -> Q, one-launch forward
CASES = [
    (150, 23, 1, 1, 180, True),
    (150, 23, 1, 6, 180, True),
    (150, 23, 1, 12, 162, False),   # the tables of twelve sources fill the LDS
    (150, 46, 2, 1, 180, True),
    (150, 46, 2, 2, 162, False),
    (155, 40, 3, 1, 162, False),
    (155, 40, 3, 2, 162, False),
    (8, 3, 1, 1, 16, True),
    (8, 5, 2, 2, 16, True),
    (13, 9, 3, 1, 16, True),
    (13, 13, 1, 1, 20, True),
    (6, 5, 3, 300, 8, False),
    (150, 80, 1, 1, 192, False),
    (150, 80, 1, 0, 192, True),
    (160, 126, 2, 0, 192, False),
]


@pytest.mark.parametrize("n,K,s,M,Q,fused", CASES)
def test_length(tmp_path, n, K, s, M, Q, fused):
    out = fake_hip.run(tmp_path, f"""
h = make_plan([{n}], [{K}], {s}, {s * n}, {M}, 1)
ci = st.ClassInfo()
assert L.starred_get_class_info(h, 0, ctypes.byref(ci)) == st.OK
print(ci.Q, ci.P, ci.fused)
""").split()
    assert [int(out[0]), int(out[1]), int(out[2]) > 0] == [Q, s * Q, fused]


@pytest.mark.gpu
@pytest.mark.parametrize("n,K,s,M", [c[:4] for c in CASES if c[4] == 162])
def test_line_passes_at_162(n, K, s, M):
    pytest.importorskip("torch")
    from oracle import oracle as ora
    from oracle import parity
    from paper_2402_08725_amd import starred as st
    from paper_2402_08725_amd import synth
    print(f"n {n} K {K} s {s} M {M}", flush=True)
    prob = synth.make_small_deconv(n + M, 2, [n], K, s, s * n, M, 1)
    rng = np.random.default_rng(n + M)
    d, w = synth.add_noise(rng.uniform(0, 300, prob.data_size), rng)
    p = synth.eval_point(prob, "near", rng)
    plan = st.Plan.for_problem(prob, conv_algo=st.CONV_FFT)
    plan.set_frames(d, w, prob.kernels, prob.W)
    loss, grad = plan.loss_grad(p)
    loss, grad = loss.cpu().numpy(), grad.cpu().numpy().astype(np.float64)
    lo, go = ora.loss_grad(prob, d, w, p)
    # the parity suite's bars
    assert abs(loss[2] - lo[2]) <= 1e-6 * abs(lo[2])
    for name, blk in parity.deconv_blocks(prob, grad).items():
        assert parity.rel_err(blk, parity.deconv_blocks(prob, go)[name]) <= 1e-4, name
