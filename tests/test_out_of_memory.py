"""Buffers that a plan makes on first use: after an allocation has failed, the next call makes
what is missing and does not run on null pointers."""
import fake_hip

SETUP = """
sides, ks, s, N, M, J = [16, 16, 12], [9, 9, 7], 2, 32, 2, 3
nd = sum(n * n for n in sides)
def fresh():
    h = make_plan(sides, ks, s, N, M, J)
    assert L.starred_set_frames(h, ptr(f32(nd)), ptr(f32(nd, 1.0)), ptr(f32(sum(k * k for k in ks), 1.0)),
                                ptr(f32(J, 1.0))) == st.OK
    return h
"""


def test_estimate_lambda_pts(tmp_path):
    fake_hip.run(tmp_path, SETUP + """
out = ctypes.c_double()
for k in (1, 2, 3):
    h = fresh()
    params = f32(L.starred_num_params(h))
    hip.fake_fail_malloc_in(k)
    assert L.starred_estimate_lambda_pts(h, ptr(params), ctypes.byref(out)) == st.ENOMEM
    m = hip.fake_mallocs()
    # (the kernels do nothing here: the norms are zero, which the call refuses)
    assert L.starred_estimate_lambda_pts(h, ptr(params), ctypes.byref(out)) == st.EINVAL
    assert hip.fake_mallocs() - m == 4 - k
    L.starred_plan_destroy(h)
""")


def test_set_frame_transforms(tmp_path):
    """The partial planes of transformed frames: no memory for them leaves the plan without
    transforms and with the planes it had."""
    fake_hip.run(tmp_path, SETUP + """
sides, ks = [12] * 40, [7] * 40
nd = 40 * 144
h = fresh()
xf = f32(3 * 40)
before = hip.fake_live_bytes()
algo = ctypes.c_int32(-1)
def info():
    assert L.starred_frame_transforms_info(h, ctypes.byref(algo), None) == st.OK
    return algo.value
hip.fake_fail_malloc_in(1)
assert L.starred_set_frame_transforms(h, ptr(xf), None, st.CONV_FFT) == st.ENOMEM
assert info() == 0 and hip.fake_live_bytes() == before
assert L.starred_set_frame_transforms(h, ptr(xf), None, st.CONV_FFT) == st.OK
assert info() == st.CONV_FFT
L.starred_plan_destroy(h)
""")
