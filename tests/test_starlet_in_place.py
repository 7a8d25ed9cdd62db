"""The starlet transform and its transpose with the image held in the coefficients' own memory."""
import pytest

import fake_hip


@pytest.mark.parametrize("mode,J", [("DECONV", 4), ("PSF", 4), ("DECONV", 1)])
def test_overlapping_input_is_copied_first(tmp_path, mode, J):
    """A pass writes while others still read: where the two overlap the input is taken from a
    copy, whichever plane the image lies in; where they do not, no copy is made."""
    fake_hip.run(tmp_path, f"""
N, J = 24, {J}
h = make_plan([12], [5], 2, N, 0, J, mode=st.{mode})
buf = f32((J + 1) * N * N)
keep.append(buf)
def at(plane):
    return ctypes.c_void_p(buf.ctypes.data + 4 * plane * N * N)
for plane in range(J):
    for f, inp, args in ((L.starred_starlet_fwd, at(plane), (at(plane), at(0))),
                         (L.starred_starlet_adj, at(0), (at(0), at(plane)))):
        before = hip.fake_copies_from(inp)
        assert f(h, *args) == st.OK
        assert hip.fake_copies_from(inp) == before + (J > 1 or plane > 0)
        assert f(h, *((at(J), at(0)) if f is L.starred_starlet_fwd else (at(0), at(J)))) == st.OK
        assert hip.fake_copies_from(inp) == before + (J > 1 or plane > 0) and hip.fake_copies_from(at(J)) == 0
L.starred_plan_destroy(h)
""")


@pytest.mark.gpu
@pytest.mark.parametrize("N,J", [(33, 3), (129, 6), (300, 8)])
def test_in_place_equals_out_of_place(N, J):
    import ctypes
    import numpy as np
    torch = pytest.importorskip("torch")
    from paper_2402_08725_amd import starred as st
    plan = st.Plan(st.DECONV, [N], [3], 1, N, 0, J, 3.0)
    img = torch.from_numpy(np.random.default_rng(N).standard_normal(N * N).astype(np.float32)).cuda()
    ref = plan.starlet_fwd(img)
    back = plan.starlet_adj(ref)
    for plane in (0, J - 1):
        buf = torch.zeros_like(ref)
        buf[plane * N * N:(plane + 1) * N * N] = img
        at = ctypes.c_void_p(buf.data_ptr() + 4 * plane * N * N)
        plan._call(st.lib().starred_starlet_fwd, at, ctypes.c_void_p(buf.data_ptr()))
        assert torch.equal(buf, ref)  # (the same launches on the same values)
        plan._call(st.lib().starred_starlet_adj, ctypes.c_void_p(buf.data_ptr()), at)
        assert torch.equal(buf[plane * N * N:(plane + 1) * N * N], back)
