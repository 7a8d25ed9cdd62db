"""The order in which an evaluation launches its kernels, where it is chosen by measurement."""
import pytest

import fake_hip


@pytest.mark.parametrize("n,s,J", [(32, 2, 1), (129, 2, 6), (33, 2, 7)])
def test_psf_prior_on_its_own_stream_is_launched_by_its_length(tmp_path, n, s, J):
    """PSF mode, the prior's passes not carried by other launches: a chain (a grid above 256) goes
    first, the one plane of J = 1 after the render. (Of the last case the passes are carried.)"""
    out = fake_hip.run(tmp_path, f"""
h = make_plan([{n}] * 3, [1] * 3, {s}, {n * s}, 0, {J}, mode=st.PSF)
assert L.starred_set_frames(h, ptr(f32(3 * {n} ** 2)), ptr(f32(3 * {n} ** 2)), None, ptr(f32({J}))) == st.OK
P = L.starred_num_params(h)
launches([])
assert L.starred_loss_grad(h, ptr(f32(P)), ptr(f32(P)), ptr(np.zeros(3))) == st.OK
print(*launches(["k_star_plane", "k_star_forward", "k_star_adjoint", "k_copy", "k_psf_render64", "k_psf_fwd",
                 "k_psf_adjsum", "k_psf_finalize"]))
""").split()
    prior = [k for k in out if k.startswith("k_star") or k == "k_copy"]
    evaluation = ["k_psf_render64", "k_psf_fwd", "k_psf_adjsum", "k_psf_finalize"]
    assert out == (evaluation[:1] + prior + evaluation[1:] if J == 1 else prior + evaluation)
    assert bool(prior) == (J == 1 or n * s > 256)


@pytest.mark.parametrize("n,s,J,carried", [(32, 2, 1, 0), (129, 2, 6, 0), (16, 2, 2, 2), (33, 2, 7, 4)])
def test_psf_launches_without_a_pass_are_compiled_without_one(tmp_path, n, s, J, carried):
    out = fake_hip.run(tmp_path, f"""
h = make_plan([{n}] * 3, [1] * 3, {s}, {n * s}, 0, {J}, mode=st.PSF)
assert L.starred_set_frames(h, ptr(f32(3 * {n} ** 2)), ptr(f32(3 * {n} ** 2)), None, ptr(f32({J}))) == st.OK
P = L.starred_num_params(h)
launches([])
assert L.starred_loss_grad(h, ptr(f32(P)), ptr(f32(P)), ptr(np.zeros(3))) == st.OK
print(*[("StarPiece" in k) + ("NoPiece" in k) * 10 for k in hip.fake_launches().decode().split() if "k_psf" in k])
""").split()
    assert sorted(out) == ["1"] * carried + ["10"] * (4 - carried)


def test_line_passes_carry_prior_jobs_only_where_some_ride(tmp_path):
    """Kernels of the spectra's and of dL/dh's passes, without and with the prior's passes in
    them: compiled for the jobs where they ride, and never elsewhere."""
    out = fake_hip.run(tmp_path, """
for J in (1, 4):  # (one plane has nothing to ride)
    h = make_plan([32] * 4, [16] * 4, 2, 64, 1, J)
    n = 4 * 32 * 32
    assert L.starred_set_frames(h, ptr(f32(n)), ptr(f32(n)), ptr(f32(4 * 256)), ptr(f32(4))) == st.OK
    P = L.starred_num_params(h)
    launches([])
    assert L.starred_loss_grad(h, ptr(f32(P)), ptr(f32(P)), ptr(np.zeros(3))) == st.OK
    names = [k for k in hip.fake_launches().decode().split() if "7k_lines" in k]
    print(sum("DensePiece" in k for k in names), sum("NoPiece" in k for k in names), len(names))
""").splitlines()
    assert out == ["0 4 4", "3 1 4"]


def test_lambda_pts_estimate_transforms_four_images_per_launch(tmp_path):
    out = fake_hip.run(tmp_path, """
h = make_plan([32] * 2, [9] * 2, 1, 32, 7, 4)
assert L.starred_set_frames(h, ptr(f32(2048)), ptr(f32(2048)), ptr(f32(162)), ptr(f32(4))) == st.OK
launches([])
L.starred_estimate_lambda_pts(h, ptr(f32(L.starred_num_params(h))), ctypes.byref(ctypes.c_double()))
print(len(launches(["k_star_forward"])))
""")
    assert int(out) == 3  # nine images, one group of three levels


def test_line_passes_go_on_while_the_prior_is_launched(tmp_path):
    """An evaluation on the line passes alone: the main stream has its spectra, product and columns
    before the host turns to the prior's branch."""
    out = fake_hip.run(tmp_path, """
h = make_plan([32] * 2, [16] * 2, 2, 64, 1, 4)
assert L.starred_set_frames(h, ptr(f32(2048)), ptr(f32(2048)), ptr(f32(512)), ptr(f32(4))) == st.OK
assert L.starred_set_fft_fused(h, 0) == st.OK
P = L.starred_num_params(h)
launches([])
assert L.starred_loss_grad(h, ptr(f32(P)), ptr(f32(P)), ptr(np.zeros(3))) == st.OK
print(*launches(["OpHCols", "k_spec_fwd", "OpMCols", "k_star_forward", "k_fwd_rows"]))
""").split()
    assert out == ["OpHCols", "k_spec_fwd", "OpMCols", "k_star_forward", "k_fwd_rows"]
