"""The bundle adjustment's solve at the edges of its 16-row tiles: with F free
keyframes the system has 6F + 1 unknowns and the right-hand side as one more
row, so F = 2, 5 and 13 end on or next to a tile's edge, F = 11 is the first
whose first panel needs a second wave, F = 20 is the largest; and steps whose
rotations pass from the exponential's power series to its closed form.  One
step against the FP64 oracle, at the same relative 1e-8 (both sides FP64, the
order of sums apart)."""
import pytest

pytest.importorskip("torch")

from paper_2607_14481_amd.ba_scenes import make_problem

from .test_gpu_ba import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_free", [1, 2, 3, 5, 8, 10, 11, 13, 16, 18, 20])
def test_system_sizes(n_free):
    P = make_problem(40 + n_free, n_cams=n_free + 2, n_landmarks=40 + 13 * n_free, n_fixed=2, max_obs=min(8, n_free + 2),
                     pixel_noise=0.5)
    _compare(P, 1)


@pytest.mark.parametrize("rot_noise", [0.1, 0.35])
def test_large_rotations(rot_noise):
    P = make_problem(70, n_cams=6, n_landmarks=200, n_fixed=2, max_obs=4, pixel_noise=0.5, rot_noise=rot_noise)
    _compare(P, 1)
