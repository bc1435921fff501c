"""Vectors of one and two cells in short chunks without absorption, on the
march loop and off it, against the one-pass step: chunks shorter than a run of
six planes and not a multiple of it, detection faces inside and at the ends."""
import pytest

from tests.test_two_step_march_gpu import test_march_is_bitwise_the_one_pass_step as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,tx,ty,zc,kdet", [
    ("f32", (37, 29, 53), 16, 9, 27, 30), ("f32", (37, 29, 53), 16, 9, 7, 52),    # W 1
    ("f64", (37, 29, 53), 16, 20, 27, 30), ("f64", (37, 29, 53), 16, 9, 20, 0),
    ("f32", (38, 30, 45), 38, 12, 23, 20), ("f32", (38, 30, 100), 38, 12, 50, 20),  # W 2: off, on
])
def test_narrow_vectors_without_absorption(prec, n, tx, ty, zc, kdet):
    check(prec, n, tx, ty, zc, 0, kdet, 0)
