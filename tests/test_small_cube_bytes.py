"""The bytes that a plan reports for cubes of n <= 64: three passes (CPU).

P1 writes W1 once and the plane pass reads it; that writes 2 n^3 complex values
once, which P5 reads.  Larger cubes move W1 four times and W2 four times."""
import pytest

psn = pytest.importorskip("paper_1612_01799_amd")


@pytest.mark.parametrize("dt,bio,b1,b2,bk", [("f32", 4, 8, 8, 4), ("f64", 8, 16, 16, 8), ("split", 8, 12, 16, 8)])
@pytest.mark.parametrize("n", [8, 32, 64, 96])
def test_bytes_of_the_passes_that_run(n, dt, bio, b1, b2, bk):
    w1, w2 = (2, 2) if n <= 64 else (4, 4)   # transfers of n^3 and of 2 n^3 elements
    want = 2 * bio * n ** 3 + w1 * b1 * n ** 3 + w2 * b2 * 2 * n ** 3 + bk * (n + 1) ** 3
    assert psn.Plan(n, 2.0, 1e-12, dt).info()["algorithmic_bytes"] == want
