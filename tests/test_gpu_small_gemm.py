"""The orbital step's products at the edges of the small GEMM's tiles: 32 x 32 up to
128 tiles of 64 x 64 (n of 704: 121 of them), 64 x 64 above (n of 705: 144), and
remainders of both.  Checked as the eigensolver tests check a diagonalisation:
residual, orthogonality and eigenvalues, with their tolerances."""
import pytest

from tests.test_gpu_eig import check, ctx, diagonalise, random_sym  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [31, 32, 33, 64, 65, 161, 704, 705])
def test_orbital_products(ctx, n):  # noqa: F811
    print("case small gemm:", n, flush=True)
    F = random_sym(n, 1000 + n)
    w, V = diagonalise(ctx, F, 3)
    check(F, w, V)
