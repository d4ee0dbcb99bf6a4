"""GPU parity of the pivoting column steps of the persistent wide-band LU:
ties between rows of one wave and of several (equal magnitudes, equal high
words), pivots below DBL_MIN, zero columns among ties, panels that interchange
followed by panels that do not and the reverse, and windows that leave waves
without candidates.  Pivots and info exactly, factors within the elementwise
tolerance (a tie decided otherwise gives another pivot)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_22099_amd import inputs  # noqa: E402
from test_gpu_wide import check  # noqa: E402

SHAPES = [(400, 32, 0), (300, 40, 64), (500, 100, 37), (700, 256, 31), (90, 64, 89)]


def ties(n, kl, ku, seed):
    """Entries of one magnitude and either sign, in band."""
    T = inputs.banded_dense(n, kl, ku, seed, check=False)
    return np.sign(T)


@pytest.mark.parametrize("n,kl,ku", SHAPES)
def test_equal_magnitudes(n, kl, ku):
    # the first columns are exact ties; later ones tie after exact sums
    check(ties(n, kl, ku, n + kl), kl, ku, f"ties n={n} kl={kl} ku={ku}")


@pytest.mark.parametrize("n,kl,ku", SHAPES)
def test_equal_high_words(n, kl, ku):
    # magnitudes that differ in the low words only: the settling path decides
    T = ties(n, kl, ku, 7 + n)
    low = np.random.default_rng(n).integers(0, 4, T.shape)
    check(T * (1.0 + low * 2.0 ** -50), kl, ku, f"low words n={n} kl={kl} ku={ku}")


@pytest.mark.parametrize("n,kl,ku", SHAPES)
def test_tiny_pivots(n, kl, ku):
    T = inputs.banded_dense(n, kl, ku, 11 + n, check=False)
    T[n // 3] *= 1e-308  # a column whose pivot is below DBL_MIN
    check(T, kl, ku, f"tiny column n={n} kl={kl} ku={ku}")


@pytest.mark.parametrize("n,kl,ku", SHAPES)
def test_panels_change_between_paths(n, kl, ku):
    # dominant columns with runs of pivoting ones, and a zero column in a run
    T = inputs.banded_dense(n, kl, ku, 13 + n, shift=4.0 * (kl + ku), check=False)
    U = inputs.banded_dense(n, kl, ku, 17 + n, check=False)
    for j in range(0, n, 192):
        T[j:j + 70] = U[j:j + 70]
    T[min(n - 1, 65)] = 0.0
    check(T, kl, ku, f"mixed n={n} kl={kl} ku={ku}")
