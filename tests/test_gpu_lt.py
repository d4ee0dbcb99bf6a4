"""GPU parity of the transposed solve's L^T pass at the edges of its matrix-core
kernel: terms in groups of four and blocks of 32, rows staged 64 at a time and
fewer, the kl = 1024 limit, an interchange at every row (near and far), signed
zeros, subnormals and infinities.  Bit for bit against the CPU oracle: the
kernel sums in the order of the definition with one rounding per term."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_22099_amd import bandlu  # noqa: E402
from test_gpu_structures import gpu, same  # noqa: E402

CASES = [(2, 1, 0), (3, 2, 1), (64, 1, 1), (65, 3, 2), (130, 4, 0), (129, 5, 3), (200, 31, 2),
         (200, 32, 1), (257, 33, 4), (300, 36, 0), (300, 63, 1), (400, 64, 0), (191, 65, 3),
         (500, 127, 2), (700, 128, 0), (600, 130, 1), (900, 257, 5), (1100, 833, 1),
         (1300, 1023, 0), (1300, 1024, 2), (1300, 1025, 1)]


def factors(n, kl, ku, seed, special):
    """Factor-shaped data (any values are valid factors for the solve)."""
    rng = np.random.default_rng(seed)
    kv = kl + ku
    AB = rng.uniform(-1.0, 1.0, (n, 2 * kl + ku + 1)) / max(1, kl) ** 0.5
    AB[:, kv] = rng.choice([-1.0, 1.0], n) * rng.uniform(1.0, 2.0, n)
    B = rng.standard_normal((2, n))
    j = np.arange(n)
    top = np.minimum(j + kl, n - 1)
    p = np.where(rng.random(n) < 0.3, np.minimum(j + 1, top), rng.integers(j, top + 1))
    if special:
        pick = rng.random(AB.shape)
        AB[(pick < 0.1) & (np.arange(AB.shape[1]) != kv)] = -0.0
        AB[(pick > 0.9) & (np.arange(AB.shape[1]) != kv)] = 0.0
        B[0, rng.random(n) < 0.3] = -0.0
        B[1] *= 1e-310  # subnormal right-hand side
    return AB, (p + 1).astype(np.int32), B


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("n,kl,ku", CASES)
def test_lt_pass(n, kl, ku, special):
    print(f"lt n={n} kl={kl} ku={ku} special={special}", flush=True)
    AB, ipiv, B = factors(n, kl, ku, 7000 + n + kl, special)
    ref = B.copy()
    oracle.gbtrs_t(AB, kl, ku, ipiv, ref)
    Bg = gpu(B)
    bandlu.band_getrs_t(gpu(AB), kl, ku, gpu(ipiv), Bg)
    torch.cuda.synchronize()
    assert same(Bg.cpu().numpy(), ref)


def test_lt_pass_infinity_and_many_systems():
    """An infinity spreads as in the definition; 600 systems take the smaller
    staging halves."""
    n, kl, ku = 150, 6, 3
    AB, ipiv, B = factors(n, kl, ku, 7100, True)
    B = np.repeat(B[:1], 600, axis=0) * np.linspace(0.5, 2.0, 600)[:, None]
    B[1::2, n - 20] = np.inf
    ref = B.copy()
    oracle.gbtrs_t(AB, kl, ku, ipiv, ref)
    Bg = gpu(B)
    bandlu.band_getrs_t(gpu(AB), kl, ku, gpu(ipiv), Bg)
    torch.cuda.synchronize()
    assert same(Bg.cpu().numpy(), ref)


@pytest.mark.parametrize("n,kl,ku", [(4, 3, 0), (5, 1, 0), (5, 4, 0), (33, 31, 1), (34, 33, 0), (60, 4, 0),
                                     (61, 4, 0), (64, 1, 0), (100, 28, 0), (100, 29, 0), (128, 64, 0),
                                     (160, 97, 0), (191, 65, 1), (192, 64, 1), (193, 63, 1), (200, 190, 0)])
def test_lt_pass_small_windows(n, kl, ku):
    """Vectors that fit the window whole: an infinity at each end and in between
    meets no padded term (a zero times it would be NaN); one system and many."""
    print(f"lt small n={n} kl={kl} ku={ku}", flush=True)
    AB, ipiv, B = factors(n, kl, ku, 7200 + n, False)
    at = [0, 1, n // 2, max(0, n - 1 - kl), n - 2, n - 1]
    B = np.repeat(B[:1], 7, axis=0)
    for r, q in enumerate(at):
        B[r, q] = np.inf
    ref = B.copy()
    oracle.gbtrs_t(AB, kl, ku, ipiv, ref)
    for copies in (1, 90):
        Bg = gpu(np.tile(B, (copies, 1)))
        bandlu.band_getrs_t(gpu(AB), kl, ku, gpu(ipiv), Bg)
        torch.cuda.synchronize()
        assert same(Bg.cpu().numpy(), np.tile(ref, (copies, 1)))
