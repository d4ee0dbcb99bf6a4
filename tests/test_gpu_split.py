"""GPU parity of the pivot-wavefront band LU at its edges: one to seven update
wavefronts (windows around each multiple of 64 columns), one to thirty-one
rows (each group of interchange offsets), more rows than columns and the
reverse, special values, and what selects it.  Bit for bit against the CPU
oracle (every entry takes the unblocked algorithm's operations in its order)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_22099_amd import bandlu  # noqa: E402
from test_gpu_structures import gpu, same  # noqa: E402


def band(m, n, kl, ku, seed, shift=0.0, ldab=None):
    """Random band; every slot the factorisation may not read holds a marker."""
    rng = np.random.default_rng(seed)
    AB = np.full((n, ldab or 2 * kl + ku + 1), 7e77)
    for j in range(n):
        for i in range(max(0, j - ku - kl), min(m - 1, j + kl) + 1):
            AB[j, kl + ku + i - j] = rng.standard_normal() if i >= j - ku else 5e55
        if j < m:
            AB[j, kl + ku] += shift
    return AB


def check(AB, m, kl, ku, what, square=False):
    print(what, flush=True)
    ABg = gpu(AB)
    ipo, info_o, _ = oracle.gbtrf_mn(AB, m, kl, ku)
    if square:
        ipiv, info = bandlu.band_getrf(ABg, kl, ku)
    else:
        ipiv, info = bandlu.band_getrf_mn(ABg, m, kl, ku)
    torch.cuda.synchronize()
    assert np.array_equal(ipiv.cpu().numpy(), ipo) and int(info.cpu()[0]) == info_o
    assert same(ABg.cpu().numpy(), AB)


# windows of 64, 65, 127, 128, 129, 191, 192, 193, 255..257, 320, 321, 447, 448
# columns; kl = 31, 30 (odd prefetch depth), 17, 16, 15, 9, 8, 1
@pytest.mark.parametrize("kl,need", [(31, 64), (16, 65), (17, 127), (31, 128), (31, 129), (30, 191),
                                     (8, 192), (9, 193), (15, 255), (1, 256), (22, 257), (26, 320),
                                     (27, 321), (30, 447), (31, 448)])
@pytest.mark.parametrize("shift", [0.0, 1.0])
def test_windows(kl, need, shift):
    ku = need - 2 * kl - 1
    n = need + 150
    check(band(n, n, kl, ku, need + kl, shift * (kl + ku), need + 2), n, kl, ku,
          f"square n={n} kl={kl} ku={ku} shift={shift}", square=True)


@pytest.mark.parametrize("m,n,kl,ku", [(200, 150, 16, 16), (150, 200, 16, 16), (161, 160, 31, 31),
                                       (160, 161, 31, 31), (300, 40, 30, 39), (40, 300, 31, 200),
                                       (1, 70, 0, 69), (2, 70, 1, 69), (70, 2, 31, 1), (190, 190, 5, 90),
                                       (65, 64, 1, 0), (64, 65, 1, 0), (130, 300, 23, 150)])
def test_rectangular(m, n, kl, ku):
    check(band(m, n, kl, ku, m + n), m, kl, ku, f"rectangular m={m} n={n} kl={kl} ku={ku}")


@pytest.mark.parametrize("m,n", [(140, 140), (170, 140), (140, 170)])
@pytest.mark.parametrize("kl,ku", [(20, 30), (31, 70), (7, 120)])
def test_specials(m, n, kl, ku):
    base = band(m, n, kl, ku, kl + ku)
    kv = kl + ku
    for what in ("zero column", "nan", "inf", "-0.0", "tiny", "zero"):
        AB = base.copy()
        known = np.zeros(AB.shape, dtype=bool)
        for j in range(n):
            known[j, kv + max(-j, -ku):kv + min(kl, m - 1 - j) + 1] = True
        if what == "zero column":
            AB[77, known[77]] = 0.0
            AB[0, known[0]] = 0.0
        elif what == "nan":
            AB[50, kv] = AB[60, kv + 2] = np.nan
        elif what == "inf":
            AB[64, kv + 1] = np.inf
        elif what == "-0.0":
            AB[known & (np.random.default_rng(3).random(AB.shape) < 0.6)] = -0.0
        elif what == "tiny":
            AB[known] *= 1e-305
        else:
            AB[known] = 0.0
        check(AB, m, kl, ku, f"{what} m={m} n={n} kl={kl} ku={ku}")


def test_batched():
    batch, n, kl, ku = 70, 150, 24, 40
    AB = np.stack([band(n, n, kl, ku, 900 + b) for b in range(batch)])
    ABg = gpu(AB)
    ipiv, info = bandlu.band_getrf_batched(ABg, kl, ku)
    torch.cuda.synchronize()
    for b in range(batch):
        ipo, info_o, _ = oracle.gbtrf(AB[b], kl, ku)
        assert np.array_equal(ipiv.cpu().numpy()[b], ipo) and int(info.cpu()[b]) == info_o
        assert same(ABg.cpu().numpy()[b], AB[b])


@pytest.mark.parametrize("batch,kl,need", [(513, 7, 65), (1024, 12, 80), (1030, 14, 66), (1025, 13, 80),
                                           (704, 15, 81), (600, 9, 128), (705, 11, 81), (768, 14, 90),
                                           (2048, 9, 65), (2048, 15, 73), (1024, 15, 65), (2050, 7, 128),
                                           (2048, 16, 57), (2049, 19, 64)])
def test_batch_rules(batch, kl, need):
    """Batches at the edges of the rules for two columns per lane and for the
    number of resident workgroups; a few matrices of each batch, and the same
    for a band of fewer rows than columns."""
    ku = need - 2 * kl - 1
    print(f"batch={batch} kl={kl} need={need}", flush=True)
    for m, n in ((need + 140, need + 140), (need + 100, need + 140)):
        base = [band(m, n, kl, ku, 1300 + b, b % 2 * 2.0 * (kl + ku)) for b in range(5)]
        AB = np.stack([base[b % 5] for b in range(batch)])
        ABg = gpu(AB)
        if m == n:
            ipiv, info = bandlu.band_getrf_batched(ABg, kl, ku, variant="split")
        else:
            ipiv, info = bandlu.band_getrf_mn_batched(ABg, m, kl, ku)
        torch.cuda.synchronize()
        ABg, ipiv, info = ABg.cpu().numpy(), ipiv.cpu().numpy(), info.cpu().numpy()
        for b in range(5):
            ipo, info_o, _ = oracle.gbtrf_mn(base[b], m, kl, ku)
            assert np.all(ipiv[b::5] == ipo) and np.all(info[b::5] == info_o)
            for k in range(b, batch, 5):
                assert same(ABg[k], base[b])
