"""GPU parity of the tiled band Cholesky at its edges: tile and panel
remainders, rows per lane, the widest window, pivots that take the step by step
path (not positive, out of the plain root's range), signed zeros past a
panel's reach, infinities and NaN.  Bit for bit against the CPU oracle (every
entry takes the unblocked algorithm's operations in its order)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_22099_amd import bandlu  # noqa: E402
from test_gpu_structures import gpu, same  # noqa: E402


def lower(n, kd, seed, ldab=None):
    """Strictly dominant lower band; slots outside the matrix hold a marker
    that nothing may read or write."""
    rng = np.random.default_rng(seed)
    AB = np.full((n, ldab or kd + 1), 7e77)
    off = rng.standard_normal((n, kd + 1))
    row = np.zeros(n)
    for j in range(n):
        km = min(kd, n - 1 - j)
        AB[j, 1:1 + km] = off[j, 1:1 + km]
        row[j] += np.abs(off[j, 1:1 + km]).sum()
        row[j + 1:j + 1 + km] += np.abs(off[j, 1:1 + km])
    AB[:, 0] = row + 1.0
    return AB


def check(AB, kd, what):
    print(what, flush=True)
    ABg = gpu(AB)
    info_o = oracle.pbtrf(AB, kd)
    info = bandlu.band_pbtrf(ABg, kd)
    torch.cuda.synchronize()
    assert int(info.cpu()[0]) == info_o
    assert same(ABg.cpu().numpy(), AB)
    return info_o


@pytest.mark.parametrize("n,kd", [(1, 0), (2, 1), (15, 3), (16, 15), (17, 16), (33, 17), (40, 0),
                                  (100, 14), (100, 15), (100, 31), (160, 47), (161, 48), (175, 49),
                                  (200, 63), (200, 64), (250, 111), (250, 112), (251, 113),
                                  (300, 127), (300, 128), (300, 143), (320, 144), (321, 145), (330, 160),
                                  (100, 99), (161, 160)])
def test_edges(n, kd):
    assert check(lower(n, kd, 100 * n + kd, kd + 3), kd, f"pbtrf n={n} kd={kd}") == 0


@pytest.mark.parametrize("kd", [0, 5, 16, 40, 70, 130])
@pytest.mark.parametrize("at", [0, 1, 31, 32, 47, 150, 203])
def test_stops_at_the_first_failing_pivot(kd, at):
    AB = lower(204, kd, 3000 + kd)
    AB[at, 0] = -1.0 if at % 2 else np.nan
    assert check(AB, kd, f"pbtrf fails at {at}, kd={kd}") == at + 1


@pytest.mark.parametrize("kd", [3, 16, 33, 70, 130])
def test_specials(kd):
    n = 230
    rng = np.random.default_rng(4000 + kd)
    AB = lower(n, kd, 4000 + kd)
    inside = np.arange(n)[:, None] + np.arange(kd + 1) < n
    pick = rng.random(AB.shape) < 0.5
    pick[:, 0] = False
    AB[pick & inside] = -0.0
    check(AB.copy(), kd, f"signed zeros kd={kd}")
    for e in (-1040, -700, 600, 900):
        check(np.where(inside, np.ldexp(AB, e), AB), kd, f"scaled by 2^{e} kd={kd}")
    AB[100, min(2, kd)] = np.inf
    check(AB.copy(), kd, f"infinity kd={kd}")
    AB[20, 0] = np.inf
    check(AB, kd, f"infinite pivot kd={kd}")


def test_more_systems_than_one_launch_holds():
    """2^23 and a few systems of two rows: of that many workgroups of 512 threads
    one launch runs only the few, without an error."""
    batch = 2 ** 23 + 5
    rng = np.random.default_rng(5000)
    few = np.stack([lower(2, 1, 5000 + k) for k in range(97)])
    few[5, 1, 0] = -1.0
    pick = rng.integers(0, 97, batch)
    ABg = gpu(few)[torch.from_numpy(pick).to("cuda")].contiguous()
    print(f"pbtrf batch={batch}", flush=True)
    info = bandlu.band_pbtrf_batched(ABg, 1)
    torch.cuda.synchronize()
    info_o = np.array([oracle.pbtrf(few[k], 1) for k in range(97)])
    assert np.array_equal(info.cpu().numpy(), info_o[pick])
    assert same(ABg.cpu().numpy(), few[pick])


@pytest.mark.parametrize("n,kd,batch", [(1, 0, 3), (8, 7, 1), (9, 3, 512), (9, 3, 513), (12, 11, 1500),
                                        (16, 1, 1100), (16, 4, 1100), (17, 16, 1024), (20, 4, 600),
                                        (25, 4, 2048), (26, 4, 2048), (24, 12, 4096), (42, 4, 16384),
                                        (43, 4, 16384), (109, 0, 16384), (50, 49, 2048), (56, 49, 2048),
                                        (53, 52, 4096)])
def test_small_systems(n, kd, batch):
    """Both sides of the lines between the column kernel and the tiles: plain
    systems, signed zeros, an infinity, scaled ones, and failing pivots."""
    print(f"pbtrf n={n} kd={kd} batch={batch}", flush=True)
    few = np.stack([lower(n, kd, 6000 + k, kd + 2) for k in range(13)])
    inside = np.arange(n)[:, None] + np.arange(kd + 2) < n
    inside[:, kd + 1] = False
    pick = (np.random.default_rng(n).random((n, kd + 2)) < 0.5) & inside
    pick[:, 0] = False
    few[3, pick] = -0.0
    few[5] = np.where(inside, np.ldexp(few[5], -900), few[5])
    few[6, n - 1, 0] = -1.0
    few[7, n // 2, 0] = np.nan
    few[8, 0, 0] = 0.0
    few[9, n // 3, 0] = np.inf
    at = np.arange(batch) % 13
    ABg = gpu(few)[torch.from_numpy(at).to("cuda")].contiguous()
    info = bandlu.band_pbtrf_batched(ABg, kd)
    torch.cuda.synchronize()
    info_o = np.array([oracle.pbtrf(few[k], kd) for k in range(13)])
    assert np.array_equal(info.cpu().numpy(), info_o[at])
    ABg = ABg.cpu().numpy()
    for k in range(min(13, batch)):
        assert all(same(a, few[k]) for a in ABg[k::13])
