"""The panel kernel behind BLOCKED (getrf_blocked.hip) for kl <= 31: that a
caller who names the variant gets it, and that the default takes it where the
pivot-wavefront kernel's registers end (kl = 0, 2kl+ku+1 > 448).  Which kernels
a call launches is read from its captured graph (never launched): a fill kernel
and one launch per panel of 32 columns, against one launch in all.  Factors bit
for bit against the CPU oracle."""
import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_22099_amd import bandlu  # noqa: E402
from test_gpu_parity import special_band  # noqa: E402
from test_gpu_structures import gpu, same  # noqa: E402


def launches(n, kl, ku, variant=None):
    """Nodes of the graph that band_getrf records on a capturing stream."""
    hip = bandlu._lib
    vp = ctypes.c_void_p
    AB = torch.zeros((n, 2 * kl + ku + 1), dtype=torch.float64, device="cuda")
    ipiv = torch.zeros(n, dtype=torch.int32, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    graph, count = vp(), ctypes.c_size_t()
    with torch.cuda.stream(s):
        assert hip.hipStreamBeginCapture(vp(s.cuda_stream), 1) == 0  # thread-local mode
        try:
            bandlu.band_getrf(AB, kl, ku, ipiv, info, variant=variant)
        finally:
            assert hip.hipStreamEndCapture(vp(s.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return count.value


@pytest.mark.parametrize("n,kl,ku", [(95, 20, 52), (300, 31, 90), (97, 12, 80), (200, 5, 120)])
def test_named_variant_runs_the_panel_kernel(n, kl, ku):
    print(f"blocked n={n} kl={kl} ku={ku}", flush=True)
    assert launches(n, kl, ku, "blocked") > (n + 31) // 32
    assert launches(n, kl, ku) == 1


# windows of 449 and more columns, kl = 0 (no window limit), panel remainders
@pytest.mark.parametrize("n,kl,ku", [(500, 31, 386), (480, 16, 416), (610, 1, 446), (700, 30, 500),
                                     (451, 5, 450), (300, 0, 140), (200, 0, 199), (513, 0, 511)])
def test_default_beyond_the_registers(n, kl, ku):
    assert bandlu.band_getrf_variant(n, kl, ku) == "blocked"
    assert launches(n, kl, ku) > (n + 31) // 32
    for k, (nz, nans, zc) in enumerate([(0.0, 0, ()), (0.3, 0, ()), (0.1, 2, ()),
                                        (0.2, 0, (n // 3, n // 3 + 1))]):
        print(f"default blocked n={n} kl={kl} ku={ku} case {k}", flush=True)
        T = special_band(n, kl, ku, 9100 + n + k, neg_zero=nz, nans=nans, zero_cols=zc)
        AB, _ = oracle.dense_to_band(T, kl, ku)
        ABg = gpu(AB)
        ipo, info_o, _ = oracle.gbtrf(AB, kl, ku)
        ipiv, info = bandlu.band_getrf(ABg, kl, ku)
        torch.cuda.synchronize()
        assert np.array_equal(ipiv.cpu().numpy(), ipo) and int(info.cpu()[0]) == info_o
        assert same(ABg.cpu().numpy(), AB)
