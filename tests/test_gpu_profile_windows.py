"""search_ms of the profile covers the scans of narrow windows, which the result
kernel of the search makes."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

PEAKS = 8


@pytest.mark.parametrize("engine", ["ENGINE_POPCOUNT", "ENGINE_MFMA_F8", "ENGINE_MFMA_F4"])
def test_search_time_covers_the_window_scans(engine):
    """6,000 windows of about 1,000 rows at D = 4096: 3 GB read by the scans,
    against the sort of 6,000 queries and the empty tiles of the search kernel"""
    import torch
    import paper_2211_16422_amd.hyperoms as h
    n, nq, value = 400_000, 6_000, 0.75  # +- value Da
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    with h.Context(h.Params(dim=4096)) as ctx:
        bins = ctx.get_codebook()[0].shape[0]

        def csr(m):
            return (torch.arange(m + 1, device="cuda") * PEAKS,
                    torch.randint(0, bins, (m, PEAKS), generator=g, device="cuda",
                                  dtype=torch.int32).sort(dim=1)[0].reshape(-1),
                    torch.randint(0, 16, (m * PEAKS,), generator=g, device="cuda",
                                  dtype=torch.uint8))

        def spectra(m):
            return (400.0 + 600.0 * torch.rand(m, generator=g, device="cuda",
                                               dtype=torch.float64),
                    torch.full((m,), 2, device="cuda", dtype=torch.int8))

        ctx.encode_library(*csr(n), *spectra(n))
        hv, (pmz, ch) = ctx.encode_queries(*csr(nq)), spectra(nq)
        lo, hi = ctx.window_bounds(pmz, ch, h.TOL_DA, value)
        assert 500 < float((hi - lo).double().mean()) < 2000
        args = (hv, pmz, ch, h.TOL_DA, value, getattr(h, engine))
        ctx.search_window(*args)
        ctx.profile_enable(True)
        ctx.profile_read()
        for _ in range(10):
            ctx.search_window(*args)
        p = ctx.profile_read()
        ctx.profile_enable(False)
        assert p["search_launches"] == 10
        assert p["search_ms"] > 2 * p["prep_ms"], p
