"""One-shot search of so many queries and library rows that its (tile, chunk)
workgroups hold more than 2^32 threads (2,200,000 queries of 4,500,000 rows at
D = 512: 8,594 tiles x 2,198 chunks, most without candidates): the result of
every query equals that of a call of its part of the queries alone."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

DIM, N_LIB, N_Q, PEAKS = 512, 4_500_000, 2_200_000, 8


def test_more_threads_than_one_grid_holds():
    import torch
    import paper_2211_16422_amd.hyperoms as h
    assert -(-N_Q // 256) * (-(-N_LIB // 2048)) * 256 > 2**32  # popcount; the others twice that
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    with h.Context(h.Params(dim=DIM, charge_match=0)) as ctx:
        span = ctx.get_codebook()[0].shape[0] // PEAKS

        def csr(m):
            bins = torch.randint(0, span, (m, PEAKS), generator=g, device="cuda",
                                 dtype=torch.int32)
            bins += span * torch.arange(PEAKS, device="cuda", dtype=torch.int32)
            level = torch.randint(0, 16, (m * PEAKS,), generator=g, device="cuda",
                                  dtype=torch.uint8)
            return torch.arange(m + 1, device="cuda") * PEAKS, bins.reshape(-1), level

        def precursors(m):
            return 400.0 + 1000.0 * torch.rand(m, generator=g, device="cuda",
                                               dtype=torch.float64)

        zeros = torch.zeros(max(N_LIB, N_Q), dtype=torch.int8, device="cuda")
        ctx.encode_library(*csr(N_LIB), precursors(N_LIB), zeros[:N_LIB])
        hv, pmz, ch = ctx.encode_queries(*csr(N_Q)), precursors(N_Q), zeros[:N_Q]
        want = None
        for engine in (h.ENGINE_POPCOUNT, h.ENGINE_MFMA_I8, h.ENGINE_MFMA_F8, h.ENGINE_MFMA_F4):
            print(f"engine {engine}", flush=True)
            idx, dist = ctx.search_window(hv, pmz, ch, h.TOL_DA, 1.5, engine)
            torch.cuda.synchronize()
            if want is None:
                want = idx, dist
                assert int((idx >= 0).sum()) == N_Q
                for a in (0, 1_000_000, N_Q - 100_000):  # launches of one piece
                    part = slice(a, a + 100_000)
                    i, d = ctx.search_window(hv[part].contiguous(), pmz[part].contiguous(),
                                             ch[part].contiguous(), h.TOL_DA, 1.5, engine)
                    assert torch.equal(i, idx[part]) and torch.equal(d, dist[part]), a
            assert torch.equal(idx, want[0]) and torch.equal(dist, want[1]), engine
