"""One-shot searches of so many queries and library rows that their workgroups hold
2^32 threads and more, in pieces: 2,200,000 queries of 4,500,000 rows at D = 512 on the
matrix cores (8,594 tiles x 2,198 chunks, a workgroup each for open windows), 16,000,000
by popcount (62,500 tiles, eight a workgroup). Against the popcount engine, whose launch
is a single one there, and the fp4 engine with a listed grid; and a call of a part of
the queries."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

DIM, N_LIB, PEAKS = 512, 4_500_000, 8


@pytest.mark.parametrize("n_q,value,one,pieces", [
    (2_200_000, 60.0, "ENGINE_POPCOUNT", ["ENGINE_MFMA_I8", "ENGINE_MFMA_F8", "ENGINE_MFMA_F4"]),
    (16_000_000, 0.02, "ENGINE_MFMA_F4", ["ENGINE_POPCOUNT"]),
])
def test_more_threads_than_one_grid_holds(n_q, value, one, pieces):
    import torch
    import paper_2211_16422_amd.hyperoms as h
    items, threads = -(-n_q // 256) * -(-N_LIB // 2048), 512
    if one != "ENGINE_POPCOUNT":
        items, threads = (-(-n_q // 2048) | 1) * -(-N_LIB // 2048), 256
    assert items * threads > 2**32
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

        zeros = torch.zeros(max(N_LIB, n_q), dtype=torch.int8, device="cuda")
        ctx.encode_library(*csr(N_LIB), precursors(N_LIB), zeros[:N_LIB])
        hv, pmz, ch = ctx.encode_queries(*csr(n_q)), precursors(n_q), zeros[:n_q]
        want = ctx.search_window(hv, pmz, ch, h.TOL_DA, value, getattr(h, one))
        assert int((want[0] >= 0).sum()) > 0.99 * n_q
        for engine in pieces:
            print(engine, flush=True)
            idx, dist = ctx.search_window(hv, pmz, ch, h.TOL_DA, value, getattr(h, engine))
            torch.cuda.synchronize()
            assert torch.equal(idx, want[0]) and torch.equal(dist, want[1]), engine
        for a in (0, n_q // 2, n_q - 50_000):
            part = slice(a, a + 50_000)
            i, d = ctx.search_window(hv[part].contiguous(), pmz[part].contiguous(),
                                     ch[part].contiguous(), h.TOL_DA, value, getattr(h, one))
            assert torch.equal(i, want[0][part]) and torch.equal(d, want[1][part]), a
