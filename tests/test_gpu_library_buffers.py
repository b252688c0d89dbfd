"""Libraries of several sizes one after the other in one context: a new library
may take the buffers of the last one, whose rows then stand behind its own (where
the tiles read past a library's end). Every search is compared with a context
that has encoded that library only. And the memory that a context keeps."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

PEAKS = 12


def _device_csr(h, ctx, n, g, n_peaks=PEAKS):
    import torch
    span = ctx.get_codebook()[0].shape[0] // n_peaks
    bins = torch.randint(0, span, (n, n_peaks), generator=g, device="cuda", dtype=torch.int32)
    bins += span * torch.arange(n_peaks, device="cuda", dtype=torch.int32)
    return (torch.arange(n + 1, device="cuda") * n_peaks, bins.reshape(-1),
            torch.randint(0, 16, (n * n_peaks,), generator=g, device="cuda", dtype=torch.uint8))


def _spectra(n, g):
    import torch
    return (500.0 + 300.0 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64),
            torch.randint(2, 4, (n,), generator=g, device="cuda", dtype=torch.int8))


def _searches(h, ctx, hv, pmz, ch):
    """all routes: open and narrow windows, hundreds and a few queries, batched"""
    import torch
    out = []
    for engine in (h.ENGINE_POPCOUNT, h.ENGINE_MFMA_I8, h.ENGINE_MFMA_F8, h.ENGINE_MFMA_F4):
        for nq in (hv.shape[0], 40, 1):
            for value in (500.0, 2.0):
                out += ctx.search_window(hv[:nq], pmz[:nq], ch[:nq], h.TOL_DA, value, engine)
    kinds = torch.zeros(hv.shape[0], dtype=torch.int8, device="cuda")
    values = torch.full((hv.shape[0],), 500.0, dtype=torch.float64, device="cuda")
    values[::3] = 2.0
    for engine in (h.ENGINE_POPCOUNT, h.ENGINE_MFMA_F8, h.ENGINE_MFMA_F4):
        ctx.set_batched_config(engine=engine)
        out += ctx.search_batched(hv, pmz, ch, kinds, values, use_graph=False)
    out.append(ctx.library_export())
    out.append(ctx.library_order())
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("sizes", [
    (5000, 4001, 4999, 4100, 5000),  # into buffers with up to a quarter to spare
    (5000, 1200, 1199, 5000),        # more than four times smaller, then larger
    (300, 257, 256, 255, 1, 300),    # edges of tiles; a library of one row
    (2000, 0, 1700),
])
def test_a_library_after_others(sizes):
    import torch
    import paper_2211_16422_amd.hyperoms as h
    hp = h.Params(dim=1024)
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(sizes))
    with h.Context(hp) as ctx:
        hv = ctx.encode_queries(*_device_csr(h, ctx, 600, g))
        pmz, ch = _spectra(600, g)
        for n in sizes:
            lib = (*_device_csr(h, ctx, n, g), *_spectra(n, g))
            ctx.encode_library(*lib)
            assert ctx.library_size() == n
            if n == 0:
                continue
            got = _searches(h, ctx, hv, pmz, ch)
            with h.Context(hp) as fresh:
                fresh.encode_library(*lib)
                want = _searches(h, fresh, hv, pmz, ch)
            for i, (a, b) in enumerate(zip(got, want)):
                assert np.array_equal(a, b), (n, i)


def test_memory_that_a_context_keeps():
    """Held behind a library of n rows: those rows, 21 bytes more for each and at
    most a quarter of both, and a workspace of 80 MiB; not the scratch of a large
    sort (20 bytes a row), nor a larger library that went before."""
    import torch
    import paper_2211_16422_amd.hyperoms as h
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    large, small, slack = 6_000_000, 2_000_000, 16 << 20

    def held():
        torch.cuda.synchronize()
        return -torch.cuda.mem_get_info()[0]

    with h.Context(h.Params(dim=512)) as ctx:
        one = _device_csr(h, ctx, large, g, 1)
        pmz, ch = _spectra(large, g)
        ctx.encode_library(one[0][:11], one[1][:10], one[2][:10], pmz[:10], ch[:10])
        start = held()
        ctx.encode_library(*one, pmz, ch)
        assert held() - start <= large * (64 + 21) + slack
        ctx.encode_library(one[0][:small + 1], one[1][:small], one[2][:small], pmz[:small],
                           ch[:small])
        assert held() - start <= small * (64 + 21) * 5 // 4 + (80 << 20)
        ctx.encode_library(one[0][:1], one[1][:0], one[2][:0], pmz[:0], ch[:0])
        assert held() - start <= 80 << 20
