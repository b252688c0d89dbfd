"""One-shot search of thousands of queries against hundreds of thousands of rows,
where a tile of 256 queries meets chunks of several 256-row blocks in patches of
8 x 4: with a workgroup for each (tile, chunk) item (open windows), and with
grids of 4,096 and of 1,024 workgroups that list theirs (windows of up to 50 Da,
many and few items), with and without a patch more per group of tiles. All engines against
each other on every query, and against the oracle on a sample."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

import oracle  # noqa: E402

PEAKS = 8


def _ceil(a, b):
    return -(-a // b)


def _matrix_map(dim, n, nq):
    """chunk rows, chunks of a patch, whether a patch is added, items (search_mfma.hip)"""
    tiles, chunk = _ceil(nq, 256), 2048
    while chunk > max(256, 16384 * 32 // dim) and tiles * _ceil(n, chunk) < 24576:
        chunk //= 2
    chunks = _ceil(n, chunk)
    per = 4 if tiles * chunks >= 2048 else 1
    groups, patches, step = _ceil(tiles, 8), _ceil(chunks, per), chunks / per / (tiles / 8)
    turn = (patches + step) % 2.0
    padded = step < 4 and not 0.2 <= turn <= 1.8
    return chunk, per, padded, _ceil(groups * (patches + padded), 8) * 8 * 8 * per


@pytest.mark.parametrize("dim,n,nq,value,chunk,grid,padded", [
    (512, 300_000, 20_000, 500.0, 1024, None, False),
    (1536, 320_000, 20_000, 500.0, 1024, None, False),
    (512, 400_000, 100_000, 3.0, 2048, 4096, True),
    (512, 400_000, 100_000, 0.05, 2048, 1024, True),
    (512, 900_000, 70_000, 2.0, 2048, 4096, False),
    (1536, 120_000, 9_000, 20.0, 256, 1024, False),
    (1536, 120_000, 9_000, 60.0, 256, None, False),
])
def test_engines_agree(dim, n, nq, value, chunk, grid, padded):
    import torch
    import paper_2211_16422_amd.hyperoms as h
    got = _matrix_map(dim, n, nq)
    many = got[3] > (32768 if value > 1 else 65536) and value > 0.1
    listed = None if value > 50 else 4096 if many else 1024
    assert got[:3] == (chunk, 4, padded) and grid == listed and (not grid or got[3] > grid)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + nq)
    with h.Context(h.Params(dim=dim)) as ctx:
        span = ctx.get_codebook()[0].shape[0] // PEAKS

        def csr(m):
            bins = torch.randint(0, span, (m, PEAKS), generator=g, device="cuda",
                                 dtype=torch.int32)
            bins += span * torch.arange(PEAKS, device="cuda", dtype=torch.int32)
            level = torch.randint(0, 16, (m * PEAKS,), generator=g, device="cuda",
                                  dtype=torch.uint8)
            return torch.arange(m + 1, device="cuda") * PEAKS, bins.reshape(-1), level

        def spectra(m):
            return (400.0 + 1100.0 * torch.rand(m, generator=g, device="cuda",
                                                dtype=torch.float64),
                    torch.randint(2, 4, (m,), generator=g, device="cuda", dtype=torch.int8))

        pmz, ch = spectra(n)
        ctx.encode_library(*csr(n), pmz, ch)
        hv, (q_pmz, q_ch) = ctx.encode_queries(*csr(nq)), spectra(nq)
        some = torch.randperm(nq, generator=g, device="cuda")[:24]
        o_idx, o_dist = oracle.search(
            oracle.Params(dim=dim), ctx.library_export().cpu().numpy().view(np.uint32),
            pmz.cpu().numpy(), ch.cpu().numpy(), hv[some].cpu().numpy().view(np.uint32),
            q_pmz[some].cpu().numpy(), q_ch[some].cpu().numpy(), h.TOL_DA, value)
        want = None
        for engine in (h.ENGINE_POPCOUNT, h.ENGINE_MFMA_I8, h.ENGINE_MFMA_F8, h.ENGINE_MFMA_F4):
            idx, dist = ctx.search_window(hv, q_pmz, q_ch, h.TOL_DA, value, engine)
            assert np.array_equal(idx[some].cpu().numpy(), o_idx), engine
            assert np.array_equal(dist[some].cpu().numpy(), o_dist), engine
            if want is None:
                want = idx, dist
            assert torch.equal(idx, want[0]) and torch.equal(dist, want[1]), engine
