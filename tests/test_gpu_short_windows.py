"""Calls of short windows (up to 1,000 ppm or 1 Da) of thousands of queries:
the tile kernel's workgroups list their items with candidates, which are few
beside the items of the whole library. A crowded stretch of precursors, whose
tiles are worth multiplying, beside a sparse one, whose windows are scanned."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

import oracle  # noqa: E402

DIM = 512


@pytest.mark.parametrize("kind,value", [(1, 1000.0), (0, 1.0), (1, 20.0)])
@pytest.mark.parametrize("n,nq", [(60_001, 4097), (150_000, 9000)])
def test_short_windows_match(n, nq, kind, value):
    import torch
    import paper_2211_16422_amd.hyperoms as h
    rng = np.random.default_rng(n)

    def precursors(m):
        return np.where(rng.random(m) < 0.7, rng.uniform(500.0, 502.0, m),
                        rng.uniform(600.0, 1400.0, m))

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")

    hp = h.Params(dim=DIM)
    with h.Context(hp) as ctx:
        span = ctx.get_codebook()[0].shape[0] // 8

        def csr(m):
            bins = rng.integers(0, span, (m, 8)) + span * np.arange(8)
            return h.to_device_csr(np.arange(m + 1, dtype=np.int64) * 8,
                                   bins.reshape(-1).astype(np.int32),
                                   rng.integers(0, 16, 8 * m).astype(np.uint8), "cuda:0")

        pmz, ch = precursors(n), rng.choice(np.array([2, 3], np.int8), size=n)
        q_pmz, q_ch = precursors(nq), rng.choice(np.array([2, 3], np.int8), size=nq)
        ctx.encode_library(*csr(n), dev(pmz), dev(ch))
        q_hv = ctx.encode_queries(*csr(nq))
        want = None
        some = rng.permutation(nq)[:48]
        lib = ctx.library_export()
        o_lib = lib.cpu().numpy().view(np.uint32)
        o_idx, o_dist = oracle.search(oracle.Params(dim=DIM), o_lib, pmz, ch,
                                      q_hv.cpu().numpy().view(np.uint32)[some], q_pmz[some],
                                      q_ch[some], kind, value)
        for engine in (h.ENGINE_POPCOUNT, h.ENGINE_MFMA_I8, h.ENGINE_MFMA_F8, h.ENGINE_MFMA_F4):
            idx, dist = ctx.search_window(q_hv, dev(q_pmz), dev(q_ch), kind, value, engine)
            idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
            assert np.array_equal(idx[some], o_idx) and np.array_equal(dist[some], o_dist), engine
            if want is None:
                want = idx, dist
            assert np.array_equal(idx, want[0]) and np.array_equal(dist, want[1]), engine
