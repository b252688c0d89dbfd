"""The popcount search's map of (tile, chunk) items: workgroups of one, two, four
and eight tiles, slot counts that get an empty slot more (even) and that don't (odd,
or few workgroups), chunks of 64 to 256 rows, and windows about where the plan turns
from window scans to tiles, by the number of pairs (3M) and by the windows' share of
the union (1/13). Against the fp4 engine on every query and the oracle on a sample."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

import oracle  # noqa: E402

PEAKS = 8


def _map(n, nq):
    """slots, tiles of a slot, chunk rows (search_popc.hip)"""
    tiles, chunk, per = -(-nq // 256), 256, 8
    while chunk < 2048 and tiles * (n // chunk) > per << 21:
        chunk *= 2
    while chunk > 64 and tiles * -(-n // chunk) < 16384:
        chunk //= 2
    chunks = -(-n // chunk)
    while per > 1 and -(-tiles // per) * chunks < 8192:
        per //= 2
    slots = -(-tiles // per)
    return slots | 1 if slots * chunks >= 4096 else slots, per, chunk


@pytest.mark.parametrize("dim,n,nq,value,slots,per,chunk", [
    (512, 100_000, 4_096, 30.0, 9, 2, 64),
    (512, 40_003, 255, 500.0, 1, 1, 64),
    (512, 40_003, 1_000, 50.0, 4, 1, 64),
    (512, 140_000, 2_001, 500.0, 5, 2, 64),
    (1024, 270_001, 8_193, 0.5, 9, 4, 256),
    (512, 300_000, 15_001, 500.0, 9, 8, 256),
    (512, 280_000, 15_400, 0.383, 9, 8, 256),   # 195 rows: 3M pairs
    (512, 700_000, 100_096, 0.23, 49, 8, 256),  # 149 rows of a union of 1,940
    (512, 700_000, 100_096, 3.0, 49, 8, 256),
    (512, 700_000, 98_304, 150.0, 49, 8, 256),
])
def test_against_fp4(dim, n, nq, value, slots, per, chunk):
    import torch
    import paper_2211_16422_amd.hyperoms as h
    assert _map(n, nq) == (slots, per, chunk)
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
        idx, dist = ctx.search_window(hv, q_pmz, q_ch, h.TOL_DA, value, h.ENGINE_POPCOUNT)
        assert np.array_equal(idx[some].cpu().numpy(), o_idx)
        assert np.array_equal(dist[some].cpu().numpy(), o_dist)
        want = ctx.search_window(hv, q_pmz, q_ch, h.TOL_DA, value, h.ENGINE_MFMA_F4)
        assert torch.equal(idx, want[0]) and torch.equal(dist, want[1])
