"""Encoding calls of up to 1,024 spectra (a workgroup per spectrum, its lane
groups sharing the peaks) against the oracle, bit for bit: 64 lane groups to
one per workgroup, shares of no peak to many, every size class, peaks out of
range."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

import oracle  # noqa: E402

SIZES = [0, 1, 2, 7, 8, 9, 20, 63, 64, 65, 168, 169, 255, 256, 300]


@pytest.mark.parametrize("dim", [512, 1536, 2048, 8192, 16384, 32768])
@pytest.mark.parametrize("n", [1, 15, 1024])
def test_few_spectra(dim, n):
    import paper_2211_16422_amd.hyperoms as h
    rng = np.random.default_rng(dim + n)
    hp, op = h.Params(dim=dim), oracle.Params(dim=dim)
    f = h.num_bins(hp)
    sizes = np.array(SIZES)[(np.arange(n) + (11 if n == 1 else 0)) % len(SIZES)]
    if n == 1024:
        sizes[64:] = sizes[64:] % 50  # the oracle's time
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(sizes)
    bins = rng.integers(0, f, int(off[-1])).astype(np.int32)
    levels = rng.integers(0, 16, int(off[-1])).astype(np.uint8)
    with h.Context(hp) as ctx:
        got = ctx.encode_queries(*h.to_device_csr(off, bins, levels, "cuda:0"))
        got = got.cpu().numpy().view(np.uint32)
        idt, lvt = ctx.get_codebook()
        assert np.array_equal(got, oracle.encode(op, idt, lvt, off, bins, levels))
        assert ctx.device_errors() == 0
        # peaks out of range are left out and flagged
        bad = rng.integers(0, off[-1], max(1, n // 4))
        b2, l2 = bins.copy(), levels.copy()
        b2[bad[::2]] = f
        b2[bad[1::4]] = -1
        l2[bad[3::4]] = 16
        got = ctx.encode_queries(*h.to_device_csr(off, b2, l2, "cuda:0"))
        got = got.cpu().numpy().view(np.uint32)
        keep = (b2 >= 0) & (b2 < f) & (l2 < 16)
        o2 = np.concatenate([[0], np.cumsum(keep)])[off]
        assert np.array_equal(got, oracle.encode(op, idt, lvt, o2.astype(np.int64), b2[keep],
                                                 l2[keep]))
        assert ctx.device_errors() != 0
