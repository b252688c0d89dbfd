"""Offsets that descend: such a spectrum holds no peaks, and its row is all ones,
on the step-function path (calls of many spectra) as on the general one."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]


@pytest.mark.parametrize("dim,n", [(512, 49_153), (8192, 3_104), (8192, 100)])
def test_rows_are_all_ones(dim, n):
    import torch
    import paper_2211_16422_amd.hyperoms as h
    rng = np.random.default_rng(n)
    hp = h.Params(dim=dim)
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(rng.integers(2, 40, n))
    total = int(off[-1])
    down = np.unique(rng.integers(1, n, 64))
    off[down] += 60  # over the next offset or two, which are then lower
    off = np.minimum(off, total)
    falls = np.flatnonzero(np.diff(off) < 0)
    assert len(falls) >= 20
    bins = rng.integers(0, h.num_bins(hp), total).astype(np.int32)
    levels = rng.integers(0, hp.n_levels, total).astype(np.uint8)
    csr = h.to_device_csr(off, bins, levels, "cuda:0")
    with h.Context(hp) as ctx, h.Context(hp) as general:
        general.set_codebook(*general.get_codebook())
        # a row that is not written keeps the fill
        fill = torch.full((n, dim // 32), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
        got = ctx.encode_queries(*csr, out=fill.clone()).cpu().numpy()
        want = general.encode_queries(*csr, out=fill.clone()).cpu().numpy()
    assert (got[falls] == -1).all()
    assert np.array_equal(got, want)
