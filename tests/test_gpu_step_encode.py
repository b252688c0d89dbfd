"""The step-function encoding (generated ID_LEVEL tables, calls of many
spectra) against the general path, which a context takes after its own tables
were set as the caller's, and against the oracle on a sample: every bit, for
spectra of 0 to 63 peaks and beyond (the general path's size classes in the
same call), in any peak order, with repeated bins and out-of-range peaks."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

import oracle  # noqa: E402


def _spectra(n, f, q, rng):
    sizes = rng.integers(0, 64, n)
    sizes[rng.integers(0, n, 5)] = [63, 64, 65, 255, 300]
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(sizes)
    total = int(off[-1])
    bins = rng.integers(0, f, total).astype(np.int32)
    levels = rng.integers(0, q, total).astype(np.uint8)
    for s in range(0, n, 2):  # half of the spectra in ascending order, as preprocessing leaves them
        bins[off[s]:off[s + 1]].sort()
    edge = rng.integers(0, total, 50)
    bins[edge] = rng.choice([0, f - 1], 50)
    return off, bins, levels


@pytest.mark.parametrize("dim,n,q,flips,seed,bins_per_da", [
    (512, 49_153, 16, 0, 1, 20.0),
    (2048, 12_289, 16, 0, 2, 20.0),
    (8192, 3_103, 16, 0, 3, 20.0),
    (8192, 3_104, 5, 8191, 4, 0.01),
    (1536, 16_500, 2, 1, 5, 25.0),
    (16384, 1_601, 9, 0, 6, 20.0),
    (32768, 801, 16, 4001, 7, 20.0),
])
def test_every_bit(dim, n, q, flips, seed, bins_per_da):
    import paper_2211_16422_amd.hyperoms as h
    rng = np.random.default_rng(seed)
    hp = h.Params(dim=dim, n_levels=q, id_flips=flips, seed=seed, bins_per_da=bins_per_da)
    op = oracle.Params(dim=dim, n_levels=q, id_flips=flips, seed=seed, bins_per_da=bins_per_da)
    f = h.num_bins(hp)
    off, bins, levels = _spectra(n, f, q, rng)
    with h.Context(hp) as ctx, h.Context(hp) as general:
        general.set_codebook(*general.get_codebook())
        csr = h.to_device_csr(off, bins, levels, "cuda:0")
        got = ctx.encode_queries(*csr).cpu().numpy().view(np.uint32)
        want = general.encode_queries(*csr).cpu().numpy().view(np.uint32)
        assert np.array_equal(got, want)
        assert ctx.device_errors() == 0
        idt, lvt = ctx.get_codebook()
        m = 200
        assert np.array_equal(got[:m], oracle.encode(op, idt, lvt, off[:m + 1], bins[:off[m]],
                                                     levels[:off[m]]))
        # peaks out of range are left out and flagged, as by the general path
        bad = rng.integers(0, off[-1], 40)
        bins[bad[:20]] = rng.choice([-1, f, 2 ** 30], 20)
        levels[bad[20:]] = q
        csr = h.to_device_csr(off, bins, levels, "cuda:0")
        assert np.array_equal(ctx.encode_queries(*csr).cpu().numpy(),
                              general.encode_queries(*csr).cpu().numpy())
        assert ctx.device_errors() == 1 and general.device_errors() == 1
