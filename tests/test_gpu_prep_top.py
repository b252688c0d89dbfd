"""Device preprocessing of spectra at the wave kernel's edges (0 to 257 raw
peaks, one to four per lane; top_n from 1 to 65) against the oracle: identical
offsets, bins and levels with intensities that tie at the top-N boundary (and
there by m/z, then position), equal, zero and widely spread intensities, peaks
sharing bins, and peaks at and beyond the range's ends."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

import oracle  # noqa: E402


def _spectra(rng):
    mz, inten = [], []
    for n in list(range(0, 6)) + [49, 50, 51, 63, 64, 65, 66, 127, 128, 129, 191, 192, 193, 255,
                                  256, 257] * 6:
        kind = rng.integers(0, 6)
        m = rng.uniform(95.0, 1510.0, n)
        if kind == 0:  # few distinct intensities
            v = rng.choice([0.25, 1.0, 2.0, 3.0], n)
        elif kind == 1:  # all equal
            v = np.full(n, 7.0)
        elif kind == 2:  # zeros (of both signs) among them
            v = rng.choice([0.0, -0.0, 1.0], n)
        elif kind == 3:  # many orders of magnitude
            v = np.exp(rng.uniform(-300, 300, n))
        else:
            v = rng.lognormal(0.0, 1.0, n)
        if kind in (0, 1, 4) and n > 4:  # shared bins and equal m/z
            m[rng.integers(0, n, n // 2)] = rng.choice(m[: 1 + n // 8], n // 2)
            m[rng.integers(0, n, n // 8)] += 1e-3
        if n > 8:
            m[rng.integers(0, n, 4)] = [101.0, 1500.0, np.nextafter(101.0, 0), 1499.9999999]
        mz.append(m)
        inten.append(v)
    off = np.zeros(len(mz) + 1, np.int64)
    off[1:] = np.cumsum([len(m) for m in mz])
    return off, np.concatenate(mz), np.concatenate(inten)


@pytest.mark.parametrize("top_n", [1, 2, 7, 50, 63, 64, 65])
@pytest.mark.parametrize("noise", [0.0, 0.01, 1.0])
def test_matches_the_oracle(top_n, noise):
    import torch
    import paper_2211_16422_amd.hyperoms as h
    off, mz, inten = _spectra(np.random.default_rng(top_n * 10 + int(noise * 100)))
    hp = h.Params(dim=512, top_n=top_n, noise_frac=noise)
    op = oracle.Params(dim=512, top_n=top_n, noise_frac=noise)
    w_off, w_bin, w_lv = oracle.preprocess(off, mz, inten, op)
    with h.Context(hp) as ctx:
        o, b, lv = ctx.preprocess_device(*[torch.from_numpy(x).to("cuda:0")
                                           for x in (off, mz, inten)])
        assert np.array_equal(o.cpu().numpy(), w_off)
        assert np.array_equal(b.cpu().numpy(), w_bin)
        assert np.array_equal(lv.cpu().numpy(), w_lv)
