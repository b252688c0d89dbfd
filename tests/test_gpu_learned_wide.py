"""Learned shortlist search over windows of 150,000 candidates.

There the sampled threshold is one of the largest few sample scores (rank 128
or less), which the search selects from a short list; with every score equal
the list overflows and the general selection takes over."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# as for the other shortlists: how far a kept score may lie below the k-th of
# the 64-bit scores (the matrix unit's sums of E4M3 products are not exact to
# fp32: a kept score was seen 1.1e-5 below)
SCORE_TOL = 1e-2

D, H, E, N, NQ, K = 2048, 256, 64, 150_000, 40, 64


def _setup(flat):
    import torch
    import paper_2211_16422_amd.hyperoms as h
    rng = np.random.default_rng(11)
    ctx = h.Context(h.Params(dim=D))
    def csr(n):
        off = np.arange(n + 1, dtype=np.int64) * 12
        span = ctx.get_codebook()[0].shape[0] // 12
        bins = rng.integers(0, span, (n, 12)) + span * np.arange(12)  # ascending, distinct
        lev = rng.integers(0, ctx.params.n_levels, (n, 12))
        return h.to_device_csr(off, bins.reshape(-1).astype(np.int32),
                               lev.reshape(-1).astype(np.uint8), "cuda:0")

    dev = lambda a: torch.from_numpy(a).to("cuda:0")
    pmz = rng.uniform(600.0, 900.0, N)
    ctx.encode_library(*csr(N), dev(pmz), dev(np.full(N, 2, np.int8)))
    q_hv = ctx.encode_queries(*csr(NQ))
    w = {"W1": rng.normal(0, D ** -0.5, (H, D)), "b1": np.zeros(H),
         "W2": rng.normal(0, H ** -0.5, (E, H)), "b2": rng.normal(0, 0.1, E)}
    if flat:
        w = {k: np.zeros_like(v) for k, v in w.items()}
        w["b2"] = np.ones(E)
    m = h.Model(ctx, {k: v.astype(np.float32) for k, v in w.items()})
    m.embed_library()
    return ctx, m, q_hv, dev(np.full(NQ, 750.0)), dev(np.full(NQ, 2, np.int8))


@pytest.mark.parametrize("flat", [False, True])
def test_thresholds_of_wide_windows(flat):
    import torch
    from oracle import mlp
    ctx, m, q_hv, pmz, ch = _setup(flat)
    try:
        idx, dist, fb, sl = m.search(q_hv, pmz, ch, K, value=500.0, shortlist=True)
        e_idx, e_dist = ctx.search_window(q_hv, pmz, ch)
        torch.cuda.synchronize()
        if flat:  # every candidate ties: the buffers overflow, the answer is exhaustive
            assert (fb == 1).all()
            assert torch.equal(idx, e_idx) and torch.equal(dist, e_dist)
            return
        assert (fb == 0).all()
        # scores of the E4M3 embeddings that the search itself uses, in 64 bits
        bf = m.library_embeddings()[1].cpu().numpy().astype(np.uint16).astype(np.uint32) << 16
        lib = np.empty((N, E))
        lib[ctx.library_order().cpu().numpy().astype(np.int64)] = bf.view(np.float32)
        eq = mlp.round_e4m3(16.0 * m.embed(q_hv).cpu().numpy().astype(np.float64)) / 16.0
        score = eq @ lib.T
        sl = sl.cpu().numpy()
        for i in range(NQ):
            assert np.unique(sl[i]).size == K and sl[i].min() >= 0
            kth = np.partition(score[i], N - K)[N - K]
            assert score[i][sl[i]].min() >= kth - SCORE_TOL
    finally:
        m.close()
        ctx.close()
