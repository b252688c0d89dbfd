"""Performance cases: what programs built on this library have it do, over the
range of sizes they do it at.

Inputs are synthetic spectra with the shapes of the repository's generator
(``synth/spectra.py``: precursor m/z, charge and peak distributions, one decoy
per reference, jittered, thinned, noisy and half mass-shifted queries), drawn
on the GPU from the seed alone. ``n_ref`` is the number of references; the
library holds as many decoys again. Every search case starts from the
queries' spectrum vectors on the device and encodes them, as a search program
does for each file of spectra.

Kinds:

* ``search``: encode the queries, open or standard window search;
* ``batched``: the same with a window per query, replayed as a graph;
* ``cascade``: standard search, FDR, open search of the rest, FDR;
* ``learned``: shortlist search with a trained-size embedding;
* ``ingest``: raw peaks to an encoded, sorted library, and its rows;
* ``embed``: embeddings of packed rows (the larger part of making a learned
  library);
* ``train``: training steps of the embedding, then the weights (a checkpoint).
"""
import math

import numpy as np
import torch

import paper_2211_16422_amd.hyperoms as h

ENGINES = {"popcount": h.ENGINE_POPCOUNT, "int8": h.ENGINE_MFMA_I8, "fp8": h.ENGINE_MFMA_F8,
           "fp4": h.ENGINE_MFMA_F4}
MZ = (101.0, 1500.0)     # fragment m/z range
PMZ = (400.0, 1500.0)    # precursor m/z range of the references
RAW_PEAKS = 85.0         # mean raw peaks of a library spectrum (20..150)
KEPT_PEAKS = 46.3        # mean peaks it keeps after preprocessing


def listed():
    return [
        # a handful of spectra against a small library, as a test or a viewer
        # asks for: launches and latency
        {"name": "search_tiny", "kind": "search", "n_ref": 2000, "nq": 37, "dim": 2048,
         "engine": "fp4", "ppm": False, "tol": 500.0},
        # an instrument's spectra as they come, against a real library
        {"name": "search_online", "kind": "search", "n_ref": 200_000, "nq": 64, "dim": 8192,
         "engine": "fp4", "ppm": False, "tol": 500.0},
        # a short file with the default engine
        {"name": "search_popcount", "kind": "search", "n_ref": 100_000, "nq": 2001, "dim": 8192,
         "engine": "popcount", "ppm": False, "tol": 500.0},
        # one file of spectra, open search
        {"name": "search_file", "kind": "search", "n_ref": 300_001, "nq": 16_003, "dim": 8192,
         "engine": "fp4", "ppm": False, "tol": 500.0},
        # the large workload: 2M library spectra, 100,000 queries, open search
        {"name": "search_large", "kind": "search", "n_ref": 1_000_000, "nq": 100_000,
         "dim": 8192, "engine": "fp4", "ppm": False, "tol": 500.0},
        # standard search of a file: +-20 ppm windows of a few dozen candidates
        {"name": "search_standard", "kind": "search", "n_ref": 500_000, "nq": 20_001,
         "dim": 8192, "engine": "fp4", "ppm": True, "tol": 20.0},
        # a mixed stream: 70% standard, 30% open windows, charges 2 to 4
        {"name": "batched_mixed", "kind": "batched", "n_ref": 500_000, "nq": 50_000,
         "dim": 8192, "narrow": 0.7},
        # a file searched as a cascade at 1% FDR
        {"name": "cascade_file", "kind": "cascade", "n_ref": 300_000, "nq": 15_999,
         "dim": 8192, "engine": "fp4"},
        # a library built from its raw peaks
        {"name": "ingest_library", "kind": "ingest", "n": 400_001, "dim": 8192},
        # shortlist search of a file against a large library
        {"name": "learned_search", "kind": "learned", "n_ref": 500_000, "nq": 30_000,
         "dim": 8192, "hidden": 1024, "embed": 256, "k": 64},
        # embeddings of a library's rows
        {"name": "embed_rows", "kind": "embed", "n": 50_001, "dim": 8192, "hidden": 1024,
         "embed": 256},
        # training steps at the default batch, and the weights after them
        {"name": "train_steps", "kind": "train", "batch": 1024, "steps": 32, "dim": 8192,
         "hidden": 1024, "embed": 256},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "search", "standard", "batched", "cascade",
                       "ingest", "learned", "embed", "train"])
    dim = rng.choice([2048, 8192, 8192, 8192, 16384, 1536])
    if kind in ("search", "standard"):
        n_ref, nq = _log(rng, 1000, 1_000_000), _log(rng, 1, 100_000)
        engine = rng.choice(["fp4", "fp4", "fp4", "popcount", "fp8", "int8"])
        ppm = kind == "standard"
        tol = rng.choice([10.0, 20.0, 50.0]) if ppm else rng.choice([250.0, 500.0])
        cost = {"fp4": 1, "popcount": 6, "fp8": 2, "int8": 2}[engine]
        while not ppm and float(n_ref) * nq * dim * cost > 0.5e11 * 8192:
            nq = max(1, nq // 2)
        return {"kind": "search", "n_ref": n_ref, "nq": nq, "dim": dim, "engine": engine,
                "ppm": ppm, "tol": tol}
    if kind == "batched":
        return {"kind": kind, "n_ref": _log(rng, 20_000, 500_000), "nq": _log(rng, 500, 50_000),
                "dim": dim, "narrow": rng.choice([0.5, 0.7, 0.9])}
    if kind == "cascade":
        return {"kind": kind, "n_ref": _log(rng, 5000, 300_000), "nq": _log(rng, 200, 20_000),
                "dim": dim, "engine": rng.choice(["fp4", "fp4", "fp8"])}
    if kind == "ingest":
        return {"kind": kind, "n": _log(rng, 500, 800_000), "dim": dim}
    dim = rng.choice([2048, 8192, 8192])
    embed = rng.choice([64, 128, 256, 256])
    if kind == "learned":
        return {"kind": kind, "n_ref": _log(rng, 20_000, 500_000), "nq": _log(rng, 500, 30_000),
                "dim": dim, "hidden": 1024, "embed": embed, "k": rng.choice([16, 64, 256])}
    if kind == "embed":
        return {"kind": kind, "n": _log(rng, 50, 100_000), "dim": dim,
                "hidden": rng.choice([512, 1024]), "embed": embed}
    return {"kind": kind, "batch": 32 * _log(rng, 4, 64), "steps": rng.choice([8, 16, 32]),
            "dim": dim, "hidden": rng.choice([512, 1024]), "embed": embed}


# ---------------------------------------------------------------------------
# synthetic spectra on the GPU

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(n, lo, hi, g):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo


def _intensity(n, g):
    return torch.randn(n, generator=g, device="cuda", dtype=torch.float64).exp_()


def _offsets(counts):
    off = torch.zeros(counts.shape[0] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(counts, 0, out=off[1:])
    return off


def _library(n, g, charges, decoys):
    """n references (and, with decoys, one decoy each): raw peaks in CSR form,
    precursors and charges."""
    cnt = torch.randint(20, 151, (n,), generator=g, device="cuda")
    off = _offsets(cnt)
    total = int(off[-1])
    inten = _intensity(total, g)
    pmz = _uniform(n, *PMZ, g)
    ch = torch.randint(charges[0], charges[1] + 1, (n,), generator=g,
                       device="cuda").to(torch.int8)
    if not decoys:
        return off, _uniform(total, *MZ, g), inten, pmz, ch
    return (torch.cat([off, off[1:] + total]), _uniform(2 * total, *MZ, g),
            torch.cat([inten, inten]), torch.cat([pmz, pmz]), torch.cat([ch, ch]))


def _queries(lib, n_ref, nq, g):
    """nq queries made from references: jitter, 20% of the peaks dropped, 10%
    noise peaks, half of them mass-shifted."""
    off, mz, inten, pmz, ch = lib
    src = torch.randint(0, n_ref, (nq,), generator=g, device="cuda")
    cnt = (off[1:] - off[:-1])[src]
    seg = _offsets(cnt)
    total = int(seg[-1])
    qid = torch.repeat_interleave(torch.arange(nq, device="cuda"), cnt, output_size=total)
    at = off[:-1][src][qid] + torch.arange(total, device="cuda") - seg[:-1][qid]
    q_mz = mz[at] + 0.01 * torch.randn(total, generator=g, device="cuda", dtype=torch.float64)
    shifted = torch.rand(nq, generator=g, device="cuda") < 0.5
    delta = torch.where(shifted, _uniform(nq, -150.0, 500.0, g), 0.0)
    move = torch.rand(total, generator=g, device="cuda") < 0.4
    q_mz = torch.where(move, q_mz + delta[qid], q_mz)
    keep = torch.rand(total, generator=g, device="cuda") >= 0.2
    noise = (0.1 * cnt + 0.5).floor().to(torch.int64)
    nn = int(noise.sum())
    nid = torch.repeat_interleave(torch.arange(nq, device="cuda"), noise, output_size=nn)
    ids = torch.cat([qid[keep], nid])
    all_mz = torch.cat([q_mz[keep], _uniform(nn, *MZ, g)])
    all_in = torch.cat([inten[at][keep], _intensity(nn, g)])
    order = torch.argsort(ids, stable=True)
    q_ch = ch[src].contiguous()
    return (_offsets(torch.bincount(ids, minlength=nq)), all_mz[order].contiguous(),
            all_in[order].contiguous(), pmz[src] + delta / q_ch.double(), q_ch)


def _rows(n, words, g):
    """Packed rows that share a large common part, as spectrum hypervectors
    do: a base row with one bit in eight flipped."""
    def bits(*shape):
        return torch.randint(-2 ** 31, 2 ** 31, shape, generator=g, device="cuda",
                             dtype=torch.int64).to(torch.int32)
    return bits(1, words) ^ (bits(n, words) & bits(n, words) & bits(n, words))


def _weights(c, seed):
    r = np.random.default_rng(int(seed))
    D, H, E = c["dim"], c["hidden"], c["embed"]

    def uniform(fan_in, *shape):
        return (r.random(shape, dtype=np.float32) * 2 - 1) / np.float32(np.sqrt(fan_in))
    return {"W1": uniform(D, H, D), "b1": uniform(D, H), "W2": uniform(H, E, H),
            "b2": uniform(H, E)}


def _mean_bipolar(rows, dim):
    bit = torch.arange(32, device="cuda", dtype=torch.int32)
    b = ((rows[:, :, None] >> bit) & 1).reshape(rows.shape[0], dim)
    return (1.0 - 2.0 * b.double().mean(dim=0)).cpu().numpy()


# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    ctx = h.Context(h.Params(dim=case["dim"]))
    s = {"kind": kind, "case": case, "ctx": ctx}
    if kind == "ingest":
        s["lib"] = _library(case["n"], g, (2, 3), False)
        return s
    if kind == "embed":
        s["model"] = h.Model(ctx, _weights(case, seed))
        s["rows"] = _rows(case["n"], ctx.words, g)
        s["out"] = torch.empty((case["n"], case["embed"]), device="cuda")
        return s
    if kind == "train":
        s["model"] = h.Model(ctx, _weights(case, seed))
        s["pairs"] = _pairs(case, ctx.words, g)
        s["loss"] = torch.empty(case["steps"], device="cuda")
        return s
    n_ref, nq = case["n_ref"], case["nq"]
    lib = _library(n_ref, g, (2, 4) if kind == "batched" else (2, 3), True)
    q = _queries(lib, n_ref, nq, g)
    ctx.encode_library(*ctx.preprocess_device(*lib[:3]), *lib[3:])
    s["csr"] = ctx.preprocess_device(*q[:3])
    s["pmz"], s["charge"] = q[3], q[4]
    s["hv"] = torch.empty((nq, ctx.words), dtype=torch.int32, device="cuda")
    s["idx"] = torch.empty(nq, dtype=torch.int64, device="cuda")
    s["dist"] = torch.empty(nq, dtype=torch.int32, device="cuda")
    if kind == "batched":
        narrow = torch.rand(nq, generator=g, device="cuda") < case["narrow"]
        s["kinds"] = narrow.to(torch.int8)
        s["values"] = torch.where(narrow, 20.0, 500.0).double()
    elif kind == "cascade":
        s["decoy"] = (torch.arange(2 * n_ref, device="cuda") >= n_ref).to(torch.uint8)
    elif kind == "learned":
        ctx.encode_queries(*s["csr"], out=s["hv"])
        w = h.sketch_weights(case["dim"], case["hidden"], case["embed"], seed=7,
                             center=_mean_bipolar(s["hv"][:4096], case["dim"]))
        s["model"] = h.Model(ctx, w)
        s["model"].embed_library()
    torch.cuda.synchronize()
    return s


def _pairs(case, words, g):
    """Query rows and their references, [steps, batch, words] each: a
    reference is its query's row with about one bit in sixteen changed."""
    n = case["steps"] * case["batch"]
    q = _rows(n, words, g)
    flip = _rows(n, words, g)
    r = q ^ (flip & torch.roll(flip, 1, 0) & torch.roll(flip, 2, 0) & torch.roll(flip, 3, 0))
    shape = (case["steps"], case["batch"], words)
    return q.reshape(shape), r.reshape(shape)


TAU, LR = 0.05, 3e-5


def run(s):
    kind, case, ctx = s["kind"], s["case"], s["ctx"]
    if kind == "ingest":
        off, mz, inten, pmz, charge = s["lib"]
        csr = ctx.preprocess_device(off, mz, inten)
        ctx.encode_library(*csr, pmz, charge)
        # the bins and levels themselves show in every bit of the rows
        return {"offsets": csr[0], "order": ctx.library_order(), "rows": ctx.library_export()}
    if kind == "embed":
        return s["model"].embed(s["rows"], out=s["out"])
    if kind == "train":
        m, loss = s["model"], s["loss"]
        for i, (q, r) in enumerate(zip(*s["pairs"])):
            m.train_step(q, r, TAU, LR, loss_out=loss[i:i + 1])
        return {"loss": loss, "weights": m.get_weights()}
    hv = ctx.encode_queries(*s["csr"], out=s["hv"])
    if kind == "search":
        idx, dist = ctx.search_window(hv, s["pmz"], s["charge"],
                                      h.TOL_PPM if case["ppm"] else h.TOL_DA, case["tol"],
                                      ENGINES[case["engine"]], s["idx"], s["dist"])
        return {"rows": hv, "idx": idx, "dist": dist}
    if kind == "batched":
        idx, dist = ctx.search_batched(hv, s["pmz"], s["charge"], s["kinds"], s["values"],
                                       out_idx=s["idx"], out_dist=s["dist"])
        return {"rows": hv, "idx": idx, "dist": dist}
    if kind == "cascade":
        idx, dist, stage, q = ctx.cascade_search(hv, s["pmz"], s["charge"], s["decoy"],
                                                 engine=ENGINES[case["engine"]])
        return {"idx": idx, "dist": dist, "stage": stage, "qvalue": q}
    idx, dist, fallback, shortlist = s["model"].search(hv, s["pmz"], s["charge"], case["k"],
                                                       shortlist=True)
    return {"idx": idx, "dist": dist, "fallback": fallback, "shortlist": shortlist}


# ---------------------------------------------------------------------------

def _candidates(n_lib, ppm, tol, charges):
    """Mean candidates of a query: uniform precursors, one charge of several."""
    width = PMZ[1] - PMZ[0]
    if ppm:
        share = 2 * 0.5 * (PMZ[0] + PMZ[1]) * tol / 1e6 / width
    else:
        share = 2 * tol / width - (tol / width) ** 2
    return n_lib / charges * share


def work(case):
    kind, D = case["kind"], case["dim"]
    row = D / 8
    if kind == "ingest":
        n = case["n"]
        raw, out = n * (RAW_PEAKS * 16 + 8 + 9), n * (KEPT_PEAKS * 5 + 8)
        return {"bytes": raw + out + n * (row + 4), "flops": 0}
    if kind == "embed":
        n, H, E = case["n"], case["hidden"], case["embed"]
        return {"bytes": n * (row + 4 * E) + 2 * H * (D + E),
                "flops": 2.0 * n * H * (D + E)}
    if kind == "train":
        m, H, E = 2 * case["batch"], case["hidden"], case["embed"]
        # forward, the weights' gradients and the hidden layer's; Adam's state
        flops = 2.0 * m * (2 * H * D + 3 * H * E) + 3 * 2.0 * case["batch"] ** 2 * E
        return {"bytes": case["steps"] * (m * row + 24.0 * H * (D + E)),
                "flops": case["steps"] * flops}
    n_lib, nq = 2 * case["n_ref"], case["nq"]
    query = nq * (KEPT_PEAKS * 5 + 8 + 9 + row + 12)
    if kind == "search":
        pairs = nq * _candidates(n_lib, case["ppm"], case["tol"], 2)
    elif kind == "batched":
        pairs = nq * (case["narrow"] * _candidates(n_lib, True, 20.0, 3) +
                      (1 - case["narrow"]) * _candidates(n_lib, False, 500.0, 3))
    else:
        pairs = nq * _candidates(n_lib, False, 500.0, 2)
    library = min(n_lib, pairs) * (row + 4)
    if kind != "learned":
        return {"bytes": library + query, "flops": 2.0 * D * pairs}
    H, E, k = case["hidden"], case["embed"], case["k"]
    return {"bytes": min(n_lib, pairs) * E + nq * k * (row + 8) + query + 2 * H * (D + E),
            "flops": 2.0 * E * pairs + 2.0 * nq * H * (D + E)}


# ---------------------------------------------------------------------------

def _bipolar(rows, dim):
    bit = torch.arange(32, device="cuda", dtype=torch.int32)
    b = ((rows[:, :, None] >> bit) & 1).reshape(rows.shape[0], dim)
    return 1.0 - 2.0 * b.double()


def _forward(x, w):
    a = x @ w["W1"].T + w["b1"]
    z = a.clamp(min=0) @ w["W2"].T + w["b2"]
    s = (z.square().sum(1, keepdim=True) + 1e-12).sqrt()
    return a, z / s, s


def exact(case, seed):
    """The network of the learned form in 64 bits. The searches, the encoding
    and the preprocessing return whole numbers (and q-values, their ratios)."""
    kind, D = case["kind"], case["dim"]
    if kind not in ("embed", "train"):
        return None
    g, words = _gen(seed), D // 32
    w = {k: torch.from_numpy(v).cuda().double() for k, v in _weights(case, seed).items()}
    if kind == "embed":
        rows = _rows(case["n"], words, g)
        return torch.cat([_forward(_bipolar(r, D), w)[1] for r in rows.split(8192)])
    B, losses = case["batch"], []
    m = {k: torch.zeros_like(v) for k, v in w.items()}
    v = {k: torch.zeros_like(x) for k, x in w.items()}
    for t, (q, r) in enumerate(zip(*_pairs(case, words, g)), 1):
        x = _bipolar(torch.cat([q, r]), D)
        a, e, s = _forward(x, w)
        logits = e[:B] @ e[B:].T / TAU
        losses.append((logits.logsumexp(1) - logits.diagonal()).mean())
        ds = (logits.softmax(1) - torch.eye(B, device="cuda", dtype=torch.float64)) / B / TAU
        de = torch.cat([ds @ e[B:], ds.T @ e[:B]])
        dz = (de - e * (e * de).sum(1, keepdim=True)) / s
        da = (dz @ w["W2"]) * (a > 0)
        grad = {"W1": da.T @ x, "b1": da.sum(0), "W2": dz.T @ a.clamp(min=0), "b2": dz.sum(0)}
        for k in w:
            m[k] = 0.9 * m[k] + 0.1 * grad[k]
            v[k] = 0.999 * v[k] + 0.001 * grad[k].square()
            w[k] = w[k] - LR * (m[k] / (1 - 0.9 ** t)) / ((v[k] / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return {"loss": torch.stack(losses), "weights": w}
