"""The work whose speed is measured: calls that a user of the filtered search
makes, through the package's public entry points, on one GPU.

A case is one call path on one index:

  query     ``query_batch_into``: predicate encoder (or caller's w_z), condition,
            distance tables and the filtered search of a batch, on an index
            whose rows are clustered by the filtered attributes
  masked    ``select_codebook_into`` + ``build_lut_into`` + ``search_into`` on an
            index in id order, where clauses are tested row by row
  sdc       ``build_sdc_lut_into`` + ``search_into`` (the SDC baseline)
  filter    ``filter_into``: selection bitmaps and pool sizes
  exact     ``exact_search_into``: exact filtered kNN over the fp32 vectors
  train     ``train_step_into``: one SGD step of the memory bank and W

``prepare`` draws what such a program holds before the call: a Gaussian-mixture
dataset quantized by PQ (component means in [-1, 1]^D, sigma 0.3), attribute
columns (one uniform, or uniform + Zipf(1.1) categories), conditioning
parameters and encoder weights, predicates of the case's selectivity, queries
from the same mixture, and the loaded index with its output buffers.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2607_22922_amd import ifvs

SIGMA = 0.3
BANK_ROWS, R, H_FUNCS = 4096, 8, 2          # memory bank rows, directions, hash functions
PARAM_STD = 0.05
WZ_CENTER, WZ_STD = math.log(math.e - 1.0), 0.1
HIDDEN, HEADS, LAYERS, FFN = 64, 4, 2, 128  # predicate encoder
SAMPLES = 64                                # encoded vectors per mixture component
KMEANS_ITERS = 4


# ------------------------------------------------------------------- cases
def listed():
    two = dict(domain=1000, categories=100)
    return [
        # A single online query against 1M SIFT-like vectors (range + category):
        # latency and launches are everything.
        dict(name="online_one", kind="query", n=1_000_000, m=16, dsub=8, comps=256, **two, sel=0.01, nq=1, k=10,
             f16=False, encoder=True, coarse=0),
        # The smallest dataset with a small batch: 100 queries over 10K vectors.
        dict(name="toy_100", kind="query", n=10_000, m=16, dsub=8, comps=32, domain=1000, categories=0, sel=0.1,
             nq=100, k=10, f16=False, encoder=True, coarse=0),
        # A product quantizer of no special shape, half-precision tables, odd
        # sizes everywhere, the caller's own weights.
        dict(name="odd_f16", kind="query", n=777_773, m=21, dsub=5, comps=200, domain=977, categories=0, sel=0.05,
             nq=37, k=33, f16=True, encoder=False, coarse=0),
        # The serving batch on 10M vectors, a narrow range per query.
        dict(name="batch_narrow", kind="query", n=10_000_000, m=48, dsub=2, comps=1024, domain=3650, categories=0,
             sel=0.01, nq=256, k=10, f16=False, encoder=True, coarse=0),
        # The same batch with half of the rows selected and the coarse quantizer.
        dict(name="batch_wide", kind="query", n=10_000_000, m=48, dsub=2, comps=1024, domain=3650, categories=0,
             sel=0.5, nq=256, k=10, f16=False, encoder=True, coarse=2048),
        # 960-dimensional descriptors, 100 neighbours.
        dict(name="deep_k100", kind="query", n=1_000_000, m=120, dsub=8, comps=128, domain=10_000, categories=0,
             sel=0.1, nq=256, k=100, f16=False, encoder=False, coarse=0),
        # The largest dataset: 100M vectors of 16-byte codes, range + category.
        dict(name="large_100m", kind="query", n=100_000_000, m=16, dsub=8, comps=4096, domain=1000, categories=1000,
             sel=0.1, nq=256, k=10, f16=False, encoder=True, coarse=0),
        # Rows in id order, small pools: the selection decides the work.
        dict(name="masked_narrow", kind="masked", n=10_000_000, m=48, dsub=2, comps=1024, domain=3650, categories=100,
             sel=0.01, nq=256, k=10, f16=False),
        # Rows in id order, half of them selected, a ragged row count.
        dict(name="masked_wide", kind="masked", n=4_000_037, m=48, dsub=2, comps=1024, domain=3650, categories=0,
             sel=0.5, nq=256, k=10, f16=False),
        # The Filter stage alone: bitmaps and pool sizes of 256 predicates.
        dict(name="filter_10m", kind="filter", n=10_000_000, domain=3650, categories=100, sel=0.1, nq=256),
        # Exact filtered kNN of a batch (ground truth, exact baseline).
        dict(name="exact_10m", kind="exact", n=10_000_000, m=48, dsub=2, comps=1024, domain=3650, categories=0,
             sel=0.1, nq=256, k=10),
        # One training step of the conditioning: 10 positives, 32 hard negatives.
        dict(name="train_256", kind="train", n=1_000_000, m=48, dsub=2, comps=1024, domain=3650, categories=0,
             sel=0.01, nq=256, n_pos=10, n_neg=32),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case: any of the paths, sizes over their whole range."""
    kind = rng.choices(["query", "masked", "sdc", "filter", "exact", "train"], [10, 4, 2, 2, 4, 3])[0]
    m, dsub = rng.choice([(16, 8), (48, 2), (120, 8), (rng.randint(4, 64), rng.randint(1, 9))])
    nq = max(1, round(_log(rng, 1, 256)))
    sel = _log(rng, 0.001, 0.5)
    k = max(1, round(_log(rng, 1, 100)))
    two = rng.random() < 0.4
    domain = rng.randint(500, 10_000)
    most = dict(query=100_000_000, sdc=30_000_000, masked=10_000_000, filter=20_000_000, exact=10_000_000,
                train=2_000_000)[kind]
    # table reads (rows x queries x subspaces) and bytes no larger than the listed ones'
    reads = (2.5e10 if kind in ("query", "sdc") else 2e10) if m in (16, 48, 120) else 8e9
    if kind in ("query", "sdc"):
        most = min(most, reads / (m * nq * sel), 1.6e9 / m)
    elif kind == "masked":
        most = min(most, reads / (m * nq), 4.8e8 / m)
    elif kind == "exact":
        most = min(most, 9.6e8 / (m * dsub))
    elif kind == "filter":
        most = min(most, 2.5e9 / nq)
    n = int(_log(rng, 10_000, max(20_000, most))) | 1
    comps = max(16, min(4096, n // 5000))
    c = dict(kind=kind, n=n, domain=domain, categories=rng.randint(20, 1000) if two else 0, sel=round(sel, 5), nq=nq)
    if kind == "filter":
        return c
    c.update(m=m, dsub=dsub, comps=comps)
    if kind == "train":
        if m > 64:                       # the tables of one query and their gradients share the LDS
            c.update(m=48, dsub=2)
        c.update(n_pos=rng.randint(1, 20), n_neg=rng.randint(8, 100))
        return c
    c.update(k=k)
    if kind != "exact":
        c.update(f16=rng.random() < 0.25)
    if kind == "query":
        lists = n >= 1_000_000 and m >= 32 and m * dsub <= 128 and rng.random() < 0.5
        c.update(encoder=rng.random() < 0.5, coarse=2048 if lists else 0)
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed, tag):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1_000_003 + tag) % (1 << 62))


def _means(case, seed):
    d = case["m"] * case["dsub"]
    return torch.rand(case["comps"], d, generator=_gen(seed, 0), device="cuda") * 2.0 - 1.0


def _codebook(sample, m, seed):
    """A few Lloyd iterations per subspace; [m][256][dsub] fp32 and the codes of the sample."""
    xs = sample.reshape(sample.shape[0], m, -1).permute(1, 0, 2).contiguous()        # [m][n][dsub]
    perm = torch.randperm(xs.shape[1], generator=_gen(seed, 4), device="cuda")[:256]
    cb = xs[:, perm, :].clone()
    for i in range(KMEANS_ITERS + 1):
        code = torch.empty(m, xs.shape[1], dtype=torch.int64, device="cuda")
        half = 0.5 * (cb * cb).sum(-1)
        for j in range(m):
            code[j] = (half[j] - xs[j] @ cb[j].t().contiguous()).argmin(1)
        if i == KMEANS_ITERS:
            return cb.contiguous(), code.to(torch.uint8)
        # sums in fixed point: atomics add in any order, the inputs stay the same bits
        fixed = (xs * 2.0 ** 20).round().long()
        count = torch.zeros(m, 256, dtype=torch.int64, device="cuda").scatter_add_(1, code, torch.ones_like(code))
        total = torch.zeros(cb.shape, dtype=torch.int64, device="cuda")
        total.scatter_add_(1, code[..., None].expand(-1, -1, cb.shape[2]), fixed)
        mean = total.double() / (count.clamp(min=1)[..., None] * 2.0 ** 20)
        cb = torch.where(count[..., None] > 0, mean.float(), cb)


def _dataset(case, seed):
    """Component of each of n mixture vectors, codebook and codes.  Given its
    component, a vector's subspaces are independent, so each code is taken
    from the codes of SAMPLES encoded vectors of the component."""
    n, m = case["n"], case["m"]
    means = _means(case, seed)
    comps, d = means.shape
    g = _gen(seed, 1)
    sample = (means[:, None, :] + SIGMA * torch.randn(comps, SAMPLES, d, generator=g, device="cuda")).reshape(-1, d)
    fit = sample if sample.shape[0] <= 65536 else sample[:: -(-sample.shape[0] // 65536)]
    cb, code = _codebook(fit, m, seed)
    if fit is not sample:
        half = 0.5 * (cb * cb).sum(-1)
        xs = sample.reshape(-1, m, case["dsub"])
        code = torch.stack([(half[j] - xs[:, j, :].contiguous() @ cb[j].t().contiguous()).argmin(1) for j in range(m)])
        code = code.to(torch.uint8)
    table = code.reshape(m, comps, SAMPLES).permute(1, 0, 2).contiguous().reshape(-1)   # [comps][m][SAMPLES]
    codes = torch.empty(n, m, dtype=torch.uint8, device="cuda")
    comp_of = torch.empty(n, dtype=torch.int16, device="cuda")
    step = max(1, (1 << 27) // m)
    off = torch.arange(m, device="cuda", dtype=torch.int32) * SAMPLES
    for s in range(0, n, step):
        rows = min(step, n - s)
        comp = torch.randint(0, comps, (rows, 1), generator=g, device="cuda", dtype=torch.int32)
        pick = torch.randint(0, SAMPLES, (rows, m), generator=g, device="cuda", dtype=torch.int32)
        comp_of[s:s + rows] = comp[:, 0]
        codes[s:s + rows] = table[(comp * (m * SAMPLES) + off + pick).reshape(-1)].reshape(rows, m)
    return comp_of, cb, codes


def _vectors(case, seed):
    means = _means(case, seed)
    n, g = case["n"], _gen(seed, 2)
    x = torch.empty(n, means.shape[1], device="cuda")
    step = max(1, (1 << 27) // means.shape[1])
    for s in range(0, n, step):
        rows = min(step, n - s)
        comp = torch.randint(0, means.shape[0], (rows,), generator=g, device="cuda")
        x[s:s + rows] = means[comp] + SIGMA * torch.randn(rows, means.shape[1], generator=g, device="cuda")
    return x


def _query_comps(case, seed):
    return torch.randint(0, case["comps"], (case["nq"],), generator=_gen(seed, 9), device="cuda")


def _queries(case, seed):
    mean = _means(case, seed)[_query_comps(case, seed)]
    return mean + SIGMA * torch.randn(*mean.shape, generator=_gen(seed, 3), device="cuda")


def _zipf(categories):
    w = np.arange(1, categories + 1, dtype=np.float64) ** -1.1
    return w / w.sum()


def _attributes(case, seed):
    n, g = case["n"], _gen(seed, 7)
    cols = [torch.randint(0, case["domain"], (n,), generator=g, device="cuda", dtype=torch.int32)]
    if case["categories"]:
        cdf = torch.from_numpy(np.cumsum(_zipf(case["categories"]))).to(device="cuda", dtype=torch.float32)
        u = torch.rand(n, generator=g, device="cuda")
        cols.append(torch.searchsorted(cdf, u, right=True).clamp_(max=case["categories"] - 1).to(torch.int32))
    return torch.stack(cols).contiguous()


def _predicates(case, seed):
    """Range clauses of the case's selectivity; with categories an equality on
    one frequent enough, else a prefix of the most frequent ones."""
    rng = random.Random(int(seed) * 7 + 3)
    s, dom, out = case["sel"], case["domain"], []
    probs = _zipf(case["categories"]) if case["categories"] else None
    frequent = [] if probs is None else [c for c, p in enumerate(probs) if p >= s / 0.9]
    for _ in range(case["nq"]):
        mass, clause = 1.0, None
        if frequent:
            c = rng.choice(frequent)
            mass, clause = float(probs[c]), (1, c, c + 1)
        elif probs is not None:
            hi = int(np.searchsorted(np.cumsum(probs), s)) + 1
            mass, clause = float(probs[:hi].sum()), (1, 0, hi)
        w = min(dom, max(1, int(s / mass * dom + 0.5)))
        lo = rng.randint(0, dom - w)
        out.append([(0, lo, lo + w)] + ([clause] if clause else []))
    return out


def _conditioning(case, seed):
    g, m = _gen(seed, 5), case["m"]
    bank = torch.randn(BANK_ROWS, m * R, generator=g, device="cuda") * PARAM_STD
    w = torch.randn(m, R, 256, case["dsub"], generator=g, device="cuda") * PARAM_STD
    w_z = WZ_CENTER + WZ_STD * torch.randn(case["nq"], m * case["dsub"], generator=g, device="cuda")
    return bank, w, w_z.contiguous()


def _encoder(case, seed):
    g, d = _gen(seed, 6), case["m"] * case["dsub"]
    domains = [case["domain"]] + ([case["categories"]] if case["categories"] else [])

    def rn(*shape, std=1.0):
        return torch.randn(*shape, generator=g, device="cuda") * std

    def layer():
        s = HIDDEN ** -0.5
        return dict(ln1_g=1 + rn(HIDDEN, std=0.1), ln1_b=rn(HIDDEN, std=0.1), Wq=rn(HIDDEN, HIDDEN, std=s),
                    Wk=rn(HIDDEN, HIDDEN, std=s), Wv=rn(HIDDEN, HIDDEN, std=s), bq=rn(HIDDEN, std=0.1),
                    bk=rn(HIDDEN, std=0.1), bv=rn(HIDDEN, std=0.1), Wo=rn(HIDDEN, HIDDEN, std=s),
                    bo=rn(HIDDEN, std=0.1), ln2_g=1 + rn(HIDDEN, std=0.1), ln2_b=rn(HIDDEN, std=0.1),
                    W1=rn(HIDDEN, FFN, std=s), b1=rn(FFN, std=0.1), W2=rn(FFN, HIDDEN, std=FFN ** -0.5),
                    b2=rn(HIDDEN, std=0.1))

    e = dict(heads=HEADS, col_offset=torch.zeros(len(domains), dtype=torch.float64),
             col_scale=torch.tensor([1.0 / v for v in domains], dtype=torch.float64), col_embed=rn(len(domains), HIDDEN),
             feat_w=rn(2, HIDDEN), feat_b=rn(HIDDEN, std=0.1), cls=rn(HIDDEN), layers=[layer() for _ in range(LAYERS)])
    e.update(lnf_g=1 + rn(HIDDEN, std=0.1), lnf_b=rn(HIDDEN, std=0.1), out_w=rn(HIDDEN, d, std=WZ_STD * HIDDEN ** -0.5),
             out_b=torch.full((d,), WZ_CENTER, device="cuda"))
    return e


def _candidates(case, seed, comp_of):
    """n_pos positives and n_neg hard negatives per query: vectors of the query's
    own component.  In one query of sixteen the last negatives are absent."""
    nc = case["n_pos"] + case["n_neg"]
    order = torch.argsort(comp_of, stable=True)
    first = torch.searchsorted(comp_of[order].long(), _query_comps(case, seed)[:, None])
    cand = order[(first + torch.arange(nc, device="cuda")) % case["n"]].to(torch.int32)
    cand[::16, case["n_pos"] + 1:] = -1
    return cand.contiguous()


def prepare(case, seed):
    kind, nq = case["kind"], case["nq"]
    attrs = _attributes(case, seed)
    preds = ifvs.pack_predicates(_predicates(case, seed))
    st = dict(case=case, preds=preds)
    dev = dict(device="cuda")
    if kind == "filter":
        codes = torch.zeros(case["n"], 1, dtype=torch.uint8, **dev)
        st["index"] = ifvs.Index(codes, torch.zeros(1, 256, 1, **dev), attrs, max_batch=nq, max_k=1)
        st["bitmap"] = torch.empty(nq, st["index"].words(), dtype=torch.int32, **dev)
        st["count"] = torch.empty(nq, dtype=torch.int64, **dev)
        return st
    m, dsub = case["m"], case["dsub"]
    k = case.get("k", 1)
    cluster = () if kind == "masked" else ((1, 0) if case["categories"] else (0,))
    st["q"] = _queries(case, seed)
    if kind == "exact":
        # the codes play no part in the exact search
        codes = torch.zeros(case["n"], 1, dtype=torch.uint8, **dev)
        index = ifvs.Index(codes, torch.zeros(1, 256, m * dsub, **dev), attrs, max_batch=nq, max_k=k,
                           cluster_cols=cluster)
        index.load_vectors(_vectors(case, seed))
    else:
        comp_of, cb, codes = _dataset(case, seed)
        bank, w, w_z = _conditioning(case, seed)
        sdc = kind == "sdc"
        index = ifvs.Index(codes, cb, attrs, None if sdc else bank, None if sdc else w, R, H_FUNCS, 0x5EED + int(seed),
                           max_batch=nq, max_k=k, cluster_cols=cluster)
        if case.get("encoder"):
            index.load_encoder(_encoder(case, seed))
            st["w_z"] = None
        elif not sdc:
            st["w_z"] = w_z
        if case.get("coarse"):
            index.build_coarse(case["coarse"], 10)
        if kind == "train":
            st["cand"] = _candidates(case, seed, comp_of)
            st["loss"] = torch.empty(nq, **dev)
            st["dwz"] = torch.empty(nq, m * dsub, **dev)
        st["wz_out"] = torch.empty(nq, m * dsub, **dev)
        st["alpha"] = torch.empty(nq, m * R, **dev)
        st["wf"] = torch.empty(nq, m * dsub, **dev)
        st["lut"] = torch.empty(nq, m, 256, dtype=torch.float16 if case.get("f16") else torch.float32, **dev)
        st["dtype"] = ifvs.LUT_F16 if case.get("f16") else ifvs.LUT_F32
    st["index"] = index
    st["ids"] = torch.empty(nq, k, dtype=torch.int32, **dev)
    st["dist"] = torch.empty(nq, k, **dev)
    return st


TAU, LAM, LR = 1.0, 0.1, 20.0


def run(st):
    case, index = st["case"], st["index"]
    kind, k = case["kind"], case.get("k", 1)
    if kind == "filter":
        index.filter_into(case["nq"], st["preds"], st["bitmap"], st["count"])
        return dict(bitmap=st["bitmap"], count=st["count"])
    if kind == "exact":
        index.exact_search_into(st["q"], st["preds"], k, st["ids"], st["dist"])
        return dict(ids=st["ids"], dist=st["dist"])
    if kind == "train":
        index.train_step_into(st["q"], st["preds"], st["w_z"], st["cand"], case["n_pos"], TAU, LAM, LR, st["loss"],
                              st["dwz"])
        bank, w = index.read_params()
        return dict(loss=st["loss"], dwz=st["dwz"], bank=bank, W=w)
    if kind == "sdc":
        index.build_sdc_lut_into(st["q"], st["dtype"], st["lut"])
        index.search_into(case["nq"], st["preds"], st["lut"], st["dtype"], k, st["ids"], st["dist"])
        return dict(ids=st["ids"], dist=st["dist"], lut=st["lut"])
    if kind == "masked":
        index.select_codebook_into(st["q"], st["preds"], st["w_z"], st["alpha"], st["wf"])
        index.build_lut_into(st["q"], st["alpha"], st["wf"], st["dtype"], st["lut"])
        index.search_into(case["nq"], st["preds"], st["lut"], st["dtype"], k, st["ids"], st["dist"])
    else:
        index.query_batch_into(st["q"], st["preds"], st["w_z"], st["wz_out"] if st["w_z"] is None else None,
                               st["alpha"], st["wf"], st["dtype"], st["lut"], k, st["ids"], st["dist"])
    out = dict(ids=st["ids"], dist=st["dist"], alpha=st["alpha"], w_f=st["wf"], lut=st["lut"])
    if kind == "query" and st["w_z"] is None:
        out["w_z"] = st["wz_out"]
    return out


def work(case):
    """Bytes: the rows that some query of the batch selects, read once, the
    inputs and the outputs.  Operations: one addition per table read of every
    (query, selected row); exact distances three per dimension; tables and
    training their multiplications and additions."""
    n, nq, s, kind = case["n"], case["nq"], case["sel"], case["kind"]
    rows = n * (1.0 - (1.0 - s) ** nq)
    n_attr = 2 if case["categories"] else 1
    if kind == "filter":
        return dict(bytes=n * 4 * n_attr + nq * n / 8, flops=2.0 * nq * n * n_attr)
    m, d = case["m"], case["m"] * case["dsub"]
    table = nq * m * 256
    if kind == "train":
        nc = case["n_pos"] + case["n_neg"]
        params = BANK_ROWS * m * R * 4 + 256 * d * R * 4
        return dict(bytes=2.0 * params + nq * nc * m + 3.0 * nq * d * 4, flops=nq * (256.0 * d * (6 * R + 10) + nc * m))
    if kind == "exact":
        return dict(bytes=rows * d * 4 + nq * (d * 4 + case["k"] * 8), flops=3.0 * d * nq * n * s)
    masks = n * 4.0 * n_attr if kind == "masked" else 0.0
    return dict(bytes=rows * m + masks + table * (2 if case["f16"] else 4) + 256 * d * (R + 1) * 4 + nq * d * 8,
                flops=nq * n * s * m + nq * 256.0 * d * (5 + 2 * R))


def tolerance(case):
    """Searches, tables and bitmaps are defined operation by operation in fp32,
    so the results are the same bits.  The encoder's projections may be summed
    in any order, which the later steps carry on; training sums over the batch
    with atomics."""
    if case["kind"] == "train":
        return dict(rel=4e-6, max=4e-4)
    if case.get("encoder"):
        return dict(rel=5e-5, max=2e-3, differ=0.005) if case["f16"] else dict(rel=1e-6, max=4e-5, differ=0.002)
    return "exact"


# ------------------------------------------------------- the same in 64 bits
MASK = (1 << 64) - 1


def _splitmix(z):
    z = (z + 0x9E3779B97F4A7C15) & MASK
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & MASK
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & MASK
    return z ^ (z >> 31)


def _bank_rows(q, preds, hash_seed):
    """Memory-bank rows of each query: FNV-1a over its bytes and clauses, then SplitMix64."""
    out = []
    for x, clauses in zip(q.cpu().numpy(), preds):
        data = x.astype("<f4").tobytes() + np.array([len(clauses)], "<i4").tobytes()
        for col, lo, hi in clauses:
            data += np.array([col], "<i4").tobytes() + np.array([lo, hi], "<i8").tobytes()
        key = 0xCBF29CE484222325
        for b in data:
            key = ((key ^ b) * 0x100000001B3) & MASK
        out.append([_splitmix(key ^ _splitmix((hash_seed + j) & MASK)) % BANK_ROWS for j in range(H_FUNCS)])
    return torch.tensor(out, device="cuda")


def _norm(x, g, b):
    return torch.nn.functional.layer_norm(x, (x.shape[-1],), g.double(), b.double(), 1e-5)


def _encode(case, enc, preds):
    """w_z of every predicate (all of one clause count) in 64 bits."""
    e = {k: v.double() if torch.is_tensor(v) else v for k, v in enc.items()}
    t = torch.tensor(preds, dtype=torch.float64, device="cuda")                  # [nq][clauses][3]
    col = t[..., 0].long()
    off, scale = e["col_offset"].cuda()[col], e["col_scale"].cuda()[col]
    f = lambda v: ((v - off) * scale).clamp(-1.0, 2.0).float().double()[..., None]
    tok = e["col_embed"][col] + f(t[..., 1]) * e["feat_w"][0] + f(t[..., 2]) * e["feat_w"][1] + e["feat_b"]
    x = torch.cat([e["cls"].expand(len(preds), 1, HIDDEN), tok], 1)
    nq, n_tok, dh = x.shape[0], x.shape[1], HIDDEN // HEADS
    for p in enc["layers"]:
        p = {k: v.double() for k, v in p.items()}
        z = _norm(x, p["ln1_g"], p["ln1_b"])
        a, b, v = ((z @ p["W" + c] + p["b" + c]).reshape(nq, n_tok, HEADS, dh).transpose(1, 2).contiguous()
                   for c in "qkv")
        w = torch.softmax(a @ b.transpose(2, 3).contiguous() / math.sqrt(dh), -1)
        x = x + (w @ v).transpose(1, 2).reshape(nq, n_tok, HIDDEN) @ p["Wo"] + p["bo"]
        z = _norm(x, p["ln2_g"], p["ln2_b"])
        x = x + torch.relu(z @ p["W1"] + p["b1"]) @ p["W2"] + p["b2"]
    return _norm(x[:, 0], e["lnf_g"], e["lnf_b"]) @ e["out_w"] + e["out_b"]


def _tables(q, wf, cb, delta):
    m, _, dsub = cb.shape
    e = q.double().reshape(-1, m, 1, dsub) - (cb.double() + delta)
    return (wf.reshape(-1, m, 1, dsub) * e * e).sum(-1)


def _selected(attrs, clauses):
    keep = torch.ones(attrs.shape[1], dtype=torch.bool, device="cuda")
    for col, lo, hi in clauses:
        keep &= (attrs[col] >= lo) & (attrs[col] < hi)
    return keep.nonzero().flatten()


def _ranked(case, score, attrs, preds):
    """Ascending k smallest scores of each query's selected rows, padded with +inf."""
    k = case["k"]
    out = torch.full((case["nq"], k), math.inf, dtype=torch.float64, device="cuda")
    for i, p in enumerate(preds):
        rows, best = _selected(attrs, p), []
        for part in rows.split(4_000_000):
            best.append(torch.topk(score(i, part), min(k, part.numel()), largest=False).values)
        if best:
            v = torch.sort(torch.cat(best)).values[:k]
            out[i, :v.numel()] = v
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "filter":
        return None
    attrs, preds, q = _attributes(case, seed), _predicates(case, seed), _queries(case, seed)
    nq, pairs = case["nq"], case["nq"] * case["n"] * case["sel"]
    if kind == "exact":
        if pairs * case["m"] * case["dsub"] > 4e10:
            return None
        x = _vectors(case, seed)
        return dict(ids=None, dist=_ranked(case, lambda i, r: (x[r].double() - q[i].double()).square().sum(1), attrs,
                                           preds))
    comp_of, cb, codes = _dataset(case, seed)
    m, dsub = case["m"], case["dsub"]
    slow = pairs * m > 2e10

    def search(lut):
        if slow:
            return None
        flat = lut.reshape(nq, m * 256)
        off = torch.arange(m, device="cuda") * 256

        def score(i, rows):
            out = torch.empty(rows.numel(), dtype=torch.float64, device="cuda")
            for s in range(0, rows.numel(), 1 << 19):
                c = codes[rows[s:s + (1 << 19)]].long() + off
                out[s:s + c.shape[0]] = flat[i][c.reshape(-1)].reshape(c.shape).sum(1)
            return out

        return _ranked(case, score, attrs, preds)

    if kind == "sdc":
        qs = q.double().reshape(nq, m, 1, dsub)
        near = (qs - cb.double()).square().sum(-1).argmin(-1)                       # [nq][m]
        own = cb.double()[torch.arange(m, device="cuda"), near].unsqueeze(2)        # [nq][m][1][dsub]
        lut = (own - cb.double()).square().sum(-1)
        return dict(ids=None, dist=search(lut), lut=lut)
    bank, w, w_z = _conditioning(case, seed)
    if case.get("encoder"):
        w_z = _encode(case, _encoder(case, seed), preds)
    rows = _bank_rows(q, preds, 0x5EED + int(seed))
    if kind != "train":
        alpha = bank.double()[rows].sum(1)
        wf = torch.nn.functional.softplus(w_z.double(), threshold=1e9)
        delta = (alpha.reshape(nq, m, R, 1, 1) * w.double()).sum(2) if nq * m * dsub < 30_000 else \
            torch.stack([(a.reshape(m, R, 1, 1) * w.double()).sum(1) for a in alpha])
        lut = _tables(q, wf, cb, delta)
        out = dict(ids=None, dist=search(lut), alpha=alpha, w_f=wf, lut=lut)
        if case.get("encoder"):
            out["w_z"] = w_z
        return out
    cand = _candidates(case, seed, comp_of).long()
    bank, w, w_z = bank.double().requires_grad_(), w.double().requires_grad_(), w_z.double().requires_grad_()
    losses, total = [], 0.0
    for i in range(nq):
        alpha = bank[rows[i]].sum(0)
        delta = (alpha.reshape(m, R, 1, 1) * w).sum(1)
        lut = _tables(q[i:i + 1], torch.nn.functional.softplus(w_z[i:i + 1], threshold=1e9), cb, delta)[0]
        live = cand[i][cand[i] >= 0]
        d = lut[torch.arange(m, device="cuda"), codes[live].long()].sum(1)
        loss = torch.logsumexp(-d / TAU, 0) + d[:case["n_pos"]].mean() / TAU + LAM * delta.square().mean()
        (loss / nq).backward()
        losses.append(loss.detach())
    return dict(loss=torch.stack(losses), dwz=w_z.grad, bank=bank.detach() - LR * bank.grad, W=w.detach() - LR * w.grad)
