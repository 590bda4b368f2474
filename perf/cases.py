"""The work a user of this library has it do, as cases with sizes: exhaustive searches from one
query over a small list to batches over ten million codes, the stage-by-stage calls, inverted-list
searches behind the coarse quantizer (both modes) and encoding.

The sizes are those of harness/synth.py's configurations and of bench.py; inputs are synthetic
with the same distributions (byte-range heavy-tailed descriptors, normalised anisotropic
Gaussians), k-means codebooks and nearest-centroid codes, all from the seed.
"""
import math

import numpy as np
import torch

from paper_1812_09162_amd import binding as qb

T_CALIB = 400  # calibration codes of the distance quantizer (Section 4.1)

# layout: bits of the sub-quantizers, width of the quantized tables
LAYOUTS = {
    "16x4": ([4] * 16, 8),             # 64-bit codes, the paper's m x {4,4} with uint8 tables
    "32x4": ([4] * 32, 8),             # 128-bit codes
    "c3": ([6, 5, 5, 6, 5, 5, 4, 4], 16),  # irregular 40-bit codes
    "655": ([6, 5, 5] * 4, 16),        # irregular 64-bit codes
    "664": ([6, 6, 4] * 4, 16),
    "664x2": ([6, 6, 4] * 8, 16),      # irregular 128-bit codes
    "8x8": ([8] * 8, 16),              # classic product quantizer, 64-bit codes
    "16x8": ([8] * 16, 16),            # ... 128-bit codes
}


def listed():
    def flat(name, **kw):
        return dict(dict(name=name, path="search", layout="16x4", data="gauss", d=96, n=10_000_000, nq=1, R=100), **kw)

    def ivf(name, **kw):
        return dict(dict(name=name, path="ivf", layout="16x4", data="gauss", d=96, n=100_000_000, nq=1, R=100,
                         K=65_536, nprobe=64), **kw)

    return [
        # the smallest call: one query over 100,000 SIFT-like descriptors (an index shard, a test set)
        flat("search_c0_q1", data="gamma", d=128, n=100_000),
        # the headline workload: one request at a time over ten million 64-bit codes
        flat("search_c1_q1"),
        # a server that collects requests into batches
        flat("search_c1_q32", nq=32),
        flat("search_c1_q256", nq=256),
        # 128-bit codes, long result lists for re-ranking
        flat("search_c2_q1_r1000", layout="32x4", data="gamma", d=128, n=20_000_000, R=1000),
        # irregular sub-quantizers with 16-bit tables, one request and a batch
        flat("search_c3_q1", layout="c3", data="gamma", d=128),
        flat("search_664_q32", layout="664", data="gamma", d=128, nq=32),
        # the stages called one by one (tables and quantizer kept for inspection), 1,000 evaluation
        # queries over a million base vectors (the paper's SIFT1M shape), odd length
        flat("stages_1m_q1000", path="stages", data="gamma", d=128, n=1_000_003, nq=1000),
        # inverted index over a hundred million codes: one request; a bulk job of 10,000 queries
        ivf("ivf_c4_q1"),
        ivf("ivf_c4_q10000", nq=10_000),
        # ... with the bound that tightens from list to list
        ivf("ivf_tight_c4_q1000", path="ivf_tight", nq=1000),
        # building the index: ten million vectors to codes
        flat("encode_c1", path="encode", nq=0, R=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["search", "search", "search", "search", "stages", "ivf", "ivf", "ivf_tight", "encode"])
    layout = rng.choice(["16x4", "16x4", "32x4", "c3", "655", "664", "664x2", "8x8", "16x8"])
    data = rng.choice(["gauss", "gamma"])
    d = rng.choice([96, 128])
    R = rng.choice([1, 10, 100, 100, 100, _log_int(rng, 2, 1000)])
    if path == "encode":
        return dict(path=path, layout=layout, data=data, d=d, n=_log_int(rng, 10_000, 4_000_000), nq=0, R=0)
    if path in ("search", "stages"):
        n = _log_int(rng, 50_000, 10_000_000)
        nq = rng.choice([1, _log_int(rng, 2, 64), _log_int(rng, 2, 256)])
        nq = max(1, min(nq, 400_000_000 // n))
        return dict(path=path, layout=layout, data=data, d=d, n=n, nq=nq, R=R)
    n = _log_int(rng, 500_000, 20_000_000)
    K = max(64, min(16_384, _log_int(rng, max(64, n // 6000), n // 400)))
    nprobe = min(_log_int(rng, 4, 128), K)
    nq = rng.choice([1, _log_int(rng, 2, 300), _log_int(rng, 300, 2000)])
    nq = max(1, min(nq, int(300_000_000 / (nprobe * (n / K)))))
    return dict(path=path, layout=layout, data=data, d=d, n=n, nq=nq, R=min(R, 200), K=K, nprobe=nprobe)


# ------------------------------------------------------------------- inputs --
def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed, stream, device):
    g = torch.Generator(device=device)
    g.manual_seed((seed * 1000003 + stream * 7919 + 12345) & 0x7FFFFFFFFFFFFFFF)
    return g


def _vectors(data, n, d, seed, stream):
    z = torch.randn((n, d), generator=_gen(seed, stream, _dev()), device=_dev(), dtype=torch.float32)
    if data == "gamma":  # non-negative integers 0..255, heavy tail, about 40 % zeros
        return z.mul_(z).mul_(7.27 / 2.0).floor_().clamp_(max=255.0)
    z.mul_(torch.rsqrt(1.0 + torch.arange(d, dtype=torch.float32, device=z.device) / 8.0))
    return z.div_(z.norm(dim=1, keepdim=True).clamp_(min=1e-20))


def _split(d, nbits):
    """Dimensions in proportion to the bits, leftovers to the first sub-quantizers."""
    B = sum(nbits)
    ds = [(d * b) // B for b in nbits]
    for j in range(d - sum(ds)):
        ds[j % len(ds)] += 1
    return ds


def _codebooks(sample, nbits, dsub, iters=5):
    """k-means per sub-space on the host in float64; concatenated float32."""
    x = sample.cpu().numpy().astype(np.float64)
    parts, o = [], 0
    for b, s in zip(nbits, dsub):
        k, xs = 1 << b, x[:, o:o + s]
        c = xs[:k].copy()
        for _ in range(iters):
            a = np.argmin((c * c).sum(1)[None, :] - 2.0 * (xs @ c.T), axis=1)
            cnt = np.bincount(a, minlength=k)
            for l in range(s):
                tot = np.bincount(a, weights=xs[:, l], minlength=k)
                c[:, l] = np.where(cnt > 0, tot / np.maximum(cnt, 1), c[:, l])
        parts.append(c.astype(np.float32).reshape(-1))
        o += s
    return torch.from_numpy(np.concatenate(parts)).to(sample.device)


def _encode(x, nbits, dsub, codebooks):
    """Packed codes (little-endian bit stream) of the rows of x: nearest centroid per sub-space."""
    cs = (sum(nbits) + 7) // 8
    out = torch.zeros((x.shape[0], cs), dtype=torch.uint8, device=x.device)
    o = cb = off = 0
    for b, s in zip(nbits, dsub):
        k = 1 << b
        c = codebooks[cb:cb + k * s].reshape(k, s)
        sub = torch.argmin(torch.addmm((c * c).sum(1), x[:, o:o + s], c.t(), alpha=-2.0), dim=1).to(torch.int16)
        sh = off & 7
        out[:, off >> 3] |= ((sub << sh) & 255).to(torch.uint8)
        if sh + b > 8:
            out[:, (off >> 3) + 1] |= (sub >> (8 - sh)).to(torch.uint8)
        o, cb, off = o + s, cb + k * s, off + b
    return out


CHUNK = 1 << 20


def _flat_inputs(case, seed):
    nbits, acc = LAYOUTS[case["layout"]]
    d, n = case["d"], case["n"]
    dsub = _split(d, nbits)
    cb = _codebooks(_vectors(case["data"], 8192, d, seed, 1), nbits, dsub)
    s = dict(nbits=nbits, acc=acc, dsub=dsub, codebooks=cb)
    if case["path"] == "encode":
        x = torch.empty((n, d), dtype=torch.float32, device=_dev())
        for c, lo in enumerate(range(0, n, CHUNK)):
            hi = min(n, lo + CHUNK)
            x[lo:hi] = _vectors(case["data"], hi - lo, d, seed, 100 + c)
        s["vectors"] = x
        return s
    codes = torch.empty((n, (sum(nbits) + 7) // 8), dtype=torch.uint8, device=_dev())
    for c, lo in enumerate(range(0, n, CHUNK)):
        hi = min(n, lo + CHUNK)
        codes[lo:hi] = _encode(_vectors(case["data"], hi - lo, d, seed, 100 + c), nbits, dsub, cb)
    s["codes"] = codes
    s["queries"] = _vectors(case["data"], case["nq"], d, seed, 2)
    return s


def _ivf_inputs(case, seed):
    """Cells, residual codebooks and list sizes from an assigned sample; every list's codes are
    drawn from the sample's encoded residuals."""
    nbits, acc = LAYOUTS[case["layout"]]
    d, n, K = case["d"], case["n"], case["K"]
    dsub = _split(d, nbits)
    coarse = _vectors(case["data"], K, d, seed, 3)
    pool = _vectors(case["data"], 1 << 18, d, seed, 4)
    cn = (coarse * coarse).sum(1)
    assign = torch.empty(pool.shape[0], dtype=torch.int64, device=pool.device)
    step = max(256, min(1 << 16, (1 << 29) // K))
    for lo in range(0, pool.shape[0], step):
        assign[lo:lo + step] = torch.argmin(torch.addmm(cn, pool[lo:lo + step], coarse.t(), alpha=-2.0), dim=1)
    res = pool - coarse[assign]
    cb = _codebooks(res[:8192], nbits, dsub)
    pool_codes = _encode(res, nbits, dsub, cb)
    w = torch.bincount(assign, minlength=K).double() + 0.5
    sizes = torch.floor(w * (n / float(w.sum()))).to(torch.int64)
    sizes[: n - int(sizes.sum())] += 1  # fewer than K codes are left over
    offsets = torch.zeros(K + 1, dtype=torch.int64, device=pool.device)
    offsets[1:] = torch.cumsum(sizes, 0)
    g = _gen(seed, 5, _dev())
    codes = torch.empty((n, pool_codes.shape[1]), dtype=torch.uint8, device=pool.device)
    big = 1 << 24
    for lo in range(0, n, big):
        hi = min(n, lo + big)
        codes[lo:hi] = pool_codes[torch.randint(0, pool.shape[0], (hi - lo,), generator=g, device=pool.device)]
    ids = torch.randperm(n, generator=g, device=pool.device, dtype=torch.int32)
    return dict(nbits=nbits, acc=acc, dsub=dsub, codebooks=cb, coarse=coarse, offsets=offsets, codes=codes, ids=ids,
                queries=_vectors(case["data"], case["nq"], d, seed, 2))


def prepare(case, seed):
    s = (_ivf_inputs if case["path"].startswith("ivf") else _flat_inputs)(case, seed)
    dev, nq, R, n = _dev(), case["nq"], case["R"], case["n"]
    s["path"], s["R"] = case["path"], R
    s["idx"] = idx = qb.PqIndex(case["d"], s["nbits"], s["dsub"], s["codebooks"], s["acc"])

    def empty(*shape, dtype):
        return torch.empty(shape, dtype=dtype, device=dev)

    if case["path"] == "encode":
        return s
    if case["path"] == "search":
        s["ws"] = empty(qb.pq_search_workspace_bytes(idx, nq, n, R), dtype=torch.uint8)
        s["out"] = (empty(nq, R, dtype=torch.int32), empty(nq, R, dtype=torch.uint16), empty(nq, R, dtype=torch.float32))
    elif case["path"] == "stages":
        s["ws"] = empty(qb.pq_workspace_bytes(idx, nq, n, R), dtype=torch.uint8)
    else:
        K, nprobe = case["K"], case["nprobe"]
        s["nprobe"] = nprobe
        need = qb.ivf_workspace_bytes(idx, nq, nprobe, R) if case["path"] == "ivf_tight" else \
            qb.ivf_sorted_workspace_bytes(idx, nq, nprobe, R, K)
        s["ws"] = empty(need, dtype=torch.uint8)
        s["cws"] = empty(qb.ivf_coarse_workspace_bytes(nq, K), dtype=torch.uint8)
        s["cout"] = (empty(nq, nprobe, dtype=torch.int32), empty(nq, nprobe, dtype=torch.float32))
        s["out"] = (empty(nq, R, dtype=torch.int32), empty(nq, R, dtype=torch.float32))
    return s


def run(s):
    path, idx, R = s["path"], s["idx"], s["R"]
    if path == "search":
        return qb.pq_search_topk(idx, s["queries"], s["codes"], T_CALIB, R, workspace=s["ws"], out=s["out"])
    if path == "stages":
        tables = qb.pq_compute_tables(idx, s["queries"])
        qtables, qparams = qb.pq_quantize_tables(idx, tables, s["codes"], T_CALIB, R)
        ids, keys, dist = qb.pq_adc_scan_topk(idx, qtables, qparams, s["codes"], R, workspace=s["ws"])
        return tables, qtables, qparams, ids, keys, dist
    if path == "encode":
        return qb.pq_encode(idx, s["vectors"])
    probe_ids, scores = qb.ivf_coarse_search(s["queries"], s["coarse"], s["nprobe"], workspace=s["cws"], out=s["cout"])
    search = qb.ivf_adc_scan_topk_tightening if path == "ivf_tight" else qb.ivf_adc_scan_topk
    ids, dist = search(idx, s["coarse"], s["offsets"], s["codes"], s["ids"], s["queries"], probe_ids, T_CALIB, R,
                       workspace=s["ws"], out=s["out"])
    return probe_ids, scores, ids, dist


def work(case):
    """Every input once, every output once; one addition per (code, sub-quantizer, query)."""
    nbits, acc = LAYOUTS[case["layout"]]
    m, cs, d, n, nq, R = len(nbits), (sum(nbits) + 7) // 8, case["d"], case["n"], case["nq"], case["R"]
    dsub = _split(d, nbits)
    cbl = sum((1 << b) * s for b, s in zip(nbits, dsub))
    T = sum(1 << b for b in nbits)
    if case["path"] == "encode":
        return {"bytes": n * (4 * d + cs) + 4 * cbl, "flops": 3.0 * n * cbl}
    if case["path"] in ("search", "stages"):
        b = n * cs + nq * 4 * d + 4 * cbl + nq * R * 10
        if case["path"] == "stages":
            b += nq * (T * (4 + acc // 8) + 24)
        return {"bytes": b, "flops": float(n) * m * nq + 3.0 * cbl * nq}
    K, nprobe = case["K"], case["nprobe"]
    touched = K * (1.0 - (1.0 - nprobe / K) ** nq)  # distinct lists of a call whose probes spread evenly
    codes = nq * nprobe * (n / K)
    return {"bytes": touched * (n / K) * cs + 4 * K * d + nq * (4 * d + R * 8 + nprobe * 8),
            "flops": 2.0 * nq * K * d + codes * m + 3.0 * cbl * nq * nprobe}


def tolerance(case):
    """Every result is defined bit for bit (fp32 terms in a stated order, integer sums, ranks with
    ties by lowest id), so another correct implementation gives the same bytes."""
    return "exact"


# ------------------------------------------------------------ in 64 bits -----
def _tables64(z, nbits, dsub, codebooks):
    """[nq, T] float64 tables of eq. (1) for the rows of z."""
    parts, o, cb = [], 0, 0
    for b, s in zip(nbits, dsub):
        k = 1 << b
        c = codebooks[cb:cb + k * s].reshape(k, s).double()
        acc = torch.zeros((z.shape[0], k), dtype=torch.float64, device=z.device)
        for l in range(s):
            acc += (z[:, o + l, None] - c[None, :, l]) ** 2
        parts.append(acc)
        o, cb = o + s, cb + k * s
    return parts


def _subcodes(codes, nbits):
    out, off = [], 0
    for b in nbits:
        byte, sh = off >> 3, off & 7
        v = codes[:, byte].to(torch.int32) >> sh
        if sh + b > 8:
            v = v | (codes[:, byte + 1].to(torch.int32) << (8 - sh))
        out.append((v & ((1 << b) - 1)).to(torch.uint8))
        off += b
    return out


def _take(tab, sub):
    """Sum over the sub-quantizers of tab[j][sub[j]]."""
    acc = tab[0][sub[0].int()]
    for j in range(1, len(tab)):
        acc = acc + tab[j][sub[j].int()]
    return acc


def _quantize(tab, dmax, qmax):
    dmin = float(sum(float(t.min()) for t in tab))
    delta = (dmax - dmin) / qmax
    if not (delta > 0.0 and math.isfinite(delta)):
        return dmin, 0.0, [torch.zeros_like(t, dtype=torch.int32) for t in tab]
    return dmin, delta, [torch.floor((t - t.min()) / delta).clamp_(max=qmax).to(torch.int32) for t in tab]


def _flat64(case, s):
    nbits, acc = s["nbits"], s["acc"]
    n, R, qmax = case["n"], case["R"], (1 << acc) - 1
    tabs = _tables64(s["queries"].double(), nbits, s["dsub"], s["codebooks"])
    sub = _subcodes(s["codes"], nbits)
    t_eff = min(n, max(T_CALIB, 4 * R))
    head = [x[:t_eff] for x in sub]
    dist = torch.empty((case["nq"], R), dtype=torch.float64, device=_dev())
    for q in range(case["nq"]):
        tab = [t[q] for t in tabs]
        dmax = float(torch.kthvalue(_take(tab, head), min(R, t_eff)).values)
        dmin, delta, qt = _quantize(tab, dmax, qmax)
        key = _take(qt, sub).clamp_(max=qmax)
        best = torch.topk(key, R, largest=False, sorted=True).values
        dist[q] = best.double() * delta + dmin
    return tabs, dist


def _ivf64(case, s):
    nbits, acc = s["nbits"], s["acc"]
    R, qmax, nprobe = case["R"], (1 << acc) - 1, case["nprobe"]
    z, cen, off = s["queries"].double(), s["coarse"].double(), s["offsets"].cpu()
    score = (cen * cen).sum(1)[None, :] - 2.0 * (z @ cen.t())
    scores, probes = torch.topk(score, nprobe, dim=1, largest=False, sorted=True)
    want = max(T_CALIB, 4 * R)
    dist = torch.full((case["nq"], R), math.inf, dtype=torch.float64, device=_dev())
    for q in range(case["nq"]):
        lists, first, seen = [], [], 0
        for c in probes[q].tolist():
            lo, hi = int(off[c]), int(off[c + 1])
            if hi == lo:
                continue
            tab = [t[0] for t in _tables64((z[q] - cen[c])[None, :], nbits, s["dsub"], s["codebooks"])]
            sub = _subcodes(s["codes"][lo:hi], nbits)
            if seen < want:
                take = min(hi - lo, want - seen)
                first.append(_take(tab, [x[:take] for x in sub]))
                seen += take
            lists.append((tab, sub))
        if not lists:
            continue
        dmax = float(torch.kthvalue(torch.cat(first), min(R, seen)).values)
        held = torch.empty(0, dtype=torch.float64, device=_dev())
        cur = dmax
        for tab, sub in lists:
            if sum(float(t.min()) for t in tab) >= cur:
                continue
            dmin, delta, qt = _quantize(tab, cur, qmax)
            key = _take(qt, sub).clamp_(max=qmax)
            if case["path"] == "ivf_tight":
                key = key[key < qmax]
            held = torch.cat([held, key.double() * delta + dmin])
            if held.numel() > R:
                held = torch.topk(held, R, largest=False).values
            if case["path"] == "ivf_tight" and held.numel() >= R:
                cur = min(cur, float(held.max()))
        held = torch.sort(held).values[:R]
        dist[q, :held.numel()] = held
    return scores, dist


def exact(case, seed):
    """Tables, scores and distances by the definitions in float64.  Ids, keys, quantized tables and
    codes are whole values decided by fp32 roundings and have no 64-bit value of their own."""
    if case["path"] == "encode" or (case["path"].startswith("ivf") and case["nq"] * case["nprobe"] > 2048):
        return None
    if not case["path"].startswith("ivf") and float(case["n"]) * case["nq"] * len(LAYOUTS[case["layout"]][0]) > 2e10:
        return None
    if case["path"].startswith("ivf"):
        scores, dist = _ivf64(case, _ivf_inputs(case, seed))
        return None, scores, None, dist
    s = _flat_inputs(case, seed)
    tabs, dist = _flat64(case, s)
    if case["path"] == "stages":
        return torch.cat(tabs, dim=1), None, None, None, None, dist
    return None, None, dist
