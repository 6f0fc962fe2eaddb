"""The work that users of this library have it do, as cases that can be timed and compared.

A case goes through the public entry points of `paper_1704_07355_amd` as a program of a user does:
the database, the codebooks, the index and the workspace are in hand before the call (`prepare`),
a pass (`run`) is what is repeated for every query, batch of queries or batch of vectors.

Six kinds of work:

  search  exhaustive Quick ADC search of one query or a batch over 4-bit codes (qadc_search), with
          the rotation of an optimized product quantizer before it where `opq` is set
  ivf     non-exhaustive search of an inverted index (qadc_ivf_search)
  multi   the same with a multi-index over its occupied cells as the partition
          (qadc_multi_index_probes, _slots, qadc_ivf_search)
  adc     the three steps as separate calls (qadc_build_luts, qadc_quantize_luts, qadc_scan_topk):
          the float ADC baseline with 8- and 4-bit codes, and uint8 tables with 8- and 6-bit codes
  build   an inverted index from raw vectors (qadc_ivf_assign, _group, _encode)
  train   codebooks by k-means and the codes of a database (qadc_pq_train, qadc_pq_encode)

Inputs: a 64-component Gaussian mixture in the range of 8-bit image descriptors, lists with
Zipf(0.8) sizes, queries around the centroids of size-weighted cells.
"""

import math

import numpy as np
import torch

import paper_1704_07355_amd as Q

ROWS = 1 << 20          # vectors generated at a time
SIGMA = 18.0            # spread of the vectors of a cell around its centroid
ROW_BYTES = {16: lambda m: m // 2, 64: lambda m: 3 * m // 4, 256: lambda m: m}
VARIANTS = {            # kind "adc": (scan variant, centroids per sub-quantizer)
    "f32_8bit": (Q.QADC_F32_8BIT, 256),
    "f32_4bit": (Q.QADC_F32_4BIT, 16),
    "u8_8bit": (Q.QADC_U8_8BIT, 256),
    "u8_6bit": (Q.QADC_U8_6BIT, 64),
}
WORKSPACES = {"f32_8bit": Q.QADC_WS_SCAN_F32_8BIT, "f32_4bit": Q.QADC_WS_SCAN_F32_4BIT,
              "u8_8bit": Q.QADC_WS_SCAN_U8_8BIT, "u8_6bit": Q.QADC_WS_SCAN_U8_6BIT}


# ---------------------------------------------------------------------------------------------
# cases

def _search(n, d, m, nq, R=100, init=200, nbins=255, qmin=0, opq=False):
    return {"kind": "search", "n": n, "d": d, "m": m, "nq": nq, "R": R, "init": init, "nbins": nbins,
            "qmin": qmin, "opq": opq}


def _ivf(n, K, d, m, nq, nprobe, R=100, init=1000):
    return {"kind": "ivf", "n": n, "K": K, "d": d, "m": m, "nq": nq, "nprobe": nprobe, "R": R, "init": init}


def _multi(n, kh, d, m, nq, nprobe, R=100, init=1000):
    return {"kind": "multi", "n": n, "kh": kh, "d": d, "m": m, "nq": nq, "nprobe": nprobe, "R": R, "init": init}


def _adc(variant, n, d, m, nq, R=100, init=200):
    return {"kind": "adc", "variant": variant, "n": n, "d": d, "m": m, "nq": nq, "R": R, "init": init}


def _build(n, K, d, m):
    return {"kind": "build", "n": n, "K": K, "d": d, "m": m}


def _train(train_n, d, m, ksub, n, iters=10):
    return {"kind": "train", "train_n": train_n, "d": d, "m": m, "ksub": ksub, "iters": iters, "n": n}


def listed():
    cases = [
        # a handful of queries over a database that fits a cache: launches and latency count
        ("search_16q_100k", _search(100_000, 128, 16, 16)),
        # the library's headline: one query at a time over 10 M 64-bit codes
        ("search_1q_10m", _search(10_000_000, 128, 16, 1)),
        # a 960-dimensional global descriptor in 128-bit codes behind an OPQ rotation, one query
        ("search_opq_1q_1m_960d", _search(1_000_000, 960, 32, 1, opq=True)),
        # a throughput job: batches of 256 queries over 100 M 128-bit codes
        ("search_256q_100m", _search(100_000_000, 128, 32, 256, init=1000)),
        # a web request's dozen of queries over 256-bit codes, a ragged size, the paper's signed bytes
        ("search_12q_3m_ragged", _search(3_000_017, 256, 64, 12, R=37, init=333, nbins=127, qmin=1)),
        # response time of one query against an index of 100 M codes
        ("ivf_1q_100m", _ivf(100_000_000, 65536, 128, 32, 1, 64)),
        # serving a billion codes, large batches
        ("ivf_4096q_1b", _ivf(1_000_000_000, 65536, 128, 32, 4096, 64)),
        # the small inverted index of the paper, a mid-sized batch of an odd size
        ("ivf_150q_1m", _ivf(1_000_000, 256, 128, 16, 150, 24, init=200)),
        # a multi-index over its occupied cells
        ("multi_512q_100m", _multi(100_000_000, 4096, 128, 32, 512, 64)),
        # the float ADC baseline with 8-bit components, one query
        ("adc_f32_8bit_1q_50m", _adc("f32_8bit", 50_000_000, 96, 8, 1)),
        # an inverted index from a million raw vectors
        ("build_1m_4096", _build(1_000_003, 4096, 128, 32)),
        # a product quantizer from a learning set, and the codes of a database
        ("train_20k_encode_2m", _train(20_000, 128, 16, 16, 2_000_003)),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "ivf", "ivf", "ivf", "multi", "adc", "build", "train"])
    d = rng.choice([64, 96, 128, 128, 256])
    R = rng.choice([1, 10, 100, 100, 100, 200, 1000])
    if kind == "search":
        m = rng.choice([8, 16, 16, 32, 32, 64])
        nq = rng.choice([1, 1, _log(rng, 2, 256)])
        n = _log(rng, 20_000, 100_000_000)
        n = max(20_000, min(n, int(3e11 / (m * nq)), 400_000_000 // m))
        return _search(n, d, m, nq, R, rng.choice([100, 200, 1000]), rng.choice([255, 255, 127]),
                       rng.choice([0, 0, 1]), rng.random() < 0.2)
    if kind == "ivf":
        K = rng.choice([256, 1000, 4096, 16384, 65536])
        n = max(1_000_000, K * _log(rng, 500, 8000))
        nprobe = rng.choice([8, 24, 64, 100])
        m = rng.choice([16, 32, 32])
        nq = rng.choice([1, _log(rng, 2, 64), _log(rng, 65, 4096)])
        nq = max(1, min(nq, int(5e10 / (nprobe * (n // K) * m))))
        return _ivf(n, K, d, m, nq, nprobe, min(R, 200), rng.choice([200, 1000]))
    if kind == "multi":
        kh = rng.choice([512, 1024, 4096])
        return _multi(_log(rng, 5_000_000, 100_000_000), kh, d, rng.choice([16, 32]), _log(rng, 1, 1024), 64, min(R, 200))
    if kind == "adc":
        variant = rng.choice(sorted(VARIANTS))
        m = rng.choice([16, 32]) if variant == "f32_4bit" else rng.choice([8, 16])
        nq = rng.choice([1, 1, _log(rng, 2, 64)])
        n = max(100_000, min(_log(rng, 100_000, 50_000_000), int(6e9 / (m * nq))))
        return _adc(variant, n, rng.choice([96, 128]), m, nq, min(R, 200), 200)
    if kind == "build":
        K = rng.choice([256, 1000, 4096, 16384])
        n = min(_log(rng, 50_000, 2_000_000), int(4e11 / (K * d)))
        return _build(n, K, d, rng.choice([16, 32]))
    ksub = rng.choice([16, 16, 64, 256])
    return _train(rng.choice([5_000, 20_000]), d, 16 if ksub == 16 else 8, ksub, _log(rng, 50_000, 2_000_000))


# ---------------------------------------------------------------------------------------------
# inputs

def _device():
    return torch.device("cuda:0")


def _gen(seed, salt):
    g = torch.Generator(device=_device())
    g.manual_seed((int(seed) * 64 + salt) & ((1 << 62) - 1))
    return g


def _means(seed, d):
    """Means of the mixture's components, f32 [64][d]."""
    return (48.0 + 32.0 * torch.randn((64, d), generator=_gen(seed, 0), device=_device())).clamp_(0.0, 255.0)


def _mixture(means, n, g):
    label = torch.randint(0, means.shape[0], (n,), generator=g, device=means.device)
    x = torch.randn((n, means.shape[1]), generator=g, device=means.device).mul_(24.0)
    return x.add_(means[label]).clamp_(0.0, 255.0)


def _rows(seed, n, k):
    return torch.randperm(n, generator=_gen(seed, 1), device=_device())[:k].contiguous()


def _rotation(seed, d):
    g = np.random.default_rng([int(seed), d])
    q, r = np.linalg.qr(g.standard_normal((d, d)))
    return torch.from_numpy((q * np.sign(np.diag(r))).astype(np.float32)).to(_device())


def _encoded(seed, cb, means, n, rot=None):
    """The codes of n vectors of the mixture."""
    m, ksub, _ = cb.shape
    codes = torch.empty((n, ROW_BYTES[ksub](m)), dtype=torch.uint8, device=_device())
    g = _gen(seed, 2)
    for s in range(0, n, ROWS):
        x = _mixture(means, min(ROWS, n - s), g)
        Q.qadc_pq_encode(cb, x if rot is None else Q.qadc_rotate(rot, x), out=codes[s:s + ROWS])
    return codes


def _residual_codes(seed, n, d, m):
    """A residual quantizer and the codes of n residuals."""
    learn = SIGMA * torch.randn((20_000, d), generator=_gen(seed, 3), device=_device())
    cb = Q.qadc_pq_train(learn, m, 16, _rows(seed, 20_000, 16), 10)
    codes = torch.empty((n, m // 2), dtype=torch.uint8, device=_device())
    g = _gen(seed, 4)
    for s in range(0, n, ROWS):
        cnt = min(ROWS, n - s)
        Q.qadc_pq_encode(cb, torch.randn((cnt, d), generator=g, device=_device()).mul_(SIGMA), out=codes[s:s + cnt])
    return cb, codes


def _zipf(n, K, seed=None):
    """Sizes of K lists, Zipf(0.8), summing to n; in a seeded order."""
    w = np.arange(1, K + 1, dtype=np.float64) ** -0.8
    sizes = np.floor(n * w / w.sum()).astype(np.int64)
    sizes[0] += n - sizes.sum()
    return sizes if seed is None else sizes[np.random.default_rng([int(seed), K]).permutation(K)]


def _workspace(nbytes):
    return Q.qadc_workspace_init(torch.empty((max(256, nbytes),), dtype=torch.uint8, device=_device()))


def _outputs(nq, R, dtype=torch.uint8):
    return (torch.empty((nq, R), dtype=torch.int32, device=_device()),
            torch.empty((nq, R), dtype=dtype, device=_device()))


def prepare(case, seed):
    c = dict(case)
    kind, d, m, n = c["kind"], c["d"], c["m"], c["n"]
    s = {"case": c}
    if kind in ("search", "adc"):
        ksub = 16 if kind == "search" else VARIANTS[c["variant"]][1]
        means = _means(seed, d)
        rot = _rotation(seed, d) if c.get("opq") else None
        learn = _mixture(means, 20_000, _gen(seed, 5))
        if rot is not None:
            learn = Q.qadc_rotate(rot, learn)
        s["cb"] = Q.qadc_pq_train(learn, m, ksub, _rows(seed, 20_000, ksub), 10)
        s["codes"] = _encoded(seed, s["cb"], means, n, rot)
        s["queries"] = _mixture(means, c["nq"], _gen(seed, 6))
        s["rot"] = rot
        if kind == "search":
            s["ws"] = _workspace(Q.qadc_workspace_bytes(Q.QADC_WS_SEARCH, n, m, c["nq"], c["R"]))
            s["out"] = _outputs(c["nq"], c["R"])
        else:
            s["ws"] = _workspace(Q.qadc_workspace_bytes(WORKSPACES[c["variant"]], n, m, c["nq"], c["R"]))
            s["out"] = _outputs(c["nq"], c["R"], torch.float32 if c["variant"].startswith("f32") else torch.uint8)
        return s
    if kind == "ivf":
        K = c["K"]
        coarse = _mixture(_means(seed, d), K, _gen(seed, 7))
        sizes = _zipf(n, K, seed)
        off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)])).to(_device())
        cb, codes = _residual_codes(seed, n, d, m)
        ids = torch.arange(n, dtype=torch.int32, device=_device())
        s["index"] = Q.IvfIndex(coarse, off, codes, ids, cb)
        g = _gen(seed, 8)
        home = torch.multinomial(torch.from_numpy(sizes / sizes.sum()).to(_device()), c["nq"], True, generator=g)
        s["queries"] = coarse[home] + SIGMA * torch.randn((c["nq"], d), generator=g, device=_device())
        s["ws"] = _workspace(Q.qadc_ivf_workspace_bytes(s["index"], c["nq"], c["nprobe"], c["R"]))
        return s
    if kind == "multi":
        kh, nq = c["kh"], c["nq"]
        means = _means(seed, d)
        g = _gen(seed, 7)
        x = _mixture(means, 2 * kh, g)
        halves = torch.stack([x[:kh, :d // 2], x[kh:, d // 2:]]).contiguous()
        homes = _mixture(means, max(4096, n // 2048), g)
        pool = torch.cat([Q.qadc_multi_index_probes(halves, homes[i:i + 8192].contiguous(), 4).reshape(-1)
                          for i in range(0, homes.shape[0], 8192)])
        cells = pool[torch.randint(0, pool.numel(), (n,), generator=g, device=_device())]
        cell_ids, off, ids = Q.qadc_multi_index_group(cells, kh)
        cb, codes = _residual_codes(seed, n, d, m)
        s["index"] = Q.IvfIndex(None, off, codes, ids, cb, halves=halves, cell_ids=cell_ids)
        s["halves"], s["cell_ids"] = halves, cell_ids
        pick = torch.randint(0, homes.shape[0], (nq,), generator=g, device=_device())
        s["queries"] = homes[pick] + SIGMA * torch.randn((nq, d), generator=g, device=_device())
        s["mws"] = torch.empty((Q.qadc_multi_index_workspace_bytes(kh, nq, c["nprobe"]),), dtype=torch.uint8,
                               device=_device())
        s["ws"] = _workspace(Q.qadc_ivf_workspace_bytes(s["index"], nq, c["nprobe"], c["R"]))
        return s
    if kind == "build":
        K = c["K"]
        s["coarse"] = _mixture(_means(seed, d), K, _gen(seed, 7))
        sizes = _zipf(n, K, seed)
        g = _gen(seed, 8)
        home = torch.multinomial(torch.from_numpy(sizes / sizes.sum()).to(_device()), n, True, generator=g)
        s["x"] = s["coarse"][home] + SIGMA * torch.randn((n, d), generator=g, device=_device())
        learn = SIGMA * torch.randn((20_000, d), generator=g, device=_device())
        s["cb"] = Q.qadc_pq_train(learn, m, 16, _rows(seed, 20_000, 16), 10)
        s["ws"] = torch.empty((max(16, Q.qadc_ivf_group_workspace_bytes(n, K)),), dtype=torch.uint8, device=_device())
        return s
    means = _means(seed, d)
    s["learn"] = _mixture(means, c["train_n"], _gen(seed, 5))
    s["rows"] = _rows(seed, c["train_n"], c["ksub"])
    s["x"] = _mixture(means, n, _gen(seed, 6))
    return s


# ---------------------------------------------------------------------------------------------
# one pass

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "search":
        q = s["queries"] if s["rot"] is None else Q.qadc_rotate(s["rot"], s["queries"])
        return Q.qadc_search(s["cb"], q, s["codes"], c["R"], c["init"], nbins=c["nbins"], qmin_mode=c["qmin"],
                             workspace=s["ws"], out_idx=s["out"][0], out_dist=s["out"][1])
    if kind == "ivf":
        return Q.qadc_ivf_search(s["index"], s["queries"], c["nprobe"], c["R"], c["init"], workspace=s["ws"])
    if kind == "multi":
        cells = Q.qadc_multi_index_probes(s["halves"], s["queries"], c["nprobe"], workspace=s["mws"])
        slots = Q.qadc_multi_index_slots(s["cell_ids"], cells)
        ids, dist = Q.qadc_ivf_search(s["index"], s["queries"], c["nprobe"], c["R"], c["init"], probes_in=slots,
                                      workspace=s["ws"])
        return cells, ids, dist
    if kind == "adc":
        variant = VARIANTS[c["variant"]][0]
        luts = Q.qadc_build_luts(s["cb"], s["queries"])
        if c["variant"].startswith("f32"):
            idx, dist = Q.qadc_scan_topk(variant, s["codes"], luts, c["R"], workspace=s["ws"], out_idx=s["out"][0],
                                         out_dist=s["out"][1])
            return luts, idx, dist
        qluts, bias, delta, qmax = Q.qadc_quantize_luts(luts, s["codes"][:c["init"]], c["R"])
        idx, dist = Q.qadc_scan_topk(variant, s["codes"], qluts, c["R"], workspace=s["ws"], out_idx=s["out"][0],
                                     out_dist=s["out"][1])
        return luts, qluts, bias, delta, qmax, idx, dist
    if kind == "build":
        cells = Q.qadc_ivf_assign(s["coarse"], s["x"])
        off, ids = Q.qadc_ivf_group(cells, c["K"], workspace=s["ws"])
        codes = Q.qadc_ivf_encode(s["coarse"], s["cb"], s["x"], cells, ids)
        return cells, off, ids, codes
    cb = Q.qadc_pq_train(s["learn"], c["m"], c["ksub"], s["rows"], c["iters"])
    return cb, Q.qadc_pq_encode(cb, s["x"])


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    """Each input read once, each output written once; operations: a lookup and an addition per component of a
    (code, query) pair count as one, distances count a subtraction and a fused multiply-add per component."""
    c = case
    kind, d, m, n = c["kind"], c["d"], c["m"], c["n"]
    if kind in ("search", "adc"):
        nq, R = c["nq"], c["R"]
        ksub = 16 if kind == "search" else VARIANTS[c["variant"]][1]
        out = nq * R * (8 if c.get("variant", "").startswith("f32") else 5)
        rot = 4 * d * d if c.get("opq") else 0
        return {"bytes": n * ROW_BYTES[ksub](m) + 4 * ksub * d + 4 * nq * d + rot + out,
                "flops": float(n) * m * nq + 3.0 * nq * ksub * d + 2.0 * nq * (rot // 4)}
    if kind in ("ivf", "multi"):
        nq, nprobe, R = c["nq"], c["nprobe"], c["R"]
        if kind == "ivf":
            K = c["K"]
            sizes = _zipf(n, K).astype(np.float64)
            share = np.minimum(1.0, sizes / n + (nprobe - 1.0) / K)  # chance of a cell to be probed by a query
            pairs = nq * float((sizes * share).sum())
            codes = float((sizes * (1.0 - (1.0 - share) ** nq)).sum())
            index_bytes, index_flops = 4.0 * K * d, 3.0 * nq * K * d
        else:
            pairs = nq * 48.0 * 512.0  # occupied cells of 64 probed, codes of an occupied cell
            codes = min(float(n), pairs)
            index_bytes, index_flops = 4.0 * c["kh"] * d, 3.0 * nq * c["kh"] * d
        return {"bytes": index_bytes + codes * (m // 2) + 4.0 * nq * d + 5.0 * nq * R,
                "flops": index_flops + pairs * m + 3.0 * nq * nprobe * 16 * d}
    if kind == "build":
        K = c["K"]
        return {"bytes": 4.0 * n * d + 4.0 * K * d + n * (4 + 4 + m // 2) + 8.0 * K,
                "flops": 3.0 * n * K * d + 3.0 * n * 16 * d}
    return {"bytes": 4.0 * n * d + 4.0 * c["train_n"] * d + n * ROW_BYTES[c["ksub"]](m) + 4.0 * c["ksub"] * d,
            "flops": 3.0 * c["ksub"] * d * (n + c["iters"] * c["train_n"])}


def tolerance(case):
    """Sums, ids, cells and codes are whole numbers with one right answer under the stated tie order, and the float
    steps before them have a stated order; only float outputs have room, for the last bit of a float32."""
    if case["kind"] in ("adc", "train"):
        return {"rel": 2e-7, "max": 1e-6}
    return "exact"


# ---------------------------------------------------------------------------------------------
# the same in 64 bits

def _exact_luts(cb, q):
    m, _, dsub = cb.shape
    y = q.double().reshape(q.shape[0], m, 1, dsub)
    return ((y - cb.double()[None]) ** 2).sum(3)


def _fields(codes, m, ksub):
    """Components of a block of codes, int64 [n][m]."""
    if ksub == 256:
        return codes.long()
    if ksub == 16:
        return torch.stack([codes & 15, codes >> 4], 2).reshape(codes.shape[0], m).long()
    b = codes.reshape(codes.shape[0], m // 4, 3).long()
    v = b[..., 0] | (b[..., 1] << 8) | (b[..., 2] << 16)
    return torch.stack([(v >> (6 * k)) & 63 for k in range(4)], 2).reshape(codes.shape[0], m)


def _sums(luts, codes, ksub):
    """Sums of one query's tables f64 [m][ksub] over a block of codes."""
    f = _fields(codes, luts.shape[0], ksub)
    total = torch.zeros(codes.shape[0], dtype=torch.float64, device=codes.device)
    for j in range(luts.shape[0]):
        total += luts[j][f[:, j]]
    return total


def exact(case, seed):
    if case["kind"] == "adc":
        s = prepare(case, seed)
        c = s["case"]
        ksub, nq, R = VARIANTS[c["variant"]][1], c["nq"], c["R"]
        luts = _exact_luts(s["cb"], s["queries"])
        if c["variant"].startswith("f32"):
            if c["n"] * c["nq"] > 400_000_000:
                return luts, None, None
            dist = torch.full((nq, R), math.inf, dtype=torch.float64, device=luts.device)
            for i in range(0, c["n"], 1 << 24):
                for q in range(nq):
                    v = torch.cat([dist[q], _sums(luts[q], s["codes"][i:i + (1 << 24)], ksub)])
                    dist[q] = torch.topk(v, R, largest=False, sorted=True).values
            return luts, None, dist
        bias = luts.amin(2)
        first = torch.stack([_sums(luts[q], s["codes"][:c["init"]], ksub) for q in range(nq)])
        qmax = first.sort(1).values[:, min(R, first.shape[1]) - 1]
        return luts, None, bias, (qmax - bias.sum(1)) / 255.0, qmax, None, None
    if case["kind"] == "train":
        # Lloyd's iterations in 64 bits; the centroids are held in 32 bits between them, as the definition says
        s = prepare(case, seed)
        c = s["case"]
        n, d, m, ksub = c["train_n"], c["d"], c["m"], c["ksub"]
        x = s["learn"].double().reshape(n, m, d // m).transpose(0, 1).contiguous()
        cb = x[:, s["rows"]].clone()
        for it in range(c["iters"]):
            for j in range(m):
                own = ((x[j][:, None] - cb[j][None]) ** 2).sum(2).argmin(1)
                hot = torch.nn.functional.one_hot(own, ksub).double()
                count = hot.sum(0)
                mean = (hot.T @ x[j]) / count.clamp(min=1.0)[:, None]
                if it + 1 < c["iters"]:
                    mean = mean.float().double()
                cb[j] = torch.where(count[:, None] > 0, mean, cb[j])
        return cb, None
    return None
