"""The work that is timed when this library's speed is judged: single calls
through the package's public entry points, from the smallest search to the
largest batch.

Inputs are the library's usual synthetic ones (a z-normalised Gaussian random
walk as the reference; every even query a time-warped noisy excerpt of it,
every odd one a walk of its own), made with NumPy from the seed alone.

A case's "path" names what is called:
  forward      sdtw_forward, plain launch (cost and end position per query)
  persistent   sdtw_forward with the persistent launch for uneven lengths
  pruned       sdtw_forward_pruned, threshold "tau"
  f16          sdtw_forward_f16
  u8           sdtw_forward_u8
  align        checkpointed sdtw_forward, then sdtw_align (the warp paths)
  train        sdtw (autograd) and the gradient of a weighted sum of the costs
  znorm        sdtw_znorm on raw series
"batch" queries have lengths spread over "n_lo".."n_hi" ("len_seed" draws
them; f16 pairs up equal lengths), "ref_len" is the reference's length and
"kind" the local cost (0 squared, 1 absolute).
"""
import numpy as np
import torch

import paper_2403_06931_amd as P


def _case(name, path, batch, n_lo, n_hi, ref_len, kind=0, tau=0.0, every=0, len_seed=0):
    return {"name": name, "path": path, "batch": batch, "n_lo": n_lo, "n_hi": n_hi,
            "ref_len": ref_len, "kind": kind, "tau": tau, "every": every, "len_seed": len_seed}


def listed():
    return [
        # a handful of short patterns in a short recording: the smallest
        # call, where the launch and the host path count
        _case("forward_4x64_1k", "forward", 4, 64, 64, 1024),
        # one pattern searched in a recording, answered at once
        _case("forward_1x2000_100k", "forward", 1, 2000, 2000, 100_000),
        # a small batch of patterns of different, odd lengths, absolute cost
        _case("forward_48ragged_9973", "forward", 48, 40, 900, 9973, kind=1, len_seed=3),
        # a few patterns in a very long recording, absolute cost
        _case("forward_16x500_2m", "forward", 16, 500, 500, 2_000_000, kind=1),
        # the paper's experiment: 512 queries of 2,000 samples, 100,000-sample
        # reference
        _case("forward_512x2000_100k", "forward", 512, 2000, 2000, 100_000),
        # a large batch of uneven lengths: the persistent launch
        _case("persistent_4096x250-4000_200k", "persistent", 4096, 250, 4000, 200_000,
              len_seed=5),
        # one training step (forward with checkpoints, walk-back gradients)
        _case("train_256x1000_50k", "train", 256, 1000, 1000, 50_000, every=1024),
        # a small training step, as with a short learned pattern bank
        _case("train_32x150_3k", "train", 32, 120, 180, 3001, every=256, len_seed=7),
        # search and alignment paths of a small batch
        _case("align_16x1000_50k", "align", 16, 700, 1000, 50_000, every=1024, len_seed=9),
        # the paper's own precision on the paper's shape
        _case("f16_512x2000_100k", "f16", 512, 2000, 2000, 100_000),
        # quantised search of a medium batch
        _case("u8_96x600_30k", "u8", 96, 400, 600, 30_011, len_seed=11),
        # normalising a batch of raw series before a search
        _case("znorm_4096x250-4000", "znorm", 4096, 250, 4000, 0, len_seed=13),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    path = rng.choice(["forward", "forward", "forward", "persistent", "pruned", "f16", "u8",
                       "align", "train", "znorm"])
    every = 0
    tau = 0.0
    while True:
        batch = _log_int(rng, 1, 4096)
        n_hi = _log_int(rng, 16, 4000)
        n_lo = n_hi if rng.random() < 0.4 else max(1, int(n_hi * rng.uniform(0.1, 1.0)))
        ref_len = _log_int(rng, 500, 2_000_000)
        cells = batch * 0.5 * (n_lo + n_hi) * ref_len
        # (a single query's passes run one after the other)
        serial = ref_len * -(-n_hi // 2048)
        if cells > 2e11 or serial > 1_000_000:
            continue
        if path in ("align", "train"):
            every = rng.choice([64, 256, 1024])
            total = batch * 0.5 * (n_lo + n_hi)
            # checkpoints, direction codes and partials stay within a few GB
            if total * (ref_len / every + ref_len / 256) > 1e9 or batch * ref_len > 2e8:
                continue
        break
    if path == "pruned":
        tau = round(rng.uniform(0.5, 4.0), 3)
    kind = rng.choice([0, 0, 1]) if path in ("forward", "persistent", "f16", "align",
                                             "train") else 0
    if path == "znorm":
        ref_len = 0
    c = _case("", path, batch, n_lo, n_hi, ref_len, kind, tau, every, rng.randrange(1 << 20))
    del c["name"]
    return c


def _lens(c):
    rng = np.random.default_rng(c["len_seed"])
    h = rng.integers(c["n_lo"], c["n_hi"] + 1, size=c["batch"]).astype(np.int32)
    if c["path"] == "f16":
        k = c["batch"] // 2
        h[1:2 * k:2] = h[0:2 * k:2]
    return h


def _znorm(x, h):
    """Every series of the packed binary64 batch, z-normalised."""
    off = np.concatenate([[0], np.cumsum(h[:-1].astype(np.int64))])
    n = h.astype(np.float64)
    x = x - np.repeat(np.add.reduceat(x, off) / n, h)
    s = np.sqrt(np.add.reduceat(x * x, off) / n)
    return x / np.repeat(np.where(s > 0, s, 1.0), h)


def _walks(rng, h):
    """A Gaussian random walk per series, packed."""
    x = np.cumsum(rng.standard_normal(int(h.sum(dtype=np.int64))))
    off = np.concatenate([[0], np.cumsum(h[:-1].astype(np.int64))])
    return x - np.repeat(x[off], h)


def _inputs(c, seed):
    """(queries float32 packed, lengths int32, reference float32 or None)."""
    rng = np.random.default_rng([seed, 240306931])
    h = _lens(c)
    total = int(h.sum(dtype=np.int64))
    off = np.concatenate([[0], np.cumsum(h[:-1].astype(np.int64))])
    if c["path"] == "znorm":
        # raw series as captured in different units
        scale = np.repeat(10.0 ** rng.uniform(-3.0, 3.0, h.size), h)
        shift = np.repeat(rng.uniform(-50.0, 50.0, h.size), h)
        return ((_walks(rng, h) + shift) * scale).astype(np.float32), h, None
    m = c["ref_len"]
    ref = _znorm(np.cumsum(rng.standard_normal(m)), np.array([m], np.int64))
    q = _walks(rng, h)
    # even queries: an excerpt of the reference, time-warped over 8 segments
    # by factors of 0.8 to 1.25, with noise
    i = np.arange(total) - np.repeat(off, h)
    seg = (8 * i) // np.repeat(h, h)
    step = 1.0 / rng.uniform(0.8, 1.25, (h.size, 8))
    pos = np.cumsum(step[np.repeat(np.arange(h.size), h), seg])
    pos = pos - np.repeat(pos[off], h)
    span = pos[off + h - 1]
    a = rng.uniform(0.0, 1.0, h.size) * np.maximum(m - 1 - span, 0.0)
    warped = np.interp(np.repeat(a, h) + pos, np.arange(m, dtype=np.float64), ref)
    warped = warped + rng.normal(0.0, 0.1, total)
    q = _znorm(np.where(np.repeat(np.arange(h.size) % 2 == 0, h), warped, q), h)
    return q.astype(np.float32), h, ref.astype(np.float32)


def prepare(case, seed):
    dev = torch.device("cuda")
    q, h, ref = _inputs(case, seed)
    s = {"case": case, "h": h, "q": torch.from_numpy(q).to(dev),
         "lens": torch.from_numpy(h).to(dev)}
    if ref is not None:
        s["r"] = torch.from_numpy(ref).to(dev)
    if case["path"] == "train":
        rng = np.random.default_rng([seed, 7])
        s["weights"] = torch.from_numpy(
            rng.uniform(0.5, 1.5, h.size).astype(np.float32) / h.size).to(dev)
        s["q"].requires_grad_(True)
        s["r"].requires_grad_(True)
    if case["path"] == "align":
        n = P.sdtw_checkpoint_floats(h, case["ref_len"], case["every"])
        s["ckpt"] = torch.empty(n, dtype=torch.float32, device=dev) if n else None
    return s


def run(s):
    c, h, q, lens = s["case"], s["h"], s["q"], s["lens"]
    path, kind, every = c["path"], c["kind"], c["every"]
    if path == "forward":
        return P.sdtw_forward(q, h, lens, s["r"], kind)
    if path == "persistent":
        return P.sdtw_forward(q, h, lens, s["r"], kind, flags=P.SDTW_F_PERSISTENT)
    if path == "pruned":
        return P.sdtw_forward_pruned(q, h, lens, s["r"], c["tau"])
    if path == "f16":
        return P.sdtw_forward_f16(q, h, lens, s["r"], kind)
    if path == "u8":
        return P.sdtw_forward_u8(q, h, lens, s["r"])
    if path == "align":
        cost, end = P.sdtw_forward(q, h, lens, s["r"], kind, ckpt=s["ckpt"], ckpt_every=every,
                                   flags=P.SDTW_F_CHECKPOINT)
        start, lo, hi = P.sdtw_align(q, h, lens, s["r"], kind, cost, end, s["ckpt"], every)
        return cost, end, start, lo, hi
    if path == "train":
        cost, end = P.sdtw(q, h, s["r"], kind, every, query_lens=lens)
        loss = (cost * s["weights"]).sum()
        gq, gr = torch.autograd.grad(loss, (q, s["r"]))
        return cost.detach(), end, gq, gr
    return P.sdtw_znorm(q, h, lens)


def work(case):
    """Each input read once and each output written once; per DP cell a
    difference, a product (not with absolute cost), two comparisons and a sum."""
    h = _lens(case)
    total, b, m = int(h.sum(dtype=np.int64)), h.size, case["ref_len"]
    path = case["path"]
    if path == "znorm":
        return {"bytes": 8 * total, "flops": 6 * total}
    nbytes = 4 * total + 4 * b + 4 * m + 12 * b
    flops = (4 if case["kind"] == 1 else 5) * total * m
    if path == "train":
        nbytes += 4 * total + 4 * m + 4 * b
    if path == "align":
        nbytes += 8 * total + 8 * b
    return {"bytes": nbytes, "flops": flops}


def _dp64(q, h, r, kind, tau=None):
    """Minimum of the last row of every query in binary64, by anti-diagonals:
    d[:, i] holds D(i, s - i) on diagonal s."""
    dev = torch.device("cuda")
    b, n, m = h.size, int(h.max()), r.size
    off = np.concatenate([[0], np.cumsum(h[:-1].astype(np.int64))])
    qp = np.zeros((b, n))
    for k in range(b):
        qp[k, :h[k]] = q[off[k]:off[k] + h[k]]
    inf = float("inf")
    qd = torch.from_numpy(qp).to(dev)
    # reversed reference, +inf outside it: rr[m + n - j] = r_j
    rr = torch.full((m + 2 * n + 1,), inf, dtype=torch.float64, device=dev)
    rr[n:n + m] = torch.from_numpy(r.astype(np.float64)[::-1].copy()).to(dev)
    d = [torch.full((b, n + 1), inf, dtype=torch.float64, device=dev) for _ in range(3)]
    for x in d:
        x[:, 0] = 0.0
    c, mn = torch.empty_like(qd), torch.empty_like(qd)
    at = torch.from_numpy(h.astype(np.int64)).to(dev)[:, None]
    best = torch.full((b, 1), inf, dtype=torch.float64, device=dev)
    for s in range(2, n + m + 1):
        k = n + m - s + 1                       # row 1's column s - 1
        torch.sub(qd, rr[k:k + n], out=c)
        c.abs_()
        if kind == 0:
            if tau is not None:
                far = c > tau
            c.mul_(c)
            if tau is not None:
                c.masked_fill_(far, inf)
        torch.minimum(d[0][:, :-1], d[0][:, 1:], out=mn)
        torch.minimum(mn, d[1][:, :-1], out=mn)
        torch.add(mn, c, out=d[2][:, 1:])
        torch.minimum(best, d[2].gather(1, at), out=best)
        d = [d[2], d[0], d[1]]
    return best[:, 0]


def exact(case, seed):
    q, h, r = _inputs(case, seed)
    path = case["path"]
    if path == "znorm":
        return torch.from_numpy(_znorm(q.astype(np.float64), h))
    n, m, b = int(h.max()), r.size, h.size
    if n + m > 110_000 or (n + m) * b * n > 1.2e11:
        return None
    if path == "u8":
        lo, hi = max(float(r.min()), -4.0), min(float(r.max()), 4.0)
        scale = 255.0 / (hi - lo) if hi > lo else 0.0
        q, r = (np.clip(np.rint((x.astype(np.float64) - lo) * scale), 0, 255) for x in (q, r))
        return _dp64(q, h, r, 0), None, torch.tensor([lo, hi], dtype=torch.float64)
    cost = _dp64(q, h, r, case["kind"], case["tau"] if path == "pruned" else None)
    return (cost,) + (None,) * {"align": 4, "train": 3}.get(path, 1)
