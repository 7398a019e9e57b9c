"""Timed cases: what a program that uses this package has it do.

Texts are EST-shaped DNA (log-normal records of mean 500, 1 % N, a newline
after each record) and pattern sets are text windows plus uniform ACGT
strings, as in the repository's benchmark and tests; everything is drawn from
the seed on the GPU. Kinds of cases:

  oneshot  ``mpm.scan`` on a text, default variant: buffers, launch and wait
           included (interactive use, small files);
  scan     ``Scanner.scan_async`` on kept buffers under the benchmark's launch
           shape: large texts against one set, sparse lists;
  dense    the same with MPM_VARIANT_DENSE: short patterns against a large
           set, about one pair per position;
  counts   a default-variant scan and the per-pattern counts of its list;
  mixed    one scan with patterns of different lengths;
  batch    many texts, several sets, one replayed graph;
  host     a text in pinned host memory streamed through the device.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_1407_2889_amd as mpm
from paper_1407_2889_amd.batch import BatchScan

KiB, MiB = 1 << 10, 1 << 20
SHAPE = dict(lane_bytes=1024, block_threads=1024)  # the benchmark's launch shape


def listed():
    return [
        # one small request, as an interactive caller makes: latency and launches
        dict(name="oneshot_ac_4k", kind="oneshot", algo="ac", n=4 * KiB + 3, d=100, m=8),
        # an ordinary file of odd size, everything allocated per call
        dict(name="oneshot_wm_3m", kind="oneshot", algo="wm", n=3_000_017, d=800, m=12),
        # the benchmark's text and set, either index
        dict(name="scan_ac_256m", kind="scan", algo="ac", n=256 * MiB, d=1000, m=16),
        dict(name="scan_wm_256m", kind="scan", algo="wm", n=256 * MiB, d=1000, m=16),
        # sets whose tables outgrow the LDS (the sweep's rows, smaller texts)
        dict(name="scan_ac_10k", kind="scan", algo="ac", n=128 * MiB, d=10_000, m=16),
        dict(name="scan_wm_100k", kind="scan", algo="wm", n=64 * MiB + 12_345, d=100_000, m=16),
        # more than one pair per position: the densest list of the sweep
        dict(name="dense_ac_100k", kind="dense", algo="ac", n=64 * MiB, d=100_000, m=8),
        # short windows, a list of a million pairs, and its per-pattern counts
        dict(name="counts_wm_m8", kind="counts", algo="wm", n=64 * MiB, d=1000, m=8),
        # patterns of lengths 8 to 32, either index
        dict(name="mixed_ac_128m", kind="mixed", algo="ac", n=128 * MiB, d=1000, lo=8, hi=32),
        dict(name="mixed_wm_32m", kind="mixed", algo="wm", n=32 * MiB + 7, d=1000, lo=8, hi=32),
        # a batch of requests: log-uniform text lengths, sets of all sizes
        dict(name="batch_256", kind="batch", texts=256, sets=8, max_len=4 * MiB, d_hi=20_000),
        # text kept in host memory: bound by the link
        dict(name="host_ac_64m", kind="host", algo="ac", n=64 * MiB, d=1000, m=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["oneshot", "oneshot", "scan", "scan", "scan", "dense", "counts", "mixed",
                       "batch", "host"])
    algo = rng.choice(["ac", "wm"])
    m = rng.choice([8, 12, 16, 24, 32])
    if kind == "oneshot":
        return dict(kind=kind, algo=algo, n=_log(rng, KiB, 16 * MiB), d=_log(rng, 100, 10_000), m=m)
    if kind == "scan":
        m = rng.choice([12, 16, 24, 32])
        d = _log(rng, 100, 100_000 if algo == "wm" or m <= 16 else 20_000)
        return dict(kind=kind, algo=algo, n=_log(rng, 4 * MiB, (256 if d <= 10_000 else 64) * MiB),
                    d=d, m=m)
    if kind == "dense":
        return dict(kind=kind, algo=algo, n=_log(rng, 4 * MiB, (64 if algo == "ac" else 16) * MiB),
                    d=_log(rng, 10_000, 100_000), m=8)
    if kind == "counts":
        return dict(kind=kind, algo=algo, n=_log(rng, 4 * MiB, 64 * MiB), d=_log(rng, 100, 10_000),
                    m=rng.choice([8, 12, 16]))
    if kind == "mixed":
        lo = rng.choice([8, 12])
        return dict(kind=kind, algo=algo, n=_log(rng, MiB, (128 if algo == "ac" else 32) * MiB),
                    d=_log(rng, 100, 1000), lo=lo, hi=rng.choice([24, 32, 64]))
    if kind == "batch":
        return dict(kind=kind, texts=_log(rng, 32, 256), sets=rng.randint(2, 8),
                    max_len=_log(rng, 256 * KiB, 4 * MiB), d_hi=_log(rng, 2000, 20_000))
    return dict(kind="host", algo=algo, n=_log(rng, 8 * MiB, 64 * MiB), d=_log(rng, 100, 2000),
                m=rng.choice([12, 16, 24, 32]))


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _text(n, g):
    """EST-shaped text: uniform bases with 1 % N, '\\n' after each record."""
    lut = torch.tensor([65] * 99 + [67] * 99 + [71] * 99 + [84] * 99 + [78] * 4,
                       dtype=torch.uint8, device="cuda")
    out = torch.empty(n, dtype=torch.uint8, device="cuda")
    for lo in range(0, n, 64 * MiB):
        hi = min(n, lo + 64 * MiB)
        out[lo:hi] = lut[torch.randint(0, 400, (hi - lo,), device="cuda", generator=g)]
    k = int(n / 501 * 1.1) + 64
    z = torch.randn(k, device="cuda", dtype=torch.float64, generator=g)
    lens = torch.exp(math.log(500) - 0.125 + 0.5 * z).round().clamp(min=1).long()
    ends = torch.cumsum(lens + 1, 0) - 1
    out[ends[ends < n]] = 10
    return out


def _windows(text, count, m, g):
    """Up to `count` newline-free windows of the text."""
    starts = torch.randint(0, text.numel() - m + 1, (2 * count + 64,), device="cuda", generator=g)
    w = text[starts[:, None] + torch.arange(m, device="cuda")]
    return w[(w != 10).all(1)][:count]


def _patterns(text, d, m, g, planted):
    win = _windows(text, min(planted, d), m, g)
    acgt = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device="cuda")
    rest = acgt[torch.randint(0, 4, (d - win.shape[0], m), device="cuda", generator=g)]
    return torch.cat([win, rest]).cpu().numpy()


def _mixed(text, d, lo, hi, g):
    """Half windows; prefixes, suffixes and copies of them; the rest uniform."""
    full = _patterns(text, d, hi, g, d // 2)
    ln = torch.randint(lo, hi + 1, (d,), device="cuda", generator=g).cpu().numpy()
    rng = np.random.default_rng(int(ln.sum()))
    pats = [full[i, :ln[i]].tobytes() for i in range(d)]
    for i in range(d // 2, d // 2 + (7 * d) // 20):
        src = pats[int(rng.integers(0, d // 2))]
        cut = int(rng.integers(lo, len(src) + 1))
        k = i % 7
        pats[i] = src[:cut] if k < 4 else src[len(src) - cut:] if k < 6 else src
    return [pats[i] for i in rng.permutation(d)]


def _planted(case):
    return (3 * case["d"]) // 10 if case["d"] <= 1000 else case["d"] // 10


def _pairs(n, d, m):
    """Expected pairs of a scan (random hits and the planted windows)."""
    return int(n * d / 4.0 ** m) + d


def _capacity(n, d, m):
    return int(1.15 * _pairs(n, d, m)) + 4096


def _inputs(case, seed):
    """Text (on the GPU) and patterns of a one-text case."""
    g = _gen(seed)
    text = _text(case["n"], g)
    if case["kind"] == "mixed":
        return text, _mixed(text, case["d"], case["lo"], case["hi"], g)
    return text, _patterns(text, case["d"], case["m"], g, _planted(case))


def _batch_inputs(case, seed):
    # the requests' shapes belong to the case, their bytes to the seed
    g = _gen(seed)
    rng = np.random.default_rng([case["texts"], case["sets"], case["max_len"], case["d_hi"]])
    lens = np.rint(np.exp(rng.uniform(math.log(1024), math.log(case["max_len"]), case["texts"]))).astype(np.int64)
    offs = np.concatenate([[0], np.cumsum((lens + 256) // 256 * 256)])
    arena = _text(int(offs[-1]) + 256, g)
    ds = np.rint(np.exp(rng.uniform(math.log(100), math.log(case["d_hi"]), case["sets"]))).astype(np.int64)
    ms = [8, 12, 16, 24, 32]
    sets = [_patterns(arena, int(ds[k]), ms[k % 5], g, int(ds[k]) // 10)
            for k in range(case["sets"])]
    pair = rng.integers(0, case["sets"], case["texts"])
    caps = [_capacity(int(lens[i]), len(sets[pair[i]]), sets[pair[i]].shape[1])
            for i in range(case["texts"])]
    return arena, offs[:-1], lens, sets, pair, caps


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        arena, offs, lens, sets, pair, caps = _batch_inputs(case, seed)
        # longer patterns suit Wu-Manber, short ones the automaton
        idx = [(mpm.build_wm if s.shape[1] >= 16 and len(s) <= 5000 else mpm.build_ac)(s, upload=True)
               for s in sets]
        var = [mpm.variant(lane_bytes=256, block_threads=512)] * len(lens)
        bs = BatchScan(arena, offs, lens, [idx[k] for k in pair], var, caps)
        bs.out.zero_()
        bs.capture()
        return dict(kind=kind, batch=bs)
    text, pats = _inputs(case, seed)
    ac = case["algo"] == "ac"
    if kind == "mixed":
        ix = (mpm.build_ac_var if ac else mpm.build_wm_var)(pats, upload=True)
        cap = case["n"] // 64 + 4096
    else:
        ix = (mpm.build_ac if ac else mpm.build_wm)(pats, upload=True)
        cap = _capacity(case["n"], case["d"], case["m"])
    if kind == "oneshot":
        return dict(kind=kind, ix=ix, text=text, keep=_fill(torch.empty(0, 2), cap))
    if kind == "host":
        pinned = torch.empty(case["n"], dtype=torch.uint8, pin_memory=True)
        pinned.copy_(text)
        return dict(kind=kind, ix=ix, text=pinned, keep=_fill(torch.empty(0, 2), cap))
    var = (mpm.variant(**SHAPE) if kind in ("scan", "mixed")
           else mpm.variant(block_threads=1024, flags=mpm.VARIANT_DENSE) if kind == "dense" else None)
    sc = mpm.Scanner(ix, case["n"], cap, var)
    sc.out.zero_()
    return dict(kind=kind, sc=sc, text=text, d=case["d"])


def run(state):
    kind = state["kind"]
    if kind in ("oneshot", "host"):
        pairs = (mpm.scan(state["ix"], state["text"]) if kind == "oneshot"
                 else mpm.scan_host(state["ix"], state["text"], chunk=16 * MiB))
        state["keep"][:len(pairs)] = pairs  # the program's own results table
        return state["keep"]
    if kind == "batch":
        bs = state["batch"]
        bs.replay()
        return bs.out, bs.totals
    sc = state["sc"]
    if kind == "counts":
        pairs = sc.scan(state["text"])
        return sc.out, mpm.count_ids(pairs, state["d"])
    sc.scan_async(state["text"])
    return sc.out, sc.total


def work(case):
    """Each text byte read once, each pair (8 bytes) and count written once;
    a lookup per byte is no floating-point work."""
    if case["kind"] == "batch":
        # mean of the log-uniform lengths; a third of a pair per byte is not
        # reached by most sets, so the lists are left out
        hi = case["max_len"]
        mean = (hi - 1024) / math.log(hi / 1024)
        return dict(bytes=int(case["texts"] * mean), flops=0)
    if case["kind"] == "mixed":
        pairs = int(case["n"] * 0.04 * case["d"] / 4.0 ** case["lo"]) + case["d"]
    else:
        pairs = _pairs(case["n"], case["d"], case["m"])
    b = case["n"] + 8 * pairs
    if case["kind"] == "counts":
        b += 8 * pairs + 4 * case["d"]
    return dict(bytes=int(b), flops=0)


# --------------------------------------------------------------------------
# The definition of the result in plain torch: polynomial hashes (modulo
# 2^64) of all windows looked up among the patterns', then compared bytewise.
# --------------------------------------------------------------------------
_BASE = 6364136223846793005


def _pow(k):
    p = pow(_BASE, k, 1 << 64)
    return p - (1 << 64) if p >= 1 << 63 else p


def _hashes(t, m):
    """int64 hash of every window of m bytes of t."""
    acc, done, h, ln = None, 0, t.long() + 1, 1
    while True:
        if m & ln:
            k = t.numel() - done - ln + 1
            acc = h[done:done + k] if acc is None else acc[:k] * _pow(ln) + h[done:done + k]
            done += ln
        if 2 * ln > m:
            return acc[:t.numel() - m + 1]
        h = h[:h.numel() - ln] * _pow(ln) + h[ln:]
        ln *= 2


def _matches(text, groups):
    """(pos, id) pairs in order; groups: (m, uint8 [k, m] patterns, ids)."""
    keys = []
    for m, P, ids in groups:
        P = torch.from_numpy(np.ascontiguousarray(P)).cuda()
        ids = torch.as_tensor(ids, dtype=torch.int64, device="cuda")
        ph = torch.cat([_hashes(r, m) for r in P]) if len(P) < 64 else _hashes(P.reshape(-1), m)[::m]
        ph, order = torch.sort(ph)
        for lo in range(0, max(0, text.numel() - m + 1), 32 * MiB):
            part = text[lo:lo + 32 * MiB + m - 1]
            th = _hashes(part, m)
            a = torch.searchsorted(ph, th)
            pos = (ph[a.clamp(max=len(ph) - 1)] == th).nonzero()[:, 0]
            b = torch.searchsorted(ph, th[pos], right=True)
            cnt = b - a[pos]
            pos_r = torch.repeat_interleave(pos, cnt)
            first = torch.cumsum(cnt, 0) - cnt
            k = torch.arange(len(pos_r), device="cuda") - torch.repeat_interleave(first, cnt)
            row = order[torch.repeat_interleave(a[pos], cnt) + k]
            same = torch.ones(len(row), dtype=torch.bool, device="cuda")
            for j in range(m):
                same &= part[pos_r + j] == P[row, j]
            keys.append(((pos_r[same] + lo) << 32) | ids[row[same]])
    key = torch.sort(torch.cat(keys))[0]
    return torch.stack([key >> 32, key & 0xFFFFFFFF], 1).to(torch.int32)


def _fill(pairs, cap):
    out = torch.zeros((max(1, cap), 2), dtype=torch.int32, device="cuda")
    k = min(cap, pairs.shape[0])
    out[:k] = pairs[:k]
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        arena, offs, lens, sets, pair, caps = _batch_inputs(case, seed)
        outs, totals = [], []
        for i in range(len(lens)):
            P = sets[pair[i]]
            t = arena[int(offs[i]):int(offs[i] + lens[i])]
            r = _matches(t, [(P.shape[1], P, np.arange(len(P)))])
            outs.append(_fill(r, caps[i]))
            totals.append(r.shape[0])
        return torch.cat(outs), torch.tensor(totals, dtype=torch.int64, device="cuda")
    text, pats = _inputs(case, seed)
    if kind == "mixed":
        ln = np.array([len(p) for p in pats])
        groups = [(int(m), np.stack([np.frombuffer(pats[i], np.uint8) for i in np.nonzero(ln == m)[0]]),
                   np.nonzero(ln == m)[0]) for m in np.unique(ln)]
        r = _matches(text, groups)
        return _fill(r, case["n"] // 64 + 4096), torch.tensor([r.shape[0]], device="cuda")
    r = _matches(text, [(case["m"], pats, np.arange(case["d"]))])
    out = _fill(r, _capacity(case["n"], case["d"], case["m"]))
    if kind in ("oneshot", "host"):
        return out
    if kind == "counts":
        return out, torch.bincount(r[:, 1].long(), minlength=case["d"]).to(torch.int32)
    return out, torch.tensor([r.shape[0]], device="cuda")
