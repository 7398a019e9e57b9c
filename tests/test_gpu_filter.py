"""GPU: the scans behind automatic placement (the q-gram filter and the
direct-address table) against the oracle and against the walkers of explicit
placements, element by element, at the sizes where they can go wrong: pattern
lengths that change the sampling step or the gram, texts ending around a
16-byte piece, a lane's 64 bytes, a 4 KiB block and a chunk, every text
alignment, low-complexity texts where every sample is a candidate, repeated
and nested strings, bytes sharing a 2-bit code with a pattern byte, and
capacities that cut the list."""

import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ACGT = np.frombuffer(b"ACGT", np.uint8)


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def mpm():
    import paper_1407_2889_amd as m
    assert torch.cuda.is_available()
    return m


def to_dev(text, mis=0):
    buf = torch.full((len(text) + mis + 64,), 65, dtype=torch.uint8, device="cuda")
    if len(text):
        buf[mis:mis + len(text)] = torch.from_numpy(np.ascontiguousarray(text)).cuda()
    return buf[mis:mis + len(text)]


def check(got, want, what):
    gp, gi = got
    assert len(gp) == len(want[0]), f"{what}: {len(gp)} pairs, oracle {len(want[0])}"
    assert np.array_equal(gp, want[0]) and np.array_equal(gi, want[1]), what


def build(mpm, algo, P):
    if isinstance(P, list):
        return (mpm.build_ac_var if algo == "ac" else mpm.build_wm_var)(P, upload=True)
    return (mpm.build_ac if algo == "ac" else mpm.build_wm)(P, upload=True)


def want_of(P, T):
    if isinstance(P, list):
        return oracle.Win(P).scan(T)
    return oracle.Win(P).scan(T) if len(T) else (np.zeros(0, np.uint32),) * 2


def run(mpm, ix, T, mis=0, var=None):
    return mpm.pairs_numpy(mpm.scan(ix, to_dev(T, mis), var=var))


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 7, 8, 9, 10, 11, 12, 13, 16, 17, 23, 24, 25, 32, 40, 100])
@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_lengths(mpm, algo, m):
    t = synth.est_text(120_000, seed=100 + m)
    for d in (1, 60, 3000):
        ps = synth.pattern_set(t, d=d, m=m, n_planted=max(1, d // 3), seed=200 + m)
        P = ps.patterns.copy()
        if d > 20:
            P[5:9] = P[0]
        ix = build(mpm, algo, P)
        for n in (len(t), 4096 + m, 4096 * 4 + m - 1, 65536 + m, 70):
            want = want_of(P, t[:n])
            for mis in (0, 7):
                say(f"[filter] {algo} m={m} d={d} n={n} mis={mis}")
                check(run(mpm, ix, t[:n], mis), want, f"{algo} m={m} d={d} n={n} mis={mis}")


@pytest.mark.parametrize("m", [6, 8, 16, 24])
def test_text_ends_and_alignments(mpm, m):
    t = synth.est_text(30_000, seed=7)
    P = synth.pattern_set(t, d=200, m=m, n_planted=150, seed=8).patterns
    P[:4] = t[0:m]
    ix = mpm.build_wm(P, upload=True)
    ends = sorted({m - 1, m, m + 1} | {b + k for b in (16, 64, 4096, 8192, 16384) for k in (-1, 0, 1, 15, 17)})
    for n in ends:
        T = t[:n].copy()
        if n >= m:
            T[n - m:] = P[10]  # an occurrence that ends with the text
        want = want_of(P, T)
        for mis in ((0, 1, 15) if n > 300 else range(16)):
            say(f"[ends] m={m} n={n} mis={mis}")
            check(run(mpm, ix, T, mis), want, f"m={m} n={n} mis={mis}")


@pytest.mark.parametrize("m,d", [(2, 9), (3, 40), (5, 900), (7, 9000), (8, 9000), (8, 60_000)])
def test_direct_address_sets(mpm, m, d):
    """Sets dense enough for the direct-address table: texts of one wave, of
    waves sharing a block (below 8 MiB), and of several blocks per wave; text
    bytes N and newline that share a code with a base, strings that hold N."""
    t = synth.est_text(9_000_000, seed=300 + m)
    P = synth.pattern_set(t, d=d, m=m, n_planted=d // 4, seed=301 + m).patterns
    if d > 100:
        P[:20] = np.where(np.arange(m) == m // 2, ord("N"), P[:20])
    ix = mpm.build_ac(P, upload=True)
    for n, mis in ((len(t), 0), (4_200_001, 5), (1_000_003, 9), (70_001, 15), (300, 2)):
        say(f"[direct] m={m} d={d} n={n} mis={mis}")
        want = oracle.parallel_scan(oracle.Win(P), t[:n])
        check(run(mpm, ix, t[:n], mis, mpm.variant(block_threads=1024, flags=mpm.VARIANT_DENSE)), want,
              f"m={m} d={d} n={n}")


def low_complexity():
    rng = np.random.default_rng(3)
    a16 = np.full((3, 16), 65, np.uint8)
    cases = [("all A, m=16", np.full(150_001, 65, np.uint8), a16)]
    cases.append(("all A, m=8", np.full(150_001, 65, np.uint8), np.full((2, 8), 65, np.uint8)))
    per = np.tile(np.frombuffer(b"ACACACGT", np.uint8), 20_000)
    P = np.stack([per[k:k + 24] for k in range(8)] + [per[0:24]] * 3)
    cases.append(("period 8, m=24", per, P))
    mix = np.frombuffer(b"ACGTN\n", np.uint8)[rng.integers(0, 6, 100_000)]
    P = np.stack([mix[s:s + 8] for s in rng.integers(0, 99_000, 400)])
    cases.append(("N and newlines in every pattern, m=8", mix, P))
    P = np.stack([mix[s:s + 12] for s in rng.integers(0, 99_000, 400)])
    cases.append(("N and newlines in every pattern, m=12", mix, P))
    t = ACGT[rng.integers(0, 4, 100_000)]
    P = ACGT[rng.integers(0, 4, (30_000, 8))]
    P[100:161] = P[0]
    P[200:204] = P[1]
    P[300:300 + 50] = np.frombuffer(b"ACGNACGT", np.uint8)
    t[5000:5008] = P[0]
    t[6000:6008] = P[300]
    cases.append(("repeated strings, m=8, d=30k", t, P))
    t = ACGT[rng.integers(0, 4, 8192 * 3 + 7)]
    cases.append(("all-A prefix, text ends early in a block", t, [b"A" * 8 + b"CGT", t[5:25].tobytes(), t[-20:].tobytes()]))
    b = rng.integers(0, 256, 60_000).astype(np.uint8)
    cases.append(("all byte values, m=9", b, np.stack([b[s:s + 9] for s in rng.integers(0, 59_000, 300)])))
    nested = [b"A" * k for k in range(8, 60)] + [b"ACACACGT" * 3, b"ACACACGT"]
    t = np.concatenate([per[:30_000], np.full(30_000, 65, np.uint8), per[:30_000]])
    cases.append(("nested strings", t, nested))
    t = synth.est_text(400_000, seed=12)
    cases.append(("lengths 8-32", t, synth.mixed_pattern_set(t, 600, 8, 32, 300, 13, 120, 60, 30)))
    cases.append(("lengths 12-90", t, synth.mixed_pattern_set(t, 300, 12, 90, 200, 14, 60, 30, 10)))
    return cases


@pytest.mark.parametrize("case", low_complexity(), ids=lambda c: c[0])
@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_low_complexity_and_capacity(mpm, algo, case):
    name, T, P = case
    want = want_of(P, T)
    assert len(want[0]) > 0
    ix = build(mpm, algo, P)
    dev = to_dev(T, 3)
    for var in (None, mpm.variant(1024, 1024), mpm.variant(64, 256, 0, 3)):
        say(f"[low] {algo} {name} {var}")
        check(mpm.pairs_numpy(mpm.scan(ix, dev, var=var)), want, f"{name} {var}")
    say(f"[low] {algo} {name} walkers")
    check(mpm.pairs_numpy(mpm.scan(ix, dev, var=mpm.variant(64, 256, mpm.PLACE_GLOBAL))), want, name)
    for cap in (0, 1, 65, len(want[0]) // 2, len(want[0])):
        say(f"[low] {algo} {name} capacity {cap}")
        sc = mpm.Scanner(ix, len(T), cap)
        sc.out.fill_(-1)
        for rep in range(3):
            sc.scan_async(dev)
        assert int(sc.total.item()) == len(want[0])
        k = min(cap, len(want[0]))
        check(mpm.pairs_numpy(sc.out[:k]), (want[0][:k], want[1][:k]), f"{name} capacity {cap}")


def test_graph_capture(mpm):
    """Captured scans replay to the eager list, with eager work between."""
    t = synth.est_text(2_000_000, seed=5)
    for P, var in ((synth.pattern_set(t, 500, 16, 200, 6).patterns, mpm.variant(1024, 1024)),
                   (synth.pattern_set(t, 20_000, 8, 2000, 6).patterns, None)):
        want = want_of(P, t)
        ix = mpm.build_ac(P, upload=True)
        dev = to_dev(t)
        sc = mpm.Scanner(ix, len(t), len(want[0]), var)
        sc.scan_async(dev)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            sc.scan_async(dev)
        for rep in range(4):
            say(f"[capture] m={P.shape[1]} rep={rep}")
            sc.out.fill_(-1)
            sc.total.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert int(sc.total.item()) == len(want[0])
            check(mpm.pairs_numpy(sc.out[:len(want[0])]), want, f"replay {rep}")
