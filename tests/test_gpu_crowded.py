"""GPU: texts where a set's grams repeat (runs of one character, of N, which
shares G's 2-bit code, and short repeats), through automatic placement,
against the oracle element by element: runs shorter and longer than a 4 KiB
block, at the text's start and end and at odd alignments, blocks before and
after a run, lists that fit the LDS and lists that do not, cut lists, strings
longer than a lane's range, repeated strings and mixed lengths. Blocks with
candidates almost everywhere are walked with the automaton (Aho-Corasick
indexes), the others are not, and the list is one."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ACGT = np.frombuffer(b"ACGT", np.uint8)


@pytest.fixture(scope="module")
def mpm():
    import paper_1407_2889_amd as m
    assert torch.cuda.is_available()
    return m


def to_dev(text, mis=0):
    buf = torch.full((len(text) + mis + 64,), 65, dtype=torch.uint8, device="cuda")
    buf[mis:mis + len(text)] = torch.from_numpy(np.ascontiguousarray(text)).cuda()
    return buf[mis:mis + len(text)]


def check(mpm, got, want, what):
    gp, gi = mpm.pairs_numpy(got)
    assert len(gp) == len(want[0]), f"{what}: {len(gp)} pairs, oracle {len(want[0])}"
    assert np.array_equal(gp, want[0]) and np.array_equal(gi, want[1]), what


def run_text(n, seed, units):
    """EST-shaped text with runs of the units: at the start, at the end, one
    shorter than a block, several over many blocks, odd places and lengths."""
    t = synth.est_text(n, seed=seed)
    for k, (at, ln) in enumerate([(0, 700), (9_001, 300), (20_003, 9_000), (60_000, 30_011), (120_005, 5),
                                  (n - 20_000, 20_000)]):
        u = np.frombuffer(units[k % len(units)], np.uint8)
        t[at:at + ln] = np.tile(u, ln // len(u) + 1)[:ln]
    return t


def fixed_set(d, m, seed, units, repeat):
    P = ACGT[np.random.default_rng(seed).integers(0, 4, (d, m))]
    for k, u in enumerate(units):
        P[k] = np.tile(np.frombuffer(u, np.uint8), m // len(u) + 1)[:m]
        P[len(units) + k, : max(4, m - 3)] = P[k, : max(4, m - 3)]
    if repeat:
        P[-6:] = P[:6]
        P[40:45] = P[0]
    return P


UNITS = [b"A", b"N", b"AT", b"G", b"CAG", b"N"]


@pytest.mark.parametrize("m", [8, 11, 12, 16, 24, 32, 100, 300])
@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_runs(mpm, algo, m):
    t = run_text(150_000, 300 + m, UNITS)
    for d, units in ((200, UNITS), (1000, [b"G"]), (3000, [b"A", b"AT"])):
        P = fixed_set(d, m, 400 + m, units, repeat=d != 1000)
        ix = (mpm.build_ac if algo == "ac" else mpm.build_wm)(P, upload=True)
        for n in (len(t), 65_536 + m):
            want = oracle.Win(P).scan(t[:n])
            for mis in (0, 9):
                print(f"[crowded] {algo} m={m} d={d} n={n} mis={mis}", flush=True)
                dev = to_dev(t[:n], mis)
                check(mpm, mpm.scan(ix, dev), want, f"{algo} m={m} d={d} n={n} mis={mis}")
            total = len(want[0])
            for cap in (0, 1, total // 2, total):
                sc = mpm.Scanner(ix, n, cap)
                sc.scan_async(dev)
                torch.cuda.synchronize()
                assert int(sc.total.item()) == total
                k = min(cap, total)
                check(mpm, sc.out[:k], (want[0][:k], want[1][:k]), f"cap {cap}")


@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_runs_32_bit_states(mpm, algo):
    t = run_text(200_000, 11, UNITS)
    P = fixed_set(10_000, 16, 12, UNITS, repeat=True)
    ix = (mpm.build_ac if algo == "ac" else mpm.build_wm)(P, upload=True)
    check(mpm, mpm.scan(ix, to_dev(t, 3)), oracle.Win(P).scan(t), algo)


@pytest.mark.parametrize("algo", ["ac", "wm"])
@pytest.mark.parametrize("lo,hi", [(8, 32), (12, 64), (9, 200)])
def test_runs_mixed_lengths(mpm, algo, lo, hi):
    rng = np.random.default_rng(lo * hi)
    P = [ACGT[rng.integers(0, 4, rng.integers(lo, hi + 1))].tobytes() for _ in range(500)]
    for k, u in enumerate(UNITS):
        for j, ln in enumerate((lo, (lo + hi) // 2, hi)):
            P[3 * k + j] = (u * hi)[:ln]
    for k in range(40):  # a crowded head
        P[100 + k] = b"A" * lo + P[100 + k][: max(1, hi - lo)]
    t = run_text(150_000, 700 + hi, UNITS)
    want = oracle.Win(P).scan(t)
    ix = (mpm.build_ac_var if algo == "ac" else mpm.build_wm_var)(P, upload=True)
    for mis in (0, 5):
        print(f"[crowded] mixed {algo} {lo}-{hi} mis={mis}", flush=True)
        check(mpm, mpm.scan(ix, to_dev(t, mis)), want, f"{algo} {lo}-{hi} mis={mis}")
    cap = len(want[0]) // 3
    sc = mpm.Scanner(ix, len(t), cap)
    sc.scan_async(to_dev(t, 5))
    torch.cuda.synchronize()
    assert int(sc.total.item()) == len(want[0])
    check(mpm, sc.out, (want[0][:cap], want[1][:cap]), "cut")


@pytest.mark.parametrize("mixed", [False, True])
def test_runs_past_2_gib(mpm, mixed):
    """Crowded blocks at the end of a text of more than 2^31 bytes."""
    rng = np.random.default_rng(41)
    P = ACGT[rng.integers(0, 4, (1000, 12))]
    P[0], P[1] = 65, np.frombuffer(b"ATATATATATAT", np.uint8)
    sets = [p.tobytes() + (b"AC" if k % 3 == 0 else b"") for k, p in enumerate(P)] if mixed else P
    tail = run_text(150_000, 43, [b"A", b"AT"])
    n = (1 << 31) + 123_457
    t = torch.full((n,), 10, dtype=torch.uint8, device="cuda")
    t[n - len(tail):] = torch.from_numpy(tail).cuda()
    want = oracle.Win(sets).scan(tail)
    assert len(want[0]) > 1000
    ix = (mpm.build_ac_var if mixed else mpm.build_ac)(sets, upload=True)
    got = mpm.pairs_numpy(mpm.scan(ix, t, capacity=len(want[0]) + 64))
    off = np.uint32(n - len(tail))
    assert len(got[0]) == len(want[0])
    assert np.array_equal(got[0], want[0] + off) and np.array_equal(got[1], want[1])


def test_runs_batched(mpm):
    from paper_1407_2889_amd.batch import BatchScan, pack_texts
    sets = [fixed_set(d, m, 900 + m, UNITS, repeat=True) for d, m in ((1000, 16), (300, 8), (2000, 24), (100, 12))]
    texts = [run_text(n, 800 + k, UNITS) for k, n in enumerate((150_000, 130_001, 700_003, 150_017))]
    idx = [(mpm.build_wm if k == 3 else mpm.build_ac)(s, upload=True) for k, s in enumerate(sets)]
    arena, offs, lens = pack_texts(texts * 2)
    sel = [0, 1, 2, 3, 1, 2, 3, 0]
    want = [oracle.Win(sets[k]).scan(t) for k, t in zip(sel, texts * 2)]
    bs = BatchScan(arena, offs, lens, [idx[k] for k in sel], [mpm.variant(256, 512)] * 8, [len(w[0]) for w in want])
    bs.capture()
    for r in range(3):
        bs.out.zero_()
        bs.replay()
        torch.cuda.synchronize()
        for i in range(8):
            gp, gi = bs.result(i)
            assert np.array_equal(gp, want[i][0]) and np.array_equal(gi, want[i][1]), f"replay {r}, text {i}"


@pytest.mark.parametrize("m", [8, 16, 24])
def test_runs_cost_about_a_walk(mpm, m):
    """A tenth of the text in runs of N, poly-G in the set: every sample of the
    runs is a candidate. Such blocks are walked, through L1 and L2 where the
    walkers have LDS and by the few waves that hold a run, so the scan takes
    about the walkers' time and not three to five times that."""
    n = 32 << 20
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    lut = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device="cuda")
    t = lut[torch.randint(0, 4, (n,), device="cuda", generator=g)]
    for s in range(0, n - (1 << 20), 5 << 20):
        t[s:s + (1 << 19)] = 78
    P = ACGT[np.random.default_rng(6).integers(0, 4, (1000, m))]
    P[0] = 71
    ix = mpm.build_ac(P, upload=True)
    us = {}
    for name, place in (("auto", mpm.PLACE_AUTO), ("walk", mpm.PLACE_LDS if m == 8 else mpm.PLACE_HOT)):
        sc = mpm.Scanner(ix, n, n // 16, mpm.variant(1024, 1024, place))
        a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ts = []
        for _ in range(8):
            a.record()
            sc.scan_async(t)
            z.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(z) * 1e3)
        us[name] = min(ts)
    print(f"[crowded] m={m}: {us}", flush=True)
    assert us["auto"] <= 2.5 * us["walk"], us
