"""GPU: the direct-address scan on runs of characters outside the set's four
main ones (N), with strings of them in the set: blocks where every window is
looked up among those strings, where more are than a wave has lanes, and
where a few are, against the oracle element by element, and timed against the
dense walk."""

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


def odd_set(d, m, seed):
    """d strings of ACGT, some of N (which shares G's code) and of N among G,
    repeated ones among both."""
    P = ACGT[np.random.default_rng(seed).integers(0, 4, (d, m))]
    P[0], P[1] = 78, 71
    for k in range(m):
        P[2 + k] = 71
        P[2 + k, k] = 78
    P[20:24] = P[0]
    P[24:27] = P[3]
    P[30:33] = P[40]
    return P


def n_text(n, seed):
    """EST-shaped text with runs of N: at both ends, over several blocks, of 90
    windows in one block, alternating with G, single ones from the text itself."""
    t = synth.est_text(n, seed=seed)
    t[:500] = 78
    t[12_301:12_400] = 78
    t[30_005:52_000] = 78
    t[60_000:66_000:2] = 78
    t[60_001:66_000:2] = 71
    t[n - 9_000:] = 78
    return t


def dev_text(t, mis):
    buf = torch.full((len(t) + mis + 64,), 65, dtype=torch.uint8, device="cuda")
    buf[mis:mis + len(t)] = torch.from_numpy(t).cuda()
    return buf[mis:mis + len(t)]


@pytest.mark.parametrize("m,d", [(5, 700), (6, 2000), (7, 6000), (8, 12_000)])
@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_odd_runs(mpm, algo, m, d):
    P = odd_set(d, m, 10 * m)
    ix = (mpm.build_ac if algo == "ac" else mpm.build_wm)(P, upload=True)
    for n in (100_000, 700_001):
        t = n_text(n, n + m)
        want = oracle.Win(P).scan(t)
        for mis in (0, 11):
            print(f"[odd] {algo} m={m} n={n} mis={mis}", flush=True)
            dev = dev_text(t, mis)
            for cap in (len(want[0]), len(want[0]) // 2, 0):
                sc = mpm.Scanner(ix, n, cap)
                sc.scan_async(dev)
                torch.cuda.synchronize()
                assert int(sc.total.item()) == len(want[0])
                gp, gi = mpm.pairs_numpy(sc.out[:cap])
                assert np.array_equal(gp, want[0][:cap]) and np.array_equal(gi, want[1][:cap]), (n, mis, cap)


def test_odd_runs_cost(mpm):
    """A tenth of the text in runs of N: every window of the runs is looked up,
    in both passes, two round trips per pair of windows of a lane. That and
    the waves that hold a run alone may take up to three times the dense
    walk's time, not nine."""
    n = 32 << 20
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    t = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device="cuda")[
        torch.randint(0, 4, (n,), device="cuda", generator=g)]
    for s in range(0, n - (1 << 20), 5 << 20):
        t[s:s + (1 << 19)] = 78
    P = ACGT[np.random.default_rng(6).integers(0, 4, (10_000, 8))]
    P[0] = 78
    ix = mpm.build_ac(P, upload=True)
    us = {}
    for name, place in (("auto", mpm.PLACE_AUTO), ("walk", mpm.PLACE_GLOBAL)):
        sc = mpm.Scanner(ix, n, n // 2, mpm.variant(block_threads=1024, placement=place, flags=mpm.VARIANT_DENSE))
        a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ts = []
        for _ in range(8):
            a.record()
            sc.scan_async(t)
            z.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(z) * 1e3)
        us[name] = min(ts)
    print(f"[odd] {us}", flush=True)
    assert us["auto"] <= 3 * us["walk"], us


def test_odd_string_with_many_ids(mpm):
    """A string outside the main characters given 40,000 times: its pairs take
    80 rounds of the output buffer, each of which deals its own ids alone."""
    rng = np.random.default_rng(9)
    P = ACGT[rng.integers(0, 4, (10_000, 8))]
    P[0] = np.frombuffer(b"ACGNACGT", np.uint8)
    P = np.concatenate([P, np.tile(P[0], (40_000, 1))])
    t = ACGT[rng.integers(0, 4, 200_000)]
    for s in (0, 777, 4090, 4110, 100_000, len(t) - 8):
        t[s:s + 8] = P[0]
    want = oracle.Win(P).scan(t)
    ix = mpm.build_ac(P, upload=True)
    dev = dev_text(t, 3)
    us = {}
    for name, place in (("auto", mpm.PLACE_AUTO), ("walk", mpm.PLACE_GLOBAL)):
        sc = mpm.Scanner(ix, len(t), len(want[0]), mpm.variant(block_threads=1024, placement=place, flags=mpm.VARIANT_DENSE))
        a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ts = []
        for _ in range(4):
            a.record()
            sc.scan_async(dev)
            z.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(z) * 1e3)
        us[name] = min(ts)
        gp, gi = mpm.pairs_numpy(sc.out[: int(sc.total.item())])
        assert np.array_equal(gp, want[0]) and np.array_equal(gi, want[1]), name
    print(f"[odd] many ids {us}", flush=True)
    assert us["auto"] <= 3 * us["walk"], us
