"""GPU: batches through the q-gram filter against the oracle (texts around the
sizes where a wave's pieces change, texts that stay with the walkers in the
same batch, lists that overflow or are cut, one workgroup, timed requests,
graph replays), and synchronous scans from more threads than there are pinned
read-back slots."""

import sys
import threading

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def mpm():
    import paper_1407_2889_amd as m
    assert torch.cuda.is_available()
    return m


def make_sets(t):
    """Filters of every sampling step (1 to 16) and gram length (8 to 10), a
    set without one, repeated strings, and bytes that share a code."""
    sets = [synth.pattern_set(t, d, m, d // 4, 7 + d).patterns
            for d, m in ((300, 8), (3000, 8), (700, 10), (900, 12), (400, 16), (6000, 24), (200, 32), (60, 5))]
    rep = sets[2].copy()
    rep[1::2] = rep[::2]
    odd = sets[3].copy()
    odd[::5, 4] = ord("N")
    return sets + [rep, odd, np.frombuffer(b"A" * 12 + b"C" * 12, np.uint8).reshape(2, 12)]


@pytest.mark.parametrize("grid", [0, 1])
@pytest.mark.parametrize("timed", [False, True])
def test_batch_filter(mpm, grid, timed):
    from paper_1407_2889_amd import batch
    t = synth.est_text(3_000_000, seed=91)
    sets = make_sets(t)
    idx = [(mpm.build_wm if k % 2 else mpm.build_ac)(P, upload=True) for k, P in enumerate(sets)]
    wins = [oracle.Win(P) for P in sets]
    rng = np.random.default_rng(17)
    lens = [0, 1, 4, 5, 8, 12, 15, 16, 31, 32, 63, 64, 65, 4080, 4081, 4095, 4096, 4097, 8192, 65_536, 65_552,
            262_144, 1_000_001]
    texts, pair = [], []
    for k in range(len(sets)):
        for n in (lens if k % 3 == 0 else lens[k % 3::2]):
            at = int(rng.integers(0, len(t) - n))
            texts.append(t[at:at + n])
            pair.append(k)
    for n in (70, 5000, 40_000):  # every sample a candidate, occurrences all along
        texts.append(np.full(n, ord("A"), np.uint8))
        pair.append(len(sets) - 1)
    want = [wins[pair[i]].scan(x) if len(x) else (np.zeros(0, np.uint32),) * 2 for i, x in enumerate(texts)]
    caps = [max(0, len(w[0]) - (i % 4 == 3) * (1 + len(w[0]) // 3)) for i, w in enumerate(want)]
    # texts back to back: every alignment
    offs = np.concatenate([[0], np.cumsum([len(x) for x in texts])])
    arena = torch.from_numpy(np.concatenate(texts + [np.zeros(64, np.uint8)])).cuda()
    var = [mpm.variant(grid=grid) if i % 7 else mpm.variant(256, 512, mpm.PLACE_GLOBAL) for i in range(len(texts))]
    bs = batch.BatchScan(arena, offs[:-1], np.array([len(x) for x in texts]), [idx[k] for k in pair], var, caps,
                         timed=timed)
    keys = {mpm.launch_key(ix, mpm.variant(grid=grid)) for ix in idx}
    say(f"[filter batch] grid {grid} timed {timed}: {len(texts)} texts, {bs.groups} launches, {len(keys)} keys")
    assert len(keys) <= 2

    def same(tag):
        tot = bs.totals_host()
        for i, w in enumerate(want):
            assert int(tot[i]) == len(w[0]), f"{tag}: text {i} of {len(texts[i])}, set {pair[i]}: {int(tot[i])}"
            c = min(caps[i], len(w[0]))
            gp, gi = mpm.pairs_numpy(bs.out[int(bs.out_offs[i]):int(bs.out_offs[i]) + c])
            assert np.array_equal(gp, w[0][:c]) and np.array_equal(gi, w[1][:c]), f"{tag}: text {i}"

    bs.run()
    torch.cuda.synchronize()
    same("run")
    if timed:
        c = bs.costs.cpu().numpy()
        long = [i for i, x in enumerate(texts) if len(x) >= 4096]
        assert np.all(c[long] > 0) and np.all(np.isfinite(c))
    bs.capture()
    for rep in range(3):
        bs.out.fill_(-1)
        bs.totals.fill_(12345)
        torch.cuda.synchronize()
        say(f"[filter batch] replay {rep}")
        bs.replay()
        torch.cuda.synchronize()
        same(f"replay {rep}")


@pytest.mark.parametrize("m,d", [(8, 400), (16, 400)])
def test_tune_time_filter(mpm, m, d):
    """The timing call under automatic placement: its workspace is enough and
    no more than it asks for is touched, and it leaves the scan's list."""
    import ctypes as C
    t = synth.est_text(70_001, seed=5)
    P = synth.pattern_set(t, d, m, 100, 6).patterns
    ix = mpm.build_ac(P, upload=True)
    want = oracle.Win(P).scan(t)
    dev = torch.from_numpy(t).cuda()
    L, v = mpm._L, mpm.variant(256, 512)
    for copies in (1, 7, 300):
        wb = int(L.mpm_tune_work_bytes(ix.handle, len(t), copies, C.byref(v)))
        assert wb > 0
        work = torch.full((wb + 512,), 0x5a, dtype=torch.uint8, device="cuda")
        base = (work.data_ptr() + 255) // 256 * 256
        out = torch.full((len(want[0]), 2), -1, dtype=torch.int32, device="cuda")
        total = torch.zeros(1, dtype=torch.int64, device="cuda")
        ms = C.c_float(-1)
        say(f"[tune_time] m {m} copies {copies} workspace {wb}")
        args = [ix.handle, C.c_void_p(dev.data_ptr()), len(t), copies, C.byref(v), C.c_void_p(out.data_ptr()),
                len(want[0]), C.c_void_p(total.data_ptr()), C.c_void_p(base), wb, 3, mpm._stream_handle(), C.byref(ms)]
        assert L.mpm_tune_time(*args) == 0 and ms.value > 0
        assert int(total.item()) == len(want[0])
        got = mpm.pairs_numpy(out)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        lo = base - work.data_ptr()
        assert bool((work[:lo] == 0x5a).all()) and bool((work[lo + wb:] == 0x5a).all())
        args[9] = wb - 1
        assert L.mpm_tune_time(*args) < 0


def test_sync_scans_from_many_threads(mpm):
    """More threads than pinned read-back slots, each with a stream, an index
    and a workspace of its own; totals inside and outside the workspace."""
    t = synth.est_text(300_000, seed=3)
    jobs = []
    for k in range(40):
        n = 200_000 + 2000 * k
        P = synth.pattern_set(t, 50 + 10 * k, 12, 30, 60 + k).patterns
        jobs.append((mpm.build_ac(P, upload=True), torch.from_numpy(t[:n]).cuda(), oracle.Win(P).scan(t[:n])))
    torch.cuda.synchronize()
    bad = []

    def work(k):
        ix, dev, want = jobs[k]
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for rep in range(3):
                got = mpm.pairs_numpy(mpm.scan(ix, dev) if (k + rep) % 2 else mpm.Scanner(ix, len(dev), 50_000).scan(dev))
                if not (np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])):
                    bad.append((k, rep))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    say("[threads] 40 scanning threads")
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not bad, bad


@pytest.mark.parametrize("lens,d", [((8, 8), 1000), ((7, 7), 150), ((5, 5), 8), ((8, 32), 900), ((12, 12), 3000),
                                    ((16, 16), 20_000), ((24, 24), 40_000)])
def test_large_workgroups(mpm, lens, d):
    """Texts of 16 MiB and a few bytes: workgroups of 1024 threads with the
    answers for two positions, ranks in LDS, 4^10 bits, and waves with uneven
    shares of the blocks; N runs and bytes that share a code."""
    lo, hi = lens
    t = synth.est_text((16 << 20) + 4 * 4096 + 77, seed=61)
    t[5_000_000:5_000_400] = ord("N")
    t[-300:] = ord("A")
    P = synth.pattern_set(t, d, hi, d // 4, 62).patterns
    P[0], P[1] = ord("A"), ord("N")
    if lo != hi:
        rng = np.random.default_rng(63)
        P = [p[:n].tobytes() for p, n in zip(P, rng.integers(lo, hi + 1, d))]
        ix = mpm.build_ac_var(P, upload=True)
    else:
        ix = mpm.build_wm(P, upload=True)
    buf = torch.zeros(len(t) + 64, dtype=torch.uint8, device="cuda")
    buf[5:5 + len(t)] = torch.from_numpy(t).cuda()
    w = oracle.Win(P)
    for n in (len(t), 16 << 20):
        want = w.scan(t[:n])
        say(f"[large] lengths {lens} d {d} n {n}: {len(want[0])} pairs")
        got = mpm.pairs_numpy(mpm.scan(ix, buf[5:5 + n], capacity=len(want[0])))
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
