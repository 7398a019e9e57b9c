"""GPU: the table walks of both index kinds where automatic placement answers by
the q-gram filter or the direct-address table. MPM_VARIANT_WALK keeps those
requests with the walkers: the sweep at 1 GiB (16- and 32-bit rows, LDS, hot and
global tables, per-lane and dense output), the benchmark's text, grid sizes, cut
lists, repeated scans on one workspace, and workspaces that walkers and filter
scans share."""

import hashlib
import json
import os
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")
sys.path.insert(0, GOLDEN)
import listdigest  # noqa: E402

ACGT = np.frombuffer(b"ACGT", np.uint8)


@pytest.fixture(scope="module")
def mpm():
    import paper_1407_2889_amd as m
    assert torch.cuda.is_available()
    return m


@pytest.fixture(scope="module")
def golden():
    with open(os.path.join(GOLDEN, "sweep_digests.json")) as f:
        return json.load(f)


@pytest.fixture(scope="module")
def sweep_text():
    print("[walk] generating 1 GiB text", flush=True)
    text = synth.workload_sweep_text()
    return text, torch.from_numpy(text).cuda()


@pytest.fixture(scope="module")
def small():
    text, ps = synth.workload_small()
    return text, ps.patterns, oracle.Win(ps.patterns).scan(text)


def check(mpm, got, want, what):
    gp, gi = mpm.pairs_numpy(got)
    assert len(gp) == len(want[0]), f"{what}: {len(gp)} pairs, oracle {len(want[0])}"
    assert np.array_equal(gp, want[0]) and np.array_equal(gi, want[1]), what


def build(mpm, algo, P):
    return (mpm.build_ac if algo == "ac" else mpm.build_wm)(P, upload=True)


@pytest.mark.parametrize("d", synth.SWEEP_D)
@pytest.mark.parametrize("m", synth.SWEEP_M)
def test_sweep_walkers(mpm, sweep_text, golden, d, m):
    """Whole lists at 1 GiB against the oracle's digests, each walker by itself."""
    text, dev = sweep_text
    ps = synth.workload_sweep_set(text, d, m)
    g = next(r for r in golden["sets"] if r["d"] == d and r["m"] == m)
    assert hashlib.sha256(ps.patterns.tobytes()).hexdigest() == g["patterns_sha256"]
    for algo in ("ac", "wm"):
        ix = build(mpm, algo, ps.patterns)
        for v in (mpm.variant(1024, 1024, flags=mpm.VARIANT_WALK),
                  mpm.variant(1024, 1024, mpm.PLACE_GLOBAL),
                  mpm.variant(block_threads=1024, flags=mpm.VARIANT_WALK | mpm.VARIANT_DENSE)):
            print(f"[walk] sweep d={d} m={m} {algo} {v}", flush=True)
            got = mpm.scan(ix, dev, capacity=g["total"], var=v)
            assert got.shape[0] == g["total"]
            assert f"{listdigest.digest_torch(got):016x}" == g["digest"]
            counts = mpm.count_ids(got, d).cpu().numpy().view(np.uint32)
            assert hashlib.sha256(counts.astype("<u4").tobytes()).hexdigest() == g["counts_sha256"]
            del got
        del ix
    torch.cuda.empty_cache()


def test_est256_walkers(mpm):
    text, ps = synth.workload_est256()
    want = oracle.parallel_scan(oracle.Win(ps.patterns), text)
    dev = torch.from_numpy(text).cuda()
    for algo in ("ac", "wm"):
        ix = build(mpm, algo, ps.patterns)
        for fl in (0, mpm.VARIANT_DENSE):
            print(f"[walk] est256 {algo} flags={fl}", flush=True)
            L = 0 if fl else 1024
            check(mpm, mpm.scan(ix, dev, var=mpm.variant(L, 1024, flags=mpm.VARIANT_WALK | fl)), want, algo)


@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_walker_grids(mpm, small, algo):
    text, P, want = small
    ix = build(mpm, algo, P)
    t = torch.from_numpy(text).cuda()
    for grid in (1, 3, 17, 256, 4096):
        sc = mpm.Scanner(ix, len(text), len(want[0]) + 16, mpm.variant(64, 256, 0, grid, mpm.VARIANT_WALK))
        for rep in range(3):
            print(f"[walk] {algo} grid={grid} rep={rep}", flush=True)
            check(mpm, sc.scan(t), want, f"{algo} grid={grid} rep={rep}")


@pytest.mark.parametrize("algo", ["ac", "wm"])
@pytest.mark.parametrize("dense", [False, True])
def test_walker_cut_lists(mpm, small, algo, dense):
    text, P, want = small
    ix = build(mpm, algo, P)
    t = torch.from_numpy(text).cuda()
    v = mpm.variant(block_threads=1024 if dense else 256,
                    flags=mpm.VARIANT_WALK | (mpm.VARIANT_DENSE if dense else 0))
    for cap in (0, 1, len(want[0]) // 3, len(want[0]) - 1):
        sc = mpm.Scanner(ix, len(text), cap, v)
        with pytest.raises(mpm.MpmError) as e:
            sc.scan(t)
        assert e.value.status == mpm.MPM_EOVERFLOW
        assert int(sc.total.item()) == len(want[0])
        check(mpm, sc.out[:cap], (want[0][:cap], want[1][:cap]), f"{algo} cap {cap}")


@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_walker_workspace_reuse(mpm, small, algo):
    text, P, want = small
    ix = build(mpm, algo, P)
    t = torch.from_numpy(text).cuda()
    w2 = oracle.Win(P).scan(text[:100_000])
    for v in (mpm.variant(16, 256, 0, 7, mpm.VARIANT_WALK), mpm.variant(64, 1024, flags=mpm.VARIANT_WALK),
              mpm.variant(48, 512, 0, 5, mpm.VARIANT_WALK)):
        sc = mpm.Scanner(ix, len(text), len(want[0]) + 10, v)
        for rep in range(4):
            print(f"[walk] {algo} {v} rep={rep}", flush=True)
            check(mpm, sc.scan(t), want, f"rep {rep}")
            check(mpm, sc.scan(t[:100_000]), w2, f"prefix {rep}")


@pytest.mark.parametrize("kind", ["ac", "ac32", "wm"])
def test_walker_hot_is_the_automatic_choice(mpm, kind):
    t = synth.est_text(2_500_000, seed=31)
    d, m, k, seed = {"ac": (3000, 20, 1500, 32), "ac32": (6000, 20, 3000, 34), "wm": (20000, 16, 2000, 33)}[kind]
    ps = synth.pattern_set(t, d=d, m=m, n_planted=k, seed=seed)
    ix = build(mpm, kind[:2], ps.patterns)
    v = mpm.variant(256, 512, flags=mpm.VARIANT_WALK)
    assert mpm.launch_key(ix, v) == mpm.launch_key(ix, mpm.variant(256, 512, mpm.PLACE_HOT))
    check(mpm, mpm.scan(ix, torch.from_numpy(t).cuda(), var=v), oracle.Win(ps.patterns).scan(t), kind)


@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_tuner_variants_in_single_scans(mpm, algo):
    """Every variant of the tuner, as a caller of single scans may use it, on a
    set of one length and one of several."""
    from paper_1407_2889_amd import tune
    t = synth.est_text(400_000, seed=81)
    ps = synth.pattern_set(t, d=500, m=14, n_planted=300, seed=82)
    mixed = [p.tobytes()[: 9 + k % 6] for k, p in enumerate(ps.patterns)]
    dev = torch.from_numpy(t).cuda()
    for P in (ps.patterns, mixed):
        want = oracle.Win(P).scan(t)
        ix = build(mpm, algo, P) if P is not mixed else (
            mpm.build_ac_var if algo == "ac" else mpm.build_wm_var)(P, upload=True)
        for k, (a, *_) in enumerate(tune.VARIANTS):
            if a == algo:
                check(mpm, mpm.scan(ix, dev, var=tune.variant_struct(k)), want, f"{algo} variant {k}")


def test_shared_workspace_walkers_and_filter(mpm):
    """Scans of both kinds and of different lengths in turn on one workspace:
    each finds words, chunks and staged pairs of the others where its own
    status words lie."""
    import ctypes as C
    rng = np.random.default_rng(91)
    sets = {m: np.unique(ACGT[rng.integers(0, 4, (600, m))], axis=0)[:256] for m in (8, 16)}
    short = sets[8][64 + np.arange(2048) % 128].reshape(-1)
    texts = [short, ACGT[rng.integers(0, 4, 3 << 20)], synth.est_text(9 << 20, seed=92)]
    dev = [torch.from_numpy(t).cuda() for t in texts]
    idx, want = {}, {}
    for m, P in sets.items():
        for algo in ("ac", "wm"):
            idx[algo, m] = build(mpm, algo, P)
        for k, t in enumerate(texts):
            want[m, k] = oracle.Win(P).scan(t)
    big = sets[8][rng.integers(0, 256, 12_000)]  # 256 strings, some 47 ids each: no direct table
    dense = ACGT[rng.integers(0, 4, (12_000, 8))]
    for name, P in (("big", big), ("dense", dense)):
        idx[name, 8] = mpm.build_ac(P, upload=True)
        for k, t in enumerate(texts):
            want[name, k] = oracle.Win(P).scan(t)
    variants = [mpm.variant(64, 256), mpm.variant(64, 256, flags=mpm.VARIANT_WALK), mpm.variant(1024, 1024),
                mpm.variant(16, 512, mpm.PLACE_GLOBAL), mpm.variant(block_threads=1024, flags=mpm.VARIANT_DENSE),
                mpm.variant(block_threads=1024, flags=mpm.VARIANT_DENSE | mpm.VARIANT_WALK)]
    nb = max(mpm.workspace_bytes(ix, len(texts[2]), v) for ix in idx.values() for v in variants)
    ws = torch.zeros((nb + 7) // 8, dtype=torch.int64, device="cuda")
    total = torch.zeros(1, dtype=torch.int64, device="cuda")
    out = torch.empty((max(len(w[0]) for w in want.values()) + 16, 2), dtype=torch.int32, device="cuda")
    keys = list(idx)
    for step in range(160):
        key, k, v = keys[rng.integers(len(keys))], int(rng.integers(3)), variants[rng.integers(len(variants))]
        w = want[key[0] if key[0] in ("big", "dense") else key[1], k]
        print(f"[share] {step} {key} text {k} {v}", flush=True)
        tot = C.c_uint64()
        st = mpm._L.mpm_scan_sync(idx[key].handle, C.c_void_p(dev[k].data_ptr()), len(texts[k]),
                                  C.c_void_p(out.data_ptr()), out.shape[0], C.c_void_p(ws.data_ptr()),
                                  ws.numel() * 8, C.c_void_p(total.data_ptr()), C.byref(v),
                                  mpm._stream_handle(None), C.byref(tot))
        assert st == mpm.MPM_OK, (st, mpm._L.mpm_last_error())
        check(mpm, out[: tot.value], w, f"step {step}")
