"""GPU: one workspace for scans of different kinds and lengths, one after
another, against the oracle element by element. The status words of a long
text lie where a shorter text's scan staged its occurrences, and where the
other scan kinds keep words and chunks of other sizes."""

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


def check(mpm, got, want, what):
    gp, gi = mpm.pairs_numpy(got)
    assert len(gp) == len(want[0]), f"{what}: {len(gp)} pairs, oracle {len(want[0])}"
    assert np.array_equal(gp, want[0]) and np.array_equal(gi, want[1]), what


@pytest.mark.parametrize("algo", ["ac", "wm"])
def test_staged_pairs_are_no_status_words(mpm, algo):
    """A lane keeps two occurrences in registers and stages the others as
    (position, string). Read as a status word of the next, longer scan, the
    pairs of strings 80 to 127 carry its epoch (1) and a set flag."""
    rng = np.random.default_rng(71)
    P = np.unique(ACGT[rng.integers(0, 4, (400, 8))], axis=0)[:128]  # string number = row
    short = P[96 + np.arange(2048) % 16].reshape(-1)
    long = ACGT[rng.integers(0, 4, 16 << 20)]
    ix = (mpm.build_ac if algo == "ac" else mpm.build_wm)(P, upload=True)
    want = [oracle.Win(P).scan(t) for t in (short, long)]
    var = mpm.variant(64, 256, mpm.PLACE_GLOBAL)
    sc = mpm.Scanner(ix, len(long), max(len(w[0]) for w in want) + 64, var)
    dev = [torch.from_numpy(t).cuda() for t in (short, long)]
    for k in range(6):
        print(f"[reuse] {algo} scan {k}", flush=True)
        check(mpm, sc.scan(dev[k & 1]), want[k & 1], f"{algo} scan {k}")
