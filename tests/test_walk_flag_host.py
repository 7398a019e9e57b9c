"""Host: MPM_VARIANT_WALK keeps automatic placement with the walkers, in single
scans and in batches, and names nothing else; the tuner's variants carry it and
fit every index kind."""

import numpy as np
import pytest

import paper_1407_2889_amd as mpm
from paper_1407_2889_amd import tune

ACGT = np.frombuffer(b"ACGT", np.uint8)


def sets():
    rng = np.random.default_rng(3)
    small = ACGT[rng.integers(0, 4, (1000, 16))]    # Aho-Corasick rows in LDS
    large = ACGT[rng.integers(0, 4, (10_000, 16))]  # rows beyond it: hot placement
    return small, large


def test_tuner_variants_fit_sets_of_different_lengths():
    P = [b"ACGTACGTAC", b"ACGTACGTTTGACC", b"GATTACAGA"]
    ix = {"ac": mpm.build_ac_var(P), "wm": mpm.build_wm_var(P)}
    for k, (algo, L, W, place) in enumerate(tune.VARIANTS):
        v = tune.variant_struct(k)
        assert (v.lane_bytes, v.block_threads, v.placement, v.grid) == (L, W, place, 0)
        assert mpm.workspace_bytes(ix[algo], 1 << 20, v) > 0


def test_walk_is_the_walkers_placement_alone():
    small, large = sets()
    for P, place in ((small, mpm.PLACE_LDS), (large, mpm.PLACE_HOT)):
        ix = mpm.build_ac(P)
        for L, W in ((64, 256), (256, 512), (1024, 512)):
            walk = mpm.variant(L, W, mpm.PLACE_AUTO, 0, mpm.VARIANT_WALK)
            same = mpm.variant(L, W, place)
            assert mpm.workspace_bytes(ix, 1 << 24, walk) == mpm.workspace_bytes(ix, 1 << 24, same)
            assert mpm.launch_key(ix, walk) == mpm.launch_key(ix, same)
            assert mpm.launch_key(ix, walk) != mpm.launch_key(ix, mpm.variant(L, W))
            k = tune.VARIANTS.index(("ac", L, W, mpm.PLACE_AUTO))
            assert mpm.workspace_bytes(ix, 1 << 24, tune.variant_struct(k)) == mpm.workspace_bytes(ix, 1 << 24, same)
            assert mpm.launch_key(ix, tune.variant_struct(k)) == mpm.launch_key(ix, same)


def test_unknown_flags_stay_refused():
    ix = mpm.build_ac(sets()[0])
    for fl in (128, 1 << 31, 128 | mpm.VARIANT_WALK):
        with pytest.raises(mpm.MpmError) as e:
            mpm.workspace_bytes(ix, 1 << 20, mpm.variant(64, 256, 0, 0, fl))
        assert e.value.status == mpm.MPM_EINVAL
