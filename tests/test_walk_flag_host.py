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


def test_workspace_of_a_refused_filter_scan():
    """1.1 M copies of one string are more ids per 4 KiB block than the filter
    and direct-address scans count: the scan is walked, so its workspace holds
    the walkers' staging area."""
    rng = np.random.default_rng(4)
    few = ACGT[rng.integers(0, 4, (40, 12))]
    many = np.concatenate([few, np.repeat(few[:1], 1_100_000, axis=0)])
    for build in (mpm.build_ac, mpm.build_wm):
        auto, walk = mpm.variant(16, 256), mpm.variant(16, 256, mpm.PLACE_AUTO, 0, mpm.VARIANT_WALK)
        n = 30_000
        ix = build(few)
        assert mpm.workspace_bytes(ix, n, auto) < mpm.workspace_bytes(ix, n, walk)
        ix = build(many)
        assert mpm.workspace_bytes(ix, n, auto) == mpm.workspace_bytes(ix, n, walk)
