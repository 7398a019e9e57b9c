"""GPU: the staging copies of a host-text scan start after the work that is
already queued on the caller's stream. A caching allocator hands out blocks
whose last kernel is only queued, so that kernel may still write the staging
buffer when the scan is called."""

import ctypes as C

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("chunk", [1 << 20, 300_000])  # one buffer; both buffers
def test_staging_waits_for_queued_work(chunk):
    import paper_1407_2889_amd as mpm
    t = synth.est_text(1_000_000, seed=61)
    ps = synth.pattern_set(t, d=500, m=12, n_planted=400, seed=62)
    want = oracle.Win(ps.patterns).scan(t)
    assert len(want[0]) >= 400
    ix = mpm.build_ac(ps.patterns, upload=True)
    pinned = torch.empty(len(t), dtype=torch.uint8, pin_memory=True)
    pinned.numpy()[:] = t
    n = len(t)
    c = min(chunk, n - 11)
    stage = torch.zeros(2 * (c + 11), dtype=torch.uint8, device="cuda")
    ws = mpm.new_workspace(ix, c + 11)
    total = torch.zeros(1, dtype=torch.int64, device="cuda")
    out = torch.empty((len(want[0]) + 16, 2), dtype=torch.int32, device="cuda")
    big = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")

    def call():
        tot = C.c_uint64()
        st = mpm._L.mpm_scan_host(ix.handle, C.c_void_p(pinned.data_ptr()), n, C.c_void_p(stage.data_ptr()),
                                  stage.numel(), c, C.c_void_p(out.data_ptr()), out.shape[0],
                                  C.c_void_p(ws.data_ptr()), ws.numel() * 8, C.c_void_p(total.data_ptr()), None,
                                  mpm._stream_handle(None), C.byref(tot))
        assert st == mpm.MPM_OK
        gp, gi = mpm.pairs_numpy(out[: tot.value])
        assert np.array_equal(gp, want[0]) and np.array_equal(gi, want[1])

    call()  # the copy stream and its events exist from here on
    for k in range(3):
        print(f"[order] chunk={chunk} call {k}", flush=True)
        for _ in range(100):  # some 15 ms of queued work, then a write to the staging buffer
            big.fill_(k)
        stage.fill_(65)
        call()
