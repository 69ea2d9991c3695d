"""Training on a handle whose stream does not wait for the null stream, while
another thread keeps the null stream busy: whatever the training call clears
or copies must be ordered with its own kernels, so the result is the one of
an idle device, bit for bit (every sum of a step has one fixed order).  A
clear of the optimizer's moments that waits behind the other thread's work
would land among the steps.
"""
import ctypes
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_training_beside_a_busy_null_stream():
    from paper_1602_05716_amd import inputs, mc
    sy = inputs.electrolyte(2048, 2048, 1.0, -1.0, 1.0, 1.0, 0.05, 0.7)
    sy.xyz = inputs.random_start(sy, 52)
    n_log = 8 * sy.n
    mc.lib()
    hip = ctypes.CDLL("libamdhip64.so.7")  # the runtime the library runs on
    size, scrap = 8 << 30, ctypes.c_void_p()
    stop = threading.Event()

    def busy():
        # some milliseconds of work in the null stream's queue at nearly any
        # time, a bounded number of rounds
        for k in range(4000):
            if stop.is_set():
                break
            assert hip.hipMemsetAsync(scrap, 0, ctypes.c_size_t(size), None) == 0
            if k % 4 == 3:
                assert hip.hipStreamSynchronize(None) == 0
        assert hip.hipStreamSynchronize(None) == 0

    print("[gpu-case] training, null stream idle and busy", flush=True)
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision="fp32", max_disp=1.5, log_moves=n_log,
                  resum_every=0) as ch:
        ch.sweep(8, 78)
        args = dict(epochs=20, batch=256, lr=2e-3, seed=6)
        ref = ch.train_surrogate(n_log, **args)
        assert hip.hipMalloc(ctypes.byref(scrap), ctypes.c_size_t(size)) == 0
        t = threading.Thread(target=busy)
        t.start()
        try:
            got = [ch.train_surrogate(n_log, **args) for _ in range(2)]
        finally:
            stop.set()
            t.join()
            assert hip.hipFree(scrap) == 0
    for g in got:
        assert np.array_equal(g["params"], ref["params"])
        assert np.array_equal(g["loss"], ref["loss"])
        assert g["val_loss"] == ref["val_loss"] and g["ref_stage2_reject"] == ref["ref_stage2_reject"]
