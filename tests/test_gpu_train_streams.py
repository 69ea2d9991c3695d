"""Training on a handle whose stream does not wait for the null stream, while
another thread keeps the null stream busy: whatever the training call clears
or copies must be ordered with its own kernels, so the result is the one of
an idle device, bit for bit (every sum of a step has one fixed order).  A
clear of the optimizer's moments that waits behind the other thread's work
would land among the steps.
"""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_training_beside_a_busy_null_stream():
    import torch
    from paper_1602_05716_amd import inputs, mc
    sy = inputs.electrolyte(2048, 2048, 1.0, -1.0, 1.0, 1.0, 0.05, 0.7)
    sy.xyz = inputs.random_start(sy, 52)
    n_log = 8 * sy.n
    stop = threading.Event()
    a = torch.zeros((4096, 4096), device="cuda")
    torch.cuda.synchronize()

    def busy():
        # about ten milliseconds of work in the queue at any time, a bounded
        # number of rounds
        ends = []
        for _ in range(2000):
            if stop.is_set():
                break
            for _ in range(4):
                torch.mm(a, a)
            e = torch.cuda.Event()
            e.record()
            ends.append(e)
            if len(ends) > 2:
                ends.pop(0).synchronize()
        torch.cuda.synchronize()

    print("[gpu-case] training, null stream idle and busy", flush=True)
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision="fp32", max_disp=1.5, log_moves=n_log,
                  resum_every=0) as ch:
        ch.sweep(8, 78)
        args = dict(epochs=20, batch=256, lr=2e-3, seed=6)
        ref = ch.train_surrogate(n_log, **args)
        t = threading.Thread(target=busy)
        t.start()
        try:
            got = [ch.train_surrogate(n_log, **args) for _ in range(2)]
        finally:
            stop.set()
            t.join()
    for g in got:
        assert np.array_equal(g["params"], ref["params"])
        assert np.array_equal(g["loss"], ref["loss"])
        assert g["val_loss"] == ref["val_loss"] and g["ref_stage2_reject"] == ref["ref_stage2_reject"]
