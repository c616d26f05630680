"""Forward passes of one thread while another trains the same network, or sets its
parameters: every pass sees the weights after some whole number of steps, never
some of a step's new values beside old ones.  An epoch of one minibatch is one step, so the weights
after k steps are those of a training of k epochs."""
import ctypes as C
import threading

import numpy as np
import pytest

from oracle import mlp_oracle as M
from paper_2511_13894_amd import pdhg

pytestmark = pytest.mark.gpu

STEPS, ROUNDS, BATCH = 60, 40, 64  # steps of a training, trainings, passes between two looks at their logits


def test_passes_beside_training_see_whole_steps():
    hip, net = pdhg._hip_runtime(), pdhg.Mlp(3)
    rng = np.random.default_rng(5)
    f = rng.standard_normal((4096, 16)).astype(np.float32)
    f[:, 12:] = 0
    y = (f[:, 0] + 0.3 * rng.standard_normal(4096) > 0.2).astype(np.float32)
    start = M.flat(M.init_params(9))
    n = 1024
    feat, out = C.c_void_p(), C.c_void_p()
    assert hip.hipMalloc(C.byref(feat), 64 * n) == 0 and hip.hipMalloc(C.byref(out), 4 * n * BATCH) == 0
    got = np.empty((BATCH, n), dtype=np.float32)

    def passes():
        for k in range(BATCH):
            net.forward_noalloc(feat, n, C.c_void_p(out.value + 4 * n * k))
        assert hip.hipDeviceSynchronize() == 0
        assert hip.hipMemcpy(got.ctypes.data_as(C.c_void_p), out, got.nbytes, 2) == 0
        return {row.tobytes() for row in got}

    def train(steps):
        net.set_params(start)
        net.train(f, y, epochs=steps, batch=65536, lr=0.05, seed=1)

    try:
        probe = np.ascontiguousarray(f[:n])
        assert hip.hipMemcpy(feat, probe.ctypes.data_as(C.c_void_p), probe.nbytes, 1) == 0
        seen = set()
        for k in range(STEPS + 1):
            train(k)
            after = passes()
            assert len(after) == 1
            seen |= after
        assert len(seen) == STEPS + 1
        print("[mlp] training beside passes", flush=True)
        trainer = threading.Thread(target=lambda: [train(STEPS) for _ in range(ROUNDS)])
        trainer.start()
        torn = total = 0
        while trainer.is_alive():
            rows = passes()
            torn += len(rows - seen)
            total += len(rows)
        trainer.join()
        print(f"[mlp] {total} different logit rows, {torn} of no whole step", flush=True)
        assert torn == 0
    finally:
        hip.hipFree(feat)
        hip.hipFree(out)
