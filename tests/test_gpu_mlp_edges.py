"""Sizes where the predictor's kernels can go wrong: partial tiles and waves,
gradient sums shorter and longer than a round of loads, loss sums past one
chunk, and the no-allocation forward on buffers that are only element-aligned
or overlap.  Tolerance of a gradient: the float32 sums' rounding, at most
(waves + 64) x 2^-24 of the summed magnitudes, which exceed the sum itself by
less than a factor of ten on these data."""
import ctypes as C

import numpy as np
import pytest

from oracle import mlp_oracle as M
from paper_2511_13894_amd import pdhg

pytestmark = pytest.mark.gpu


def _data(n, seed):
    rng = np.random.default_rng(seed)
    f = rng.standard_normal((n, 16)).astype(np.float32)
    f[:, 12:] = 0
    return f, (f[:, 0] + 0.3 * rng.standard_normal(n) > 0.2).astype(np.float32)


@pytest.mark.parametrize("n", [1, 16, 33, 1023, 1025, 4097, 40000])
def test_gradient_at_partial_tiles_and_long_sums(n):
    f, y = _data(n, n)
    net = pdhg.Mlp(3)
    net.set_params(M.flat(M.init_params(9)))
    q = M.unflat(net.get_params())
    g, loss = net.gradient(f, y, 1.5)
    lo, go, _ = M.loss_and_grad(q, f.astype(np.float64), y.astype(np.float64), 1.5)
    go = M.flat(go)
    tol = 10 * (n / 32 + 64) * 2.0 ** -24
    rel = np.linalg.norm(g - go) / np.linalg.norm(go)
    print(f"[mlp] gradient of {n} samples: relative l2 error {rel:.2e} (bound {tol:.2e})", flush=True)
    assert loss == pytest.approx(lo, rel=tol)
    assert rel <= tol


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("n", [1, 17, 4099])
def test_forward_noalloc_on_element_aligned_and_overlapping_buffers(n, shift):
    hip, net = pdhg._hip_runtime(), pdhg.Mlp(3)
    f, _ = _data(n, 5)
    want = net.forward(f)
    size = 4 * (18 * n + 64)
    buf, host = C.c_void_p(), np.zeros(18 * n + 64, dtype=np.float32)
    host[shift:shift + 16 * n] = f.reshape(-1)
    assert hip.hipMalloc(C.byref(buf), size) == 0
    try:
        for at in (shift + 16 * n, shift + 8 * n):  # after the features; inside them
            assert hip.hipMemcpy(buf, host.ctypes.data_as(C.c_void_p), size, 1) == 0
            net.forward_noalloc(C.c_void_p(buf.value + 4 * shift), n, C.c_void_p(buf.value + 4 * at))
            assert hip.hipDeviceSynchronize() == 0
            got = np.empty_like(host)
            assert hip.hipMemcpy(got.ctypes.data_as(C.c_void_p), buf, size, 2) == 0
            np.testing.assert_array_equal(got[at:at + n], want)
            np.testing.assert_array_equal(got[at + n:], host[at + n:])
    finally:
        hip.hipFree(buf)


@pytest.mark.parametrize("n", [3000, 20000, 65536])
def test_forward_noalloc_of_networks_by_turns_into_one_buffer(n):
    """Passes on the networks' own streams run in the order of the calls: the
    last one's logits are what the buffer holds."""
    hip = pdhg._hip_runtime()
    f, _ = _data(n, 5)
    for seed in range(6):
        nets = [pdhg.Mlp(seed + k) for k in (10, 20, 30)]
        want = nets[0].forward(f)
        got = np.empty(n, np.float32)
        df, dl = C.c_void_p(), C.c_void_p()
        assert hip.hipMalloc(C.byref(df), f.nbytes) == 0
        assert hip.hipMalloc(C.byref(dl), got.nbytes) == 0
        assert hip.hipMemcpy(df, f.ctypes.data_as(C.c_void_p), f.nbytes, 1) == 0
        for k in (0, 1, 2, 0, 1, 0):
            nets[k].forward_noalloc(df.value, n, dl.value)
        del nets[1]  # the networks share the stream
        assert hip.hipDeviceSynchronize() == 0
        assert hip.hipMemcpy(got.ctypes.data_as(C.c_void_p), dl, got.nbytes, 2) == 0
        np.testing.assert_array_equal(got, want)
        assert hip.hipFree(df) == 0 and hip.hipFree(dl) == 0


@pytest.mark.parametrize("n", [16384, 16385, 32769, 65520, 131089, 262145, 1048593])
def test_forward_of_many_tiles_a_wave_equals_that_of_its_parts(n):
    """One to sixteen tiles a wave, the last one of each wave missing or partial:
    a variable's logit does not depend on the others."""
    f, _ = _data(n, n)
    net = pdhg.Mlp(5)
    whole = net.forward(f)
    parts = np.concatenate([net.forward(f[k:k + 9999]) for k in range(0, n, 9999)])
    np.testing.assert_array_equal(whole, parts)
