"""Codes at the midpoints between integers, where the rounding of the quotient decides, and at scales from the smallest to
the largest that fp32 holds: the quantizer against the oracle, bit for bit.  Rows in registers in each of the three lengths
and longer rows; one group per row, groups of one 64-feature segment, of several, and of two."""
import numpy as np
import pytest

from paper_2305_14152_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available()
    from paper_2305_14152_amd import peqa
    peqa.lib()
    import gpu_util
    return gpu_util


def _midpoints(seed, N, K, group, qmax, magnitude):
    """Rows whose weights lie on midpoints of their own scale, and an fp32 step to either side."""
    g = group or K
    W = np.zeros((N, K // g, g), np.float32)
    u = synth.normal_f32(seed, (N, K // g), 1.0)
    step = np.float32(magnitude) * (1 + np.abs(u)).astype(np.float32)
    W[:, :, 0], W[:, :, 1] = -step * np.float32(qmax // 2), step * np.float32(qmax - qmax // 2)
    s = (W[:, :, 1] - W[:, :, 0]) / np.float32(qmax)
    m = (np.arange(2, g) % qmax - qmax // 2).astype(np.float32)
    mid = s[:, :, None] * (m + np.float32(0.5))
    which = np.arange(2, g) // qmax % 3
    mid = np.where(which == 0, mid, np.nextafter(mid, np.where(which == 1, np.inf, -np.inf).astype(np.float32)))
    W[:, :, 2:] = np.clip(mid, W[:, :, :1], W[:, :, 1:2])
    return W.reshape(N, K)


@pytest.mark.parametrize("bits,K,group", [
    (4, 128, 0), (3, 4096, 0), (4, 4224, 0), (3, 8320, 0), (4, 12288, 0), (4, 12416, 0), (3, 12416, 0),
    (4, 384, 64), (3, 5376, 192), (4, 12288, 6144), (4, 16384, 128),
])
def test_codes_at_midpoints(gpu, oracle, bits, K, group):
    N = 128
    for magnitude in (1e-38, 3e-37, 0.01, 1e36):
        print("midpoints bits=%d K=%d g=%d magnitude=%g" % (bits, K, group, magnitude), flush=True)
        W = _midpoints(81000 + K + group, N, K, group, (1 << bits) - 1, magnitude)
        layer = gpu.GpuLayer(W, bits, group)
        codes, s0, z0 = oracle.quantize(W, bits, group)
        packed, gs0, gz0 = layer.host_quant()
        assert (gz0 == z0).all()
        assert (gs0.view(np.uint32) == s0.view(np.uint32)).all()
        assert (packed == oracle.pack(codes, bits)).all()
