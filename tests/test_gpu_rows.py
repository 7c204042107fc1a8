"""Tiles of 64, 96, 112 and 128 token rows (chosen by the number of tokens): every call against the oracle at the edges of
each, and Y and dX bit for bit against the same tokens in a call of 128-row tiles, since the rows of a tile do not change the
order in which a contraction is added up."""
import numpy as np
import pytest

from paper_2305_14152_amd import synth

pytestmark = pytest.mark.gpu

Y_TOL = 2e-2
EDGES = (17, 63, 64, 65, 96, 97, 112, 113, 129, 192, 193, 224, 225, 257, 288, 336, 337)


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available()
    from paper_2305_14152_amd import peqa
    peqa.lib()
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("bits,group", [(4, 0), (3, 0), (4, 64), (3, 128)])
def test_rows_of_a_tile(gpu, oracle, bits, group, waves):
    from paper_2305_14152_amd import peqa
    N, K, most = 384, 640, 384                     # an odd number of 128-wide units both ways; 384 tokens: 128-row tiles
    seed = 81000 + 10 * bits + group
    W = synth.normal_f32(seed, (N, K), 0.02)
    X, dY = synth.normal_bf16(seed + 1, (most, K), 1.0), synth.normal_bf16(seed + 2, (most, N), 1.0)
    layer = gpu.GpuLayer(W, bits, group)
    codes, s0, z0 = oracle.quantize(W, bits, group)
    ds = synth.normal_f32(seed + 3, s0.shape, 1e-3)
    Yref = oracle.fwd(codes, s0, ds, z0, X, group)
    peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, waves)
    try:
        Y128, dX128 = gpu.to_host(layer.fwd(X, ds)), gpu.to_host(layer.bwd(X, dY, ds)[0])
        assert np.abs(gpu.bf16_dev_to_f64(layer.fwd(X, ds)) - Yref).max() <= Y_TOL * np.abs(Yref).max()
        for T in EDGES:
            print("rows bits=%d g=%d waves=%d T=%d" % (bits, group, waves, T), flush=True)
            Y = layer.fwd(X[:T], ds)
            dX, g = layer.bwd(X[:T], dY[:T], ds)
            assert (gpu.to_host(Y) == Y128[:T]).all() and (gpu.to_host(dX) == dX128[:T]).all(), T
            dXref, gref, _ = oracle.bwd(codes, s0, ds, z0, X[:T], dY[:T], group)
            assert np.abs(gpu.bf16_dev_to_f64(dX) - dXref).max() <= Y_TOL * np.abs(dXref).max()
            gpu.assert_scale_grad_close(gpu.to_host(g), gref)
    finally:
        peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 0)


@pytest.mark.parametrize("T", [40, 90, 110, 180, 200, 300])
@pytest.mark.parametrize("bits", [3, 4])
def test_rows_of_a_tile_split_and_paired(gpu, oracle, bits, T):
    """Few tiles of a long contraction: pieces, the scale gradient's with row sums of their own; the block calls too."""
    import torch
    from paper_2305_14152_amd import peqa
    print("rows, split, bits=%d T=%d" % (bits, T), flush=True)
    N, K = 256, 6144
    seed = 82000 + 10 * bits + T
    W = synth.normal_f32(seed, (N, K), 0.02)
    X, dY = synth.normal_bf16(seed + 1, (T, K), 1.0), synth.normal_bf16(seed + 2, (T, N), 1.0)
    layer = gpu.GpuLayer(W, bits, 0)
    codes, s0, z0 = oracle.quantize(W, bits, 0)
    Yref = oracle.fwd(codes, s0, None, z0, X)
    dXref, gref, _ = oracle.bwd(codes, s0, None, z0, X, dY)
    assert peqa.workspace_bytes(layer.L, T, peqa.PEQA_OP_FWD) > 4 * T * N     # (pieces)
    d = dict(L=layer.L, packed=layer.packed, s0=layer.s0, z0=layer.z0, X=gpu.to_dev(X), dY=gpu.to_dev(dY),
             Y=torch.zeros((T, N), dtype=torch.int16, device="cuda"), dX=torch.zeros((T, K), dtype=torch.int16, device="cuda"),
             d_ds=torch.zeros((N, 1), dtype=torch.float32, device="cuda"))
    items = peqa.block_items([d])
    nb = max(peqa.block_workspace_bytes(items, T, op) for op in (peqa.PEQA_OP_FWD, peqa.PEQA_OP_BWD))
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    peqa.block_fwd(items, T, ws, nb)
    peqa.block_bwd(items, T, ws, nb)
    single = (layer.fwd(X),) + tuple(layer.bwd(X, dY))
    for Y, dX, g in (single, (d["Y"], d["dX"], d["d_ds"])):
        assert np.abs(gpu.bf16_dev_to_f64(Y) - Yref).max() <= Y_TOL * np.abs(Yref).max()
        assert np.abs(gpu.bf16_dev_to_f64(dX) - dXref).max() <= Y_TOL * np.abs(dXref).max()
        gpu.assert_scale_grad_close(gpu.to_host(g), gref)


@pytest.mark.parametrize("N,T", [(14336, 530), (16384, 400)])
@pytest.mark.parametrize("group", [0, 128])
def test_fewer_rows_where_idle(gpu, N, T, group):
    """Whole contractions that take tiles of 96 or 112 rows for their number: the bits of 128-row tiles, whose form is asked for."""
    from paper_2305_14152_amd import peqa
    print("fewer rows, N=%d T=%d group=%d" % (N, T, group), flush=True)
    K, seed = 512, 83000 + N + T + group
    layer = gpu.GpuLayer(synth.normal_f32(seed, (N, K), 0.02), 4, group)
    X = synth.normal_bf16(seed + 1, (T, K), 1.0)
    Y, forms = gpu.to_host(layer.fwd(X)), []
    for waves in (4, 8):
        peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, waves)
        try:
            forms.append(gpu.to_host(layer.fwd(X)))
        finally:
            peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 0)
    assert np.abs(Y).max() > 0 and any((Y == f).all() for f in forms)


@pytest.mark.parametrize("group", [64, 128, 256])
@pytest.mark.parametrize("N,K,T", [(4096, 4096, 900), (3072, 4096, 900), (3200, 4096, 1000)])
def test_few_long_chains_of_the_backward(gpu, N, K, T, group):
    """Group-wise backward on both sides of the rule that takes few, long and whole dX contractions out of the token
    contractions' launch: whole contractions, so the bits of a forced form; the block call agrees."""
    import torch
    from paper_2305_14152_amd import peqa
    print("chains, N=%d K=%d T=%d group=%d" % (N, K, T, group), flush=True)
    seed = 84000 + N + T + group
    layer = gpu.GpuLayer(synth.normal_f32(seed, (N, K), 0.02), 4, group)
    X, dY = synth.normal_bf16(seed + 1, (T, K), 1.0), synth.normal_bf16(seed + 2, (T, N), 1.0)
    dX, g = (gpu.to_host(v) for v in layer.bwd(X, dY))
    forms = []
    for waves in (4, 8):
        peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, waves)
        try:
            forms.append([gpu.to_host(v) for v in layer.bwd(X, dY)])
        finally:
            peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 0)
    assert np.abs(dX).max() > 0 and any((dX == f[0]).all() for f in forms)
    assert (g == forms[0][1]).all()
    d = dict(L=layer.L, packed=layer.packed, s0=layer.s0, z0=layer.z0, X=gpu.to_dev(X), dY=gpu.to_dev(dY),
             Y=torch.zeros((T, N), dtype=torch.int16, device="cuda"), dX=torch.zeros((T, K), dtype=torch.int16, device="cuda"),
             d_ds=torch.zeros_like(layer.s0))
    items = peqa.block_items([d])
    nb = peqa.block_workspace_bytes(items, T, peqa.PEQA_OP_BWD)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    peqa.block_bwd(items, T, ws, nb)
    assert any((gpu.to_host(d["dX"]) == f[0]).all() for f in forms)
    assert (gpu.to_host(d["d_ds"]).reshape(g.shape) == g).all()
