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


@pytest.mark.parametrize("N,K,T,group,rows", [
    (14336, 512, 530, 0, 4), (14336, 512, 530, 128, 6), (16384, 512, 400, 0, 4), (16384, 512, 400, 128, 7),
    (2304, 512, 256, 0, 4), (13184, 512, 640, 0, 6), (17152, 896, 490, 0, 7), (2304, 512, 256, 128, 4), (16640, 512, 1024, 128, 6),
    (11008, 2048, 490, 64, 7),
])
def test_fewer_rows_where_idle(gpu, oracle, N, K, T, group, rows):
    """Whole contractions planned in tiles of 64, 96 and 112 rows, all but one where gemm_row_tiles gives more (112 at T = 530 and
    400, else 128): the bits of that height's tiles, which a form that is asked for has, and rows of Y against the oracle."""
    from paper_2305_14152_amd import peqa
    from test_plan_host import Planner
    print("fewer rows, N=%d K=%d T=%d group=%d" % (N, K, T, group), flush=True)
    assert Planner(peqa.lib()).plan([(N, K, 4 * T * N)], T, group > 0, True, most=peqa.STATIC_SCRATCH_BYTES) == (rows, [1])
    seed = 83000 + N + T + group
    W = synth.normal_f32(seed, (N, K), 0.02)
    layer = gpu.GpuLayer(W, 4, group)
    X = synth.normal_bf16(seed + 1, (T, K), 1.0)
    Ydev, forms = layer.fwd(X), []
    Y = gpu.to_host(Ydev)
    for waves in (4, 8):
        peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, waves)
        try:
            forms.append(gpu.to_host(layer.fwd(X)))
        finally:
            peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 0)
    assert np.abs(Y).max() > 0 and any((Y == f).all() for f in forms)
    codes, s0, z0 = oracle.quantize(W, 4, group)
    some = [0, 63, 64, 95, 96, 111, 112, 127, 128, T - 1]
    Yref = oracle.fwd(codes, s0, None, z0, X[some], group)
    assert np.abs(gpu.bf16_dev_to_f64(Ydev)[some] - Yref).max() <= Y_TOL * np.abs(Yref).max()


@pytest.mark.parametrize("group", [64, 128, 256])
@pytest.mark.parametrize("N,K,T", [(4096, 4096, 900), (3072, 4096, 900), (3200, 4096, 1000)])
def test_few_long_chains_of_the_backward(gpu, N, K, T, group):
    """Group-wise backward on both sides of the rule that takes few, long and whole dX contractions out of the token
    contractions' launch: whole contractions, so the bits of a forced form; the block call agrees."""
    import torch
    from paper_2305_14152_amd import peqa
    from test_plan_host import Planner
    planner, beside = Planner(peqa.lib()), (K // 128) * ((N + 255) // 256) * (0.55 * ((T + 63) // 64 * 2) + 8)
    jobs = [(K, N, 4 * T * K)]
    assert planner.plan(jobs, T, True, False, other=beside)[1] == [1]
    assert planner.chains(jobs, [1], T) == (N > 3072)
    print("chains, N=%d K=%d T=%d group=%d" % (N, K, T, group), flush=True)
    seed = 84000 + N + T + group
    layer = gpu.GpuLayer(synth.normal_f32(seed, (N, K), 0.02), 4, group)
    X, dY = synth.normal_bf16(seed + 1, (T, K), 1.0), synth.normal_bf16(seed + 2, (T, N), 1.0)
    peqa.trace_begin(16)
    dX, g = (gpu.to_host(v) for v in layer.bwd(X, dY))
    assert ("gemm_dx" in peqa.trace_end()) == (N > 3072)             # a launch of its own, or shared with the token contractions
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
