"""Host-side tests of the C-ABI library: it loads, exports every declared symbol, its
host-only helpers agree with the stated layout, and argument validation returns status
codes before the device is touched.  No GPU needed."""
import ctypes
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def peqa():
    from paper_2305_14152_amd import peqa as p
    if not os.path.exists(p.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    p.lib()
    return p


def test_library_exports_every_declared_symbol(peqa):
    header = open(os.path.join(ROOT, "include", "peqa.h")).read()
    declared = set(re.findall(r"\b(peqa_[a-z_0-9]+)\s*\(", header))
    assert {"peqa_quantize", "peqa_linear_fwd", "peqa_linear_bwd", "peqa_scale_update"} <= declared
    L = ctypes.CDLL(peqa.LIB_PATH)
    for name in declared:
        assert hasattr(L, name), name
    assert declared == set(peqa.EXPORTS)


def test_layout_helpers(peqa):
    L = peqa.layout(4096, 11008, 4)
    assert peqa.check_layout(L) == peqa.PEQA_OK
    assert peqa.packed_words(L) == 4096 * 11008 * 4 // 32
    assert peqa.num_scales(L) == 4096
    L3 = peqa.layout(5120, 13824, 3, 128)
    assert peqa.packed_words(L3) == 5120 * 13824 * 3 // 32
    assert peqa.num_scales(L3) == 5120 * 108
    assert peqa.workspace_bytes(L, 2048, peqa.PEQA_OP_FWD) > 0
    assert peqa.workspace_bytes(L, 2048, peqa.PEQA_OP_BWD) > 2048 * 4096 * 2
    assert peqa.workspace_bytes(L, 0, peqa.PEQA_OP_FWD) == 0
    assert peqa.workspace_bytes(L, 8, 7) == 0


@pytest.mark.parametrize("args,status", [
    ((4096, 4096, 5, 0), 3), ((4096, 4096, 2, 0), 3), ((4000, 4096, 4, 0), 2), ((4096, 100, 4, 0), 2),
    ((0, 4096, 4, 0), 2), ((4096, 4096, 4, 96), 4), ((4096, 4096, 4, -1), 4), ((4096, 4096 + 128, 3, 256), 4),
])
def test_bad_layouts_are_rejected(peqa, args, status):
    L = peqa.layout(*args)
    assert peqa.check_layout(L) == status
    assert peqa.packed_words(L) == 0 and peqa.num_scales(L) == 0
    assert peqa.status_string(status) != "unknown status"


@pytest.mark.parametrize("bits", [3, 4])
def test_bit_location_matches_the_oracles_map(peqa, oracle, bits):
    """The library's statement of its packing layout against the oracle's independent one."""
    L = peqa.layout(256, 256, bits)
    r = np.random.default_rng(bits)
    pts = [(int(r.integers(256)), int(r.integers(256)), int(r.integers(bits))) for _ in range(500)]
    pts += [(i, k, t) for i in range(8) for k in range(8) for t in range(bits)]
    for (i, k, t) in pts:
        assert peqa.bit_location(L, i, k, t) == oracle.bit_location(256, bits, i, k, t)
    with pytest.raises(peqa.PeqaError):
        peqa.bit_location(L, 256, 0, 0)


def test_argument_validation_needs_no_device(peqa):
    L = peqa.layout(256, 256, 4)
    good, bad = 0x10000, 0x10004            # never dereferenced: validation fails first
    lib = peqa.lib()
    byref = ctypes.byref
    assert lib.peqa_quantize(byref(L), None, good, good, good, None) == peqa.PEQA_ERR_NULL
    assert lib.peqa_quantize(byref(L), good, bad, good, good, None) == peqa.PEQA_ERR_ALIGN
    assert lib.peqa_quantize(None, good, good, good, good, None) == peqa.PEQA_ERR_NULL
    Lbad = peqa.layout(256, 256, 7)
    assert lib.peqa_quantize(byref(Lbad), good, good, good, good, None) == peqa.PEQA_ERR_BITS
    f = lib.peqa_linear_fwd
    assert f(byref(L), good, good, None, good, None, 8, good, good, 1 << 20, None) == peqa.PEQA_ERR_NULL
    assert f(byref(L), good, good, None, good, good, 0, good, good, 1 << 20, None) == peqa.PEQA_ERR_SHAPE
    assert f(byref(L), good, good, bad, good, good, 8, good, good, 1 << 20, None) == peqa.PEQA_ERR_ALIGN
    assert f(byref(L), good, good, None, good, good, 8, good, None, 0, None) == peqa.PEQA_ERR_WORKSPACE
    assert f(byref(L), good, good, None, good, good, 8, good, good, 16, None) == peqa.PEQA_ERR_WORKSPACE
    b = lib.peqa_linear_bwd
    assert b(byref(L), good, good, None, good, good, None, 8, good, good, good, 1 << 30, None) == peqa.PEQA_ERR_NULL
    assert b(byref(L), good, good, None, good, None, good, 8, None, good, good, 1 << 30, None) == peqa.PEQA_ERR_NULL
    assert b(byref(L), good, good, None, good, good, good, 8, good, good, good, 64, None) == peqa.PEQA_ERR_WORKSPACE
    opt = peqa.AdamW(1e-3, 0.9, 0.999, 1e-8, 0.0, 0)
    u = lib.peqa_scale_update
    assert u(16, good, good, good, good, good, byref(opt), None) == peqa.PEQA_ERR_PARAM
    opt.step = 1
    assert u(16, good, None, good, good, good, byref(opt), None) == peqa.PEQA_ERR_NULL
    assert u(0, good, good, good, good, good, byref(opt), None) == peqa.PEQA_ERR_SHAPE
    opt.beta1 = 1.0
    assert u(16, good, good, good, good, good, byref(opt), None) == peqa.PEQA_ERR_PARAM


def test_kept_product_validation_needs_no_device(peqa):
    L, Lg = peqa.layout(256, 256, 4), peqa.layout(256, 256, 4, 128)
    good, bad = 0x10000, 0x10004
    lib, byref = peqa.lib(), ctypes.byref
    assert peqa.workspace_bytes(L, 100, peqa.PEQA_OP_FWD_KEEP) > 0
    assert peqa.workspace_bytes(L, 100, peqa.PEQA_OP_BWD_KEPT) >= 100 * 256 * 2 + 2 * 256 * 4
    assert peqa.workspace_bytes(Lg, 100, peqa.PEQA_OP_FWD_KEEP) == 0
    assert peqa.workspace_bytes(Lg, 100, peqa.PEQA_OP_BWD_KEPT) == 0
    assert peqa.workspace_bytes(L, 100, 9) == 0
    f = lib.peqa_linear_fwd_keep
    assert f(byref(Lg), good, good, None, good, good, 8, good, good, good, 1 << 20, None) == peqa.PEQA_ERR_GROUP
    assert f(byref(L), good, good, None, good, good, 8, good, None, good, 1 << 20, None) == peqa.PEQA_ERR_NULL
    assert f(byref(L), good, good, None, good, good, 8, good, bad, good, 1 << 20, None) == peqa.PEQA_ERR_ALIGN
    assert f(byref(L), good, good, None, good, good, 8, good, good, good, 16, None) == peqa.PEQA_ERR_WORKSPACE
    b = lib.peqa_linear_bwd_kept
    assert b(byref(Lg), good, good, None, good, good, good, 8, good, good, good, 1 << 30, None) == peqa.PEQA_ERR_GROUP
    assert b(byref(L), good, good, None, good, None, good, 8, good, good, good, 1 << 30, None) == peqa.PEQA_ERR_NULL
    assert b(byref(L), good, good, None, good, good, None, 8, good, good, good, 1 << 30, None) == peqa.PEQA_ERR_NULL
    assert b(byref(L), good, good, None, good, good, good, 8, good, good, good, 64, None) == peqa.PEQA_ERR_WORKSPACE


def test_zero_point_training_validation_needs_no_device(peqa):
    L, Lg = peqa.layout(256, 256, 4), peqa.layout(256, 256, 4, 128)
    good, bad = 0x10000, 0x10004
    lib, byref = peqa.lib(), ctypes.byref
    assert peqa.workspace_bytes(L, 100, peqa.PEQA_OP_FWD_Z) == peqa.workspace_bytes(L, 100, peqa.PEQA_OP_FWD)
    for lay in (L, Lg):
        assert peqa.workspace_bytes(lay, 100, peqa.PEQA_OP_BWD_Z) > peqa.workspace_bytes(lay, 100, peqa.PEQA_OP_BWD)
    f = lib.peqa_linear_fwd_z
    assert f(byref(L), good, good, None, good, bad, good, 8, good, good, 1 << 20, None) == peqa.PEQA_ERR_ALIGN
    assert f(byref(L), good, good, None, good, good, None, 8, good, good, 1 << 20, None) == peqa.PEQA_ERR_NULL
    assert f(byref(L), good, good, None, good, good, good, 8, good, good, 16, None) == peqa.PEQA_ERR_WORKSPACE
    b = lib.peqa_linear_bwd_z
    # the zero-point gradient needs X
    assert b(byref(L), good, good, None, good, None, None, good, 8, None, None, good, good, 1 << 30, None) == peqa.PEQA_ERR_NULL
    assert b(byref(L), good, good, None, good, None, good, good, 8, None, None, bad, good, 1 << 30, None) == peqa.PEQA_ERR_ALIGN
    need = peqa.workspace_bytes(L, 8, peqa.PEQA_OP_BWD_Z)
    assert b(byref(L), good, good, None, good, None, good, good, 8, good, good, good, good, need - 1, None) == peqa.PEQA_ERR_WORKSPACE


def test_quantize_search_validation_needs_no_device(peqa):
    L = peqa.layout(256, 256, 4)
    good, bad = 0x10000, 0x10004
    f, byref = peqa.lib().peqa_quantize_search, ctypes.byref
    assert f(byref(L), good, 0, 0.5, good, good, good, None) == peqa.PEQA_ERR_PARAM
    assert f(byref(L), good, 8, 0.0, good, good, good, None) == peqa.PEQA_ERR_PARAM
    assert f(byref(L), good, 8, 1.5, good, good, good, None) == peqa.PEQA_ERR_PARAM
    assert f(byref(L), None, 8, 0.5, good, good, good, None) == peqa.PEQA_ERR_NULL
    assert f(byref(L), good, 8, 0.5, bad, good, good, None) == peqa.PEQA_ERR_ALIGN
    # rows that do not fit on chip are refused, not mis-handled
    assert f(byref(peqa.layout(128, 22016, 4)), good, 8, 0.5, good, good, good, None) == peqa.PEQA_ERR_SHAPE
    assert f(byref(peqa.layout(128, 12288, 4, 64)), good, 8, 0.5, good, good, good, None) == peqa.PEQA_ERR_SHAPE


def test_scale_update_multi_validation_needs_no_device(peqa):
    good, bad = 0x10000, 0x10004
    lib, byref = peqa.lib(), ctypes.byref
    opt = peqa.AdamW(1e-3, 0.9, 0.999, 1e-8, 0.0, 1)
    def items(*rows):
        arr = (peqa.UpdateItem * len(rows))()
        for i, row in enumerate(rows):
            arr[i] = peqa.UpdateItem(*row)
        return arr
    f = lib.peqa_scale_update_multi
    ok = (16, good, good, good, good, good)
    arr = items(ok, ok)
    assert f(0, ctypes.addressof(arr), byref(opt), None) == peqa.PEQA_ERR_PARAM
    assert f(17, ctypes.addressof(arr), byref(opt), None) == peqa.PEQA_ERR_PARAM
    assert f(2, None, byref(opt), None) == peqa.PEQA_ERR_NULL
    arr = items(ok, (16, good, None, good, good, good))
    assert f(2, ctypes.addressof(arr), byref(opt), None) == peqa.PEQA_ERR_NULL
    arr = items(ok, (16, good, good, bad, good, good))
    assert f(2, ctypes.addressof(arr), byref(opt), None) == peqa.PEQA_ERR_ALIGN
    arr = items(ok, (0, good, good, good, good, good))
    assert f(2, ctypes.addressof(arr), byref(opt), None) == peqa.PEQA_ERR_SHAPE
    opt.step = 0
    arr = items(ok)
    assert f(1, ctypes.addressof(arr), byref(opt), None) == peqa.PEQA_ERR_PARAM


def test_row_sums_validation_needs_no_device(peqa):
    good, bad = 0x10000, 0x10004
    f = peqa.lib().peqa_row_sums
    assert f(None, 8, 256, good, None) == peqa.PEQA_ERR_NULL
    assert f(good, 0, 256, good, None) == peqa.PEQA_ERR_SHAPE
    assert f(good, 8, 192, good, None) == peqa.PEQA_ERR_SHAPE
    assert f(good, 8, 256, bad, None) == peqa.PEQA_ERR_ALIGN
    L = peqa.layout(256, 256, 4)
    b = peqa.lib().peqa_linear_bwd_rs
    assert b(ctypes.byref(L), good, good, None, good, good, bad, good, 8, good, good, good, 1 << 30, None) == peqa.PEQA_ERR_ALIGN


def test_fused_forward_validation_needs_no_device(peqa):
    a, b = peqa.layout(256, 512, 4), peqa.layout(128, 512, 4)
    assert peqa.workspace_bytes_fused([(a, 16, 16, None, 16, 16), (b, 16, 16, None, 16, 16)], 4) > 0
    odd = peqa.layout(128, 256, 4)                      # another K
    assert peqa.workspace_bytes_fused([(a, 16, 16, None, 16, 16), (odd, 16, 16, None, 16, 16)], 4) == 0
    with pytest.raises(peqa.PeqaError):
        peqa.linear_fwd_fused([(a, 16, 16, None, 16, 16), (odd, 16, 16, None, 16, 16)], 16, 4, 16, 1 << 20, stream=0)
    with pytest.raises(peqa.PeqaError):                 # too many layers
        peqa.linear_fwd_fused([(a, 16, 16, None, 16, 16)] * 5, 16, 4, 16, 1 << 20, stream=0)
    with pytest.raises(peqa.PeqaError):                 # a NULL output
        peqa.linear_fwd_fused([(a, 16, 16, None, 16, None)], 16, 4, 16, 1 << 20, stream=0)


def test_product_package_does_not_touch_the_oracle():
    """The product path may not import, read or link anything under oracle/."""
    pkg = os.path.join(ROOT, "paper_2305_14152_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.lower() or f == "synth.py", f


def test_fp64_reciprocal_product_is_the_correctly_rounded_fp32_quotient():
    """The quantize kernels take w / s as (float)((double)w * (1.0 / (double)s)).  The identity with the
    correctly rounded fp32 divide (what Eq. 1's reference arithmetic uses) is checked here on the host:
    random operands over many binades, the operand ranges the quantizer sees, and quotients placed next
    to points midway between two fp32 numbers."""
    rng = np.random.default_rng(2024)

    def check(w, s):
        w = w.astype(np.float32)
        s = s.astype(np.float32)
        ref = w / s                                                   # IEEE fp32 divide
        alt = (w.astype(np.float64) * (1.0 / s.astype(np.float64))).astype(np.float32)
        bad = np.nonzero(ref.view(np.uint32) != alt.view(np.uint32))[0]
        assert bad.size == 0, (w[bad[:3]], s[bad[:3]])

    n = 2_000_000
    check(rng.standard_normal(n) * 0.02, np.abs(rng.standard_normal(n)) * 0.01 + 1e-4)
    check(np.ldexp(rng.uniform(1, 2, n), rng.integers(-60, 60, n)) * rng.choice([-1.0, 1.0], n),
          np.ldexp(rng.uniform(1, 2, n), rng.integers(-60, 60, n)))
    # quotients as close to a midpoint as fp32 operands allow: w = fl(m * s) for 25-bit odd m
    m = (rng.integers(1 << 23, 1 << 24, n).astype(np.float64) * 2 + 1) / (1 << 24)      # 25 significant bits
    s = rng.integers(1 << 23, 1 << 24, n).astype(np.float64) / (1 << 23)
    for nudge in (0, 1, -1):
        w = (m * s).astype(np.float32)
        w = (w.view(np.int32) + nudge).view(np.float32)
        check(w, s)


def test_options_are_explicit_and_validated(peqa):
    """The test switches are set through peqa_set_option only (nothing is read from the environment); unknown
    options and values are refused and change nothing."""
    assert peqa.get_option(peqa.PEQA_OPT_GEMM_WAVES) == 0
    assert peqa.get_option(peqa.PEQA_OPT_BWD_PAIR) == -1
    assert peqa.get_option(peqa.PEQA_OPT_GROUPED_DDS) == 0
    lib = peqa.lib()
    for opt, bad in ((peqa.PEQA_OPT_GEMM_WAVES, 2), (peqa.PEQA_OPT_BWD_PAIR, 2), (peqa.PEQA_OPT_GROUPED_DDS, -1), (99, 0)):
        assert lib.peqa_set_option(opt, bad) == peqa.PEQA_ERR_PARAM
    assert peqa.get_option(99) == -2 ** 31
    try:
        peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 8)
        assert peqa.get_option(peqa.PEQA_OPT_GEMM_WAVES) == 8
    finally:
        peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 0)
    src = "".join(open(os.path.join(ROOT, "paper_2305_14152_amd", "csrc", f)).read()
                  for f in os.listdir(os.path.join(ROOT, "paper_2305_14152_amd", "csrc")))
    assert "getenv" not in src


@pytest.mark.parametrize("N,K,bits,group,T", [
    (135808, 9216, 3, 64, 16), (144384, 15872, 4, 256, 13), (154624, 26112, 4, 192, 13), (409472, 8192, 4, 256, 10),
    (4096, 4096, 4, 0, 16), (256, 49152, 3, 0, 5), (184576, 35200, 4, 64, 12), (5504, 4096, 3, 128, 17), (256, 8192, 4, 0, 40),
])
def test_static_forward_takes_only_what_runs_alike_in_its_scratch(peqa, N, K, bits, group, T):
    """What peqa_linear_fwd_static accepts has to run as peqa_linear_fwd does with the workspace it asks for, so that
    workspace must fit the static scratch: the same slices, the same pieces, the same bits."""
    L = peqa.layout(N, K, bits, group)
    refused = peqa.lib().peqa_linear_fwd_static(ctypes.byref(L), None, None, None, None, None, T, None, None)
    assert refused in (peqa.PEQA_ERR_WORKSPACE, peqa.PEQA_ERR_NULL)     # (the size is looked at before the pointers)
    assert (refused == peqa.PEQA_ERR_WORKSPACE) == (peqa.workspace_bytes(L, T, peqa.PEQA_OP_FWD) > peqa.STATIC_SCRATCH_BYTES)


@pytest.mark.parametrize("bits,N,K,group,T", [(4, 384, 1152, 64, 70), (3, 640, 1280, 128, 200), (3, 256, 768, 192, 33), (4, 128, 1024, 512, 300)])
def test_group_wise_backward_asks_for_what_it_uses(peqa, bits, N, K, group, T):
    """Whole contractions (a forced form): table, group sums and partials, transposed copies, and the chunk sums of groups
    of more than 128 features; groups of 64 and 128 are complete in the token contraction's tiles."""
    def r(n):
        return (n + 255) // 256 * 256
    G, Tp, tiles = K // group, (T + 63) // 64 * 64, (T + 127) // 128
    chunks = r(4 * N * (K // 64)) if group > 128 else 0
    L = peqa.layout(N, K, bits, group)
    peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 4)
    try:
        single = peqa.workspace_bytes(L, T, peqa.PEQA_OP_BWD)
        block = peqa.block_workspace_bytes(peqa.block_items([dict(L=L, packed=None, s0=None, z0=None)]), T, peqa.PEQA_OP_BWD)
    finally:
        peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 0)
    assert single == r(8 * N * G) + r(4 * T * G) + r(4 * tiles * N * G) + r(2 * K * Tp) + r(2 * N * Tp) + chunks
    assert block == r(8 * N * G) + r(2 * K * Tp) + r(2 * N * Tp) + chunks


_QUERIES = """
import ctypes, sys
lib = ctypes.CDLL(sys.argv[1])
class Layout(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("n_out", "k_in", "bits", "group_size")]
class Fused(ctypes.Structure):
    _fields_ = [("layout", Layout)] + [(n, ctypes.c_void_p) for n in ("packed", "s0", "ds", "z0", "Y")]
class Item(ctypes.Structure):
    _fields_ = [("layout", Layout)] + [(n, ctypes.c_void_p) for n in ("packed", "s0", "ds", "z0", "X", "Y", "dY", "dX", "d_ds", "row_sums")]
p = ctypes.c_void_p(4096)
for group in (0, 128):
    L = Layout(4096, 11008, 4, group)
    fused, item = Fused(layout=L), Item(layout=L, packed=4096, s0=4096, z0=4096, X=4096, Y=4096, dY=4096, d_ds=4096)
    for T in (1, 40, 2048):
        for op in range(6):
            lib.peqa_workspace_bytes(ctypes.byref(L), T, op)
        lib.peqa_workspace_bytes_fused(1, ctypes.byref(fused), T)
        for op in (0, 1):
            lib.peqa_block_workspace_bytes(1, ctypes.byref(item), T, op)
        # calls that are refused: no workspace
        assert lib.peqa_linear_fwd(ctypes.byref(L), p, p, None, p, p, T, p, None, ctypes.c_size_t(0), None) == 6
        assert lib.peqa_linear_bwd(ctypes.byref(L), p, p, None, p, p, p, T, p, p, None, ctypes.c_size_t(0), None) == 6
        assert lib.peqa_block_fwd(1, ctypes.byref(item), T, None, ctypes.c_size_t(0), None) == 6
        assert lib.peqa_block_bwd(1, ctypes.byref(item), T, None, ctypes.c_size_t(0), None) == 6
        assert lib.peqa_linear_fwd_static(ctypes.byref(L), None, p, None, p, p, T, p, None) in (1, 6)
print("QUERIES DONE", file=sys.stderr, flush=True)
a, b = ctypes.c_int32(), ctypes.c_int32()
lib.peqa_device_info(ctypes.byref(a), ctypes.byref(b))
"""


def test_queries_and_refusals_do_not_touch_the_device(peqa):
    """The size queries are host-only, and a call that is refused is refused before the runtime is asked for a device: the
    HIP runtime's own call log stays empty until the one call that does ask."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, "-c", _QUERIES, peqa.LIB_PATH], stderr=subprocess.PIPE, text=True, timeout=120,
                       env=dict(os.environ, AMD_LOG_LEVEL="3"))
    assert r.returncode == 0, r.stderr[-2000:]
    before, _, after = r.stderr.partition("QUERIES DONE")
    if "hipGetDevice" not in after:
        pytest.skip("this HIP runtime writes no call log")
    assert "hip" not in before.replace(peqa.LIB_PATH, ""), before[-2000:]


def test_item_arrays_take_and_refuse_what_the_structures_do(peqa):
    """Items of the fused forward and of the joint update, marshalled as bytes: the same bytes as ctypes' own structures, a
    layout given as a tuple, numbers modulo 2^64, TypeError for what is no layout, PeqaError for a negative n_scales."""
    L, good = peqa.layout(256, 512, 3, 128), 0x10000
    want = bytes(peqa.FwdItem(L, good, good, None, good, 2 ** 63))
    assert peqa._items([(L, good, good, None, good, 2 ** 63)] * 2) == 2 * want
    assert peqa._items([((256, 512, 3, 128), good, good, None, good, 2 ** 63)]) == want
    assert peqa._items([(L, good, good, 2 ** 64, good, 2 ** 63 - 2 ** 64)]) == want
    assert peqa.workspace_bytes_fused([((256, 256, 4, 0), 16, 16, None, 16, 16)], 4) > 0
    for bad in (b"x" * 16, b"x" * 40, 16, None, [256, 256, 4, 0], peqa.AdamW()):
        with pytest.raises(TypeError):
            peqa.workspace_bytes_fused([(bad, 16, 16, None, 16, 16)], 4)
    for n, status in ((-1, peqa.PEQA_ERR_SHAPE), (2 ** 64, peqa.PEQA_ERR_SHAPE), (0, peqa.PEQA_ERR_SHAPE)):
        with pytest.raises(peqa.PeqaError) as e:
            peqa.scale_update_multi([(n, good, good, good, good, good)], 1e-3, stream=0)
        assert e.value.status == status
    with pytest.raises(peqa.PeqaError) as e:
        peqa.scale_update_multi([(16, good, None, good, good, 2 ** 64 + good)], 1e-3, stream=0)
    assert e.value.status == peqa.PEQA_ERR_NULL
