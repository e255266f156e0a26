"""CPU tests of libbitcos.so: exported symbols, host packers vs the oracle, error codes.

The packers are C++ written independently of the oracle; their blobs must be
byte-identical to the oracle's serialisation of the same (W, scales, unit).
No GPU work is done here.
"""

import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

import oracle as O
import workloads as wl

api = pytest.importorskip("paper_2609_16338_amd.api")
from paper_2609_16338_amd import _native as N  # noqa: E402

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "bitcos.h")


def header_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"^\s*(?:const\s+)?\w+\**\s+\**(\w+)\s*\(", text, flags=re.M)))


def test_library_loads_and_exports_every_declared_function():
    names = header_functions()
    assert "bitcos_gemv" in names and "bit2_unpack" in names and len(names) == 24
    lib = N.lib()
    for nm in names:
        assert hasattr(lib, nm), nm
    out = subprocess.run(["nm", "-D", "--defined-only", N.LIB_PATH], capture_output=True, text=True).stdout
    exported = set(re.findall(r"\sT\s(\w+)$", out, flags=re.M))
    assert set(names) <= exported
    assert set(names) == set(N.SIGNATURES)


def test_version_and_strerror():
    assert N.lib().bitcos_version() == N.LAYOUT_VERSION
    for st in (N.OK, N.E_ARG, N.E_VALUE, N.E_SPACE, N.E_HIP, N.E_UNSUPPORTED):
        assert N.strerror(st)
    assert N.strerror(-99) == "unknown status"


def test_layout_struct_size():
    assert ctypes.sizeof(N.Layout) == 112
    assert ctypes.sizeof(N.LaunchInfo) == 40


ENC = {N.FMT_BITCOS: O.bitcos_encode, N.FMT_TRIT5: O.trit5_encode, N.FMT_BIT2: O.bit2_encode}


def _oracle_blob(fmt, w, sc, group, unit):
    p = O.bitcos_encode(w, sc, group, unit) if fmt == N.FMT_BITCOS else ENC[fmt](w, sc, group)
    return p, O.serialize(p)


@pytest.mark.parametrize("fmt", [N.FMT_BITCOS, N.FMT_TRIT5, N.FMT_BIT2])
@pytest.mark.parametrize("z", [0.0, 0.3, 0.42, 0.5, 1.0])
@pytest.mark.parametrize("group", [128, 0])
def test_packers_match_oracle_bytes(fmt, z, group):
    for (n, k) in [(1, 128), (7, 384), (33, 1024), (5, 2560)]:
        w = wl.ternary(n, k, z, wl.rng_for(40, n, k, int(z * 100)))
        ns = n * k // 128 if group else 1
        sc = wl.fp16_uniform((ns,), 0.005, 0.1, wl.rng_for(41, n))
        unit = 3 if fmt == N.FMT_BITCOS else 0
        if fmt == N.FMT_BITCOS:
            L = api.bitcos_plan(w, group, unit)
        else:
            L = api.trit5_plan(w, group) if fmt == N.FMT_TRIT5 else api.bit2_plan(w, group)
        blob = {N.FMT_BITCOS: api.bitcos_pack, N.FMT_TRIT5: api.trit5_pack, N.FMT_BIT2: api.bit2_pack}[fmt](w, sc, L)
        p, (ob, offs) = _oracle_blob(fmt, w, sc, group, unit)
        assert bytes(blob) == ob
        assert L.total_bytes == len(ob)
        assert L.payload_bits == O.payload_bits(p)
        assert L.nnz == int(np.count_nonzero(w))
        idx = [0, 1, 2, 3] if fmt == N.FMT_BITCOS else [0, 3]
        assert [(L.sec_off[i], L.sec_bytes[i]) for i in idx] == offs
        unpack = {N.FMT_BITCOS: api.bitcos_unpack, N.FMT_TRIT5: api.trit5_unpack, N.FMT_BIT2: api.bit2_unpack}[fmt]
        w2, s2 = unpack(L, blob)
        assert np.array_equal(w2, w) and np.array_equal(s2, sc)


def test_bitcos_per_tensor_k_multiple_of_32():
    w = wl.ternary(5, 96, 0.4, wl.rng_for(42))
    sc = np.array([0x2E66], np.uint16)
    L = api.bitcos_plan(w, 0, 2)
    blob = api.bitcos_pack(w, sc, L)
    assert bytes(blob) == O.serialize(O.bitcos_encode(w, sc, 0, 2))[0]


def test_default_unit_rows_is_positive_and_oracle_agrees():
    w = wl.ternary(100, 2560, 0.42, wl.rng_for(43))
    sc = np.array([0x2E66], np.uint16)
    L = api.bitcos_plan(w, 0, 0)
    assert L.unit_rows >= 1
    assert bytes(api.bitcos_pack(w, sc, L)) == O.serialize(O.bitcos_encode(w, sc, 0, L.unit_rows))[0]


def test_payload_bits_exact_two_minus_z():
    n, k = 64, 1024
    w = wl.ternary(n, k, 0.5, wl.rng_for(44))
    L = api.bitcos_plan(w, 128, 0)
    zeros = int(np.count_nonzero(w == 0))
    assert L.payload_bits == n * k + (n * k - zeros) + 16 * n * (k // 128)


def _status(fn, *args):
    return getattr(N.lib(), fn)(*args)


def test_error_codes():
    L = N.Layout()
    w = np.zeros((4, 128), np.int8)
    p = ctypes.c_void_p(w.ctypes.data)
    assert _status("bitcos_plan", None, 4, 128, 128, 0, ctypes.byref(L)) == N.E_ARG
    assert _status("bitcos_plan", p, 0, 128, 128, 0, ctypes.byref(L)) == N.E_ARG
    assert _status("bitcos_plan", p, 4, 100, 128, 0, ctypes.byref(L)) == N.E_ARG    # K % 128
    assert _status("bitcos_plan", p, 4, 128, 64, 0, ctypes.byref(L)) == N.E_ARG     # bad group
    assert _status("bitcos_plan", p, 4, 128, 128, -1, ctypes.byref(L)) == N.E_ARG
    assert _status("trit5_plan", p, 4, 96, 0, ctypes.byref(L)) == N.E_ARG          # blocks of 128
    bad = w.copy()
    bad[1, 5] = 3
    assert _status("bitcos_plan", ctypes.c_void_p(bad.ctypes.data), 4, 128, 128, 0, ctypes.byref(L)) == N.E_VALUE
    assert _status("bit2_plan", ctypes.c_void_p(bad.ctypes.data), 4, 128, 128, ctypes.byref(L)) == N.E_VALUE
    # pack: scale checks and capacity
    L = api.bitcos_plan(w, 128, 0)
    dst = np.zeros(L.total_bytes, np.uint8)
    neg = np.full(4, 0xBC00, np.uint16)
    inf = np.full(4, 0x7C00, np.uint16)
    ok = np.full(4, 0x3C00, np.uint16)
    d = ctypes.c_void_p(dst.ctypes.data)
    assert _status("bitcos_pack", p, ctypes.c_void_p(neg.ctypes.data), ctypes.byref(L), d, dst.nbytes) == N.E_VALUE
    assert _status("bitcos_pack", p, ctypes.c_void_p(inf.ctypes.data), ctypes.byref(L), d, dst.nbytes) == N.E_VALUE
    assert _status("bitcos_pack", p, ctypes.c_void_p(ok.ctypes.data), ctypes.byref(L), d, dst.nbytes - 1) == N.E_SPACE
    # W different from the one planned (more non-zeros) is rejected
    more = np.ones((4, 128), np.int8)
    assert _status("bitcos_pack", ctypes.c_void_p(more.ctypes.data), ctypes.c_void_p(ok.ctypes.data),
                   ctypes.byref(L), d, dst.nbytes) == N.E_VALUE
    assert _status("bitcos_pack", p, ctypes.c_void_p(ok.ctypes.data), ctypes.byref(L), d, dst.nbytes) == N.OK
    # wrong version / format
    L2 = N.Layout.from_buffer_copy(L)
    L2.version = 99
    assert _status("bitcos_pack", p, ctypes.c_void_p(ok.ctypes.data), ctypes.byref(L2), d, dst.nbytes) == N.E_ARG
    L3 = N.Layout.from_buffer_copy(L)
    L3.format = N.FMT_TRIT5
    assert _status("bitcos_unpack", ctypes.byref(L3), d, dst.nbytes, p, ctypes.c_void_p(ok.ctypes.data)) == N.E_ARG


def test_unpack_detects_corruption():
    w = wl.ternary(6, 256, 0.4, wl.rng_for(45))
    sc = wl.fp16_uniform((12,), 0.01, 0.1, wl.rng_for(46))
    L = api.bitcos_plan(w, 128, 2)
    blob = api.bitcos_pack(w, sc, L)
    bad = blob.copy()
    bad[L.sec_off[N.SEC_OFFSETS] + 4] ^= 1          # a unit offset
    with pytest.raises(N.BitcosError):
        api.bitcos_unpack(L, bad)
    bad = blob.copy()
    bad[L.sec_off[N.SEC_BITMAP]] ^= 0x10            # one presence bit -> popcount != nnz
    with pytest.raises(N.BitcosError):
        api.bitcos_unpack(L, bad)
    Lt = api.trit5_plan(w, 128)
    bt = api.trit5_pack(w, sc, Lt)
    bt[Lt.sec_off[N.SEC_CODES]] = 250               # not a five-trit byte
    with pytest.raises(N.BitcosError):
        api.trit5_unpack(Lt, bt)
    Lb = api.bit2_plan(w, 128)
    bb = api.bit2_pack(w, sc, Lb)
    bb[Lb.sec_off[N.SEC_CODES]] |= 3                # code 3
    with pytest.raises(N.BitcosError):
        api.bit2_unpack(Lb, bb)


def test_gemv_validation_happens_before_any_device_work():
    # No GPU needed: every one of these is rejected by the host checks.
    w = wl.ternary(4, 256, 0.4, wl.rng_for(47))
    L = api.bitcos_plan(w, 128, 0)
    dummy = ctypes.c_void_p(16)
    g = N.lib().bitcos_gemv
    assert g(ctypes.byref(L), None, 1, dummy, N.X_I8, None, dummy, N.Y_F32, None) == N.E_ARG
    assert g(ctypes.byref(L), dummy, 0, dummy, N.X_I8, None, dummy, N.Y_F32, None) == N.E_ARG
    assert g(ctypes.byref(L), dummy, 17, dummy, N.X_I8, None, dummy, N.Y_F32, None) == N.E_ARG
    assert g(ctypes.byref(L), dummy, 4, dummy, 7, None, dummy, N.Y_F32, None) == N.E_ARG
    assert g(ctypes.byref(L), dummy, 16, dummy, N.X_BF16, None, dummy, N.Y_I32_RAW, None) == N.E_ARG
    assert g(ctypes.byref(L), None, 2, dummy, N.X_I8, None, dummy, N.Y_F32, None) == N.E_ARG
    L4 = api.bitcos_plan(w, 128, 4)   # four rows per sign offset: m batch-1 launches, same checks first
    assert g(ctypes.byref(L4), dummy, 3, dummy, 7, None, dummy, N.Y_F32, None) == N.E_ARG
    assert g(ctypes.byref(L), dummy, 1, dummy, 7, None, dummy, N.Y_F32, None) == N.E_ARG
    assert g(ctypes.byref(L), dummy, 1, dummy, N.X_BF16, None, dummy, N.Y_I32_RAW, None) == N.E_ARG
    Lt = api.trit5_plan(w, 128)
    assert N.lib().trit5_gemv(ctypes.byref(L), dummy, 1, dummy, N.X_I8, None, dummy, N.Y_F32, None) == N.E_ARG
    assert N.lib().bit2_gemv(ctypes.byref(Lt), dummy, 1, dummy, N.X_I8, None, dummy, N.Y_F32, None) == N.E_ARG
    assert N.lib().trit5_gemv(ctypes.byref(Lt), dummy, 17, dummy, N.X_I8, None, dummy, N.Y_F32, None) == N.E_ARG
    assert N.lib().trit5_gemv(ctypes.byref(Lt), dummy, 5, dummy, 9, None, dummy, N.Y_F32, None) == N.E_ARG


def test_add_partials_argument_checks():
    """bitcos_add_partials rejects null buffers, no parts and empty outputs
    before anything is enqueued (no GPU needed)."""
    f = N.lib().bitcos_add_partials
    dummy = ctypes.c_void_p(16)
    assert f(None, dummy, 1, 4, None) == N.E_ARG
    assert f(dummy, None, 1, 4, None) == N.E_ARG
    assert f(dummy, dummy, 0, 4, None) == N.E_ARG
    assert f(dummy, dummy, 1, 0, None) == N.E_ARG


def test_describe_small_batch():
    w = np.zeros((100, 2560), np.int8)
    L = api.bitcos_plan(w, 128, 0)
    info = api.describe(L, 16, N.X_BF16)
    assert (info.seg_lanes, info.rows_per_step, info.per_lane) == (4, 32, 1)
    assert info.waves == 4                      # ceil(100 / 32) units of 32 rows
    with pytest.raises(N.BitcosError) as e:
        api.describe(L, 17, N.X_I8)
    assert e.value.status == N.E_ARG


def test_describe_tiles():
    # fewest idle lanes first, then the widest tile up to 8 words per lane;
    # int8 rows over 16384 take up to 16
    for k, per_lane, seg in [(2560, 5, 16), (8192, 8, 32), (6912, 7, 32), (1024, 8, 4), (4096, 8, 16),
                             (12288, 6, 64), (25600, 13, 64)]:
        w = np.zeros((8, k), np.int8)
        L = api.bitcos_plan(w, 128, 0)
        info = api.describe(L, 1, N.X_I8)
        assert (info.per_lane, info.seg_lanes) == (per_lane, seg), k
        assert info.rows_per_step * info.seg_lanes == 64
        assert info.lanes_used * info.per_lane >= k // 32
    # bf16: the widest equally full tile with at most 5 words per lane, if any
    for k, per_lane, seg in [(2560, 5, 16), (4096, 4, 32), (8192, 4, 64), (6912, 7, 32), (12288, 6, 64),
                             (1024, 4, 8)]:
        L = api.bitcos_plan(np.zeros((8, k), np.int8), 128, 0)
        info = api.describe(L, 1, N.X_BF16)
        assert (info.per_lane, info.seg_lanes) == (per_lane, seg), k


def test_describe_trit5_tiles():
    # five-trit: at most 4 blocks per lane with int8 activations, 2 with bf16;
    # rows of 20 or 40 blocks take the 20-lane segment (3 rows, 60 lanes)
    for k, kind, per_lane, seg, rows in [(2560, N.X_BF16, 1, 20, 3), (5120, N.X_BF16, 2, 20, 3),
                                         (4096, N.X_BF16, 1, 32, 2), (12288, N.X_BF16, 2, 64, 1),
                                         (6912, N.X_BF16, 1, 64, 1), (1280, N.X_BF16, 1, 16, 4),
                                         (2560, N.X_I8, 1, 20, 3), (5120, N.X_I8, 2, 20, 3),
                                         (4096, N.X_I8, 1, 32, 2), (12288, N.X_I8, 3, 32, 2),
                                         (6912, N.X_I8, 1, 64, 1), (16384, N.X_I8, 2, 64, 1)]:
        L = api.trit5_plan(np.zeros((8, k), np.int8), 128)
        info = api.describe(L, 1, kind)
        assert (info.per_lane, info.seg_lanes, info.rows_per_step) == (per_lane, seg, rows), (k, kind)
        assert info.lanes_used == -(-(k // 128) // per_lane) <= seg
        assert info.waves == -(-8 // rows)


def test_describe_bit2_tiles():
    # 2-bit: int8 up to 16 words per lane where a tile fits, else up to 32;
    # bf16 up to 16
    for k, kind, per_lane, seg in [(6912, N.X_I8, 7, 64), (6912, N.X_BF16, 7, 64), (16384, N.X_I8, 16, 64),
                                   (25600, N.X_I8, 25, 64), (5120, N.X_I8, 5, 64), (12288, N.X_BF16, 12, 64)]:
        L = api.bit2_plan(np.zeros((8, k), np.int8), 128)
        info = api.describe(L, 1, kind)
        assert (info.per_lane, info.seg_lanes) == (per_lane, seg), (k, kind)
    L = api.bit2_plan(np.zeros((8, 32768 + 128), np.int8), 128)
    with pytest.raises(N.BitcosError):
        api.describe(L, 1, N.X_I8)


def test_describe_kernel_choice():
    """Which kernel a table of batch-1 GEMVs on a layout runs; a call too, but for rows longer
    than a tile (test_gpu_launches.py has what is launched)."""
    def kind(group, unit_rows, k=2560, fmt=N.FMT_BITCOS, m=1, x=N.X_BF16):
        w = np.zeros((40, k), np.int8)
        if fmt == N.FMT_BITCOS:
            L = api.bitcos_plan(w, group, unit_rows)
        elif fmt == N.FMT_TRIT5:
            L = api.trit5_plan(w, group)
        else:
            L = api.bit2_plan(w, group)
        return api.describe(L, m, x).kernel
    # one scale per tensor, one offset per row: matrix cores (either activation type)
    assert kind(0, 1) == N.KERNEL_MATRIX
    assert kind(0, 1, x=N.X_I8) == N.KERNEL_MATRIX
    # group scales: the streaming kernel
    assert kind(128, 1) == N.KERNEL_STREAMING
    # several rows per offset at 16 lanes per row (K = 2560): the prefix needs per-row offsets
    assert kind(0, 2) == N.KERNEL_STREAMING
    # ... but not at 32 or more lanes per row (K = 6912: 32 lanes, 2 rows per step)
    assert kind(0, 2, k=6912) == N.KERNEL_MATRIX
    # a unit that does not divide the wave step: the general kernel
    assert kind(0, 3) == N.KERNEL_GENERAL
    assert kind(128, 3) == N.KERNEL_GENERAL
    # rows longer than every batch-1 tile (bf16 K > 16384, int8 K > 32768): the small-batch kernel at m = 1
    assert kind(0, 1, k=16384) == N.KERNEL_MATRIX
    assert kind(128, 1, k=16512) == N.KERNEL_SMALL_BATCH
    assert kind(0, 1, k=25600) == N.KERNEL_SMALL_BATCH
    assert kind(0, 1, k=25600, x=N.X_I8) == N.KERNEL_MATRIX
    assert kind(128, 1, k=32896, x=N.X_I8) == N.KERNEL_SMALL_BATCH
    with pytest.raises(N.BitcosError):
        kind(0, 2, k=25600)  # several rows per offset: no kernel takes such rows
    # small batch and the baselines
    assert kind(0, 1, m=4) == N.KERNEL_SMALL_BATCH
    assert kind(0, 0, fmt=N.FMT_TRIT5) == N.KERNEL_FIXED
    assert kind(128, 0, fmt=N.FMT_BIT2) == N.KERNEL_FIXED
