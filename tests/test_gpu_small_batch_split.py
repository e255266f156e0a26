"""GPU parity of the small-batch kernel where several waves share a unit of 32
rows (they split its K): every number of parts at its smallest and largest
launch, parts of unequal length or with no step at all, rows past the matrix
end, batch tables of mixed K, and all output modes.  int8 raw sums bit-exact,
the others at the bars of parity_checks.py on sampled rows."""

import numpy as np
import pytest

import oracle as O
import workloads as wl
from parity_checks import bf16_bound, check_bf16, check_grouped, group_bound, inputs, sampled_rows, say, to_dev_x

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
api = pytest.importorskip("paper_2609_16338_amd.api")
from launches import captured  # noqa: E402
from paper_2609_16338_amd import _native as N  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N.lib()


# (n, k, m): 32-row units x parts against 2048 waves, steps of 512 weights.
# 8 parts up to n = 8192 (of 16-row units up to 4096, where k has 8 steps), 4 up
# to 16384, 2 up to 32768, then whole units; no
# more parts than steps (k = 384: one step, 1024: two, 2560: five).
SHAPES = [(1, 128, 2), (33, 384, 3), (45, 1024, 16), (40, 2560, 5), (70, 4096, 4), (8192, 4224, 2), (50, 2560, 8), (8193, 4224, 7),
          (16384, 2176, 2), (16385, 2176, 9), (32768, 1152, 2), (32769, 1152, 3), (64, 25600, 1),
          (37, 33024, 1), (5, 65664, 1), (4096, 4096, 3), (4097, 4096, 2), (2000, 4224, 16), (17, 4096, 6)]


def _run(L, bd, xd, y, xscale=None, y_mode=N.Y_F32):
    """One GEMV on the small-batch kernel: a call, or with one activation row, where calls of
    rows up to twice a batch-1 tile run another kernel, a table of one."""
    call = lambda: api.gemv(L, bd, xd, y, xscale, y_mode)  # noqa: E731
    if y.shape[0] == 1 and L.k <= (65536 if xd.dtype == torch.int8 else 32768):
        call = api.Batch([L], [bd], [xd], [y], None if xscale is None else [xscale], y_mode).run
    if y_mode in (N.Y_F32, N.Y_I32_RAW):  # asking runs it too, and it overwrites y
        (name, _, _), = captured(call)
        assert "bitcos_mfma_kernel" in name
    call()


def _rows(n):
    return np.arange(n) if n <= 128 else sampled_rows(n, 40, n)


def _sub(w, sc, rows, k, group):
    return w[rows], (sc.reshape(-1, k // 128)[rows].reshape(-1) if group == 128 else sc)


@pytest.mark.parametrize("n,k,m", SHAPES)
def test_parts_int8(n, k, m):
    w, sc = inputs(n, k, 0.42, 128, 601)
    rows = _rows(n)
    ws, ss = _sub(w, sc, rows, k, 128)
    L, blob = api.plan_and_pack(N.FMT_BITCOS, w, sc, 128)
    bd = torch.from_numpy(blob).cuda()
    if m == 1 and api.describe(L, 1, N.X_I8).kernel != N.KERNEL_SMALL_BATCH:
        pytest.skip("batch-1 tile")
    say("split int8", n, k, m)
    x = wl.act_int8(m, k, wl.rng_for(602, k, m))
    xd = to_dev_x(x, "int8")
    y = torch.full((m, n), 3, dtype=torch.int32, device="cuda")
    _run(L, bd, xd, y, y_mode=N.Y_I32_RAW)
    ref = O.dense_gemv_raw(ws, x)
    assert np.array_equal(y.cpu().numpy()[:, rows], ref)
    _run(L, bd, xd, y, y_mode=N.Y_I32_RAW_ADD)
    assert np.array_equal(y.cpu().numpy()[:, rows], 2 * ref)
    q, a = O.quantize_activations(wl.act_bf16(m, k, wl.rng_for(603, k, m)))
    f = torch.empty((m, n), dtype=torch.float32, device="cuda")
    _run(L, bd, to_dev_x(q, "int8"), f, torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda())
    check_grouped(f.cpu().numpy()[:, rows], O.dense_gemv(ws, ss, 128, q, a), group_bound(ws, ss, 128, q, a))


@pytest.mark.parametrize("group", [128, 0])
@pytest.mark.parametrize("n,k,m", SHAPES)
def test_parts_bf16(n, k, m, group):
    w, sc = inputs(n, k, 0.42, group, 604)
    rows = _rows(n)
    ws, ss = _sub(w, sc, rows, k, group)
    L, blob = api.plan_and_pack(N.FMT_BITCOS, w, sc, group)
    if m == 1 and api.describe(L, 1, N.X_BF16).kernel != N.KERNEL_SMALL_BATCH:
        pytest.skip("batch-1 tile")
    say("split bf16", n, k, m, group)
    x = wl.act_bf16(m, k, wl.rng_for(605, k, m))
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    bd = torch.from_numpy(blob).cuda()
    _run(L, bd, to_dev_x(x, "bf16"), y)
    first = y.cpu().numpy()
    check_bf16(first[:, rows], O.dense_gemv(ws, ss, group, x, x_is_bf16_bits=True), bf16_bound(ws, ss, group, x))
    _run(L, bd, to_dev_x(x, "bf16"), y)
    assert np.array_equal(first.view(np.uint32), y.cpu().numpy().view(np.uint32))  # a fixed order of the parts


@pytest.mark.parametrize("kind", ["int8", "bf16"])
def test_table_of_mixed_rows(kind):
    """Units of different K share a launch: some have fewer steps than parts."""
    m, shapes = 4, [(70, 512), (33, 4096), (5, 128), (64, 2560), (96, 1152)]
    say("split table", kind)
    Ls, bs, xs, ys, refs = [], [], [], [], []
    for i, (n, k) in enumerate(shapes):
        w, sc = inputs(n, k, 0.42, 128, 606 + i)
        L, blob = api.plan_and_pack(N.FMT_BITCOS, w, sc, 128)
        x = wl.act_int8(m, k, wl.rng_for(607, i)) if kind == "int8" else wl.act_bf16(m, k, wl.rng_for(608, i))
        Ls.append(L)
        bs.append(torch.from_numpy(blob).cuda())
        xs.append(to_dev_x(x, kind))
        ys.append(torch.empty((m, n), dtype=torch.float32, device="cuda"))
        refs.append((w, sc, x))
    api.Batch(Ls, bs, xs, ys).run()
    torch.cuda.synchronize()
    for y, (w, sc, x) in zip(ys, refs):
        if kind == "int8":
            check_grouped(y.cpu().numpy(), O.dense_gemv(w, sc, 128, x), group_bound(w, sc, 128, x))
        else:
            check_bf16(y.cpu().numpy(), O.dense_gemv(w, sc, 128, x, x_is_bf16_bits=True), bf16_bound(w, sc, 128, x))
