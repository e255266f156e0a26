"""GPU parity of batch-1 GEMVs whose rows two waves share (bf16 rows above
16384 weights, int8 rows above 32768, one call each): the narrowest and widest
row of every tile, a second half of almost nothing, rows of all, one or no
non-zeros (their signs are fetched from either end), every scale and output
mode, and launches of fewer and more rows than waves.  Bars as in
parity_checks.py; int8 raw sums bit-exact."""

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


def _mixed(n, k, seed):
    w, sc = inputs(n, k, 0.42, 128, seed)
    if n >= 4:
        w[1] = 0
        w[2] = -1
        w[3] = 0
        w[3, k - 1] = 1
    return w, sc


@pytest.mark.parametrize("n,k", [(1, 16512), (6, 20480), (7, 20608), (70, 25600), (5, 28672), (9, 32768), (1100, 16640)])
def test_long_rows_bf16(n, k):
    say("long bf16", n, k)
    w, sc = _mixed(n, k, 801)
    rows = np.arange(n) if n <= 128 else sampled_rows(n, 40, n)
    x = wl.act_bf16(1, k, wl.rng_for(802, k))
    for group in (128, 0):
        s = sc if group else sc[:1]
        L, blob = api.plan_and_pack(N.FMT_BITCOS, w, s, group)
        bd, xd = torch.from_numpy(blob).cuda(), to_dev_x(x, "bf16")
        y = torch.full((1, n), 5.0, dtype=torch.float32, device="cuda")
        api.gemv(L, bd, xd, y)
        ss = s.reshape(n, -1)[rows].reshape(-1) if group else s
        ref, bound = O.dense_gemv(w[rows], ss, group, x, x_is_bf16_bits=True), bf16_bound(w[rows], ss, group, x)
        first = y.cpu().numpy()
        check_bf16(first[:, rows], ref, bound)
        api.gemv(L, bd, xd, y, y_mode=N.Y_F32_ADD)
        check_bf16(y.cpu().numpy()[:, rows], 2 * ref, 2 * bound)
        again = torch.empty_like(y)
        api.gemv(L, bd, xd, again)
        assert np.array_equal(first.view(np.uint32), again.cpu().numpy().view(np.uint32))
        (name, _, _), = captured(lambda: api.gemv(L, bd, xd, again))
        assert "bitcos_fast_kernel" in name
        a = wl.rng_for(806, k).uniform(0.5, 2.0, size=(1, k // 128)).astype(np.float32)
        api.gemv(L, bd, xd, y, torch.from_numpy(a).cuda())
        refa = O.dense_gemv(w[rows], ss, group, x, a, x_is_bf16_bits=True)
        check_bf16(y.cpu().numpy()[:, rows], refa, bound * float(a.max()))


@pytest.mark.parametrize("n,k", [(1, 32896), (6, 36864), (9, 40960), (70, 33024), (5, 65536), (1100, 32896)])
def test_long_rows_int8(n, k):
    say("long int8", n, k)
    w, sc = _mixed(n, k, 803)
    rows = np.arange(n) if n <= 128 else sampled_rows(n, 40, n)
    x = wl.act_int8(1, k, wl.rng_for(804, k))
    xd = to_dev_x(x, "int8")
    L, blob = api.plan_and_pack(N.FMT_BITCOS, w, sc, 128)
    bd = torch.from_numpy(blob).cuda()
    raw = O.dense_gemv_raw(w[rows], x)
    y = torch.empty((1, n), dtype=torch.int32, device="cuda")
    api.gemv(L, bd, xd, y, y_mode=N.Y_I32_RAW)
    assert np.array_equal(y.cpu().numpy()[:, rows], raw)
    api.gemv(L, bd, xd, y, y_mode=N.Y_I32_RAW_ADD)
    assert np.array_equal(y.cpu().numpy()[:, rows], 2 * raw)
    f = torch.empty((1, n), dtype=torch.float32, device="cuda")
    ss = sc.reshape(n, -1)[rows].reshape(-1)
    api.gemv(L, bd, xd, f)
    check_grouped(f.cpu().numpy()[:, rows], O.dense_gemv(w[rows], ss, 128, x), group_bound(w[rows], ss, 128, x))
    q, a = O.quantize_activations(wl.act_bf16(1, k, wl.rng_for(805, k)))
    ad = torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    api.gemv(L, bd, to_dev_x(q, "int8"), f, ad)
    check_grouped(f.cpu().numpy()[:, rows], O.dense_gemv(w[rows], ss, 128, q, a), group_bound(w[rows], ss, 128, q, a))
    Lt, bt = api.plan_and_pack(N.FMT_BITCOS, w, sc[:1], 0)
    (name, _, _), = captured(lambda: api.gemv(L, bd, xd, y, y_mode=N.Y_I32_RAW))
    assert "bitcos_fast_kernel" in name
    api.gemv(Lt, torch.from_numpy(bt).cuda(), xd, f)  # one scale per tensor: bit-exact
    assert np.array_equal(f.cpu().numpy()[:, rows], np.asarray(O.dense_gemv(w[rows], sc[:1], 0, x), np.float32))
