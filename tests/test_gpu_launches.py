"""What calls launch: the kernel and its grid, read back from a recorded graph."""

import pytest

import workloads as wl
from parity_checks import say

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


def _packed(n, k, group=128, unit=0, fmt=N.FMT_BITCOS):
    w = wl.ternary(n, k, 0.45, wl.rng_for(901, n, k))
    sc = wl.fp16_uniform((n * (k // 128) if group else 1,), 0.005, 0.05, wl.rng_for(902, n, k))
    L, blob = api.plan_and_pack(fmt, w, sc, group, unit)
    return L, torch.from_numpy(blob).cuda()


def _gemv_call(L, blob, m, dtype):
    x = torch.ones((m, L.k), dtype=dtype, device="cuda")
    y = torch.empty((m, L.n), dtype=torch.float32, device="cuda")
    return lambda: api.gemv(L, blob, x, y)


@pytest.mark.parametrize("dtype", ["bfloat16", "int8"])
@pytest.mark.parametrize("kernel,n,k,unit,m,steps", [
    ("bitcos_gemv_kernel", 300 * 64, 256, 64, 1, 300),   # units of 64 rows: the general kernel
    ("bitcos_gemv_kernel", 9 * 100, 512, 100, 1, 9),
    ("bitcos_mfma_kernel", 4096, 512, 0, 4, 128),        # whole units of 32 rows, one step each
    ("bitcos_mfma_kernel", 40, 128, 0, 16, 2),
])
def test_every_workgroup_has_units(kernel, n, k, unit, m, steps, dtype):
    """Kernels whose waves take consecutive runs of ceil(units / waves) units: no workgroup
    of the launch builds its tables for nothing."""
    say("launch", kernel, n, k, unit, m, dtype)
    L, blob = _packed(n, k, unit=unit)
    (name, blocks, threads), = captured(_gemv_call(L, blob, m, getattr(torch, dtype)))
    assert kernel in name
    waves = threads // 64
    per_wave = -(-steps // (blocks * waves))
    assert (blocks - 1) * waves * per_wave < steps, f"{blocks} workgroups of {waves} waves for {steps} units"


KERNEL_NAMES = {N.KERNEL_GENERAL: "bitcos_gemv_kernel", N.KERNEL_STREAMING: "bitcos_fast_kernel",
                N.KERNEL_MATRIX: "bitcos_diag_kernel", N.KERNEL_SMALL_BATCH: "bitcos_mfma_kernel"}


@pytest.mark.parametrize("dtype", ["bfloat16", "int8"])
@pytest.mark.parametrize("n,k,group,unit,m", [
    (40, 2560, 0, 1, 1), (40, 2560, 128, 1, 1), (40, 2560, 0, 3, 1), (40, 2560, 128, 2, 1), (40, 2560, 0, 1, 4),
    (40, 16384, 128, 1, 1), (40, 16512, 128, 1, 1), (5, 32768, 0, 1, 1), (5, 32896, 128, 1, 1),
    (5, 65536, 128, 1, 1), (5, 65664, 0, 1, 1), (5, 65664, 128, 1, 16),
])
def test_described_kernel_is_launched(n, k, group, unit, m, dtype):
    """bitcos_describe names what a table launches, and what a call launches but for rows of
    one to two batch-1 tiles, which a call runs on the streaming kernel."""
    say("route", n, k, group, unit, m, dtype)
    L, blob = _packed(n, k, group, unit)
    described = api.describe(L, m, N.X_I8 if dtype == "int8" else N.X_BF16).kernel
    tile = 32768 if dtype == "int8" else 16384
    x = torch.ones((m, k), dtype=getattr(torch, dtype), device="cuda")
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    (table, _, _), = captured(api.Batch([L], [blob], [x], [y]).run)
    assert KERNEL_NAMES[described] in table
    (single, _, _), = captured(lambda: api.gemv(L, blob, x, y))
    call = N.KERNEL_STREAMING if m == 1 and tile < k <= 2 * tile else described
    assert KERNEL_NAMES[call] in single
