"""Activations that are aligned to their element only: a contiguous view at an odd
element offset gives the same bits as an aligned copy, on every kernel."""

import numpy as np
import pytest

import workloads as wl
from parity_checks import FMT_NAME, inputs, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
api = pytest.importorskip("paper_2609_16338_amd.api")
from paper_2609_16338_amd import _native as N  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N.lib()


# (format, n, K, scale group, rows per sign offset, activation rows): ragged and full tiles of
# each kernel; rows of two waves; whole and split units.
CASES = [(N.FMT_BITCOS, 37, 2560, 128, 1, 1), (N.FMT_BITCOS, 37, 6912, 0, 1, 1), (N.FMT_BITCOS, 37, 2560, 128, 7, 1),
         (N.FMT_BITCOS, 9, 96, 0, 1, 1), (N.FMT_BITCOS, 5, 33024, 128, 1, 1), (N.FMT_BITCOS, 37, 4096, 128, 1, 4),
         (N.FMT_BITCOS, 37, 384, 128, 1, 16), (N.FMT_TRIT5, 37, 2560, 128, 0, 1), (N.FMT_TRIT5, 37, 6912, 128, 0, 1),
         (N.FMT_BIT2, 37, 640, 128, 0, 1), (N.FMT_BIT2, 37, 2560, 128, 0, 1), (N.FMT_BIT2, 37, 6912, 128, 0, 1)]


@pytest.mark.parametrize("kind", ["int8", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_odd_element_offsets(case, kind):
    fmt, n, k, group, unit, m = case
    say("alignment", FMT_NAME[fmt], kind, case)
    w, sc = inputs(n, k, 0.42, group, 521)
    L, blob = api.plan_and_pack(fmt, w, sc, group, unit)
    bd = torch.from_numpy(blob).cuda()
    if kind == "int8":
        x = torch.from_numpy(wl.act_int8(m, k, wl.rng_for(522, k))).cuda()
    else:
        x = torch.from_numpy(wl.act_bf16(m, k, wl.rng_for(523, k)).view(np.int16)).cuda().view(torch.bfloat16)
    want = torch.empty((m, n), dtype=torch.float32, device="cuda")
    api.gemv(L, bd, x.contiguous(), want)
    room = torch.zeros(m * k + 16, dtype=x.dtype, device="cuda")
    table = fmt != N.FMT_BITCOS or (unit == 1 and k % 128 == 0) or m == 1
    want_t = torch.empty_like(want)
    if table:
        api.Batch([L], [bd], [x.contiguous()], [want_t]).run()
    for offset in (1, 2, 3, 7, 8):
        xo = room[offset:offset + m * k].view(m, k)
        xo.copy_(x)
        y = torch.full_like(want, -7.0)
        api.gemv(L, bd, xo, y)
        assert torch.equal(y.view(torch.int32), want.view(torch.int32)), offset
        if table:
            y.fill_(-7.0)
            api.Batch([L], [bd], [xo], [y]).run()
            assert torch.equal(y.view(torch.int32), want_t.view(torch.int32)), offset
