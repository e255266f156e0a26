"""GPU parity of how a batched launch starts: tables of more than 64 GEMVs (the
search for a wave's first one compares 64 at a time), workgroups whose waves
start on GEMVs with different activations, and rows whose activations pass
through the LDS in several rounds.  Bars as in parity_checks.py."""

import numpy as np
import pytest

import oracle as O
import workloads as wl
from parity_checks import FMT_NAME, bf16_bound, group_bound, inputs, say, to_dev_x

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
api = pytest.importorskip("paper_2609_16338_amd.api")
from paper_2609_16338_amd import _native as N  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N.lib()


# (count, rows of a GEMV, K, scale group, distinct activations): one matrix
# packed once and multiplied with several activation vectors.
CASES = [(1, 5, 256, 128, 1), (64, 3, 256, 128, 64), (65, 3, 256, 128, 5), (130, 9, 1024, 128, 2),
         (4100, 2, 128, 128, 7), (70, 7, 640, 0, 3), (9, 33, 8192, 128, 2)]


@pytest.mark.parametrize("fmt", [N.FMT_BITCOS, N.FMT_TRIT5, N.FMT_BIT2])
@pytest.mark.parametrize("kind", ["int8", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_batch_starts(fmt, kind, case):
    count, n, k, group, nx = case
    say(FMT_NAME[fmt], kind, case)
    w, sc = inputs(n, k, 0.42, group, 501)
    L, blob = api.plan_and_pack(fmt, w, sc, group)
    bd = torch.from_numpy(blob).cuda()
    xs = [wl.act_int8(1, k, wl.rng_for(502, i)) if kind == "int8" else wl.act_bf16(1, k, wl.rng_for(503, i))
          for i in range(nx)]
    xd = [to_dev_x(x, kind).reshape(-1) for x in xs]
    pick = [(i * 3) % nx if i % 2 else i // 2 % nx for i in range(count)]  # neighbours share or differ
    y = torch.full((count, n), -7.0, dtype=torch.float32, device="cuda")
    b = api.Batch([L] * count, [bd] * count, [xd[p] for p in pick], [y[i] for i in range(count)])
    b.run()
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    for p in sorted(set(pick)):
        rows = got[[i for i in range(count) if pick[i] == p]]
        if kind == "int8":
            ref, bound = O.dense_gemv(w, sc, group, xs[p]), 1e-5 * group_bound(w, sc, group, xs[p])
        else:
            ref, bound = O.dense_gemv(w, sc, group, xs[p], x_is_bf16_bits=True), 1e-3 * bf16_bound(w, sc, group, xs[p])
        assert np.all(np.abs(rows - np.asarray(ref).reshape(1, n)) <= np.asarray(bound).reshape(1, n) + 1e-30)
