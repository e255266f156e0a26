"""2-bit int8 launches on both sides of where waves share their activations (3 / 4
words a lane single, 5 / 6 in a table): int32 row sums, exact, for single calls and
for tables whose neighbours have other activations, with fewer and more units than
waves and a last wave without any."""

import numpy as np
import pytest

import oracle as O
import workloads as wl
from parity_checks import inputs, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
api = pytest.importorskip("paper_2609_16338_amd.api")
from paper_2609_16338_amd import _native as N  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N.lib()


# (K, words of 16 a lane): 1 to 7 words, rows of 8 to 64 lanes, ragged ones among them.
TILES = [(128, 1), (1024, 1), (2048, 2), (2944, 3), (384, 3), (3968, 4), (4096, 4), (4736, 5), (640, 5), (5760, 6), (896, 7)]


@pytest.mark.parametrize("n", [1, 70, 2501])
@pytest.mark.parametrize("k,words", TILES)
def test_single_and_table(k, words, n):
    say("bit2 int8", n, k)
    w, sc = inputs(n, k, 0.42, 128, 511)
    L, blob = api.plan_and_pack(N.FMT_BIT2, w, sc, 128)
    assert api.describe(L, 1, N.X_I8).per_lane == words
    bd = torch.from_numpy(blob).cuda()
    xs = [wl.act_int8(1, k, wl.rng_for(512, i)) for i in range(3)]
    xd = [torch.from_numpy(x).cuda().reshape(-1) for x in xs]
    ref = [np.asarray(O.dense_gemv_raw(w, x)).reshape(n) for x in xs]
    y = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    api.gemv(L, bd, xd[0], y, y_mode=N.Y_I32_RAW)
    assert np.array_equal(y.cpu().numpy(), ref[0])
    pick = [0, 0, 1, 2, 2, 0, 1]
    ys = torch.full((len(pick), n), -7, dtype=torch.int32, device="cuda")
    api.Batch([L] * len(pick), [bd] * len(pick), [xd[p] for p in pick], [ys[i] for i in range(len(pick))],
              y_mode=N.Y_I32_RAW).run()
    got = ys.cpu().numpy()
    for i, p in enumerate(pick):
        assert np.array_equal(got[i], ref[p]), i
