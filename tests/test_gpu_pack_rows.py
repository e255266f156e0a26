"""Device packer where rows meet inside a sign dword and passes inside a row:
blobs byte for byte against the host packer, for rows of no, one or all
non-zeros, rows shorter than a dword of signs, and rows of several passes of
2048 weights; and what the one-call packer leaves alone when it refuses."""

import numpy as np
import pytest

import workloads as wl
from parity_checks import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
api = pytest.importorskip("paper_2609_16338_amd.api")
from paper_2609_16338_amd import _native as N  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N.lib()


def _weights(n, k, kind):
    rng = wl.rng_for(701, n, k)
    if kind == "dense":
        return rng.choice(np.array([-1, 1], dtype=np.int8), size=(n, k))
    w = wl.ternary(n, k, 0.45, rng)
    if kind == "sparse":  # zero to three non-zeros a row: dozens of rows in one dword
        w[:] = 0
        for r in range(n):
            w[r, rng.choice(k, size=r % 4, replace=False)] = rng.choice([-1, 1], size=r % 4)
    elif kind == "mixed":  # empty, single, full and ordinary rows next to each other
        w[0::4] = 0
        w[1::4] = 0
        w[1::4, k - 1] = -1
        w[2::4] = -1
    return w


@pytest.mark.parametrize("kind", ["dense", "sparse", "mixed", "plain"])
@pytest.mark.parametrize("n,k,group,unit", [(1, 32, 0, 1), (5, 96, 0, 2), (70, 2048, 128, 1), (33, 2080, 0, 3),
                                            (9, 4128, 0, 1), (130, 6144, 128, 1), (4097, 128, 128, 7)])
def test_rows_and_passes(kind, n, k, group, unit):
    say("pack", kind, n, k, group, unit)
    w = _weights(n, k, kind)
    sc = wl.fp16_uniform((n * (k // 128) if group else 1,), 0.005, 0.05, wl.rng_for(702, n, k))
    L_ref, ref = api.plan_and_pack(N.FMT_BITCOS, w, sc, group, unit)
    wd, sd = torch.from_numpy(w).cuda(), torch.from_numpy(sc.view(np.int16)).cuda()
    L, blob = api.bitcos_pack_device(wd, sd, group, unit)
    assert bytes(L) == bytes(L_ref) and np.array_equal(blob.cpu().numpy(), ref)
    dst = torch.full((L_ref.total_bytes + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    L2 = api.bitcos_pack_device_noalloc(wd, sd, dst, group, unit)
    got = dst.cpu().numpy()
    assert bytes(L2) == bytes(L_ref) and np.array_equal(got[:L2.total_bytes], ref) and np.all(got[L2.total_bytes:] == 0x5A)


@pytest.mark.parametrize("value", [2, -2, -128, 127, -127])
def test_one_call_packer_refuses_without_writing(value):
    n, k = 21, 2176
    w = _weights(n, k, "plain")
    w[n - 1, k - 1] = value
    sc = wl.fp16_uniform((n * (k // 128),), 0.005, 0.05, wl.rng_for(703))
    dst = torch.full((65536,), 0x33, dtype=torch.uint8, device="cuda")
    with pytest.raises(N.BitcosError) as e:
        api.bitcos_pack_device_noalloc(torch.from_numpy(w).cuda(), torch.from_numpy(sc.view(np.int16)).cuda(), dst, 128)
    assert e.value.status == N.E_VALUE and np.all(dst.cpu().numpy() == 0x33)
    w[n - 1, k - 1] = 0
    L, ref = api.plan_and_pack(N.FMT_BITCOS, w, sc, 128)
    short = torch.full((L.total_bytes - 1,), 0x33, dtype=torch.uint8, device="cuda")
    with pytest.raises(N.BitcosError) as e:
        api.bitcos_pack_device_noalloc(torch.from_numpy(w).cuda(), torch.from_numpy(sc.view(np.int16)).cuda(), short, 128)
    assert e.value.status == N.E_SPACE and e.value.layout.total_bytes == L.total_bytes
    assert np.all(short.cpu().numpy() == 0x33)
