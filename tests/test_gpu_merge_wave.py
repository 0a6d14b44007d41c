"""Merge tails with 32 keys per lane (tiles of 2^11 to 2^14 keys) against the oracle.

Bar: bit-exact. Arrays of a few tiles, whole ones and with an end inside a wave's 2048
keys, in either direction of a tile; arrays that are not 16-byte aligned; all 0/1
thresholds; the nontemporal variant on an array beyond the caches.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")


@pytest.mark.parametrize("log_t", [11, 12, 13, 14])
def test_tiles(log_t):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    meld.set_option(0, meld.OPT_SORT_LOG_TILE, log_t)
    try:
        tile = 1 << log_t
        for n in (2 * tile, 8 * tile, tile + 1, 2 * tile - 1, 3 * tile, 3 * tile + 2047,
                  5 * tile + 2049, 7 * tile + 77):
            keys = workloads.keys_u32(n, n)
            ones = (np.arange(n) * 40503 % 65536 < n % 60000).astype(np.uint32)
            for k in (keys, keys % np.uint32(9), ones):
                for offset in (0, 1):
                    buf = torch.zeros(n + offset, dtype=torch.int32, device="cuda:0")
                    buf[offset:] = torch.from_numpy(k.view(np.int32)).cuda()
                    for v in ("melded", "divergent"):
                        b = buf.clone()
                        meld.sort(b[offset:], variant=v)
                        got = b.cpu().numpy().view(np.uint32)
                        assert np.array_equal(got[offset:], oracle.sort_u32(k)), (n, v)
    finally:
        meld.set_option(0, meld.OPT_SORT_LOG_TILE, 0)


def test_beyond_the_caches():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = (1 << 26) + 12_345  # padded to 2^27 keys, 512 MiB
    g = torch.Generator(device="cuda:0")
    g.manual_seed(3)
    k = torch.randint(-(1 << 31), 1 << 31, (n,), dtype=torch.int32, device="cuda:0", generator=g)
    want = torch.sort(k.to(torch.int64) & 0xFFFFFFFF).values
    meld.sort(k, variant="melded")
    assert torch.equal(k.to(torch.int64) & 0xFFFFFFFF, want)
