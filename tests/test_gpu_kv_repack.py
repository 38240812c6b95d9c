"""spec_kv_repack_mfma against the layout as the header states it: head counts that do not fill the last
block, both head dims, and pools that start at an odd element."""
import numpy as np
import pytest

from paper_2406_14066_amd import spec_verify as sv

pytestmark = pytest.mark.gpu


def _tiled(k, v):
    """Token-major [nb][Hkv][16][d] to K [nb][Hkv][d/8][16][8] and V [nb][Hkv][d/32][4][16][2][4] (flat)."""
    nb, H, S, d = k.shape
    kt = k.reshape(nb, H, S, d // 8, 8).transpose(0, 1, 3, 2, 4)
    # [.., token group, token, dim pair, half, dim] -> [.., pair, group, dim, half, token]
    vt = v.reshape(nb, H, 4, 4, d // 32, 2, 16).transpose(0, 1, 4, 2, 6, 5, 3)
    return kt.reshape(-1), vt.reshape(-1)


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "odd_element"])
@pytest.mark.parametrize("blocks,Hkv,d", [(1, 1, 64), (3, 1, 128), (5, 3, 64), (2, 8, 128), (33, 5, 128)])
def test_repack(blocks, Hkv, d, offset):
    import torch
    print("case repack", blocks, Hkv, d, offset, flush=True)
    rng = np.random.default_rng(blocks * 1000 + Hkv)
    n = blocks * Hkv * 16 * d
    src = rng.integers(-32768, 32767, size=(2, n), dtype=np.int16)   # every bit pattern counts
    want = _tiled(*(x.reshape(blocks, Hkv, 16, d) for x in src))
    dev_src = [torch.zeros(n + 2, dtype=torch.int16, device="cuda") for _ in range(2)]
    dev_dst = [torch.full((n + 2,), 77, dtype=torch.int16, device="cuda") for _ in range(2)]
    for t, x in zip(dev_src, src):
        t[offset: offset + n] = torch.from_numpy(x).cuda()
    shape = (blocks, Hkv, 16, d)
    sv.spec_kv_repack_mfma(*(t[offset: offset + n].view(shape) for t in dev_src + dev_dst))
    torch.cuda.synchronize()
    for t, x in zip(dev_dst, want):
        got = t.cpu().numpy()
        np.testing.assert_array_equal(got[offset: offset + n], x)
        assert (got[:offset] == 77).all() and (got[offset + n:] == 77).all()
