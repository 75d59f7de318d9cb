"""GPU parity at the sizes where a kernel changes its path: edges of tiles,
remainders, the smallest and largest of a rule's range, against the oracle.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sf():
    import paper_2407_06107_amd as sf
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sf.lib()
    return sf


def _case(*args):
    print("CASE", *args, flush=True)


def _pyramid(w, h, seed):
    """Independent random RGBA8 levels down to 1 x 1."""
    rng = np.random.default_rng(seed)
    lv, l = [], 0
    while True:
        lv.append(rng.integers(0, 256, (max(1, h >> l), max(1, w >> l), 4), dtype=np.uint8))
        if max(w, h) >> l == 1:
            return lv
        l += 1


# 128 x 128 is one workgroup of 256 blocks, 136 x 128 starts a second; the
# odd sizes have edge blocks, and small levels share a workgroup
@pytest.mark.parametrize("w, h", [(1, 1), (7, 3), (8, 8), (9, 17), (128, 128), (136, 128), (250, 1031), (2051, 64)])
def test_dct_codes_at_block_and_workgroup_edges(sf, orc, w, h):
    """Codes and AC ranges equal the oracle's bit for bit, also where the rows
    of a level are only 4-byte aligned."""
    _case("dct_codes", w, h)
    lv = _pyramid(w, h, 100 * w + h)
    lv[0][...] = lv[0][:1, :1] if min(w, h) == 3 else lv[0]   # a constant level: all ranges 0 or tiny
    ot = orc.Tex2D.dct(lv)
    gt = sf.Texture2D.dct(sf.Texture2D(lv))
    torch.cuda.synchronize()
    buf = gt.buffer.cpu().numpy()
    for l, x in enumerate(lv):
        n = 16 * (-(-x.shape[1] // 8)) * (-(-x.shape[0] // 8))
        assert np.array_equal(buf[gt.offsets[l]:gt.offsets[l] + n], ot.buf[ot.off[l]:ot.off[l] + n]), l
    assert np.array_equal(gt.ranges.cpu().numpy(), ot.dct_range)
