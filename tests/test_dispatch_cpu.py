"""Which kernel the library's own choice runs a call on, asked on the host: the lines between the kernels as they were
measured, and that the sizes which other tests name reach the kernels that those tests are about."""
import pytest

from paper_2604_04451_amd import binding as B

CUS = 256  # compute units of the GPU


def _attention(Lq, Lk, H, dh, factor, pad=128):
    return B.load().chorus_attention_variant(Lq, Lk, -(-Lk // pad) * pad, H, dh, int(factor), CUS)


@pytest.mark.parametrize("factor", [False, True])
def test_attention_long_and_short_keys(factor):
    assert _attention(13104, 512, 12, 128, factor) == _attention(300, 2049, 3, 64, factor) == 5
    assert _attention(13104, 570, 12, 128, factor, pad=64) == 3      # padded to 64 only
    assert _attention(480, 64, 12, 128, factor) == _attention(32760, 16, 12, 128, factor) == 3
    for Lq, Lk, H in ((480, 480, 12), (1200, 77, 12), (128, 128, 4), (300, 300, 12)):  # half tiles all at once
        assert _attention(Lq, Lk, H, 128, factor) == 5
    for Lk in (129, 180, 300):                                       # half of the last 128-key tile would be padding
        assert _attention(13104, Lk, 40, 128, factor) == 3
    assert _attention(13104, 400, 40, 128, factor) == (5 if factor else 3)


def test_attention_full_tiles():
    for Lq, H in ((3271, 12), (13104, 12), (13104, 40)):             # 156, 624, 2080 tiles of 256 rows
        for Lk in (65, 77, 96, 200, 226, 480, 511):
            assert _attention(Lq, Lk, H, 128, True) == 5
            assert _attention(Lq, Lk, 2 * H, 64, True) == 5
        for Lk in (97, 128):                                         # few keys masked, or none
            assert _attention(Lq, Lk, H, 128, True) == 3
        assert _attention(Lq, 300, 2 * H, 64, True) == 5
        for Lk in (65, 77, 128):
            assert _attention(Lq, Lk, H, 128, False) == 3
    assert _attention(3271, 226, 12, 128, False) == 3                # less than a round
    assert _attention(13104, 226, 12, 128, False) == _attention(13104, 480, 40, 128, False) == 5


def test_attention_variant_refuses():
    lib = B.load()
    for bad in ((0, 8, 64, 2, 64), (8, 0, 64, 2, 64), (8, 80, 64, 2, 64), (8, 8, 64, 0, 64)):
        assert lib.chorus_attention_variant(*bad, 0, CUS) == B.E_ARG
    assert lib.chorus_attention_variant(8, 8, 64, 2, 64, 0, 0) == B.E_ARG
    assert lib.chorus_attention_variant(8, 8, 64, 2, 96, 0, CUS) == lib.chorus_attention_variant(8, 8, 72, 2, 64, 0, CUS) == B.E_SHAPE
