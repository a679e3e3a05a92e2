"""The mask kernels at the edges of their pieces: rows that end one site before, on and behind a word of 64, radii beyond a
word, strips that fill the LDS; pixel rows of every length modulo 16 that start anywhere, more frames in a window than are
looked up together, frames without a key frame. Against max pooling and a loop over the windows; results are exact."""
import pytest
import torch
import torch.nn.functional as F

from paper_2604_04451_amd import binding as B

pytestmark = pytest.mark.gpu


def _mask(shape, p, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return (torch.rand(shape, generator=g, device="cuda") < p).to(torch.uint8) * 200  # any non-zero byte is set


def _dilate(m, r):
    r = [min(a, n) for a, n in zip(r, m.shape)]  # further there is nothing to reach
    k = [2 * a + 1 for a in r]
    return F.max_pool3d((m != 0).double()[None, None], k, 1, r)[0, 0].to(torch.uint8)


@pytest.mark.parametrize("T,H,W,re,rs", [
    (1, 1, 1, (0, 0, 0), (2, 2, 2)), (3, 5, 63, (1, 1, 1), (1, 2, 2)), (3, 5, 64, (0, 1, 2), (1, 2, 3)), (2, 7, 65, (1, 0, 1), (6, 1, 4)),
    (9, 4, 130, (2, 1, 65), (5, 2, 70)), (2, 3, 200, (0, 0, 64), (0, 1, 128)), (21, 30, 52, (1, 1, 1), (1, 2, 2)),
    (3, 30, 52, (0, 1, 10 ** 6), (0, 1, 10 ** 6)), (3, 9, 70, (1, 2, 3), (2 ** 31 - 1,) * 3), (1, 1100, 3, (2 ** 31 - 1,) * 3, (2 ** 31 - 1,) * 3),
    (1, 4, 90000, (0, 2 ** 31 - 1, 1), (2 ** 31 - 1, 2 ** 31 - 1, 2)),
    (1, 40, 3000, (0, 2, 1), (0, 3, 2)), (1, 9, 30000, (0, 1, 1), (0, 1, 2)), (1, 4, 90000, (0, 0, 1), (0, 1, 2))])
def test_hierarchy(T, H, W, re, rs):
    print(f"[case] hierarchy {T}x{H}x{W} {re} {rs}", flush=True)
    m = _mask((T, H, W), 0.004 if W > 8 else 0.5, W)
    m[0, 0, W - 1] = 1
    edit, see = B.chorus_mask_hierarchy(m, re, rs)
    assert torch.equal(edit, _dilate(m, re)) and torch.equal(see, _dilate(m, rs))


@pytest.mark.parametrize("Hp,Wp,kt,kh,kw", [(33, 854, 4, 16, 16), (20, 207, 11, 16, 16), (64, 1000, 17, 16, 12), (7, 5, 3, 3, 2),
                                            (40, 17, 9, 18, 16), (17, 16, 1, 1, 1), (65, 33, 8, 64, 32), (9, 37, 2 ** 31 - 1, 4, 8),
                                            (9, 37, 4, 2 ** 31 - 1, 2 ** 31 - 1), (9, 36, 20, 10, 40)])
def test_project(Hp, Wp, kt, kh, kw):
    Tp, Kf = 1 + 2 * (kt if kt < 100 else 4) + 1, 6
    print(f"[case] project {Hp}x{Wp} window {kt} {kh} {kw}", flush=True)
    store = _mask((Kf * Hp * Wp + 5,), 3.0 / (min(kh, Hp) * min(kw, Wp)), Wp)
    for off in (0, 5):  # from an aligned address and from another
        keys = store[off:off + Kf * Hp * Wp].view(Kf, Hp, Wp)
        fk = torch.tensor([(i * 5) % (Kf + 2) - 1 for i in range(Tp)], dtype=torch.int32, device="cuda")  # -1 and Kf: none
        got = B.chorus_mask_project(keys, fk, Tp, (kt, kh, kw), 1)
        wins = [[0]] + [list(range(t, min(t + kt, Tp))) for t in range(1, Tp, kt)]
        for o, frames in enumerate(wins):
            ks = [int(fk[t]) for t in frames if 0 <= int(fk[t]) < Kf]
            any_ = (keys[ks] != 0).any(0) if ks else torch.zeros(Hp, Wp, dtype=torch.bool, device="cuda")
            win = (min(kh, Hp), min(kw, Wp))
            want = F.max_pool2d(any_.double()[None, None], win, win, ceil_mode=True)[0, 0].to(torch.uint8)
            assert torch.equal(got[o], want[:got.shape[1], :got.shape[2]]), (off, o)
