"""Which kernel the library's own choice runs a call on, asked on the host: the lines between the kernels as they were
measured, and that the sizes which other tests name reach the kernels that those tests are about."""
import pytest

from paper_2604_04451_amd import binding as B
from test_gpu_block_text import CASES as TEXT_CASES
from test_gpu_gemm_slices import DEFAULT_TILES, FFN_SLICES, ffn2_scratch

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


def test_attention_few_keys():
    for Lq, Lk, H in ((128, 128, 4), (1, 1, 1), (300, 77, 8), (2048, 16, 16), (8192, 65, 4)):  # up to 128 tiles of 256 queries
        for factor in (False, True):
            assert _attention(Lq, Lk, H, 64, factor) == _attention(Lq, Lk, H, 64, factor, pad=64) == 7
            assert _attention(Lq, Lk, H, 128, factor) != 7
    assert _attention(128, 129, 4, 64, False) == _attention(2049, 128, 16, 64, True) == 5 and _attention(2049, 16, 16, 64, False) == 3


def _slices(L, H, dh=128, first=None, rest=None):
    D = H * dh  # a block's scratch: its normalised rows and its projection
    return B.chorus_attention_slices_plan(L, H, dh, CUS, 2 * L * D if first is None else first, 6 * L * D if rest is None else rest)


def test_attention_slices():
    assert _slices(13104, 12) == (512, 2) and _slices(75600, 40) == (11776, 4) and _slices(8100, 12) == (256, 2)
    assert _slices(32760, 12) == _slices(16380, 12) == (0, 0)          # whole rounds
    assert _slices(3271, 12) == _slices(3000, 40) == (0, 0)            # a last round that is more than half full
    assert _slices(1200, 12) == _slices(2560, 12) == _slices(1792, 40) == (0, 0)  # too few keys
    assert _slices(5120, 3, 128, 1 << 30) == (0, 4) and _slices(5121, 4, 128, 1 << 30) == (0, 3)
    assert _slices(5120, 3) == (0, 2) and _slices(3584, 4, 64) == (0, 0)  # as many slices as there is scratch for
    assert _slices(8840, 12) == (256, 3) and _slices(9400, 12) == (0, 0)  # 164 and 188 tiles
    need = 2 * 112 * 4 + 112 * 4
    need = -(-need // 256) * 256 + 112 * 139264
    assert _slices(13104, 12, 128, need, 0) == (512, 2) and _slices(13104, 12, 128, need - 1, 0) == (0, 0)
    assert _slices(13104, 12, 128, need - 1, 139264) == (512, 2) and _slices(13104, 12, 128, 0, 1 << 30) == (0, 0)


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


def test_gemm_cases_reach_their_tiles():
    for (M, N, K), want in DEFAULT_TILES.items():
        for epi, kernel in zip((B.EPI_BF16, B.EPI_RESID), want):
            assert B.chorus_gemm_bf16_plan(M, N, K, epi) == (0, kernel, 1), (M, N, K, epi)
    for epi in range(4):  # rows cut behind the last whole round
        assert B.chorus_gemm_bf16_plan(4099, 4608, 1536, epi) == (3584, 5, 1)
    assert B.chorus_gemm_bf16_plan(4452, 4096, 512, B.EPI_BF16)[0] == 4096
    assert B.chorus_gemm_bf16_plan(13104, 1536, 8960, B.EPI_RESID) == (10752, 5, 1)
    assert B.chorus_gemm_bf16_plan(32760, 8960, 1536, B.EPI_GELU_BF16)[1] == 3


def test_rows_are_not_cut_with_few_steps():
    for M, N in ((3700, 4608), (4500, 4608), (8000, 4608), (13104, 1536), (2300, 8960), (30000, 768)):
        for K in (64, 128, 192):
            for epi in range(4):
                head, kernel, _ = B.chorus_gemm_bf16_plan(M, N, K, epi)
                assert head == 0 and (epi < B.EPI_F32 or kernel == 4), (M, N, K, epi)
    assert B.chorus_gemm_bf16_plan(3700, 4608, 256, B.EPI_RESID)[0] == 3584


def test_small_tiles_up_to_two_workgroups_a_unit():
    """A third workgroup on a unit waits for a place: 64 x 64 tiles were never the fastest with more than 512 of them."""
    for M, N, K, epi in ((691, 3072, 8960, B.EPI_BF16), (700, 3072, 8960, B.EPI_RESID), (691, 3072, 4096, B.EPI_RESID),
                         (1382, 1536, 8960, B.EPI_RESID), (1382, 1536, 8960, B.EPI_BF16), (1382, 1536, 4096, B.EPI_GELU_BF16)):
        assert B.chorus_gemm_bf16_plan(M, N, K, epi) == (0, 5, 1), (M, N, K, epi)
    assert B.chorus_gemm_bf16_plan(1240, 1536, 8960, B.EPI_RESID) == (0, 1, 1)
    for M in range(64, 6000, 96):
        for N in (256, 768, 1536, 3072, 4608, 5120):
            for K in (256, 1536, 8960):
                head, kernel, _ = B.chorus_gemm_bf16_plan(M, N, K, B.EPI_BF16)
                assert kernel != 1 or -(-(M - head) // 64) * -(-N // 64) <= 512, (M, N, K)


def _ffn2(D, H, F, Lt, Ls):
    shape = B.make_block_shape(D, H, D // H, F, Lt, (21, 60, 90))
    return B.chorus_gemm_bf16_plan(Ls, D, F, B.EPI_RESID, *ffn2_scratch(shape, Ls))


def test_second_ffn_product_in_slices():
    for (Ls, Lt, F), slices in FFN_SLICES.items():
        assert _ffn2(256, 4, F, Lt, Ls) == (0, 1, slices), (Ls, Lt, F)
    for Ls, kernel, slices in ((128, 1, 4), (300, 1, 2), (480, 5, 4), (700, 5, 3), (960, 4, 3), (1200, 5, 2), (1500, 4, 2),
                               (2000, 2, 2), (3000, 4, 1), (4000, 2, 1)):
        assert _ffn2(1536, 12, 8960, 512, Ls) == (0, kernel, slices), Ls
    for Ls, kernel, slices in ((64, 1, 3), (128, 5, 4), (300, 2, 4), (480, 2, 3), (700, 2, 2), (960, 3, 3), (2000, 3, 3),
                               (4000, 3, 3), (5000, 3, 1)):
        assert _ffn2(5120, 40, 13824, 512, Ls) == (0, kernel, slices), Ls
    # the scratch bounds the slices: none at all, one result in front, further ones behind the hidden rows
    one = 480 * 1536 * 4
    assert B.chorus_gemm_bf16_plan(480, 1536, 8960, B.EPI_RESID)[2] == 1
    assert B.chorus_gemm_bf16_plan(480, 1536, 8960, B.EPI_RESID, one - 1, 8 * one)[2] == 1
    assert B.chorus_gemm_bf16_plan(480, 1536, 8960, B.EPI_RESID, one, 0)[2] <= 2
    assert B.chorus_gemm_bf16_plan(480, 1536, 8960, B.EPI_RESID, one, 2 * one - 1)[2] <= 3
    assert B.chorus_gemm_bf16_plan(480, 1536, 8960, B.EPI_RESID, one, 2 * one)[2] == 4
    assert B.chorus_gemm_bf16_plan(480, 1536, 8960, B.EPI_F32, one, 2 * one)[2] == 1  # the gated residual only
    assert B.chorus_gemm_bf16_plan(64, 64, 128, B.EPI_RESID, one, 2 * one)[2] <= 2    # no more slices than steps


def test_residual_products_in_chained_slices():
    """The choice that a block makes: a chain where every slice has a unit and 16 steps or more, and it is estimated to be faster."""
    plan = lambda M, N, K, first=0, rest=0: B.chorus_gemm_bf16_chain_plan(M, N, K, first, rest)  # noqa: E731
    for M, want in ((3271, (0, 3, 3, True)), (4500, (0, 3, 2, True)), (2000, (0, 2, 2, True)), (1350, (0, 2, 3, True)), (1100, (0, 5, 2, True))):
        assert plan(M, 1536, 8960, 4 * M * 1536) == want, M
    assert plan(480, 1536, 8960, 4 * 480 * 1536, 8 * 480 * 1536) == (0, 5, 4, False)  # slices with scratch
    assert plan(13104, 1536, 8960) == (10752, 2, 2, True)                            # the rows behind the last whole round
    for M in (300, 1200, 3271, 13104):
        assert not plan(M, 1536, 1536)[3] and not plan(M, 256, 1024)[3]              # too few steps
    assert plan(6000, 1536, 8960)[2:] == plan(32760, 1536, 8960)[2:] == plan(75600, 5120, 13824)[2:] == (1, False)
    assert plan(960, 5120, 13824) == plan(960, 5120, 5120) == (0, 3, 3, True)
    assert not plan(300, 1 << 21, 4096)[3] and not plan(64, 64, 1 << 22)[3]          # out of the 32-bit offsets' reach
    for M in range(64, 6000, 160):
        for N, K in ((768, 3072), (1536, 8960), (3072, 4096), (5120, 5120)):
            head, kernel, slices, chained = plan(M, N, K)
            rows, cols = {1: (64, 64), 2: (128, 256), 3: (256, 256), 4: (128, 128), 5: (128, 128)}[kernel]
            assert not chained or (-(-(M - head) // rows) * -(-N // cols) * slices <= 256 and K // 64 // slices >= 16), (M, N, K)
    out, chained = B.GemmPlan(), B.C.c_int32()
    for bad, status in (((0, 64, 64), B.E_ARG), ((8, 64, 100), B.E_SHAPE), ((8, 60, 64), B.E_SHAPE)):
        assert B.load().chorus_gemm_bf16_chain_plan(*bad, 0, 0, B.C.byref(out), B.C.byref(chained)) == status
    assert B.load().chorus_gemm_bf16_chain_plan(8, 64, 64, 0, 0, None, B.C.byref(chained)) == B.E_ARG


def test_two_products_in_one_launch():
    """Where one launch for both is the faster one as measured: by the tiles of both together, not of the first alone."""
    two = lambda D, Ls, Lt: B.chorus_gemm_bf16_two_plan(Ls, 3 * D, Lt, 2 * D, D)  # noqa: E731
    for D, _, _, Ls, Lt, kernel in TEXT_CASES:
        assert two(D, Ls, Lt) == kernel, (D, Ls, Lt)
    for D, Ls, Lt in ((256, 128, 16), (256, 1200, 512), (1536, 100, 16), (1536, 200, 77)):
        assert two(D, Ls, Lt) == 1, (D, Ls, Lt)
    for D, Ls, Lt in ((256, 4000, 512), (1536, 640, 226), (1536, 900, 512), (5120, 100, 77), (5120, 100, 512)):
        assert two(D, Ls, Lt) == 5, (D, Ls, Lt)
    for D, Ls, Lt in ((1536, 800, 16), (1536, 800, 512), (1536, 300, 2048), (5120, 64, 512), (5120, 160, 16), (5120, 160, 77),
                      (5120, 200, 16), (5120, 200, 512), (5120, 256, 512), (5120, 100, 2048)):
        assert two(D, Ls, Lt) == 0, (D, Ls, Lt)
    assert B.chorus_gemm_bf16_two_plan(64, 64, 64, 64, 1 << 22) == 0  # rows beyond 32-bit offsets
    out = B.C.c_int32()
    for bad in ((0, 64, 8, 64, 64), (8, 64, 0, 64, 64), (8, 0, 8, 64, 64), (8, 64, 8, 64, 0)):
        assert B.load().chorus_gemm_bf16_two_plan(*bad, B.C.byref(out)) == B.E_ARG
    for bad in ((8, 60, 8, 64, 64), (8, 64, 8, 60, 64), (8, 64, 8, 64, 100)):
        assert B.load().chorus_gemm_bf16_two_plan(*bad, B.C.byref(out)) == B.E_SHAPE


def test_rows_beyond_32_bit_offsets_are_planned_as_they_run():
    for M, N in ((70, 72), (4500, 4608), (20000, 8960)):
        for epi in range(4):
            assert B.chorus_gemm_bf16_plan(M, N, (1 << 22) + 64, epi) == (0, 1, 1), (M, N, epi)
    head, kernel, slices = B.chorus_gemm_bf16_plan(70, 72, (1 << 22) + 64, B.EPI_RESID, 1 << 20, 1 << 20)
    assert (head, kernel) == (0, 1) and slices > 1
    assert B.chorus_gemm_bf16_plan(20000, 8960, (1 << 22) - 64, B.EPI_BF16)[1] == 3


def test_gemm_plan_refuses():
    lib, out = B.load(), B.GemmPlan()
    for bad in ((0, 64, 64, 0), (8, 0, 64, 0), (8, 64, 0, 0), (8, 64, 64, 4), (8, 64, 64, -1)):
        assert lib.chorus_gemm_bf16_plan(*bad, 0, 0, B.C.byref(out)) == B.E_ARG
    assert lib.chorus_gemm_bf16_plan(8, 64, 64, 0, 0, 0, None) == B.E_ARG
    assert lib.chorus_gemm_bf16_plan(8, 64, 100, 0, 0, 0, B.C.byref(out)) == B.E_SHAPE
    assert lib.chorus_gemm_bf16_plan(8, 60, 64, 0, 0, 0, B.C.byref(out)) == B.E_SHAPE


@pytest.mark.parametrize("T,H,W", [(1, 1, 1), (21, 30, 52), (21, 45, 80), (1, 1024, 64), (1, 1500, 40), (3, 900, 100), (1, 40, 3000),
                                   (2, 4, 90000), (1, 4, 400000)])
def test_mask_hierarchy_radii_end_at_the_grid(T, H, W):
    """A radius beyond the grid reaches what the grid's extent reaches; the kernels loop over what they are given."""
    last, held_before = (T - 1, H - 1, W - 1), None
    for big in (max(T, H, W), 10 ** 6, 2 ** 30, 2 ** 31 - 1):
        for re in ((0, 0, 0), (big, big, big)):
            got = B.chorus_mask_hierarchy_plan(T, H, W, re, (big, big, big))
            assert got[0] == (last if re[0] else (0, 0, 0)) and got[1] == last
            assert held_before is None or got[2:] == held_before
            held_before = got[2:]
    for r in range(5):
        re, rs, strip, nstrips, lds = B.chorus_mask_hierarchy_plan(T, H, W, (r, 0, r), (r + 1, r, r + 2))
        assert re == (min(r, T - 1), 0, min(r, W - 1)) and rs == (min(r + 1, T - 1), min(r, H - 1), min(r + 2, W - 1))
        if strip:  # two sets of bits per row held, before and after the pass along x, and one per row of the strip
            assert (nstrips - 1) * strip < H <= nstrips * strip
            assert lds == (4 * min(H, strip + 2 * rs[1]) + 2 * strip) * -(-W // 64) * 8 <= 48 * 1024
        else:
            assert W > 64 * 100


def test_mask_hierarchy_plan_refuses():
    for T, H, W, re, rs, want in ((0, 1, 1, (0,) * 3, (0,) * 3, B.E_ARG), (1, 1, 1, (1, 0, 0), (0,) * 3, B.E_ARG),
                                  (1, 1, 1, (0, -1, 0), (0,) * 3, B.E_ARG), (2, 2 ** 15, 2 ** 15, (0,) * 3, (0,) * 3, B.E_SHAPE)):
        assert B.load().chorus_mask_hierarchy_plan(T, H, W, B._Radii(*re), B._Radii(*rs), B.C.byref(B.HierarchyPlan())) == want


def test_batch_workspace_is_what_it_was():
    """A caller may have kept the size: partial sums of as many equal slices of 64-float steps as 1024 workgroups of 64 rows allow (16 at
    most), then 32 scores a row."""
    up = lambda v, a: -(-v // a) * a  # noqa: E731
    for N in (1, 63, 64, 65, 370, 1000, 4096, 7740, 20000, 65537, 300000):
        for d in (4, 64, 380, 1024, 1096, 2056, 2640, 3420, 4076, 4096, 8192):
            for Q in (1, 16, 17, 48):
                blocks, steps = -(-N // 64), -(-d // 64)
                want = max(1, min(1024 // blocks, steps, 16))
                slices = -(-steps // -(-steps // want))
                size = up(slices * blocks * 64 * (32 if Q > 16 else 16) * 4, 256) + up(slices * blocks * 64 * 4, 256) + up(32 * blocks * 64 * 4, 256)
                assert B.load().chorus_cache_lookup_batch_workspace_bytes(N, d, Q) == size, (N, d, Q)
