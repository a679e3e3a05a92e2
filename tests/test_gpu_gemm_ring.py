"""The GEMM's ring of operand halves in LDS: products of one to nine k-steps (fewer than the ring holds, as many, more) on
every tile, with rows and columns that end inside a tile, on its edge and one behind it; rows longer than 32-bit offsets
reach. The operands are small integers, so every order of summation gives the same bits."""
import pytest
import torch

from paper_2604_04451_amd import binding as B

pytestmark = pytest.mark.gpu
TILES = {1: (64, 64), 2: (128, 256), 3: (256, 256), 4: (128, 128), 5: (128, 128)}


def _ints(shape, seed, lo=-2, hi=3):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randint(lo, hi, shape, generator=g, device="cuda").to(torch.float32)


def _check(M, N, K, kernel, epi):
    print(f"[case] gemm ring kernel={kernel} M={M} N={N} K={K} epi={epi}", flush=True)
    A, W, b = _ints((M, K), 1), _ints((N, K), 2), _ints((N,), 3)
    out = _ints((M, N), 4)
    want = A @ W.T + b + (out if epi == B.EPI_RESID else 0)
    guard = torch.full((2, N), 7.0, device="cuda")
    buf = torch.cat((out, guard))
    B.chorus_gemm_bf16(A.bfloat16(), W.bfloat16(), epi, buf[:M], b, kernel=kernel)
    torch.cuda.synchronize()
    assert torch.equal(buf[:M], want) and torch.equal(buf[M:], guard)


@pytest.mark.parametrize("kernel", list(TILES))
@pytest.mark.parametrize("steps", range(1, 10))
def test_steps_and_edges(kernel, steps):
    rows, cols = TILES[kernel]
    for M, N in ((1, 8), (rows - 1, cols), (rows, cols - 8), (rows + 1, cols + 8), (2 * rows + 3, 2 * cols + 24)):
        _check(M, N, 64 * steps, kernel, B.EPI_F32 if steps % 2 else B.EPI_RESID)


FAR_K = (1 << 22) + 64


def _far_operands(M, N):
    """256 rows of 2 K bytes pass 2^31 from K = 2^22 on; sums of 2^22 products of -1, 0 and 1 stay whole in fp32."""
    A, W = _ints((M, FAR_K), 5, -1, 2), _ints((N, FAR_K), 6, -1, 2)
    want = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    for k in range(0, FAR_K, 1 << 16):
        want += (A[:, k:k + (1 << 16)] @ W[:, k:k + (1 << 16)].T).double()
    return A.bfloat16(), W.bfloat16(), want


@pytest.mark.parametrize("kernel", [0, 3])  # the default choice and a named kernel, which stands for the one by 64-bit addresses
def test_rows_beyond_32_bit_offsets(kernel):
    M, N = 130, 72
    A, W, want = _far_operands(M, N)
    out = torch.empty(M, N, device="cuda")
    print(f"[case] gemm far rows kernel={kernel}", flush=True)
    B.chorus_gemm_bf16(A, W, B.EPI_F32, out, None, kernel=kernel)
    assert torch.equal(out.double(), want)


def test_rows_beyond_32_bit_offsets_in_slices():
    M, N = 70, 136
    A, W, want = _far_operands(M, N)
    for slices in (2, 3, 4):
        print(f"[case] gemm far rows slices={slices}", flush=True)
        out = _ints((M, N), 7)
        ref = out.double() + want
        parts = torch.full((slices - 1, M, N), float("nan"), device="cuda")
        B.chorus_gemm_bf16_slices(A, W, out, 1, slices, parts=parts.view(-1))
        assert torch.equal(out.double(), ref)
