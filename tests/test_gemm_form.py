"""Which GEMM kernel a product takes (host logic, no GPU), and that the kernel's 32-bit addresses reach it."""
import pytest

LIMIT = 0xFFFFFFF0 - 16   # bytes of an operand that a product accepts


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


def rows_that_wrap(rows, width):
    """Rows past the end of a [rows, width] bf16 operand that a whole last k-tile of 64 reads at a 32-bit offset
    which falls into the operand again."""
    pitch, end = 2 * width, -(-rows // 64) * 64
    return [r for r in range(rows, end) if (r * pitch + 2 * (width - 8)) % 2 ** 32 < rows * pitch or (r * pitch) % 2 ** 32 < rows * pitch]


# widths of both operands; the last ones only one of the two close to 4 GiB
@pytest.mark.parametrize("m,n", [(3200, 3200), (5120, 5120), (32760, 32760), (28672, 64), (64, 28672)])
def test_ragged_contraction_near_4_gib_keeps_to_the_kernel_that_compares_rows(B, m, n):
    most = LIMIT // (2 * max(m, n))
    seen = set()
    for k in range(most - 200, most + 1):
        wraps = bool(rows_that_wrap(k, m) or rows_that_wrap(k, n))
        tiled = B.mllm_gemm_form(m, n, k, 1, 0)[0] != 0
        assert not (tiled and wraps), k
        assert tiled or k % 64, k          # whole k-tiles have no row past the end
        seen.add((tiled, wraps))
    assert (True, False) in seen           # further from the limit the tile kernel stays


def test_ragged_contraction_examples(B):
    assert rows_that_wrap(671050, 3200)                        # 247 KB short of 4 GiB
    assert B.mllm_gemm_form(3200, 3200, 671050, 1, 0) == (0, 0, 1)
    assert B.mllm_gemm_form(3200, 3200, 671040, 1, 0)[0] != 0    # a multiple of 64
    assert B.mllm_gemm_form(5120, 5120, 419400, 1, 0) == (0, 0, 1)
    assert B.mllm_gemm_form(4096, 4096, 777, 1, 0)[0] != 0
    assert B.mllm_gemm_form(4096, 4096, 776, 0, 0) == (0, 0, 1)  # k along the rows of only one operand
    assert B.mllm_gemm_form(64, 64, 0, 1, 0) == (0, 0, 1)


def test_no_plan_leaves_a_part_empty(B):
    """A part is a whole number of k-tiles, at least eight, and the last one has some: over shapes of every layout, with
    all the scratch a plan wants and with less."""
    cut = 0
    for m in (72, 777, 1024, 1280, 3200):
        for n in (192, 1024, 1280, 4096):
            for k in list(range(64, 8000, 64 * 7)) + [6720, 26496, 37888]:
                for a_layout, b_layout in ((0, 0), (0, 1), (1, 0)):
                    for scratch in (1 << 40, 5 * m * n * 4):
                        parts = B.mllm_gemm_form(m, n, k, a_layout, b_layout, scratch)[2]
                        tiles = k // 64
                        per = -(-tiles // parts)
                        assert (parts - 1) * per < tiles and (parts == 1 or per >= 8) and parts * m * n * 4 <= max(scratch, m * n * 4)
                        cut += parts > 1
    assert cut > 100


# the last product in quarters of 128x128 tiles and the first that is not; rows that fill as many tiles of 224 as of 256 and others
@pytest.mark.parametrize("m,n,k,a_layout,b_layout,tile", [
    (1024, 1024, 64, 0, 0, 64), (1025, 1024, 64, 0, 0, 128), (576, 1024, 1024, 0, 1, 64), (1024, 1024, 77, 1, 0, 64), (1032, 1024, 77, 1, 0, 128), (200, 520, 320, 1, 1, 128),
    (896, 14336, 4096, 0, 0, 224), (897, 14336, 4096, 0, 0, 256), (1568, 8320, 704, 0, 1, 224), (1569, 8320, 704, 0, 1, 256), (896, 28672, 4096, 1, 0, 256)])
def test_the_tile_that_runs_is_named(B, m, n, k, a_layout, b_layout, tile):
    assert B.mllm_gemm_form(m, n, k, a_layout, b_layout) == (tile, 256 if tile > 128 else tile, 1)


# rows x columns x contraction of a decoder's down projection for a few hundred tokens: fewer tiles than compute units over a long
# contraction
@pytest.mark.parametrize("m", [444, 600, 763, 900])
@pytest.mark.parametrize("n,k", [(3584, 18944), (4096, 14336), (4096, 11008)])
def test_long_contractions_of_few_tiles_are_cut(B, m, n, k):
    """Uncut they take 1.1 to 1.4 times as long with weights that come from memory."""
    assert B.mllm_gemm_form(m, n, k, 0, 0, 1 << 40)[2] > 1
