"""Products in quarters of 128x128 tiles (64 x 64, eight LDS stages of a k-tile) at their edges: rows and columns around 16, 32
and 64, fewer k-tiles than stages, as many and more, a ragged last k-tile of weight gradients, as many quarters as are taken and one row more;
bias, residual, accumulation; operands off 16 bytes (another kernel).  Against float64 products of the same operands: one bf16 rounding
of the result (1e-2 of the maximum), or fp32 sums of bf16 products (2e-3); and to the bit against the tiles they stand for."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import nmax_err, host_f64  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


def operand(g, rows, cols, offset=0):
    """Rows x cols of unit variance, `offset` elements into an allocation, large values behind it."""
    flat = torch.full((offset + rows * cols + 64 * cols,), 1000.0, dtype=torch.bfloat16, device="cuda")
    flat[offset:offset + rows * cols] = torch.randn(rows * cols, generator=g, device="cuda").bfloat16()
    return flat[offset:], flat[offset:offset + rows * cols].reshape(rows, cols).double()


def product(B, m, n, k, a_layout, b_layout, out_fp32, extras=False, offset=0):
    g = torch.Generator(device="cuda").manual_seed(m + 3 * n + 7 * k)
    a, ad = operand(g, *((k, m) if a_layout else (m, k)), offset)
    b, bd = operand(g, *((n, k) if b_layout else (k, n)))
    want = (ad.t().contiguous() if a_layout else ad) @ (bd.t().contiguous() if b_layout else bd)
    c = torch.full((m + 2, n), 7.0, dtype=torch.float32 if out_fp32 else torch.bfloat16, device="cuda")
    kw = {}
    if extras and out_fp32:
        c[:m], kw["accumulate"], want = 3.0, 1, want + 3.0
    elif extras:
        bias, res = torch.randn(n, generator=g, device="cuda").bfloat16(), torch.randn(m, n, generator=g, device="cuda").bfloat16()
        kw, want = dict(bias=bias, residual=res), want + bias.double() + res.double()
    B.mllm_op_gemm(a, b, c, m, n, k, a_layout, b_layout, out_fp32, **kw)
    assert bool((c[m:] == 7.0).all())
    assert nmax_err(host_f64(c[:m]), want.cpu().numpy()) < (2e-3 if out_fp32 else 1e-2)


@pytest.mark.parametrize("extras", [False, True])
@pytest.mark.parametrize("b_layout", [0, 1])
@pytest.mark.parametrize("m,n,k", [(1, 8, 64), (15, 16, 128), (16, 24, 192), (17, 64, 448), (63, 72, 512), (64, 136, 576), (65, 128, 1024), (200, 264, 1088),
                                   (1024, 1024, 64), (1025, 1024, 64), (64, 1016, 1024), (64, 1024, 1024)])
def test_forward_and_input_gradient(B, m, n, k, b_layout, extras):
    product(B, m, n, k, 0, b_layout, 0, extras)


@pytest.mark.parametrize("extras", [False, True])
@pytest.mark.parametrize("m,n,k", [(8, 8, 1), (16, 72, 63), (64, 64, 64), (72, 136, 65), (128, 40, 511), (192, 576, 513), (1024, 1000, 77), (1032, 1000, 200)])
def test_weight_gradient(B, m, n, k, extras):
    product(B, m, n, k, 1, 0, 1, extras)


@pytest.mark.parametrize("a_layout,b_layout", [(0, 0), (0, 1), (1, 0)])
def test_operands_off_16_bytes(B, a_layout, b_layout):
    product(B, 136, 192, 320, a_layout, b_layout, a_layout, True, offset=3)


# A quarter adds up in the order of every other tile, so the form cannot be seen in a result.  Operands off 16 bytes take 128x128 tiles.
@pytest.mark.parametrize("a_layout,b_layout", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("m,n,k", [(72, 72, 64), (104, 200, 448), (200, 264, 512), (328, 192, 576), (576, 1024, 1024), (64, 768, 3584)])
def test_to_the_bit_the_tiles_they_stand_for(B, m, n, k, a_layout, b_layout):
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    c = [torch.empty(m, n, dtype=torch.float32, device="cuda") for _ in range(2)]
    a, b = (torch.randn(r, s, generator=g, device="cuda").bfloat16() for r, s in ((k, m) if a_layout else (m, k), (n, k) if b_layout else (k, n)))
    for out, offset in zip(c, (0, 3)):
        flat = torch.zeros(a.numel() + offset, dtype=torch.bfloat16, device="cuda")
        flat[offset:] = a.flatten()
        B.mllm_op_gemm(flat[offset:], b, out, m, n, k, a_layout, b_layout, 1)
    assert B.mllm_gemm_form(m, n, k, a_layout, b_layout)[0] == 64
    assert torch.equal(c[0], c[1])


# tokens either side of the line of both gradients, with the same parts of dX's K loop: 4 of 256 x 2048, none of 512 x 512
@pytest.mark.parametrize("k,n,few,many", [(256, 2048, (64, 128, 129, 288), 577), (512, 512, (64, 576, 1536), 1600)])
def test_rows_of_both_gradients_do_not_depend_on_the_other_rows(B, k, n, few, many):
    g = torch.Generator(device="cuda").manual_seed(k)
    dy, x, w = (torch.randn(*s, generator=g, device="cuda").bfloat16() for s in ((many, n), (many, k), (k, n)))
    dw, got = torch.empty(k, n, device="cuda"), {}
    for t in few + (many,):
        size = B.mllm_linear_bwd_form(t, k, n)[1]
        ws = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        got[t] = torch.empty(t, k, dtype=torch.bfloat16, device="cuda")
        B.mllm_op_linear_bwd(dy, x, w, got[t], dw, t, k, n, workspace=ws, scratch_bytes=size)
        assert B.mllm_linear_bwd_form(t, k, n)[0][1][2] == B.mllm_linear_bwd_form(many, k, n)[0][1][2]
    for t in few:
        assert torch.equal(got[t], got[many][:t])


# tokens, k, n: both gradients, dX uncut and (200 and 777 tokens x 256 x 2048) planned in parts; 256 quarters and one more
@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("t,k,n", [(1, 64, 64), (63, 64, 192), (65, 72, 128), (148, 192, 576), (129, 256, 2048), (200, 256, 2048), (777, 256, 2048),
                                   (576, 512, 512), (576, 512, 1472), (576, 512, 1536), (1025, 192, 64)])
def test_both_gradients(B, t, k, n, accumulate):
    g = torch.Generator(device="cuda").manual_seed(t + k + n)
    (dy, dyd), (x, xd), (w, wd) = operand(g, t, n), operand(g, t, k), operand(g, k, n)
    size = B.mllm_linear_bwd_form(t, k, n)[1]
    ws = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
    dx = torch.full((t + 2, k), 7.0, dtype=torch.bfloat16, device="cuda")
    dw = torch.full((k, n), 3.0 if accumulate else float("nan"), device="cuda")
    B.mllm_op_linear_bwd(dy, x, w, dx, dw, t, k, n, accumulate, workspace=ws, scratch_bytes=size)
    assert bool((dx[t:] == 7.0).all())
    assert nmax_err(host_f64(dx[:t]), (dyd @ wd.t().contiguous()).cpu().numpy()) < 1e-2
    assert nmax_err(host_f64(dw), (xd.t().contiguous() @ dyd + 3.0 * accumulate).cpu().numpy()) < 2e-3


@pytest.mark.parametrize("a_layout,b_layout", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_whole_tiles_with_more_quarters_than_compute_units(B, a_layout, b_layout, tiles):
    """128x128 tiles with a CU each that are not quartered: any number of k-tiles over their four LDS stages."""
    m, n, k = 1096, 1160, 64 * tiles - (13 if a_layout else 0)
    assert B.mllm_gemm_form(m, n, k, a_layout, b_layout)[0] == 128
    for out_fp32 in (0, 1):
        for extras in (False, True):
            product(B, m, n, k, a_layout, b_layout, out_fp32, extras)
