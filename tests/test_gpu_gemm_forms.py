"""Products on four and on eight wavefronts where the choice between them turns, against float64 products of the same operands.

bf16 results carry one rounding (1e-2 of the maximum), fp32 sums of bf16 products 2e-3."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import host_f64, nmax_err  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


def product(B, m, n, k, a_layout, b_layout, f32, offset=0):
    """Relative error of the product; the rows of the operands behind K hold large values."""
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    rows = k + 64
    a = torch.randn(rows if a_layout else m, m if a_layout else k, generator=g, device="cuda").bfloat16()
    b = (torch.randn(n if b_layout else rows, k if b_layout else n, generator=g, device="cuda") * 0.125).bfloat16()
    for t, turned in ((a, a_layout), (b, not b_layout)):
        if turned:
            t[k:] = 1000.0
    av, bv = (a[:k].double().t().contiguous() if a_layout else a.double()), (b.double().t().contiguous() if b_layout else b[:k].double())
    if offset:
        flat = torch.zeros(a.numel() + offset, dtype=torch.bfloat16, device="cuda")
        flat[offset:] = a.flatten()
        a = flat[offset:]
    c = torch.full((m + 2, n), 7.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
    B.mllm_op_gemm(a, b, c, m, n, k, a_layout, b_layout, out_fp32=f32)
    assert bool((c[m:] == 7.0).all())
    return nmax_err(host_f64(c[:m]), (av @ bv).cpu().numpy())


LAYOUTS = [(0, 0), (0, 1), (1, 0)]


@pytest.mark.parametrize("a_layout,b_layout", LAYOUTS)
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_every_remainder_of_the_four_stages(B, a_layout, b_layout, tiles):
    """128x128 tiles with a CU each: any number of k-tiles over four LDS stages, a ragged last one where k runs along the rows."""
    m, n, k = 1096, 1160, 64 * tiles - (13 if a_layout else 0)
    assert B.mllm_gemm_form(m, n, k, a_layout, b_layout)[0] == 128
    for f32 in (0, 1):
        assert product(B, m, n, k, a_layout, b_layout, f32) < (2e-3 if f32 else 1e-2)


# rows of tiles x columns of tiles: the last number of workgroups on eight wavefronts and the first on four
@pytest.mark.parametrize("a_layout,b_layout", LAYOUTS)
@pytest.mark.parametrize("m,n", [(2040, 2048), (2040, 2056), (2056, 2056)])
def test_as_many_small_tiles_as_compute_units_and_more(B, a_layout, b_layout, m, n):
    assert B.mllm_gemm_form(m, n, 192, a_layout, b_layout)[0] == 128
    for offset in (0, 3):
        assert product(B, m, n, 192, a_layout, b_layout, 0, offset) < 1e-2


@pytest.mark.parametrize("k", [8128, 8192, 8256])
def test_forward_layout_at_the_line_in_the_contraction(B, k):
    assert B.mllm_gemm_form(3336, 5128, k)[0] in (192, 256)
    assert product(B, 3336, 5128, k, 0, 0, 0) < 1e-2


@pytest.mark.parametrize("k", [64, 128, 192, 200, 457])
def test_large_tiles_on_eight_wavefronts_stored_by_k(B, k):
    """Both operands stored [K, .], the last k-tile whole and ragged; operands off 16 bytes go through registers."""
    assert B.mllm_gemm_form(704, 20944, k, 1, 0)[0] == 256
    for offset in (0, 5):
        assert product(B, 704, 20944, k, 1, 0, 1, offset) < 2e-3


# k-tiles either side of the lines between four and eight wavefronts: 192-row tiles 24 (64 from two rounds on), 256-row tiles 32 for at most a
# round and 64 beyond, weight gradients 64 (any number from a round of a matrix wider than high on)
@pytest.mark.parametrize("m,n,k,a_layout", [(5960, 1312, 1536, 0), (5960, 1312, 1600, 0), (2216, 5536, 2048, 0), (2216, 5536, 2112, 0),
                                            (6000, 7000, 4096, 0), (6000, 7000, 4160, 0), (640, 20944, 4096, 1), (640, 20944, 4097, 1),
                                            (20944, 640, 4096, 1), (20944, 640, 4100, 1), (1024, 20736, 4161, 1), (20736, 1024, 4161, 1)])
def test_either_side_of_the_lines_of_the_large_tiles(B, m, n, k, a_layout):
    assert B.mllm_gemm_form(m, n, k, a_layout, 0)[0] == (192 if n == 1312 else 256)
    for offset in (0, 3):
        assert product(B, m, n, k, a_layout, 0, a_layout, offset) < (2e-3 if a_layout else 1e-2)


def shifted(t, offset):
    """The same values, `offset` elements behind an allocation's start."""
    flat = torch.zeros(t.numel() + offset, dtype=t.dtype, device="cuda")
    flat[offset:] = t.flatten()
    return flat[offset:]


# operands off 16 bytes and contractions over 4096 keep the fused epilogues on four wavefronts
@pytest.mark.parametrize("x_at,w_at", [(0, 0), (0, 1), (3, 0), (3, 3)])
@pytest.mark.parametrize("m,f,k", [(4200, 1536, 320), (6401, 1024, 64), (2900, 2304, 4160)])
def test_swiglu_epilogue_on_four_wavefronts(B, m, f, k, x_at, w_at):
    """[gate | up] carries one rounding (1e-2), silu(gate) * up another (2e-2)."""
    g = torch.Generator(device="cuda").manual_seed(m + k)
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    w = (torch.randn(k, 2 * f, generator=g, device="cuda") * 0.125).bfloat16()
    pre, act = (torch.full((m, c), float("nan"), dtype=torch.bfloat16, device="cuda") for c in (2 * f, f))
    B.mllm_op_gemm_swiglu(shifted(x, x_at), shifted(w, w_at), pre, act, m, f, k)
    ref = x.double() @ w.double()
    gate, up = ref[:, :f], ref[:, f:]
    assert nmax_err(host_f64(pre), ref.cpu().numpy()) < 1e-2
    assert nmax_err(host_f64(act), (gate * torch.sigmoid(gate) * up).cpu().numpy()) < 2e-2


@pytest.mark.parametrize("x_at,w_at", [(0, 0), (0, 1), (3, 0)])
@pytest.mark.parametrize("k", [64, 320, 4160])
def test_rotary_epilogue_of_64_wide_heads_on_four_wavefronts(B, k, x_at, w_at):
    m, n, rot, hd = 4101, 3584, 2560, 64
    g = torch.Generator(device="cuda").manual_seed(k)
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    w = (torch.randn(k, n, generator=g, device="cuda") * 0.06).bfloat16()
    pos = torch.arange(m, device="cuda", dtype=torch.int32)
    table = torch.empty(m, hd, device="cuda")
    B.mllm_op_rope_table(table, m, hd, 10000.0)
    y = torch.zeros(m, n, dtype=torch.bfloat16, device="cuda")
    B.mllm_op_gemm_rope(shifted(x, x_at), shifted(w, w_at), None, y, m, n, k, pos, table, rot, hd)
    ref = x.double() @ w.double()
    cos, sin = (t.double()[:, None, :] for t in table.split(hd // 2, dim=1))
    a, b = ref[:, :rot].reshape(m, rot // hd, 2, hd // 2).unbind(2)
    want = torch.cat([torch.stack([a * cos - b * sin, b * cos + a * sin], dim=2).reshape(m, rot), ref[:, rot:]], dim=1)
    assert nmax_err(host_f64(y), want.cpu().numpy()) < 1e-2
