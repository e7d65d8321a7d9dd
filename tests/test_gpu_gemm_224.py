"""Products planned in 256-row tiles whose rows fit as many tiles of 224: rows at the edges of those tiles and one more (256 again), in
forward layout with and without bias and residual, with the SwiGLU and the rotary epilogues, cut, and as the input gradient beside
a weight gradient, with and without the SwiGLU gradient.  Against float64 products of the same operands: one bf16 rounding of the
result (1e-2 of the maximum; activations and gradients through SwiGLU 2e-2), fp32 sums 2e-3."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


def error(got, want):
    return float((got.double() - want).abs().max() / want.abs().max())


def randn(g, *shape, scale=1.0):
    return (torch.randn(*shape, generator=g, device="cuda") * scale).bfloat16()


@pytest.mark.parametrize("k", [64, 192, 704])
@pytest.mark.parametrize("m", [193, 224, 225, 447, 448, 449, 672, 1343, 1568])
def test_fused_epilogues(B, m, k):
    g = torch.Generator(device="cuda").manual_seed(m + k)
    f = 6272 * (1 + 1024 // m)                 # 200 tiles of 256 x 256 and more
    x, w, bias = randn(g, m, k), randn(g, k, 2 * f, scale=0.125), randn(g, 2 * f)
    ref = x.double() @ w.double()
    y = torch.full((m + 1, 2 * f), 7.0, dtype=torch.bfloat16, device="cuda")
    pre, act = (torch.full((m + 1, c), 7.0, dtype=torch.bfloat16, device="cuda") for c in (2 * f, f))
    B.mllm_op_gemm_swiglu(x, w, pre, act, m, f, k)
    gate, up = ref.split(f, dim=1)
    assert error(pre[:m], ref) < 1e-2 and error(act[:m], gate * torch.sigmoid(gate) * up) < 2e-2
    assert bool((pre[m:] == 7.0).all()) and bool((act[m:] == 7.0).all())
    pos = torch.arange(m, device="cuda", dtype=torch.int32)
    for hd in (64, 128):
        rot = 2 * f - 256
        table = torch.empty(m, hd, device="cuda")
        B.mllm_op_rope_table(table, m, hd, 10000.0)
        B.mllm_op_gemm_rope(x, w, bias, y, m, 2 * f, k, pos, table, rot, hd)
        cos, sin = (t.double()[:, None, :] for t in table.split(hd // 2, dim=1))
        b = ref + bias.double()
        lo, hi = b[:, :rot].reshape(m, rot // hd, 2, hd // 2).unbind(2)
        want = torch.cat([torch.stack([lo * cos - hi * sin, hi * cos + lo * sin], dim=2).reshape(m, rot), b[:, rot:]], dim=1)
        assert error(y[:m], want) < 1e-2


# rows and columns whose plan is tiles of 256, and one row more than the last that takes 224
@pytest.mark.parametrize("k", [64, 192, 704])
@pytest.mark.parametrize("b_layout", [0, 1])
@pytest.mark.parametrize("m,n,tile", [(430, 22320, 224), (448, 21800, 224), (449, 21800, 256), (672, 17120, 224), (896, 14000, 224), (897, 14000, 256), (1343, 9840, 224),
                                      (1568, 8280, 224), (1569, 8280, 256)])
def test_plain_products(B, m, n, tile, b_layout, k):
    assert B.mllm_gemm_form(m, n, k, 0, b_layout) == (tile, 256, 1)
    g = torch.Generator(device="cuda").manual_seed(m + k)
    x, w, bias, res = randn(g, m, k), randn(g, *((n, k) if b_layout else (k, n)), scale=0.125), randn(g, n), randn(g, m, n)
    ref = x.double() @ (w.double().t().contiguous() if b_layout else w.double())
    y = torch.full((m + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")
    B.mllm_op_gemm(x, w, y, m, n, k, 0, b_layout, bias=bias, residual=res)
    assert error(y[:m], ref + bias.double() + res.double()) < 1e-2 and bool((y[m:] == 7.0).all())
    c = torch.full((m + 1, n), 3.0, device="cuda")
    B.mllm_op_gemm(x, w, c, m, n, k, 0, b_layout, out_fp32=1, accumulate=1)
    assert error(c[:m], ref + 3.0) < 2e-3 and bool((c[m:] == 3.0).all())


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("t,k,n", [(224, 3584, 18944), (430, 4096, 8192), (448, 14336, 4096), (449, 14336, 4096), (777, 4096, 6144), (777, 14336, 4096)])
def test_both_gradients(B, t, k, n, accumulate):
    """Accumulating and not; with the scratch that is wanted and with none (then uncut)."""
    (one, x_form, _, _), want = B.mllm_linear_bwd_form(t, k, n)
    assert one and x_form[0] == (256 if t == 449 else 224)
    g = torch.Generator(device="cuda").manual_seed(t + k)
    dy, x, w = randn(g, t, n), randn(g, t, k), randn(g, k, n, scale=0.125)
    ref_x, ref_w = dy.double() @ w.double().t().contiguous(), x.double().t().contiguous() @ dy.double()
    for size in {want, 0}:
        dx = torch.full((t + 2, k), 7.0, dtype=torch.bfloat16, device="cuda")
        dw = torch.full((k, n), 3.0 if accumulate else float("nan"), device="cuda")
        ws = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        B.mllm_op_linear_bwd(dy, x, w, dx, dw, t, k, n, accumulate, workspace=ws, scratch_bytes=size)
        assert error(dx[:t], ref_x) < 1e-2 and error(dw, ref_w + 3.0 * accumulate) < 2e-3 and bool((dx[t:] == 7.0).all())


@pytest.mark.parametrize("t,f,n", [(448, 25728, 192), (777, 14336, 1024), (1560, 8320, 4096)])
def test_swiglu_gradient(B, t, f, n):
    g = torch.Generator(device="cuda").manual_seed(t)
    dy, act, pre, w = randn(g, t, n), randn(g, t, f), randn(g, t, 2 * f), randn(g, f, n, scale=0.125)
    (one, x_form, _, _), want = B.mllm_linear_bwd_form(t, f, n, swiglu=1)
    assert one and x_form == (224, 256, 1)
    dpre, dw = torch.full((t + 1, 2 * f), 7.0, dtype=torch.bfloat16, device="cuda"), torch.full((f, n), float("nan"), device="cuda")
    ws = torch.empty(want + 256, dtype=torch.uint8, device="cuda")
    B.mllm_op_linear_bwd(dy, act, w, dpre, dw, t, f, n, swiglu_pre=pre, workspace=ws, scratch_bytes=want)
    da, gate, up = dy.double() @ w.double().t().contiguous(), pre[:, :f].double(), pre[:, f:].double()
    s = torch.sigmoid(gate)
    assert error(dpre[:t, :f], da * up * s * (1.0 + gate * (1.0 - s))) < 2e-2 and error(dpre[:t, f:], da * gate * s) < 2e-2
    assert error(dw, act.double().t().contiguous() @ dy.double()) < 2e-3 and bool((dpre[t:] == 7.0).all())
