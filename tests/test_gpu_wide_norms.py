"""Norms of rows wider than 1024 (a workgroup a row) and the sums over tokens at the edges of their tiles, against float64.

One bf16 rounding of y and dx (1e-2 of the maximum); fp32 sums of bf16 values and their second stage 2e-3."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import host_f64, nmax_err, scratch  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


# rows: one, fewer than workgroups, several a workgroup; widths: the first wide one, ragged, each number of vectors a thread
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("t,d", [(1, 1032), (3, 2048), (770, 2056), (2400, 1096), (777, 4096), (1601, 4104), (40, 8192)])
def test_wide_norm(B, kind, t, d):
    g = torch.Generator(device="cuda").manual_seed(t + d + kind)
    x, dy, dres = (torch.randn(t, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    gam = (1 + 0.02 * torch.randn(1, d, generator=g, device="cuda")).bfloat16()
    bet = (0.02 * torch.randn(1, d, generator=g, device="cuda")).bfloat16()
    y, dx = (torch.full_like(x, float("nan")) for _ in range(2))
    stats = torch.empty(2, t, device="cuda")
    B.mllm_op_norm_fwd(kind, x, gam, bet if kind == 0 else None, y, stats, t, d, 1e-5)
    X, G = x.double(), gam.double()
    if kind == 0:
        X = X - X.mean(1, keepdim=True)
    r = torch.rsqrt((X * X).mean(1, keepdim=True) + 1e-5)
    xh = X * r
    assert nmax_err(host_f64(y), (xh * G + (bet.double() if kind == 0 else 0.0)).cpu().numpy()) < 1e-2
    dgam, dbet = torch.full((1, d), float("nan"), device="cuda"), torch.full((1, d), float("nan"), device="cuda")
    part = scratch(B.mllm_op_norm_bwd_partial_bytes(t, d))
    B.mllm_op_norm_bwd(kind, dy, x, gam, stats, dres, dx, dgam, dbet if kind == 0 else None, 0, part, t, d)
    dxh = dy.double() * G
    want = dxh - xh * (dxh * xh).mean(1, keepdim=True) - (dxh.mean(1, keepdim=True) if kind == 0 else 0.0)
    assert nmax_err(host_f64(dx), (want * r + dres.double()).cpu().numpy()) < 1e-2
    assert nmax_err(host_f64(dgam), (dy.double() * xh).sum(0, keepdim=True).cpu().numpy()) < 2e-3
    if kind == 0:
        assert nmax_err(host_f64(dbet), dy.double().sum(0, keepdim=True).cpu().numpy()) < 2e-3


@pytest.mark.parametrize("t,n", [(1, 8), (15, 40), (16 * 33, 136), (16 * 255, 1032), (16 * 257, 24), (9000, 264)])
def test_column_sums(B, t, n):
    """Rows of partial sums below, at and above the slices of a workgroup and the loads it keeps in flight."""
    x = torch.randn(t, n, generator=torch.Generator(device="cuda").manual_seed(t), device="cuda").bfloat16()
    init = torch.randn(1, n, device="cuda")
    out = init.clone()
    B.mllm_op_colsum(x, out, 1, scratch(B.mllm_op_colsum_partial_bytes(t, n)), t, n)
    ref = (x.double().sum(0, keepdim=True) + init.double()).cpu().numpy()
    assert nmax_err(host_f64(out), ref) < 2e-3
