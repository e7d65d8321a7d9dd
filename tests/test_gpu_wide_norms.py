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


# either side of each line between a wavefront and a workgroup a row: 1536 rows up to 2048 columns; RMSNorm up to 4096 columns
# between 3/4 of the columns and 5120 rows; and more rows than a grid's first dimension is given
@pytest.mark.parametrize("kind,t,d", [(0, 1536, 1288), (0, 1537, 1288), (1, 1536, 2048), (1, 1537, 2048), (1, 1728, 2304), (1, 1729, 2304),
                                      (1, 5120, 2056), (1, 5121, 2056), (1, 3073, 4096), (0, 3073, 4096), (1, 4000, 4104),
                                      (0, (1 << 20) + 3, 2056), (1, (1 << 20) + 3, 2056), (1, (1 << 24) + 3, 1032)])
def test_norm_at_the_lines_between_its_forms(B, kind, t, d):
    """The first and last rows, and those around multiples of a million, against float64; the others' results are written by the
    same code.  y 1e-2 of the maximum (one rounding), rstd and mean 1e-5 (fp32 sums of at most 8192 terms)."""
    torch.cuda.empty_cache()
    if t * d * 4 > torch.cuda.mem_get_info()[0] * 3 // 4:
        pytest.skip("needs %d GB" % (t * d * 4 >> 30))
    g = torch.Generator(device="cuda").manual_seed(t + d + kind)
    x, y = (torch.empty(t, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    rows = torch.tensor(sorted({r for c in range(0, t + (1 << 20), 1 << 20) for r in range(c - 2, c + 3) if 0 <= r < t} | {t - 2, t - 1}), device="cuda")
    x[rows] = torch.randn(len(rows), d, generator=g, device="cuda").bfloat16()
    gam = (1 + 0.02 * torch.randn(d, generator=g, device="cuda")).bfloat16()
    bet = (0.02 * torch.randn(d, generator=g, device="cuda")).bfloat16()
    stats = torch.full((2, t), float("nan"), device="cuda")
    B.mllm_op_norm_fwd(kind, x, gam, bet if kind == 0 else None, y, stats, t, d, 1e-5)
    X = x[rows].double()
    mean = X.mean(1, keepdim=True) if kind == 0 else torch.zeros(len(rows), 1, dtype=torch.float64, device="cuda")
    r = torch.rsqrt(((X - mean) ** 2).mean(1, keepdim=True) + 1e-5)
    want = (X - mean) * r * gam.double() + (bet.double() if kind == 0 else 0.0)
    assert nmax_err(host_f64(y[rows]), want.cpu().numpy()) < 1e-2
    assert nmax_err(stats[0][rows].double().cpu().numpy(), r.flatten().cpu().numpy()) < 1e-5
    assert float((stats[1][rows].double() - mean.flatten()).abs().max()) < 1e-5
