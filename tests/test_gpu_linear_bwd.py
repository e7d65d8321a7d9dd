"""Both gradients of a linear map in one launch, against float64 products of the same operands.

dX carries one bf16 rounding (2^-9 relative, and sums of at most n products in fp32: 1e-2 of the maximum), dW is an fp32
sum of bf16 products (2e-3)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import dev_bf16, host_f64, nmax_err  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


# tokens, k, n and the form that is meant: a tile each of dX and dW, alone and in parts, either one first
CASES = [(1, 64, 64, 64, 1, 64, 1), (77, 192, 576, 64, 1, 64, 1), (200, 256, 2048, 64, 4, 64, 1), (130, 520, 64, 64, 1, 64, 1), (577, 256, 2048, 128, 4, 128, 1),
         (2880, 1024, 1024, 128, 1, 128, 3), (200, 4096, 8192, 128, 4, 128, 1), (5125, 640, 3200, 128, 1, 128, 2),
         (1025, 3200, 3200, 128, 1, 128, 1), (5125, 3200, 3200, 192, 1, 256, 1), (6000, 3200, 1024, 256, 1, 128, 1),
         (9216, 1024, 1024, 256, 1, 256, None)]


def gradients(B, t, k, n, accumulate, scratch_bytes, seed):
    """(dX, dW) of the launch and their float64 references; the operands' rows past t hold large values."""
    dy, x = W.draw_tensor(seed, t + 64, n), W.draw_tensor(seed + 1, t + 64, k)
    dy[t:], x[t:] = 1000.0, 1000.0
    w = W.bf16_round(W.draw_tensor(seed + 2, k, n) * np.float32(0.125))
    init = np.random.default_rng(seed).standard_normal((k, n)).astype(np.float32)
    dev = [dev_bf16(v) for v in (dy, x, w)]
    want_dw = (dev[1][:t].double().t().contiguous() @ dev[0][:t].double()).cpu().numpy() + (init if accumulate else 0.0)
    want_dx = (dev[0][:t].double() @ dev[2].double().t().contiguous()).cpu().numpy()
    dx = torch.full((t + 3, k), 7.0, dtype=torch.bfloat16, device="cuda")
    dw = torch.from_numpy(init.copy()).cuda() if accumulate else torch.full((k, n), float("nan"), device="cuda")
    ws = torch.full((scratch_bytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    B.mllm_op_linear_bwd(dev[0], dev[1], dev[2], dx, dw, t, k, n, accumulate, workspace=ws, scratch_bytes=scratch_bytes)
    assert bool((ws[scratch_bytes:] == 0x5A).all()) and bool((dx[t:] == 7.0).all())
    return host_f64(dx[:t]), host_f64(dw), want_dx, want_dw


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("t,k,n,x_tile,x_parts,w_tile,w_parts", CASES)
def test_pair(B, t, k, n, x_tile, x_parts, w_tile, w_parts, accumulate):
    (one, x, w, _), want = B.mllm_linear_bwd_form(t, k, n)
    assert one
    assert all(a is None or a == b for a, b in ((x_tile, x[0]), (x_parts, x[2]), (w_tile, w[0]), (w_parts, w[2])))
    for scratch in (want, 0) if want else (0,):
        dx, dw, want_dx, want_dw = gradients(B, t, k, n, accumulate, scratch, 900 + t)
        assert nmax_err(dx, want_dx) < 1e-2 and nmax_err(dw, want_dw) < 2e-3


def test_pair_with_the_swiglu_gradient(B):
    t, f, n = 4200, 3080, 192
    assert B.mllm_linear_bwd_form(t, f, n, swiglu=1)[0][0]
    dy, w = W.draw_tensor(391, t, n), W.bf16_round(W.draw_tensor(392, f, n) * np.float32(0.125))
    pre, act = W.draw_tensor(393, t, 2 * f), W.draw_tensor(394, t, f)
    da = dy.astype(np.float64) @ w.astype(np.float64).T
    g, u = pre[:, :f].astype(np.float64), pre[:, f:].astype(np.float64)
    s = 1.0 / (1.0 + np.exp(-g))
    dpre = torch.full((t, 2 * f), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw = torch.full((f, n), float("nan"), device="cuda")
    B.mllm_op_linear_bwd(dev_bf16(dy), dev_bf16(act), dev_bf16(w), dpre, dw, t, f, n, swiglu_pre=dev_bf16(pre))
    assert nmax_err(host_f64(dpre), np.concatenate([da * u * s * (1.0 + g * (1.0 - s)), da * g * s], axis=1)) < 2e-2
    assert nmax_err(host_f64(dw), act.astype(np.float64).T @ dy.astype(np.float64)) < 2e-3


@pytest.mark.parametrize("oa,ob", [(1, 0), (0, 3)])
def test_operands_off_16_bytes_make_two_launches(B, oa, ob):
    t, k, n = 300, 520, 192
    flat = [torch.zeros(r * c + 8, dtype=torch.bfloat16, device="cuda") for r, c in ((t, n), (t, k), (k, n))]
    host = [W.draw_tensor(395 + i, r, c) for i, (r, c) in enumerate(((t, n), (t, k), (k, n)))]
    at = (oa, 0, ob)
    for f, h, o in zip(flat, host, at):
        f[o:o + h.size] = dev_bf16(h).flatten()
    dy, x, w = (f[o:o + h.size] for f, h, o in zip(flat, host, at))
    dx, dw = torch.empty(t, k, dtype=torch.bfloat16, device="cuda"), torch.empty(k, n, device="cuda")
    B.mllm_op_linear_bwd(dy, x, w, dx, dw, t, k, n)
    d64 = [h.astype(np.float64) for h in host]
    assert nmax_err(host_f64(dx), d64[0] @ d64[2].T) < 1e-2 and nmax_err(host_f64(dw), d64[1].T @ d64[0]) < 2e-3


# every kind of shared launch that the plan takes for the layers' widths: tokens, k, n; rows of dX's tiles and whether it is cut; the
# same of dW; whether dX's workgroups come first
FORMS = [(129, 5120, 1280, 128, 0, 256, 0, 1), (67, 1280, 5120, 128, 1, 256, 0, 1), (67, 1280, 1280, 128, 1, 128, 0, 1), (4099, 4096, 1024, 128, 0, 128, 0, 0),
         (963, 192, 192, 64, 0, 64, 1, 1), (996, 768, 192, 128, 0, 128, 1, 1), (2435, 1280, 1280, 192, 0, 128, 0, 1), (4099, 768, 192, 192, 0, 128, 1, 1), (513, 1280, 3840, 192, 1, 128, 0, 1),
         (1985, 5120, 1280, 192, 0, 256, 0, 0), (705, 5120, 1280, 192, 0, 256, 0, 1), (8099, 1280, 1280, 192, 0, 256, 1, 0), (4293, 1280, 1280, 192, 0, 256, 1, 1),
         (641, 2048, 2560, 192, 1, 256, 0, 1), (3397, 1280, 1280, 256, 0, 128, 0, 1), (6151, 1024, 1024, 256, 0, 128, 1, 1), (2883, 5120, 1280, 256, 0, 256, 0, 0),
         (1155, 5120, 1280, 256, 0, 256, 0, 1), (9263, 4096, 1024, 256, 0, 256, 1, 0), (7817, 1024, 1024, 256, 0, 256, 1, 1), (961, 1280, 3840, 256, 1, 128, 0, 1),
         (193, 3200, 9600, 224, 1, 256, 0, 1), (225, 3200, 9600, 256, 1, 256, 0, 1)]


@pytest.mark.parametrize("t,k,n,x_tile,x_cut,w_tile,w_cut,x_first", FORMS)
def test_every_form(B, t, k, n, x_tile, x_cut, w_tile, w_cut, x_first):
    """Accumulating and not; with the scratch that is wanted and with none (then uncut)."""
    (one, x, w, first), want = B.mllm_linear_bwd_form(t, k, n)
    assert one and (x[0], x[2] > 1, w[0], w[2] > 1, first) == (x_tile, bool(x_cut), w_tile, bool(w_cut), bool(x_first))
    g = torch.Generator(device="cuda").manual_seed(t + k + n)
    dy, act = (torch.randn(t + 64, c, generator=g, device="cuda").bfloat16() for c in (n, k))
    dy[t:], act[t:] = 1000.0, 1000.0
    weight = (torch.randn(k, n, generator=g, device="cuda") * 0.125).bfloat16()
    want_dx = dy[:t].double() @ weight.double().t().contiguous()
    want_dw = act[:t].double().t().contiguous() @ dy[:t].double()
    for accumulate, size in ((0, want), (1, want), (1, 0)):
        dx = torch.full((t + 3, k), 7.0, dtype=torch.bfloat16, device="cuda")
        dw = torch.full((k, n), 3.0 if accumulate else float("nan"), device="cuda")
        ws = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        B.mllm_op_linear_bwd(dy, act, weight, dx, dw, t, k, n, accumulate, workspace=ws, scratch_bytes=size)
        assert bool((ws[size:] == 0x5A).all()) and bool((dx[t:] == 7.0).all())
        assert float((dx[:t].double() - want_dx).abs().max() / want_dx.abs().max()) < 1e-2
        assert float((dw.double() - want_dw - 3.0 * accumulate).abs().max() / want_dw.abs().max()) < 2e-3


# with the SwiGLU gradient: dW in small and in large tiles, first and second
@pytest.mark.parametrize("t,f,n,w_tile,x_first", [(4200, 3080, 1024, 128, 1), (4200, 3080, 2048, 256, 0), (4200, 3080, 4096, 256, 1)])
def test_pair_with_the_swiglu_gradient_of_a_layer(B, t, f, n, w_tile, x_first):
    """bf16 gradients of the gate and up halves: 2e-2 of the maximum (dA stays in fp32, three factors and one rounding)."""
    (one, x, w, first), want = B.mllm_linear_bwd_form(t, f, n, swiglu=1)
    assert one and (x, w[0], first) == ((256, 256, 1), w_tile, bool(x_first))
    g = torch.Generator(device="cuda").manual_seed(n)
    dy, act, pre = (torch.randn(t, c, generator=g, device="cuda").bfloat16() for c in (n, f, 2 * f))
    weight = (torch.randn(f, n, generator=g, device="cuda") * 0.125).bfloat16()
    dpre = torch.full((t, 2 * f), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw = torch.full((f, n), float("nan"), device="cuda")
    ws = torch.empty(want + 256, dtype=torch.uint8, device="cuda")
    B.mllm_op_linear_bwd(dy, act, weight, dpre, dw, t, f, n, swiglu_pre=pre, workspace=ws, scratch_bytes=want)
    da, gate, up = dy.double() @ weight.double().t().contiguous(), pre[:, :f].double(), pre[:, f:].double()
    s = torch.sigmoid(gate)
    for got, ref in ((dpre[:, :f], da * up * s * (1.0 + gate * (1.0 - s))), (dpre[:, f:], da * gate * s)):
        assert float((got.double() - ref).abs().max() / ref.abs().max()) < 2e-2
    ref = act.double().t().contiguous() @ dy.double()
    assert float((dw.double() - ref).abs().max() / ref.abs().max()) < 2e-3
