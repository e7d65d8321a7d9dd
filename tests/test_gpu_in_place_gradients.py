"""Gradients written in the place of inputs that are not needed any more, against the same call with buffers of their own.

bf16 probabilities and dS between the contractions on both sides: 3e-2 of the maximum, the stage tolerance of gradients."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import host_f64, nmax_err, scratch  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("what", ["dk dv", "dq", "dq dk dv"])
def test_attention_gradients_over_their_inputs(B, head_dim, causal, what):
    lengths, hq, hkv = [700, 65, 1], 6, 3
    T = sum(lengths)
    g = torch.Generator(device="cuda").manual_seed(T + head_dim + causal)
    q, o, do = (torch.randn(T, hq * head_dim, generator=g, device="cuda").bfloat16() for _ in range(3))
    k, v = (torch.randn(T, hkv * head_dim, generator=g, device="cuda").bfloat16() for _ in range(2))
    pack = W.make_pack(lengths, W.MASK_CAUSAL if causal else W.MASK_BIDIR)
    lse, delta = torch.empty(hq, T, device="cuda"), torch.empty(hq, T, device="cuda")
    ws = scratch(B.mllm_op_attn_workspace_bytes(len(lengths), T, hq))
    dims = (pack, hq, hkv, head_dim, hq * head_dim, hkv * head_dim, hq * head_dim, ws)
    B.mllm_op_attn_fwd(q, k, v, o, lse, *dims)
    own = [torch.full_like(t, float("nan")) for t in (q, k, v)]
    B.mllm_op_attn_bwd(q, k, v, o, lse, do, *own, delta, *dims)
    place = [torch.full_like(t, float("nan")) if n not in what else t.clone() for n, t in (("dq", o), ("dk", k), ("dv", v))]
    kin, vin = (place[1], place[2]) if "dk" in what else (k, v)
    B.mllm_op_attn_bwd(q, kin, vin, place[0] if "dq" in what else o, lse, do, *place, delta, *dims)
    for got, want in zip(place, own):
        assert nmax_err(host_f64(got), host_f64(want)) < 3e-2


@pytest.mark.parametrize("t,k,n", [(600, 1024, 192), (130, 256, 64), (2050, 640, 3200)])
def test_input_gradient_over_the_input(B, t, k, n):
    """Sizes whose gradients share a launch: dX over X makes two.  dX carries one bf16 rounding, dW is an fp32 sum (2e-3)."""
    (one, *_), want = B.mllm_linear_bwd_form(t, k, n)
    assert one
    g = torch.Generator(device="cuda").manual_seed(t + k + n)
    dy, x = (torch.randn(t, c, generator=g, device="cuda").bfloat16() for c in (n, k))
    w = (torch.randn(k, n, generator=g, device="cuda") * 0.125).bfloat16()
    want_dx, want_dw = dy.double() @ w.double().t().contiguous(), x.double().t().contiguous() @ dy.double()
    dw = torch.full((k, n), float("nan"), device="cuda")
    B.mllm_op_linear_bwd(dy, x, w, x, dw, t, k, n, workspace=scratch(want), scratch_bytes=want)
    assert nmax_err(host_f64(x), want_dx.cpu().numpy()) < 1e-2 and nmax_err(host_f64(dw), want_dw.cpu().numpy()) < 2e-3
