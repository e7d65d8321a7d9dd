"""Backward attention at head_dim 64 in one launch and in two, against float64 attention: probabilities and dS are rounded to
bf16 between the contractions (3e-2 of the maximum, the stage tolerance of gradients)."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import nmax_err, host_f64, scratch  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


def reference(q, k, v, do, lengths, causal, grp):
    outs, grads = [], [torch.zeros_like(t) for t in (q, k, v)]
    at = 0
    for n in lengths:
        part = [t[at:at + n].clone().requires_grad_() for t in (q, k, v)]
        kk, vv = (t.repeat_interleave(grp, dim=1) for t in part[1:])
        s = torch.einsum("qhd,khd->hqk", part[0], kk) / 8.0
        if causal:
            s = s.masked_fill(torch.ones(n, n, dtype=torch.bool, device=s.device).triu(1), float("-inf"))
        o = torch.einsum("hqk,khd->qhd", torch.softmax(s, dim=2), vv)
        o.backward(do[at:at + n])
        outs.append(o.detach())
        for g, t in zip(grads, part):
            g[at:at + n] = t.grad
        at += n
    return torch.cat(outs), grads


# (the last two: more workgroups than one launch takes)
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("lengths,hq,hkv", [([1], 1, 1), ([63, 64, 65], 4, 2), ([127, 1, 130], 3, 3), ([577], 16, 16), ([200, 3], 8, 1),
                                            ([40] * 52, 32, 32), ([129] * 13, 64, 64)])
def test_backward(B, lengths, hq, hkv, causal):
    T, hd = sum(lengths), 64
    g = torch.Generator(device="cuda").manual_seed(T + hq)
    qkv = torch.randn(T, (hq + 2 * hkv) * hd, generator=g, device="cuda").bfloat16()
    do = torch.randn(T, hq * hd, generator=g, device="cuda").bfloat16()
    pack = W.make_pack(lengths, W.MASK_CAUSAL if causal else W.MASK_BIDIR)
    o, dqkv = torch.empty_like(do), torch.full_like(qkv, float("nan"))
    lse, delta = torch.empty(hq, T, device="cuda"), torch.full((hq, T), float("nan"), device="cuda")
    ws = scratch(B.mllm_op_attn_workspace_bytes(len(lengths), T, hq))
    width, at = (hq + 2 * hkv) * hd, [0, 2 * hq * hd, 2 * (hq + hkv) * hd]
    q, k, v = (qkv.data_ptr() + a for a in at)
    B.mllm_op_attn_fwd(q, k, v, o, lse, pack, hq, hkv, hd, width, width, hq * hd, ws)
    B.mllm_op_attn_bwd(q, k, v, o, lse, do, *(dqkv.data_ptr() + a for a in at), delta, pack, hq, hkv, hd, width, width, hq * hd, ws)
    Q, K, V = (t.double().reshape(T, -1, hd) for t in qkv.split([hq * hd, hkv * hd, hkv * hd], dim=1))
    ref, grads = reference(Q, K, V, do.double().reshape(T, hq, hd), lengths, causal, hq // hkv)
    assert nmax_err(host_f64(o), ref.reshape(T, -1).cpu().numpy()) < 2e-2
    for got, want in zip(dqkv.split([hq * hd, hkv * hd, hkv * hd], dim=1), grads):
        assert nmax_err(host_f64(got.contiguous()), want.reshape(T, -1).cpu().numpy()) < 3e-2
    assert nmax_err(host_f64(delta), (ref * do.double().reshape(T, hq, hd)).sum(2).t().cpu().numpy()) < 2e-2
