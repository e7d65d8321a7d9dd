"""Attention forward and backward at the edges of their blocks, for both head widths: segments of one row, of 16- and 32-row groups
and key tiles plus or minus one, wavefronts without a row, one key tile, an odd and an even number of them, parts of the dK/dV
pass; and scores that grow from key tile to key tile, so that the forward pass has to move its reference, within the range of fp32
and by more than that.  Against float64 attention: probabilities and dS are rounded to bf16 between the contractions (the stage
tolerances); lse is a sum in fp32 of at most 1025 exponentials whose arguments carry 2^-24 of at most 600 (2e-5 of its maximum)."""
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


def reference(q, k, v, do, lengths, causal, grp, hd):
    outs, lses, grads, at = [], [], [torch.zeros_like(t) for t in (q, k, v)], 0
    for n in lengths:
        part = [t[at:at + n].clone().requires_grad_() for t in (q, k, v)]
        kk, vv = (t.repeat_interleave(grp, dim=1) for t in part[1:])
        s = torch.einsum("qhd,khd->hqk", part[0], kk) / hd ** 0.5
        if causal:
            s = s.masked_fill(torch.ones(n, n, dtype=torch.bool, device=s.device).triu(1), float("-inf"))
        o = torch.einsum("hqk,khd->qhd", torch.softmax(s, dim=2), vv)
        o.backward(do[at:at + n])
        outs.append(o.detach())
        lses.append(torch.logsumexp(s, dim=2).detach())
        for g, t in zip(grads, part):
            g[at:at + n] = t.grad
        at += n
    return torch.cat(outs), torch.cat(lses, dim=1), grads


def run(B, lengths, hq, hkv, hd, causal, growth=None):
    T = sum(lengths)
    g = torch.Generator(device="cuda").manual_seed(T * hq + hd)
    qkv = torch.randn(T, (hq + 2 * hkv) * hd, generator=g, device="cuda")
    if growth:   # keys scaled by the key tile they fall into
        tile = torch.cat([torch.arange(n, device="cuda") // 64 for n in lengths])
        qkv[:, hq * hd:(hq + hkv) * hd] *= torch.tensor(growth, device="cuda")[tile.clamp(max=len(growth) - 1)][:, None]
    qkv = qkv.bfloat16()
    do = torch.randn(T, hq * hd, generator=g, device="cuda").bfloat16()
    pack = W.make_pack(lengths, W.MASK_CAUSAL if causal else W.MASK_BIDIR)
    o, dqkv = torch.empty_like(do), torch.full_like(qkv, float("nan"))
    lse, delta = torch.empty(hq, T, device="cuda"), torch.empty(hq, T, device="cuda")
    ws = scratch(B.mllm_op_attn_workspace_bytes(len(lengths), T, hq))
    width, at = (hq + 2 * hkv) * hd, [0, 2 * hq * hd, 2 * (hq + hkv) * hd]
    q, k, v = (qkv.data_ptr() + a for a in at)
    B.mllm_op_attn_fwd(q, k, v, o, lse, pack, hq, hkv, hd, width, width, hq * hd, ws)
    B.mllm_op_attn_bwd(q, k, v, o, lse, do, *(dqkv.data_ptr() + a for a in at), delta, pack, hq, hkv, hd, width, width, hq * hd, ws)
    Q, K, V = (t.double().reshape(T, -1, hd) for t in qkv.split([hq * hd, hkv * hd, hkv * hd], dim=1))
    ref, ref_lse, grads = reference(Q, K, V, do.double().reshape(T, hq, hd), lengths, causal, hq // hkv, hd)
    assert nmax_err(host_f64(o), ref.reshape(T, -1).cpu().numpy()) < 2e-2
    assert nmax_err(host_f64(lse), ref_lse.cpu().numpy()) < 2e-5
    for got, want in zip(dqkv.split([hq * hd, hkv * hd, hkv * hd], dim=1), grads):
        assert nmax_err(host_f64(got.contiguous()), want.reshape(T, -1).cpu().numpy()) < 3e-2


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("lengths,hq,hkv", [([1, 15, 16, 17], 2, 2), ([31, 32, 33, 63], 2, 1), ([64, 65, 95, 97], 4, 2), ([127, 128, 129], 2, 2),
                                            ([161, 193], 3, 1), ([320, 257], 5, 5), ([1025], 4, 1)])
def test_edges(B, lengths, hq, hkv, causal, hd):
    run(B, lengths, hq, hkv, hd, causal)


def forward_us(B, hd, higher):
    """Median time of a forward pass whose keys behind the first tile of each segment score `higher` nats more."""
    n, segments, heads = 1500, 4, 16
    T, g = n * segments, torch.Generator(device="cuda").manual_seed(hd)
    q, k, v = (torch.randn(T, heads, hd, generator=g, device="cuda") * s for s in (1.0, 0.2, 1.0))
    q[:, :, 0] = hd ** 0.5
    k[:, :, 0] = (torch.arange(T, device="cuda") % n >= 64).float()[:, None] * higher
    q, k, v = (t.bfloat16().reshape(T, -1) for t in (q, k, v))
    o, lse, w = torch.empty_like(q), torch.empty(heads, T, device="cuda"), heads * hd
    pack, ws = W.make_pack([n] * segments, W.MASK_BIDIR), scratch(B.mllm_op_attn_workspace_bytes(segments, T, heads))
    times = []
    for _ in range(12):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(30):
            B.mllm_op_attn_fwd(q, k, v, o, lse, pack, heads, heads, hd, w, w, w, ws)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return sorted(times[2:])[5]


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("higher", [2.5, 4.0])
def test_keys_within_the_reference_cost_no_more(B, higher, hd):
    """Below 2^8 of the reference no tile is formed again, whatever its sum.  1.5 times the time where the sum alone decided."""
    assert forward_us(B, hd, higher) < 1.2 * forward_us(B, hd, 0.0)


# times 1, 8 and 64 at unit variance: scores of about 4, 35 and 270 (390 in units of log2); falling again, the reference stays
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("growth", [[1, 8], [1, 8, 64], [1, 1, 64, 1], [64, 1, 64, 1], [0, 0, 64]])
def test_scores_that_grow(B, growth, causal, hd):
    run(B, [300, 65, 130], 4, 2, hd, causal, growth)
