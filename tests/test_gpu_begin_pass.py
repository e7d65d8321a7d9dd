"""What a pass begins with (metadata read from pinned host memory, rotary tables, the text rows) and the connector's gradient in one
launch: microbatches of different lengths through one handle and its ring of four slots, over and over, bit for bit as on their
first pass; input gradients of the sequence written over the incoming gradient, and not wanted at all."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import dev_bf16, scratch  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


def test_slots_of_the_ring_are_read_fresh(B):
    wls = [W.workload_tiny(s) for s in range(6)]
    layers = wls[0].layers
    h = B.mllm_stage_create(layers)
    try:
        sizes = [B.mllm_stage_sizes(h, w.batch) for w in wls]
        saved, ws = scratch(max(a for a, _ in sizes)), scratch(max(b for _, b in sizes))
        params = [dev_bf16(p) for p in wls[0].params]
        infos = [B.mllm_stage_param_info(h, i) for i in range(len(params))]
        first = {}
        for turn in range(60):
            i = (turn * 5 + turn // 7) % len(wls)
            w = wls[i]
            x_img, x_seq, dy = dev_bf16(w.x_img), dev_bf16(w.x_seq), dev_bf16(w.dy)
            y, dx_img, dx_seq = torch.zeros_like(dy), torch.zeros_like(x_img), torch.zeros_like(x_seq)
            dparams = [torch.empty(r, c, device="cuda") for _, _, r, c in infos]
            B.mllm_stage_fwd(h, w.batch, params, x_img, x_seq, y, saved, ws)
            B.mllm_stage_bwd(h, w.batch, params, dy, saved, dx_img, dx_seq, dparams, 0, ws)
            got = [y, dx_img, dx_seq] + dparams
            if i in first:
                assert all(torch.equal(a, b) for a, b in zip(first[i], got)), (turn, i)
            first.setdefault(i, got)
        assert len(first) == len(wls)
    finally:
        B.mllm_stage_destroy(h)


@pytest.mark.parametrize("wanted", ["apart", "in place", "none"])
def test_gradient_of_the_scattered_rows(B, wanted):
    """A connector on its own: its rows' gradient, and the others' as they came."""
    wl = W.workload_tiny(3)
    layers, batch = [wl.layers[1]], wl.batch
    d_in, d_out, T = layers[0].d_model, layers[0].d_out, int(batch.seq.cu_seqlens[-1])
    n = int(batch.img.cu_seqlens[-1])
    g = torch.Generator(device="cuda").manual_seed(5)
    w, b = (torch.randn(r, d_out, generator=g, device="cuda").bfloat16() * 0.05 for r in (d_in, 1))
    x_img, x_seq, dy = (torch.randn(r, c, generator=g, device="cuda").bfloat16() for r, c in ((n, d_in), (T, d_out), (T, d_out)))
    came, rows = dy.clone(), torch.from_numpy(batch.img_to_seq_row.astype("int64")).cuda()
    h = B.mllm_stage_create(layers)
    try:
        sb, wb = B.mllm_stage_sizes(h, batch)
        saved, ws, y = scratch(sb), scratch(wb), torch.empty_like(dy)
        B.mllm_stage_fwd(h, batch, [w, b], x_img, x_seq, y, saved, ws)
        want = x_seq.double().index_copy(0, rows, x_img.double() @ w.double() + b.double())
        assert float((y.double() - want).abs().max() / want.abs().max()) < 1e-2
        dx_img, dparams = torch.empty_like(x_img), [torch.empty(d_in, d_out, device="cuda"), torch.empty(1, d_out, device="cuda")]
        dx_seq = {"apart": torch.empty_like(dy), "in place": dy, "none": None}[wanted]
        B.mllm_stage_bwd(h, batch, [w, b], dy, saved, dx_img, dx_seq, dparams, 0, ws)
        rest = came.clone()
        rest[rows] = 0
        if dx_seq is not None:
            assert torch.equal(dx_seq, rest)
        dproj = came[rows].double()
        for got, ref, tol in ((dx_img, dproj @ w.double().t().contiguous(), 1e-2), (dparams[0], x_img.double().t().contiguous() @ dproj, 2e-3),
                              (dparams[1], dproj.sum(0, keepdim=True), 2e-3)):
            assert float((got.double() - ref).abs().max() / ref.abs().max()) < tol
    finally:
        B.mllm_stage_destroy(h)
