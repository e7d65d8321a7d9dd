"""Stage calls whose workspace holds less than mllm_stage_sizes says, against the fp64 oracle at the stage tolerances:
products and dK/dV passes in fewer parts or none, and nothing written past the end of the buffer."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import GpuStage, compare, dev_bf16, oracle_run, scratch  # noqa: E402
from tests.test_workspace_reuse import status  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


def least_workspace(B, st, batch, sb, wb):
    lo, hi = 0, wb
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if status(B, st.h, batch, (sb, mid), len(st.infos)) == 7: lo = mid
        else: hi = mid
    return hi


@pytest.mark.parametrize("share", [0.0, 0.4, 1.0])
@pytest.mark.parametrize("kind", ["decoder", "encoder"])
def test_less_scratch(B, kind, share):
    if kind == "decoder":
        layer, batch = W.decoder_layer(1024, 8, 1, 128, 4096, 10000.0, qkv_bias=1), W.Batch(None, W.make_pack([641, 1, 130], W.MASK_CAUSAL), None, [])
    else:
        layer, batch = W.vit_layer(1024, 16, 64, 4096), W.Batch(W.make_pack([577, 66], W.MASK_BIDIR), None, None, [])
    wl = W.make_workload(kind, [layer], batch, 351)
    st = GpuStage(B, [layer])
    try:
        sb, wb = B.mllm_stage_sizes(st.h, wl.batch)
        least = least_workspace(B, st, wl.batch, sb, wb)
        assert least < wb                                  # this microbatch does want scratch
        use = least + int(share * (wb - least))
        ws = torch.full((use + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
        saved, params, dy = scratch(sb), [dev_bf16(p) for p in wl.params], dev_bf16(wl.dy)
        x = dev_bf16(wl.x_img if kind == "encoder" else wl.x_seq)
        y, dx = torch.zeros_like(dy), torch.zeros_like(x)
        dparams = [torch.full((r, c), float("nan"), dtype=torch.float32, device="cuda") for _, _, r, c in st.infos]
        x_img, x_seq, dx_img, dx_seq = (x, None, dx, None) if kind == "encoder" else (None, x, None, dx)
        B.mllm_stage_fwd(st.h, wl.batch, params, x_img, x_seq, y, saved, ws, workspace_bytes=use)
        B.mllm_stage_bwd(st.h, wl.batch, params, dy, saved, dx_img, dx_seq, dparams, 0, ws, workspace_bytes=use)
        torch.cuda.synchronize()
        assert bool((ws[use:] == 0x5A).all())
        compare(st, wl, (y, dx_img, dx_seq, dparams), oracle_run(wl))
        if share == 1.0:                                   # exactly the size asked for: the same bits as with room to spare
            got = st.run(wl)
            assert torch.equal(got[0], y) and all(torch.equal(a, b) for a, b in zip(got[3], dparams))
    finally:
        st.close()
