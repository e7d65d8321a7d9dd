"""The sums over the tokens (norm and bias gradients) of a backward pass are finished by one launch for several
layers: more sums than the list holds, scratch that fills up, and layers that share gradient buffers."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import GpuStage, host_f64  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


# 9 layers hold 8 sums each (the list holds 32); 3000 tokens 1024 and 8192 wide fills the scratch between two layers
@pytest.mark.parametrize("layers,d,ff,tokens", [(2, 128, 256, [5]), (9, 128, 256, [70, 1, 33]), (3, 1024, 8192, [3000])])
def test_shared_gradients_get_the_sum(B, layers, d, ff, tokens):
    batch = W.Batch(W.make_pack(tokens, W.MASK_BIDIR), None, None, [])
    wl = W.make_workload("shared", [W.vit_layer(d, d // 64, 64, ff) for _ in range(layers)], batch, 5)
    st = GpuStage(B, wl.layers)
    try:
        own = st.run(wl)[3]
        per = len(own) // layers
        shared = [torch.zeros_like(g) for g in own[:per]] * layers
        st.run(wl, accumulate=1, dparams=shared)
        for j in range(per):
            ref = np.sum([host_f64(own[i * per + j]) for i in range(layers)], axis=0)
            # a layer adds its gradient in one fp32 addition, a weight's in up to 17 (16 parts of a split K loop)
            mag = np.max(np.sum([np.abs(host_f64(own[i * per + j])) for i in range(layers)], axis=0))
            assert np.max(np.abs(host_f64(shared[j]) - ref)) <= 17 * layers * 2.0 ** -23 * mag
    finally:
        st.close()
