"""The dK/dV pass walked in parts (few tokens, few kv heads), against the fp64 oracle at the stage tolerances:
parts that end inside a query head, more parts than a light key tile has query tiles, ragged and one-row
segments, with and without rotary gradient, both head widths."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import GpuStage, compare, oracle_run  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


CASES = {
    "gqa_128_one_sample": (W.decoder_layer(1024, 8, 1, 128, 256, 10000.0), [700], W.MASK_CAUSAL),
    "gqa_128_odd_group_ragged": (W.decoder_layer(896, 7, 1, 128, 256, 10000.0, qkv_bias=1), [641, 1, 130], W.MASK_CAUSAL),
    "gqa_64": (W.decoder_layer(512, 8, 2, 64, 256, 500000.0), [1000, 65], W.MASK_CAUSAL),
    "bidirectional_64": (W.vit_layer(128, 2, 64, 256), [1500], W.MASK_BIDIR),
    "bidirectional_128_qk_norm": (W.vit_layer(128, 1, 128, 256, qk_norm=1), [1025, 300], W.MASK_BIDIR),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_divided_key_pass_matches_oracle(B, name):
    layer, lengths, mask = CASES[name]
    pack = W.make_pack(lengths, mask)
    batch = W.Batch(pack, None, None, []) if mask == W.MASK_BIDIR else W.Batch(None, pack, None, [])
    wl = W.make_workload(name, [layer], batch, 331)
    st = GpuStage(B, [layer])
    try:
        got = st.run(wl)
        compare(st, wl, got, oracle_run(wl))
        again = st.run(wl)
        assert all(torch.equal(x, y) for x, y in zip(got[3], again[3]))
    finally:
        st.close()
