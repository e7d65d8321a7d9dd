"""Buffers sized for the longest microbatch serve every shorter one (host only: calls are refused or pass their
buffer checks before anything is launched)."""
import pytest

import workloads as W


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


STACKS = {
    "dec8b": ([W.dec8b_layer()], W.MASK_CAUSAL),
    "dec_qkv_bias": ([W.decoder_layer(3584, 28, 4, 128, 18944, 1000000.0, qkv_bias=1)], W.MASK_CAUSAL),
    "dec7b": ([W.dec7b_layer()], W.MASK_CAUSAL),
    "vit_l": ([W.vit_l_layer()] * 2, W.MASK_BIDIR),
    "internvit": ([W.vit_layer(3200, 25, 128, 12800, qk_norm=1)], W.MASK_BIDIR),
}


def one_segment(tokens, mask):
    pack = W.make_pack([tokens], mask)
    return W.Batch(pack, None, None, []) if mask == W.MASK_BIDIR else W.Batch(None, pack, None, [])


def status(B, h, batch, sizes, n):
    """Status of a forward call whose buffers pass (1: the input is NULL) or are too small (7)."""
    with pytest.raises(B.MllmError) as e:
        B.mllm_stage_fwd(h, batch, [4096] * n, None, None, 4096, 4096, 4096, stream=1, saved_bytes=sizes[0], workspace_bytes=sizes[1])
    return e.value.status


@pytest.mark.parametrize("name", sorted(STACKS))
def test_buffers_of_a_longer_microbatch_are_accepted(B, name):
    layers, mask = STACKS[name]
    h = B.mllm_stage_create(layers)
    n = B.mllm_stage_param_count(h)
    try:
        tokens = list(range(64, 3000, 97)) + list(range(3000, 16000, 391))
        sizes = [B.mllm_stage_sizes(h, one_segment(t, mask)) for t in tokens]
        for i, t in enumerate(tokens):
            batch = one_segment(t, mask)
            # every later size: the smallest of them decides
            least = (min(s[0] for s in sizes[i:]), min(s[1] for s in sizes[i:]))
            assert status(B, h, batch, least, n) == 1, t
            assert status(B, h, batch, (sizes[i][0] - 1, sizes[i][1]), n) == 7
            assert status(B, h, batch, (sizes[i][0], 4096), n) == 7
    finally:
        B.mllm_stage_destroy(h)


def test_scratch_decides_the_parts_of_a_product(B):
    """The most parts that fit, none without scratch; more scratch than wanted changes nothing."""
    m, n, k = 1232, 1024, 28672
    tr, tc, want = B.mllm_gemm_form(m, n, k, scratch_bytes=1 << 40)
    assert want > 1
    one = m * n * 4
    assert B.mllm_gemm_form(m, n, k, scratch_bytes=want * one) == (tr, tc, want)
    assert B.mllm_gemm_form(m, n, k, scratch_bytes=want * one - 1)[2] < want
    assert B.mllm_gemm_form(m, n, k, scratch_bytes=one)[2] == 1 and B.mllm_gemm_form(m, n, k)[2] == 1
