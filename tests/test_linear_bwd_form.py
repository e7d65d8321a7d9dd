"""The plan of a linear map's two gradients in one launch (host logic, no GPU)."""
import pytest


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


WIDTHS = [(192, 576), (256, 2048), (1024, 1024), (1024, 4096), (4096, 1024), (1280, 3840), (3200, 9600), (4096, 4096), (4096, 28672), (18944, 3584)]


@pytest.mark.parametrize("k,n", WIDTHS)
def test_no_part_is_empty_and_the_parts_fit_the_scratch(B, k, n):
    """A part is a whole number of k-tiles, at least eight; both products' parts together stay inside the scratch that the
    plan was given, which is what the stage's workspace holds of it."""
    paired = 0
    for t in list(range(1, 1200, 131)) + [64, 576, 2880, 5125, 7488, 26496]:
        want = B.mllm_linear_bwd_form(t, k, n)[1]
        for scratch in (0, 4 * t * k, want // 2 // 4 * 4, max(want - 4, 0), want, 1 << 40):
            (one, x, w, first), _ = B.mllm_linear_bwd_form(t, k, n, scratch_bytes=scratch)
            used = 0
            for (rows, cols, parts), tiles, (m, c) in ((x, n // 64, (t, k)), (w, -(-t // 64), (k, n))):
                assert (rows, cols) in ((256, 256), (224, 256), (192, 256), (128, 128), (64, 64))
                per = -(-tiles // parts)
                assert (parts - 1) * per < tiles and (parts == 1 or per >= 8)
                used += parts * m * c * 4 if parts > 1 else 0
            assert w[0] not in (192, 224) and (not one or (x[0] == 64) == (w[0] == 64))
            assert (used if one else 0) <= scratch
            paired += one
        assert B.mllm_linear_bwd_form(t, k, n, scratch_bytes=want)[0] == B.mllm_linear_bwd_form(t, k, n)[0]
    assert paired > 20


# both gradients in quarters of 128x128 tiles up to 256 of them, in as many parts as the larger tiles
@pytest.mark.parametrize("t,k,n,tile,parts", [(64, 256, 2048, 64, 4), (288, 256, 2048, 64, 4), (577, 256, 2048, 128, 4), (576, 512, 512, 64, 1), (600, 512, 1472, 128, 1),
                                              (193, 3200, 9600, 224, 6), (225, 3200, 9600, 256, 6)])
def test_the_tile_of_the_input_gradient_that_runs_is_named(B, t, k, n, tile, parts):
    (one, x, w, _), _ = B.mllm_linear_bwd_form(t, k, n)
    assert one and (x[0], x[2]) == (tile, parts) and w[0] == (256 if tile > 128 else tile)


def test_what_the_tile_kernel_does_not_take_stays_apart(B):
    assert not B.mllm_linear_bwd_form(640, 136, 200)[0][0]       # dX contracts over 200 columns
    assert not B.mllm_linear_bwd_form(671050, 3200, 3200)[0][0]   # the last k-tile of dW would pass 4 GiB
    assert B.mllm_linear_bwd_form(0, 1024, 1024)[0][0] is False   # no tokens: dW is still written
    assert B.mllm_linear_bwd_form(777, 1024, 1024)[0][0]


def test_swiglu_form_keeps_the_tile_of_its_epilogue(B):
    for t in (777, 2999, 8192, 32768):
        (one, x, _, _), _ = B.mllm_linear_bwd_form(t, 18944, 3584, swiglu=1)
        assert one and x == (224 if t == 777 else 256, 256, 1)


@pytest.mark.parametrize("t,k,n", [(20000, 512, 520), (9000, 512, 712), (4000, 256, 72), (671050, 3200, 3200), (2880, 1024, 1024), (200, 4096, 8192)])
def test_scratch_wanted_is_enough_for_two_launches(B, t, k, n):
    """Maps whose gradients cannot share a launch (n no multiple of 64, or past 4 GiB) and maps whose operands may start off 16
    bytes: what the scratch is sized for is the form without a limit, one launch or two."""
    form, want = B.mllm_linear_bwd_form(t, k, n)
    assert B.mllm_linear_bwd_form(t, k, n, scratch_bytes=want)[0] == form
    for m, c, depth, al, bl in ((t, k, n, 0, 1), (k, n, t, 1, 0)):
        assert B.mllm_gemm_form(m, c, depth, al, bl, want) == B.mllm_gemm_form(m, c, depth, al, bl, 1 << 40)
