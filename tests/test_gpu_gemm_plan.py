"""The GEMM tile kernel where its tiles and its split K loop can go wrong, against the fp64 oracle.

Single products: bf16 results carry one rounding (2^-9 relative; 1e-2 of the maximum), fp32 results of bf16
products accumulated in fp32 2e-3.  Layers: the stage tolerances (2e-2 outputs, 3e-2 gradients)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.gpu_util import GpuStage, compare, dev_bf16, empty_bf16, host_f64, nmax_err, oracle_run  # noqa: E402


@pytest.fixture(scope="module")
def B():
    from paper_2603_25120_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("k", [1, 7, 63, 64, 65, 130, 193])
@pytest.mark.parametrize("m,n", [(8, 8), (136, 264), (640, 120), (1096, 1160)])
def test_weight_gradient_small_tiles_any_token_count(B, m, n, k):
    """128x128 tiles and quarters of them, both operands stored [K, .]: a last k-tile of any length, tile edges inside the matrix.  The
    rows behind the operands hold large values, so a row read past K would show."""
    a, b = W.draw_tensor(301, k + 64, m), W.draw_tensor(302, k + 64, n)
    a[k:], b[k:] = 1000.0, 1000.0
    ref = a[:k].T.astype(np.float64) @ b[:k].astype(np.float64)
    a_dev, b_dev = dev_bf16(a), dev_bf16(b)
    init = np.random.default_rng(303).standard_normal((m, n)).astype(np.float32)
    c = torch.from_numpy(init.copy()).cuda()
    B.mllm_op_gemm(a_dev, b_dev, c, m, n, k, 1, 0, out_fp32=1, accumulate=1)
    assert nmax_err(host_f64(c), ref + init) < 2e-3
    c = empty_bf16(m, n)
    B.mllm_op_gemm(a_dev, b_dev, c, m, n, k, 1, 0)
    assert nmax_err(host_f64(c), ref) < 1e-2


@pytest.mark.parametrize("m,n,k", [(1, 8, 64), (127, 136, 128), (129, 120, 192), (513, 264, 320), (1025, 1032, 320), (1151, 1160, 192)])
@pytest.mark.parametrize("b_layout,f32", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_small_tiles_edges_and_epilogue_terms(B, m, n, k, b_layout, f32):
    a = W.draw_tensor(311, m, k)
    b = W.bf16_round(W.draw_tensor(312, k, n) * np.float32(0.125))
    ref = a.astype(np.float64) @ b.astype(np.float64)
    bias = W.draw_tensor(313, 1, n)
    b_dev = dev_bf16(np.ascontiguousarray(b.T) if b_layout else b)
    # guard rows behind C: nothing past the last row may be written
    c = torch.full((m + 3, n), 7.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
    if f32:
        B.mllm_op_gemm(dev_bf16(a), b_dev, c, m, n, k, 0, b_layout, out_fp32=1, bias=dev_bf16(bias))
        want = ref + bias
    else:
        res = W.draw_tensor(314, m, n)
        B.mllm_op_gemm(dev_bf16(a), b_dev, c, m, n, k, 0, b_layout, bias=dev_bf16(bias), residual=dev_bf16(res))
        want = ref + bias + res
    got = host_f64(c)
    assert nmax_err(got[:m], want) < (2e-3 if f32 else 1e-2)
    assert np.all(got[m:] == 7.0)


# sizes that take a tile with one, two, an odd and an even number of k-tiles alike
TILES = [(256, 2216, 5536, 0, 0), (256, 2216, 5536, 0, 1), (256, 704, 20944, 1, 0), (256, 704, 20944, 1, 1),
         (192, 5960, 1312, 0, 0), (192, 5960, 1312, 0, 1),
         (224, 896, 14000, 0, 0), (224, 896, 14000, 0, 1), (224, 1343, 9840, 0, 0),
         (128, 1096, 1160, 0, 0), (128, 1096, 1160, 0, 1), (128, 1096, 1160, 1, 0), (128, 200, 520, 1, 1),
         (64, 200, 520, 0, 0), (64, 200, 520, 0, 1), (64, 200, 520, 1, 0)]


@pytest.mark.parametrize("k", [64, 128, 192, 320])
@pytest.mark.parametrize("f32", [0, 1])
@pytest.mark.parametrize("tile,m,n,a_layout,b_layout", TILES)
def test_every_tile_with_few_k_tiles(B, tile, m, n, a_layout, b_layout, f32, k):
    """Ragged M and N, every layout and output type of a tile, all epilogue terms."""
    assert B.mllm_gemm_form(m, n, k, a_layout, b_layout)[0] == tile
    a = W.draw_tensor(361, m, k)
    b = W.bf16_round(W.draw_tensor(362, k, n) * np.float32(0.125))
    ref = a.astype(np.float64) @ b.astype(np.float64)
    bias = W.draw_tensor(363, 1, n)
    a_dev, b_dev = (dev_bf16(np.ascontiguousarray(t.T) if turned else t) for t, turned in ((a, a_layout), (b, b_layout)))
    if f32:
        init = np.random.default_rng(364).standard_normal((m, n)).astype(np.float32)
        c = torch.from_numpy(init.copy()).cuda()
        B.mllm_op_gemm(a_dev, b_dev, c, m, n, k, a_layout, b_layout, out_fp32=1, accumulate=1, bias=dev_bf16(bias))
        assert nmax_err(host_f64(c), ref + bias + init) < 2e-3
    else:
        res = W.draw_tensor(365, m, n)
        c = empty_bf16(m, n)
        B.mllm_op_gemm(a_dev, b_dev, c, m, n, k, a_layout, b_layout, bias=dev_bf16(bias), residual=dev_bf16(res))
        assert nmax_err(host_f64(c), ref + bias + res) < 1e-2
        B.mllm_op_gemm(a_dev, b_dev, c, m, n, k, a_layout, b_layout)
        assert nmax_err(host_f64(c), ref) < 1e-2


@pytest.mark.parametrize("k", [1, 63, 65, 130, 193])
@pytest.mark.parametrize("f32", [0, 1])
def test_weight_gradient_large_tiles_short_ragged_contraction(B, k, f32):
    """256x256 tiles whose last k-tile is partial, also the only one; the rows behind the operands hold large values."""
    m, n = 704, 20944
    assert B.mllm_gemm_form(m, n, k, 1, 0)[0] == 256
    a, b = W.draw_tensor(371, k + 64, m), W.draw_tensor(372, k + 64, n)
    a[k:], b[k:] = 1000.0, 1000.0
    ref = a[:k].T.astype(np.float64) @ b[:k].astype(np.float64)
    c = torch.full((m, n), float("nan"), dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
    B.mllm_op_gemm(dev_bf16(a), dev_bf16(b), c, m, n, k, 1, 0, out_fp32=f32)
    assert nmax_err(host_f64(c), ref) < (2e-3 if f32 else 1e-2)


SCRATCH = 1 << 40   # more than any product wants


@pytest.mark.parametrize("lengths", [[5], [77, 130], [300, 1, 64]])
def test_layers_whose_products_split_the_k_loop(B, lengths):
    """A few tokens against wide matrices: products with too few tiles to fill the chip go through partial products, the
    down projection forward (bias, residual) and the input gradients of the up and QKV projections among them.  (The
    weight gradients here contract over too few tokens to be cut; the test below has some.)"""
    T = sum(lengths)
    assert B.mllm_gemm_form(T, 1024, 4096, 0, 1, SCRATCH)[2] > 1 and B.mllm_gemm_form(T, 1024, 3072, 0, 1, SCRATCH)[2] > 1
    assert B.mllm_gemm_form(T, 1024, 4096, 0, 0, SCRATCH)[2] > 1                # the down projection: bias, residual
    assert B.mllm_gemm_form(4096, 1024, T, 1, 0, SCRATCH)[2] == 1
    for layer, pack in ((W.vit_layer(1024, 16, 64, 4096), "img"), (W.decoder_layer(1024, 8, 2, 128, 4096, 10000.0, qkv_bias=1), "seq")):
        p = W.make_pack(lengths, W.MASK_BIDIR if pack == "img" else W.MASK_CAUSAL)
        batch = W.Batch(p, None, None, []) if pack == "img" else W.Batch(None, p, None, [])
        wl = W.make_workload("split", [layer], batch, 321)
        st = GpuStage(B, [layer])
        try:
            got, ref = st.run(wl), oracle_run(wl)
            compare(st, wl, got, ref)
            again = st.run(wl)
            assert all(torch.equal(x, y) for x, y in zip(got[3], again[3])) and torch.equal(got[0], again[0])
        finally:
            st.close()


@pytest.mark.parametrize("d_in,d_out,images,img_tokens,tile,parts", [(512, 1024, 19, 79, 128, 3), (2048, 2560, 5, 1025, 256, 3)])
def test_split_weight_gradient_over_ragged_tokens_accumulates(B, d_in, d_out, images, img_tokens, tile, parts):
    """A connector's weight gradient in parts, the last of which ends in a partial k-tile, added to what is there."""
    T = images * img_tokens
    assert T % 64 and B.mllm_gemm_form(d_in, d_out, T, 1, 0, SCRATCH) == (tile, tile, parts)
    layers = [W.projector_layer(d_in, d_out)]
    wl = W.make_workload("split_dw", layers, W.batch_from_samples([(1, 3)] * images, img_tokens=img_tokens), 331)
    st = GpuStage(B, layers)
    try:
        ref = oracle_run(wl)
        scale = float(np.max(np.abs(ref[3][0])))
        rng = np.random.default_rng(332)
        init = [(rng.standard_normal((r, c)) * scale).astype(np.float32) for _, _, r, c in st.infos]
        dparams = [torch.from_numpy(t.copy()).cuda() for t in init]
        got = st.run(wl, accumulate=1, dparams=dparams)
        compare(st, wl, got, (*ref[:3], [g + t for g, t in zip(ref[3], init)]))
        assert nmax_err(host_f64(dparams[0]), ref[3][0] + init[0]) < 2e-3      # fp32 sums of bf16 products
    finally:
        st.close()


def test_ragged_contraction_close_to_4_gib(B):
    """Both operands are 247 KB short of 4 GiB with a partial last k-tile: 32-bit offsets of the rows past
    K would come round to the first rows, which are the only non-zero ones here besides the last."""
    k, w, head, tail = 671050, 3200, 64, 10
    a, b = (torch.zeros(k, w, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    ref = 0.0
    for t, seed in ((a, 341), (b, 342)):
        rows = W.draw_tensor(seed, head + tail, w)
        t[:head], t[k - tail:] = dev_bf16(rows[:head]), dev_bf16(rows[head:])
        ref = rows.T.astype(np.float64) if t is a else ref @ rows.astype(np.float64)
    c = torch.empty(w, w, dtype=torch.float32, device="cuda")
    B.mllm_op_gemm(a, b, c, w, w, k, 1, 0, out_fp32=1)
    assert nmax_err(host_f64(c), ref) < 2e-3


def placed(x, offset):
    """The values of x in a contiguous device tensor that starts `offset` elements into its allocation."""
    flat = torch.zeros(x.size + offset, dtype=torch.bfloat16, device="cuda")
    flat[offset:] = dev_bf16(x).flatten()
    return flat[offset:].view(x.shape)


@pytest.mark.parametrize("oa,ob", [(1, 0), (0, 1), (3, 6), (8, 4), (0, 0)])
@pytest.mark.parametrize("m,n,k,a_layout,b_layout", [(2216, 5536, 192, 0, 1), (5960, 1312, 128, 0, 1), (264, 328, 192, 0, 1),
                                                     (2216, 5536, 192, 0, 0), (704, 20944, 130, 1, 0)])
def test_operands_anywhere_in_a_buffer(B, m, n, k, a_layout, b_layout, oa, ob):
    """Tensors that start at any element of a larger buffer, results included; nothing beside the result is written."""
    a = W.draw_tensor(381, m, k)
    b = W.bf16_round(W.draw_tensor(382, k, n) * np.float32(0.125))
    ref = a.astype(np.float64) @ b.astype(np.float64)
    a_dev, b_dev = (placed(np.ascontiguousarray(t.T) if turned else t, o) for t, turned, o in ((a, a_layout, oa), (b, b_layout, ob)))
    c = torch.full((m * n + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    at = 1 + oa
    B.mllm_op_gemm(a_dev, b_dev, c[at:at + m * n], m, n, k, a_layout, b_layout)
    assert nmax_err(host_f64(c[at:at + m * n]).reshape(m, n), ref) < 1e-2
    assert bool((c[:at] == 7.0).all()) and bool((c[at + m * n:] == 7.0).all())


@pytest.mark.parametrize("oa,ob", [(1, 0), (0, 5)])
def test_swiglu_gradient_of_operands_anywhere_in_a_buffer(B, oa, ob):
    m, f, k = 4200, 3080, 192
    dy, w = W.draw_tensor(391, m, k), W.bf16_round(W.draw_tensor(392, f, k) * np.float32(0.125))
    pre = W.draw_tensor(393, m, 2 * f)
    da = dy.astype(np.float64) @ w.astype(np.float64).T
    g, u = pre[:, :f].astype(np.float64), pre[:, f:].astype(np.float64)
    s = 1.0 / (1.0 + np.exp(-g))
    dpre = torch.full((m, 2 * f), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.mllm_op_gemm_swiglu_bwd(placed(dy, oa), placed(w, ob), dev_bf16(pre), dpre, m, f, k)
    assert nmax_err(host_f64(dpre), np.concatenate([da * u * s * (1.0 + g * (1.0 - s)), da * g * s], axis=1)) < 2e-2
