"""Kernels against the oracle at the sizes where they can go wrong: edges of tiles, remainders, ends of their ranges."""
import pytest

pytestmark = pytest.mark.gpu

import oracle as O
import workloads as W
from oracle import graph as OG
from helpers import assert_close, error_budget, run_hip


def steps_of(spec, opts=None):
    from paper_1810_00952_amd import binding
    return [st["kernel"] for st in binding.Plan(binding.graph_from_spec(binding.Context(), spec), opts).describe()["steps"]]


def check(spec, data, dtype, what, opts=None):
    # where the plan has a contraction without LDS tiles, the kernels with them are held to the same
    steps = steps_of(spec, opts)
    print(what, steps, flush=True)
    ref = OG.run(spec, data)
    forms = [opts]
    if not (opts or {}).get("no_direct") and any("_direct" in k and "stem" not in k for k in steps):
        forms.append(dict(opts or {}, no_direct=1, direct_all=0))
    for form in forms:
        got, _ = run_hip(spec, data, opts=form)
        for v in spec.outputs:
            dt = spec.values[v].type.dtype
            assert_close(got[v], ref[v], dt, f"{what} {form}", budget=(lambda: error_budget(spec, data)[v]) if dt == "f32" else None)


# ---- weight gradients that contract over the rows of both operands (igemm_tn.hip) ---------------------------------------
ROWS_CASES = [
    # kind           dims                        stride pad
    ("dense_grad_w", (512, 1000, 784), 1, 0),            # 64 x 64 tiles, ragged last ones, one slice
    ("dense_grad_w", (20, 192, 1536), 1, 0),             # fewer rows than a K tile
    ("dense_grad_w", (4099, 72, 40), 1, 0),              # long and narrow: slices, a last K tile of three rows
    ("dense_grad_w", (167, 391, 173), 1, 0),             # both feature counts padded to whole vectors
    ("conv2d_grad_w", (5, 64, 31, 30, 64, 3), 1, 1),     # odd batch, taps outside the image, slices
    ("conv2d_grad_w", (6, 40, 33, 29, 72, 3), 2, 1),     # stride 2: (H + 2p - K) % s = 0 for both; tiles that span taps
    ("conv2d_grad_w", (2, 93, 20, 19, 36, 5), 1, 2),     # 25 taps, x padded to whole vectors
    ("conv2d_grad_w", (7, 128, 24, 26, 136, 1), 1, 0),   # 1x1: rows as they lie
    ("conv2d_grad_w", (12, 128, 23, 21, 200, 1), 2, 0),   # the strided projection
    ("conv2d_grad_w", (1, 512, 7, 7, 512, 3), 1, 1),     # one K tile and a remainder, many tiles: no slices
    ("conv2d_grad_w", (40, 128, 36, 1, 72, 3), 1, 1),    # rows of one pixel
    ("dense_grad_w", (4, 16384, 8192), 1, 0),            # as many results as partial sums may be: one slice
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", ROWS_CASES, ids=[f"rows{i}" for i in range(len(ROWS_CASES))])
def test_weight_gradient_over_rows(dtype, case):
    kind, dims, stride, pad = case
    for out_dtype in (None, "f32") if dtype == "bf16" else (None,):
        spec, data = W.grad_case(kind, dims, dtype, stride, pad, second_is_param=False, out_dtype=out_dtype)
        assert any("_rows" in k for k in steps_of(spec)), steps_of(spec)
        check(spec, data, dtype, f"rows {case} {dtype} {out_dtype}")


def test_weight_gradient_over_rows_beside_the_input_gradient():
    # a batch of 64 in bf16, both gradients in one graph: dy is held channel-last for the first, so the second takes the rows;
    # 128 x 128 tiles on both sides
    import numpy as np
    for dtype, n in (("bf16", 64), ("f32", 5)):
        rng = np.random.default_rng(7)
        g = W.GraphSpec("layer_backward")
        dy = g.input("dy", dtype, (n, 128, 17, 16)); w = g.param("w", dtype, (128, 192, 3, 3)); x = g.input("x", dtype, (n, 192, 17, 16))
        at = dict(stride=(1, 1), pad=(1, 1))
        o, (dx,) = g.op("conv2d_grad_x", [dy, w], [(dtype, (n, 192, 17, 16))], **at); g.group([o])
        o, (dw,) = g.op("conv2d_grad_w", [dy, x], [("f32", (128, 192, 3, 3))], out_dtype="f32", **at); g.group([o])
        g.output(dx); g.output(dw)
        data = {"dy": W.as_dtype(rng.standard_normal((n, 128, 17, 16)), dtype), "x": W.as_dtype(rng.standard_normal((n, 192, 17, 16)), dtype),
                "w": W.as_dtype(rng.standard_normal((128, 192, 3, 3)) / 40, dtype)}
        assert any("_rows" in k for k in steps_of(g)), steps_of(g)
        check(g, data, dtype, f"layer backward {dtype}")
        first, _ = run_hip(g, data)
        again, _ = run_hip(g, data)
        np.testing.assert_array_equal(first[dw], again[dw])           # slices are added in a fixed order


# ---- contractions whose K tiles span filter taps, padded channels, results in Shape order (igemm_dma.hip) ------------------
TAPS_CASES = [
    # batch cin cout h  w  k s p residual relu acts tail
    (17, 96, 136, 29, 29, 3, 1, 1, True, True, (), False),       # tiles across taps, ragged N, images of 841 pixels (one-pixel stores)
    (3, 8, 24, 20, 22, 3, 1, 1, True, False, (), False),         # eight taps per bf16 K tile; four-pixel stores
    (2, 24, 40, 17, 16, 7, 2, 3, False, True, (), False),        # 49 taps
    (40, 5, 12, 33, 31, 3, 1, 1, False, True, (), False),         # channels padded to whole vectors
    (60, 1, 20, 28, 28, 5, 1, 0, False, False, ("tanh",), False), # one channel; tanh in the pixel-order store
    (60, 1, 20, 28, 28, 5, 1, 0, False, False, ("tanh",), True),  # the same kept channel-last: 20 channels per pixel
    (2, 37, 50, 20, 20, 5, 1, 2, True, True, (), True),          # padded channels, channel-last result that is no multiple of eight
    (12, 3, 64, 64, 62, 7, 2, 3, False, True, (), False),         # three channels, even tile
    (70, 3, 18, 57, 57, 1, 2, 0, False, False, (), False),       # one tap, K of three channels, many tiles
    (2, 104, 264, 28, 28, 3, 1, 1, True, True, ("sigmoid", "neg"), False),
    (64, 104, 192, 28, 28, 3, 1, 1, False, True, (), False),     # 128-wide tiles
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", TAPS_CASES, ids=[f"taps{i}" for i in range(len(TAPS_CASES))])
def test_convolution_with_ragged_channels(dtype, case):
    b, ci, co, h, w, k, s, p, res, relu, acts, tail = case
    spec, data = W.conv_group(b, ci, co, h, w, k, s, p, dtype, residual=res, relu=relu, acts=acts, tail=tail)
    # one channel of f32: padding it fourfold costs more than the element gather
    by_gather, opts = ci == 1 and dtype == "f32", {"no_direct": 1}
    assert any("_gather" in x for x in steps_of(spec, opts) if x.startswith("igemm")) == by_gather, steps_of(spec, opts)
    check(spec, data, dtype, f"taps {case} {dtype}")


def two_convs():
    import numpy as np
    rng = np.random.default_rng(9)
    spec, dtype, at = W.GraphSpec("two_layers"), "bf16", dict(stride=(2, 2), pad=(1, 1))
    shapes = dict(x=(64, 53, 53, 53), w1=(64, 53, 3, 3), w2=(24, 64, 3, 3))
    data = {k: W.as_dtype(rng.standard_normal(s) * (1.0 if k == "x" else (2 / np.prod(s[1:])) ** 0.5), dtype) for k, s in shapes.items()}
    x, w1, w2 = spec.input("x", dtype, shapes["x"]), spec.param("w1", dtype, shapes["w1"]), spec.param("w2", dtype, shapes["w2"])
    o, (y,) = spec.op("conv2d", [x, w1], [(dtype, (64, 64, 27, 27))], **at); spec.group([o])
    o, (y,) = spec.op("conv2d", [y, w2], [(dtype, (64, 24, 14, 14))], **at); spec.group([o])
    spec.output(y)
    return spec, data


def test_direct_load_contractions_repeat_to_the_bit():
    # a stage that is requested again while another wave still reads it shows as a pixel that differs from run to run
    import torch
    from paper_1810_00952_amd import harness
    spec, data = two_convs()
    assert [k.rsplit("64x64", 1)[-1] for k in steps_of(spec)][1:] == ["_dma_taps", "_dma"], steps_of(spec)
    check(spec, data, "bf16", "two convolutions")
    s = harness.Session(spec); s.load(data); s.run()
    first = s.output().clone()
    for _ in range(40):
        s.run()
        assert torch.equal(first.view(torch.int16), s.output().view(torch.int16))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dims", [(10, 1446, 128, 45), (150, 867, 20, 100), (300, 235, 57, 33), (1, 1627, 450, 5), (513, 1001, 391, 77), (40, 112, 130, 70)])
def test_dense_with_ragged_features(dtype, dims):
    spec, data = W.mlp(*dims, dtype=dtype)
    check(spec, data, dtype, f"ragged mlp {dims} {dtype}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_input_gradient_with_ragged_channels(dtype):
    for kind, dims, stride, pad in (("dense_grad_x", (167, 391, 720), 1, 0), ("conv2d_grad_x", (3, 93, 19, 19, 45, 5), 1, 2), ("conv2d_grad_x", (6, 40, 26, 26, 30, 3), 1, 1)):
        spec, data = W.grad_case(kind, dims, dtype, stride, pad)
        check(spec, data, dtype, f"ragged {kind} {dims} {dtype}")


# ---- weights in the order of the fragments: last tiles of few channels, K ending inside a step, every tile and slicing; a weight that two
# convolutions read stays in rows
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("form", [32 * 16 + 1, 32 * 16 + 8, 16 * 16 + 8])
def test_convolution_weights_in_fragment_order(dtype, form):
    for ci, co, k in ((8, 1, 3), (16, 33, 3), (12, 17, 5), (3, 40, 2), (24, 64, 3)):
        spec, data = W.conv_group(2, ci, co, 9, 11, k, 1, 1, dtype, residual=True)
        check(spec, data, dtype, f"fragments {ci} {co} {k} {form}", {"direct_all": form})


# a single pixel's second layer on the adding launch of the first, ragged channels between them; by itself; and where there is no slice to add
@pytest.mark.parametrize("dtype,dims,chained", [("f32", (8, 2048, 50, 10), True), ("bf16", (8, 4096, 100, 30), True), ("f32", (70, 4096, 33, 64), True), ("bf16", (5, 72, 50, 10), False)])
def test_layers_of_a_single_pixel(dtype, dims, chained):
    spec, data = W.pixel_layers(*dims, dtype)
    assert any(k.endswith("+dense") for k in steps_of(spec)) == chained, steps_of(spec)
    check(spec, data, dtype, f"pixel {dims} {dtype}")
    check(spec, data, dtype, f"pixel {dims} {dtype}", {"no_dense_chain": 1})


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_weight_of_two_convolutions_stays_in_rows(dtype):
    import numpy as np
    rng = np.random.default_rng(21)
    spec, at = W.GraphSpec("shared"), dict(pad=(1, 1))
    data = {"x": W.as_dtype(rng.standard_normal((1, 16, 10, 10)), dtype), "w": W.as_dtype(rng.standard_normal((16, 16, 3, 3)) / 12, dtype)}
    y, w = spec.input("x", dtype, (1, 16, 10, 10)), spec.param("w", dtype, (16, 16, 3, 3))
    for _ in range(2):
        o, (y,) = spec.op("conv2d", [y, w], [(dtype, (1, 16, 10, 10))], **at); spec.group([o])
    spec.output(y)
    check(spec, data, dtype, f"shared weight {dtype}")


# ---- bf16 layers of whole K tiles, and short K, on the kernel without LDS tiles: from channels in planes, inside a channel-last network, dense;
# the larger neighbour of each stays on LDS tiles
@pytest.mark.parametrize("small,case", [(True, (2, 128, 72, 9, 9, 3, 1, 1)), (True, (1, 64, 112, 24, 24, 3, 2, 0)), (False, (64, 128, 128, 28, 28, 3, 1, 1)), (False, (3, 64, 64, 14, 14, 3, 1, 1))])
def test_small_bf16_convolutions_of_whole_k_tiles(small, case):
    spec, data = W.conv_group(*case, dtype="bf16", residual=True)
    assert any("_direct" in x for x in steps_of(spec)) == small, steps_of(spec)
    check(spec, data, "bf16", f"small {case}")


@pytest.mark.parametrize("small,batch,c,h", [(True, 2, 128, 7), (True, 4, 192, 14), (True, 1, 512, 7), (False, 32, 128, 28)])
def test_small_bf16_convolutions_of_a_channel_last_network(small, batch, c, h):
    import numpy as np
    rng = np.random.default_rng(22)
    spec, t = W.GraphSpec("chain"), ("bf16", (batch, c, h, h))
    data = {"x": W.as_dtype(rng.standard_normal(t[1]), "bf16")}
    y = spec.input("x", *t)
    for i in range(3):
        data[f"w{i}"], data[f"b{i}"] = W.as_dtype(rng.standard_normal((c, c, 3, 3)) * (2 / (9 * c)) ** 0.5, "bf16"), W.as_dtype(rng.uniform(-1, 1, c), "f32")
        o0, (v,) = spec.op("conv2d", [y, spec.param(f"w{i}", "bf16", (c, c, 3, 3))], [t], pad=(1, 1))
        o1, (v,) = spec.op("bias_add", [v, spec.param(f"b{i}", "f32", (c,))], [t], axis=1)
        o2, (y,) = spec.op("relu", [v], [t])
        spec.group([o0, o1, o2])
    spec.output(y)
    assert any("_direct" in x for x in steps_of(spec)) == small, steps_of(spec)
    check(spec, data, "bf16", f"chain {batch} {c} {h}")


@pytest.mark.parametrize("small,dtype,dims", [(True, "bf16", (28, 320, 446)), (True, "bf16", (16, 1024, 64)), (True, "f32", (616, 128, 16)), (True, "bf16", (48, 1280, 980)),
                                              (False, "bf16", (657, 1728, 1152)), (False, "bf16", (341, 320, 832)), (False, "f32", (1000, 128, 1000))])
def test_small_dense_layers_of_whole_or_few_k_tiles(small, dtype, dims):
    import numpy as np
    m, k, n = dims
    rng = np.random.default_rng(23)
    spec, t = W.GraphSpec("dense"), (dtype, (m, n))
    data = {"x": W.as_dtype(rng.standard_normal((m, k)), dtype), "w": W.as_dtype(rng.standard_normal((n, k)) / k ** 0.5, dtype), "b": W.as_dtype(rng.uniform(-1, 1, n), "f32")}
    o0, (v,) = spec.op("dense", [spec.input("x", dtype, (m, k)), spec.param("w", dtype, (n, k))], [t])
    o1, (v,) = spec.op("bias_add", [v, spec.param("b", "f32", (n,))], [t], axis=1)
    o2, (v,) = spec.op("relu", [v], [t])
    spec.group([o0, o1, o2]); spec.output(v)
    assert any("_direct" in x for x in steps_of(spec)) == small, steps_of(spec)
    check(spec, data, dtype, f"dense {dims} {dtype}")


# ---- a backward pass of a small dense layer: the weights' gradient from dy and x as they lie; batches that end inside a step, last tiles of
# few rows and columns, and a batch past the form
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("columns,dims", [(True, (1, 5, 3)), (True, (14, 128, 88)), (True, (9, 33, 17)), (True, (257, 31, 65)), (True, (300, 72, 40)), (True, (70, 200, 144)), (False, (6200, 21, 16))])
def test_both_gradients_of_a_small_dense_layer(dtype, columns, dims):
    import numpy as np
    m, n, k = dims
    rng = np.random.default_rng(24)
    for out in {dtype, "f32"}:
        spec = W.GraphSpec("dense_grads")
        data = {"dy": W.as_dtype(rng.standard_normal((m, n)), dtype), "x": W.as_dtype(rng.standard_normal((m, k)), dtype), "w": W.as_dtype(rng.standard_normal((n, k)) / n ** 0.5, dtype)}
        dy, x, w = spec.input("dy", dtype, (m, n)), spec.input("x", dtype, (m, k)), spec.param("w", dtype, (n, k))
        o, (dx,) = spec.op("dense_grad_x", [dy, w], [(dtype, (m, k))]); spec.group([o])
        o, (dw,) = spec.op("dense_grad_w", [dy, x], [(out, (n, k))], out_dtype=out); spec.group([o])
        spec.output(dx); spec.output(dw)
        assert any("_columns" in s for s in steps_of(spec)) == columns, steps_of(spec)
        check(spec, data, dtype, f"dense gradients {dims} {dtype} {out}")


# the longest batches of the column form, 24 steps a wave (whole, and ending inside the last step), and one row past it
@pytest.mark.parametrize("dtype,batch,columns", [("bf16", 6143, True), ("bf16", 6144, True), ("bf16", 6145, False), ("f32", 3070, True), ("f32", 3072, True), ("f32", 3073, False)])
def test_longest_batches_of_the_column_form(dtype, batch, columns):
    import numpy as np
    rng = np.random.default_rng(30)
    spec = W.GraphSpec("dense_grads")
    data = {"dy": W.as_dtype(rng.standard_normal((batch, 21)), dtype), "x": W.as_dtype(rng.standard_normal((batch, 16)), dtype), "w": W.as_dtype(rng.standard_normal((21, 16)) / 21 ** 0.5, dtype)}
    dy, x, w = spec.input("dy", dtype, (batch, 21)), spec.input("x", dtype, (batch, 16)), spec.param("w", dtype, (21, 16))
    o, (dx,) = spec.op("dense_grad_x", [dy, w], [(dtype, (batch, 16))]); spec.group([o])
    o, (dw,) = spec.op("dense_grad_w", [dy, x], [("f32", (21, 16))], out_dtype="f32"); spec.group([o])
    spec.output(dx); spec.output(dw)
    assert any("_columns" in s for s in steps_of(spec)) == columns, steps_of(spec)
    check(spec, data, dtype, f"columns {batch} {dtype}")


# ---- x of a weight gradient changes its layout beside dy, ahead of the input gradient that stands between them
@pytest.mark.parametrize("case", [(8, 128, 28, 28, 128, 3), (3, 64, 20, 20, 64, 3)])
def test_both_operands_of_a_backward_pass_change_layout_in_one_launch(case):
    import numpy as np
    b, c, h, w, o, k = case
    rng = np.random.default_rng(26)
    spec, at, dtype = W.GraphSpec("moves"), dict(pad=(1, 1)), "bf16"
    shapes = dict(dy=(b, o, h, w), x=(b, c, h, w), w=(o, c, k, k))
    data = {n: W.as_dtype(rng.standard_normal(t) * ((o * k * k) ** -0.5 if n == "w" else 1.0), dtype) for n, t in shapes.items()}
    dy, x, wt = spec.input("dy", dtype, shapes["dy"]), spec.input("x", dtype, shapes["x"]), spec.param("w", dtype, shapes["w"])
    q, (dx,) = spec.op("conv2d_grad_x", [dy, wt], [(dtype, shapes["x"])], **at); spec.group([q])
    q, (dw,) = spec.op("conv2d_grad_w", [dy, x], [("f32", shapes["w"])], out_dtype="f32", **at); spec.group([q])
    spec.output(dx); spec.output(dw)
    steps = steps_of(spec)
    assert steps[0] == "nchw_to_nhwc | nchw_to_nhwc" and not any("_to_nhwc" in s for s in steps[2:]), steps
    check(spec, data, dtype, f"moves {case}")


# ---- one channel's pixels turned behind the convolution that computes them
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_one_channels_pixels_are_turned(dtype):
    for dims in ((5, 7, 5, 8), (2, 64, 9, 12)):
        spec, data = W.one_channel_turned(*dims, dtype)
        check(spec, data, dtype, f"one channel {dims} {dtype}")


# ---- a change of layout does not overtake the cell whose h or c it turns
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("out", ["h", "c"])
def test_a_cells_result_changes_its_layout_behind_the_cell(dtype, out):
    for dims in ((16, 64, 128), (33, 128, 256)):
        spec, data = W.lstm_cell_transposed(*dims, dtype, out)
        check(spec, data, dtype, f"transposed {out} {dims} {dtype}")


# ---- a backward pass of a small convolution: the weights' gradient over the rows of dy and x however few they are
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(1, 3, 4, 4, 2, 3, 1, 1), (2, 16, 12, 12, 24, 3, 1, 1), (3, 9, 15, 14, 17, 3, 2, 1), (5, 31, 7, 9, 33, 1, 1, 0), (4, 12, 11, 11, 10, 5, 2, 0), (1, 64, 9, 9, 8, 1, 2, 0)])
def test_both_gradients_of_a_small_convolution(dtype, case):
    import numpy as np
    b, c, h, w, o, k, s, p = case
    rng = np.random.default_rng(25)
    oh, ow = W.conv_out(h, k, s, p), W.conv_out(w, k, s, p)
    at = dict(stride=(s, s), pad=(p, p))
    for out in {dtype, "f32"}:
        spec = W.GraphSpec("conv_grads")
        shapes = dict(dy=(b, o, oh, ow), x=(b, c, h, w), w=(o, c, k, k))
        data = {n: W.as_dtype(rng.standard_normal(t) * ((o * k * k) ** -0.5 if n == "w" else 1.0), dtype) for n, t in shapes.items()}
        dy, x, wt = spec.input("dy", dtype, shapes["dy"]), spec.input("x", dtype, shapes["x"]), spec.param("w", dtype, shapes["w"])
        q, (dx,) = spec.op("conv2d_grad_x", [dy, wt], [(dtype, shapes["x"])], **at); spec.group([q])
        q, (dw,) = spec.op("conv2d_grad_w", [dy, x], [(out, shapes["w"])], out_dtype=out, **at); spec.group([q])
        spec.output(dx); spec.output(dw)
        # (at a stride dy is spread out with zeros, its rows padded where its channels are no whole vectors)
        assert any("_rows" in n for n in steps_of(spec)) and ("dilate_nhwc" in steps_of(spec)) == (s > 1), steps_of(spec)
        check(spec, data, dtype, f"convolution gradients {case} {dtype} {out}")


# ---- direct-load tiles of 64x64 with the steps of a K tile over two halves of the waves: grids of up to 256 workgroups, and one past it; the
# fewest K tiles, a part-filled last one, one beyond a round of the stages; rows of channels, any order, K tiles across taps, K slices
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dims", [(1024, 136, 1024, 10), (1032, 136, 1024, 10), (1000, 200, 1001, 3), (70, 264, 72, 50), (65, 1000, 130, 9)])
def test_dense_on_two_halves_of_the_waves(dtype, dims):
    spec, data = W.mlp(*dims, dtype=dtype)
    check(spec, data, dtype, f"two halves {dims} {dtype}", {"no_direct": 1})


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(4, 96, 136, 29, 29, 3, 1, 1, True), (2, 64, 72, 15, 13, 3, 1, 1, False), (5, 24, 65, 21, 21, 5, 2, 2, True), (9, 40, 130, 29, 28, 1, 1, 0, True)])
def test_convolution_on_two_halves_of_the_waves(dtype, case):
    b, ci, co, h, w, k, s, p, res = case
    for tail in (False, True):
        spec, data = W.conv_group(b, ci, co, h, w, k, s, p, dtype, residual=res, tail=tail)
        check(spec, data, dtype, f"two halves {case} {dtype} {tail}", {"no_direct": 1})


# ---- f32 tiles and K slices chosen by how the grid fills the chip ----------------------------------------------------------
@pytest.mark.parametrize("case", [(8, 256, 256, 14, 14, 3, 1, 1), (4, 64, 128, 28, 28, 3, 2, 1), (9, 72, 200, 14, 14, 3, 1, 1)])
def test_f32_half_filled_grids_split_k(case):
    spec, data = W.conv_group(*case, dtype="f32", residual=True)
    opts = {"no_direct": 1}
    assert any(x.endswith("_splitk") for x in steps_of(spec, opts)), steps_of(spec, opts)
    check(spec, data, "f32", f"half-filled {case}")                # as planned, and with LDS tiles


# ---- 256 x 256 tiles (igemm_big.hip) -----------------------------------------------------------------------------------------
@pytest.mark.parametrize("m,n,k,res", [(4096, 4096, 64, False), (3841, 4000, 192, False), (4100, 3336, 128, True)])
def test_dense_at_matrix_multiplication_scale(m, n, k, res):
    # ragged last tiles both ways, the shortest K and one that ends between two rounds of the stages, with and without a residual
    import numpy as np
    rng = np.random.default_rng(3)
    g = W.GraphSpec("dense_big")
    x = g.input("x", "bf16", (m, k)); w = g.param("w", "bf16", (n, k)); b = g.param("b", "f32", (n,))
    t = ("bf16", (m, n))
    data = {"x": W.as_dtype(rng.standard_normal((m, k)), "bf16"), "w": W.as_dtype(rng.standard_normal((n, k)) / k ** 0.5, "bf16"), "b": W.as_dtype(rng.uniform(-1, 1, n), "f32")}
    o0, (y,) = g.op("dense", [x, w], [t]); ops = [o0]
    o1, (y,) = g.op("bias_add", [y, b], [t], axis=1); ops.append(o1)
    if res:
        r = g.input("r", "bf16", (m, n)); data["r"] = W.as_dtype(rng.standard_normal((m, n)), "bf16")
        o2, (y,) = g.op("add", [y, r], [t]); ops.append(o2)
    o3, (y,) = g.op("relu", [y], [t]); ops.append(o3)
    g.group(ops); g.output(y)
    assert any("256x256" in s for s in steps_of(g)), steps_of(g)
    check(g, data, "bf16", f"dense {m}x{n}x{k}")


# ---- bf16, a very long K on few tiles: cut along K by the direct-load kernel -------------------------------------------------
@pytest.mark.parametrize("case", [(2, 512, 512, 7, 7, 3, 1, 1, True, True), (1, 512, 136, 9, 8, 3, 2, 1, True, False)])
def test_bf16_long_k_on_few_tiles(case):
    b, ci, co, h, w, k, s, p, res, tail = case
    spec, data = W.conv_group(b, ci, co, h, w, k, s, p, "bf16", residual=res, tail=tail)
    assert any(x.endswith("_dma_splitk") for x in steps_of(spec)), steps_of(spec)
    check(spec, data, "bf16", f"long K {case}")


# ---- a whole sequence in one launch (lstm_seq.hip) ---------------------------------------------------------------------------
def run_sequence(T, B, I, H, d, opts=None, room=None, c0=None, h0=None, h0_slot=None, capture=False):
    import torch
    from paper_1810_00952_amd import harness
    spec = W.lstm_cell_graph(B, I, H, "bf16", True)
    s = harness.Session(spec, opts=opts)
    s.load({"w": d["w"], "b": d["b"]})
    x = harness.to_device(d["x"], "bf16")
    h0 = torch.zeros((B, H), dtype=torch.bfloat16, device="cuda:0") if h0 is None else harness.to_device(h0, "bf16")
    c = torch.zeros((B, H), dtype=torch.float32, device="cuda:0") if c0 is None else harness.to_device(c0, "f32")
    hs = torch.full((T, B, H), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    if h0_slot is not None:
        at = int(h0_slot * B * H)                         # a fraction: across two slots
        hs.view(-1)[at:at + B * H] = h0.view(-1)
        h0 = hs.view(-1)[at:at + B * H]
    ws = torch.empty(max(256, s.plan.recurrent_workspace_bytes(room or T)), dtype=torch.uint8, device="cuda:0")
    n = s.by_name
    roles = {"x": n["x"], "h_in": n["h"], "c_in": n["c"], "c_out": spec.outputs[0], "h_out": spec.outputs[1]}

    def run():
        s.plan.run_recurrent(T, roles, x.data_ptr(), B * I * 2, h0.data_ptr(), c.data_ptr(), hs.data_ptr(), B * H * 2,
                             {n["w"]: s.tensors[n["w"]].data_ptr(), n["b"]: s.tensors[n["b"]].data_ptr()}, ws.data_ptr(), ws.numel(), harness.stream_handle())
    if capture:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run()
        graph.replay()
    else:
        run()
    torch.cuda.synchronize()
    return O.widen(harness.to_host(hs), "bf16"), O.widen(harness.to_host(c), "f32")


# batches that leave XCDs without rows, with ragged last groups, and at the limit; every hidden size the kernel is built for; odd
# and even step counts from the fewest the kernel takes; the sequence whole and in chunks (the second starts from the first one's last h and c)
SEQ_CASES = [(16, 5, 128, 256, None), (17, 70, 192, 512, None), (18, 33, 128, 768, None), (16, 64, 256, 1024, None), (13, 128, 128, 1024, None), (17 + 17, 1, 128, 1024, 17)]


@pytest.mark.parametrize("case", SEQ_CASES, ids=[f"seq{i}" for i in range(len(SEQ_CASES))])
def test_lstm_sequence_in_one_launch(case):
    import numpy as np
    T, B, I, H, room = case
    d = W.lstm_data(T, B, I, H, "bf16")
    rng = np.random.default_rng(11)
    c0, h0 = W.as_dtype(rng.standard_normal((B, H)), "f32"), W.as_dtype(rng.uniform(-1, 1, (B, H)), "bf16")
    ref_h, ref_c = O.lstm_sequence(O.widen(d["x"], "bf16"), O.widen(d["w"], "bf16"), O.widen(d["b"], "f32"), O.widen(h0, "bf16"), O.widen(c0, "f32"), h_dtype="bf16")
    for opts in (None, {"no_seq": 2}, {"no_seq": 1}):
        print(f"sequence {case} {opts}", flush=True)
        h, c = run_sequence(T, B, I, H, d, opts, room, c0, h0)
        assert_close(h, ref_h, "bf16", f"sequence h {case} {opts}")
        assert_close(c, ref_c, "bf16", f"sequence c {case} {opts}")
    # one result whichever form runs it: a launch per step, and one launch whose workgroups are all there, whoever is there, or too
    # few (one XCD a workgroup short, two blocks each, XCDs with none, three in all)
    first = run_sequence(T, B, I, H, d, {"no_seq": 1}, room, c0, h0)
    for no_seq in (0, 0, 2, H // 4 - 1, H // 8 + 3, 9, 3):
        print(f"sequence {case} bits, no_seq {no_seq}", flush=True)
        again = run_sequence(T, B, I, H, d, {"no_seq": no_seq}, room, c0, h0)
        np.testing.assert_array_equal(first[0], again[0])
        np.testing.assert_array_equal(first[1], again[1])


# whole XCDs beside ones without a workgroup: each works off several groups of rows, one behind the other, its weights in registers and the
# exchange in that group's ring; odd and even step counts, at most eight rows a group and more, last groups of fewer rows
@pytest.mark.parametrize("T,B,H", [(17, 64, 256), (18, 64, 256), (19, 70, 512), (17, 9, 1024), (16, 128, 768)])
def test_lstm_sequence_of_several_groups_of_rows_an_xcd(T, B, H):
    import numpy as np
    I = 128
    d = W.lstm_data(T, B, I, H, "bf16")
    rng = np.random.default_rng(13)
    c0, h0 = W.as_dtype(rng.standard_normal((B, H)), "f32"), W.as_dtype(rng.uniform(-1, 1, (B, H)), "bf16")
    first = run_sequence(T, B, I, H, d, {"no_seq": 1}, None, c0, h0)
    for n in (1, 3, 7):
        print(f"sequence {T} {B} {H} on {n} XCDs", flush=True)
        again = run_sequence(T, B, I, H, d, {"no_seq": -n}, None, c0, h0)
        np.testing.assert_array_equal(first[0], again[0])
        np.testing.assert_array_equal(first[1], again[1])


# what the waiting members must not take for a word that is still to come: NaN in a row's h and c from some step on, infinite c, h at
# its largest (1 exactly in bf16), the sign of zero; rows beside them stay what they are
@pytest.mark.parametrize("B", [5, 64, 70])
def test_lstm_sequence_with_nan_and_extreme_rows(B):
    import numpy as np
    T, I, H = 19, 128, 512
    d = dict(W.lstm_data(T, B, I, H, "bf16"))
    c0 = np.zeros((B, H), np.float32)
    c0[1], c0[2], c0[3, ::2] = np.inf, 1e30, -np.inf
    x = O.widen(d["x"], "bf16").copy()
    x[7, 0, :], x[4, 4, 3] = np.nan, np.inf
    x[:, 2] *= 1e4                                       # saturated gates
    d["x"] = W.as_dtype(x, "bf16")
    first, again = (run_sequence(T, B, I, H, d, {"no_seq": n}, None, c0) for n in (1, 0))
    assert np.isnan(first[0][7:, 0]).all() and np.abs(first[0][:, 2]).max() == 1.0
    np.testing.assert_array_equal(first[0], again[0])
    np.testing.assert_array_equal(first[1], again[1])


def test_lstm_sequence_captured_and_eager_agree():
    import numpy as np
    T, B, I, H = 16, 64, 128, 1024
    d = W.lstm_data(T, B, I, H, "bf16")
    eager, captured = run_sequence(T, B, I, H, d), run_sequence(T, B, I, H, d, capture=True)
    np.testing.assert_array_equal(eager[0], captured[0])
    np.testing.assert_array_equal(eager[1], captured[1])


# a sequence continued from the last state of the one before, in the same buffer: h0 is the slot that the last step will write
@pytest.mark.parametrize("room", [None, 16])
def test_lstm_sequence_from_the_last_slot_of_its_own_results(room):
    import numpy as np
    T, B, I, H = 33, 9, 128, 1024
    d = W.lstm_data(T, B, I, H, "bf16")
    h0 = W.as_dtype(np.random.default_rng(12).uniform(-1, 1, (B, H)), "bf16")
    ref_h, ref_c = O.lstm_sequence(O.widen(d["x"], "bf16"), O.widen(d["w"], "bf16"), O.widen(d["b"], "f32"), O.widen(h0, "bf16"), np.zeros((B, H)), h_dtype="bf16")
    for at in (None, T - 1, 1, T - 1.5):
        print(f"sequence from slot {at}, room {room}", flush=True)
        h, c = run_sequence(T, B, I, H, d, None, room, None, h0, at)
        assert_close(h, ref_h, "bf16", f"sequence h, h0 in slot {at}")
        assert_close(c, ref_c, "bf16", f"sequence c, h0 in slot {at}")


def test_lstm_sequences_on_two_streams_do_not_wait_for_each_other():
    import numpy as np
    import torch
    T, B, I, H = 40, 64, 128, 1024
    ds = [W.lstm_data(T, B, I, H, "bf16", config=5 + i) for i in (0, 20)]
    alone = [run_sequence(T, B, I, H, d) for d in ds]
    import threading
    got = [None, None]

    def work(i):
        torch.cuda.set_device(0)
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                got[i] = run_sequence(T, B, I, H, ds[i])
    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    for i in range(2):
        np.testing.assert_array_equal(got[i][0], alone[i][0])
        np.testing.assert_array_equal(got[i][1], alone[i][1])


# plans whose quicker forms (padded rows, weight gradients over rows) need more than the built-in workspace: the allocation-free
# entry point runs the form that fits, from its own packed weights behind the plan's
@pytest.mark.parametrize("case", ["conv", "two_convs", "grad_w"])
def test_built_in_workspace_holds_a_smaller_form(case):
    import torch
    from paper_1810_00952_amd import binding, harness
    if case == "conv":
        spec, data = W.conv_group(64, 53, 384, 53, 53, 1, 2, 0, "bf16")
        dtype = "bf16"
    elif case == "two_convs":                          # the second layer's weights are read alike by both forms, and packed once
        spec, data = two_convs()
        dtype = "bf16"
    else:
        spec, data = W.grad_case("conv2d_grad_w", (32, 235, 36, 36, 24, 1), "f32", 1, 0, second_is_param=False)
        dtype = "f32"
    s = harness.Session(spec); s.load(data); s.alloc()
    assert s.plan.workspace_bytes() > binding.STATIC_WORKSPACE_BYTES
    ref = OG.run(spec, data)[spec.outputs[0]]
    budget = (lambda: error_budget(spec, data)[spec.outputs[0]]) if dtype == "f32" else None
    for static in (False, True):
        print(case, static, flush=True)
        s.output().zero_()
        if static:
            s.plan.run_static({vid: t.data_ptr() for vid, t in s.tensors.items()}, harness.stream_handle())
        else:
            s.run()
        torch.cuda.synchronize()
        assert_close(O.widen(harness.to_host(s.output()), dtype), ref, dtype, f"{case} static={static}", budget=budget)


# ---- operands straight into registers, K over the waves of a workgroup (igemm_direct.hip) ------------------------------------
DIRECT_CASES = [
    # batch cin cout h  w  k s p residual relu acts tail
    (1, 64, 64, 56, 56, 3, 1, 1, False, True, (), False),      # planes read and written as they are
    (3, 8, 33, 9, 11, 3, 1, 1, True, True, (), False),         # one channel past a tile; images of 99 pixels
    (2, 72, 31, 13, 7, 5, 2, 2, True, False, ("tanh", "neg"), True),     # stride 2, channel-last result of odd rows
    (1, 20, 50, 12, 12, 5, 1, 0, False, True, (), True),       # f32 vectors, bf16 element by element
    (5, 7, 40, 10, 9, 3, 1, 1, True, True, ("sigmoid",), False),    # every element decoded, padding
    (2, 1, 20, 28, 28, 5, 1, 0, False, False, ("tanh",), False),    # one channel
    (4, 24, 16, 1, 1, 1, 1, 0, False, True, (), False),        # one pixel per image, fewer K steps than slices
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("form", [32 * 16 + 1, 32 * 16 + 2, 32 * 16 + 4, 32 * 16 + 8, 16 * 16 + 8])
def test_contractions_without_lds_tiles(dtype, form):
    for case in DIRECT_CASES:
        b, ci, co, h, w, k, s, p, res, relu, acts, tail = case
        spec, data = W.conv_group(b, ci, co, h, w, k, s, p, dtype, residual=res, relu=relu, acts=acts, tail=tail)
        assert any("_direct" in x for x in steps_of(spec, {"direct_all": form})), steps_of(spec, {"direct_all": form})
        check(spec, data, dtype, f"direct {case} {dtype} {form}", {"direct_all": form})
    for dims in ((1, 4, 8, 8), (33, 784, 130, 31), (70, 515, 17, 5), (129, 30, 64, 3)):
        spec, data = W.mlp(*dims, dtype=dtype)
        check(spec, data, dtype, f"direct mlp {dims} {dtype} {form}", {"direct_all": form})
    # channel-last input, two layers (the second reads what the first wrote, channels fastest), channel-last output
    spec, data = W.channel_last_block(2, 24, 9, 7, dtype)
    check(spec, data, dtype, f"direct channel-last block {dtype} {form}", {"direct_all": form})


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("b,c,h,w,k,pool,tail", [(3, 12, 12, 14, 3, 2, False), (2, 33, 9, 11, 3, 2, True), (5, 6, 7, 7, 5, 2, False), (2, 8, 9, 9, 3, 3, False)])
def test_max_pool_over_a_contraction_without_lds_tiles(dtype, b, c, h, w, k, pool, tail):
    # odd images (their last row and column are in no window), values of both signs, the pooled result in Shape order and
    # channel-last; 3x3 windows stay a kernel of their own.  The two-kernel form gives the same bits
    import numpy as np
    rng = np.random.default_rng(b * c)
    g = W.GraphSpec("conv_pool")
    oh, ow = h - k + 1, w - k + 1
    shapes = dict(x=(b, 5, h, w), w=(c, 5, k, k))
    data = {n: W.as_dtype(rng.standard_normal(s), dtype) for n, s in shapes.items()}
    data["b"] = W.as_dtype(rng.uniform(-1, 1, c), "f32")
    x, wv, bv = g.input("x", dtype, shapes["x"]), g.param("w", dtype, shapes["w"]), g.param("b", "f32", (c,))
    o0, (y,) = g.op("conv2d", [x, wv], [(dtype, (b, c, oh, ow))])
    o1, (y,) = g.op("bias_add", [y, bv], [(dtype, (b, c, oh, ow))], axis=1)
    g.group([o0, o1])
    q = (dtype, (b, c, (oh - pool) // pool + 1, (ow - pool) // pool + 1))
    o, (y,) = g.op("maxpool2d", [y], [q], kernel=(pool, pool), stride=(pool, pool)); g.group([o])
    if tail:
        o, (y,) = g.op("neg", [y], [q]); g.group([o])
    g.output(y)
    opts = {"direct_all": 1}
    assert any(s.endswith("_maxpool") for s in steps_of(g, opts)) == (pool == 2), steps_of(g, opts)
    check(g, data, dtype, f"direct pool {dtype} {(b, c, h, w, k, pool)}", opts)
    if pool == 2:
        got, _ = run_hip(g, data, opts=opts)
        # the contraction's result as an output too: the pool then is a kernel of its own
        o_mid = g.ops[1].outputs[0]
        g.output(o_mid)
        assert not any(s.endswith("_maxpool") for s in steps_of(g, opts)), steps_of(g, opts)
        apart, _ = run_hip(g, data, opts=opts)
        np.testing.assert_array_equal(got[g.outputs[0]], apart[g.outputs[0]])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_contraction_with_k_split_over_workgroups_where_another_kernel_is_planned(dtype):
    # the adding launch at the sizes the kernel without LDS tiles has taken over
    for b, ci, co, h, w, k, s, p, res, tail in ((1, 256, 256, 14, 14, 3, 1, 1, True, False), (2, 64, 72, 9, 11, 3, 1, 1, True, False), (64, 20, 50, 12, 12, 5, 1, 0, False, False),
                                                (3, 36, 24, 9, 7, 3, 2, 1, True, False), (2, 40, 40, 8, 8, 5, 1, 2, False, True)):
        if dtype == "bf16" and ci % 8:
            continue
        spec, data = W.conv_group(b, ci, co, h, w, k, s, p, dtype, residual=res, tail=tail)
        opts = {"no_direct": 1}
        assert any(x.endswith("_splitk") for x in steps_of(spec, opts)) and not any("_direct" in x for x in steps_of(spec, opts)), steps_of(spec, opts)
        check(spec, data, dtype, f"split-K {(b, ci, co, h, w)} {dtype}", opts)


def test_one_param_read_by_layers_of_different_batches():
    # one layer small enough for the kernel without LDS tiles, one not: both read the same packed weights
    import numpy as np
    rng = np.random.default_rng(4)
    for k in (200, 203, 256):
        g = W.GraphSpec("shared")
        xs = [g.input("xa", "f32", (9, k)), g.input("xb", "f32", (3000, k))]
        w = g.param("w", "f32", (500, k))
        data = {"xa": W.as_dtype(rng.standard_normal((9, k)), "f32"), "xb": W.as_dtype(rng.standard_normal((3000, k)), "f32"), "w": W.as_dtype(rng.standard_normal((500, k)), "f32")}
        for x, m in zip(xs, (9, 3000)):
            o, (y,) = g.op("dense", [x, w], [("f32", (m, 500))]); g.group([o]); g.output(y)
        check(g, data, "f32", f"shared param {k}")


# ---- the recurrent cell without LDS tiles ---------------------------------------------------------------------------------------
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,I,H,opts", [(1, 8, 16, {}), (17, 96, 48, {}), (5, 656, 80, {}), (33, 24, 272, {}), (70, 104, 336, {}), (129, 40, 144, {}), (9, 128, 64, {"direct_all": 1}),
                                        (48, 16, 32, {"direct_all": 4}), (16, 200, 64, {"direct_all": 8})])
def test_recurrent_cell_without_lds_tiles(dtype, B, I, H, opts):
    # a step whose x and h end inside a K tile, one unit block and many, rows past a tile of 16, both widths of a workgroup
    import numpy as np
    spec = W.lstm_cell_graph(B, I, H, dtype, True)
    assert steps_of(spec, opts)[0].endswith("_direct_gates"), steps_of(spec, opts)
    rng = np.random.default_rng(B + H)
    data = {"x": W.as_dtype(rng.standard_normal((B, I)), dtype), "h": W.as_dtype(rng.standard_normal((B, H)) / 2, dtype), "c": W.as_dtype(rng.standard_normal((B, H)), "f32"),
            "w": W.as_dtype(rng.uniform(-1, 1, (4 * H, I + H)) * H ** -0.5, dtype), "b": W.as_dtype(rng.uniform(-1, 1, 4 * H) * H ** -0.5, "f32")}
    print(f"cell {dtype} {B} {I} {H}", flush=True)
    ref = OG.run(spec, data)
    got, _ = run_hip(spec, data, opts=opts)
    for v in spec.outputs:
        assert_close(got[v], ref[v], spec.values[v].type.dtype, f"cell {dtype} {(B, I, H)}")


# ---- both gradients of a layer in one launch (igemm_grads.hip) ------------------------------------------------------------------
def layer_backward(kind, dims, dtype, stride=1, pad=1, weights_first=False, inner=False):
    import numpy as np
    rng = np.random.default_rng(sum(dims))
    g = W.GraphSpec("layer_backward")
    if kind == "dense":
        m, n, k = dims
        sdy, sx, sw, at, dx, dw = (m, n), (m, k), (n, k), {}, "dense_grad_x", "dense_grad_w"
    else:
        b, c, h, w, o, k = dims
        oh, ow = (h + 2 * pad - k) // stride + 1, (w + 2 * pad - k) // stride + 1
        sdy, sx, sw, at, dx, dw = (b, o, oh, ow), (b, c, h, w), (o, c, k, k), dict(stride=(stride, stride), pad=(pad, pad)), "conv2d_grad_x", "conv2d_grad_w"
    dy, wv, x = g.input("dy", dtype, sdy), g.param("w", dtype, sw), g.input("x", dtype, sx)
    data = {"dy": W.as_dtype(rng.standard_normal(sdy), dtype), "x": W.as_dtype(rng.standard_normal(sx), dtype), "w": W.as_dtype(rng.standard_normal(sw) / np.prod(sw[1:]) ** 0.5, dtype)}
    out = []
    for which in ((dw, dx) if weights_first else (dx, dw)):
        o_, (y,) = g.op(which, [dy, wv] if which == dx else [dy, x], [(dtype, sx)] if which == dx else [("f32", sw)], **(at if which == dx else dict(at, out_dtype="f32")))
        g.group([o_])
        out.append(y)
    if inner:                                           # dx goes on to a group of its own: stored channel-last
        at_dx = 1 if weights_first else 0
        o_, (out[at_dx],) = g.op("neg", [out[at_dx]], [(dtype, sx)]); g.group([o_])
    for y in out:
        g.output(y)
    return g, data


PAIR_CASES = [
    # kind   dims                      stride pad weights_first inner
    ("dense", (512, 1000, 784), 1, 0, False, False),      # one slice; f32: the other contraction cut along K as well
    ("dense", (2050, 136, 72), 1, 0, True, False),        # slices; the other order
    ("conv", (8, 64, 20, 19, 64, 3), 1, 1, False, False),     # taps inside a K tile, result in Shape order
    ("conv", (9, 40, 17, 21, 72, 3), 1, 1, False, True),      # K tiles across taps, result kept channel-last
    ("conv", (24, 64, 14, 14, 128, 1), 1, 0, True, False),    # one tap: rows as they lie
    ("conv", (6, 40, 33, 29, 64, 3), 2, 1, False, False),     # stride 2: dy spread out beside dy as it is
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", PAIR_CASES, ids=[f"pair{i}" for i in range(len(PAIR_CASES))])
def test_both_gradients_of_a_layer_in_one_launch(dtype, case):
    import numpy as np
    kind, dims, stride, pad, weights_first, inner = case
    spec, data = layer_backward(kind, dims, dtype, stride, pad, weights_first, inner)
    opts = {"no_direct": 1, "no_lp": 1}                # bf16 too on the direct-load kernel
    ks = steps_of(spec, opts)
    together = [k for k in ks if " | " in k and "_rows" in k and "_dma" in k]
    assert len(together) == 1 and "(launched with the step before)" in ks, ks
    check(spec, data, dtype, f"both gradients {case} {dtype}", opts)
    first, _ = run_hip(spec, data, opts=opts)
    again, _ = run_hip(spec, data, opts=opts)
    for v in spec.outputs:
        np.testing.assert_array_equal(first[v], again[v])
    assert not any(" | " in k for k in steps_of(spec, dict(opts, no_pair=1)))


# ---- two changes of layout in one launch -------------------------------------------------------------------------------------------
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shapes", [((3, 40, 16, 24), (2, 64, 56, 8)), ((1, 8, 4, 2), (5, 33, 7, 9)), ((2, 31, 29, 3), (1, 1000, 1, 72)), ((9, 24, 28, 28), (70, 3, 5, 5))])
def test_two_changes_of_layout_in_one_launch(dtype, shapes):
    # whole vectors and ragged tiles, either first, sizes far apart: every element, bit for bit
    import numpy as np
    rng = np.random.default_rng(8)
    g = W.GraphSpec("moves")
    data, want = {}, []
    for i, shape in enumerate(shapes):
        data[f"x{i}"] = W.as_dtype(rng.standard_normal(shape), dtype)
        o, (y,) = g.op("layout_transform", [g.input(f"x{i}", dtype, shape)], [(dtype, (shape[0], shape[2], shape[3], shape[1]))], perm=(0, 2, 3, 1))
        g.group([o]); g.output(y)
    assert steps_of(g) == ["transpose_tiled | transpose_tiled", "(launched with the step before)"] and steps_of(g, {"no_pair": 1}) == ["transpose_tiled"] * 2, steps_of(g)
    ref = OG.run(g, data)
    for opts in ({}, {"no_pair": 1}):
        got, _ = run_hip(g, data, opts=opts)
        for v in g.outputs:
            np.testing.assert_array_equal(got[v], ref[v])


# ---- 3x3 weight gradients with the taps of a filter row from one copy of the rows (igemm_tn_run.hip) ---------------------------------
TN_RUN_CASES = [
    # n  c    h   w   o
    (4, 64, 16, 16, 64),        # every size whole: one tile of channels, whole K tiles
    (5, 40, 17, 19, 72),        # channels past the tile on both sides, a last K tile of 15 pixels, images that end inside a K tile
    (40, 64, 33, 1, 64),        # one column: kw = 1 alone is inside the image
    (5, 136, 2, 131, 64),       # rows longer than two K tiles, every line at an edge
    (1, 24, 40, 35, 200),       # one image
    (70, 72, 5, 6, 40),         # lines and images shorter than a wave's pixels
]


@pytest.mark.parametrize("case", TN_RUN_CASES, ids=[f"tn_run{i}" for i in range(len(TN_RUN_CASES))])
def test_weight_gradient_with_a_filter_rows_taps_from_one_copy(case):
    import numpy as np
    n, c, h, w, o = case
    for slices in (2, 5, 512):                          # one or many K tiles a slice: shorter and longer than the ring of stages
        for out_dtype in ("f32", None):
            spec, data = W.grad_case("conv2d_grad_w", (n, c, h, w, o, 3), "bf16", 1, 1, second_is_param=False, out_dtype=out_dtype)
            opts = {"tn_run": slices}
            assert any("64x64x3_rows_run" in k for k in steps_of(spec, opts)), steps_of(spec, opts)
            check(spec, data, "bf16", f"tn_run {case} {slices} {out_dtype}", opts)
            if out_dtype == "f32":
                first, _ = run_hip(spec, data, opts=opts)
                again, _ = run_hip(spec, data, opts=opts)
                for v in spec.outputs:
                    np.testing.assert_array_equal(first[v], again[v])


# ---- results of the pixel-on-lane kernels stored in Shape order (lp_planes.h) --------------------------------------------------------
PLANES_CASES = [
    # n   c    h   w   o    k  s  p  options
    (16, 64, 28, 28, 128, 3, 1, 1, {}),                 # nine taps from one copy of the rows, whole tiles
    (25, 320, 20, 20, 40, 3, 1, 1, {}),
    (16, 128, 28, 28, 128, 3, 1, 1, {}),                # in place of K split over the waves
    (70, 64, 30, 58, 512, 1, 1, 0, {}),                 # in place of 256x256 tiles
    (9, 64, 22, 26, 200, 3, 1, 1, {}),                  # images that end inside a wave's pixels, channels past the tile, a ragged last tile
    (50, 256, 14, 14, 264, 3, 1, 1, {}),                # 196 pixels: four at a time and no more
    (64, 128, 28, 28, 128, 3, 1, 1, {}),
    (5, 64, 36, 33, 72, 3, 1, 1, {}),                   # rows too long for one copy
    (33, 192, 30, 30, 136, 1, 1, 0, {}),
    (17, 128, 31, 29, 256, 3, 2, 1, {}),                # 16 x 15
    (16, 128, 28, 28, 128, 3, 1, 1, {"no_run": 1}),
    (301, 256, 2, 2, 512, 3, 1, 1, {"no_run": 1}),      # images of four pixels
    (301, 256, 2, 2, 512, 3, 1, 1, {}),
]


@pytest.mark.parametrize("steps", ["none", "bias", "bias_relu", "bias_residual_relu", "residual"])
@pytest.mark.parametrize("case", PLANES_CASES, ids=[f"planes{i}" for i in range(len(PLANES_CASES))])
def test_result_stored_in_shape_order(case, steps):
    import numpy as np
    n, c, h, w, o, k, s, p, opts = case
    oh, ow = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
    rng = np.random.default_rng(n + o)
    g = W.GraphSpec("conv")
    x, wv, b = g.input("x", "bf16", (n, c, h, w)), g.param("w", "bf16", (o, c, k, k)), g.param("b", "f32", (o,))
    t = [("bf16", (n, o, oh, ow))]
    ops = [g.op("conv2d", [x, wv], t, stride=(s, s), pad=(p, p))]
    if "bias" in steps:
        ops.append(g.op("bias_add", [ops[-1][1][0], b], t, axis=1))
    if "residual" in steps:
        ops.append(g.op("add", [ops[-1][1][0], g.input("r", "bf16", (n, o, oh, ow))], t))
    if "relu" in steps:
        ops.append(g.op("relu", [ops[-1][1][0]], t))
    g.group([q[0] for q in ops])
    g.output(ops[-1][1][0])
    data = {"x": W.as_dtype(rng.standard_normal((n, c, h, w)), "bf16"), "w": W.as_dtype(rng.standard_normal((o, c, k, k)) / (c * k * k) ** 0.5, "bf16"),
            "b": rng.standard_normal(o).astype(np.float32), "r": W.as_dtype(rng.standard_normal((n, o, oh, ow)), "bf16")}
    data = {q: data[q] for q in data if q != "r" or "residual" in steps}
    from paper_1810_00952_amd import binding
    order = lambda o: [q.get("shape_order", 0) for q in binding.Plan(binding.graph_from_spec(binding.Context(), g), o).describe()["steps"]]
    assert 1 in order(opts) and 1 in order(dict(opts, no_pair=1)) and 1 not in order(dict(opts, no_shape_order=1)), steps_of(g, opts)
    print(case, steps_of(g, opts), flush=True)
    got, _ = run_hip(g, data, opts=opts)
    # rows of channels, then the transposition: the same sums and rounding, K not split over the waves, and the same tiles
    rows, _ = run_hip(g, data, opts=dict(opts, no_shape_order=1, no_run_ks=1))
    other_tiles = any("256x256" in q for q in steps_of(g, dict(opts, no_shape_order=1)))
    if other_tiles:
        assert_close(got[g.outputs[0]], rows[g.outputs[0]], "bf16", f"planes against rows {case} {steps}")      # other sums
    else:
        np.testing.assert_array_equal(got[g.outputs[0]], rows[g.outputs[0]])
    if n * c * h * w * o < 2e8 or (other_tiles and steps in ("bias_relu", "bias_residual_relu")):
        check(g, data, "bf16", f"planes {case} {steps}", opts)
