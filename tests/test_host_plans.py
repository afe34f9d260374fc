"""Routes, limits, refusals and workspaces of calls, planned on the host without a GPU (see host_device.py)."""
import pytest

import host_device as hd


@pytest.fixture(scope="session")
def child(tmp_path_factory):
    so = hd.build(tmp_path_factory)
    return lambda function, *args: hd.in_child(so, "test_host_plans", function, *args)


# ---- weight records past the product kernels' 32-bit byte offsets ----

def _large_records(n, options, kw):
    before = hd.live_bytes()
    layer = hd.Layer(max_n=n, **kw)
    held = hd.live_bytes() - before
    return layer.set(**options).describe(n), layer.forward(n), held


BIG = 131136     # outputs: with K = 8192 the records hold 2.15 GB


@pytest.mark.parametrize("n,options,kw,route,weights", [
    (64, {}, dict(C_out=BIG, K=8192, M=1, B=16, x="bf16", cb="bf16", tile="bf16", y="f32"), "generic", None),
    (64, {}, dict(C_out=BIG, K=8192, M=3, x="bf16", cb="bf16", tile="bf16"), "generic", None),
    (64, {}, dict(C_out=BIG, K=8192, M=3), "generic", None),                            # fp16, records only
    (4, {"weights": 2, "lut_max_tokens": -1}, dict(C_out=BIG, K=8192, M=2, x="i8"), "fused", "in-loop-lds-fp16"),
    (1024, {}, dict(C_out=BIG, K=8192, M=1, B=16), "fused", "in-loop-l2-fp16"),         # records where they fit
    (4, {}, dict(C_out=28800, M=1, B=16, conv=(4352, 3, 1, 1, 16, 16)), "fused", "in-loop-l2-fp16"),
    (64, {}, dict(C_out=131008, K=8192, M=1, B=16, x="bf16", cb="bf16", tile="bf16"), "rec-linear", "records"),   # just below
])
def test_records_past_32_bit_offsets(child, n, options, kw, route, weights):
    """Records of 2 GiB and more are not indexable by the kernels that read them: such layers decode in the loop or,
    where their format has no such decode, run the generic kernel; no buffer is held for records that never exist."""
    d, kernels, held = child("_large_records", n, options, kw)
    assert (d["route"], d.get("weights")) == (route, weights)
    if weights != "records":
        assert kernels == [{"generic": "mfma_fwd_kernel", "fused": "fused_fwd_kernel"}[route]]
        assert held < 2**31


def test_g9_records_past_32_bit_offsets_are_refused(child):
    kw = dict(C_out=28800, M=2, g=9, conv=(4160, 3, 1, 1, 16, 16))
    assert child("_large_records_g9", kw) == "AQ_ERR_UNSUPPORTED"


def _large_records_g9(kw):
    return hd.Layer(max_n=1, **kw).set(lut_max_tokens=-1).forward(1)


# ---- convolutions past the kernels' 24-bit index arithmetic ----

def _conv_limit(n, options, kw):
    return hd.Layer(max_n=n, **kw).set(lut_max_tokens=-1, **options).forward(n)


@pytest.mark.parametrize("n,options,kw,kernels", [
    # 2^25 (image, channel) planes of 2 x 2 pixels, and just below 2^24 of them
    (1 << 19, {}, dict(C_out=64, conv=(64, 1, 1, 0, 2, 2)), ["mfma_fwd_kernel"]),
    ((1 << 18) - 1, {"weights": 1}, dict(C_out=64, conv=(64, 1, 1, 0, 2, 2)), ["fused_fwd_kernel"]),
    # odd widths, as before
    (1 << 20, {}, dict(C_out=8, conv=(16, 3, 2, 1, 3, 3)), ["mfma_fwd_kernel"]),
])
def test_convolutions_past_24_bit_indices(child, n, options, kw, kernels):
    assert child("_conv_limit", n, options, kw) == kernels


# ---- the allocation-free forward's static array ----

def _static(n, kw):
    layer = hd.Layer(max_n=n, **kw)
    return layer.forward(n), layer.forward(n, static=True)


@pytest.mark.parametrize("kw,product", [
    # 65.5 MB of records fit the array's 66.8, the 2 MB of a K split's partial tiles beside them do not
    (dict(C_out=4000, K=8192, M=3), "rec_linear_kernel"),
    (dict(C_out=4000, K=8192, M=3, x="bf16", cb="bf16", tile="bf16"), "rec_linear_kernel"),
    (dict(C_out=3000, K=8192, M=3), "fused_fwd_kernel"),      # both fit
])
def test_static_forward_of_records_only_layers(child, kw, product):
    """A call that the array's records allow is not refused for partial tiles, and takes the forward's kernels."""
    forward, static = child("_static", 8, kw)
    assert forward == static and static[-1] == product


@pytest.mark.parametrize("n,kw,product", [
    # in-loop layers that take records for the wave-split kernel: 3x3 on rows under 16 pixels, and 1x1 on small
    # planes read as longer rows
    (16, dict(C_out=8192, M=2, conv=(512, 3, 1, 1, 8, 8)), "fused_fwd_kernel"),       # 75 MB of records
    (16, dict(C_out=2048, M=2, conv=(512, 3, 1, 1, 8, 8)), "fused_fwd_kernel"),       # 19 MB, too few tiles
    (24, dict(C_out=2048, M=2, conv=(512, 3, 1, 1, 8, 8)), "rec_conv_kernel"),
    (256, dict(C_out=8192, M=2, conv=(4160, 1, 1, 0, 8, 8)), "fused_fwd_kernel"),     # 68 MB
    (256, dict(C_out=2048, M=2, conv=(1024, 1, 1, 0, 8, 8)), "rec_conv_kernel"),      # 4 MB
])
def test_static_forward_of_layers_switched_to_records(child, n, kw, product):
    forward, static = child("_static", n, kw)
    assert forward == static and static[-1] == product


# ---- a forward allocates nothing ----

def _allocations(static):
    counts = []
    for n, kw in ((64, dict(C_out=256, K=256, x="f32", y="f32", cb="f32", tile="f32")), (1, dict(C_out=960, K=8640)),
                  (2, dict(C_out=192, conv=(192, 3, 1, 1, 64, 64))), (512, dict(C_out=1728, K=576, x="i8"))):
        hd.Layer(max_n=n, **kw).forward(n, static=static)      # the process's first use of these kernels
        layer = hd.Layer(max_n=n, **kw)
        before = hd.news()
        f = layer.aq.aq_layer_forward_static if static else layer.aq.aq_layer_forward
        f(layer.handle, 4096, layer.x_scales, 4096, n, 0)
        counts.append(hd.news() - before)
    return counts


@pytest.mark.parametrize("static", [False, True])
def test_first_forward_of_a_layer_allocates_nothing(child, static):
    assert child("_allocations", static) == [0, 0, 0, 0]


# ---- device memory that no route reads is not held ----

def _held(n, kw):
    before = hd.live_bytes()
    hd.Layer(max_n=n, **kw)
    return hd.live_bytes() - before


@pytest.mark.parametrize("n,kw,limit", [
    (4096, dict(C_out=16, conv=(16, 3, 1, 1, 25, 25)), 8e6),      # 82 MB of input, never repacked for the dense product
    (4096, dict(C_out=16, conv=(24, 3, 1, 1, 16, 16)), 8e6),      # 50 MB
    (1, dict(C_out=1024, M=1, B=10, cb="f32", conv=(1024, 3, 1, 1, 25, 25)), 4e6),      # 19 MB of records
    (1, dict(C_out=1024, M=1, B=10, g=9, conv=(1024, 3, 1, 1, 24, 24)), 4e6),
])
def test_device_memory_of_uneven_convolutions(child, n, kw, limit):
    assert child("_held", n, kw) < limit


# ---- choices that were measured ----

def _route(n, kw, options=None):
    d = hd.Layer(max_n=n, **kw).set(**(options or {})).describe(n)
    return [d.get(k) for k in ("route", "weights", "tile", "split_k")]


@pytest.mark.parametrize("M,cin,C_out,side,n,tile,split", [
    (2, 192, 192, 8, 1, "64x64", 3),       # 10.1 us, unsplit 11.1
    (2, 192, 384, 16, 2, "64x64", 3),      # 10.1, 10.7
    (1, 192, 192, 8, 4, "64x64", 3),       # 10.3, 10.5
    (2, 192, 384, 32, 1, "64x64", 1),      # 11.0, three splits 15.8
    (2, 256, 256, 8, 1, "64x64", 4),       # 10.5, two splits 11.2
    (2, 256, 256, 32, 1, "64x64", 2),      # 11.3, four 11.9
    (2, 960, 960, 8, 8, "64x96", 3),       # 21.4, 64 x 64 with two 22.9
    (2, 1920, 960, 8, 8, "64x96", 3),      # 32.1, 128 x 64 with four 34.9
])
def test_splits_of_under_filled_in_loop_convolutions(child, M, cin, C_out, side, n, tile, split):
    route = child("_route", n, dict(C_out=C_out, M=M, conv=(cin, 3, 1, 1, side, side)))
    assert route == ["fused", "in-loop-lds-fp16", tile, str(split)]


@pytest.mark.parametrize("M,cin,C_out,side,n,route", [
    (2, 64, 64, 64, 8, "fused"),          # 10.7 us, by records 13.4: one round of in-loop tiles
    (2, 32, 64, 64, 12, "rec-conv"),      # 13.1, in the loop 18.2
    (1, 16, 96, 64, 64, "rec-conv"),      # 33.7, 88
    (2, 32, 96, 64, 4, "fused"),
    (2, 32, 96, 64, 8, "rec-conv"),       # 11.9, 14.4
    (1, 16, 32, 32, 4, "fused"),          # 6.6, 8.6
    (1, 16, 32, 64, 8, "rec-conv"),       # 7.9, 9.2
])
def test_convolutions_of_few_weights(child, M, cin, C_out, side, n, route):
    got = child("_route", n, dict(C_out=C_out, M=M, conv=(cin, 3, 1, 1, side, side)))
    assert got[:2] == [route, "in-loop-lds-fp16" if route == "fused" else "records"]


def test_strided_convolutions_of_few_weights(child):
    """512 tiles of 64 x 64: by records 10.5 us, in the loop 13.9; 320 tiles: 15.5 and 13.5."""
    assert child("_route", 32, dict(C_out=32, M=2, conv=(32, 3, 2, 1, 64, 64)))[1] == "records"
    assert child("_route", 20, dict(C_out=32, M=2, conv=(32, 3, 2, 1, 64, 64)))[:2] == ["fused", "in-loop-lds-fp16"]


@pytest.mark.parametrize("k,cin,C_out,n,route", [
    (3, 80, 64, 32, "rec-conv"),          # 30.7 us, fused kernel 35.2
    (3, 192, 64, 32, "fused"),            # rec-conv 1.14 times longer
    (1, 576, 32, 16, "rec-conv"),         # 19.3, 23.2
    (1, 960, 64, 16, "fused"),
    (1, 576, 64, 8, "fused"),
])
def test_convolutions_to_few_channels(child, k, cin, C_out, n, route):
    assert child("_route", n, dict(C_out=C_out, M=2, conv=(cin, k, 1, k // 2, 64, 64)))[0] == route


@pytest.mark.parametrize("n,K,C_out,route", [
    (4096, 192, 576, "rec-linear"),       # 8.7 us, in the loop 10.8
    (4096, 2304, 576, "fused"),           # 23.7, by records 25.0
    (1024, 952, 2304, "fused"),           # 16.4, 19.2
    (1024, 192, 2304, "rec-linear"),      # 9.4, 10.8
    (1590, 952, 3456, "rec-linear"),      # 28.5, 31.3
    (3000, 2304, 700, "rec-linear"),      # 26.0, 29.9: rows that are no multiple of 16 bytes
    (1000, 2304, 700, "fused"),           # 12.6, 25.4
])
@pytest.mark.parametrize("x", ["f16", "i8"])
def test_linear_layers_of_one_codebook(child, n, K, C_out, route, x):
    got = child("_route", n, dict(C_out=C_out, K=K, M=1, x=x), {"lut_max_tokens": -1})
    assert got[:2] == [route, "in-loop-lds-fp16" if route == "fused" else "records"]


@pytest.mark.parametrize("n,K,C_out,M,B,route", [
    (1, 64, 1152, 1, 8, "generic"),       # 4.0 us, fused 4.5
    (40, 64, 1152, 1, 8, "fused"),
    (1000, 64, 1152, 3, 8, "generic"),    # 8.4, 9.4
    (1000, 144, 1152, 3, 8, "fused"),     # 10.0, generic 11.2
    (3, 88, 1152, 1, 12, "generic"),      # 4.3, 6.7
    (70, 144, 4608, 1, 12, "generic"),    # 7.4, 8.9
    (4, 304, 1030, 1, 12, "generic"),     # 7.2, 9.0
    (1025, 192, 109, 1, 12, "generic"),   # 7.8, 8.8
    (633, 280, 64, 1, 12, "fused"),       # 8.4, 9.0
    (1, 144, 1472, 3, 4, "generic"),      # 6.8, 8.6
    (2, 240, 630, 3, 4, "fused"),         # 8.4, 9.8
    (361, 144, 3451, 1, 8, "generic"),    # 8.8, 10.2
    (3561, 64, 1007, 2, 8, "generic"),    # 12.6, 19.3
    (9894, 640, 1007, 2, 8, "generic"),   # 57.3, 82.4
    (1000, 640, 1007, 2, 8, "fused"),
    (1000, 2304, 576, 2, 8, "fused"),     # 15.8, 56
])
def test_bf16_linear_layers(child, n, K, C_out, M, B, route):
    kw = dict(C_out=C_out, K=K, M=M, B=B, x="bf16", cb="bf16", tile="bf16", y="f32")
    assert child("_route", n, kw, {"lut_max_tokens": -1})[0] == route


@pytest.mark.parametrize("n,cin,C_out,k,M,side,route,weights", [
    (2, 16, 256, 1, 1, 50, "generic", None),             # 10.2 us, fused 11.0
    (2, 48, 320, 1, 1, 50, "fused", "records"),
    (9, 8, 64, 3, 2, 50, "generic", None),               # 15.0, 18.3
    (2, 8, 64, 3, 2, 50, "fused", "records"),
    (9, 64, 256, 1, 4, 50, "fused", "records"),          # 25.4, in the loop 39.2
    (1, 64, 256, 1, 4, 50, "fused", "in-loop-lds-fp16"),
])
def test_short_reductions_of_uneven_convolutions(child, n, cin, C_out, k, M, side, route, weights):
    got = child("_route", n, dict(C_out=C_out, M=M, conv=(cin, k, 1, k // 2, side, side)))
    assert got[:2] == [route, weights]


@pytest.mark.parametrize("n,k,cin,C_out,H,W,M,B,route", [
    (6, 3, 16, 400, 61, 71, 1, 8, "generic"),        # 59 us, fused 108
    (37, 3, 24, 290, 11, 65, 1, 8, "generic"),       # 52, 84
    (117, 3, 24, 638, 7, 69, 4, 8, "generic"),       # 226, 316
    (80, 3, 16, 720, 7, 41, 1, 12, "generic"),       # 83, 101: two tiles on a compute unit
    (63, 3, 64, 209, 13, 57, 2, 8, "fused"),         # 121, generic 130
    (47, 1, 136, 832, 29, 39, 2, 8, "generic"),      # 202, 359
    (13, 1, 272, 272, 61, 29, 1, 12, "generic"),     # 70, 84
    (25, 1, 400, 304, 13, 33, 2, 8, "fused"),        # 46, 68
    (1, 1, 152, 360, 13, 33, 2, 8, "fused"),         # one round
    (1, 1, 24, 512, 62, 54, 1, 8, "generic"),        # 10.3, 11.0
    (1, 1, 24, 784, 48, 60, 1, 16, "fused"),         # 13.6, 16.0
    (1, 1, 40, 512, 62, 54, 1, 8, "fused"),
])
def test_uneven_convolutions_in_many_tiles(child, n, k, cin, C_out, H, W, M, B, route):
    assert child("_route", n, dict(C_out=C_out, M=M, B=B, conv=(cin, k, 1, k // 2, H, W)))[0] == route


@pytest.mark.parametrize("n,cin,C_out,H,W,M,B,route", [
    (932, 192, 143, 33, 7, 1, 8, "generic"),         # 80 us, fused 110
    (126, 160, 288, 59, 16, 1, 16, "generic"),       # 53, 72
    (71, 104, 468, 9, 32, 1, 16, "fused"),           # 24, 32
])
def test_strided_uneven_convolutions_in_many_tiles(child, n, cin, C_out, H, W, M, B, route):
    assert child("_route", n, dict(C_out=C_out, M=M, B=B, conv=(cin, 1, 2, 0, H, W)))[0] == route


@pytest.mark.parametrize("n,cin,C_out,side,weights", [
    (324, 176, 112, 8, "records"),               # 22.7 us, in the loop 27.9
    (89, 48, 120, 16, "records"),                # 15.0, 17.1
    (78, 48, 88, 16, "in-loop-lds-fp16"),        # 12.8, 14.8: one round of 64 x 96 tiles
    (89, 16, 120, 16, "in-loop-lds-fp16"),
])
def test_convolutions_of_one_codebook(child, n, cin, C_out, side, weights):
    assert child("_route", n, dict(C_out=C_out, M=1, conv=(cin, 3, 1, 1, side, side)))[:2] == ["fused", weights]


@pytest.mark.parametrize("n,K,C_out,M,dt,route,weights", [
    (6270, 144, 1891, 1, "f16", "fused", "records"),           # 38 us, in the loop 63
    (6893, 1616, 1386, 1, "f16", "fused", "records"),          # 74, 89
    (1260, 2712, 4234, 1, "f16", "fused", "in-loop-lds-fp16"),   # 68, 85
    (1250, 152, 806, 1, "f16", "fused", "in-loop-lds-fp16"),     # one round
    (4325, 1144, 2433, 1, "bf16", "fused", "records"),         # 75, 90
    (11162, 672, 197, 4, "bf16", "fused", "records"),          # 20, 42
    (417, 400, 3339, 4, "bf16", "fused", "in-loop-lds-bf16"),  # 14.6, 18.6
    (6976, 1144, 1415, 2, "bf16", "fused", "records"),         # 61, 104
    (6386, 344, 438, 2, "bf16", "fused", "records"),           # 16.4, 21.6
    (1094, 488, 1389, 2, "bf16", "fused", "in-loop-lds-bf16"),   # 13.2, 14.8
    (1174, 728, 4279, 2, "bf16", "fused", "in-loop-lds-bf16"),   # 35, 39
    (1088, 312, 2603, 1, "bf16", "generic", None),             # 17.5, 20.8
])
def test_linear_layers_of_odd_output_rows(child, n, K, C_out, M, dt, route, weights):
    kw = dict(C_out=C_out, K=K, M=M, x=dt, cb=dt, tile=dt, y="f32" if dt == "bf16" else "f16")
    assert child("_route", n, kw, {"lut_max_tokens": -1})[:2] == [route, weights]


@pytest.mark.parametrize("n,K,C_out,M,route", [
    (3, 13392, 2160, 4, "fused"),         # 16.2 us, few-token kernel 26.2
    (4, 4176, 2720, 4, "fused"),          # 11.3, 11.9
    (4, 3912, 2224, 4, "few-token"),      # 10.3, 10.9
    (4, 14184, 1152, 4, "fused"),         # 15.4, 16.8
    (4, 10896, 432, 4, "few-token"),      # 9.9, 13.5
    (4, 17208, 464, 4, "few-token"),      # 13.1, 16.0
    (2, 12400, 2320, 4, "fused"),         # 16.3, 17.1
    (2, 10096, 4048, 4, "few-token"),     # 14.8, 16.9
    (4, 4040, 4288, 2, "fused"),          # 10.1, 11.3
    (4, 5528, 3952, 2, "few-token"),      # 10.0, 17.0
])
@pytest.mark.parametrize("x", ["f16", "i8"])
def test_few_token_layers(child, n, K, C_out, M, route, x):
    assert child("_route", n, dict(C_out=C_out, K=K, M=M, x=x))[0] == route


def _grad(n, kw):
    layer = hd.Layer(**{"max_n": n, **kw})
    kernels, launches = hd.launches(lambda: layer.grad(n, "f16"))
    product = [i for i, k in enumerate(kernels) if k.startswith("wgrad")][0]
    return kernels[product], launches[product - len(kernels)][0]


@pytest.mark.parametrize("n,K,C_out,splits", [
    (7495, 400, 3800, 3),       # 80 us; one split 91, two 93
    (300, 400, 3800, 1),        # 22.9, three 31.5
    (16384, 200, 4608, 8),      # 102, three 119
    (5432, 320, 320, 10),       # 19.6, sixteen 21.0
])
def test_token_splits_of_linear_gradients(child, n, K, C_out, splits):
    kernel, blocks = child("_grad", n, dict(C_out=C_out, K=K))
    tiles = -(-K // 64) * -(-C_out // 64)
    assert kernel.startswith("wgrad_linear_dma_kernel") and blocks == -(-tiles * splits // 8) * 8


@pytest.mark.parametrize("n,k,cin,C_out,H,halves,splits", [
    (16, 1, 360, 696, 64, 1, 11),       # 81 us; the best with eight waves 125
    (9, 1, 360, 696, 64, 1, 11),
    (16, 3, 384, 384, 32, 1, 6),        # 74, eight waves 91
    (16, 3, 192, 192, 64, 1, 16),       # 72, eight waves 80
    (16, 3, 64, 64, 64, 2, 16),         # 52.0, four waves 57.8
    (1, 3, 320, 320, 16, 1, 1),         # 20.3; eight splits 27.6 (512 tokens)
])
def test_waves_and_splits_of_convolution_gradients(child, n, k, cin, C_out, H, halves, splits):
    kw = dict(C_out=C_out, conv=(cin, k, 1, k // 2, H, H))
    kernel, blocks = child("_grad", n, kw)
    tiles = -(-C_out // 64) * -(-cin * k // 64)
    assert kernel.endswith(f"64, {halves}>") and blocks == -(-tiles * splits // 8) * 8
    # the tokens of the call decide, not the most that the layer takes
    assert child("_grad", n, dict(kw, max_n=8 * n)) == [kernel, blocks]


@pytest.mark.parametrize("n,K,C_out,conv,M,g,x,kernel", [
    (16511, 8, 3172, None, 2, 8, "f32", "f32_tile_kernel"),      # 107 us, matrix cores 353
    (5393, 72, 1097, None, 1, 8, "f32", "f32_tile_kernel"),      # 38, 64
    (4554, 24, 338, None, 2, 8, "f32", "f32_tile_kernel"),       # 12.0, 16.4
    (5711, 256, 611, None, 1, 8, "f32", "f32_fwd_kernel"),
    (5000, 40, 600, None, 4, 8, "f32", "f32_fwd_kernel"),
    (2639, 80, 2198, None, 2, 8, "f32", "f32_tile_kernel"),      # 50, 58
    (914, 48, 3844, None, 4, 4, "f32", "f32_tile_kernel"),       # 35, 53
    (1332, 144, 694, None, 4, 16, "f32", "f32_fwd_kernel"),      # 43.6, tiles 48.5
    (3, 0, 675, (64, 1, 1, 0, 40, 49), 2, 8, "f32", "f32_tile_kernel"),
    (3, 0, 675, (64, 1, 1, 0, 40, 49), 4, 8, "f32", "f32_fwd_kernel"),
    (64, 256, 256, None, 2, 8, "f32", "f32_fwd_kernel"),
    (512, 24, 512, None, 2, 8, "f32", "f32_fwd_kernel"),
])
def test_fp32_layers(child, n, K, C_out, conv, M, g, x, kernel):
    kw = dict(C_out=C_out, M=M, g=g, x=x, cb="f32", tile="f32", y="f32", conv=conv)
    assert child("_conv_limit", n, {}, dict(kw, K=K)) == [kernel]


# ---- launches ----

def _f32_large(n, C_out):
    layer = hd.Layer(C_out, 200, M=1, B=4, max_n=n, x="f32", cb="f32", tile="f32").set(lut_max_tokens=-1)
    kernels, launches = hd.launches(lambda: layer.forward(n))
    return kernels, launches[-1]


def test_f32_launch_past_the_threads_of_one_dimension(child):
    """33 million tiles of 256 threads: more than a launch holds along x."""
    kernels, grid = child("_f32_large", 1 << 20, 1 << 16)
    assert kernels == ["f32_fwd_kernel"] and grid[0] * grid[1] >= 1 << 25 and grid[0] * grid[3] < 2**32
