"""GPU parity of the kernels on shapes where their index arithmetic can go wrong: image widths and heights that
do not tile a token tile, odd widths, channel counts that leave a chunk partly empty, ragged token counts.

Every element of Y is compared with the fp64 oracle, by infinity-norm relative error and by the per-element
rounding bound of the path's arithmetic; a second forward must give the same bits.
"""
import numpy as np
import pytest
import torch

import oracle as O
from parity_checks import check_against_oracle, sampled_outputs
from workloads import ConvGeom, LayerSpec, generate

pytestmark = pytest.mark.gpu

TOL = 2e-3


def _conv(name, n, cin, C_out, k, H, W, stride=1, M=2, B=8, **kw):
    geom = ConvGeom(cin, k, k, stride, (k - 1) // 2, H, W)
    return LayerSpec(name=name, C_out=C_out, K=geom.K, g=8, M=M, B=B, n=n, conv=geom, **kw)


def _forward(spec, inp, opts=None):
    import paper_2506_05960_amd as P
    layer = P.AQLayer(spec, inp)
    for k, v in (opts or {}).items():
        layer.set_option(k, v)
    route = layer.describe(spec.n)
    print(spec.name, opts or {}, route, flush=True)
    x = torch.from_numpy(np.ascontiguousarray(inp["x"])).cuda()
    y, y2 = layer.forward(x), layer.forward(x)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    layer.close()
    return y.float().cpu().numpy().astype(np.float64), route


def _check(spec, inp, y):
    tok, ch = np.arange(spec.tokens), np.arange(spec.C_out)
    check_against_oracle(spec, inp, sampled_outputs(spec, y, tok, ch), tok, ch, "decode", TOL)


UNEVEN = [
    _conv("u24", 2, 32, 64, 3, 24, 24),                       # rows that start mid-tile, one image border per tile
    _conv("u24_m4_long", 1, 256, 96, 3, 24, 24, M=4),         # a K split over a partial last tile
    _conv("u72", 1, 16, 40, 3, 6, 72),                        # rows longer than a tile
    _conv("u10", 5, 48, 72, 3, 10, 10),                       # two image borders in one tile, planes not a multiple of 8
    _conv("u9_odd", 3, 16, 33, 3, 9, 9),                      # odd width, planes not a multiple of 4
    _conv("u25x31_odd", 2, 24, 64, 3, 25, 31),                # odd width, a half-empty last chunk
    _conv("u13x15_s2", 3, 64, 48, 3, 13, 15, stride=2),       # odd width, stride 2
    _conv("u7x2", 4, 8, 16, 3, 7, 2),                         # the narrowest width, half a chunk in all
    _conv("u40x132", 1, 16, 64, 3, 40, 132),                  # the most staged pixels per lane
    _conv("u36_rec", 4, 64, 256, 3, 36, 36, M=1),             # records only
    _conv("u28_b16", 2, 48, 64, 3, 28, 28, M=1, B=16),        # codewords from memory
    _conv("u1x1_24", 3, 80, 96, 1, 24, 24),                   # 1x1, a partly empty chunk, planes of 64-pixel rows
    _conv("u1x1_odd", 2, 136, 64, 1, 15, 17),                 # 1x1, odd planes
    _conv("u1x1_10", 7, 40, 50, 1, 10, 10, M=4),              # 1x1, 4-pixel rows
    _conv("u48_wide", 8, 48, 256, 3, 48, 48, y_dtype="f32"),  # enough tiles for the wave-split kernel
    _conv("u1x1_wide", 12, 144, 192, 1, 54, 52),
]


@pytest.mark.parametrize("spec", UNEVEN, ids=lambda s: s.name)
@pytest.mark.parametrize("weights", [0, 1, 2])
def test_uneven_convolutions(spec, weights):
    inp = generate(spec, 7001)
    y, route = _forward(spec, inp, {"weights": weights})
    # (forced to decode in its loop, the fused kernel stages fewer pixels than the longest and odd 1x1 rows need)
    assert route["route"] in ("fused", "rec-conv") or weights == 1
    _check(spec, inp, y)
    if weights == 0:
        y_gen, route = _forward(spec, inp, {"generic": 1})
        assert route["route"] == "generic"
        _check(spec, inp, y_gen)


@pytest.mark.parametrize("spec", [
    _conv("w8x8", 64, 16, 736, 3, 8, 8),                      # 192 tiles, the fewest; a partial channel tile, a half-empty chunk
    _conv("w8x8_b12", 64, 16, 736, 3, 8, 8, M=1, B=12),        # records only
    _conv("w4x4", 256, 32, 768, 3, 4, 4, M=4),                # 8 images to a tile
    _conv("w8x8_s2", 64, 32, 768, 3, 16, 16, stride=2, y_dtype="f32"),
    _conv("w4x4_192", 512, 16, 768, 3, 4, 4),                 # 256 tiles of 192 channels instead of 384 of 128
], ids=lambda s: s.name)
def test_narrow_images_on_the_wave_split_kernel(spec):
    inp = generate(spec, 7004)
    y, route = _forward(spec, inp)
    assert route["route"] == "rec-conv" and route["tile"] == ("128x192" if spec.name.endswith("_192") else "128x128")
    _check(spec, inp, y)


def test_uneven_convolution_static_and_limits():
    """The allocation-free forward gives the forward's bits; g = 9 on an odd width stays refused."""
    import paper_2506_05960_amd as P
    spec = UNEVEN[0]
    inp = generate(spec, 7002)
    layer = P.AQLayer(spec, inp)
    x = torch.from_numpy(inp["x"]).cuda()
    assert torch.equal(layer.forward(x), layer.forward(x, static=True))
    layer.close()
    g9 = LayerSpec(name="g9_24", C_out=64, K=32 * 9, g=9, M=2, B=8, n=1, conv=ConvGeom(32, 3, 3, 1, 1, 24, 24))
    layer = P.AQLayer(g9, generate(g9, 7003))
    with pytest.raises(P.AQError) as e:
        layer.forward(torch.zeros((1, 32, 24, 24), dtype=torch.float16, device="cuda"))
    assert e.value.status == 2
    layer.close()


def _bf16(name, n, K, C_out, M=2, B=8, cb="bf16", y="f32"):
    return LayerSpec(name=name, C_out=C_out, K=K, g=8, M=M, B=B, n=n, codebook_dtype=cb, x_dtype="bf16", y_dtype=y,
                     tile_dtype="bf16")


BF16 = [
    _bf16("b_1", 1, 64, 64),
    _bf16("b_ragged", 77, 200, 131, M=2, B=6),                # a partial chunk, a C_out that is no multiple of 4
    _bf16("b_m4_splitk", 130, 2304, 96, M=4),                 # a K split
    _bf16("b_m3", 70, 136, 72, M=3),                          # records, M loop
    _bf16("b_m1_b12", 65, 64, 68, M=1, B=12),                 # 16-bit codes
    _bf16("b_cb16", 90, 264, 100, M=1, cb="f16", y="f16"),
    _bf16("b_cb32", 90, 264, 100, M=2, cb="f32", y="f16"),
    _bf16("b_wide", 2100, 128, 1664, y="f16"),                # enough tiles for the wave-split linear kernel
]


@pytest.mark.parametrize("spec", BF16, ids=lambda s: s.name)
@pytest.mark.parametrize("weights", [0, 2])
def test_bf16_linear(spec, weights):
    """bf16 linear layers against the 64-bit product of the inputs and the decode's rounded weights (host
    emulation): within the rounding of an fp32 sum of K exact products and the two scalings, |dY| <= 4 K 2^-24
    sum |x w|, plus that of an fp16 output; the generic kernel, on the same weights, within twice that."""
    import paper_2506_05960_amd as P
    inp = generate(spec, 7101)
    xb = torch.from_numpy(inp["x"].view(np.int16)).cuda().view(torch.bfloat16)
    layer = P.AQLayer(spec, inp)
    layer.set_option("lut_max_tokens", -1)
    layer.set_option("weights", weights)
    route = layer.describe(spec.n)
    print(spec.name, weights, route, flush=True)
    assert route["route"] in ("fused", "rec-linear")
    y, y2 = layer.forward(xb), layer.forward(xb)
    assert torch.equal(y, y2)
    assert torch.equal(y, layer.forward(xb, static=True))
    layer.set_option("generic", 1)
    assert layer.describe(spec.n)["route"] == "generic"
    y_gen = layer.forward(xb)
    w = O.decode_emulate(inp["codebooks"], inp["codes"], inp["scales"], 8, spec.codebook_dtype, "bf16", scaled=False)
    w = torch.from_numpy(w.view(np.int16)).cuda().view(torch.bfloat16).double() * torch.from_numpy(
        inp["scales"]).cuda().double()[:, None]
    bound = 4 * spec.K * 2.0**-24 * (xb.double().abs() @ w.abs().t())
    ref = xb.double() @ w.t()
    if spec.y_dtype == "f16":
        bound = bound + 2.0**-11 * ref.abs() + 2.0**-24
    assert torch.all((y.double() - ref).abs() <= bound)
    assert torch.all((y.double() - y_gen.double()).abs() <= 2 * bound)
    layer.close()


@pytest.mark.parametrize("tile,split,dt,y", [
    ("64x96", 1, "f16", "f16"), ("64x64", 2, "f16", "f32"), ("32x128", 2, "f16", "f16"), ("32x64", 1, "f16", "f32"),
    ("64x96", 2, "bf16", "f32"), ("32x128", 1, "bf16", "f16"),
])
def test_unaligned_output_rows(tile, split, dt, y):
    """Outputs whose rows are no multiple of 16 bytes leave through LDS: the bits are those of the same channels in
    a layer of whole rows, and nothing is written past the last one."""
    import paper_2506_05960_amd as P
    wide = LayerSpec(name="rows_136", C_out=136, K=840, g=8, M=2, B=8, n=77, codebook_dtype=dt, x_dtype=dt, y_dtype=y, tile_dtype=dt)
    inp = generate(wide, 7111)
    x = torch.from_numpy(inp["x"].view(np.int16)).cuda().view(torch.bfloat16) if dt == "bf16" else torch.from_numpy(inp["x"]).cuda()
    outs = []
    for C_out in (136, 131, 7):
        spec = LayerSpec(**{**wide.__dict__, "name": f"rows_{C_out}", "C_out": C_out})
        layer = P.AQLayer(spec, {**inp, "codes": inp["codes"][:C_out], "scales": inp["scales"][:C_out]})
        layer.set_path("decode")
        for k, v in {"weights": 1, "fused_tile": tile, "split_k": split}.items():
            layer.set_option(k, v)
        d = layer.describe(spec.n)
        assert d["route"] == "fused" and d["tile"] == tile and (C_out == 7 or d["split_k"] == str(split))
        buf = torch.full((spec.n * C_out + 64,), 9.0, dtype=torch.float16 if y == "f16" else torch.float32, device="cuda")
        layer.forward(x, out=buf[:spec.n * C_out].view(spec.n, C_out))
        assert bool((buf[spec.n * C_out:] == 9.0).all())
        outs.append(buf[:spec.n * C_out].view(spec.n, C_out))
        layer.close()
    assert torch.equal(outs[1], outs[0][:, :131])
    if split == 1:
        assert torch.equal(outs[2], outs[0][:, :7])


def _f32(name, n, K, C_out, g=8, M=2, B=8, x="f32", conv=None, y="f32"):
    return LayerSpec(name=name, C_out=C_out, K=K, g=g, M=M, B=B, n=n, codebook_dtype="f32", x_dtype=x, y_dtype=y,
                     tile_dtype="f32", conv=conv)


F32 = [
    _f32("s_1", 1, 8, 1),                                     # one step, one output
    _f32("s_k24", 33, 24, 33),                                # fewer steps than waves
    _f32("s_k264", 70, 264, 40, M=3, B=5),                    # a last wave with fewer steps
    _f32("s_g3", 40, 27, 50, g=3),                            # groups across lanes, rows not 16-byte multiples
    _f32("s_g16", 20, 48, 30, g=16, M=1, B=12),               # 16-bit codes
    _f32("s_wide", 600, 200, 500, M=4),                       # four waves per tile
    _f32("s_wide_g9", 520, 90, 512, g=9, B=6),
    _f32("s_i8", 50, 64, 40, x="i8", y="f16"),
    _f32("s_bf16", 50, 64, 40, x="bf16"),
    _f32("s_conv", 2, 12 * 9, 36, g=4, conv=ConvGeom(12, 3, 3, 2, 1, 9, 7)),
    _f32("s_conv_m1", 3, 24 * 9, 70, M=1, conv=ConvGeom(24, 3, 3, 1, 1, 9, 11)),     # a chunk that ends in its first half
    _f32("s_conv1_s2", 3, 40, 36, M=4, conv=ConvGeom(40, 1, 1, 2, 0, 11, 7)),
    # short reductions in many tiles: the tile kernel, partial tiles on both edges
    _f32("t_k8", 1001, 8, 715),
    _f32("t_k24", 1280, 24, 1025, M=1, y="f16"),
    _f32("t_g3", 1290, 27, 1030, g=3, B=5),
    _f32("t_i8", 1300, 40, 970, M=3, x="i8"),
    _f32("t_conv", 3, 8 * 9, 460, M=1, conv=ConvGeom(8, 3, 3, 1, 1, 25, 33)),
    _f32("t_conv1", 5, 32, 300, M=2, B=10, conv=ConvGeom(32, 1, 1, 2, 0, 51, 49)),
]


@pytest.mark.parametrize("spec", F32, ids=lambda s: s.name)
def test_f32_kernel(spec):
    """fp32 layers against the oracle on every output: 1e-5 (fp32 output) and the rounding bound."""
    import paper_2506_05960_amd as P
    inp = generate(spec, 7201)
    layer = P.AQLayer(spec, inp)
    layer.set_path("decode")
    x = torch.from_numpy(inp["x"].view(np.int16) if spec.x_dtype == "bf16" else inp["x"]).cuda()
    xs = None if inp["x_scales"] is None else torch.from_numpy(inp["x_scales"]).cuda()
    y, y2 = layer.forward(x, xs), layer.forward(x, xs)
    print(spec.name, layer.last_launches(), flush=True)
    assert torch.equal(y, y2)
    layer.close()
    tok, ch = np.arange(spec.tokens), np.arange(spec.C_out)
    check_against_oracle(spec, inp, sampled_outputs(spec, y.double().cpu().numpy(), tok, ch), tok, ch, "decode",
                         1e-5 if spec.y_dtype == "f32" else TOL)


def test_f32_infinite_codeword():
    """A codeword that no code of a row selects does not reach that row, whatever steps its waves share."""
    import paper_2506_05960_amd as P
    spec = _f32("s_inf", 5, 24, 40, M=1, B=2)
    inp = generate(spec, 7202)
    inp["codebooks"][0, 3] = np.inf
    inp["codes"][:, :, 0] = inp["codes"][:, :, 0] % 3
    inp["codes"][7, 2, 0] = 3
    layer = P.AQLayer(spec, inp)
    layer.set_path("decode")
    inp["x"][:, 16:] = np.abs(inp["x"][:, 16:])
    y = layer.forward(torch.from_numpy(inp["x"]).cuda()).cpu().numpy()
    layer.close()
    assert np.all(np.isposinf(y[:, 7])) and np.all(np.isfinite(np.delete(y, 7, axis=1)))


def test_f32_more_tiles_than_one_grid_row():
    """1050624 tiles: the last ones, in the grid's second row, and the first against the 64-bit product."""
    import paper_2506_05960_amd as P
    spec = _f32("s_grid", 65600, 200, 32800, M=1, B=8, y="f16")
    rng = np.random.default_rng(7203)
    inp = {"codebooks": rng.standard_normal((1, 256, 8)).astype(np.float32),
           "codes": rng.integers(0, 256, (spec.C_out, 25, 1), dtype=np.uint8),
           "scales": rng.uniform(0.5, 1.5, spec.C_out).astype(np.float32)}
    x = torch.from_numpy(rng.standard_normal((spec.n, spec.K)).astype(np.float32)).cuda()
    layer = P.AQLayer(spec, inp)
    layer.set_path("decode")
    y = layer.forward(x)
    assert layer.last_launches()[1][0].startswith("f32_fwd_kernel")
    w = torch.from_numpy(inp["codebooks"][0][inp["codes"][:, :, 0]].reshape(spec.C_out, spec.K) * inp["scales"][:, None]).cuda().double()
    for rows in (slice(0, 40), slice(spec.n // 2, spec.n // 2 + 40), slice(spec.n - 80, spec.n)):
        ref = x[rows].double() @ w.t()
        assert torch.all((y[rows].double() - ref).abs() <= 2.0**-11 * ref.abs() + 2.0**-24 + 2e-6 * (x[rows].double().abs() @ w.abs().t()))
    layer.close()


def _glin(name, C_out, K, n, M=2, B=8):
    return LayerSpec(name=name, C_out=C_out, K=K, g=8, M=M, B=B, n=n)


GRAD = [
    # (layer, dtype, options): the 128 x 192 linear tile forced on edges of its tile, of a token chunk and of a split
    (_glin("gw_one_tile", 128, 192, 64), "f16", {"grad_tile": "128x192"}),
    (_glin("gw_less", 8, 8, 1), "bf16", {"grad_tile": "128x192"}),
    (_glin("gw_edges", 136, 200, 65), "f16", {"grad_tile": "128x192"}),
    (_glin("gw_long", 264, 392, 700, M=4), "bf16", {"grad_tile": "128x192"}),
    (_glin("gw_auto", 1160, 584, 1500, M=1), "f16", {}),
    # convolutions with few tiles (two waves' token halves) and many, whole and ragged tiles
    (_conv("gc_few", 2, 24, 40, 3, 16, 16), "f16", {}),
    (_conv("gc_one_chunk", 1, 8, 8, 3, 8, 8), "bf16", {}),
    (_conv("gc_w64", 1, 16, 72, 3, 4, 64, M=1), "f16", {}),
    (_conv("gc_1x1", 3, 88, 72, 1, 16, 16, M=4), "bf16", {}),
    (_conv("gc_many", 1, 352, 1032, 3, 8, 8, M=1), "f16", {}),
    # rows of K that are not whole 16-byte pieces (g = 9, odd channel count)
    (LayerSpec(name="gc_k_odd", C_out=40, K=27 * 9, g=9, M=2, B=6, n=2, conv=ConvGeom(27, 3, 3, 1, 1, 8, 8)), "f16", {}),
]


@pytest.mark.parametrize("spec,dt,opts", GRAD, ids=lambda v: getattr(v, "name", None))
def test_codebook_gradient_tiles(spec, dt, opts):
    """Codebook gradients against the oracle, bar as in the gradient's own tests (2e-5, fp32 sums)."""
    import paper_2506_05960_amd as P
    from workloads import generate_grad_inputs
    inp, gi = generate(spec, 7301), generate_grad_inputs(spec, 7302, dt)
    layer = P.AQLayer(spec, inp)
    for k, v in opts.items():
        layer.set_option(k, v)
    dev = [torch.from_numpy(gi[k].view(np.int16)).cuda().view(torch.bfloat16) if dt == "bf16"
           else torch.from_numpy(gi[k]).cuda() for k in ("x", "dy")]
    a, b = layer.codebook_grad(*dev), layer.codebook_grad(*dev)
    print(spec.name, layer.last_launches(), flush=True)
    assert torch.equal(a, b)
    layer.close()
    ref = O.codebook_grad(spec, {"codes": inp["codes"], "scales": inp["scales"], "x": gi["x"]}, gi["dy"], x_dtype=dt,
                          dy_dtype=dt)
    assert O.rel_err_inf(a.double().cpu().numpy(), ref) <= 2e-5


FEW = [
    # (C_out, K, M, B, tokens, x dtype, y dtype)
    (1, 8, 1, 8, 1, "f16", "f32"),            # one group
    (5, 128, 2, 8, 1, "f16", "f16"),          # a partial row tile, one whole chunk
    (70, 136, 2, 4, 2, "i8", "f32"),          # a chunk past K, few codewords
    (33, 264, 4, 8, 3, "f16", "f32"),         # three tokens in four slots
    (300, 1000, 4, 6, 4, "i8", "f16"),
    (130, 16384, 1, 8, 4, "f16", "f32"),      # exactly as many chunks as lanes
    (40, 17280, 4, 8, 1, "f16", "f32"),       # several rounds of codes per lane
    (24, 40960, 2, 8, 1, "f16", "f32"),       # more rounds than are loaded ahead
    (20, 65536, 2, 8, 1, "f16", "f32"),       # the largest K that fits LDS, nearly
    (1541, 520, 2, 8, 4, "f16", "f32"),       # eight rows per workgroup, a partial tile
    (3077, 264, 4, 8, 2, "i8", "f16"),        # sixteen
    (1030, 13152, 1, 8, 4, "i8", "f16"),      # eight, as LDS holds one workgroup of more than 256
    (2060, 13152, 1, 8, 3, "f16", "f32"),     # sixteen, likewise
    (4100, 264, 4, 8, 4, "f16", "f32"),       # more rows than sixteen per unit
]


@pytest.mark.parametrize("case", FEW, ids=lambda c: "x".join(str(v) for v in c))
def test_few_token_kernel(case):
    """One to four tokens: every output against the oracle and the table path's bound (fp32 products and sums)."""
    import paper_2506_05960_amd as P
    C_out, K, M, B, n, xd, yd = case
    spec = LayerSpec(name="few", C_out=C_out, K=K, g=8, M=M, B=B, n=n, x_dtype=xd, y_dtype=yd)
    inp = generate(spec, 7401)
    layer = P.AQLayer(spec, inp)
    layer.set_option("lut_max_tokens", 4)      # the table path's token count: the kernel replaces it
    x = torch.from_numpy(inp["x"]).cuda()
    xs = None if inp["x_scales"] is None else torch.from_numpy(inp["x_scales"]).cuda()
    assert layer.describe(n)["route"] == "few-token"
    y, y2 = layer.forward(x, xs), layer.forward(x, xs)
    print(case, layer.last_launches(), flush=True)
    assert torch.equal(y, y2) and torch.equal(y, layer.forward(x, xs, static=True))
    tok, ch = np.arange(n), np.arange(C_out)
    check_against_oracle(spec, inp, y.double().cpu().numpy(), tok, ch, "lut", 1e-5 if yd == "f32" else TOL)
    layer.set_path("lut")                      # the table kernels stay behind their path
    assert layer.describe(n)["route"] == "table"
    layer.close()


def test_few_token_infinite_codeword():
    """The codeword that pads a last chunk does not reach a row that does not select it."""
    import paper_2506_05960_amd as P
    spec = LayerSpec(name="few_inf", C_out=9, K=24, g=8, M=1, B=2, n=2, y_dtype="f32")
    inp = generate(spec, 7402)
    inp["codebooks"][0, 0] = np.inf
    inp["codes"][:, :, 0] = 1 + inp["codes"][:, :, 0] % 3
    inp["codes"][4, 1, 0] = 0
    inp["x"][:] = np.abs(inp["x"]) + 1
    layer = P.AQLayer(spec, inp)
    layer.set_option("lut_max_tokens", 4)
    assert layer.describe(2)["route"] == "few-token"
    y = layer.forward(torch.from_numpy(inp["x"]).cuda()).cpu().numpy()
    layer.close()
    assert np.all(np.isposinf(y[:, 4])) and np.all(np.isfinite(np.delete(y, 4, axis=1)))


PAD = [
    # (M, B, dtype, K): in-loop formats of a linear layer whose last 64-wide chunk is partly empty
    (1, 8, "f16", 72),
    (2, 4, "f16", 200),
    (4, 8, "f16", 56),
    (1, 12, "f16", 72),                       # codewords from memory
    (1, 8, "bf16", 72),
    (2, 8, "bf16", 200),
    (4, 4, "bf16", 88),
]


@pytest.mark.parametrize("weights", [1, 2])
@pytest.mark.parametrize("case", PAD, ids=lambda c: "x".join(str(v) for v in c))
def test_codeword_of_no_row_past_k(case, weights):
    """An infinite or NaN codeword that no code selects reaches no output: not through the codes past K either."""
    import paper_2506_05960_amd as P
    M, B, dt, K = case
    spec = LayerSpec(name="pad", C_out=40, K=K, g=8, M=M, B=B, n=70, codebook_dtype=dt, x_dtype=dt, y_dtype="f32",
                     tile_dtype=dt)
    inp = generate(spec, 7501)
    inp["codes"][inp["codes"] == 0] = 1
    clean = {k: np.copy(v) for k, v in inp.items() if v is not None} | {"x_scales": None}
    inp["codebooks"][:, 0] = np.array([np.inf, -np.inf, np.nan, np.inf] * 2, np.float16) if dt == "f16" else 0x7F80
    x = torch.from_numpy(inp["x"].view(np.int16)).cuda().view(torch.bfloat16) if dt == "bf16" else torch.from_numpy(inp["x"]).cuda()
    ys = []
    for w in (inp, clean):
        layer = P.AQLayer(spec, w)
        layer.set_path("decode")
        layer.set_option("weights", weights)
        d = layer.describe(spec.n)
        print(case, d, flush=True)
        assert d["route"] in ("fused", "rec-linear") and d["weights"].startswith("in-loop" if weights == 1 else "records")
        ys.append(layer.forward(x))
        layer.close()
    assert bool(torch.isfinite(ys[0]).all()) and torch.equal(ys[0], ys[1])


def test_codewords_too_large_to_pad_take_records():
    """No code's padding sum is surely finite: the layer decodes records, which hold zeros past K."""
    import paper_2506_05960_amd as P
    spec = LayerSpec(name="pad_big", C_out=40, K=72, g=8, M=4, B=4, n=70, y_dtype="f32")
    inp = generate(spec, 7502)
    signs = np.array([1.0, -1.0, 1.0, -1.0])[:, None, None]
    inp["codebooks"] = (signs * 30000.0 + 2000.0 * inp["codebooks"].astype(np.float64)).astype(np.float16)
    layer = P.AQLayer(spec, inp)
    layer.set_path("decode")
    layer.set_option("weights", 1)
    assert layer.describe(spec.n)["weights"] == "records"
    y = layer.forward(torch.from_numpy(inp["x"]).cuda()).double().cpu().numpy()
    layer.close()
    tok, ch = np.arange(spec.n), np.arange(spec.C_out)
    check_against_oracle(spec, inp, y, tok, ch, "decode", TOL)
