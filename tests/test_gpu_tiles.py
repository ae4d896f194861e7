"""The tile shapes the dispatch chooses between, each on sizes that end inside a tile, a 16-row block, a k-step and (where the k-steps
are dealt out to groups of waves) inside a round of the groups: every element against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import linear as OL
from oracle import projection as OP
from paper_2409_09099_amd import workloads as WL
from test_gpu_parity import bf16_dev, dt, operand, rel_err, sste, TOL, z_to_f64  # noqa: F401

pytestmark = pytest.mark.gpu


def packed_weight(sste, O, I, wdt, beta=np.float32(1.4830322)):
    """(oracle values, oracle positions, scale, GPU values, GPU positions) of one projected weight."""
    wb = WL.weight_bits(WL.WORKLOADS[1], 0, O=O, I=I)
    ws = np.float32(1.0)
    if wdt == "e4m3":
        ws = np.float32(OP.project_pack(wb, beta)[2] / np.float32(448.0))
    rv, rm, _ = OP.project_pack(wb, beta, wdt, ws)
    vals, meta = sste.project_pack(bf16_dev(wb), float(beta), dt(sste, wdt), float(ws))
    return rv, rm, ws, vals, meta


@pytest.mark.parametrize("dtype", ["bf16", "e4m3", "e5m2"])
@pytest.mark.parametrize("T,O,I,tile16,tile8", [
    (200, 48, 64, "64x64 kg 1", "64x64 kg 1"),             # fewer k-steps than the pipeline is deep
    (65, 1040, 64, "64x64 kg 4", "64x64 kg 2"),            # the last round of the groups incomplete; one row in the last tile
    (500, 4112, 128, "64x64 kg 4", "64x64 kg 4"),
    (1100, 1552, 832, "64x64 kg 4", "64x64 kg 2"),
    (20000, 48, 320, "128x128 kg 1", "128x128 kg 1"),      # ragged features
    (5100, 656, 704, "128x128 kg 2", "128x128 kg 2"),
    (9000, 272, 448, "256x128 kg 1", "256x128 kg 1"),
    (4100, 144, 2112, "256x256 kg 1", "256x256 kg 1"),     # 64 features in the last tile
    (16500, 400, 1152, "256x256+256x128 kg 1", "256x256+256x128 kg 1"),       # both axes ragged
])
def test_linear_dgrad_tiles(sste, dtype, T, O, I, tile16, tile8):  # noqa: F811
    if dtype != "bf16" and I % 128:
        I += 64
    assert sste.describe_plan("dgrad", T, O, I, dt(sste, dtype)).startswith((tile16 if dtype == "bf16" else tile8) + " ")
    wl = WL.WORKLOADS[1]
    dyc, dys, dY = operand(sste, WL.output_gradient(wl, 0, T=T, O=O)[0], dtype)
    wdt = "bf16" if dtype == "bf16" else "e4m3"
    rv, rm, ws, vals, meta = packed_weight(sste, O, I, wdt)
    ref = OL.linear_dgrad(dyc, rv, rm, dtype, dys, ws, w_dtype=wdt)
    got = z_to_f64(sste.linear_dgrad(dY, vals, meta, I, dt(sste, dtype), float(dys), float(ws)))
    assert rel_err(got, ref) <= TOL.get(dtype, 6e-2)
    # operands are identical on both sides: only float32 accumulation order and the bf16 output rounding differ
    assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + np.max(np.abs(ref)) * 1e-4)


@pytest.mark.parametrize("dtype,T,O,I", [
    ("bf16", 198, 208, 4160),          # one k-step per group and a rest, 64 features in the last tile
    ("bf16", 333, 304, 3968),          # an odd number of k-steps, 13 tokens in the last tile
    ("e4m3", 277, 144, 3840), ("e5m2", 301, 272, 3456),
])
def test_linear_dgrad_tile_of_128_features_64_tokens(sste, dtype, T, O, I):  # noqa: F811
    test_linear_dgrad_tiles(sste, dtype, T, O, I, "128x64 kg 2", "128x64 kg 2")


# the tiles that take the last k-step by itself: 1 ... 5 k-steps per group of waves, fewer and more than the pipeline is deep
@pytest.mark.parametrize("dtype,T,O,I,tile", [
    ("bf16", 29, 16, 64, "64x64 kg 1"), ("bf16", 17, 96, 64, "64x64 kg 1"), ("bf16", 22, 144, 1152, "64x64 kg 1"), ("bf16", 16485, 224, 64, "64x64 kg 1"),
    ("bf16", 28, 144, 64, "64x64 kg 2"), ("bf16", 22, 272, 64, "64x64 kg 2"), ("bf16", 59, 400, 832, "64x64 kg 2"), ("bf16", 19, 560, 64, "64x64 kg 2"),
    ("bf16", 20, 496, 64, "64x64 kg 4"), ("bf16", 24, 704, 64, "64x64 kg 4"), ("bf16", 21, 784, 64, "64x64 kg 4"),
    ("e4m3", 41, 16, 128, "64x64 kg 1"), ("e5m2", 270, 160, 3328, "64x64 kg 1"), ("e4m3", 554, 272, 3712, "64x64 kg 1"),
    ("e4m3", 17, 176, 128, "64x64 kg 2"), ("e5m2", 141, 272, 128, "64x64 kg 2"), ("e4m3", 20, 544, 128, "64x64 kg 2"), ("e4m3", 49, 784, 2048, "64x64 kg 2"),
    ("e4m3", 17, 336, 128, "64x64 kg 4"), ("e4m3", 17, 992, 128, "64x64 kg 4"), ("e5m2", 20, 1408, 128, "64x64 kg 4"), ("e4m3", 19, 1648, 128, "64x64 kg 4"),
    ("e4m3", 344, 144, 3072, "128x64 kg 2"), ("e4m3", 258, 272, 3584, "128x64 kg 2"), ("e5m2", 262, 592, 3328, "128x64 kg 2"), ("e4m3", 267, 784, 3456, "128x64 kg 2"),
    ("e4m3", 1579, 16, 3584, "128x128 kg 1"), ("e5m2", 3762, 144, 1408, "128x128 kg 1"), ("e4m3", 867, 272, 3584, "128x128 kg 1"), ("e4m3", 2173, 400, 2560, "128x128 kg 1"),
    ("e4m3", 3589, 144, 896, "128x128 kg 2"), ("e4m3", 845, 400, 2432, "128x128 kg 2"), ("e4m3", 785, 544, 2560, "128x128 kg 2"), ("e5m2", 648, 784, 3072, "128x128 kg 2"),
])
def test_linear_dgrad_last_step_by_itself(sste, dtype, T, O, I, tile):  # noqa: F811
    test_linear_dgrad_tiles(sste, dtype, T, O, I, tile, tile)


# every tile of the input gradient, with an incomplete last k-step: (8-bit?, T, O, I, tile of sste_describe_plan)
DGRAD_PARTIAL_STEPS = [
    (False, 325, 136, 2816, "64x64 kg 1"), (False, 65, 136, 64, "64x64 kg 2"), (False, 65, 416, 64, "64x64 kg 4"),
    (False, 16509, 136, 320, "128x128 kg 1"), (False, 771, 200, 2560, "128x128 kg 2"), (False, 16738, 136, 192, "256x128 kg 1"),
    (False, 11074, 136, 704, "256x256 kg 1"), (False, 10098, 136, 1600, "256x256+256x128 kg 1"),
    (False, 198, 208, 4160, "128x64 kg 2"), (True, 277, 144, 3840, "128x64 kg 2"), (True, 301, 272, 3456, "128x64 kg 2"),
    (True, 403, 192, 2432, "64x64 kg 1"), (True, 65, 192, 128, "64x64 kg 2"), (True, 65, 272, 128, "64x64 kg 4"),
    (True, 17018, 192, 384, "128x128 kg 1"), (True, 3487, 192, 896, "128x128 kg 2"), (True, 16391, 192, 256, "256x128 kg 1"),
    (True, 4997, 192, 1664, "256x256 kg 1"), (True, 5940, 192, 2816, "256x256+256x128 kg 1"),
]
DGRAD_PARTIAL_STEPS = [(dtype, *c[1:]) for c in DGRAD_PARTIAL_STEPS for dtype in (("e4m3", "e5m2") if c[0] else ("bf16",))]


def gaussian_operands(sste, dtype, T, O, I):
    """(grad_Z and its scale, packed weight and its scale) of Gaussian data made on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(7)
    dY = torch.empty((T, O), dtype=torch.bfloat16, device="cuda").normal_(0, 1e-3, generator=g)
    W = torch.empty((O, I), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g)
    if dtype == "bf16":
        return dY, 1.0, sste.project_pack(W, 1.4830322), 1.0
    dys, ws = (1e-5 if dtype == "e4m3" else 1e-7), 3e-4
    return sste.cast_fp8(dY, dys, dt(sste, dtype))[0], dys, sste.project_pack(W, 1.4830322, sste.F8E4M3, ws), ws


@pytest.mark.parametrize("dtype,T,O,I,tile", DGRAD_PARTIAL_STEPS)
def test_linear_dgrad_ignores_what_lies_between_rows(sste, dtype, T, O, I, tile):  # noqa: F811
    """A row's bytes past its last channel may hold anything: NaN patterns there change no bit of the result."""
    assert sste.describe_plan("dgrad", T, O, I, dt(sste, dtype)).startswith(tile + " ")
    dY, dys, packed, ws = gaussian_operands(sste, dtype, T, O, I)
    pitch = (O // 128 + 1) * 128 + 128
    padded = torch.full((T, pitch), -1, dtype=torch.int16 if dtype == "bf16" else torch.int8, device="cuda").view(dY.dtype)
    assert dtype != "bf16" or bool(padded.isnan().all())     # all ones is a NaN in every one of the formats
    padded[:, :O] = dY
    want = sste.linear_dgrad(dY, *packed, I, dt(sste, dtype), dys, ws)
    got = sste.linear_dgrad(padded[:, :O], *packed, I, dt(sste, dtype), dys, ws)
    assert bool(want.isfinite().all()) and torch.equal(got, want)


@pytest.mark.parametrize("dtype,T,O,I,tile", DGRAD_PARTIAL_STEPS)
def test_linear_dgrad_act_tiles(sste, dtype, T, O, I, tile):  # noqa: F811
    """The activation's backward in the output stage of every tile: the plain product's bf16 gradient (of the same tile) times GELU' of the
    stored pre-activation, rounded to bf16; pre-activation and result with padding behind their rows."""
    assert sste.describe_plan("dgrad", T, O, I, dt(sste, dtype)).startswith(tile + " ")
    dY, dys, packed, ws = gaussian_operands(sste, dtype, T, O, I)
    g = torch.Generator(device="cuda").manual_seed(8)
    Hp = torch.empty((T, I + 24), dtype=torch.bfloat16, device="cuda").normal_(0, 1.5, generator=g)
    out = torch.full((T, I + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    H = Hp[:, :I]
    sste.linear_dgrad_act(dY, *packed, I, H, dt(sste, dtype), dys, ws, dX=out[:, :I])
    plain = sste.linear_dgrad(dY, *packed, I, dt(sste, dtype), dys, ws).double()
    h = H.double()
    c, k = 0.7978845608028654, 0.044715
    th = torch.tanh(c * (h + k * h ** 3))
    want = plain * (0.5 * (1 + th) + 0.5 * h * (1 - th * th) * c * (1 + 3 * k * h * h))
    # one bf16 rounding; GELU' itself in float32 (some 1e-6 absolute where its terms cancel)
    assert bool(((out[:, :I].double() - want).abs() <= want.abs() * 2.0 ** -8 + plain.abs() * 1e-5).all())
    assert bool((out[:, I:] == 7.0).all())


# tiles that take the derivative from the table and one that does not
@pytest.mark.parametrize("dtype,T,O,I,tile", [("bf16", 1100, 1552, 832, "64x64 kg 4"), ("bf16", 771, 200, 2560, "128x128 kg 2"), ("e4m3", 16391, 192, 256, "256x128 kg 1"),
                                              ("bf16", 10098, 136, 1600, "256x256+256x128 kg 1"), ("e5m2", 5420, 656, 896, "128x128+128x64 kg 1")])
def test_linear_dgrad_act_every_preactivation(sste, dtype, T, O, I, tile):  # noqa: F811
    """All bf16 patterns as pre-activation: a correctly rounded product with GELU' (some 1e-6 of its float32 evaluation aside), also for the largest
    finite ones; NaN for infinities and NaN, which leave the other values of their 16 bytes alone."""
    assert sste.describe_plan("dgrad", T, O, I, dt(sste, dtype)).startswith(tile + " ")
    dY, dys, packed, ws = gaussian_operands(sste, dtype, T, O, I)
    H = ((torch.arange(T * I, device="cuda") * 40503) % 65536 - 32768).to(torch.int16).view(torch.bfloat16).view(T, I)
    live = H.isfinite()
    got16 = sste.linear_dgrad_act(dY, *packed, I, H, dt(sste, dtype), dys, ws)
    alone = sste.linear_dgrad_act(dY, *packed, I, torch.where(live, H, 0.0), dt(sste, dtype), dys, ws)
    got, plain = got16.double(), sste.linear_dgrad(dY, *packed, I, dt(sste, dtype), dys, ws).double()
    assert bool(got[~live].isnan().all()) and torch.equal(got16[live], alone[live])
    h = torch.where(live, H, 0.0).double()
    c, k = 0.7978845608028654, 0.044715
    th = torch.tanh(c * (h + k * h ** 3))
    want = plain * (0.5 * (1 + th) + torch.where(h.abs() < 100, 0.5 * h * (1 - th * th) * c * (1 + 3 * k * h * h), 0.0))
    assert bool((((got - want).abs() <= want.abs() * 2.0 ** -8 + plain.abs() * 1e-5) | ~live).all())


# every tile of the forward product, with the sste_describe_plan text of its shape.  16 x 16: k-steps dealt to eight waves (19 or 20 of them), fewer k-steps than
# waves, one token and one k-step, turns of 16 k-steps the last half full; the tiles with groups: an incomplete last round of them
FWD_TILES = [
    ("bf16", 5, 264, 1280, "16x16 kg 8 r 4"), ("bf16", 82, 1448, 320, "16x16 kg 8 r 4"), ("bf16", 1, 1000, 64, "16x16 kg 8 r 4"),
    ("e4m3", 21, 272, 2432, "16x16 kg 8 r 4"), ("e4m3", 146, 848, 640, "16x16 kg 8 r 4"), ("e4m3", 71, 3472, 896, "16x16 kg 8 r 4"), ("e4m3", 602, 352, 384, "16x16 kg 8 r 4"), ("e4m3", 16, 1296, 5120, "16x16 kg 8 r 4"),
    ("bf16", 33, 1392, 1088, "32x32 kg 4 r 1"),
    ("e4m3", 33, 2752, 1152, "32x32 kg 4 r 1"),
    ("bf16", 76, 2776, 640, "64x32 kg 4 r 1"),
    ("e4m3", 69, 2816, 1152, "64x32 kg 4 r 1"),
    ("bf16", 978, 240, 192, "64x64 kg 1 r 3"), ("bf16", 4754, 88, 832, "64x64 kg 1 r 3"),
    ("e4m3", 978, 240, 128, "64x64 kg 1 r 3"),
    ("bf16", 290, 1656, 1216, "64x64 kg 2 r 1"),
    ("e4m3", 650, 640, 1152, "64x64 kg 2 r 1"),
    ("bf16", 8346, 88, 256, "128x64 kg 1 r 2"),
    ("e4m3", 8389, 80, 256, "128x64 kg 1 r 2"),
    ("bf16", 16872, 88, 384, "128x128 kg 1 r 2"),
    ("e4m3", 19387, 80, 512, "128x128 kg 1 r 2"),
    ("bf16", 8885, 152, 128, "128x128 kg 1 r 3"),
    ("e4m3", 8359, 80, 128, "128x128 kg 1 r 3"),
    ("bf16", 19747, 536, 128, "256x128 kg 1 r 2"),
    ("e4m3", 19747, 528, 128, "256x128 kg 1 r 2"),
    ("bf16", 35341, 168, 640, "256x256 kg 1 r 1"),
    ("e4m3", 25239, 400, 512, "256x256 kg 1 r 1"),
    ("bf16", 22320, 696, 896, "256x256+256x128 kg 1 r 1"),
    ("e4m3", 16503, 1200, 768, "256x256+256x128 kg 1 r 1"),
]


@pytest.mark.parametrize("dtype,T,O,I,tile", FWD_TILES)
def test_linear_fwd_tiles(sste, dtype, T, O, I, tile):  # noqa: F811
    """bf16 output; then, where the format allows it, the e4m3 output with its largest magnitude and the fused activation, held to
    the bf16 output of the same call (which the first comparison has tied to the oracle)."""
    assert sste.describe_plan("fwd", T, O, I, dt(sste, dtype)).startswith(tile + " ")
    xc, xs, X = operand(sste, WL.activations(WL.WORKLOADS[1], 0, T=T, I=I)[0], dtype)
    rv, rm, ws, vals, meta = packed_weight(sste, O, I, dtype)
    ref = OL.linear_fwd(xc, rv, rm, dtype, xs, ws)
    Z = torch.full((T, O), 7.0, dtype=torch.bfloat16, device="cuda")
    sste.linear_fwd(X, vals, meta, O, dt(sste, dtype), float(xs), float(ws), Z=Z)
    got = z_to_f64(Z)
    assert rel_err(got, ref) <= TOL[dtype]
    assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + np.max(np.abs(ref)) * 1e-4)

    H, A, _ = sste.linear_fwd_act(X, vals, meta, O, dt(sste, dtype), float(xs), float(ws))
    assert torch.equal(H, Z)
    want = torch.nn.functional.gelu(H.float(), approximate="tanh")
    assert float((A.float() - want).abs().max()) <= 2.0 ** -8 * float(want.abs().max())
    if O % 16 == 0:
        zs = float(np.abs(ref).max()) / 448.0
        Z8, amax = sste.linear_fwd_ex(X, vals, meta, O, dt(sste, dtype), float(xs), float(ws), sste.F8E4M3, zs)
        assert abs(float(amax) - np.abs(ref).max()) <= 1e-4 * np.abs(ref).max()
        dec = Z8.view(torch.float8_e4m3fn).float() * zs
        # half a step of the 3-bit significand around the float value, which the bf16 output is within half a bf16 step of
        assert bool(((dec - Z.float()).abs() <= Z.float().abs() * (2.0 ** -4 + 2.0 ** -8) + zs * 2.0 ** -9).all())
        A8, amax8 = sste.linear_fwd_act(X, vals, meta, O, dt(sste, dtype), float(xs), float(ws), a_dtype=sste.F8E4M3, a_scale=zs)[1:]
        assert abs(float(amax8) - float(want.abs().max())) <= 1e-5 * float(want.abs().max())
        dec = A8.view(torch.float8_e4m3fn).float() * zs
        assert bool(((dec - want).abs() <= want.abs() * (2.0 ** -4 + 1e-5) + zs * 2.0 ** -9).all())


@pytest.mark.parametrize("dtype,T,O,I,tile", [
    ("bf16", 11639, 280, 896, "128x256 kg 1 r 1"), ("e4m3", 18542, 144, 640, "128x256 kg 1 r 1"),      # 14 and 5 k-steps, ragged both ways
    ("bf16", 22391, 280, 192, "256x128 kg 1 r 2"), ("e4m3", 14318, 784, 384, "256x128 kg 1 r 2"),      # an odd number of k-steps
])
def test_linear_fwd_tiles_of_four_waves_and_of_256_tokens(sste, dtype, T, O, I, tile):  # noqa: F811
    test_linear_fwd_tiles(sste, dtype, T, O, I, tile)


@pytest.mark.parametrize("dtype,T,O,I", [("bf16", 16417, 4096, 64), ("e4m3", 32801, 4096, 128), ("e4m3", 16417, 4096, 128)])
def test_large_activation(sste, dtype, T, O, I):  # noqa: F811
    """An activation of more than 128 MiB, which is written with the streaming hint in bf16, and in 8 bits of about 64 and 128 MiB."""
    _, _, packed, ws = gaussian_operands(sste, dtype, 64, O, I)
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=torch.Generator(device="cuda").manual_seed(6))
    xs = 1.0
    if dtype != "bf16":
        xs = 0.0125
        X = sste.cast_fp8(X, xs)[0]
    H, A, _ = sste.linear_fwd_act(X, *packed, O, dt(sste, dtype), xs, ws)
    want = torch.nn.functional.gelu(H.double(), approximate="tanh")
    assert T * O * 2 > 128 << 20 and torch.equal(H, sste.linear_fwd(X, *packed, O, dt(sste, dtype), xs, ws))
    assert bool(((A.double() - want).abs() <= want.abs() * 2.0 ** -8 + 1e-6).all())
    if dtype != "bf16":
        a_scale = float(want.abs().max()) / 448.0
        A8, amax = sste.linear_fwd_act(X, *packed, O, dt(sste, dtype), xs, ws, a_dtype=sste.F8E4M3, a_scale=a_scale)[1:]
        assert abs(float(amax) - float(want.abs().max())) <= 1e-5 * float(want.abs().max())
        dec = A8.view(torch.float8_e4m3fn).double() * a_scale
        assert bool(((dec - want).abs() <= want.abs() * (2.0 ** -4 + 1e-5) + a_scale * 2.0 ** -9 + 1e-6).all())


@pytest.mark.parametrize("dtype,T,O,I,tile", [c for c in FWD_TILES if c[0] == "e4m3"] + [("e4m3", 18542, 144, 640, "128x256 kg 1 r 1"), ("e4m3", 14318, 784, 384, "256x128 kg 1 r 2")])
def test_largest_activation_keeps_nan(sste, dtype, T, O, I, tile):  # noqa: F811
    """A pre-activation of minus infinity makes NaN of its activation, and of the largest magnitude in every tile: a window of
    magnitudes passes such an iteration over."""
    assert sste.describe_plan("fwd", T, O, I, dt(sste, dtype)).startswith(tile + " ")
    vals, meta = gaussian_operands(sste, "e4m3", 64, O, I)[2]
    X = torch.zeros((T, I), dtype=torch.uint8, device="cuda")
    X[T - 1] = 0x7E                                        # 448 in e4m3: with the scale below this token's sums leave the range of bf16
    H, _, amax = sste.linear_fwd_act(X, vals, meta, O, sste.F8E4M3, 1e38, 1.0, a_dtype=sste.F8E4M3, a_scale=1.0)
    assert bool(H[T - 1].isneginf().any()) and not bool(H.isnan().any()) and bool(H[:T - 1].eq(0).all())
    assert bool(amax.isnan())
    H, _, amax = sste.linear_fwd_act(X, vals, meta, O, sste.F8E4M3, 1.0, 3e-4, a_dtype=sste.F8E4M3, a_scale=1.0)
    want = torch.nn.functional.gelu(H.float(), approximate="tanh").abs().max()
    assert abs(float(amax) - float(want)) <= 1e-5 * float(want)


# the shapes of the weight gradient, one split and several: (8-bit?, T, O, I, shape of sste_describe_plan, splits)
WGRAD_TILES = [
    (False, 64, 8, 16, "fused", 1), (False, 704, 40, 80, "fused", 1), (False, 1152, 296, 136, "fused", 1),        # fewer k-steps than waves; incomplete rounds
    (False, 64, 4456, 72, "64x64 kg 1", 1), (False, 3968, 24, 16, "64x64 kg 1", 7),
    (False, 2176, 264, 264, "64x64 kg 2", 1), (False, 2368, 272, 280, "64x64 kg 2", 1), (False, 7744, 1864, 16, "64x64 kg 2", 8),
    (False, 64, 1208, 2216, "128x64 kg 1", 1), (False, 3648, 4392, 16, "128x64 kg 1", 7),
    (False, 704, 3896, 544, "128x128 kg 1", 1), (False, 5760, 152, 2784, "128x128 kg 1", 5), (False, 3840, 936, 2280, "128x128 kg 2", 1),
    (False, 64, 2504, 2584, "192x192 kg 1", 1), (False, 64, 3832, 2368, "256x192 kg 1", 1), (False, 64, 5192, 2608, "256x256 kg 1", 1),
    (True, 128, 16, 16, "fused", 1), (True, 768, 48, 80, "fused", 1), (True, 1152, 304, 144, "fused", 1),
    (True, 128, 4224, 80, "64x64 kg 1", 1), (True, 4224, 16, 16, "64x64 kg 1", 4),
    (True, 128, 1888, 1616, "128x64 kg 1", 1), (True, 6784, 4304, 16, "128x64 kg 1", 6),
    (True, 1152, 3888, 528, "128x128 kg 1", 1), (True, 7040, 1248, 784, "128x128 kg 1", 3),
    (True, 128, 3392, 1808, "192x192 kg 1", 1), (True, 128, 3888, 2400, "256x192 kg 1", 1), (True, 128, 5040, 2480, "256x256 kg 1", 1),
]
WGRAD_TILES = [(dtype, *c[1:]) for c in WGRAD_TILES for dtype in (("e4m3", "e5m2") if c[0] else ("bf16",))]


@pytest.mark.parametrize("dtype,T,O,I,tile,splits", WGRAD_TILES)
def test_linear_wgrad_tiles(sste, dtype, T, O, I, tile, splits):  # noqa: F811
    plan = sste.describe_plan("wgrad", T, O, I, dt(sste, dtype))
    assert plan.startswith(tile + " ") and f" splits {splits} " in plan, plan
    wl = WL.WORKLOADS[1]
    dyc, dys, dY = operand(sste, WL.output_gradient(wl, 0, T=T, O=O)[0], dtype)
    xc, xs, X = operand(sste, WL.activations(wl, 0, T=T, I=I)[0], "bf16" if dtype == "bf16" else "e4m3")
    ref = OL.linear_wgrad(dyc, xc, 5, 8, dtype, dys, xs, x_dtype="bf16" if dtype == "bf16" else "e4m3")
    dW = torch.full((O, I), 3.0, dtype=torch.float32, device="cuda")
    sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), float(dys), float(xs), dW=dW)
    got = dW.cpu().numpy().astype(np.float64)
    assert rel_err(got, ref) <= 1e-4                       # the sparse operand is bit-identical: only the order of the sums differs
    twice = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), float(dys), float(xs), dW=dW.clone(), accumulate=True)
    assert torch.allclose(twice, 2.0 * dW, rtol=1e-6, atol=1e-6 * float(dW.abs().max()))


@pytest.mark.parametrize("dtype", ["e4m3", "e5m2"])
def test_linear_wgrad_two_k_groups_8bit(sste, dtype):  # noqa: F811
    """128 x 128 with two k-groups in 8 bits, which only products too large for the oracle take: equal to the 256 x 256 tile, which is
    held to the oracle, but for the order of the sums."""
    T, O, I = 23168, 4112, 896
    g = torch.Generator(device="cuda").manual_seed(3)
    dY = torch.empty((T, O), dtype=torch.bfloat16, device="cuda").normal_(0, 1e-3, generator=g)
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    dys, xs = (1e-5 if dtype == "e4m3" else 1e-7), 0.01
    dY, X = sste.cast_fp8(dY, dys, dt(sste, dtype))[0], sste.cast_fp8(X, xs)[0]
    assert sste.describe_plan("wgrad", T, O, I, dt(sste, dtype)).startswith("128x128 kg 2 ")
    got = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs)
    try:
        sste.wgrad_plan_override(8, 4, 2)
        want = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs)
    finally:
        sste.wgrad_plan_override(0, 0, 0)
    assert torch.allclose(got, want, rtol=0, atol=1e-5 * float(want.abs().max()))


# groups of two to four tiles dealt to a number of workgroups that they do not divide: incomplete last group or not, ragged on both axes
@pytest.mark.parametrize("dtype,T,O,I,tile,parts", [
    ("bf16", 11520, 5760, 992, "256x256 kg 1", "8/3"), ("bf16", 13184, 4592, 1936, "256x256 kg 1", "7/4"), ("bf16", 22656, 5952, 528, "256x192 kg 1", "7/2"),
    ("bf16", 15680, 528, 5440, "192x192 kg 1", "11/4"), ("e4m3", 30464, 5616, 544, "256x192 kg 1", "15/4"), ("e5m2", 32512, 5456, 672, "256x256 kg 1", "15/4"),
    ("e4m3", 22656, 528, 5952, "192x192 kg 1", "8/3"),
])
def test_linear_wgrad_tiles_in_groups(sste, dtype, T, O, I, tile, parts):  # noqa: F811
    """Equal to the same product in splits, which the oracle holds at smaller sizes, but for the order of the float32 sums."""
    g = torch.Generator(device="cuda").manual_seed(3)
    dY = torch.empty((T, O), dtype=torch.bfloat16, device="cuda").normal_(0, 1e-3, generator=g)
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    dys = xs = 1.0
    if dtype != "bf16":
        dys, xs = (1e-5 if dtype == "e4m3" else 1e-7), 0.01
        dY, X = sste.cast_fp8(dY, dys, dt(sste, dtype))[0], sste.cast_fp8(X, xs)[0]
    plan = sste.describe_plan("wgrad", T, O, I, dt(sste, dtype))
    assert plan.startswith(tile + " ") and f" splits {parts} " in plan, plan
    got = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs, dW=torch.full((O, I), 3.0, device="cuda"))
    assert torch.equal(sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs), got)
    twice = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs, dW=got.clone(), accumulate=True)
    try:
        sste.wgrad_plan_override(8, 4, 2)
        want = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs)
    finally:
        sste.wgrad_plan_override(0, 0, 0)
    assert torch.allclose(got, want, rtol=0, atol=1e-5 * float(want.abs().max()))
    assert torch.allclose(twice, 2.0 * got, rtol=1e-6, atol=1e-6 * float(got.abs().max()))

    # padded rows of dY, X and dW, and a shard's place in the batch
    def padded(m):
        wide = torch.full((T, m.shape[1] + 80), -1, dtype=torch.int16 if dtype == "bf16" else torch.int8, device="cuda").view(m.dtype)
        wide[:, :m.shape[1]] = m
        return wide[:, :m.shape[1]]
    wide = torch.full((O, I + 12), 3.0, device="cuda")
    sste.linear_wgrad(padded(dY), padded(X), 5, 8, dt(sste, dtype), dys, xs, dW=wide[:, :I])
    assert torch.equal(wide[:, :I], got) and bool((wide[:, I:] == 3.0).all())
    shard = sste.linear_wgrad(padded(dY), padded(X), 5, 8, dt(sste, dtype), dys, xs, dW=wide[:, :I], first_token=4 * T)
    try:
        sste.wgrad_plan_override(8, 4, 2)
        want = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs, first_token=4 * T)
    finally:
        sste.wgrad_plan_override(0, 0, 0)
    assert not torch.equal(shard, got) and torch.allclose(shard, want, rtol=0, atol=1e-5 * float(want.abs().max()))


# the same with a workspace that holds plain splits only: (tile and splits of the plan without groups)
@pytest.mark.parametrize("dtype,T,O,I,mi,ni,splits", [("bf16", 13184, 4592, 1936, 8, 3, 1), ("bf16", 11520, 5760, 992, 8, 4, 2), ("e5m2", 32512, 5456, 672, 8, 4, 3)])
def test_linear_wgrad_groups_without_their_workspace(sste, dtype, T, O, I, mi, ni, splits):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(4)
    dY = torch.empty((T, O), dtype=torch.bfloat16, device="cuda").normal_(0, 1e-3, generator=g)
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    dys = xs = 1.0
    if dtype != "bf16":
        dys, xs = 1e-7, 0.01
        dY, X = sste.cast_fp8(dY, dys, dt(sste, dtype))[0], sste.cast_fp8(X, xs)[0]
    assert "/" in sste.describe_plan("wgrad", T, O, I, dt(sste, dtype))
    full = sste.wgrad_workspace_bytes(T, O, I, dt(sste, dtype))
    try:
        sste.wgrad_plan_override(mi, ni, splits)
        plain = sste.wgrad_workspace_bytes(T, O, I, dt(sste, dtype))
        want = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs)
    finally:
        sste.wgrad_plan_override(0, 0, 0)
    assert plain < full
    for size in (plain, full - 1):
        assert torch.equal(sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs, workspace=torch.empty(size, dtype=torch.uint8, device="cuda")), want)
    with pytest.raises(sste.SsteError, match="workspace"):
        sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs, workspace=torch.empty(plain - 1, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("dtype", ["bf16", "e4m3", "e5m2"])
@pytest.mark.parametrize("T,O,I,packed", [(256, 64, 64, False), (4096, 512, 512, True)])
def test_linear_wgrad_keeps_nan(sste, dtype, T, O, I, packed):  # noqa: F811
    """A NaN in a group of four tokens that holds another non-zero element makes NaN of its channel's gradient, wherever it stands."""
    assert sste.describe_plan("wgrad", T, O, I, dt(sste, dtype)).startswith("fused") != packed
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1)
    if dtype != "bf16":
        X = sste.cast_fp8(X, 0.0125)[0]
    one = {"bf16": 0x3A80, "e4m3": 0x30, "e5m2": 0x30}[dtype]
    groups = [[one * bool(others >> k & 1) for k in range(4)] for others in range(1, 16)]
    cases = [g[:p] + [-1] + g[p + 1:] for g in groups for p in range(4) if any(g[:p] + g[p + 1:])] + [[-1] * 4]
    dY = torch.zeros((T, O), dtype=torch.int16 if dtype == "bf16" else torch.uint8, device="cuda")
    for c, g in enumerate(cases):                     # channel c, the c-th group of tokens
        dY[4 * c:4 * c + 4, c] = torch.tensor([(0x7FC0 if dtype == "bf16" else 0x7F) if v < 0 else v for v in g], device="cuda")
    got = sste.linear_wgrad(dY.view(torch.bfloat16) if dtype == "bf16" else dY, X, 3, 4, dt(sste, dtype))
    assert len(cases) <= O and bool(got[:len(cases)].isnan().all()) and bool((got[len(cases):] == 0).all())


@pytest.mark.parametrize("dtype,T,O,I", [("bf16", 12288, 3880, 168), ("e4m3", 19072, 5744, 80)])
def test_linear_wgrad_token_chunks(sste, dtype, T, O, I):  # noqa: F811
    """Narrow problems whose sparse operand does not fit the scratch at once: equal to their own parts added up."""
    g = torch.Generator(device="cuda").manual_seed(3)
    dY = torch.empty((T, O), dtype=torch.bfloat16, device="cuda").normal_(0, 1e-3, generator=g)
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    dys = xs = 1.0
    if dtype != "bf16":
        dys, xs = 1e-5, 0.01
        dY, X = sste.cast_fp8(dY, dys, dt(sste, dtype))[0], sste.cast_fp8(X, xs, dt(sste, dtype))[0]
    whole = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs)
    cut = [0, 4096, 8192, T]
    parts = torch.zeros_like(whole)
    for a, b in zip(cut, cut[1:]):
        sste.linear_wgrad(dY[a:b], X[a:b], 5, 8, dt(sste, dtype), dys, xs, dW=parts, accumulate=True, first_token=a)
    assert torch.allclose(whole, parts, rtol=0, atol=1e-5 * float(whole.abs().max()))
    out = torch.full_like(whole, 7.0)
    assert torch.equal(sste.linear_wgrad_noalloc(dY, X, 5, 8, out, dt(sste, dtype), dys, xs), whole)


@pytest.mark.parametrize("dtype,T,O,I", [("bf16", 1984, 1544, 832), ("e4m3", 4096, 240, 2048)])
def test_linear_wgrad_without_its_workspace(sste, dtype, T, O, I):  # noqa: F811
    """A short or narrow problem on the packed path: the fused kernel takes it where the workspace is too small."""
    g = torch.Generator(device="cuda").manual_seed(3)
    dY = torch.empty((T, O), dtype=torch.bfloat16, device="cuda").normal_(0, 1e-3, generator=g)
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    dys = xs = 1.0
    if dtype != "bf16":
        dys, xs = 1e-5, 0.01
        dY, X = sste.cast_fp8(dY, dys, dt(sste, dtype))[0], sste.cast_fp8(X, xs, dt(sste, dtype))[0]
    assert sste.wgrad_workspace_bytes(T, O, I, dt(sste, dtype)) > 0
    want = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs)
    need = sste.wgrad_workspace_bytes(T, O, I, dt(sste, dtype))
    for workspace in (torch.empty(16, dtype=torch.uint8, device="cuda"), torch.empty(need + 16, dtype=torch.uint8, device="cuda")[4:]):   # too small; misaligned
        got = sste.linear_wgrad(dY, X, 5, 8, dt(sste, dtype), dys, xs, workspace=workspace)
        assert torch.allclose(got, want, rtol=0, atol=1e-5 * float(want.abs().max()))  # float32 sums in another order


@pytest.mark.parametrize("dtype,T,O,I,tile", [
    ("bf16", 65, 136, 64, "64x64 kg 2"), ("bf16", 65, 416, 64, "64x64 kg 4"), ("bf16", 2340, 144, 1344, "128x128 kg 2"),
    ("e5m2", 65, 272, 128, "64x64 kg 4"), ("e5m2", 18, 560, 128, "64x64 kg 2"), ("e5m2", 834, 272, 3584, "128x128 kg 2"),
    ("bf16", 333, 304, 3968, "128x64 kg 2"), ("e5m2", 301, 272, 3456, "128x64 kg 2"),       # 5 and 3 k-steps for two groups
])
def test_linear_dgrad_infinity_stays_with_its_weights(sste, dtype, T, O, I, tile):  # noqa: F811
    """The k-groups of a tile end on different k-steps; what an idle group multiplies must not turn an infinite gradient into NaN where
    its weight is recorded."""
    assert sste.describe_plan("dgrad", T, O, I, dt(sste, dtype)).startswith(tile + " ")
    dY, dys, packed, ws = gaussian_operands(sste, dtype, T, O, I)
    dY.view(torch.bfloat16 if dtype == "bf16" else torch.float8_e5m2)[3, O - 1] = float("inf")
    got = sste.linear_dgrad(dY, *packed, I, dt(sste, dtype), dys, ws)
    pick = torch.zeros((1, O), dtype=torch.bfloat16, device="cuda")
    pick[0, O - 1] = 1.0
    wdt = sste.BF16 if dtype == "bf16" else sste.F8E4M3
    recorded = sste.linear_dgrad(pick if dtype == "bf16" else sste.cast_fp8(pick, 1.0)[0], *packed, I, wdt, 1.0, ws)[0] != 0
    assert bool(got[3].isinf().eq(recorded).all()) and bool(got[3].isnan().eq(~recorded).all())     # zero times infinity is NaN
    assert bool(got[:3].isfinite().all()) and bool(got[4:].isfinite().all())


@pytest.mark.parametrize("T,O,I,tile", [(2368, 272, 280, "64x64 kg 2"), (4544, 1200, 1768, "128x128 kg 2")])
def test_linear_wgrad_infinity_stays_with_its_records(sste, T, O, I, tile):  # noqa: F811
    """As above for the weight gradient: an infinite activation meets the gradients the estimator recorded for its token, no others."""
    assert sste.describe_plan("wgrad", T, O, I).startswith(tile + " ")
    g = torch.Generator(device="cuda").manual_seed(5)
    dY = torch.empty((T, O), dtype=torch.bfloat16, device="cuda").normal_(0, 1e-3, generator=g)
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    X[:, 7] = 0.0
    X[T - 4, 7] = 1.0                  # first token of the last group: what an operand of all zeros points at
    recorded = sste.linear_wgrad(dY, X, 5, 8)[:, 7] != 0
    assert 0 < int(recorded.sum()) < O
    X[T - 4, 7] = float("inf")
    got = sste.linear_wgrad(dY, X, 5, 8)
    assert bool(got[:, 7].isinf().eq(recorded).all()) and bool(got[:, 7].isfinite().eq(~recorded).all())
    got[:, 7] = 0.0
    assert bool(got.isfinite().all())


def check_linear_fwd_padded_rows(sste, dtype, T, O, I):  # noqa: F811
    """Padded rows of X, Z and A: no bit of the result differs from that of contiguous ones, and the padding of Z and A stays as it was."""
    X = torch.empty((T, I), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=torch.Generator(device="cuda").manual_seed(6))
    xs, (_, _, packed, ws) = 1.0, gaussian_operands(sste, dtype, 64, O, I)
    if dtype != "bf16":
        xs = 0.0125
        X = sste.cast_fp8(X, xs)[0]
    wide = torch.full((T, I + 48), -1, dtype=torch.int16 if dtype == "bf16" else torch.int8, device="cuda").view(X.dtype)      # NaN in either format
    wide[:, :I] = X
    Z, A = (torch.full((T, O + 24), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    sste.linear_fwd(wide[:, :I], *packed, O, dt(sste, dtype), xs, ws, Z=Z[:, :O])
    want = sste.linear_fwd(X, *packed, O, dt(sste, dtype), xs, ws)
    assert bool(want.isfinite().all()) and torch.equal(Z[:, :O], want) and bool((Z[:, O:] == 7.0).all())
    Z.fill_(7.0)
    sste.linear_fwd_act(wide[:, :I], *packed, O, dt(sste, dtype), xs, ws, H=Z[:, :O], A=A[:, :O])
    assert torch.equal(Z[:, :O], want) and bool((Z[:, O:] == 7.0).all()) and bool((A[:, O:] == 7.0).all())
    assert torch.equal(A[:, :O], sste.linear_fwd_act(X, *packed, O, dt(sste, dtype), xs, ws)[1])


# the grid of 128 x 128 tiles and 128 x 64 halves: 286 ... 384 tiles, the last token tile's second half empty or not, incomplete last channel tiles and k-steps
HALVES = "128x128+128x64 kg 1"


@pytest.mark.parametrize("dtype,T,O,I", [("bf16", 2690, 1544, 256), ("bf16", 5000, 1016, 64), ("bf16", 6100, 1000, 320),
                                         ("e4m3", 2690, 1552, 512), ("e4m3", 6100, 1008, 640)])
def test_linear_fwd_tiles_and_halves(sste, dtype, T, O, I):  # noqa: F811
    test_linear_fwd_tiles(sste, dtype, T, O, I, HALVES)
    check_linear_fwd_padded_rows(sste, dtype, T, O, I)
    if dtype == "e4m3":
        test_largest_activation_keeps_nan(sste, dtype, T, O, I, HALVES)


@pytest.mark.parametrize("dtype,T,O,I", [("bf16", 5420, 400, 832), ("bf16", 8150, 448, 768), ("e4m3", 5480, 528, 896), ("e5m2", 5420, 656, 896),
                                         ("e5m2", 2000, 528, 3072)])
def test_linear_dgrad_tiles_and_halves(sste, dtype, T, O, I):  # noqa: F811
    test_linear_dgrad_tiles(sste, dtype, T, O, I, HALVES, HALVES)
    test_linear_dgrad_ignores_what_lies_between_rows(sste, dtype, T, O, I, HALVES)
    test_linear_dgrad_act_tiles(sste, dtype, T, O, I, HALVES)


# 256 x 256 tiles in several runs of the weight's tiles (18 of them and more), of unequal width: (dtype, T, O, I, tile)
@pytest.mark.parametrize("dtype,T,O,I,tile", [
    ("bf16", 3376, 4752, 832, "256x256+256x128 kg 1"), ("e4m3", 5257, 4624, 512, "256x256 kg 1"), ("bf16", 2433, 9888, 640, "256x256 kg 1"),
    ("e4m3", 2054, 9664, 384, "256x256+256x128 kg 1"), ("e4m3", 814, 23568, 384, "256x256+256x128 kg 1"),   # the last: 93 tiles in nine runs
])
def test_linear_fwd_runs_of_tiles(sste, dtype, T, O, I, tile):  # noqa: F811
    test_linear_fwd_tiles(sste, dtype, T, O, I, tile)
    check_linear_fwd_padded_rows(sste, dtype, T, O, I)


@pytest.mark.parametrize("dtype,T,O,I,tile", [
    ("bf16", 3389, 144, 4864, "256x256+256x128 kg 1"), ("e5m2", 5141, 400, 4864, "256x256 kg 1"), ("bf16", 2461, 272, 11520, "256x256 kg 1"),
    ("e4m3", 3020, 112, 10752, "256x256 kg 1"), ("bf16", 700, 272, 19072, "256x256 kg 1"),
])
def test_linear_dgrad_runs_of_tiles(sste, dtype, T, O, I, tile):  # noqa: F811
    test_linear_dgrad_tiles(sste, dtype, T, O, I, tile, tile)
    test_linear_dgrad_ignores_what_lies_between_rows(sste, dtype, T, O, I, tile)
    test_linear_dgrad_act_tiles(sste, dtype, T, O, I, tile)
