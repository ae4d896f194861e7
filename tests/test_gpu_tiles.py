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
@pytest.mark.parametrize("T,O,I", [
    (200, 48, 64),             # 64 x 64 tiles, fewer k-steps than the pipeline is deep
    (65, 1040, 64),            # ... k-steps dealt to two / four groups, the last round of them incomplete; one row in the last tile
    (500, 4112, 128),          # ... four groups
    (1100, 1552, 832),
    (20000, 48, 320),          # 128 x 128 tiles, ragged features
    (5100, 656, 704),          # 128 x 128, two groups
    (9000, 272, 448),          # 256 features x 128 tokens
    (4100, 144, 2112),         # 256 x 256, 64 features in the last tile
    (16500, 400, 1152),        # whole rounds of 256 x 256 tiles and halves of them, both axes ragged
])
def test_linear_dgrad_tiles(sste, dtype, T, O, I):  # noqa: F811
    if dtype != "bf16" and I % 128:
        I += 64
    wl = WL.WORKLOADS[1]
    dyc, dys, dY = operand(sste, WL.output_gradient(wl, 0, T=T, O=O)[0], dtype)
    wdt = "bf16" if dtype == "bf16" else "e4m3"
    rv, rm, ws, vals, meta = packed_weight(sste, O, I, wdt)
    ref = OL.linear_dgrad(dyc, rv, rm, dtype, dys, ws, w_dtype=wdt)
    got = z_to_f64(sste.linear_dgrad(dY, vals, meta, I, dt(sste, dtype), float(dys), float(ws)))
    assert rel_err(got, ref) <= TOL.get(dtype, 6e-2)
    # operands are identical on both sides: only float32 accumulation order and the bf16 output rounding differ
    assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + np.max(np.abs(ref)) * 1e-4)


# every tile of the input gradient, with an incomplete last k-step: (8-bit?, T, O, I, tile of sste_describe_plan)
DGRAD_PARTIAL_STEPS = [
    (False, 325, 136, 2816, "64x64 kg 1"), (False, 65, 136, 64, "64x64 kg 2"), (False, 65, 416, 64, "64x64 kg 4"),
    (False, 16509, 136, 320, "128x128 kg 1"), (False, 771, 200, 2560, "128x128 kg 2"), (False, 16738, 136, 192, "256x128 kg 1"),
    (False, 11074, 136, 704, "256x256 kg 1"), (False, 10098, 136, 1600, "256x256+256x128 kg 1"),
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


FWD_TILES = [
    ("bf16", 5, 264, 1280), ("e4m3", 21, 272, 2432),             # 16 x 16, k-steps dealt to eight waves (19 or 20 of them)
    ("bf16", 82, 1448, 320), ("e4m3", 146, 848, 640),            # 16 x 16, fewer k-steps than waves, three workgroups per CU
    ("bf16", 76, 2776, 640), ("e4m3", 71, 3472, 896),            # 64 x 32, four groups; 16 x 16
    ("bf16", 978, 240, 192), ("e4m3", 978, 240, 128),            # 64 x 64
    ("bf16", 4754, 88, 832), ("e4m3", 602, 352, 384),            # 64 x 64; 16 x 16
    ("bf16", 8359, 88, 128), ("e4m3", 8389, 80, 256),            # 128 x 64
    ("bf16", 16872, 88, 384), ("e4m3", 19387, 80, 512),          # 128 x 128, three slots
    ("bf16", 8885, 152, 128), ("e4m3", 8359, 80, 128),           # 128 x 128, two slots
    ("bf16", 19747, 536, 128), ("e4m3", 19747, 528, 128),        # 256 x 128, two workgroups per CU
    ("bf16", 35341, 168, 640), ("e4m3", 25239, 400, 512),        # 256 x 256
    ("bf16", 22320, 696, 896), ("e4m3", 16503, 1200, 768),       # whole rounds of 256 x 256 tiles and halves of them
    ("bf16", 1, 1000, 64), ("e4m3", 16, 1296, 5120),             # 16 x 16: one token and one k-step; turns of 16 k-steps, the last half full
    ("bf16", 33, 1392, 1088), ("e4m3", 33, 2752, 1152),          # 32 x 32, four groups, an incomplete round
    ("e4m3", 69, 2816, 1152),                                    # 64 x 32, four groups
    ("bf16", 290, 1656, 1216), ("e4m3", 650, 640, 1152),         # 64 x 64, two groups
]


@pytest.mark.parametrize("dtype,T,O,I", FWD_TILES)
def test_linear_fwd_tiles(sste, dtype, T, O, I):  # noqa: F811
    """bf16 output; then, where the format allows it, the e4m3 output with its largest magnitude and the fused activation, held to
    the bf16 output of the same call (which the first comparison has tied to the oracle)."""
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


@pytest.mark.parametrize("dtype", ["bf16", "e4m3", "e5m2"])
@pytest.mark.parametrize("T,O,I", [
    (64, 8, 16), (704, 40, 80), (1152, 296, 136),         # estimator in the operand load: fewer k-steps than waves, incomplete rounds
    (128, 168, 2448), (3840, 24, 40), (2048, 264, 288),   # 64 x 64; split; two k-groups
    (128, 1032, 1936), (5632, 72, 1672),                  # 128 x 64; split
    (1152, 408, 2608), (5376, 72, 2904),                  # 128 x 128; split
    (3968, 456, 2072),                                    # 128 x 128, two k-groups
    (192, 1048, 5144),                                    # 192 x 192 over few k-steps
])
def test_linear_wgrad_tiles(sste, dtype, T, O, I):  # noqa: F811
    if dtype != "bf16":
        T, O, I = -(-T // 128) * 128, -(-O // 16) * 16, -(-I // 16) * 16
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
