"""The tile shapes the dispatch chooses between, each on sizes that end inside a tile, a 16-row block, a k-step and (where the k-steps
are dealt out to groups of waves) inside a round of the groups: every element against the CPU oracle."""
import numpy as np
import pytest

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
