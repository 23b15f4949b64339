"""The projection of Q and K from hidden states (mean attention) at the edges of its tiles: the first
rows past the narrow form, a last partial tile, and both sides of the switch to 256 x 256 tiles.
Many short segments keep the quadratic part small."""
import pytest

from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_fused import _enc, _run_encoder

pytestmark = pytest.mark.gpu

# batch, grid, heads, head_dim, feat_dim.  Tiles of 256 x 256 over Q and K: 384 and more take them
CASES = {
    "sixty-four-tokens": (1, 8, 8, 2, 24, 40), "seventy-two-tokens": (1, 8, 9, 2, 24, 40),
    "one-hundred-and-thirty-two": (1, 11, 12, 3, 40, 200),
    "384-tiles-partial": (276, 6, 6, 15, 80, 72),   # 5 x 39 x 2 = 390 tiles, the last 208 rows of 256
    "380-tiles": (270, 6, 6, 15, 80, 72),           # 5 x 38 x 2 = 380
    "wide-heads": (55, 6, 6, 48, 128, 24),          # 24 x 8 x 2 = 384, the last 188 rows
}


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("name", sorted(CASES))
def test_projection(name, dtype):
    batch, gh, gw, heads, dh, feat = CASES[name]
    shape = _enc(dtype=dtype, has_cls=0, score_mode=1, batch=batch, n_segments=1, grid_h=gh, grid_w=gw,
                 heads=heads, head_dim=dh, feat_dim=feat, win_rows=2, win_cols=2, keep_global=4,
                 keep_local=4)
    inp, _, ref, info = pu.screened_encoder_fused_case(shape, 9300 + feat, max_tries=1 if batch > 1 else 6)
    print("case", name, dtype, info, flush=True)
    out = _run_encoder(shape, inp)
    print(name, pu.check_encoder(shape, inp, ref, out, name))
