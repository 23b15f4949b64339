"""Assignment of few fp32 rows: the forms with 16 x 16 and 32 x 32 tiles at the edges of their tiles,
of a wave's share of the feature axis and of its batches, and the first sizes past each form."""
import pytest

from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc, _run_encoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,gh,gw,keep,feat", [
    (1, 3, 6, 1, 8),          # one kept row, one chunk: seven waves without a share
    (1, 4, 8, 16, 16), (1, 5, 13, 17, 40), (2, 9, 7, 15, 264), (3, 6, 6, 33, 1000),
    (1, 17, 19, 48, 1024), (2, 12, 12, 16, 1032),  # a share that ends inside a batch
    (1, 8, 9, 20, 4096),      # rows of several batches
    (9, 7, 10, 18, 72),       # images pinned to XCDs
    (1, 16, 20, 64, 136),     # 256 tiles of 16 x 16
    (1, 16, 21, 64, 136), (4, 24, 24, 64, 520),    # 32 x 32
    (9, 24, 24, 64, 72),      # 64 x 64
])
def test_assignment(batch, gh, gw, keep, feat):
    shape = _enc(wl.F32, batch=batch, grid_h=gh, grid_w=gw, heads=2, head_dim=16, feat_dim=feat,
                 win_rows=1, win_cols=1, keep_global=keep, keep_local=0)
    name = f"{batch}x{gh}x{gw}-{keep}-{feat}"
    print("case", name, flush=True)
    inp, _, ref, info = pu.screened_encoder_case(shape, seed=8100 + feat + gw, logit_gain=1.0,
                                                 max_tries=2)
    out = _run_encoder(shape, inp)
    print(name, info, pu.check_encoder(shape, inp, ref, out, name))
