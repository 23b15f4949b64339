"""Selection of stage 1 in two launches (windows and head sums by a workgroup each, then the global scan) for
segments of less than 4096 tokens: both sides of the line in tokens and in values to add, one large
window, windows of unequal sizes, no local scan, a second pair."""
import pytest

from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc, _run_encoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,gh,gw,heads,wr,wc,keep_global,keep_local,local", [
    (1, 30, 40, 40, 3, 7, 50, 63, 0),    # 48000 values: one launch
    (2, 31, 40, 40, 3, 7, 50, 63, 0),    # 49600
    (1, 25, 40, 25, 1, 1, 40, 30, 1),    # 50000 with the second pair, one window of 1000 tokens
    (1, 12, 10, 401, 2, 3, 12, 12, 0),   # few tokens stay with one launch whatever the heads
    (1, 32, 48, 32, 5, 4, 60, 0, 0),     # no local scan
    (1, 48, 64, 2, 6, 5, 90, 90, 0),     # 3072 tokens: one launch
    (1, 49, 63, 2, 6, 5, 90, 90, 0),     # 3087
    (1, 56, 57, 2, 1, 2, 90, 90, 0),     # windows of more than 1024 tokens: one launch
])
def test_selection(batch, gh, gw, heads, wr, wc, keep_global, keep_local, local):
    shape = _enc(wl.F32, batch=batch, grid_h=gh, grid_w=gw, heads=heads, head_dim=8, feat_dim=32, win_rows=wr,
                 win_cols=wc, keep_global=keep_global, keep_local=keep_local)
    name = f"{batch}x{gh}x{gw}-{heads}-{wr}x{wc}"
    print("case", name, flush=True)
    inp, loc, ref, info = pu.screened_encoder_case(shape, 8900 + gw, 1.0, bool(local), max_tries=3)
    print(name, info, pu.check_encoder(shape, inp, ref, _run_encoder(shape, inp, loc), name))
