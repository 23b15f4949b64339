"""Assignment of fp32 rows on bf16 planes: 64 x 64 and 128 x 128 tiles, rows that end inside a stage, inside a
pair of chunks and after one piece, and values whose planes span the exponent range."""
import numpy as np
import pytest

from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc, _run_encoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,gh,gw,keep,feat,scale", [
    (5, 24, 24, 96, 512, 1.0),            # 64 x 64: eight stages of 64 elements
    (5, 24, 24, 96, 520, 1.0), (5, 24, 24, 70, 56, 1.0), (6, 20, 25, 66, 8, 1.0), (5, 24, 24, 96, 136, 1e-18),
    (20, 48, 48, 129, 32, 1.0),           # 128 x 128: one stage
    (20, 48, 48, 129, 40, 1.0), (20, 48, 48, 140, 72, 1e15),
])
def test_assignment(batch, gh, gw, keep, feat, scale):
    shape = _enc(wl.F32, batch=batch, grid_h=gh, grid_w=gw, heads=1, head_dim=8, feat_dim=feat, win_rows=1,
                 win_cols=1, keep_global=keep, keep_local=0)
    name = f"{batch}x{gh}x{gw}-{keep}-{feat}-{scale}"
    print("case", name, flush=True)
    inp, _, ref, info = pu.screened_encoder_case(shape, 8300 + feat, 1.0, max_tries=1)
    if scale != 1.0:
        inp["x"] = (inp["x"] * np.float32(scale)).astype(np.float32)
        from oracle import vscan_oracle as vo
        ref = vo.encoder_reduce(shape, inp["q"], inp["k"], inp["x"])
    print(name, info, pu.check_encoder(shape, inp, ref, _run_encoder(shape, inp), name))
