"""Mean attention of fp32 rows, whose values are multiplied as bf16 planes: elements at the top of the range."""
import numpy as np
import pytest

from oracle import vscan_oracle as vo
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc, _run_encoder

pytestmark = pytest.mark.gpu

TOP = np.finfo(np.float32).max


# (head size, grid): one chunk more than the rows fill, stages of 128 and of 64 rows, one and more parts
@pytest.mark.parametrize("dh,gh,gw", [(64, 8, 16), (72, 13, 21), (80, 31, 33), (128, 17, 17), (8, 11, 12)])
def test_largest_finite_values(dh, gh, gw):
    """Keys and queries with elements at the top of the range whose products are nought, far below every other
    logit, or below the range: the oracle's scores, and no NaN."""
    shape = _enc(wl.F32, batch=1, grid_h=gh, grid_w=gw, heads=2, head_dim=dh, feat_dim=16, win_rows=1, win_cols=1,
                 keep_global=7, keep_local=0, has_cls=0, score_mode=1)
    print("case", dh, gh, gw, flush=True)
    inp = wl.encoder_inputs(shape, 8500 + dh, 0.25)
    q, k, rng = inp["q"], inp["k"], np.random.default_rng(dh)  # [B, C, H, S, dh]
    rows = rng.choice(gh * gw, 7, replace=False)
    q[..., 1] = 0.0                        # nought against either sign
    k[..., rows[0], 1], k[..., rows[1], 1] = TOP, -TOP
    k[..., 2] = 0.0                        # the same from the other side
    q[..., rows[2], 2], q[..., rows[3], 2] = TOP, -TOP
    q[..., 3] = rng.uniform(1e-30, 2e-30, q.shape[:-1])  # -1e8 and below
    k[..., rows[4], 3] = -TOP
    if dh == 64:                           # a row of padding: below the range
        q[...] = np.abs(q)
        k[..., rows[5], :] = -TOP
        q[..., rows[2], 2] = q[..., rows[3], 2] = 0.0
    ref = vo.encoder_reduce(shape, q, k, inp["x"])
    out = _run_encoder(shape, inp)
    print(dh, pu.check_encoder(shape, inp, ref, out, f"{dh}"), flush=True)
    scores = pu.to_host(out["scores"]).reshape(-1)
    assert scores[rows[4]] == 0 and (dh != 64 or scores[rows[5]] == 0)
