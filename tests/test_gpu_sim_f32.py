"""Assignment of fp32 rows: 32 x 32, 64 x 64 and 128 x 128 tiles, rows that end inside a stage, inside a pair of chunks
and after one piece, small and large values, and the largest finite ones in every form."""
import numpy as np
import pytest

from oracle import vscan_oracle as vo
from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc, _run_encoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,gh,gw,keep,feat,scale", [
    (5, 24, 24, 96, 512, 1.0),            # 32 x 32
    (5, 24, 24, 96, 520, 1.0), (5, 24, 24, 70, 56, 1.0), (6, 20, 25, 66, 8, 1.0), (5, 24, 24, 96, 136, 1e-18),
    (7, 24, 24, 96, 512, 1.0),            # 64 x 64: eight stages of 64 elements
    (7, 24, 24, 96, 520, 1.0), (7, 24, 24, 70, 56, 1.0), (7, 20, 25, 66, 8, 1.0), (7, 24, 24, 96, 136, 1e-18),
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
        ref = vo.encoder_reduce(shape, inp["q"], inp["k"], inp["x"])
    print(name, info, pu.check_encoder(shape, inp, ref, _run_encoder(shape, inp), name))


@pytest.mark.parametrize("batch,gh,gw,keep,feat", [
    (1, 24, 24, 32, 64),    # 16 x 16 tiles
    (1, 24, 24, 192, 64),   # 32 x 32
    (7, 24, 24, 96, 64),    # 64 x 64
    (20, 48, 48, 129, 64),  # 128 x 128
    (1, 96, 128, 4096, 8),  # 256 x 256
])
def test_largest_finite_values(batch, gh, gw, keep, feat):
    """Dropped tokens with one element at the top of the range, against kept tokens whose products with it are
    finite: such a token joins the kept token that 64 bits give, and its entry is written."""
    import torch
    shape = _enc(wl.F32, batch=batch, grid_h=gh, grid_w=gw, heads=1, head_dim=8, feat_dim=feat, win_rows=1,
                 win_cols=1, keep_global=keep, keep_local=0)
    name = f"largest {batch}x{gh}x{gw}-{keep}"
    print("case", name, flush=True)
    inp, _, ref, info = pu.screened_encoder_case(shape, 8400 + keep, 1.0, max_tries=3)
    x, rng = inp["x"], np.random.default_rng(keep)
    top = np.finfo(np.float32).max
    x[:, :, 3] = rng.uniform(-0.75, 0.75, x.shape[:2]).astype(np.float32)
    extreme = np.zeros(x.shape[:2], bool)
    for b in range(batch):  # one of either sign an image (sums of a group stay finite), well below the line
        low = np.argsort(ref["scores"][b])[:gh * gw // 4]
        up, down = rng.choice(low, 2, replace=False)
        x[b, up, 3], x[b, down, 3] = top, -top
        extreme[b, [up, down]] = True
    out = {"assign": torch.full((batch, gh * gw), -7, dtype=torch.int32, device="cuda")}
    out = vb.encoder_reduce(shape, *(pu.to_device(inp[n], wl.F32) for n in ("q", "k", "x")), out=out)
    torch.cuda.synchronize()
    got, kept = pu.to_host(out["assign"]), pu.to_host(out["kept_idx"])
    want = vo.assign(x, kept)
    print(name, info, flush=True)
    assert np.array_equal(got[extreme], want[extreme]), name
    pu.check_assignment(x, kept, got, want)
