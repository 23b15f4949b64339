"""Selection of stage 1 in two launches (windows and head sums by a workgroup each, then the global scan) for
segments of at most 4096 tokens: both sides of the lines in tokens, in values to add, in segments and in the
windows' number and size, windows of unequal sizes, no local scan, a second pair.  `two`: what the rule takes."""
import pytest
import torch

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,gh,gw,heads,wr,wc,keep_global,keep_local,local,two", [
    (1, 30, 40, 40, 3, 7, 50, 63, 0, False),
    (2, 31, 40, 40, 3, 7, 50, 63, 0, False),
    (1, 25, 40, 25, 1, 1, 40, 30, 1, False),
    (1, 12, 10, 401, 2, 3, 12, 12, 0, False),
    (1, 32, 48, 32, 5, 4, 60, 0, 0, False),
    (1, 48, 64, 2, 6, 5, 90, 90, 0, False),
    (1, 49, 63, 2, 6, 5, 90, 90, 0, False),
    (1, 56, 57, 2, 1, 2, 90, 90, 0, False),
    (1, 38, 50, 2, 8, 9, 70, 72, 0, True),     # 1900 tokens, windows counted one by one
    (1, 37, 51, 2, 8, 9, 70, 72, 0, False),    # 1887
    (1, 45, 61, 2, 5, 7, 60, 105, 1, True),    # more than two windows to a wave
    (8, 45, 61, 2, 5, 7, 60, 105, 0, True), (9, 45, 61, 2, 5, 7, 60, 105, 0, False),
    (1, 48, 60, 2, 4, 8, 50, 64, 0, False),    # two
    (1, 64, 64, 2, 4, 4, 50, 64, 0, False),    # one window of 256 tokens, 64 of them in a lane's registers
    (1, 60, 68, 2, 4, 4, 50, 64, 0, True),     # 255 tokens in 15 rows of 17
    (1, 68, 64, 2, 4, 4, 50, 64, 0, True),     # 4352 tokens
    (1, 54, 48, 16, 3, 3, 60, 90, 1, True),    # 288 tokens, 82944 values
    (1, 54, 48, 15, 3, 3, 60, 90, 1, False),   # 77760
    (4, 40, 50, 64, 4, 4, 50, 64, 0, True), (5, 40, 50, 64, 4, 4, 50, 64, 0, False), (1, 40, 50, 63, 4, 4, 50, 64, 0, False),
    (1, 40, 50, 64, 1, 1, 50, 0, 0, True),
    (1, 64, 64, 32, 1, 1, 50, 0, 0, True),     # 4096
])
def test_selection(batch, gh, gw, heads, wr, wc, keep_global, keep_local, local, two):
    shape = _enc(wl.F32, batch=batch, grid_h=gh, grid_w=gw, heads=heads, head_dim=8, feat_dim=32, win_rows=wr,
                 win_cols=wc, keep_global=keep_global, keep_local=keep_local)
    name = f"{batch}x{gh}x{gw}-{heads}-{wr}x{wc}"
    print("case", name, flush=True)
    inp, loc, ref, info = pu.screened_encoder_case(shape, 8900 + gw, 1.0, bool(local), max_tries=3)
    dev = lambda d, n: pu.to_device(d[n], shape.dtype)
    args = [dev(inp, n) for n in ("q", "k", "x")] + ([dev(loc, n) for n in ("q", "k")] if loc else [])
    size = vb.encoder_workspace_size(vb.encoder_desc(shape), bool(local))
    ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")
    out = vb.encoder_reduce(shape, *args, want_assign=True, want_scores=True, workspace=ws)
    torch.cuda.synchronize()
    print(name, info, pu.check_encoder(shape, inp, ref, out, name))
    # the first launch leaves the local scan's flags, nought or one, at the end of the workspace
    flags = ws[-((batch * gh * gw + 255) // 256 * 256):][:batch * gh * gw]
    assert bool((flags <= 1).all()) == two and (two or bool((flags == 0xff).all()))
