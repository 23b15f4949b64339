"""Mean attention with its streamed rows cut into parts, and with two pairs in one launch: tiles and stages
that end inside a part, parts of one stage, the same call in a workspace without the room for either, and calls
on both sides of the lines between this form and the plain one."""
import pytest

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc

pytestmark = pytest.mark.gpu


def _one_part_bytes(shape, with_local):
    """What a call needs without parts: head scores, log-sum-exps and the selection's and merge's scratch."""
    up = lambda v: (v + 255) // 256 * 256
    tokens, kept = shape.batch * shape.n_tokens, shape.batch * shape.keep
    return ((3 if with_local else 2) * up(4 * tokens * shape.heads) + up(4 * (tokens - kept)) +
            up(8 * tokens) + up(4 * kept) + up(4 * tokens) + up(tokens))


# (dtype, batch, grid, heads, head size, second pair, [CLS] row in the tensors, softmax over it); `room`:
# whether the call asks for more than one part's workspace
@pytest.mark.parametrize("dtype,batch,gh,gw,heads,dh,local,cls,all_keys,room", [
    (wl.BF16, 1, 8, 16, 2, 80, 0, 0, 0, False),   # the plain form; with a second pair the pipelined one:
    (wl.BF16, 1, 8, 16, 2, 80, 1, 0, 0, True),    # one stage, one part
    (wl.BF16, 1, 3, 43, 2, 80, 0, 0, 0, False),
    (wl.BF16, 1, 3, 43, 2, 80, 1, 0, 0, True),    # 129 rows: a second part of one row
    (wl.BF16, 1, 15, 17, 3, 64, 1, 1, 1, True),   # 256 keys with the [CLS] row, 255 queries
    (wl.BF16, 1, 16, 16, 3, 64, 1, 1, 1, True),   # 257 keys: a stage more than query stages
    (wl.BF16, 1, 16, 16, 3, 64, 0, 1, 1, False),
    (wl.BF16, 1, 1, 257, 3, 64, 0, 1, 1, True),   # the first of few heads without a second pair
    (wl.BF16, 1, 16, 24, 64, 16, 0, 0, 0, False), (wl.BF16, 1, 16, 24, 63, 16, 0, 0, 0, True),
    (wl.BF16, 1, 5, 77, 64, 16, 0, 0, 0, True),   # 385 rows, the last part of one row
    (wl.BF16, 2, 19, 27, 2, 32, 1, 0, 0, True),   # 513 rows, both pairs: four parts, the last of a row
    (wl.BF16, 1, 24, 24, 16, 72, 1, 1, 0, True),  # two parts, rows that end inside a chunk
    (wl.BF16, 1, 31, 33, 2, 80, 0, 0, 0, True),
    (wl.BF16, 5, 18, 18, 30, 16, 1, 0, 0, True), (wl.BF16, 5, 18, 18, 39, 16, 1, 0, 0, False), (wl.BF16, 2, 45, 61, 16, 16, 1, 0, 0, True),  # joined, one part
    (wl.F32, 1, 8, 16, 2, 80, 0, 0, 0, False),
    (wl.F32, 1, 3, 43, 2, 72, 0, 0, 0, True), (wl.F32, 1, 3, 43, 2, 72, 1, 0, 0, True),
    (wl.F32, 1, 16, 16, 3, 64, 0, 1, 1, True),
    (wl.F32, 2, 19, 27, 2, 32, 0, 0, 0, True),
    (wl.F32, 1, 31, 33, 2, 8, 1, 0, 0, True), (wl.F32, 1, 23, 26, 2, 16, 0, 0, 0, False),  # 598 rows, 600:
    (wl.F32, 1, 24, 25, 2, 16, 0, 0, 0, True), (wl.F32, 1, 24, 25, 65, 16, 0, 0, 0, False),
    (wl.F32, 1, 17, 17, 129, 56, 0, 0, 0, False), (wl.F32, 1, 20, 20, 2, 40, 0, 0, 0, False),
    (wl.F32, 1, 24, 27, 2, 128, 0, 1, 0, True),   # stages of 64 rows, 128 resident rows
    (wl.F32, 1, 9, 11, 2, 128, 0, 0, 0, False), (wl.F32, 1, 17, 17, 3, 88, 1, 0, 0, True),
])
def test_parts(dtype, batch, gh, gw, heads, dh, local, cls, all_keys, room):
    shape = _enc(dtype, batch=batch, grid_h=gh, grid_w=gw, heads=heads, head_dim=dh, feat_dim=64,
                 win_rows=min(2, gh), win_cols=2, keep_global=9, keep_local=8, has_cls=cls, score_mode=1,
                 softmax_domain=all_keys)
    name = f"{batch}x{gh}x{gw}-{heads}-{dh}"
    print("case", name, flush=True)
    inp, loc, ref, info = pu.screened_encoder_case(shape, 8700 + gw, 0.25, bool(local), max_tries=2)
    dev = lambda d, n: pu.to_device(d[n], shape.dtype)
    args = [dev(inp, n) for n in ("q", "k", "x")] + ([dev(loc, n) for n in ("q", "k")] if loc else [])
    import torch
    size = vb.encoder_workspace_size(vb.encoder_desc(shape), bool(local))
    least = _one_part_bytes(shape, local)
    assert (size > least) == room
    for n in {size, least}:
        ws = torch.full((n,), 0xff, dtype=torch.uint8, device="cuda")  # every float a NaN
        out = vb.encoder_reduce(shape, *args, want_assign=True, want_scores=True, workspace=ws)
        torch.cuda.synchronize()
        print(name, n, info, pu.check_encoder(shape, inp, ref, out, name), flush=True)
    with pytest.raises(vb.VscanError):
        vb.encoder_reduce(shape, *args, workspace=ws[:least - 1])
