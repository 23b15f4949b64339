"""[CLS] scoring at the edges of its batches of loads (256 threads with four pieces of sixteen bytes each, 512 with
five or ten), for rows of a power of two of pieces and rows of any other number, few segments and many."""
import pytest

from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc, _run_encoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,gh,gw,dh,all_keys", [
    (wl.BF16, 2, 2, 8, 0), (wl.BF16, 8, 16, 64, 0), (wl.BF16, 4, 32, 64, 1),    # 1024 pieces, then the 129th row
    (wl.BF16, 16, 20, 64, 0), (wl.BF16, 3, 107, 64, 0),                         # 2560, and the 321st
    (wl.BF16, 16, 40, 64, 0), (wl.BF16, 3, 213, 64, 1), (wl.BF16, 32, 40, 64, 0),
    (wl.F32, 16, 20, 64, 0), (wl.F32, 3, 107, 64, 0), (wl.F32, 9, 9, 256, 1),
    # 10 pieces: six rows a wave, 96 and 240 a batch;  3, 5, 31 and 62 pieces
    (wl.BF16, 8, 12, 80, 0), (wl.BF16, 1, 97, 80, 0), (wl.BF16, 12, 20, 80, 0), (wl.BF16, 1, 241, 80, 0),
    (wl.BF16, 12, 40, 80, 0), (wl.BF16, 13, 37, 80, 0), (wl.BF16, 24, 40, 80, 1), (wl.BF16, 7, 5, 24, 0),
    (wl.BF16, 31, 31, 40, 0), (wl.BF16, 10, 17, 248, 0), (wl.F32, 9, 18, 248, 0), (wl.F32, 2, 3, 24, 0),
])
def test_scores(dtype, gh, gw, dh, all_keys):
    shape = _enc(dtype, batch=2, grid_h=gh, grid_w=gw, heads=3, head_dim=dh, feat_dim=32, win_rows=1,
                 win_cols=2, keep_global=1, keep_local=2, softmax_domain=all_keys)
    name = f"{gh}x{gw}-{dh}"
    print("case", name, flush=True)
    inp, _, ref, info = pu.screened_encoder_case(shape, 8600 + gw, 1.0, max_tries=3)
    print(name, info, pu.check_encoder(shape, inp, ref, _run_encoder(shape, inp), name))


@pytest.mark.parametrize("dtype,gh,gw,dh,batch,all_keys", [
    (wl.BF16, 1, 3, 64, 40, 0), (wl.BF16, 8, 16, 64, 40, 1), (wl.BF16, 16, 24, 64, 40, 0),  # 24, 1032, 3072 pieces
    (wl.BF16, 16, 24, 64, 38, 1), (wl.BF16, 16, 24, 64, 40, 1),                            # 760 workgroups; 3080 pieces
    (wl.BF16, 17, 18, 80, 40, 0), (wl.F32, 10, 15, 80, 40, 1), (wl.BF16, 7, 11, 40, 40, 0),
])
def test_many_segments(dtype, gh, gw, dh, batch, all_keys):
    shape = _enc(dtype, batch=batch, grid_h=gh, grid_w=gw, heads=20, head_dim=dh, feat_dim=32, win_rows=1,
                 win_cols=1, keep_global=1, keep_local=1, softmax_domain=all_keys)
    name = f"{batch}x{gh}x{gw}-{dh}"
    print("case", name, flush=True)
    inp, _, ref, info = pu.screened_encoder_case(shape, 8650 + gw, 1.0, max_tries=3)
    print(name, info, pu.check_encoder(shape, inp, ref, _run_encoder(shape, inp), name))
