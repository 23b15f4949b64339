"""Scores from hidden states where few query rows are projected by one launch and the selection adds
the softmax rows itself: the edges of the sixteen-row blocks, of a wave's share of the contraction
axis and of its batches, and the first sizes past each rule, against the definition in 64 bits."""
import pytest

from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_fused import _enc, _run, _run_encoder, _shape

pytestmark = pytest.mark.gpu

LLM = {  # batch, n_query, q_heads, kv_heads, head_dim, hidden, vis_len
    "one-row-one-chunk": (1, 1, 1, 1, 8, 8, 40), "sixteen-rows": (16, 1, 4, 2, 24, 264, 33),
    "seventeen-rows": (17, 1, 2, 2, 40, 136, 64), "thirty-two-rows": (8, 4, 3, 1, 16, 1000, 50),
    "thirty-three-rows": (11, 3, 2, 1, 16, 72, 50), "several-batches": (2, 2, 2, 1, 32, 4096, 70),
    "most-rows-kept": (1, 8, 8, 8, 16, 64, 512), "summed-before": (1, 8, 8, 8, 16, 64, 513),
}
EDGES = {  # the same fields
    "rows-past-the-rule": (1, 9, 8, 8, 16, 64, 400),
    # the widest weights that q takes in one launch, and the first wider ones
    "two-batches-f32": (9, 1, 2, 1, 16, 2048, 40), "past-two-or-four-batches": (1, 2, 2, 1, 16, 4104, 40),
    "past-two-batches-f32": (9, 1, 2, 1, 16, 2056, 40),
    "one-batch": (9, 2, 2, 1, 16, 2048, 40), "past-one-batch": (9, 2, 2, 1, 16, 2056, 40),
    "one-batch-f32": (9, 2, 2, 1, 16, 1024, 40), "past-one-batch-f32": (9, 2, 2, 1, 16, 1032, 40),
    "most-outputs": (1, 1, 32, 32, 128, 64, 40), "past-most-outputs": (1, 1, 33, 33, 128, 64, 40),
}


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("name", sorted(LLM))
@pytest.mark.parametrize("in_place", [0, 1])
def test_stage2(name, dtype, in_place):
    batch, n_query, hq, hkv, dh, hidden, vis = LLM[name]
    shape = _shape(dtype=dtype, batch=batch, n_query=n_query, q_heads=hq, kv_heads=hkv, head_dim=dh,
                   hidden=hidden, vis_len=vis, keep=vis // 3, in_place=in_place)
    inp, ref, info = pu.screened_fused_case(shape, 7300 + sorted(LLM).index(name) * 31)
    print("case", name, dtype, in_place, info, flush=True)
    out = _run(shape, inp)
    print(pu.check_fused(shape, ref, out, name, hidden=inp["hidden"]))


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("name", sorted(EDGES))
def test_stage2_at_the_edges_of_the_rules(name, dtype):
    batch, n_query, hq, hkv, dh, hidden, vis = EDGES[name]
    shape = _shape(dtype=dtype, batch=batch, n_query=n_query, q_heads=hq, kv_heads=hkv, head_dim=dh,
                   hidden=hidden, vis_len=vis, keep=vis // 3)
    inp, ref, info = pu.screened_fused_case(shape, 7500 + sorted(EDGES).index(name) * 31)
    print("case", name, dtype, info, flush=True)
    out = _run(shape, inp)
    print(pu.check_fused(shape, ref, out, name, hidden=inp["hidden"]))


@pytest.mark.parametrize("batch,crops,heads,dh,feat", [(1, 1, 1, 8, 8), (3, 5, 3, 40, 200), (3, 6, 2, 24, 1000),
                                                       (11, 3, 2, 16, 72)])
def test_stage1(batch, crops, heads, dh, feat):
    shape = _enc(batch=batch, n_segments=crops, grid_h=6, grid_w=7, heads=heads, head_dim=dh, feat_dim=feat,
                 win_rows=2, win_cols=2, keep_global=5, keep_local=6)
    inp, _, ref, info = pu.screened_encoder_fused_case(shape, 7400 + feat, max_tries=6)
    print("case", batch, crops, heads, dh, feat, info, flush=True)
    out = _run_encoder(shape, inp)
    print(pu.check_encoder(shape, inp, ref, out, "fused encoder, few query rows"))
