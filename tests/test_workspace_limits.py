"""Workspace sizes are part of what a caller may have kept: a buffer of the size once asked for, and
the fixed scratch of vscan_llm_prune_static, hold what they always held."""
import pytest

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl


def _shape(**kw):
    base = dict(dtype=wl.BF16, batch=3, prefix=7, vis_len=700, text=33, n_query=1, q_heads=8,
                kv_heads=4, head_dim=64, hidden=256, keep=200)
    base.update(kw)
    return wl.LlmShape(**base)


# stage 2 needs the partial scores (and the split form's logits and statistics) and nothing else
@pytest.mark.parametrize("kw,qk,fused", [
    (dict(batch=32, vis_len=4096, kv_heads=32, q_heads=32), 16 << 20, 19791872),
    (dict(batch=64, vis_len=2048, kv_heads=32, q_heads=32), 16 << 20, None),
    (dict(batch=16, vis_len=8192, kv_heads=32, q_heads=32), 16 << 20, 18546688),
    (dict(), 33792, 201216),
    (dict(batch=1, vis_len=4096, q_heads=28), 538624, 1001984),
])
@pytest.mark.parametrize("in_place", [0, 1])
def test_stage2_sizes_hold_scores_only(kw, qk, fused, in_place):
    desc = vb.llm_desc(_shape(in_place=in_place, **kw))
    assert vb.llm_workspace_size(desc) == qk
    if fused is not None:
        assert vb.llm_fused_workspace_size(desc) == fused


@pytest.mark.gpu
@pytest.mark.parametrize("batch,vis_len", [(32, 4096), (64, 2048), (16, 8192)])
def test_static_scratch_takes_calls_of_exactly_its_size(batch, vis_len):
    import torch
    shape = _shape(batch=batch, vis_len=vis_len, kv_heads=32, q_heads=32, head_dim=8, hidden=8,
                   prefix=1, text=1, keep=64)
    assert vb.llm_workspace_size(vb.llm_desc(shape)) == vb.STATIC_SCRATCH_BYTES
    g = torch.Generator(device="cuda").manual_seed(vis_len)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    S = shape.seq_len
    args = r(batch, 32, 1, 8), r(batch, 32, S, 8), r(batch, 32, S, 8), r(batch, S, 8)
    got = vb.llm_prune(shape, *args, want_scores=True, static_scratch=True)
    want = vb.llm_prune(shape, *args, want_scores=True)
    torch.cuda.synchronize()
    for name in ("kept_idx", "scores", "k", "v", "hidden"):
        assert torch.equal(got[name], want[name]), name
