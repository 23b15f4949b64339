"""Ragged batches scored in chunks of 64 keys: sequences that end inside a chunk, on its edge, with one chunk
or one key, next to one that fills the capacities; both sides of the lines in longest keys and in logits; every
sequence against the oracle on it alone."""
import pytest
import torch

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests import test_gpu_parity as tp

pytestmark = pytest.mark.gpu

LENS = [  # prefix, visual tokens, text, keep
    (10, 2060, 60, 300), (0, 64, 26, 64), (3, 65, 27, 1), (40, 640, 20, 0), (5, 1, 18, 1), (0, 1024, 66, 512),
]


# `longest`: visual tokens of the first sequence; `chunks`: what the rule takes
@pytest.mark.parametrize("dtype,longest,q_heads,kv_heads,n_query,head_dim,all_keys,in_place,chunks", [
    (wl.BF16, 2060, 14, 2, 1, 128, 0, 0, False), (wl.BF16, 2060, 14, 2, 1, 128, 1, 1, False),
    (wl.F32, 2060, 4, 2, 4, 40, 0, 0, False), (wl.F32, 2060, 8, 1, 2, 72, 1, 0, True),
    (wl.BF16, 2060, 4, 4, 8, 64, 0, 1, False),
    (wl.BF16, 2815, 14, 2, 1, 128, 0, 0, False), (wl.BF16, 2816, 14, 2, 1, 128, 0, 1, True),  # 704 KB of keys
    (wl.BF16, 2746, 14, 2, 1, 128, 1, 0, True),            # with the 70 others
    (wl.BF16, 2900, 48, 8, 1, 128, 0, 0, True), (wl.BF16, 2900, 56, 8, 1, 128, 0, 0, True),  # 336 rows of logits
    (wl.BF16, 2900, 72, 8, 1, 128, 0, 0, False),           # 432
    (wl.BF16, 2210, 28, 2, 1, 128, 0, 0, False), (wl.BF16, 2260, 28, 2, 1, 128, 0, 0, True),  # no room to stage 14 rows
    (wl.F32, 1024, 7, 1, 1, 128, 0, 1, True), (wl.F32, 2560, 4, 2, 4, 56, 0, 0, True), (wl.F32, 1023, 7, 1, 1, 128, 0, 0, False),
])
def test_ragged_chunks(monkeypatch, dtype, longest, q_heads, kv_heads, n_query, head_dim, all_keys, in_place, chunks):
    base = wl.LlmShape(dtype=dtype, batch=1, prefix=0, vis_len=1, text=n_query, n_query=n_query,
                       q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim, hidden=64, keep=1,
                       softmax_domain=all_keys, in_place=in_place)
    name = f"{longest} {q_heads}/{kv_heads}x{head_dim} all {all_keys}"
    print("case", name, flush=True)
    lens = [(10, longest, 60, 300)] + [l for l in LENS[1:] if l[1] <= longest]
    caps, meta, inp, refs = pu.ragged_llm_case(base, lens, seed=7300 + head_dim)
    q, k, v, h = (pu.to_device(inp[n], dtype) for n in ("q", "k", "v", "hidden"))
    setup = vb._ragged_setup

    def filled(*args):
        host, workspace, table = setup(*args)
        workspace.fill_(0xff)
        return host, workspace, table

    monkeypatch.setattr(vb, "_ragged_setup", filled)
    out = vb.llm_prune_ragged(caps, meta, q, k, v, h, want_scores=True)
    torch.cuda.synchronize()
    print(name, pu.check_llm_ragged(caps, meta, inp, refs, out, caps.in_place, name))
    # behind the table and the sums lie the chunks' logits and statistics
    up = lambda n: (n + 255) // 256 * 256
    rest = out["workspace"][up(16 * len(lens)) + up(4 * len(lens) * kv_heads * longest):]
    assert bool((rest != 0xff).any()) == chunks
