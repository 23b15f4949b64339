"""Ragged batches scored in chunks of 64 keys: sequences that end inside a chunk, on its edge, with one chunk
or one key, next to one that fills the capacities; longest keys on both sides of half a megabyte; every
sequence against the oracle on it alone."""
import pytest

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests import test_gpu_parity as tp

pytestmark = pytest.mark.gpu

LENS = [  # prefix, visual tokens, text, keep
    (10, 2060, 60, 300), (0, 64, 26, 64), (3, 65, 27, 1), (40, 640, 20, 0), (5, 1, 18, 1), (0, 1024, 66, 512),
]


@pytest.mark.parametrize("dtype,q_heads,kv_heads,n_query,head_dim,all_keys,in_place", [
    (wl.BF16, 14, 2, 1, 128, 0, 0), (wl.BF16, 14, 2, 1, 128, 1, 1), (wl.F32, 4, 2, 4, 40, 0, 0),
    (wl.F32, 8, 1, 2, 72, 1, 0), (wl.BF16, 4, 4, 8, 64, 0, 1),
])
def test_ragged_chunks(dtype, q_heads, kv_heads, n_query, head_dim, all_keys, in_place):
    base = wl.LlmShape(dtype=dtype, batch=1, prefix=0, vis_len=1, text=n_query, n_query=n_query,
                       q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim, hidden=64, keep=1,
                       softmax_domain=all_keys, in_place=in_place)
    name = f"{q_heads}/{kv_heads}x{head_dim} all {all_keys}"
    print("case", name, flush=True)
    caps, meta, inp, refs = pu.ragged_llm_case(base, LENS, seed=7300 + head_dim)
    q, k, v, h = (pu.to_device(inp[n], dtype) for n in ("q", "k", "v", "hidden"))
    out = vb.llm_prune_ragged(caps, meta, q, k, v, h, want_scores=True)
    import torch
    torch.cuda.synchronize()
    print(name, pu.check_llm_ragged(caps, meta, inp, refs, out, caps.in_place, name))
