"""The ragged entry points that take the caller's device table (vscan_llm_prune_ragged and
vscan_llm_prune_fused_ragged), out of place and in place, each sequence against the oracle run on
that sequence alone.  The binding's ragged functions use the padded entry points instead."""
import ctypes

import numpy as np
import pytest

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests import test_gpu_fused as tf
from tests import test_gpu_parity as tp

pytestmark = pytest.mark.gpu


def _call(caps, meta, tensors, fused):
    """tensors: q, k, v, hidden, or hidden, w_q, w_k_t."""
    import torch
    desc, B = vb.llm_desc(caps), caps.batch
    host = (ctypes.c_int32 * (4 * B))(*[int(x) for m in meta for x in m])
    table = torch.tensor([list(map(int, m)) for m in meta], dtype=torch.int32, device="cuda")
    size = vb.llm_fused_workspace_size if fused else vb.llm_workspace_size
    ws = torch.empty(size(desc), dtype=torch.uint8, device="cuda")
    out = {"kept_idx": torch.zeros((B, caps.keep), dtype=torch.int32, device="cuda"),
           "scores": torch.zeros((B, caps.vis_len), dtype=torch.float32, device="cuda")}
    names = ("hidden",) if fused else ("k", "v", "hidden")
    moved = tensors[:1] if fused else tensors[1:]
    for n, t in zip(names, moved):
        out[n] = t if caps.in_place else torch.zeros_like(t)
    p = lambda t: t.data_ptr()
    dst = [None if caps.in_place else p(out[n]) for n in names]
    call = vb.lib().vscan_llm_prune_fused_ragged if fused else vb.lib().vscan_llm_prune_ragged
    rc = call(ctypes.byref(desc), ctypes.addressof(host), p(table), *map(p, tensors), p(out["kept_idx"]),
              *dst, p(out["scores"]), p(ws), ws.numel(), None)
    torch.cuda.synchronize()
    assert rc == 0
    return out


@pytest.mark.parametrize("variant", ["bf16", "bf16-inplace", "f32-all-keys", "bf16-gqa-inplace"])
def test_llm_ragged_with_a_device_table(variant):
    base = {
        "bf16": tp._llm(n_query=1),
        "bf16-inplace": tp._llm(in_place=1, n_query=2),
        "f32-all-keys": tp._llm(wl.F32, softmax_domain=1, head_dim=64, n_query=1),
        "bf16-gqa-inplace": tp._llm(in_place=1, q_heads=8, kv_heads=2, head_dim=128, n_query=3),
    }[variant]
    caps, meta, inp, refs = pu.ragged_llm_case(base, tp.RAGGED_SEQS, seed=7100 + len(variant))
    out = _call(caps, meta, [pu.to_device(inp[n], caps.dtype) for n in ("q", "k", "v", "hidden")], False)
    print(variant, pu.check_llm_ragged(caps, meta, inp, refs, out, caps.in_place, variant))


@pytest.mark.parametrize("variant", ["plain", "in-place-queries", "all-keys-gqa", "f32-in-place"])
def test_fused_ragged_with_a_device_table(variant):
    base = {
        "plain": tf._shape(hidden=256, q_heads=4, kv_heads=4, head_dim=32),
        "in-place-queries": tf._shape(in_place=1, n_query=2, hidden=136, q_heads=4, kv_heads=4, head_dim=32),
        "all-keys-gqa": tf._shape(softmax_domain=1, n_query=3, q_heads=8, kv_heads=2, head_dim=16,
                                  hidden=128),
        "f32-in-place": tf._shape(dtype=wl.F32, in_place=1, hidden=72, q_heads=4, kv_heads=2, head_dim=16),
    }[variant]
    seqs = [(p, v, max(t, base.n_query), k) for p, v, t, k in tf.RAGGED_SEQS]
    caps, meta, inp, refs = pu.ragged_fused_case(base, seqs, seed=9700 + len(variant))
    dev = [pu.to_device(inp["hidden"], caps.dtype), pu.to_device(inp["w_q"], caps.dtype),
           pu.to_device(np.ascontiguousarray(inp["w_k"].T), caps.dtype)]
    out = _call(caps, meta, dev, True)
    print(variant, pu.check_fused_ragged(caps, meta, inp, refs, out, caps.in_place, variant))
