"""The out-of-place stage-2 launch (selection, rows around the span and kept rows in one grid) at
the edges of its dispatch, and the two kinds of ragged call against each other."""
import ctypes

import pytest

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu

pytestmark = pytest.mark.gpu


def _llm(**kw):
    base = dict(dtype=wl.BF16, batch=2, prefix=5, vis_len=150, text=9, n_query=1, q_heads=4,
                kv_heads=2, head_dim=64, hidden=264, keep=40)
    base.update(kw)
    return wl.LlmShape(**base)


EDGES = {f"span-{v}": _llm(vis_len=v, keep=max(1, v // 3)) for v in
         (1, 2, 255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097)}
EDGES.update({
    # whole and partial tiles of 128 kept rows; nothing and everything kept; no prefix
    "keep-127": _llm(keep=127), "keep-128": _llm(keep=128), "keep-129": _llm(keep=129),
    "keep-none": _llm(keep=0), "keep-all": _llm(keep=150), "no-prefix": _llm(prefix=0),
    # static rows of several units per slab, and rows of more than one 256-byte strip
    "long-text": _llm(text=700, prefix=300, head_dim=256, hidden=1032),
    "f32": _llm(dtype=wl.F32, head_dim=128),
    # more sequences than the chip holds workgroups: the selections alone take several rounds
    "many-sequences": _llm(batch=2500, vis_len=33, keep=11, q_heads=2, hidden=64),
})


@pytest.mark.parametrize("name", sorted(EDGES))
def test_selection_and_copies_in_one_launch(name):
    import torch
    shape = EDGES[name]
    inp, ref, info = pu.screened_llm_case(shape, 9700, max_tries=2 if shape.batch > 2 else 16)
    dev = [pu.to_device(inp[n], shape.dtype) for n in ("q", "k", "v", "hidden")]
    out = vb.llm_prune(shape, *dev, want_scores=True)
    torch.cuda.synchronize()
    print(name, info, pu.check_llm(shape, inp, ref, out, name))


@pytest.mark.parametrize("batch", [1, 3, 128, 129, 300])
def test_padded_ragged_call_equals_the_one_with_a_device_table(batch):
    """Same results; rows and scores past them zero in the padded call, untouched in the other."""
    import torch
    caps = _llm(batch=batch, prefix=0, vis_len=60, text=40, keep=25, head_dim=32, hidden=72)
    g = torch.Generator(device="cuda").manual_seed(batch)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    q, k = r(batch, 4, 1, 32), r(batch, 2, 100, 32)
    v, h = torch.randn_like(k), r(batch, 100, 72)
    meta = [(60 + 7 * b % 41, b % 9, 1 + 13 * b % 50, min(1 + 13 * b % 50, b % 26)) for b in range(batch)]
    pad = vb.llm_prune_ragged(caps, meta, q, k, v, h, want_scores=True)
    assert pad["meta_device"].cpu().tolist() == [list(m) for m in meta]
    desc = vb.llm_desc(caps)
    host = (ctypes.c_int32 * (4 * batch))(*[x for m in meta for x in m])
    table = torch.tensor(meta, dtype=torch.int32, device="cuda")
    ws = torch.empty(vb.llm_workspace_size(desc), dtype=torch.uint8, device="cuda")
    kept = torch.empty_like(pad["kept_idx"])
    ko, vo, ho = (torch.full_like(t, 7.0) for t in (k, v, h))
    sc = torch.full((batch, 60), 7.0, device="cuda")
    p = lambda t: t.data_ptr()
    rc = vb.lib().vscan_llm_prune_ragged(ctypes.byref(desc), ctypes.addressof(host), p(table), p(q), p(k),
                                         p(v), p(h), p(kept), p(ko), p(vo), p(ho), p(sc), p(ws),
                                         ws.numel(), None)
    torch.cuda.synchronize()
    assert rc == 0 and torch.equal(kept, pad["kept_idx"])
    for b, (S, vs, V, kp) in enumerate(meta):
        n = S - V + kp
        assert torch.equal(sc[b, :V], pad["scores"][b, :V])
        assert (sc[b, V:] == 7).all() and not pad["scores"][b, V:].any()
        for a, c in ((ko, pad["k"]), (vo, pad["v"]), (ho, pad["hidden"])):
            assert torch.equal(a[b, ..., :n, :], c[b, ..., :n, :])
            assert (a[b, ..., n:, :] == 7).all() and not c[b, ..., n:, :].any()


def test_more_workgroups_than_one_grid_dimension_holds():
    """4.48 million slabs of three 16-byte rows: four workgroups to a slab, and a grid dimension ends
    below 2^32 threads."""
    import torch
    shape = _llm(batch=140000, prefix=0, vis_len=2, text=1, q_heads=32, kv_heads=32, head_dim=8,
                 hidden=8, keep=1)
    assert shape.batch * shape.kv_heads * 4 * 256 > 2 ** 32
    g = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    B = shape.batch
    q, k, v, h = r(B, 32, 1, 8), r(B, 32, 3, 8), r(B, 32, 3, 8), r(B, 3, 8)
    out = vb.llm_prune(shape, q, k, v, h, want_scores=True)
    torch.cuda.synchronize()
    kept = out["kept_idx"].long()
    assert torch.equal(kept[:, 0], (out["scores"][:, 1] > out["scores"][:, 0]).long())
    rows = torch.cat([kept, torch.full_like(kept, 2)], dim=1)
    for got, src in ((out["k"], k), (out["v"], v), (out["hidden"][:, None], h[:, None])):
        want = torch.gather(src, 2, rows[:, None, :, None].expand(-1, src.shape[1], -1, 8))
        assert torch.equal(got, want)
