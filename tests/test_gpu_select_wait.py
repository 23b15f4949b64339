"""The wait of the out-of-place stage-2 launch is bounded: a gathering workgroup that does not find
its indices makes the selection itself, with the same result."""
import ctypes
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    from paper_2505_22654_amd import binding as vb
    vb.lib()
    path = str(tmp_path_factory.mktemp("shim") / "libselect_shim.so")
    pkg = os.path.dirname(vb.LIB_PATH)
    subprocess.check_call(["g++", "-O1", "-fPIC", "-shared", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", "-Wno-unused-result",
                           os.path.join(ROOT, "tests", "select_shim.cpp"), "-o", path, vb.LIB_PATH,
                           f"-Wl,-rpath,{pkg}"])
    return ctypes.CDLL(path)


# one span per instantiation of the launch (spans up to 256, 512, 1024, 2048, 4096, 16384, above),
# kept rows of one and of several tiles
@pytest.mark.parametrize("V,keep,B", [(33, 11, 3), (300, 129, 2), (1000, 400, 2), (1500, 600, 1),
                                      (4000, 513, 1), (9000, 1000, 1), (20000, 700, 1)])
def test_gathering_workgroups_that_select_themselves(shim, V, keep, B):
    import torch
    Hkv, dh, Dh, vis_start, text = 2, 24, 136, 3, 5
    S = vis_start + V + text
    So = S - V + keep
    g = torch.Generator(device="cuda").manual_seed(V)
    part = torch.randint(0, 4 * V, (B, Hkv, V), generator=g, device="cuda").float()
    src = [torch.randint(0, 9999, shape, generator=g, device="cuda", dtype=torch.int16)
           for shape in ((B, Hkv, S, dh), (B, Hkv, S, dh), (B, S, Dh))]
    dims = (ctypes.c_int * 9)(B, Hkv, S, dh, Dh, vis_start, V, keep, 2)
    # ties to the lowest index: a stable descending sort of whole numbers
    want = part.sum(1).sort(dim=1, descending=True, stable=True).indices[:, :keep].sort(dim=1).values
    rows = torch.cat([torch.arange(vis_start, device="cuda").expand(B, -1), vis_start + want,
                      torch.arange(vis_start + V, S, device="cuda").expand(B, -1)], dim=1)
    for polls in (0, -1):  # nobody waits; the usual wait
        kept = torch.full((B, keep), -2, dtype=torch.int32, device="cuda")
        scores = torch.full((B, V), -1.0, device="cuda")
        dst = [torch.zeros((B, Hkv, So, dh), dtype=torch.int16, device="cuda"),
               torch.zeros((B, Hkv, So, dh), dtype=torch.int16, device="cuda"),
               torch.zeros((B, So, Dh), dtype=torch.int16, device="cuda")]
        p = lambda ts: (ctypes.c_void_p * 3)(*[t.data_ptr() for t in ts])
        rc = shim.vscan_test_select_compact(dims, polls, ctypes.c_void_p(part.data_ptr()), None,
                                            ctypes.c_void_p(kept.data_ptr()),
                                            ctypes.c_void_p(scores.data_ptr()), p(src), p(dst), None)
        torch.cuda.synchronize()
        assert rc == 0
        assert torch.equal(kept.long(), want) and torch.equal(scores, part.sum(1))
        for a, b in zip(src, dst):
            a = a if a.dim() == 4 else a[:, None]
            b = b if b.dim() == 4 else b[:, None]
            for i in range(B):
                assert torch.equal(b[i], a[i][:, rows[i]])


def test_a_device_table_that_keeps_more_than_there_is_ends():
    """The host table is what gets validated; a device table whose `keep` exceeds its `vis_len` counts
    as keeping the whole span."""
    import torch
    from paper_2505_22654_amd import binding as vb
    from paper_2505_22654_amd import workloads as wl
    B, S = 3, 90
    caps = wl.LlmShape(dtype=wl.BF16, batch=B, prefix=0, vis_len=60, text=30, n_query=1, q_heads=4,
                       kv_heads=2, head_dim=32, hidden=72, keep=40)
    g = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v, h = r(B, 4, 1, 32), r(B, 2, S, 32), r(B, 2, S, 32), r(B, S, 72)
    good = [(90, 5, 50, 20), (70, 3, 7, 7), (80, 0, 60, 40)]
    bad = [(90, 5, 50, 20), (70, 3, 7, 39), (80, 0, 60, 60)]  # 39 of 7 tokens; above the capacity
    want = vb.llm_prune_ragged(caps, good, q, k, v, h, want_scores=True)
    desc = vb.llm_desc(caps)
    host = (ctypes.c_int32 * (4 * B))(*[x for m in good for x in m])
    table = torch.tensor(bad, dtype=torch.int32, device="cuda")
    ws = torch.empty(vb.llm_workspace_size(desc), dtype=torch.uint8, device="cuda")
    kept = torch.empty_like(want["kept_idx"])
    ko, vo, ho = (torch.full_like(t, 7.0) for t in (k, v, h))
    sc = torch.full((B, 60), 7.0, device="cuda")
    p = lambda t: t.data_ptr()
    rc = vb.lib().vscan_llm_prune_ragged(ctypes.byref(desc), ctypes.addressof(host), p(table), p(q), p(k),
                                         p(v), p(h), p(kept), p(ko), p(vo), p(ho), p(sc), p(ws),
                                         ws.numel(), None)
    torch.cuda.synchronize()
    assert rc == 0 and torch.equal(kept, want["kept_idx"])
    for b, (n, _, V, kp) in enumerate(good):
        for a, c in ((ko, want["k"]), (vo, want["v"]), (ho, want["hidden"])):
            assert torch.equal(a[b, ..., :n - V + kp, :], c[b, ..., :n - V + kp, :])
