"""Stage-2 scores of few items with long key domains (chunks of 64 keys on the matrix cores): row
lengths that end inside a chunk, inside and past a batch of loads, query-row counts at their limits,
domains that end inside a wave's keys, causal rows; against the oracle."""
import pytest

from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _llm, _run_llm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("batch,vis,hq,hkv,n_query,dh,all_keys", [
    (1, 1024, 1, 1, 1, 8, 0), (1, 1025, 16, 1, 1, 24, 0), (2, 1087, 3, 3, 5, 40, 1),
    (1, 1030, 7, 1, 1, 128, 1), (1, 1041, 2, 2, 16, 136, 0), (3, 1100, 4, 2, 8, 256, 1)])
def test_scores(dtype, batch, vis, hq, hkv, n_query, dh, all_keys):
    dh = dh if dtype == wl.BF16 else min(dh, 128)  # rows of up to 512 bytes
    shape = _llm(dtype, batch=batch, prefix=5, vis_len=vis, text=17, n_query=n_query, q_heads=hq,
                 kv_heads=hkv, head_dim=dh, hidden=64, keep=200, softmax_domain=all_keys)
    name = f"{dtype} {batch}x{vis} {hq}/{hkv}x{n_query} {dh} {all_keys}"
    inp, ref, info = pu.screened_llm_case(shape, 6100 + vis)
    print("case", name, info, flush=True)
    out = _run_llm(shape, inp)
    print(pu.check_llm(shape, inp, ref, out, name))
