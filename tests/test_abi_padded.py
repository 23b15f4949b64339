"""Host checks of the ragged calls that bring their own device table (no GPU involved)."""
import ctypes

import pytest

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl

FAKE = 0x7F0000001000


@pytest.mark.parametrize("rows,kw,status", [
    ([(139, 35, 64, 32), (139, 35, 65, 32)], {}, vb.VSCAN_ERR_SHAPE),
    ([(139, 35, 64, 32), (139, 35, 64, 33)], {}, vb.VSCAN_ERR_BUDGET),
    ([(139, 35, 64, 32)] * 2, {"hidden": None}, vb.VSCAN_ERR_NULL),
    ([(139, 35, 64, 32)] * 2, {"ws": None}, vb.VSCAN_ERR_WORKSPACE),
    ([(139, 35, 64, 32)] * 2, {"short": 1}, vb.VSCAN_ERR_WORKSPACE),
    ([(139, 35, 64, 32)] * 2, {"ws": FAKE + 8}, vb.VSCAN_ERR_ALIGN),
])
@pytest.mark.parametrize("from_hidden", [0, 1])
def test_padded_ragged_calls_validate_before_they_enqueue(rows, kw, status, from_hidden):
    shape = wl.LlmShape(dtype=wl.BF16, batch=2, prefix=35, vis_len=64, text=40, n_query=1, q_heads=8,
                        kv_heads=8, head_dim=64, hidden=512, keep=32)
    desc = vb.llm_desc(shape)
    host = (ctypes.c_int32 * 8)(*[x for r in rows for x in r])
    n = ctypes.c_size_t(0)
    assert vb.lib().vscan_llm_ragged_workspace_size(ctypes.byref(desc), from_hidden, ctypes.byref(n)) == 0
    size = vb.llm_fused_workspace_size if from_hidden else vb.llm_workspace_size
    assert n.value >= size(desc) + 2 * 16
    hidden, ws, nbytes = kw.get("hidden", FAKE), kw.get("ws", FAKE), n.value - kw.get("short", 0)
    args = ctypes.byref(desc), ctypes.addressof(host)
    if from_hidden:
        rc = vb.lib().vscan_llm_prune_fused_ragged_padded(*args, hidden, FAKE, FAKE, FAKE, FAKE, FAKE,
                                                          ws, nbytes, None)
    else:
        rc = vb.lib().vscan_llm_prune_ragged_padded(*args, FAKE, FAKE, FAKE, hidden, FAKE, FAKE, FAKE,
                                                    FAKE, FAKE, ws, nbytes, None)
    assert rc == status


@pytest.mark.parametrize("rows,error", [
    ([(139, 35, 64, 32), (139 + 2 ** 32, 35, 64, 32)], OverflowError),
    ([(139, 35, 64, 32), (139, 35, 64)], ValueError),
    ([(139, 35, 64, 32, 139), (35, 64, 32)], ValueError),
])
def test_binding_refuses_tables_that_are_no_rows_of_four_32_bit_numbers(rows, error):
    shape = wl.LlmShape(dtype=wl.BF16, batch=2, prefix=35, vis_len=64, text=40, n_query=1, q_heads=8,
                        kv_heads=8, head_dim=64, hidden=512, keep=32)
    desc = vb.llm_desc(shape)
    with pytest.raises(error):
        vb._ragged_setup(desc, rows, 2, False, "cpu")
    host, _, table = vb._ragged_setup(desc, rows[:1] * 2 if error is OverflowError else [(1, 2, 3, 4)] * 2,
                                      2, False, "cpu")
    assert len(host) == 8 and host[4] == host[0] and tuple(table.shape) == (2, 4)
