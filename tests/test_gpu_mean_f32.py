"""Mean attention of fp32 rows, whose values the pipelined form multiplies as bf16 planes: elements at the top of the range, and
the error of the scores against 64 bits."""
import numpy as np
import pytest

from oracle import vscan_oracle as vo
from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu
from tests.test_gpu_parity import _enc, _run_encoder

pytestmark = pytest.mark.gpu

TOP = np.finfo(np.float32).max


# (head size, grid): one chunk more than the rows fill, stages of 128 and of 64 rows, one and more parts
@pytest.mark.parametrize("dh,gh,gw", [(64, 12, 11), (72, 13, 21), (80, 31, 33), (128, 17, 17), (8, 24, 26),
                                      (64, 8, 16), (8, 11, 12)])  # (these two: the plain form)
def test_largest_finite_values(dh, gh, gw):
    """Keys and queries with elements at the top of the range whose products are nought, far below every other
    logit, or below the range: the oracle's scores, and no NaN."""
    shape = _enc(wl.F32, batch=1, grid_h=gh, grid_w=gw, heads=2, head_dim=dh, feat_dim=16, win_rows=1, win_cols=1,
                 keep_global=7, keep_local=0, has_cls=0, score_mode=1)
    print("case", dh, gh, gw, flush=True)
    inp = wl.encoder_inputs(shape, 8500 + dh, 0.25)
    q, k, rng = inp["q"], inp["k"], np.random.default_rng(dh)  # [B, C, H, S, dh]
    rows = rng.choice(gh * gw, 7, replace=False)
    q[..., 1] = 0.0                        # nought against either sign
    k[..., rows[0], 1], k[..., rows[1], 1] = TOP, -TOP
    k[..., 2] = 0.0                        # the same from the other side
    q[..., rows[2], 2], q[..., rows[3], 2] = TOP, -TOP
    q[..., 3] = rng.uniform(1e-30, 2e-30, q.shape[:-1])  # -1e8 and below
    k[..., rows[4], 3] = -TOP
    if dh == 64:                           # a row of padding: below the range
        q[...] = np.abs(q)
        k[..., rows[5], :] = -TOP
        q[..., rows[2], 2] = q[..., rows[3], 2] = 0.0
    ref = vo.encoder_reduce(shape, q, k, inp["x"])
    out = _run_encoder(shape, inp)
    print(dh, pu.check_encoder(shape, inp, ref, out, f"{dh}"), flush=True)
    scores = pu.to_host(out["scores"]).reshape(-1)
    assert scores[rows[4]] == 0 and (dh != 64 or scores[rows[5]] == 0)


def _two_norm(out, ref):
    got, want = pu.to_host(out["scores"]).astype(np.float64).reshape(-1), ref["scores"].reshape(-1)
    return np.linalg.norm(got - want) / np.linalg.norm(want)


# What the planes leave out, mid x lo and lo x mid, is up to 2^-24 of a product: as much as the rounding of an fp32
# product, where every element has both planes at the end of their range.  `most`: the error that fp32 instructions
# left on the same inputs; on planes 0.7, 2.4, 0.9, 3.3, 1.9 and 1.1e-7.
@pytest.mark.parametrize("dh,heads,gh,gw,gain,most", [
    (64, 8, 18, 18, 1.0, 1.9e-7), (64, 8, 18, 18, 8.0, 3.4e-7), (80, 4, 31, 33, 1.0, 1.9e-7),
    (80, 4, 31, 33, 8.0, 4.2e-7), (128, 2, 24, 27, 4.0, 2.7e-7), (72, 3, 17, 19, 2.0, 2.0e-7),
])
def test_products_with_the_most_left_out(dh, heads, gh, gw, gain, most):
    shape = _enc(wl.F32, batch=1, grid_h=gh, grid_w=gw, heads=heads, head_dim=dh, feat_dim=16, win_rows=1,
                 win_cols=1, keep_global=7, keep_local=0, has_cls=0, score_mode=1)
    print("case", dh, gh, gw, gain, flush=True)
    inp = wl.encoder_inputs(shape, 8600 + dh, 0.25)
    rng = np.random.default_rng(dh)
    x = np.float32(1 + 2.0 ** -8 - 2.0 ** -17 - 2.0 ** -23)
    for name, size in (("q", np.float32(gain)), ("k", np.float32(1))):
        inp[name] = (rng.choice(np.array([-x, x], np.float32), inp[name].shape) * size).astype(np.float32)
    error = _two_norm(_run_encoder(shape, inp), vo.encoder_reduce(shape, inp["q"], inp["k"], inp["x"]))
    print("error", error, flush=True)
    assert error < most


# Given rows and rows projected from hidden states: fp32 instructions left up to 5.6e-7 and 12.8e-7 on these inputs,
# planes 1.6e-7 and 4.8e-7.
@pytest.mark.parametrize("hidden,most", [(0, 2.5e-7), (1, 8e-7)])
@pytest.mark.parametrize("dh,heads,gh,gw", [(64, 8, 18, 18), (80, 4, 31, 33), (80, 16, 24, 24), (128, 2, 24, 27)])
def test_scores_against_64_bits(dh, heads, gh, gw, hidden, most):
    import torch
    shape = _enc(wl.F32, batch=1, grid_h=gh, grid_w=gw, heads=heads, head_dim=dh, feat_dim=dh * heads, win_rows=1,
                 win_cols=1, keep_global=7, keep_local=0, has_cls=0, score_mode=1)
    dev = lambda a: pu.to_device(np.ascontiguousarray(a), wl.F32)
    for seed in range(3):
        print("case", dh, gh, gw, hidden, seed, flush=True)
        if hidden:
            inp = wl.encoder_hidden_inputs(shape, 8700 + seed)
            ref = vo.encoder_reduce_fused(shape, inp["hidden"], inp["w_q"], inp["w_k"], inp["x"])
            out = vb.encoder_reduce_fused(shape, dev(inp["hidden"]), dev(inp["w_q"]), dev(inp["w_k"].T),
                                          dev(inp["x"]), want_scores=True)
            torch.cuda.synchronize()
        else:
            inp = wl.encoder_inputs(shape, 8700 + seed, 0.25)
            ref = vo.encoder_reduce(shape, inp["q"], inp["k"], inp["x"])
            out = _run_encoder(shape, inp)
        error = _two_norm(out, ref)
        print("error", error, flush=True)
        assert error < most


@pytest.mark.parametrize("power", [60, 100])
def test_far_apart_exponents(power):
    """Small values against large ones: the planes of 2^-100 are still whole."""
    shape = _enc(wl.F32, batch=1, grid_h=18, grid_w=18, heads=8, head_dim=64, feat_dim=16, win_rows=1, win_cols=1,
                 keep_global=7, keep_local=0, has_cls=0, score_mode=1)
    print("case", power, flush=True)
    for small, large in (("q", "k"), ("k", "q")):
        inp = wl.encoder_inputs(shape, 8800, 0.25)
        inp[small], inp[large] = inp[small] * np.float32(2.0 ** -power), inp[large] * np.float32(2.0 ** power)
        error = _two_norm(_run_encoder(shape, inp), vo.encoder_reduce(shape, inp["q"], inp["k"], inp["x"]))
        print(small, "error", error, flush=True)
        assert error < 2.5e-7  # as for drawn rows
