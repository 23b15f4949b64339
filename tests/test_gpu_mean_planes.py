"""Mean-attention scores of fp32 queries and keys: the form that carries them as pairs of fp16
planes, at the edges of its blocks (128 rows), stages (64) and tiles (32), for every operand width
it is built for, against the definition in 64 bits."""
import numpy as np
import pytest

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl
from tests import parity_utils as pu

pytestmark = pytest.mark.gpu

# The repository's score tolerance.  A logit of a few units is off by less than 2^-21 of the sum of
# its products' magnitudes (operands to 2^-23, the dropped product 2^-22, five roundings of 2^-24),
# here below 2e-6; the exponential turns that into the same relative error of a score.
RTOL = 2e-5


def _shape(gh, gw, dh, heads=2, batch=1, crops=1, has_cls=0, all_keys=0):
    return wl.EncoderShape(dtype=wl.F32, batch=batch, n_segments=crops, grid_h=gh, grid_w=gw,
                           has_cls=has_cls, score_mode=1, heads=heads, head_dim=dh, feat_dim=64,
                           win_rows=1, win_cols=1, keep_global=2, keep_local=1,
                           softmax_domain=all_keys)


def _scores(q, k, has_cls, all_keys):
    """[B, C, H, S, dh] -> [B, C*N]"""
    q, k = q.astype(np.float64), k.astype(np.float64)
    dh = q.shape[-1]
    z = np.matmul(q[..., has_cls:, :], np.swapaxes(k if all_keys else k[..., has_cls:, :], -1, -2))
    z = z / np.sqrt(dh)
    z = np.exp(z - z.max(axis=-1, keepdims=True))
    p = z / z.sum(axis=-1, keepdims=True)
    if all_keys:
        p = p[..., has_cls:]
    s = p.mean(axis=-2).mean(axis=2)
    return s.reshape(s.shape[0], -1)


def _run(shape, q, k, cut=0):
    import torch
    x = torch.randn((shape.batch, shape.tokens_per_image, shape.feat_dim), device="cuda")
    ws = torch.empty(vb.encoder_workspace_size(vb.encoder_desc(shape)) - cut, dtype=torch.uint8, device="cuda")
    out = vb.encoder_reduce(shape, pu.to_device(q, wl.F32), pu.to_device(k, wl.F32), x,
                            want_scores=True, workspace=ws)
    torch.cuda.synchronize()
    return pu.to_host(out["scores"])


@pytest.mark.parametrize("gh,gw,dh,heads,crops,has_cls,all_keys", [
    (1, 3, 8, 1, 1, 0, 0), (1, 31, 16, 2, 1, 0, 0), (4, 8, 32, 2, 1, 1, 1), (3, 11, 40, 2, 1, 1, 1),
    (7, 9, 64, 3, 1, 0, 0), (8, 8, 64, 2, 2, 1, 1), (5, 13, 72, 2, 1, 0, 0), (8, 16, 80, 2, 2, 1, 1),
    (3, 43, 80, 2, 1, 1, 0), (16, 16, 80, 2, 1, 1, 1), (1, 257, 80, 1, 1, 0, 0), (12, 16, 88, 2, 1, 0, 0),
    (11, 12, 128, 2, 2, 1, 1), (20, 20, 128, 2, 1, 0, 0),
    # enough heads and rows for the form with 64 resident rows per wave, in every width
    (12, 20, 32, 256, 1, 0, 0), (16, 27, 64, 128, 1, 1, 1), (16, 16, 80, 256, 1, 1, 1),
    (17, 27, 80, 128, 1, 0, 0)])
def test_scores(gh, gw, dh, heads, crops, has_cls, all_keys):
    shape = _shape(gh, gw, dh, heads, 1, crops, has_cls, all_keys)
    rng = np.random.default_rng(gh * 1000 + gw * 10 + dh)
    q, k = (rng.standard_normal((1, crops, heads, shape.rows, dh)).astype(np.float32) for _ in range(2))
    print("case", gh, gw, dh, heads, crops, has_cls, all_keys, flush=True)
    want = _scores(q, k, has_cls, all_keys)
    got = _run(shape, q, k)
    np.testing.assert_allclose(got, want, rtol=RTOL)
    # a workspace without room for the planes: the fp32 matrix instructions
    if heads <= 3:
        np.testing.assert_allclose(_run(shape, q, k, cut=1), want, rtol=RTOL)


@pytest.mark.parametrize("gain", [1e30, 1e-30, 3e-39])
def test_scores_far_from_one(gain):
    """Magnitudes outside the range of fp16: what q loses k gains, so the logits stay the same (the
    last gain makes q subnormal)."""
    shape = _shape(9, 15, 80)
    rng = np.random.default_rng(7)
    q, k = (rng.standard_normal((1, 1, 2, 135, 80)).astype(np.float32) for _ in range(2))
    q, k = (q * np.float64(gain)).astype(np.float32), (k / max(gain, 1e-35)).astype(np.float32)
    # fp32 holds fewer bits of a subnormal q, in the reference as here
    np.testing.assert_allclose(_run(shape, q, k), _scores(q, k, 0, 0), rtol=RTOL)


def test_blocks_of_unlike_magnitude():
    """Rows of one head whose blocks differ in scale by 2^20, and a block of zeros."""
    shape = _shape(17, 25, 64)
    rng = np.random.default_rng(8)
    q, k = (rng.standard_normal((1, 1, 2, 425, 64)).astype(np.float32) for _ in range(2))
    k[..., 128:256, :] *= 2.0 ** -20
    k[..., 300:, :] *= 0.25
    q[..., 256:384, :] = 0.0
    np.testing.assert_allclose(_run(shape, q, k), _scores(q, k, 0, 0), rtol=RTOL)


def test_zero_and_infinite_inputs():
    shape = _shape(6, 7, 64)
    z = np.zeros((1, 1, 2, 42, 64), np.float32)
    np.testing.assert_allclose(_run(shape, z, z), np.full((1, 42), 1 / 42, np.float32), rtol=1e-6)
    rng = np.random.default_rng(9)
    q, k = (rng.standard_normal(z.shape).astype(np.float32) for _ in range(2))
    q[0, 0, 1, 5, 3] = np.inf
    assert np.isnan(_run(shape, q, k)).all()   # as one infinite logit does in the fp32 form
