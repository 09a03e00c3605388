"""The MXFP4 cast of values that are not ordinary numbers: NaN becomes a zero (of its sign, which the
transform does not fix), an infinity saturates to 6, and blocks of fp32 subnormals keep the cast's
rule; activations in both forms of the prep (tile 128, and longer tiles through LDS), and weights whose
tile norm is infinite or NaN."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from tests import parity as PT
from tests.test_gpu_mxfp4 import pack_nibbles
from tests.test_gpu_parity import encode_gpu, gauss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hq():
    from paper_2606_23406_amd import hq as H
    H.lib()
    assert torch.cuda.is_available()
    return H


def nibbles(x):
    x = x.cpu().numpy()
    return np.stack((x & 15, x >> 4), -1).reshape(x.shape[0], -1)


def cast(y):
    """Codes, scale bytes and the NaN mask of fp32 values: the scale comes from the largest magnitude
    that is a number (an infinite one counts as 0.5 <= m 2^0), infinities saturate."""
    b = y.reshape(y.shape[0], -1, 32).astype(np.float64)
    nan = np.isnan(b)
    amax = np.where(nan, 0.0, np.abs(b)).max(axis=2)
    X = O.mx_scale_exponent(np.where(np.isinf(amax), 0.5, amax))
    codes = O.e2m1_bits(np.where(nan, 0.0, b) / np.ldexp(1.0, X)[:, :, None])
    return codes.reshape(y.shape), (X + 127).astype(np.uint8), nan.reshape(y.shape)


@pytest.mark.parametrize("tile", [128, 512])
def test_act_prep_mxfp4_unusual_rows(hq, tile):
    print(f"[parity] act_prep_mxfp4 unusual rows, tile {tile}", flush=True)
    K = 1024
    a = gauss(16, K, 93, 1.0, torch.bfloat16)
    a[0, 5] = float("nan")
    a[1, 7] = float("inf")
    a[2, 7], a[2, 300] = -float("inf"), float("nan")
    a[3, 3], a[3, 9] = float("inf"), -float("inf")
    for i, e in enumerate((-140, -133, -130, -128, -126, -124)):
        a[4 + i] = (a[4 + i].double() * 2.0 ** e).to(torch.bfloat16)
    for i, e in enumerate((120, 123, 125, 126)):  # sums past fp32's range, in some blocks
        a[10 + i] = (a[10 + i].double() * 2.0 ** e).clamp(-3e38, 3e38).to(torch.bfloat16)
    a[14, 600:] = 0.0
    P = PT.oracle_params(O.E8, 20.0, rht_seed=47, tile=tile)
    plan = PT.gpu_plan(hq, P, 20.0, K)
    xq, xs = hq.hq_act_prep_mxfp4(plan, a.cuda())
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        y = (a.float().numpy() * O.signs(47, K).astype(np.float32)).reshape(16, K // tile, tile)
        codes, scales, nan = cast(O.fwht(y).reshape(16, K))
    assert nan.any() and np.isinf(a.float().numpy()).any()
    got = nibbles(xq)
    assert np.array_equal(xs.cpu().numpy(), scales)
    assert np.all(got[nan] & 7 == 0)
    assert np.array_equal(got[~nan], codes[~nan])


def test_decode_mxfp4_unusual_norms(hq):
    print("[parity] decode_mxfp4 unusual norms", flush=True)
    P = PT.oracle_params(O.E8, 20.0, rht_seed=29)
    x = gauss(12, 1024, 95, 0.02, torch.float32)
    x[3, 5] = float("nan")
    x[4, 200] = float("inf")
    for i, e in enumerate((-60, -58, -66, -120)):
        x[5 + i] *= 2.0 ** e
    plan, s = encode_gpu(hq, P, 20.0, x)
    codes, scales = hq.hq_decode_mxfp4(plan, s)
    torch.cuda.synchronize()
    norms = s.norms[:12 * 8].cpu().numpy().reshape(12, 8)
    bad = ~np.isfinite(norms)
    assert bad[3, 0] and bad[4, 1] and bad.sum() == 2
    got = nibbles(codes).reshape(12, 8, 128)
    assert np.all(got[bad] & 7 == 0)
    assert np.all(scales.cpu().numpy().reshape(12, 8, 4)[bad] == 0)
    ok = [r for r in range(12) if r not in (3, 4)]
    oc, onorms, _, _ = O.frontend(P, x.numpy()[ok])
    o4, os_ = O.weight_codes_mxfp4(oc, O.weight_factors(P, onorms, len(ok), 1024), 128)
    assert np.array_equal(scales.cpu().numpy()[ok], os_)
    assert np.array_equal(codes.cpu().numpy()[ok], pack_nibbles(o4))
