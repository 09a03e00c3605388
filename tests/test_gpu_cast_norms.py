"""The three weight casts of plans that store fp16 norms (no rotation, no dither): the tile factors,
and for MXFP4 the cast itself, come from the fp16 values, against the oracle bit for bit."""
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


@pytest.mark.parametrize("lat", [O.E8, O.D4, O.Z])
def test_casts_with_fp16_norms(hq, lat):
    print(f"[parity] casts with fp16 norms, lattice {lat}", flush=True)
    P = PT.oracle_params(lat, 20.0, rht_seed=31, norm_fp16=True)
    x = gauss(37, 1024, 91, 0.02, torch.bfloat16)
    plan, s = encode_gpu(hq, P, 20.0, x)
    assert s.norms.dtype == torch.float16
    oc, norms, _, _ = O.frontend(P, x.float().numpy())
    g = O.weight_factors(P, norms, 37, 1024)
    c8, g8 = hq.hq_decode_int8(plan, s)
    cf, gf = hq.hq_decode_fp8(plan, s)
    c4, s4 = hq.hq_decode_mxfp4(plan, s)
    last, gl = hq.hq_decode_fp8(plan, s, row0=36, rows=1)
    torch.cuda.synchronize()
    assert np.array_equal(g8.cpu().numpy(), g) and np.array_equal(gf.cpu().numpy(), g)
    assert np.array_equal(c8.cpu().numpy(), np.clip(oc, -127, 127))
    assert np.array_equal(cf.cpu().numpy(), O.weight_codes_fp8(oc))
    o4, os_ = O.weight_codes_mxfp4(oc, g, 128)
    assert np.array_equal(s4.cpu().numpy(), os_)
    assert np.array_equal(c4.cpu().numpy(), pack_nibbles(o4))
    assert np.array_equal(gl.cpu().numpy(), g[36:]) and torch.equal(last, cf[36:])
