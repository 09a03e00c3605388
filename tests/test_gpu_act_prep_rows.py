"""The activation prep's register form at the edges of its row lengths (512 .. 16384 columns, every
count of 2048-column steps it is built for), and the LDS form of longer tiles, all three casts, against
the oracle byte for byte; rows of zeros and strided rows among them."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from tests import parity as PT

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hq():
    from paper_2606_23406_amd import hq as H
    H.lib()
    assert torch.cuda.is_available()
    return H


@pytest.mark.parametrize("K", [512, 2048, 2560, 4096, 4608, 8192, 8704, 14336, 16384])
def test_act_prep_row_lengths(hq, K):
    check_rows(hq, K, 128)


@pytest.mark.parametrize("tile,K", [(256, 512), (256, 2560), (512, 512), (512, 14336), (1024, 3072), (2048, 2048),
                                    (2048, 16384)])
def test_act_prep_long_tiles(hq, tile, K):
    check_rows(hq, K, tile)


def check_rows(hq, K, tile):
    from paper_2606_23406_amd import workloads
    M = 5
    wide = workloads.activations(tokens=M, features=K + 512, seed=K)
    wide[2] = 0.0
    a = wide[:, :K]
    P = PT.oracle_params(O.E8, 20.0, rht_seed=49, tile=tile)
    plan = PT.gpu_plan(hq, P, 20.0, K)
    print(f"[parity] act prep K={K} tile={tile}", flush=True)
    ad = wide.cuda()[:, :K]  # rows K + 512 apart
    x8, s8 = hq.hq_act_prep(plan, ad)
    xf, sf = hq.hq_act_prep_fp8(plan, ad)
    x4, s4 = hq.hq_act_prep_mxfp4(plan, ad)
    torch.cuda.synchronize()
    an = a.float().numpy()
    for (x, s), (ox, os_) in (((x8, s8), O.act_prep(an, tile, 49)), ((xf, sf), O.act_prep_fp8(an, tile, 49))):
        assert np.array_equal(s.cpu().numpy(), os_)
        assert np.array_equal(x.cpu().numpy(), ox)
    o4, os4 = O.act_prep_mxfp4(an, tile, 49)
    assert np.array_equal(s4.cpu().numpy(), os4)
    assert np.array_equal(x4.cpu().numpy(), (o4[:, 0::2] | (o4[:, 1::2] << 4)).astype(np.uint8))
