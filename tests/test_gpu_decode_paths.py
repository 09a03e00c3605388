"""Sub-streams on either side of every turn of the decoder's parse, against the oracle bit for bit.

The parse has a path without per-lane branches for sub-streams of at most 126 words and 64 unary
words whose groups of 8 codes fit 32 bits (remainders too), and a general one; plain weight plans
then transform codes below 25 2^4 on the matrix cores and others on the VALU.  A fixed Rice parameter
moves a stream over those lines: small k makes long unary parts and windows past 32 bits, large k
long remainders.
"""
import pytest
import torch

from oracle import oracle as O
from tests import parity as PT
from tests.test_gpu_parity import check_roundtrip, gauss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hq():
    from paper_2606_23406_amd import hq as H
    H.lib()
    assert torch.cuda.is_available()
    return H


@pytest.mark.parametrize("lat", [O.E8, O.D4, O.A2, O.Z])
@pytest.mark.parametrize("snr,rice_k", [
    (8.0, 0),    # short codes: every unary part in few words, no remainders (E8, Z)
    (22.7, 0),   # unary parts past 64 words: the general path
    (22.7, 1),   # up to 64 unary words, some windows past 32 bits
    (22.7, 3), (30.0, 4),   # the common path; the largest k of the matrix-core transform
    (36.0, 4),   # codes in the hundreds: both transforms, windows past 32 bits
    (36.0, 5),   # past it (lrem 40 for E8 and Z: the general path; D4 and A2 mixed)
    (40.0, 7),   # 56 remainder bits
])
@pytest.mark.parametrize("rows", [3, 4100])   # one sub-stream per wave, and four (a ragged last wave)
def test_parse_paths(hq, lat, snr, rice_k, rows):
    cols = 512 if rows == 3 else 2048
    P = PT.oracle_params(lat, snr, rht_seed=71, rice_k=rice_k)
    x = gauss(rows, cols, 500 + rows, 0.02, torch.bfloat16)
    check_roundtrip(hq, P, snr, x, f"parse paths lattice {lat} {snr} dB k={rice_k}")
