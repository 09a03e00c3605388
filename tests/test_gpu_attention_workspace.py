"""The attention's workspace size over batch and token counts: never less for a larger call (one
workspace for the largest serves every smaller one), also where the tokens a wave takes step up, and
a workspace of a larger call is accepted by a smaller one whose own split count is higher."""
import pytest
import torch

from oracle import oracle as O
from tests import parity as PT
from tests.test_gpu_attention import SNR, N, kv_pair, paged

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hq():
    from paper_2606_23406_amd import hq as H
    H.lib()
    assert torch.cuda.is_available()
    return H


@pytest.mark.parametrize("heads_kv", [4, 8, 32])
def test_workspace_never_falls(hq, heads_kv):
    plan = PT.gpu_plan(hq, PT.oracle_params(O.E8, SNR[O.E8], rht_seed=41), SNR[O.E8], heads_kv * N)
    tokens = sorted({t for b in range(0, 19) for t in ((1 << b) - 1, 1 << b, (1 << b) + 1, 5 << b) if t > 0})
    for group in (1, 8):
        size = {(b, t): hq.hq_attention_workspace_bytes(plan, b, group * heads_kv, t)
                for b in (1, 2, 3, 15, 16, 17, 64, 512) for t in tokens}
        for (b, t), n in size.items():
            assert all(n <= m for (b2, t2), m in size.items() if b2 >= b and t2 >= t), (b, t)


def test_workspace_of_a_larger_call(hq):
    # 4 KV heads in one sub-stream per row: 16 sequences of 4096 tokens take 4 tokens a wave, 4160
    # take 5 and a fifth fewer splits
    import numpy as np
    rng = np.random.default_rng(3)
    K, V = kv_pair(hq, O.E8, 64, 4, 13)
    lens = [20, 16, 10]
    table = np.zeros((16, 256), dtype=np.int32)
    table[:3, :2] = paged(rng, lens, 16, 4)
    q = torch.randn((16, 4, N), device="cuda")
    ln = torch.tensor(lens + [0] * 13, dtype=torch.int32, device="cuda")
    t = torch.from_numpy(table).cuda()
    ws = torch.empty(hq.hq_attention_workspace_bytes(K[1], 16, 4, 260 * 16), dtype=torch.uint8, device="cuda")
    a = hq.hq_decode_attention(K[1], K[2], V[1], V[2], q, t, ln, 16, workspace=ws)
    b = hq.hq_decode_attention(K[1], K[2], V[1], V[2], q, t, ln, 16)
    torch.cuda.synchronize()
    assert torch.equal(a[:3], b[:3])
