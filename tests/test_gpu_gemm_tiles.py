"""The block-scaled GEMMs in every workgroup tile the dispatch picks, against a 64-bit product.

Sizes: 64 x 64 tiles up to 512 of them, then 128 x 128, 256 x 128 or 256 x 256 (the last not for factor
tiles longer than 128), whichever take the fewest weighted rounds of the chip; edges off every tile in
both directions, the shortest K (no more stages than the LDS ring holds) and a K that fills the ring
again at least twice, MXFP4's stages of 256 included.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

E2M1 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]


@pytest.fixture(scope="module")
def hq():
    from paper_2606_23406_amd import hq as m
    m.lib()
    return m


def _operands(cast, M, N, K, tile):
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 7 + N * 3 + K)

    def rand(lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=g, device="cuda")

    def factors(*shape):
        return torch.rand(shape, generator=g, device="cuda") + 0.5

    if cast == "mxfp4":
        val = torch.tensor(E2M1 + [-v for v in E2M1], dtype=torch.float64, device="cuda")
        ops, dense = [], []
        for rows in (M, N):
            c, s = rand(0, 256, rows, K // 2), rand(121, 130, rows, K // 32)
            v = torch.stack((val[c & 15], val[c >> 4]), -1).reshape(rows, K // 32, 32)
            dense.append((v * torch.exp2(s.double() - 127)[..., None]).reshape(rows, K))
            ops += [c.to(torch.uint8), s.to(torch.uint8)]
        return ops, dense[0], dense[1]
    sx, gw = factors(M), factors(N, K // tile)
    if cast == "int8":
        x, w = rand(-128, 128, M, K).to(torch.int8), rand(-128, 128, N, K).to(torch.int8)
        X, W = x.double(), w.double()
    else:
        xf = (torch.randn((M, K), generator=g, device="cuda") * 60).clamp(-448, 448).to(torch.float8_e4m3fn)
        wf = (torch.randn((N, K), generator=g, device="cuda") * 12).to(torch.float8_e4m3fn)
        x, w, X, W = xf.view(torch.uint8), wf.view(torch.uint8), xf.double(), wf.double()
    W = (W.reshape(N, K // tile, tile) * gw.double()[..., None]).reshape(N, K)
    return [x, sx, w, gw], X * sx.double()[:, None], W


@pytest.mark.parametrize("cast,tile", [("int8", 128), ("int8", 512), ("fp8", 128), ("fp8", 512),
                                       ("mxfp4", 128)])
@pytest.mark.parametrize("M,N,K", [
    (1, 1, 512), (63, 130, 512), (65, 64, 2560),          # 64 x 64
    (1100, 2050, 1024), (1100, 2050, 2560),               # 128 x 128
    (500, 11000, 512), (500, 11000, 2560),                # 256 x 128
    (2000, 3900, 1024),                                   # long factor tiles: 256 x 128
    (3000, 3001, 512), (3000, 3001, 1536),                # 256 x 256
])
def test_gemm_workgroup_tiles(hq, cast, tile, M, N, K):
    print(f"[parity] gemm {cast} tile {tile} {M}x{N}x{K}", flush=True)
    plan = hq.hq_plan(tile=tile, lattice=hq.HQ_E8, bps=4.0, cols=K)
    ops, X, W = _operands(cast, M, N, K, tile)
    ref = X @ W.T.contiguous()
    fn = {"int8": hq.hq_gemm_int8_blockscaled, "fp8": hq.hq_gemm_fp8_blockscaled,
          "mxfp4": hq.hq_gemm_mxfp4_blockscaled}[cast]
    # rows past the output stay as they were
    buf = torch.full((M + 1, N), 7.0, device="cuda")
    out = fn(plan, *ops, out=buf[:M])
    out16 = fn(plan, *ops, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    rel = float((out.double() - ref).norm() / ref.norm())
    print(f"relative error {rel:.3g}", flush=True)
    # fp32 accumulation: int8 tile sums are exact and MXFP4 products too; each of
    # the K / tile (K / 64) additions rounds by 2^-24 of a running sum that the
    # result's size bounds on average.  The E4M3 matrix cores align the products
    # of a step before they add them, to about 2^-16 of the largest: 1.5e-5 measured
    # at every size here (9.5e-6 in the longer factor tiles), half the bound.
    assert rel < {"int8": 1e-6, "fp8": 2.0 ** -15, "mxfp4": 2e-6}[cast]
    assert torch.equal(out16, out.to(torch.bfloat16))
    assert torch.all(buf[M] == 7.0)
