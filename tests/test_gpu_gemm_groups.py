"""The 32 x 32 tile of the plain-matrix products with register groups of one and of two
chunks (chosen by the number of workgroups and the contraction): the same bits.  The same
product is taken one to five times in a batch, which crosses the lines between them."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api

N = 512   # 256 workgroups a product


# a wave's quarter of K: one chunk, less, a group of two, one over, several and a remainder
@pytest.mark.parametrize("K", [64, 100, 256, 384, 500, 1056, 2100])
@pytest.mark.parametrize("kinds", ["row row", "row col", "col col", "row1 col1"])
@pytest.mark.parametrize("prec", [0, 1])
def test_groups_of_one_and_two_chunks(prec, kinds, K):
    print(f"register groups prec={prec} {kinds} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)

    def operand(kind):
        odd = kind.endswith("1")
        if kind.startswith("row"):
            return torch.randn((N, (K + 3) // 4 * 4 + odd), generator=gen, device="cuda")[:, :K]
        return torch.randn((K, N + odd), generator=gen, device="cuda").t()[:N]

    A, B = (operand(k) for k in kinds.split())
    one = api.gemm(prec, A, B)[0]
    for z in (2, 3, 4, 5):
        C = api.gemm(prec, A.expand(z, -1, -1), B.expand(z, -1, -1))
        for i in range(z):
            assert torch.equal(C[i], one), (z, i)
    ref = A.double() @ B.double().t().contiguous()
    # rounding of the operands (bfloat16: 2^-8 together with the second order), then K products summed in FP32
    unit = (2.0 ** -7 if prec else 0.0) + (K + 8) * 2.0 ** -24
    assert ((one.double() - ref).abs() <= unit * (A.double().abs() @ B.double().abs().t().contiguous())).all()
