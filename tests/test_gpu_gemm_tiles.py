"""The 64 x 64 tile of the plain-matrix products against the 32 x 32 tile: a product
large enough for the former equals, bit for bit, the same product taken in row blocks
small enough for the latter (the serving loop relies on a row's result not depending on
the rows that share its launch), and FP64 within FP32 accumulation."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api

# rows, columns off the tile, batch: (Z ceil(M / 64) ceil(N / 64) tiles: 672, at least the
# 448 from which both forms of operands take the 64 x 64 tile)
Z, M, N = 16, 390, 333
STEP = 130   # rows of a block: at most 16 x 3 x 6 = 288 tiles; two batches of it 36


def _rows(gen, z, r, K, kind):
    """[z, r, K] views: k-contiguous rows (16-byte aligned or not), contiguous rows at
    every k (aligned or not)."""
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
    up = lambda n, q: (n + q - 1) // q * q
    if kind == "row":
        return rnd(z, r, up(K, 4))[..., :K]
    if kind == "row1":
        return rnd(z, r, up(K, 2) + 1)[..., :K]
    ld = up(r, 4) if kind == "col4" else up(r, 2) + 1
    return rnd(z, K, ld).transpose(1, 2)[:, :r]


# around a chunk (32), a quarter's chunks, several stages, and the update's widths
@pytest.mark.parametrize("K", [1, 31, 32, 33, 64, 100, 129, 274, 512])
@pytest.mark.parametrize("kinds", ["row row", "row row1", "row1 col", "row col4", "row1 row", "col4 col4", "col col4",
                                   "col4 row"])
@pytest.mark.parametrize("prec", [0, 1])
def test_large_tile_equals_small_tile(prec, kinds, K):
    print(f"large tile prec={prec} {kinds} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K + 1000 * prec)
    ka, kb = kinds.split()
    A, B = _rows(gen, Z, M, K, ka), _rows(gen, Z, N, K, kb)
    bias = torch.randn((Z, N), generator=gen, device="cuda")
    C = api.gemm(prec, A, B, bias=bias)
    for z in range(0, Z, 2):
        for r in range(0, M, STEP):
            part = api.gemm(prec, A[z:z + 2, r:r + STEP], B[z:z + 2], bias=bias[z:z + 2])
            assert torch.equal(C[z:z + 2, r:r + STEP], part), (z, r)
    if prec == 0:
        # each output sums K products in FP32: error below K 2^-24 of the terms' magnitude
        Ad, Bd = A.double().contiguous(), B.double().transpose(1, 2).contiguous()
        ref = torch.matmul(Ad, Bd) + bias.double()[:, None]
        bound = (K + 8) * 2.0 ** -24 * (torch.matmul(Ad.abs(), Bd.abs()) + bias.double().abs()[:, None])
        assert ((C.double() - ref).abs() <= bound).all()


@pytest.mark.parametrize("K", [1, 31, 32, 33, 64, 100, 129, 274, 512])
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, True), (True, False)])
def test_large_tile_on_copies_equals_small_tile(ta, tb, K):
    print(f"large tile copies ta={ta} tb={tb} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    r8 = lambda x: (x + 7) // 8 * 8

    def operand(rows, t):
        full = torch.randn((Z, K, r8(rows)) if t else (Z, rows, r8(K)), generator=gen, device="cuda").bfloat16()
        full[..., rows if t else K:] = float("nan")   # padding that must not reach the product
        return full.transpose(1, 2)[:, :rows] if t else full[..., :K]

    m = 392   # row blocks of a transposed operand start at multiples of 8
    A, B = operand(m, ta), operand(N, tb)
    C = api.gemm_bf16(A, B)
    assert torch.isfinite(C).all()
    for z in range(0, Z, 2):
        for r in range(0, m, 136):
            part = api.gemm_bf16(A[z:z + 2, r:r + 136], B[z:z + 2])
            assert torch.equal(C[z:z + 2, r:r + 136], part), (z, r)


def test_large_tile_accumulates():
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    A, B = _rows(gen, Z, M, 96, "row"), _rows(gen, Z, N, 96, "row")
    C0 = torch.randn((Z, M, N), generator=gen, device="cuda")
    C = api.gemm(0, A, B, C=C0.clone(), accumulate=True)
    assert torch.equal(C, api.gemm(0, A, B) + C0)


@pytest.mark.parametrize("K", [1, 3, 31, 32, 33, 64, 127, 129, 274])
@pytest.mark.parametrize("kinds", ["row row1", "row1 row", "row1 row1", "row1 col", "col row1"])
@pytest.mark.parametrize("prec", [0, 1])
def test_unaligned_rows_equal_aligned_rows(prec, kinds, K):
    """k-contiguous rows at any float's address, in the 32 x 32 tile."""
    print(f"unaligned rows prec={prec} {kinds} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    z, m, n = 2, 70, 101
    ops = [_rows(gen, z, r, K, kind) for kind, r in zip(kinds.split(), (m, n))]
    want = api.gemm(prec, *(_aligned(t) for t in ops))
    assert torch.equal(api.gemm(prec, *ops), want)
    for by in (1, 2, 3):   # and a first element off its alignment
        assert torch.equal(api.gemm(prec, *(_moved(t, by) for t in ops)), want), by


def _aligned(t):
    """t with k-contiguous, 16-byte aligned rows."""
    z, r, K = t.shape
    out = torch.zeros((z, r, (K + 3) // 4 * 4), device="cuda")[..., :K]
    out.copy_(t)
    return out


def _moved(t, by):
    """t at the same strides, its storage `by` floats off its alignment."""
    size = sum((n - 1) * s for n, s in zip(t.shape, t.stride())) + 1
    out = torch.zeros(size + 4, device="cuda")[by:].as_strided(t.shape, t.stride())
    out.copy_(t)
    return out
