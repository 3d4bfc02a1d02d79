"""Every tile shape of the bf16 GEMM and the split of K, at ragged sizes that the tile choice gives to each shape
(its comment names the shape), against the same contraction in fp64."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pop():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03295_amd import pop as p
    return p


def draw(M, N, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.empty(M, K, device="cuda").normal_(generator=g).to(torch.bfloat16)
    W = torch.empty(N, K, device="cuda").normal_(generator=g).to(torch.bfloat16)
    return A, W


def rel(got, ref):
    return float((got.double() - ref).abs().max() / ref.abs().max())


SIZES = [
    (1281, 8196, 64),     # 256 x 256, a single K-step
    (3000, 12292, 192),   # 256 x 256, the last round as 160 x 128 in a second launch
    (2047, 6140, 448),    # 256 x 192
    (1281, 8196, 128),    # 192 x 256
    (257, 28668, 64),     # 160 x 256, a single K-step
    (700, 12292, 448),    # 160 x 256
    (2047, 4100, 64),     # 192 x 192, a single K-step
    (2049, 4100, 192),    # 192 x 192
    (385, 12292, 192),    # 256 x 128
    (529, 12292, 448),    # 128 x 256
    (161, 20484, 64),     # 192 x 128, a single K-step
    (529, 8196, 192),     # 192 x 128
    (1000, 6140, 448),    # 128 x 192
    (257, 20484, 192),    # 96 x 256
    (97, 20484, 64),      # 160 x 128, a single K-step
    (1281, 3080, 192),    # 160 x 128
    (193, 12292, 448),    # 128 x 128
    (65, 20484, 64),      # 96 x 128, a single K-step
    (257, 8196, 448),     # 96 x 128
    (193, 3080, 64),      # 64 x 128, a single K-step
    (65, 8196, 448),      # 96 x 64
    (385, 1000, 448),     # 64 x 64
    (2047, 28668, 2048),  # 256 x 256, three rounds, the rest as 256 x 128 in a second launch
    (8, 14336, 4096),     # few rows: the column tiles start at different K offsets
    (250, 9000, 4096),    # the same, several row tiles
    (129, 1000, 2112),    # rows that are not a multiple of 4 KB apart: all start at offset 0
]


@pytest.mark.parametrize("M,N,K", SIZES)
def test_tile_shapes(pop, M, N, K):
    A, W = draw(M, N, K, M + N + K)
    got = pop.pop_op_gemm(A, W, epilogue=pop.EPI_STORE_F32)
    ref = A.double() @ W.double().t()
    # fp32 sums of K products: sqrt(K) 2^-24 of a row's scale, far inside 1e-5 of the largest value
    assert rel(got, ref) <= 1e-5
    half = N // 2 // 4 * 4
    glu = pop.pop_op_gemm(A, W[:2 * half], epilogue=pop.EPI_GLU_BF16, act=0)
    # one rounding to bf16 (2^-9) of a product whose factors carry fp32 sums and a fast exp2
    assert rel(glu, torch.nn.functional.silu(ref[:, :half]) * ref[:, half:2 * half]) <= 2.0 ** -7


@pytest.mark.parametrize("M,N,K", [(5, 6144, 4096), (31, 4096, 4096), (100, 4096, 14336), (250, 6140, 4096),
                                   (529, 4096, 14336), (700, 4100, 12288), (1030, 4096, 14336), (77, 2048, 3840)])
@pytest.mark.parametrize("epi", [0, 1, 3])
def test_split_k(pop, M, N, K, epi):
    A, W = draw(M, N, K, M + N + K + epi)
    ref = A.double() @ W.double().t()
    out = None
    if epi == pop.EPI_ADD_F32:
        out = torch.ones(M, N, device="cuda")
        ref = ref + 1
    scratch = torch.full((32 * M * N,), 0xff, dtype=torch.uint8, device="cuda")   # NaN unless written
    got = pop.pop_op_gemm_splitk(A, W, epilogue=epi, out=out, scratch=scratch)
    assert rel(got, ref) <= (2.0 ** -8 if epi == pop.EPI_STORE_BF16 else 1e-5)
