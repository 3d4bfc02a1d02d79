"""Every tile shape of the bf16 GEMM and the split of K, at ragged sizes that the tile choice gives to each shape
(tests/test_gemm_plan.py holds the choice to what the list says), against the same contraction in fp64."""
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


# M, N, K and what pop_op_gemm takes for them: the tile and, where the columns go to two launches, the second one's
SIZES = [
    (641, 16388, 64, (256, 256), None),           # a single K-step
    (3000, 12292, 192, (256, 256), (160, 128)),   # the last round in a second launch
    (2047, 6140, 448, (256, 192), None),
    (1281, 8196, 64, (192, 256), None),           # a single K-step
    (1281, 8196, 128, (192, 256), None),
    (257, 28668, 64, (160, 256), None),           # a single K-step
    (700, 12292, 448, (160, 256), None),
    (2047, 4100, 64, (192, 192), None),           # a single K-step
    (2049, 4100, 192, (192, 192), None),
    (385, 12292, 192, (256, 128), None),
    (529, 12292, 448, (128, 256), None),
    (161, 20484, 64, (192, 128), None),           # a single K-step
    (529, 8196, 192, (192, 128), None),
    (1000, 6140, 448, (128, 192), None),
    (257, 20484, 192, (96, 256), None),
    (97, 20484, 64, (160, 128), None),            # a single K-step
    (1281, 3080, 192, (160, 128), None),
    (193, 12292, 448, (128, 128), None),
    (65, 20484, 64, (96, 128), None),             # a single K-step
    (257, 8196, 448, (96, 128), None),
    (193, 3080, 64, (64, 128), None),             # a single K-step
    (65, 8196, 448, (96, 64), None),
    (65, 9000, 448, (96, 64), None),
    (385, 1000, 448, (64, 64), None),
    (2047, 28668, 2048, (256, 256), (256, 128)),  # three rounds, the rest in a second launch
    (8, 14336, 4096, (64, 64), None),     # few rows: the column tiles start at different K offsets
    (250, 9000, 4096, (96, 128), None),   # the same, several row tiles
    (129, 1000, 2112, (64, 64), None),    # rows that are not a multiple of 4 KB apart: all start at offset 0
    # K that is no multiple of a K-step
    (385, 16388, 72, (256, 256), None),
    (2047, 6140, 1000, (256, 192), None),
    (529, 16388, 456, (192, 256), None),
    (257, 28668, 72, (160, 256), None),
    (1281, 6140, 72, (192, 192), None),
    (193, 20484, 72, (256, 128), None),
    (300, 20484, 72, (128, 256), None),
    (161, 20484, 72, (192, 128), None),
    (193, 20484, 456, (128, 192), None),
    (257, 20484, 72, (96, 256), None),
    (97, 20484, 72, (160, 128), None),
    (97, 16388, 200, (128, 128), None),
    (65, 20484, 72, (96, 128), None),
    (65, 1000, 72, (64, 128), None),
    (65, 9000, 200, (96, 64), None),
    (65, 1000, 200, (64, 64), None),
    (1000, 12292, 1000, None, None),      # (gate|up: 256 x 192)
    (1281, 8196, 456, None, None),        # (gate|up: 192 x 256)
    (97, 20484, 200, None, None),         # (gate|up: 128 x 128)
    (2047, 28668, 2040, (256, 256), "any"),       # a second launch for the last round
]


@pytest.mark.parametrize("M,N,K,tile,tail", SIZES)
def test_tile_shapes(pop, M, N, K, tile, tail):
    A, W = draw(M, N, K, M + N + K)
    ref = A.double() @ W.double().t()
    # fp32 sums of K products: sqrt(K) 2^-24 of a row's scale, far inside 1e-5 of the largest value
    assert rel(pop.pop_op_gemm(A, W, epilogue=pop.EPI_STORE_F32), ref) <= 1e-5
    old = torch.linspace(-3.0, 5.0, M * N, device="cuda").view(M, N)
    assert rel(pop.pop_op_gemm(A, W, epilogue=pop.EPI_ADD_F32, out=old.clone()), ref + old.double()) <= 1e-5
    # one rounding to bf16, half a step of 2^-8
    assert rel(pop.pop_op_gemm(A, W, epilogue=pop.EPI_STORE_BF16), ref) <= 2.0 ** -8
    half = N // 2 // 4 * 4
    glu = pop.pop_op_gemm(A, W[:2 * half], epilogue=pop.EPI_GLU_BF16, act=0)
    # one rounding to bf16 (2^-9) of a product whose factors carry fp32 sums and a fast exp2
    assert rel(glu, torch.nn.functional.silu(ref[:, :half]) * ref[:, half:2 * half]) <= 2.0 ** -7


# (with room for them, all take parts of K: tests/test_gemm_plan.py)
SPLIT_SIZES = [(5, 6144, 4096), (31, 4096, 4096), (100, 4096, 14336), (250, 6140, 4096), (529, 4096, 14336),
               (700, 4100, 12288), (1030, 4096, 14336), (77, 2048, 3840)]


@pytest.mark.parametrize("M,N,K", SPLIT_SIZES)
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
