"""Which tile shapes, K parts and launches the bf16 GEMM takes for a problem, as the library reports it.  No GPU needed."""
import csv
import os

import pytest

from tests.test_gpu_gemm_tiles import SIZES, SPLIT_SIZES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pop = pytest.importorskip("paper_2602_03295_amd.pop", reason="libpop.so not built")


@pytest.mark.parametrize("M,N,K,epi", [(2048, 14344, 4104, 2), (4096, 14344, 4104, 2), (1536, 6144, 4104, 3),
                                       (768, 5632, 1000, 2), (2048, 4104, 4104, 1)])
def test_partly_filled_rounds_with_any_k(M, N, K, epi):
    """256 x 256 tiles would leave most of a round of work-groups idle here: with a K that is no multiple of a K-step, too,
    smaller tiles or a second launch take their place."""
    p = pop.pop_op_gemm_plan(M, N, K, epi)
    assert p["tile"] != (256, 256) or p["tail"] is not None


def test_shapes_for_any_k():
    """All sixteen shapes are built for such K: nothing sends it to a few of them."""
    masked, full = set(), set()
    for M in range(16, 4200, 88):
        for N, K in ((4096, 14336), (6144, 4096), (28672, 4096), (2048, 1024), (12288, 448)):
            full.add(pop.pop_op_gemm_plan(M, N, K, 3)["tile"])
            masked.add(pop.pop_op_gemm_plan(M, N, K - 8, 3)["tile"])
    assert len(full) >= 12 and len(masked) >= 12, (sorted(full), sorted(masked))


def test_plan_arguments():
    for bad in [dict(M=0, N=8, K=8), dict(M=8, N=0, K=8), dict(M=8, N=8, K=0), dict(M=8, N=8, K=12),
                dict(M=8, N=8, K=8, epilogue=4)]:
        with pytest.raises(pop.PopError):
            pop.pop_op_gemm_plan(**bad)
    p = pop.pop_op_gemm_plan(8, 64, 64)
    assert p["k_parts"] == 1 and p["head_cols"] == 64 and p["tail"] is None
    # scratch for the parts is what a split needs
    assert pop.pop_op_gemm_plan(16, 4096, 14336, 3)["k_parts"] == 1
    assert pop.pop_op_gemm_plan(16, 4096, 14336, 3, scratch_bytes=32 * 16 * 4096)["k_parts"] > 1


@pytest.mark.parametrize("M,N,K", [(12000, 3840, 15360), (14000, 4096, 14336)])
def test_long_k_and_many_rows_take_the_largest_tiles(M, N, K):
    """Rows of A that are too long to stay cached between column tiles: smaller tiles fill the rounds better here but
    fetch the rows more often."""
    assert pop.pop_op_gemm_plan(M, N, K, 1)["tile"] == (256, 256)


@pytest.mark.parametrize("M,N,K,tile,tail", SIZES)
def test_sizes_of_the_tile_tests_take_the_shapes_they_name(M, N, K, tile, tail):
    p = pop.pop_op_gemm_plan(M, N, K, 3)
    if tile is not None:
        assert p["tile"] == tile
    if tail == "any":
        assert p["tail"] is not None
    elif tile is not None:
        assert p["tail"] == tail


def test_sizes_of_the_tile_tests_cover_every_shape():
    """Plain and gate|up projections, K a multiple of a K-step and not: all sixteen shapes each."""
    for epi in (3, 2):
        for masked in (False, True):
            seen = set()
            for M, N, K, _, _ in SIZES:
                if (K % 64 != 0) == masked:
                    p = pop.pop_op_gemm_plan(M, N // 2 // 4 * 4 if epi == 2 else N, K, epi)
                    seen |= {p["tile"], p["tail"]} - {None}
            assert len(seen) == 16, (epi, masked, sorted(seen))


def test_sizes_of_the_split_tests_are_split():
    parts = [pop.pop_op_gemm_plan(M, N, K, 3, scratch_bytes=32 * M * N)["k_parts"] for M, N, K in SPLIT_SIZES]
    assert min(parts) >= 2 and {2, 4, 8} <= set(parts), parts


def test_choice_against_the_measured_times():
    """profiles/gemm_tile_timings.csv: every shape's time for 488 problems (MI355X).  Where the library takes one launch and
    no split, its choice is the fastest shape or near it."""
    best, times = {}, {}
    with open(os.path.join(ROOT, "profiles", "gemm_tile_timings.csv")) as f:
        for row in csv.DictReader(f):
            if row["k_parts"] != "1":
                continue
            problem = tuple(int(row[c]) for c in ("M", "N", "K", "epilogue"))
            for name, t in row.items():
                if "x" in name and t:
                    times[problem + tuple(map(int, name.split("x")))] = float(t)
                    best[problem] = min(best.get(problem, 1e30), float(t))
    lost = []
    for problem, t in best.items():
        p = pop.pop_op_gemm_plan(*problem)
        if p["tail"] is None and problem + p["tile"] in times:
            lost.append(times[problem + p["tile"]] / t - 1)
    assert len(lost) >= 400
    assert sum(lost) / len(lost) <= 0.01 and max(lost) <= 0.12


@pytest.mark.parametrize("M", [3, 8, 32])
@pytest.mark.parametrize("N,K,epi,cols", [(8192, 4096, 2, 64), (8448, 4096, 2, 128), (9216, 4096, 2, 128), (10240, 4096, 2, 128),
                                          (14336, 4096, 2, 128), (9728, 2560, 2, 128), (8960, 1536, 2, 128), (5632, 4096, 2, 64),
                                          (16032, 4096, 3, 64), (16384, 4096, 3, 64), (16864, 4096, 3, 128), (28672, 4096, 3, 128)])
def test_row_scaled_tiles_do_not_start_a_second_round(M, N, K, epi, cols):
    """Gate|up and LM head of 3 to 32 rows: 64-column tiles are one work-group per CU, and from 16385 columns on a second round
    of them is slower than 128-column tiles (gate|up of 2 x 8448 rows of 4096, 32 rows: a step of four layers 504 and 473 us)."""
    assert pop.pop_op_gemm_row_scaled_tile_cols(M, N, K, epi) == cols


def test_row_scaled_tile_arguments():
    for bad in [(0, 8, 8, 2), (33, 8, 8, 2), (8, 0, 8, 2), (8, 8, 12, 2), (8, 8, 8, 1)]:
        assert pop.pop_op_gemm_row_scaled_tile_cols(*bad) == 0
