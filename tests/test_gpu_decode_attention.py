"""Decode attention over the paged cache at the edges of its key blocks and splits: every bound of query heads per KV
head, every head size, one and two rows (RoPE and append inside the kernel) and more, both cache types, a sliding window."""
import numpy as np
import pytest
import torch

from oracle import pop_oracle as O
from paper_2602_03295_amd import synth
from tests.gpu_util import DeviceRun, TOL, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pop():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03295_amd import pop as p
    return p


def check(pop, lens, steps, tol=TOL, l_keep=1, d_ffn=256, **kw):
    cfg = synth.get_config("tiny", dtype=synth.DTYPE_BF16, n_layers=2, d_ffn=d_ffn, vocab=512, **kw)
    W = synth.make_weights(cfg, seed=21)
    synth.add_qk_norms(W, cfg)
    tokens = synth.make_tokens(cfg["vocab"], sum(lens), seed=22)
    run = DeviceRun(pop, cfg, W, lens, reserve_pages=2, shuffle_seed=23, poison=float("nan"))
    logits = run.prefill(tokens, l_keep)
    outs = O.pop_prefill_batch(cfg, W, tokens, run.cu, l_keep)
    state = []
    for b, (Kc, Vc, ref) in enumerate(outs):
        assert rel_err(logits[b], ref) <= tol, ("prefill", b, lens[b])
        state.append((Kc, Vc))
    for s in range(steps):
        tok = synth.make_tokens(cfg["vocab"], len(lens), seed=30 + s)
        got = run.decode(tok)
        for b in range(len(lens)):
            ref, Kc, Vc = O.decode_step(cfg, W, O.embed_rows(W, tok[b:b + 1], np.float64)[0], *state[b])
            state[b] = (Kc, Vc)
            assert rel_err(got[b], ref) <= tol, (s, b, lens[b])
            for l in range(cfg["n_layers"]):       # the new entries, where the step stored them
                k, v = run.kv(l, b, lens[b] + s + 1)
                assert rel_err(k[-1], Kc[l][-1]) <= 2 * tol and rel_err(v[-1], Vc[l][-1]) <= 2 * tol


EDGES = [1, 15, 16, 17, 31, 63, 64, 65, 129]


@pytest.mark.parametrize("hd,hq,hkv", [(64, 2, 2), (64, 6, 3), (128, 3, 1), (128, 8, 1), (256, 4, 2), (256, 5, 1)])
@pytest.mark.parametrize("rows", [1, 2, 3, 9])
def test_edges(pop, hd, hq, hkv, rows):
    for i in range(0, 9, rows):
        check(pop, EDGES[i:i + rows], 2, head_dim=hd, n_q_heads=hq, n_kv_heads=hkv)


@pytest.mark.parametrize("rows", [1, 2, 3, 9])
@pytest.mark.parametrize("hd", [64, 128, 256])
def test_window_and_page_sizes(pop, rows, hd):
    lens = [40, 129, 65, 16, 33, 100, 250, 7, 64]
    for P in (1, 8, 64):
        for i in range(0, 9 if rows < 3 else 1, rows):
            check(pop, lens[i:i + rows], 2, head_dim=hd, n_q_heads=4, n_kv_heads=2, sliding_window=33, global_every=2,
                  page_size=P)


@pytest.mark.parametrize("rows", [1, 2, 3, 9])
@pytest.mark.parametrize("hd", [64, 128, 256])
def test_8_bit_cache(pop, rows, hd):
    # code flips put one code step (6 to 12 % of an element) on a few entries: the bound of the 8-bit cache's own tests
    for i in range(0, 9 if rows < 3 else 1, rows):
        check(pop, EDGES[i:i + rows], 2, tol=8e-2, head_dim=hd, n_q_heads=4, n_kv_heads=2, kv_dtype=1, k_scale=0.02,
              v_scale=0.02)


# lengths whose last block of 32 keys holds 31, 32, 1, 15, 16, 17, 18 of them
LAST_BLOCKS = [31, 32, 33, 47, 48, 49, 50]


@pytest.mark.parametrize("kv_dtype", [0, 1])
@pytest.mark.parametrize("hd,hq,hkv", [(64, 16, 8), (128, 8, 8), (64, 32, 4)])
def test_splits_of_256_keys_and_more(pop, hd, hq, hkv, kv_dtype):
    """Six sequences x 8 KV heads (13 x 4) of about 3300 keys: at most 16 (14) splits of 256 keys, which an 8-bit cache
    takes in blocks of two key groups and a bf16 cache in blocks of one; the last block of a sequence partly filled."""
    n = 6 if hkv == 8 else 13
    check(pop, [3264 + LAST_BLOCKS[i % 7] for i in range(n)], 1, l_keep=0, tol=8e-2 if kv_dtype else TOL, head_dim=hd,
          n_q_heads=hq, n_kv_heads=hkv, kv_dtype=kv_dtype, k_scale=0.02, v_scale=0.02)


@pytest.mark.parametrize("hd,hq", [(64, 32), (64, 64), (128, 32)])
@pytest.mark.parametrize("lens", [[4672 + 31], [4672 + 33], [2336 + 15, 2336 + 17], [2336 + 16, 2336]])
def test_splits_of_256_keys_with_rope_and_append_inside(pop, hd, hq, lens):
    """One and two sequences of an 8-bit cache with 32 KV heads: at most 24 and 12 splits, so of 256 keys here."""
    check(pop, lens, 2, l_keep=0, tol=8e-2, head_dim=hd, n_q_heads=hq, n_kv_heads=32, kv_dtype=1, k_scale=0.02, v_scale=0.02)


def test_one_split_for_many_sequences(pop):
    """More (sequence, KV head) pairs than half the work-groups that run at once: one split, whatever the length."""
    check(pop, [EDGES[i % 9] + 40 * (i % 3) for i in range(49)], 1, head_dim=64, n_q_heads=8, n_kv_heads=8)


@pytest.mark.parametrize("rows", [3, 4, 5])
def test_few_rows_of_a_width_that_is_no_multiple_of_64(pop, rows):
    """Projections of three and four rows by the GEMV kernel's 4-row form (QKV, O, gate|up and down, all of 2048 rows or
    more), of five by the tiled GEMM."""
    check(pop, [33, 20, 65, 7, 16][:rows], 2, d_model=2056, d_ffn=2072, head_dim=64, n_q_heads=24, n_kv_heads=4)
