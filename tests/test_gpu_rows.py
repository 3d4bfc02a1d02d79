"""Projections of 3 to 32 decode-style rows (residual update, next norm's input, RoPE and append in their epilogues): row counts
around the groups of 8 rows, K ranges that four waves share unevenly, one work-group per CU and two, both cache types."""
import numpy as np
import pytest
import torch

from oracle import pop_oracle as O
from paper_2602_03295_amd import synth
from tests.gpu_util import DeviceRun, TOL, rel_err



def model(**kw):
    cfg = synth.get_config("tiny", dtype=synth.DTYPE_BF16, n_layers=2, **{"vocab": 512, **kw})
    # q, k and v of magnitude one (scores too), and blocks that weigh as much as the residual they are added to; norm scales of one
    # would hide a wrong scale, or a wrong column of it
    W = synth.make_weights(cfg, seed=41, std=0.96 / cfg["d_model"] ** 0.5)
    synth.randomize_norms(W, cfg)
    return cfg, W


def check(rows, tol=TOL, qk_norm=False, **kw):
    """A prefill whose second layer's boundary rows run decode-style, then two decode steps, against the oracle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03295_amd import pop
    cfg, W = model(**kw)
    if qk_norm:
        synth.add_qk_norms(W, cfg)
    lens = [3 + 7 * b % 37 for b in range(rows)]
    tokens = synth.make_tokens(cfg["vocab"], sum(lens), seed=42)
    run = DeviceRun(pop, cfg, W, lens, reserve_pages=2, shuffle_seed=43, poison=float("nan"))
    logits = run.prefill(tokens, 1)
    state = [(Kc, Vc, ref) for Kc, Vc, ref in O.pop_prefill_batch(cfg, W, tokens, run.cu, 1)]
    for b in range(rows):
        assert rel_err(logits[b], state[b][2]) <= tol, ("prefill", b)
    state = [s[:2] for s in state]
    for s in range(2):
        tok = synth.make_tokens(cfg["vocab"], rows, seed=50 + s)
        got = run.decode(tok)
        for b in range(rows):
            ref, Kc, Vc = O.decode_step(cfg, W, O.embed_rows(W, tok[b:b + 1], np.float64)[0], *state[b])
            state[b] = (Kc, Vc)
            assert rel_err(got[b], ref) <= tol, (s, b)
            for l in range(2):       # the new entries, where the step stored them
                k, v = run.kv(l, b, lens[b] + s + 1)
                assert rel_err(k[-1], Kc[l][-1]) <= 2 * tol and rel_err(v[-1], Vc[l][-1]) <= 2 * tol


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [3, 7, 8, 9, 16, 17, 24, 25, 32, 33])
def test_row_counts(rows):
    check(rows, head_dim=64, n_q_heads=8, n_kv_heads=2, d_ffn=256)


# d_model (K of QKV, gate|up), Dq (K of O) and d_ffn (K of down) in K-steps of 64: 4 (one per wave), 5, 7, 37; a width whose
# QKV projection has more than 256 work-groups
@pytest.mark.gpu
@pytest.mark.parametrize("d_model,hd,hq,hkv,d_ffn", [(256, 64, 5, 1, 320), (320, 64, 4, 4, 448), (512, 128, 3, 1, 2368),
                                                     (448, 256, 2, 1, 256), (256, 128, 32, 4, 256)])
@pytest.mark.parametrize("rows", [3, 12, 20, 30])
def test_shapes(rows, d_model, hd, hq, hkv, d_ffn):
    check(rows, d_model=d_model, head_dim=hd, n_q_heads=hq, n_kv_heads=hkv, d_ffn=d_ffn)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [4, 19])
@pytest.mark.parametrize("kv_dtype,qk_norm", [(1, False), (0, True), (1, True)])
def test_cache_types_and_key_norms(rows, kv_dtype, qk_norm):
    # code flips of the 8-bit cache put one code step (6 to 12 % of an element) on a few entries
    check(rows, tol=8e-2 if kv_dtype else TOL, head_dim=128, n_q_heads=4, n_kv_heads=2, d_ffn=256, kv_dtype=kv_dtype,
          k_scale=0.02, v_scale=0.02, qk_norm=qk_norm)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d_ffn", [(24, 14336), (25, 14336), (24, 14400)])
def test_longest_k_of_the_down_projection_with_its_epilogue(rows, d_ffn):
    """Both sides of where a split GEMM takes over."""
    check(rows, head_dim=64, n_q_heads=4, n_kv_heads=2, d_ffn=d_ffn)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [16, 17, 32])
def test_long_k_of_the_down_projection(rows):
    """K above 8192: beyond 24 rows down is a split GEMM between projections of this path."""
    check(rows, head_dim=64, n_q_heads=4, n_kv_heads=2, d_ffn=8256)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [3, 12, 20])
@pytest.mark.parametrize("hd", [64, 128])
def test_sliding_window_layers_with_their_own_rope_base(rows, hd):
    check(rows, head_dim=hd, n_q_heads=4, n_kv_heads=2, d_ffn=256, sliding_window=9, global_every=2, rope_theta_local=50.0)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [16, 20, 30])
def test_key_norms_over_a_wide_qkv_projection(rows):
    """fp32 rows of more than 4096 columns, for the separate rotate-and-append kernel: 32 columns per work-group from 17 rows on."""
    check(rows, head_dim=128, n_q_heads=32, n_kv_heads=4, d_ffn=256, qk_norm=True)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [3, 32])
@pytest.mark.parametrize("vocab,cols", [(16384, 64), (16420, 128), (20548, 128)])
def test_lm_head_tiles(rows, vocab, cols):
    from paper_2602_03295_amd import pop
    assert pop.pop_op_gemm_row_scaled_tile_cols(rows, vocab, 256, 3) == cols
    check(rows, head_dim=64, n_q_heads=4, n_kv_heads=2, d_ffn=256, vocab=vocab)


# gate|up and LM head with 64 to 128 weight rows per work-group: 4 to 8 blocks of 16, whole and ragged last work-groups, K-steps of
# four waves even (256) and uneven (448), both activations; one width below and one above go through the tiled GEMM.  One and two
# rows are normalised inside this kernel.
@pytest.mark.gpu
@pytest.mark.parametrize("rows", [1, 2, 3, 9, 17, 32])
@pytest.mark.parametrize("d_model,d_ffn,vocab,act", [(256, 6144, 12288, 0), (256, 6208, 12292, 1), (448, 8256, 20480, 0),
                                                     (256, 12288, 24580, 1), (448, 14336, 28676, 0), (256, 16384, 32772, 0)])
def test_wide_projections(rows, d_model, d_ffn, vocab, act):
    check(rows, d_model=d_model, head_dim=64, n_q_heads=4, n_kv_heads=2, d_ffn=d_ffn, vocab=vocab, act=act)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d_model", [(5, 4160), (20, 4160), (32, 8192)])
def test_more_than_256_sums_of_squares_per_row(rows, d_model):
    check(rows, d_model=d_model, head_dim=64, n_q_heads=4, n_kv_heads=2, d_ffn=256)


def _swap(W, l):
    lw = W["layers"][l]
    lw["norm_in"], lw["norm_post"] = lw["norm_post"], lw["norm_in"]


MISTAKES = {
    "input and post-attention scale swapped": lambda W: _swap(W, 0),
    "own input scale in the next layer": lambda W: W["layers"][1].update(norm_in=W["layers"][0]["norm_in"]),
    "input scale of the wrong columns": lambda W: W["layers"][1].update(norm_in=W["layers"][1]["norm_in"].roll(16)),
    "post-attention scale of the wrong columns": lambda W: W["layers"][1].update(norm_post=W["layers"][1]["norm_post"].roll(16)),
    "final scale of the wrong columns": lambda W: W.update(final_norm=W["final_norm"].roll(16)),
    "final scale left out": lambda W: W.update(final_norm=torch.ones_like(W["final_norm"])),
}


@pytest.mark.parametrize("name", MISTAKES)
def test_a_wrong_norm_scale_is_beyond_the_tolerance(name):
    """The inputs of the tests above tell such mistakes apart: planted in the oracle, each moves a decode step by more."""
    kw = dict(head_dim=64, n_q_heads=8, n_kv_heads=2, d_ffn=256)
    cfg, W = model(**kw)
    tokens = synth.make_tokens(cfg["vocab"], 21, seed=42)
    Kc, Vc, _ = O.pop_prefill(cfg, W, tokens, 1)
    x = O.embed_rows(W, tokens[:1], np.float64)[0]
    ref, Kr, Vr = O.decode_step(cfg, W, x, Kc, Vc)
    _, wrong = model(**kw)
    MISTAKES[name](wrong)
    got, Kg, Vg = O.decode_step(cfg, wrong, x, Kc, Vc)
    assert max(rel_err(got, ref), *(rel_err(g[-1], r[-1]) for g, r in zip(Kg + Vg, Kr + Vr))) > 2 * TOL
