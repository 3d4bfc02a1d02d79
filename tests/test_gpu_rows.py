"""Projections of 3 to 32 decode-style rows (residual update, next norm's input, RoPE and append in their epilogues): row counts
around the groups of 8 rows, K ranges that four waves share unevenly, one work-group per CU and two, both cache types."""
import numpy as np
import pytest
import torch

from oracle import pop_oracle as O
from paper_2602_03295_amd import synth
from tests.gpu_util import DeviceRun, TOL, rel_err

pytestmark = pytest.mark.gpu


def check(rows, tol=TOL, qk_norm=False, **kw):
    """A prefill whose second layer's boundary rows run decode-style, then two decode steps, against the oracle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03295_amd import pop
    cfg = synth.get_config("tiny", dtype=synth.DTYPE_BF16, n_layers=2, vocab=512, **kw)
    W = synth.make_weights(cfg, seed=41)
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


@pytest.mark.parametrize("rows", [3, 7, 8, 9, 16, 17, 24, 25, 32, 33])
def test_row_counts(rows):
    check(rows, head_dim=64, n_q_heads=8, n_kv_heads=2, d_ffn=256)


# d_model (K of QKV, gate|up), Dq (K of O) and d_ffn (K of down) in K-steps of 64: 4 (one per wave), 5, 7, 37; a width whose
# QKV projection has more than 256 work-groups
@pytest.mark.parametrize("d_model,hd,hq,hkv,d_ffn", [(256, 64, 5, 1, 320), (320, 64, 4, 4, 448), (512, 128, 3, 1, 2368),
                                                     (448, 256, 2, 1, 256), (256, 128, 32, 4, 256)])
@pytest.mark.parametrize("rows", [3, 12, 20, 30])
def test_shapes(rows, d_model, hd, hq, hkv, d_ffn):
    check(rows, d_model=d_model, head_dim=hd, n_q_heads=hq, n_kv_heads=hkv, d_ffn=d_ffn)


@pytest.mark.parametrize("rows", [4, 19])
@pytest.mark.parametrize("kv_dtype,qk_norm", [(1, False), (0, True), (1, True)])
def test_cache_types_and_key_norms(rows, kv_dtype, qk_norm):
    # code flips of the 8-bit cache put one code step (6 to 12 % of an element) on a few entries
    check(rows, tol=8e-2 if kv_dtype else TOL, head_dim=128, n_q_heads=4, n_kv_heads=2, d_ffn=256, kv_dtype=kv_dtype,
          k_scale=0.02, v_scale=0.02, qk_norm=qk_norm)
