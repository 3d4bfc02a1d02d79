"""Prefill attention, head sizes 64 and 128: the forms of the kernel (256 query rows that share their key tiles, 128 rows with
the key tiles dealt to two groups of waves, sequences of one key tile by themselves or among longer ones), at the edges of
waves, tiles and windows."""
import numpy as np
import pytest
import torch

from oracle import pop_oracle as O

# The form is chosen by the estimated time of each: many short sequences (few key tiles each) take the 256-row form, a single
# one whose tiles do not fill the chip the 128-row form, sequences of up to 64 tokens alone a form of their own.
FORMS = [([1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300], 32, 4, 256), ([700], 24, 2, 128), ([257], 4, 4, 128),
         ([65, 640, 130], 6, 1, 128), ([513], 3, 1, 128), ([50, 400, 64], 4, 2, 128), ([1, 2, 31, 32, 33, 63, 64], 6, 2, 64),
         ([64], 1, 1, 64), ([17], 8, 1, 64)]


@pytest.mark.parametrize("lens,hq,hkv,rows", FORMS)
@pytest.mark.parametrize("hd", [64, 128, 256])
def test_forms_are_what_the_cases_name(lens, hq, hkv, rows, hd):
    pop = pytest.importorskip("paper_2602_03295_amd.pop", reason="libpop.so not built")
    cu = np.concatenate([[0], np.cumsum(lens)])
    assert pop.pop_op_rope_attention_tile_rows(cu, hq, hd) == (rows if hd <= 128 else 128)


@pytest.mark.parametrize("n,length,rows", [(32, 16, 64), (64, 64, 64), (1, 64, 64), (64, 65, 128), (1, 65, 256), (32, 300, 256)])
def test_short_sequences_have_a_form_of_their_own(n, length, rows):
    """32 query heads of 128.  Two waves a sequence: with eight, 32 sequences of 64 tokens took 67 us, with four 63, with two 52."""
    pop = pytest.importorskip("paper_2602_03295_amd.pop", reason="libpop.so not built")
    assert pop.pop_op_rope_attention_tile_rows(np.arange(n + 1) * length, 32, 128) == rows
    assert pop.pop_op_rope_attention_tile_rows([0, 5, 5], 32, 128) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("lens,hq,hkv", [f[:3] for f in FORMS])
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("window", [0, 1, 64, 97, 200])
def test_forms(lens, hq, hkv, hd, window):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03295_amd import pop
    cu = np.concatenate([[0], np.cumsum(lens)])
    rng = np.random.default_rng(hd + window + len(lens))
    qkv = torch.from_numpy(rng.standard_normal((int(cu[-1]), (hq + 2 * hkv) * hd)).astype(np.float32)).to(torch.bfloat16)
    got = pop.pop_op_rope_attention(qkv.cuda(), cu, hq, hkv, hd, 10000.0, window).double().cpu().numpy()
    heads = [0, hq - 1]      # first and last query head (every head is a work-group of its own)
    for b, n in enumerate(lens):
        x = qkv[cu[b]:cu[b + 1]].double().numpy().reshape(n, hq + 2 * hkv, hd)
        kv = [h // (hq // hkv) for h in heads]
        q, k = O.rope(x[:, heads], np.arange(n), 10000.0), O.rope(x[:, [hq + i for i in kv]], np.arange(n), 10000.0)
        ref = O.attention_rows(q, np.arange(n), k, x[:, [hq + hkv + i for i in kv]], window).reshape(n, 2, hd)
        out = got[cu[b]:cu[b + 1]].reshape(n, hq, hd)[:, heads]
        # q, k and P are fp16 (2^-11 each; scores of these inputs are below 8 in magnitude), the result is bf16 (2^-9)
        assert np.abs(out - ref).max() / np.abs(ref).max() <= 2.0 ** -7
