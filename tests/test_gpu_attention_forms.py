"""Prefill attention, head sizes 64 and 128: both forms of the kernel (256 query rows that share their key tiles, 128 rows with
the key tiles dealt to two groups of waves), at the edges of waves, tiles and windows."""
import numpy as np
import pytest
import torch

from oracle import pop_oracle as O

pytestmark = pytest.mark.gpu


# The form is chosen by the estimated time of each: many short sequences (few key tiles each) take the 256-row form, a single
# one whose tiles do not fill the chip the 128-row form.
@pytest.mark.parametrize("lens,hq,hkv", [([1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300], 32, 4),     # 256 rows
                                         ([700], 24, 2), ([257], 4, 4), ([65, 640, 130], 6, 1), ([513], 3, 1)])       # 128 rows
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
