"""Projections whose K range is split and whose partial products the RoPE + append kernel adds: kept layers (q, k, v) and
a single pruned layer (k, v), against the CPU oracle."""
import pytest
import torch

from paper_2602_03295_amd import synth
from tests.gpu_util import DeviceRun, compare_with_oracle

pytestmark = pytest.mark.gpu

# (few rows and a long K range: 64-row tiles of a 1024- to 1536-wide result leave most of the chip idle, so the parts are
# taken; 65 and 130 rows cross a 64-row tile of the append kernel)
CASES = [
    dict(n_q_heads=8, n_kv_heads=4, head_dim=64, lens=[5], l_keep=2),
    dict(n_q_heads=8, n_kv_heads=2, head_dim=128, lens=[65], l_keep=3, qk_norms=True),
    dict(n_q_heads=4, n_kv_heads=1, head_dim=256, lens=[3, 64, 63], l_keep=1),
    dict(n_q_heads=8, n_kv_heads=4, head_dim=64, lens=[130, 1], l_keep=3),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"hd{c['head_dim']}-{sum(c['lens'])}-{c['l_keep']}")
def test_parts_added_by_the_append_kernel(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03295_amd import pop
    case = dict(case)
    lens, l_keep, qk_norms = case.pop("lens"), case.pop("l_keep"), case.pop("qk_norms", False)
    cfg = synth.get_config("tiny", dtype=synth.DTYPE_BF16)
    cfg.update(n_layers=4, d_model=2048, d_ffn=512, vocab=256, **case)
    W = synth.make_weights(cfg, seed=11)
    synth.randomize_norms(W, cfg)
    if qk_norms:
        synth.add_qk_norms(W, cfg)
    tokens = synth.make_tokens(cfg["vocab"], sum(lens), seed=12)
    run = DeviceRun(pop, cfg, W, lens, reserve_pages=2, poison=float("nan"))
    logits = run.prefill(tokens, l_keep)
    compare_with_oracle(run, W, tokens, l_keep, logits)
