"""The cost model's choices where two of its terms meet."""
from dataclasses import replace

import pytest

from paper_2509_15965_amd import configs
from paper_2509_15965_amd.inputs import make_weights
from paper_2509_15965_amd.rl_decode import Engine

pytestmark = pytest.mark.gpu


def test_gate_up_over_32_rows_is_not_sliced():
    # SwiGLU slices cost a launch of their own: one round of 128 x 256 tiles is the faster plan here (7B shape, 2 layers,
    # 40 rows: 298 us a step against 327 with two slices of 128 x 128 tiles)
    s = replace(configs.QWEN_7B, n_layers=1, vocab=1024)
    eng = Engine(s, make_weights(s, 1, device="cuda", init="fanin"), max_seqs=64, max_ctx=64, max_prefill_tokens=64)
    splits = [eng.gemm_plan("gemm_gate_up", rows)[0] >> 8 & 0xff for rows in range(33, 65)]
    eng.close()
    assert splits == [0] * 32
