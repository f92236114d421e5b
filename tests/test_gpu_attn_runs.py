"""Decode attention over equal runs of all rows' keys, against one item per row (a chunk that holds the longest):
runs that start and end inside rows, rows shorter than a step, a row cut into the most items, more rows than
waves, keys that end on and off 32-position steps and pages."""
import numpy as np
import pytest
import torch

from harness import ATTENTION_REL_TOL, attention_alone
from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.inputs import make_weights
from paper_2509_15965_amd.rl_decode import RL_OPT_ATTN_CHUNK, Engine

pytestmark = pytest.mark.gpu

SHAPES = {"g7": ModelShape(1, 448, 14, 2, 64, 128, 264, 1e-6, 1e4, "bf16"),
          "g1": ModelShape(1, 256, 2, 2, 128, 128, 264, 1e-6, 1e4, "bf16"),
          "g16": ModelShape(1, 1024, 16, 1, 64, 128, 264, 1e-6, 1e4, "bf16")}


@pytest.mark.parametrize("shape,lens,page", [
    ("g7", [0], 0), ("g7", [31], 0), ("g7", [32], 0), ("g7", [63, 0, 1, 31, 32, 33, 500, 64], 0),
    ("g1", [4100, 3, 2, 1], 0), ("g16", [6000], 0), ("g7", [5, 40, 100, 7] * 200, 0),
    ("g1", [255, 256, 257, 31, 700, 0], 64), ("g7", [95, 96, 97, 64, 1000, 2], 96)])
def test_runs(shape, lens, page):
    s = SHAPES[shape]
    n = len(lens)
    w = attention_alone(make_weights(s, 4, device="cuda", init="fanin"))
    eng = Engine(s, w, max_seqs=n, max_ctx=max(lens) + 2, max_prefill_tokens=64, kv_page_size=page)
    slots = list(range(n))
    if page:
        eng.set_lengths(slots, [max(lens) + 1] * n)   # every page taken, so the whole pool holds finite values
    eng.kv.view(torch.bfloat16).normal_(generator=torch.Generator("cuda").manual_seed(2))
    tok = torch.arange(n, dtype=torch.int32, device="cuda") % s.vocab
    ot, lp = torch.empty_like(tok), torch.empty(n, device="cuda")
    out = []
    for chunk in (65536, 0):
        eng.set_option(RL_OPT_ATTN_CHUNK, chunk)
        z = torch.empty((n, s.vocab), device="cuda")
        eng.set_lengths(slots, lens)
        eng.step(slots, slots, tok, ot, lp, out_logits=z)
        torch.cuda.synchronize()
        out.append(z.double())
    eng.close()
    assert torch.isfinite(out[1]).all()
    # a 32-key step left out (or taken twice) moves a row by 0.07 of its norm at 6000 keys, one key by 0.013
    err = (out[1] - out[0]).norm(dim=1) / out[0].norm(dim=1)
    assert float(err.max()) < ATTENTION_REL_TOL
