"""Prefill attention in 32-column tiles against the split-KV work items, at the edges of tokens per wave and per
tile for every grouping of q-heads, ragged last steps, and pages."""
import numpy as np
import pytest
import torch

from harness import ATTENTION_REL_TOL, attention_alone
from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.inputs import make_weights
from paper_2509_15965_amd.rl_decode import RL_OPT_PREFILL_ATTENTION, Engine

pytestmark = pytest.mark.gpu


# (q-heads per kv-head, head_dim); tokens per wave 32, 16, 10, 6, 4, 2 in tiles of 4 waves, or of 8 where these make
# 224 workgroups (never with up to two q-heads)
@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("G,d,page", [(1, 64, 0), (1, 128, 64), (2, 128, 0), (3, 64, 32), (5, 128, 0), (7, 128, 96), (16, 64, 0)])
def test_tiles(G, d, page, many):
    s = ModelShape(1, 256, 2 * G, 2, d, 128, 264, 1e-6, 1e4, "bf16")
    w = attention_alone(make_weights(s, 6, device="cuda", init="fanin"))
    per_wave = 32 // G
    tile = per_wave * (8 if many and G > 2 else 4)
    lens = [1, 2, 31, 32, 33, per_wave, per_wave + 1, tile - 1, tile, tile + 1, 2 * tile + 3]

    def workgroups():   # if they had eight waves
        return 2 * sum(-(-m // (8 * per_wave)) for m in lens)
    while many and workgroups() < 224:
        lens = lens + lens[:11]
    assert many or workgroups() < 224
    n, rows = len(lens), sum(lens)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    toks = torch.randint(0, s.vocab, (rows,), device="cuda", dtype=torch.int32, generator=torch.Generator("cuda").manual_seed(1))
    eng = Engine(s, w, max_seqs=n, max_ctx=max(lens) + 2, max_prefill_tokens=2 * rows, kv_page_size=page)
    # keys past a sequence's end are not finite: a step that let one through would show it
    eng.kv.view(torch.bfloat16).fill_(float("nan"))
    out = []
    for items in (1, 0):
        eng.set_option(RL_OPT_PREFILL_ATTENTION, items)
        lp = torch.empty(rows - n, device="cuda")
        two = [i for i in range(n) if lens[i] > 1]
        # every position's output counts: score each prompt's own tokens as responses of its first one
        first = torch.cat([toks[offs[i]:offs[i] + 1] for i in two])
        rest = torch.cat([toks[offs[i] + 1:offs[i + 1]] for i in two])
        eng.score(two, np.arange(len(two) + 1), first, offsets([lens[i] - 1 for i in two]), rest, lp)
        z, tok, l0 = torch.empty((n, s.vocab), device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")
        eng.prefill(list(range(n)), list(range(n)), offs, toks, tok, l0, out_logits=z)
        torch.cuda.synchronize()
        out.append((z.double(), lp.double()))
        eng.release(list(range(n)))
    eng.close()
    (za, la), (zb, lb) = out
    assert torch.isfinite(zb).all() and torch.isfinite(lb).all()
    # one key of 260 left out moves a row by 0.06 of its norm; logits of about 1, up to 4 of them apart by their bound
    assert float(((zb - za).norm(dim=1) / za.norm(dim=1)).max()) < ATTENTION_REL_TOL
    assert float((lb - la).abs().max()) < 4 * ATTENTION_REL_TOL


def offsets(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
