"""The experts' projections in MFMA tiles of 128 and 256 pairs: part-filled, exactly full and several row tiles
per expert, column tiles past the width.  Every expert is chosen by every token, so no routing decision is a
near tie, and every row is compared."""
import numpy as np
import pytest
import torch

from harness import LOGIT_REL_TOL, LOGP_ABS_TOL, build_models, row_rel_err
from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.rl_decode import Engine
import oracle

pytestmark = pytest.mark.gpu


# pairs per expert = rows.  1 row, and 2 rows of 8 narrow experts: the GEMV form; 1100 and 1024: tiles of 256.  16
# experts of 2048 at hidden 128: gate|up alone in tiles (256) from 2 rows; at hidden 4096 and 8 rows: down alone
@pytest.mark.parametrize("E,rows,hidden,ffn", [(8, 1, 128, 64), (8, 2, 128, 64), (3, 128, 192, 192), (4, 129, 320, 64),
                                               (4, 600, 128, 320), (2, 1100, 128, 64), (2, 1024, 192, 192),
                                               (4, 63, 128, 64), (4, 64, 128, 64), (16, 8, 4096, 64), (16, 2, 128, 2048)])
def test_expert_tiles(E, rows, hidden, ffn):
    shape = ModelShape(1, hidden, 2, 1, 64, 0, 264, 1e-6, 1e4, "bf16", n_experts=E, top_k=E, expert_ffn=ffn)
    w, _, om = build_models(shape, 11, init="fanin")
    toks = (torch.arange(rows, dtype=torch.int64) * 37 % shape.vocab).to(torch.int32)
    eng = Engine(shape, w, max_seqs=1, max_ctx=rows + 2, max_prefill_tokens=rows)
    tok, lp = torch.empty(1, dtype=torch.int32, device="cuda"), torch.empty(1, device="cuda")
    z = torch.empty((1, shape.vocab), device="cuda")
    target = torch.tensor([5], dtype=torch.int32, device="cuda")
    eng.prefill([0], [0], [0, rows], toks.cuda(), tok, lp, forced=target, out_logits=z)
    out = torch.empty(rows - 1, device="cuda")
    if rows > 1:   # every row's experts, not the last row's alone
        eng.score([0], [0, 1], toks[:1].cuda(), [0, rows - 1], toks[1:].cuda(), out)
    torch.cuda.synchronize()
    s = om.new_seq(rows + 2)
    ref, lps = None, []
    for i in range(rows):
        ref = s.forward(int(toks[i]))
        if i + 1 < rows:
            lps.append(oracle.logprob(ref.astype(np.float32), 1.0, int(toks[i + 1])))
    eng.close()
    assert row_rel_err(z.cpu().numpy(), ref) < LOGIT_REL_TOL
    assert abs(float(lp[0]) - oracle.logprob(ref.astype(np.float32), 1.0, 5)) < LOGP_ABS_TOL
    if rows > 1:
        assert np.abs(out.cpu().numpy() - np.array(lps)).max() < LOGP_ABS_TOL
