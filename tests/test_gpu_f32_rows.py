"""fp32 projections at the edges of their two kernels: row counts around the activation blocks of 2, 4 and
8, output widths and K that no block divides, and enough rows for the tiled kernel."""
import numpy as np
import pytest
import torch

from harness import F32_LOGIT_REL_TOL, build_models, row_rel_err
from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.rl_decode import Engine

pytestmark = pytest.mark.gpu


# ffn 3096: 194 workgroups a row block, so 300 prompt rows (38 blocks) pass the limit of 6144
@pytest.mark.parametrize("ffn,lens", [(40, [1]), (40, [1, 1]), (40, [1, 2]), (40, [4]), (40, [2, 3]), (40, [9]),
                                      (3096, [7]), (3096, [300])])
def test_fp32_rows(ffn, lens):
    shape = ModelShape(2, 72, 2, 1, 64, ffn, 104, 1e-6, 1e4, "fp32")
    w, _, om = build_models(shape, 5, init="normal")
    n = len(lens)
    eng = Engine(shape, w, max_seqs=n, max_ctx=320, max_prefill_tokens=sum(lens))
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    toks = torch.arange(sum(lens), dtype=torch.int32, device="cuda") * 7 % shape.vocab
    tok, lp = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")
    z0, z1 = (torch.empty((n, shape.vocab), device="cuda") for _ in range(2))
    eng.prefill(list(range(n)), list(range(n)), offs, toks, tok, lp, out_logits=z0)
    first = tok.clone()
    eng.step(list(range(n)), list(range(n)), first, tok, lp, out_logits=z1)
    torch.cuda.synchronize()
    for i in range(n):
        s = om.new_seq(320)
        for t in toks[offs[i]:offs[i + 1]].tolist():
            ref = s.forward(t)
        assert row_rel_err(z0[i].cpu().numpy(), ref) < F32_LOGIT_REL_TOL
        assert row_rel_err(z1[i].cpu().numpy(), s.forward(int(first[i]))) < F32_LOGIT_REL_TOL
    eng.close()
