"""The 256 x 256 GEMM whose tiles past the whole rounds are cut in K (the planner's choice for these sizes),
for each epilogue: a prefill against the same prefill with plain 256 x 256 tiles forced."""
import numpy as np
import pytest
import torch

from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.inputs import make_weights
from paper_2509_15965_amd.rl_decode import RL_GEMM_T256, RL_OPT_GEMM_PLAN, Engine, gemm_plan_code

pytestmark = pytest.mark.gpu


# 33 row tiles (the last one of 100 rows).  hidden 2048 + 64: 9 column tiles, the last 64 wide: 297 tiles, 41 of
# them cut in 6 (o, down).  q|k|v 2048: 264 tiles, 8 cut in 8 (K 2112) ; gate|up 2 * 2000: 528 tiles, 16 cut
@pytest.mark.parametrize("rows,hidden,heads,ffn", [(33 * 256 - 156, 2112, 12, 2048), (33 * 256, 2048, 12, 2000)])
def test_cut_remainder(rows, hidden, heads, ffn):
    shape = ModelShape(2, hidden, heads, 2, 128, ffn, 8192 - 8, 1e-6, 1e4, "bf16")
    w = make_weights(shape, 3, device="cuda", init="fanin")
    n = 33
    lens = [rows // n + (1 if i < rows % n else 0) for i in range(n)]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    toks = torch.randint(0, shape.vocab, (rows,), device="cuda", dtype=torch.int32,
                         generator=torch.Generator("cuda").manual_seed(1))
    eng = Engine(shape, w, max_seqs=n, max_ctx=max(lens) + 2, max_prefill_tokens=rows)
    out = []
    for plan in (gemm_plan_code(RL_GEMM_T256), 0):
        eng.set_option(RL_OPT_GEMM_PLAN, plan)
        tok, lp = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")
        z = torch.empty((n, shape.vocab), device="cuda")
        eng.prefill(list(range(n)), list(range(n)), offs, toks, tok, lp, out_logits=z)
        torch.cuda.synchronize()
        out.append(z.double())
        eng.set_lengths(list(range(n)), [0] * n)
    eng.close()
    # the slices are summed in another order: fp32 rounding, which flips bf16 storage roundings of both layers
    # (each flip 2^-8 of an element; two bf16 versions of this depth differ by about 2e-3 of the norm)
    assert torch.isfinite(out[1]).all()
    assert float((out[1] - out[0]).norm() / out[0].norm()) < 1e-2
    assert not torch.equal(out[0], out[1])   # the cut kernel ran
