"""The 256 x 256 GEMM whose tiles past the whole rounds are cut in K, for each projection and epilogue: a prefill
against the same prefill with plain 256 x 256 tiles, tile by tile of the residual stream."""
import numpy as np
import pytest
import torch

from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.inputs import make_weights
from paper_2509_15965_amd.rl_decode import RL_GEMM_T256, RL_GEMM_T256_CUT, RL_OPT_GEMM_PLAN, Engine, RLError, gemm_plan_code

pytestmark = pytest.mark.gpu

CLASSES = ("gemm_qkv", "gemm_o", "gemm_gate_up", "gemm_down")


def run(eng, shape, rows, plan):
    """The residual stream [rows][hidden] after a prefill of 33 prompts (the first region of the workspace)."""
    n = 33
    lens = [rows // n + (1 if i < rows % n else 0) for i in range(n)]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    toks = torch.randint(0, shape.vocab, (rows,), device="cuda", dtype=torch.int32,
                         generator=torch.Generator("cuda").manual_seed(1))
    tok, lp = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")
    eng.set_option(RL_OPT_GEMM_PLAN, plan)
    eng.prefill(list(range(n)), list(range(n)), offs, toks, tok, lp)
    torch.cuda.synchronize()
    x = eng.ws[:4 * rows * shape.hidden].view(torch.float32).view(rows, shape.hidden).double()
    eng.set_lengths(list(range(n)), [0] * n)
    return x


# 33 row tiles, the last one of 100 rows.  q|k|v (30 + 2 * 2) * 64 = 2176: 9 column tiles, the last 128 wide, 297 tiles,
# 41 of them cut in 6 slices of 384 (the last of 192).  o and down: hidden 2112, the last column tile 64 wide, cut in 6 of
# 320 (K 1920) and 6 of 384.  gate|up: 2112 columns of act in 17 tiles, 561 tiles, 49 cut in 5 of 448 (the last of 320).
# The second shape: whole tiles, 8 or 32 of them cut in 8, 6, 8 and 16 whole slices of 256
@pytest.mark.parametrize("rows,hidden,q_heads,d,ffn", [(33 * 256 - 156, 2112, 30, 64, 2112), (33 * 256, 2048, 12, 128, 4096)])
def test_cut_remainder(rows, hidden, q_heads, d, ffn):
    shape = ModelShape(1, hidden, q_heads, 2, d, ffn, 264, 1e-6, 1e4, "bf16")
    w = make_weights(shape, 3, device="cuda", init="fanin")
    w["embed"] /= 128   # the projections' outputs are the residual stream
    eng = Engine(shape, w, max_seqs=33, max_ctx=300, max_prefill_tokens=rows)
    plain = run(eng, shape, rows, gemm_plan_code(RL_GEMM_T256))
    cut = run(eng, shape, rows, RL_GEMM_T256_CUT)
    again = run(eng, shape, rows, RL_GEMM_T256_CUT)
    assert [eng.gemm_plan(c, rows)[0] for c in CLASSES] == [RL_GEMM_T256_CUT] * 4
    eng.close()
    assert torch.equal(cut, again) and not torch.equal(plain, cut)
    # the slices are summed in another order: fp32 roundings, and the bf16 ones of attention, act and norms that they flip,
    # each 2^-8 of an element at most; one 64-wide step of K left out of a tile is 0.15 of it
    diff, ref = (cut - plain).square(), plain.square()
    for m in range(0, rows, 256):
        for c in range(0, hidden, 256):
            t = (slice(m, m + 256), slice(c, c + 256))
            assert float((diff[t].sum() / ref[t].sum()).sqrt()) < 2.0 ** -8, (m, c)


def test_plan_codes():
    # the cost model takes the cut for q|k|v of this shape and reports it by its own code, which the override takes alone
    shape = ModelShape(1, 2048, 12, 2, 128, 2000, 264, 1e-6, 1e4, "bf16")
    eng = Engine(shape, make_weights(shape, 3, device="cuda", init="fanin"), max_seqs=1, max_ctx=300, max_prefill_tokens=33 * 256)
    assert eng.gemm_plan("gemm_qkv", 33 * 256)[0] == RL_GEMM_T256_CUT
    for bad in (8, RL_GEMM_T256_CUT | 2 << 8, RL_GEMM_T256_CUT | RL_GEMM_T256 << 16, RL_GEMM_T256 | RL_GEMM_T256_CUT << 16):
        with pytest.raises(RLError):
            eng.set_option(RL_OPT_GEMM_PLAN, bad)
    eng.close()
