"""The scoring head that reduces logits inside its GEMM tiles against the one that writes them (each sequence scored
alone), on the same hidden states."""
import numpy as np
import pytest
import torch

from harness import LOGP_ABS_TOL
from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.inputs import make_weights
from paper_2509_15965_amd.rl_decode import (KERNEL_CLASSES, RL_GEMM_T128, RL_GEMM_T256, RL_OPT_GEMM_PLAN, RL_OPT_PROFILE,
                                            Engine, gemm_plan_code)

pytestmark = pytest.mark.gpu


def score(eng, prompts, group, resp, T):
    po = np.concatenate([[0], np.cumsum([len(p) for p in prompts])]).astype(np.int32)
    ro = np.concatenate([[0], np.cumsum([len(r) for r in resp])]).astype(np.int32)
    out = torch.empty(int(ro[-1]), device="cuda")
    i32 = lambda a: torch.as_tensor(np.concatenate(a), dtype=torch.int32, device="cuda")
    eng.score(list(range(len(resp))), po, i32(prompts), ro, i32(resp), out, group=group, temperature=T)
    torch.cuda.synchronize()
    return out.cpu().numpy()


# head rows 130, 256 (a whole row tile), 257 and 585, in tiles by override; vocabularies of one ragged column tile, whole
# tiles and a ragged last one
@pytest.mark.parametrize("vocab,rlens,T", [(200, [65, 65, 1, 1], 1.0), (512, [64, 64, 64, 66], 0.6), (1032, [64, 64, 64, 67], 0.0),
                                           (1288, [100, 120, 40, 90, 110, 128], 0.6)])
def test_head_in_tiles(vocab, rlens, T):
    shape = ModelShape(1, 256, 4, 2, 64, 512, vocab, 1e-6, 1e4, "bf16")
    w = make_weights(shape, 9, device="cuda", init="fanin")
    w["lm_head"][min(vocab - 1, 130)] *= 12   # one entry far above the rest: a column tile that dominates the sum
    rng = np.random.default_rng(vocab)
    group = 2
    prompts = [rng.integers(0, vocab, 9).astype(np.int32) for _ in range(len(rlens) // group)]
    resp = [rng.integers(0, vocab, m).astype(np.int32) for m in rlens]
    resp[0][3], resp[1][0] = -1, vocab   # not scored: NaN
    eng = Engine(shape, w, max_seqs=len(rlens), max_ctx=160, max_prefill_tokens=1024)
    # tile kernels for every row count, both adding up K in the same order: the hidden states are then the same
    # bits in both calls, and the 256 x 256 one reduces the logits in its tiles
    eng.set_option(RL_OPT_GEMM_PLAN, gemm_plan_code(RL_GEMM_T256))
    together = score(eng, prompts, group, resp, T)
    eng.set_option(RL_OPT_GEMM_PLAN, gemm_plan_code(RL_GEMM_T128))
    alone = np.concatenate([score(eng, [prompts[i // group]], 1, [resp[i]], T) for i in range(len(resp))])
    eng.close()
    assert np.array_equal(np.isnan(together), np.isnan(alone)) and np.isnan(alone).sum() == 2
    # fp32 sums in another order: logits of |z| < 64 and their LSE, each a few units of 2^-24 relative, over T
    np.testing.assert_allclose(together[~np.isnan(alone)], alone[~np.isnan(alone)], rtol=0, atol=64 * 2.0 ** -21)


def test_certain_tokens_are_not_above_zero():
    # a greedy rollout scored again: every target is its row's largest logit, far above the rest.  The log-sum-exp
    # is never below the largest of its terms, so no log-probability is above 0 when both come from one logit.
    shape = ModelShape(1, 256, 4, 2, 64, 512, 1032, 1e-6, 1e4, "bf16")
    w = make_weights(shape, 3, device="cuda", init="fanin")
    w["lm_head"] *= 64
    n, steps = 8, 40
    rng = np.random.default_rng(1)
    prompts = [rng.integers(0, shape.vocab, 5 + i).astype(np.int32) for i in range(n)]
    eng = Engine(shape, w, max_seqs=n, max_ctx=96, max_prefill_tokens=1024)
    tok, lp = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")
    ids, offs = list(range(n)), np.concatenate([[0], np.cumsum([len(p) for p in prompts])])
    eng.prefill(ids, ids, offs, torch.as_tensor(np.concatenate(prompts), device="cuda"), tok, lp, temperature=0.0)
    out = [tok.clone()]
    for _ in range(steps - 1):
        eng.step(ids, ids, out[-1], tok, lp, temperature=0.0)
        out.append(tok.clone())
    eng.release(ids)
    resp = list(torch.stack(out, 1).cpu().numpy())
    eng.set_option(RL_OPT_GEMM_PLAN, gemm_plan_code(RL_GEMM_T256))
    together = score(eng, prompts, 1, resp, 1.0)   # in tiles
    eng.set_option(RL_OPT_GEMM_PLAN, 0)
    alone = np.concatenate([score(eng, [prompts[i]], 1, [resp[i]], 1.0) for i in range(n)])
    eng.close()
    for lps in (together, alone):
        assert lps.max() <= 0.0 and np.mean(lps > -1e-3) > 0.5   # most of them certain


# a whole column tile of the logit (and whole lanes of the other head's sum), or one of its columns
@pytest.mark.parametrize("rows", [slice(256, 512), slice(700, 701), slice(0, 4)])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_logits_that_are_not_finite(rows, value):
    shape = ModelShape(1, 256, 4, 2, 64, 512, 1032, 1e-6, 1e4, "bf16")
    w = make_weights(shape, 3, device="cuda", init="fanin")
    w["embed"].fill_(1.0), w["final_norm"].fill_(1.0), w["w_o"].zero_(), w["w_down"].zero_()   # hidden states of 1
    w["lm_head"][rows, 0] = value
    rng = np.random.default_rng(2)
    prompts = [rng.integers(0, shape.vocab, 9).astype(np.int32)]
    resp = [rng.integers(4, 200, 70).astype(np.int32) for _ in range(4)]
    eng = Engine(shape, w, max_seqs=4, max_ctx=96, max_prefill_tokens=1024)
    eng.set_option(RL_OPT_GEMM_PLAN, gemm_plan_code(RL_GEMM_T256))   # in tiles
    together = score(eng, prompts, 4, resp, 0.7)
    eng.set_option(RL_OPT_GEMM_PLAN, 0)
    alone = score(eng, prompts, 1, resp[:1], 0.7)
    eng.close()
    if value == -np.inf:   # left out of the sum
        assert np.isfinite(together).all()
        np.testing.assert_allclose(together[:70], alone, rtol=0, atol=64 * 2.0 ** -21)
    else:   # the row has no log-sum-exp
        assert np.isnan(alone).all() and np.isnan(together).all()


@pytest.mark.parametrize("vocab,spread", [(264, 4.0), (4096, 1.0), (32000, 2.0)])
def test_error_against_64_bits(vocab, spread):
    # logits that are exact in every kernel (hidden states of 1, one weight a row), so that the sums alone differ: the
    # head in tiles is no further from 64 bits than the one over written logits
    s = ModelShape(1, 64, 1, 1, 64, 64, vocab, 1e-6, 1e4, "bf16")
    w = make_weights(s, 3, device="cuda", init="fanin")
    w["embed"].fill_(1.0), w["final_norm"].fill_(1.0), w["w_o"].zero_(), w["w_down"].zero_(), w["lm_head"].zero_()
    eng = Engine(s, w, max_seqs=2, max_ctx=96, max_prefill_tokens=512)
    err = {RL_GEMM_T256: [], RL_GEMM_T128: []}
    for seed in range(8):
        z = torch.randn(vocab, generator=torch.Generator("cuda").manual_seed(seed), device="cuda") * spread
        w["lm_head"][:, 0] = z.bfloat16()
        zz = w["lm_head"][:, 0].float()
        resp = [np.array([int(zz.argmax())] + list(range(69)), np.int32)] * 2
        for T in (1.0, 0.6, 0.83):
            zt = (zz / np.float32(T)).double()
            ref = (zt[torch.as_tensor(np.concatenate(resp), device="cuda").long()] - torch.logsumexp(zt, 0)).cpu().numpy()
            for plan in err:
                eng.set_option(RL_OPT_GEMM_PLAN, gemm_plan_code(plan))
                err[plan].append(score(eng, [resp[0][:1]], 2, resp, T) - ref)
    eng.close()
    tiles, logits = (np.sqrt(np.mean(np.square(np.array(err[p], dtype=np.float64)))) for p in err)
    # both are mostly the final roundings (half an ulp of values up to 40: 1.9e-6); rms over 24 sums, so a fifth apart at most
    assert tiles < 1.2 * logits and tiles < 1.9e-6


# the default choice: 128 head rows over written logits, 129 in tiles where the vocabulary has enough of them (41 column
# tiles at hidden 256, and not 39) or where the logits buffer takes the rows in more than one chunk
@pytest.mark.parametrize("vocab,rlens,ffn,tiles", [(10248, [65, 64], 512, False), (10248, [65, 65], 512, True),
                                                   (9800, [65, 65], 512, False), (9800, [65, 65], 64, True)])
def test_default_choice(vocab, rlens, ffn, tiles):
    shape = ModelShape(1, 256, 4, 2, 64, ffn, vocab, 1e-6, 1e4, "bf16")
    w = make_weights(shape, 9, device="cuda", init="fanin")
    rng = np.random.default_rng(vocab)
    prompt = [rng.integers(0, vocab, 9).astype(np.int32)]
    resp = [rng.integers(0, vocab, m).astype(np.int32) for m in rlens]
    rows = 1 + sum(rlens) - 2
    # max_prefill_tokens sets the MLP buffer: 8192 * 512 / (2 * vocab) rows of logits, or 8192 * 64 / (2 * vocab)
    eng = Engine(shape, w, max_seqs=2, max_ctx=160, max_prefill_tokens=8192)
    eng.set_option(RL_OPT_PROFILE, 1 << KERNEL_CLASSES.index("gemm_lm_head"))
    together = score(eng, prompt, 2, resp, 1.0)
    st = eng.kernel_stats()["gemm_lm_head"]
    alone = np.concatenate([score(eng, prompt, 1, [r], 1.0) for r in resp])
    eng.close()
    logits_bytes = 4 * rows * vocab
    assert (st["alg_bytes"] - 2 * 256 * (vocab + rows) < logits_bytes / 2) == tiles
    # the projections' plans differ with the row count: bf16 roundings of one layer
    assert np.abs(together - alone).max() < LOGP_ABS_TOL
