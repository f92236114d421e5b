"""Test helpers: run the GPU library (through the C ABI binding) and the CPU
oracle on the same seeded inputs and compare them.

The two sides share only the seeded input generators.  Expected values come
from the oracle; the GPU outputs are only ever compared against them.
"""
import numpy as np
import torch

import oracle
from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.inputs import bf16_bits_to_f64, make_weights, to_host_numpy, weights_to_host

# bf16 tolerances: per-row relative max error of the logits, absolute log-prob error
LOGIT_REL_TOL = 3e-2
LOGP_ABS_TOL = 2e-2
# fp32 tolerances (fp32 accumulation against the fp64 oracle)
F32_LOGIT_REL_TOL = 1e-4
F32_LOGP_ABS_TOL = 1e-4
NEAR_TIE = 1e-4

# Two bf16 versions of attention_alone's model differ by the roundings of the attention output and of the final norm,
# each half an ulp (2^-9 of the element at most) where they flip: 2 * 2^-9 * sqrt(2) of a row's norm if all did
ATTENTION_REL_TOL = 2.0 ** -7.5


def attention_alone(w):
    """Weights whose logits are the last layer's attention output and next to nothing else: embeddings (whose
    normalised rows are as they were) at 1/128, the output projection at 128, no MLP."""
    w["embed"] /= 128
    w["w_o"] *= 128
    w["w_down"].zero_()
    return w


def oracle_mode(shape: ModelShape) -> int:
    return oracle.MODE_BF16 if shape.dtype == "bf16" else oracle.MODE_FP32


def build_models(shape: ModelShape, seed: int, device="cuda", init: str = "normal"):
    """Same seeded weights for both sides: device tensors and an oracle model."""
    w_dev = make_weights(shape, seed, device=device, init=init)
    w_host = weights_to_host(w_dev)
    om = oracle.OracleModel(shape.as_dict(), w_host, oracle_mode(shape))
    return w_dev, w_host, om


def row_rel_err(gpu: np.ndarray, ref: np.ndarray) -> float:
    """max over rows of max|gpu - ref| / max|ref|"""
    gpu = np.atleast_2d(gpu).astype(np.float64)
    ref = np.atleast_2d(ref).astype(np.float64)
    return float(np.max(np.abs(gpu - ref).max(axis=1) / np.abs(ref).max(axis=1)))


def check_token(gpu_tok: int, z_orc: np.ndarray, T: float, seed: int, uid: int, pos_new: int, excused: list):
    """fp32 parity: the GPU token equals the oracle's sample, or the draw is a
    near tie (top-two perturbed-score margin < 1e-4) and the GPU picked the
    runner-up."""
    o_tok, _ = oracle.sample(z_orc.astype(np.float32), T, seed, uid, pos_new)
    if gpu_tok == o_tok:
        return True
    a, b, margin = oracle.sample_margin(z_orc.astype(np.float32), T, seed, uid, pos_new)
    if margin < NEAR_TIE and gpu_tok == b:
        excused.append((uid, pos_new, margin))
        return True
    return False


class OracleRollout:
    """Oracle-side sequences for a prefill + decode run with given tokens."""

    def __init__(self, om: oracle.OracleModel, max_ctx: int):
        self.om = om
        self.max_ctx = max_ctx
        self.seqs = {}

    def prefill(self, key, prompt_tokens, embed_rows=None):
        """prompt_tokens: ids (< 0 select embed_rows[-id-1]); returns last logits."""
        s = self.om.new_seq(self.max_ctx)
        z = None
        for t in prompt_tokens:
            t = int(t)
            if t < 0:
                z = s.forward(t, embed_row=embed_rows[-t - 1])
            else:
                z = s.forward(t)
        self.seqs[key] = s
        return z

    def step(self, key, tok):
        return self.seqs[key].forward(int(tok))

    def length(self, key):
        return self.seqs[key].length


def inject_random_kv(engine, om, slots, lengths, seed: int):
    """Fill slots' caches with seeded N(0,1) rows (model dtype) through the
    documented pool layout, declare their lengths, and give the oracle the
    same rows.  Returns the oracle sequences, keyed by slot."""
    shape = engine.shape
    Kv, Vv = engine.kv_views()
    L, Hkv, D = shape.n_layers, shape.n_kv_heads, shape.head_dim
    dt = torch.float32 if shape.dtype == "fp32" else torch.bfloat16
    gen = torch.Generator(device=engine.device)
    gen.manual_seed(int(seed))
    seqs = {}
    for slot, n in zip(slots, lengths):
        K = torch.randn((L, Hkv, n, D), generator=gen, device=engine.device, dtype=torch.float32).to(dt)
        V = torch.randn((L, Hkv, n, D), generator=gen, device=engine.device, dtype=torch.float32).to(dt)
        Kv[:, slot, :, :n, :] = K
        nb = (n + 7) // 8
        Vpad = torch.zeros((L, Hkv, nb * 8, D), device=engine.device, dtype=dt)
        Vpad[:, :, :n] = V
        # [L][Hkv][nb][8][D] -> [L][Hkv][nb][D][8]
        Vv[:, slot, :, :nb] = Vpad.view(L, Hkv, nb, 8, D).transpose(3, 4)
        s = om.new_seq(engine.cfg.max_ctx)
        Kh, Vh = to_host_numpy(K), to_host_numpy(V)
        Kh = bf16_bits_to_f64(Kh) if Kh.dtype == np.uint16 else Kh.astype(np.float64)
        Vh = bf16_bits_to_f64(Vh) if Vh.dtype == np.uint16 else Vh.astype(np.float64)
        for l in range(L):
            for g in range(Hkv):
                s.set_kv_block(l, g, Kh[l, g], Vh[l, g])
        s.set_length(n)
        seqs[slot] = s
        del K, V, Vpad
    engine.set_lengths(list(slots), list(lengths))
    torch.cuda.synchronize()
    return seqs
