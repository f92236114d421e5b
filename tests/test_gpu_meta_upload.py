"""A call's metadata around the size where its upload changes from a kernel to a copy: a paged pool whose page table is
a little under and over 1 MiB, against the same steps with a table of a few entries."""
import numpy as np
import pytest
import torch

from paper_2509_15965_amd.configs import ModelShape
from paper_2509_15965_amd.inputs import make_weights
from paper_2509_15965_amd.rl_decode import Engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seqs", [1019, 1024])   # tables of 4 * seqs * 256 bytes; about 1 KiB of other metadata
def test_upload_sizes(seqs):
    s = ModelShape(1, 128, 2, 1, 64, 128, 264, 1e-6, 1e4, "bf16")
    w = make_weights(s, 4, device="cuda", init="fanin")
    out = []
    for max_seqs, max_ctx in ((5, 160), (seqs, 8192)):
        eng = Engine(s, w, max_seqs=max_seqs, max_ctx=max_ctx, max_prefill_tokens=512, kv_page_size=32, kv_pages=64)
        slots = [max_seqs - 1, 1, 2, max_seqs // 2 + 1, 0]
        offs = np.cumsum([0, 100, 33, 32, 1, 64])
        toks = torch.arange(offs[-1], dtype=torch.int32, device="cuda") * 7 % s.vocab
        tok, lp, z = torch.empty(5, dtype=torch.int32, device="cuda"), torch.empty(5, device="cuda"), torch.empty((5, s.vocab), device="cuda")
        eng.prefill(slots, range(5), offs, toks, tok, lp)
        for _ in range(4):   # more calls than staging buffers
            eng.step(slots, range(5), tok.clone(), tok, lp, out_logits=z)
        torch.cuda.synchronize()
        out.append((z.clone(), tok.clone(), lp.clone()))
        eng.close()
    assert all(torch.equal(a, b) for a, b in zip(*out))
