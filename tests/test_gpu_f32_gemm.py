"""The fp32 matrix-core GEMM through whole fp32 steps, at widths and token
counts where its launcher takes each of its tile shapes, with and without a K
split, under each epilogue.

``products`` names a block's products and ``STACKS`` the steps; the host test
``test_gpu_steps_cover_every_tile`` (test_f32_gemm_choice.py) holds them to
the launcher's choice, so that a change of its rule cannot drop the coverage
unseen.  Widths are multiples of 8 that no tile divides, token counts are
ragged too.  A step covers the three operand orientations (both k-contiguous,
only A, neither), the K-concatenated output projection and every epilogue; the
vocabulary steps have a head whose width and contraction are no multiple of 4.
The oracle is fp64 and the tolerance that of the other fp32 tests.
"""
import numpy as np
import pytest

import oracle
from paper_2510_14614_amd import synth
from paper_2510_14614_amd.config import ARCH_FAL, SCHED_SEQ, SCHED_STREAMS_MERGED, Config

from gpu_helpers import compare_step, gpu_model_step, gpu_stack_step, log

pytestmark = pytest.mark.gpu

# (d, heads, head_dim, f, seq_len, batch)
STACKS = [(136, 2, 16, 328, 300, 3), (328, 4, 16, 840, 300, 4), (520, 8, 64, 2056, 300, 7),
          (264, 2, 64, 3080, 1153, 2),    # FFN up and its data gradient on 128 x 128, unsplit
          (3080, 2, 64, 264, 1153, 2),    # the K-concatenated projection and the plain data gradients on 128 x 128
          (1032, 16, 64, 264, 1065, 2)]   # that projection on 64 x 64, a weight gradient split on 128 x 128


def products(d, heads, hd, f, seq, batch):
    """{product: (M, N, K, K2, may split)} of a block with its branches on streams."""
    M, dA = batch * seq, heads * hd
    return {"qkv": (M, 3 * dA, d, 0, 0), "ffn up, GELU": (M, f, d, 0, 0), "projection, residual": (M, d, dA, f, 0),
            "ffn up gradient, GELU'": (M, f, d, 0, 0), "dO": (M, dA, d, 0, 1), "dH2": (M, d, f, 0, 1),
            "dH1": (M, d, 3 * dA, 0, 1), "dW_o": (dA, d, M, 0, 1), "dW_2": (f, d, M, 0, 1), "dW_fc": (d, f, M, 0, 1),
            "dW_qkv": (d, 3 * dA, M, 0, 1)}


@pytest.mark.parametrize("sched", [SCHED_SEQ, SCHED_STREAMS_MERGED])
@pytest.mark.parametrize("d,heads,hd,f,seq,batch", STACKS)
def test_f32_stack_step_tile_shapes(d, heads, hd, f, seq, batch, sched):
    cfg = Config(n_layer=2, d_model=d, n_head=heads, head_dim=hd, d_ff=f, vocab=0, seq_len=seq, batch=batch,
                 arch=ARCH_FAL, dtype=0, has_embed_head=0, sched=sched)
    log(f"fp32 stack step d={d} f={f} tokens={cfg.tokens} sched={sched}")
    _, blocks = synth.make_params(cfg, seed=90)
    x1, gout = synth.make_stack_inputs(cfg, seed=91)
    ref = oracle.stack_step(cfg, blocks, x1, gout)
    ref["loss_scale"] = float(np.abs(gout * ref["y"]).sum())
    compare_step(cfg, gpu_stack_step(cfg, blocks, x1, gout), ref, label=f"fp32 d{d} f{f} sched{sched}")


@pytest.mark.parametrize("vocab,seq,batch", [(1003, 101, 3), (5003, 333, 3), (259, 37, 1)])
def test_f32_model_step_ragged_head(vocab, seq, batch):
    # odd vocabulary: dHf contracts over it (k-contiguous, a scalar tail in
    # every row) and dwte has it as its strided rows, with an odd token count
    cfg = Config(n_layer=2, d_model=200, n_head=3, head_dim=64, d_ff=328, vocab=vocab, seq_len=seq, batch=batch,
                 arch=ARCH_FAL, dtype=0)
    log(f"fp32 model step V={vocab} tokens={cfg.tokens}")
    g, blocks = synth.make_params(cfg, seed=92)
    tok = synth.make_tokens(cfg, seed=93, dist="zipf")
    compare_step(cfg, gpu_model_step(cfg, g, blocks, tok), oracle.train_step(cfg, g, blocks, tok),
                 label=f"fp32 V{vocab} T{seq}")
