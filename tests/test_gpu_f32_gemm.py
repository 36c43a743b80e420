"""The fp32 matrix-core GEMM through whole fp32 stack steps, at widths and
token counts where its launcher takes each of its tile shapes and K splits:

* 900 tokens, d 136, f 328: every product on 32 x 32 tiles, K not a multiple
  of the 128-wide slice, ragged tiles on both sides;
* 1200 tokens, d 328, f 840: 32 x 32, 128 x 64 (FFN up, GELU backward) and
  64 x 64 (FFN weight gradients, K split three ways);
* 2100 tokens, d 520, f 2056: 128 x 64, 64 x 64 and 128 x 128 (the FFN-up
  weight gradient), K splits of 1, 3, 5 and 7.

Widths are multiples of 8 that no tile divides.  Each step covers the four
operand orientations, the K-concatenated output projection and every
epilogue; the oracle is fp64 and the tolerance that of the other fp32 tests.
"""
import numpy as np
import pytest

import oracle
from paper_2510_14614_amd import synth
from paper_2510_14614_amd.config import ARCH_FAL, SCHED_SEQ, SCHED_STREAMS_MERGED, Config

from gpu_helpers import compare_step, gpu_stack_step, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sched", [SCHED_SEQ, SCHED_STREAMS_MERGED])
@pytest.mark.parametrize("d,heads,hd,f,batch", [(136, 2, 16, 328, 3), (328, 4, 16, 840, 4), (520, 8, 64, 2056, 7)])
def test_f32_stack_step_tile_shapes(d, heads, hd, f, batch, sched):
    cfg = Config(n_layer=2, d_model=d, n_head=heads, head_dim=hd, d_ff=f, vocab=0, seq_len=300, batch=batch,
                 arch=ARCH_FAL, dtype=0, has_embed_head=0, sched=sched)
    log(f"fp32 stack step d={d} f={f} tokens={cfg.tokens} sched={sched}")
    _, blocks = synth.make_params(cfg, seed=90)
    x1, gout = synth.make_stack_inputs(cfg, seed=91)
    ref = oracle.stack_step(cfg, blocks, x1, gout)
    ref["loss_scale"] = float(np.abs(gout * ref["y"]).sum())
    compare_step(cfg, gpu_stack_step(cfg, blocks, x1, gout), ref, label=f"fp32 d{d} f{f} sched{sched}")
