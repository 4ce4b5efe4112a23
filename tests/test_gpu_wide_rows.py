"""Wide layers (separate normalisations) of few rows in one launch: parity at the edges of its tiles, where it ends, and with repeated calls."""
import pytest

from paper_2511_13587_amd import synth
from test_gpu_parity import gc, run_bf16_case, show  # noqa: F401

pytestmark = pytest.mark.gpu


# d 1536: 2 rows; 12 and 24 heads (head size 128, 64); 32, 34 and 64 rows, one row-block to a tile; 66, 98 and 128 rows, two; 130 rows, a launch per projection;
# d_ff no multiple of 48 and no whole share of 32 (4160 / 32 = 130); more pairs than CUs, so that rows share an attention unit.  d 2304: two from 34 rows on, up to 64
@pytest.mark.parametrize("d,heads,d_ff,prompts,tokens,n_forced", [
    (1536, 12, 4096, 1, 2, 9), (1536, 24, 4096, 1, 16, 40), (1536, 12, 4096, 1, 17, 70), (1536, 12, 4096, 1, 32, 33), (1536, 24, 4160, 2, 16, 31), (1536, 24, 4096, 8, 4, 20),
    (1536, 12, 4096, 16, 2, 20), (1536, 24, 4096, 3, 11, 20), (1536, 12, 4160, 7, 7, 20), (1536, 24, 4096, 4, 16, 20), (1536, 12, 4096, 13, 5, 9), (2304, 18, 2304, 1, 17, 20),
    (2304, 36, 2368, 2, 11, 20), (2304, 18, 2304, 4, 8, 20), (2304, 18, 2304, 3, 11, 20)])
def test_wide_layers_in_one_launch(gc, d, heads, d_ff, prompts, tokens, n_forced):  # noqa: F811
    shape = synth.SEVEN_B.replace(d_model=d, n_heads=heads, d_ff=d_ff, n_layers=2, vocab=1024, logit_lo=0, logit_hi=1024, prefix_len=8, n_prompts=prompts,
                                  n_nodes=tokens - 1, tree_widths=None)
    sample = {"sample": [0, prompts - 1]} if prompts > 4 else {}
    show(f"d {d} heads {heads} d_ff {d_ff} {prompts} x {tokens}", run_bf16_case(gc, shape, n_forced=n_forced, calls=2, **sample))
