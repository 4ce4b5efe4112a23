"""GPU parity of verify calls whose q/k/v projection and attention are launches of their own at head size 64: few (head, prompt)
pairs, with the projection on 32 x 32 tiles and attention workgroups that read ahead, and more pairs than CUs."""
import pytest

from paper_2511_13587_amd import synth
from test_gpu_parity import gc, run_bf16_case, show  # noqa: F401

pytestmark = pytest.mark.gpu


# 20 pairs: 14, 54, 64, 66 and 122 rows (one row-block, two, the last with every tile on a CU, one more); 40 pairs and 64 rows; 264 pairs
@pytest.mark.parametrize("model,prompts,n_nodes,widths,n_forced", [("xl", 1, 6, None, 33), ("xl", 1, 26, (4, 6, 6, 5, 5), 45), ("xl", 1, 31, (4, 6, 8, 8, 5), 20),
                                                                  ("xl", 1, 32, (4, 6, 8, 8, 6), 20), ("xl", 1, 60, (8, 12, 12, 10, 10, 8), 31),
                                                                  ("xl", 2, 15, (4, 5, 6), 40), ("b", 22, 5, None, 9)])
def test_projection_and_attention_apart(gc, model, prompts, n_nodes, widths, n_forced):  # noqa: F811
    base = synth.XL_TREE if model == "xl" else synth.B_SHAPE
    shape = base.replace(n_layers=2, n_prompts=prompts, n_nodes=n_nodes, tree_widths=widths)
    sample = [0, prompts - 1] if prompts > 8 else None
    show(f"{model} {prompts} x {n_nodes + 1}", run_bf16_case(gc, shape, n_forced=n_forced, calls=2, **({"sample": sample} if sample else {})))
