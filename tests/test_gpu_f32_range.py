"""fp32 expert products at the ends of the fp32 range, where the sums of bf16 parts give way to the fp32 instruction."""
import pytest
import torch

import paper_2504_19925_amd as symi
from tests.test_gpu_f32_split import layer, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [1.0, 2.0 ** 41, float("inf")])
def test_active_leaves_classes_without_rows(value):
    """Some seven tiles to a workgroup, those of the classes without rows behind the others: none of them is written, whatever
    the values of the others are."""
    rows = [64] * 24 + [0] * 40
    s = layer(rows, list(range(65)), 264, 520, seed=5)
    run(s)
    s["Xp"][7::64, 5] = value
    s["dYp"][9::64, 3] = value
    s["dW1"].fill_(7.0)
    s["dW2"].fill_(7.0)
    symi.symi_expert_bwd_active(s["ctx"], s["dYp"], s["Xp"], s["UV"], s["H"], s["off"], s["first"], s["W1"], s["W2"], s["dXp"],
                                s["dW1"], s["dW2"], s["ws"])
    for e in range(64):
        kept = bool((s["dW1"][e] == 7.0).all()) and bool((s["dW2"][e] == 7.0).all())
        assert kept == (e >= 24), e
