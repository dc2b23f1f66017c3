"""The score-only kernels of the predictors at 1-2 tokens (a threshold of +inf gathers nothing):
the same scores, bit for bit, as the kernels that gather, no active neuron and y = 0. Every
rank, token widths of every chunk count, neuron counts off the 32-neuron blocks."""
import numpy as np
import pytest

from gpu_support import dev_bf16
from workloads import make_layer, make_predictor, make_ternary, make_tokens

pytestmark = pytest.mark.gpu

CASES = [("dual_pred", 264, 8, 1, 8), ("dual_pred", 520, 40, 2, 16), ("dual_pred", 8, 72, 1, 32),
         ("dual_pred", 1032, 136, 2, 64), ("dual_pred", 2056, 200, 1, 128),
         ("dual_pred", 4096, 264, 2, 256), ("dual_pred", 264, 1000, 1, 512),
         ("dual_pred", 520, 104, 2, 1024), ("dual_pred", 8192, 104, 1, 1024),
         ("dual_tern", 8, 8, 1, 0), ("dual_tern", 520, 40, 1, 0), ("dual_tern", 2048, 72, 1, 0),
         ("dual_tern", 4096, 1000, 1, 0), ("dual_tern", 8192, 136, 1, 0)]


@pytest.mark.parametrize("variant,dm,dff,B,rank", CASES)
def test_scores_alone(variant, dm, dff, B, rank):
    import torch
    from paper_2505_17701_amd import binding as cd

    D = {n: dev_bf16(v) for n, v in make_layer(920, dm, dff, 0.05).items()}
    x = dev_bf16(make_tokens(920, B, dm))
    plan = cd.Plan(dm, dff, max_batch=B, d_rank=rank, keep_coef=True)
    if rank:
        P = {n: dev_bf16(v) for n, v in make_predictor(920, dm, rank, dff, 0.05).items()}
    else:
        packed = torch.from_numpy(
            cd.countdown_ternary_pack(make_ternary(920, dm, dff)).view(np.int32)).cuda()

    def call(thld):
        mats = (D["W_gate"], D["W_up"], D["W_down"])
        y = torch.full((B, dm), float("nan"), device="cuda")
        if rank:
            cd.countdown_ffn_dual(plan, x, *mats, thld, A_t=P["A_t"], B_t=P["B_t"], y=y)
        else:
            cd.countdown_ffn_tern(plan, x, *mats, packed, thld, y=y)
        idx, _, coef = cd.countdown_export_active(plan)
        return y, idx, coef.clone()

    _, idx_all, gathered = call(-float("inf"))
    assert len(idx_all) == dff
    y, idx, scores = call(float("inf"))
    assert len(idx) == 0 and not y.any()
    assert torch.equal(scores, gathered)
    if rank and B == 2:  # a plan for two tokens, one in use
        x = x[:1].contiguous()
        B = 1
        assert torch.equal(call(float("inf"))[2][0], gathered[0])
    plan.close()
