"""The MFMA kernels of batches of 3-8 tokens (the ternary predictor: 2-8) at the edges of
their tiling, against the oracle: the columns a wave owns (128-column steps, pairs and odd
steps, 512-column units of the packed ternary weights), row quads over the workgroups (one
quad each, an uneven share, whole and partial blocks, more than one generation), batches
that fill, overflow and leave empty the token quads, every rank."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import Layer, compare, plan_for
from test_gpu_topk import check_topk
from workloads import make_layer, make_predictor, make_ternary, make_tokens

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (variant, d_model, d_ff, B, rank)
CASES = [
    # columns: S = 1 (even one chunk), 2, 3, 4, 6, 8 steps a wave, and their ragged ends
    ("mono", 8, 64, 3, 0), ("mono", 128, 40, 8, 0), ("mono", 1016, 72, 5, 0),
    ("mono", 1032, 136, 8, 0), ("cats", 2048, 64, 4, 0), ("mono", 2056, 72, 3, 0),
    ("mono", 3064, 72, 8, 0), ("cats", 3080, 72, 6, 0), ("mono", 4096, 136, 8, 0),
    ("mono", 4104, 72, 4, 0), ("mono", 6144, 40, 3, 0), ("cats", 6152, 40, 4, 0),
    ("mono", 8192, 72, 4, 0),
    ("dual_ideal", 8, 8, 8, 0), ("dual_ideal", 1400, 264, 7, 0), ("dual_ideal", 4096, 72, 5, 0),
    ("dual_ideal", 5000, 72, 3, 0), ("dual_ideal", 8192, 40, 4, 0),
    # ternary: one unit, two, four, eight, sixteen
    ("dual_tern", 8, 64, 2, 0), ("dual_tern", 504, 72, 8, 0), ("dual_tern", 520, 72, 3, 0),
    ("dual_tern", 1024, 40, 2, 0), ("dual_tern", 1032, 72, 5, 0), ("dual_tern", 2048, 72, 4, 0),
    ("dual_tern", 2056, 72, 8, 0), ("dual_tern", 4096, 72, 2, 0), ("dual_tern", 4104, 72, 3, 0),
    ("dual_tern", 8192, 72, 2, 0),
    # low-rank predictor: ranks by one to eight loads a wave, the latent in LDS at 1024
    ("dual_pred", 264, 136, 3, 8), ("dual_pred", 264, 136, 8, 32), ("dual_pred", 1032, 136, 4, 128),
    ("dual_pred", 2048, 72, 8, 512), ("dual_pred", 520, 136, 3, 1024), ("dual_pred", 520, 136, 8, 1024),
    ("dual_pred", 8192, 72, 4, 64),
    # rows: one quad a workgroup (up to 1024 neurons), 256 workgroups of 1-2 quads, 512 of
    # 1-2, of 8, and the first size with two generations
    ("mono", 64, 1016, 3, 0), ("mono", 64, 1032, 8, 0), ("dual_pred", 64, 2056, 4, 16),
    ("dual_ideal", 64, 2048, 3, 0), ("mono", 64, 16384, 5, 0), ("dual_tern", 64, 16392, 4, 0),
    # one workgroup per CU up to three quads each, or eight with the latent in LDS; two past it
    ("mono", 64, 3072, 5, 0), ("mono", 64, 3080, 8, 0), ("dual_pred", 64, 8192, 4, 1024),
    ("dual_pred", 64, 8200, 8, 1024),
    # the kernels of 1-2 tokens with a tile of 4 or 8 on one side of the lines of small layers,
    # the batch kernels (one or two steps a wave at 3-4 tokens) on the other
    ("mono", 1024, 7168, 3, 0), ("mono", 1024, 7176, 4, 0), ("cats", 8, 7176, 3, 0),
    ("cats", 2048, 3072, 4, 0), ("mono", 2048, 3080, 3, 0), ("dual_ideal", 512, 7168, 4, 0),
    ("dual_ideal", 512, 7176, 3, 0), ("dual_ideal", 1024, 3080, 4, 0), ("mono", 2056, 40, 4, 0),
    ("dual_pred", 512, 3080, 8, 256), ("dual_pred", 520, 3080, 5, 8), ("dual_pred", 8, 3080, 5, 16),
]


def _layer(variant, dm, dff, rank, wid):
    P = make_predictor(wid, dm, rank, dff, 0.05) if rank else None
    T = make_ternary(wid, dm, dff) if variant == "dual_tern" else None
    return Layer(make_layer(wid, dm, dff, 0.05), P, T), P, T


def _coefficients(variant, layer, P, T, x):
    if variant == "dual_pred":
        return oracle.predictor(x, P["A_t"], P["B_t"])[1]
    if variant == "dual_tern":
        return oracle.ternary_predictor(x, T)
    u, g, s = oracle.coefficients(x, layer.h["W_gate"], layer.h["W_up"])
    return np.abs({"mono": u, "dual_ideal": s, "cats": g / (1.0 + np.exp(-g))}[variant])


@pytest.mark.parametrize("variant,dm,dff,B,rank", CASES)
def test_batch_kernel_edges(variant, dm, dff, B, rank):
    layer, P, T = _layer(variant, dm, dff, rank, 910)
    x = make_tokens(910, B, dm)
    c = _coefficients(variant, layer, P, T, x)
    plan = plan_for(layer, max_batch=B)
    # few active neurons, about half, none and all
    for thld in (float(np.float32(np.quantile(c, 0.95))), float(np.float32(np.quantile(c, 0.4))),
                 np.inf, -np.inf):
        compare(plan, variant, layer, x, thld, f"{variant} {dm}x{dff} B{B} thld {thld}")
    plan.close()
    check_topk(variant, layer, x, 0.8, f"{variant} {dm}x{dff} B{B} per token")


@pytest.mark.parametrize("B", [3, 8])
def test_batch_kernels_keep_tokens_and_neurons_apart(B):
    """Infinite and NaN weights stay in their neuron and a NaN token in its own row of y:
    neither leaks through the matrix instructions' empty columns or shared registers."""
    from paper_2505_17701_amd import binding as cd

    dm, dff = 264, 136
    layer, _, _ = _layer("mono", dm, dff, 0, 911)
    D = layer.d
    x = torch.from_numpy(make_tokens(911, B, dm).view(np.int16)).view(torch.bfloat16).cuda()
    plan = cd.Plan(dm, dff, max_batch=B, keep_coef=True)
    W = D["W_up"].clone()
    W[5, 3], W[77, 200] = float("inf"), float("nan")
    cd.countdown_ffn_mono(plan, x, D["W_gate"], D["W_up"], D["W_down"], 0.5)
    ref = cd.countdown_export_active(plan)[2].clone()
    cd.countdown_ffn_mono(plan, x, D["W_gate"], W, D["W_down"], 0.5)
    got = cd.countdown_export_active(plan)[2]
    same = torch.ones(dff, dtype=torch.bool, device="cuda")
    same[5] = same[77] = False
    assert torch.equal(got[:, same], ref[:, same])
    assert torch.isinf(got[:, 5]).all() and torch.isnan(got[:, 77]).all()
    # a NaN token: its own coefficients only
    x2 = x.clone()
    x2[1, 7] = float("nan")
    y = cd.countdown_ffn_dense(plan, x2, D["W_gate"], D["W_up"], D["W_down"])
    bad = torch.isnan(y).any(dim=1)
    assert bad[1] and int(bad.sum()) == 1
    plan.close()
