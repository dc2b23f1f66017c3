"""Calibration as a matrix product: tile edges in tokens, neurons and columns, every
variant, against the oracle; chunks of tokens; infinite and NaN coefficients."""
import math

import numpy as np
import pytest

import oracle
from gpu_support import dev_bf16
from workloads import make_layer, make_predictor, make_ternary, make_tokens
from workloads.synth import T_CALIB

pytestmark = pytest.mark.gpu

RTOL = 2e-5  # of the quantiles at k 0.9: an fp32 dot product's error, as in the parity tests


def _calibrate(cd, plan, variant, X, k, D):
    if variant == "dual_tern":
        return cd.countdown_calibrate_tern(plan, X, D["Tp"], k)
    v = {"mono": cd.CD_VARIANT_MONO, "dual_ideal": cd.CD_VARIANT_DUAL_IDEAL,
         "dual_pred": cd.CD_VARIANT_DUAL_PRED, "cats": cd.CD_VARIANT_CATS}[variant]
    need = {"mono": ("W_up",), "cats": ("W_gate",), "dual_ideal": ("W_gate", "W_up"),
            "dual_pred": ("A_t", "B_t")}[variant]
    return cd.countdown_calibrate(plan, v, X, k, **{n: D[n] for n in need})


# tokens around the 32 / 64 token tiles and the 256-token chunk; columns around the 64-
# and 128-column tiles and past 2048 (the longer chains); d_ff around the 32 / 64 tiles
CASES = [
    ("mono", 2, 8, 8, 0), ("mono", 31, 72, 40, 0), ("mono", 33, 136, 72, 0),
    ("mono", 257, 264, 136, 0), ("mono", 65, 2056, 128, 0), ("mono", 32, 4096, 688, 0),
    ("cats", 64, 200, 64, 0), ("cats", 17, 520, 1000, 0),
    ("dual_ideal", 32, 64, 96, 0), ("dual_ideal", 100, 1032, 200, 0),
    ("dual_pred", 20, 512, 200, 8), ("dual_pred", 65, 264, 136, 64),
    ("dual_pred", 300, 1544, 264, 256), ("dual_pred", 33, 136, 72, 1024),
    ("dual_tern", 31, 256, 136, 0), ("dual_tern", 70, 1544, 200, 0),
    ("dual_tern", 33, 8192, 64, 0),
    # two batches of the plan's one token past 4096 columns: the decode kernels; three: the product
    ("mono", 2, 4104, 40, 0), ("dual_ideal", 2, 8192, 40, 0), ("dual_tern", 2, 4104, 72, 0),
    ("cats", 3, 4104, 40, 0), ("dual_tern", 3, 8192, 72, 0), ("mono", 2, 4104, 2056, 0),
    ("dual_pred", 2, 264, 72, 512), ("dual_pred", 3, 136, 72, 1024),
]


@pytest.mark.parametrize("variant,T,dm,dff,rank", CASES)
def test_calibration_tiles(variant, T, dm, dff, rank):
    import torch
    from paper_2505_17701_amd import binding as cd

    wid = 870 + len(variant)
    L = make_layer(wid, dm, dff, 0.02)
    P = make_predictor(wid, dm, rank, dff, 0.05) if rank else {}
    theta = make_ternary(wid, dm, dff) if variant == "dual_tern" else None
    X = make_tokens(wid, T, dm, purpose=T_CALIB)
    t_o, q_o = oracle.calibrate(variant, X, 0.9, W_gate=L["W_gate"], W_up=L["W_up"],
                                A_t=P.get("A_t"), B_t=P.get("B_t"), theta_t=theta)
    D = {n: dev_bf16(v) for n, v in {**L, **P}.items()}
    if theta is not None:
        D["Tp"] = torch.from_numpy(cd.countdown_ternary_pack(theta).view(np.int32)).to("cuda")
    plan = cd.Plan(dm, dff, 1, rank)
    for _ in range(2):  # the second call finds the plan's workspace in place
        thld, q = _calibrate(cd, plan, variant, dev_bf16(X), 0.9, D)
        q = q.cpu().numpy()
        # a quantile near zero carries the coefficients' absolute error
        np.testing.assert_allclose(q, q_o, rtol=RTOL, atol=RTOL * float(np.abs(q_o).max()))
        assert abs(float(thld.item()) - t_o) <= RTOL * float(np.abs(q_o).max())
        assert float(thld.item()) == float(np.float32(sum(q.tolist()) / T))  # in order, fp64
    # a decode-sized plan takes the decode kernels up to its batch: the same tokens
    small = cd.Plan(dm, dff, 2, rank)
    _, q2 = _calibrate(cd, small, variant, dev_bf16(X[:2]), 0.9, D)
    np.testing.assert_allclose(q2.cpu().numpy(), q[:2], rtol=RTOL,
                               atol=RTOL * float(np.abs(q_o).max()))


@pytest.mark.parametrize("variant", ["mono", "dual_pred"])
def test_calibration_keeps_infinities_and_nan(variant):
    """One infinite weight and one NaN weight: their neurons' coefficients, and no others,
    are infinite and NaN, as in the decode kernels (the compensated sums must not turn an
    infinite sum into NaN)."""
    import torch
    from paper_2505_17701_amd import binding as cd

    dm, dff, rank, T = 512, 136, 64, 40
    L = make_layer(880, dm, dff, 0.02)
    P = make_predictor(880, dm, rank, dff, 0.05)
    D = {n: dev_bf16(v) for n, v in {**L, **P}.items()}
    X = dev_bf16(make_tokens(880, T, dm, purpose=T_CALIB))
    W = D["W_up"] if variant == "mono" else D["B_t"]
    W[5, 3] = math.inf
    plan1 = cd.Plan(dm, dff, 1, rank)
    for k in (0.5, 0.9999):  # 0.9999: between the two largest, infinite where the product is
        _, q = _calibrate(cd, plan1, variant, X, k, D)
        ref = torch.cat([_calibrate(cd, plan1, variant, X[t:t + 1], k, D)[1] for t in range(T)])
        assert torch.equal(torch.isinf(q), torch.isinf(ref))
        assert not torch.isnan(q).any() and (k < 0.9 or torch.isinf(q).any())
        f = torch.isfinite(ref)
        if f.any():
            torch.testing.assert_close(q[f], ref[f], rtol=RTOL,
                                       atol=RTOL * float(ref[f].abs().max()))
    W[5, 3] = math.nan
    _, q = _calibrate(cd, plan1, variant, X, 0.5, D)
    assert torch.isfinite(q).all()  # one NaN neuron among 136 does not reach the median
