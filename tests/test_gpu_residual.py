"""GPU parity of the residual-stream entry point (countdown_ffn_residual):
h_out = h_in + y_prev, x = bf16(RMSNorm(h_out)), then the FFN on x. The
residual/normalisation step joins the layers of the stack workload; the FFN
part is checked against the oracle on the GPU's own x (teacher forcing), the
normalisation against the oracle's residual_rmsnorm."""
import numpy as np
import pytest

import oracle
from gpu_support import dev_bf16
from test_gpu_parity import Layer, calibrated, check_call, plan_for
from workloads import WORKLOADS, make_layer, make_predictor
from workloads.synth import bf16_to_f32, stream

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = 1e-5
X_SLACK = 1e-5  # relative: fp32 sum of squares and scaling against the fp64 oracle

VID = {"mono": 0, "dual_ideal": 1, "dual_pred": 2, "dense": 3, "cats": 4}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def residual_inputs(seed, B, d_model, with_y=True):
    rng = stream(9000 + seed, B, d_model)
    h = rng.standard_normal((B, d_model)).astype(np.float32)
    y = (0.5 * rng.standard_normal((B, d_model))).astype(np.float32) if with_y else None
    return h, y


def run_residual(plan, variant, layer, h_in, y_prev, thld):
    from paper_2505_17701_amd import binding as cd

    B, dm = h_in.shape
    hd = torch.from_numpy(h_in).cuda()
    yp = None if y_prev is None else torch.from_numpy(y_prev).cuda()
    h_out = torch.empty_like(hd)
    x_out = torch.empty((B, dm), dtype=torch.bfloat16, device="cuda")
    D = layer.d
    y = cd.countdown_ffn_residual(plan, VID[variant], hd, yp, h_out, x_out, D["W_gate"],
                                  D["W_up"], D["W_down"], thld, A_t=D.get("A_t"),
                                  B_t=D.get("B_t"), eps=EPS)
    idx, s_c, coef = cd.countdown_export_active(plan)
    x_bits = x_out.view(torch.int16).cpu().numpy().view(np.uint16)
    return (h_out.cpu().numpy(), x_bits,
            (y.cpu().numpy().astype(np.float64), idx.cpu().numpy(), s_c.cpu().numpy(),
             None if coef is None else coef.cpu().numpy()))


def check_norm(h_in, y_prev, h_gpu, x_bits, label):
    # h_out: one fp32 addition of two fp32 values, correctly rounded
    ref_h = h_in if y_prev is None else (h_in.astype(np.float64) + y_prev).astype(np.float32)
    np.testing.assert_array_equal(h_gpu.view(np.uint32), ref_h.view(np.uint32), err_msg=label)
    # x: within half a bf16 ulp of the exact normalised value (plus the fp32 slack)
    x = bf16_to_f32(x_bits).astype(np.float64)
    for b in range(h_in.shape[0]):
        _, r = oracle.residual_rmsnorm(h_in[b], None if y_prev is None else y_prev[b], eps=EPS)
        mag = np.maximum(np.abs(r), np.abs(x[b]))
        ulp = np.exp2(np.floor(np.log2(np.maximum(mag, 1e-30))) - 7)
        err = np.abs(x[b] - r)
        bad = err > 0.5 * ulp + X_SLACK * np.abs(r)
        assert not bad.any(), f"{label}: token {b}, {bad.sum()} x values off, worst {err.max():.3e}"


@pytest.mark.parametrize("variant", ["mono", "dual_ideal", "dual_pred", "dense"])
@pytest.mark.parametrize("shape", [(264, 520, 1), (1032, 1000, 3), (4096, 1376, 2), (2048, 776, 8)])
def test_residual_layer(variant, shape):
    dm, dff, B = shape
    L = make_layer(950 + dm, dm, dff, 0.03)
    P = make_predictor(950 + dm, dm, 64, dff, 0.05) if variant == "dual_pred" else None
    layer = Layer(L, P)
    h_in, y_prev = residual_inputs(dm + B, B, dm, with_y=(B != 2))
    # threshold: the variant's calibrated value on normalised inputs of the same recipe
    X = np.stack([oracle.residual_rmsnorm(h_in[b], None if y_prev is None else y_prev[b],
                                          eps=EPS)[1] for b in range(B)])
    Xb = np.array([np.float32(v) for v in X.ravel()], dtype=np.float32).reshape(X.shape)
    from workloads.synth import bf16_round
    thld = 0.0 if variant == "dense" else float(np.float32(oracle.calibrate(
        variant, bf16_round(Xb), 0.8, W_gate=L["W_gate"], W_up=L["W_up"],
        A_t=None if P is None else P["A_t"], B_t=None if P is None else P["B_t"])[0]))
    plan = plan_for(layer, max_batch=B)
    label = f"residual {variant} {shape}"
    h_gpu, x_bits, out = run_residual(plan, variant, layer, h_in, y_prev, thld)
    check_norm(h_in, y_prev, h_gpu, x_bits, label)
    check_call(variant, layer, x_bits, thld, out, label)


# The kernels that only residual layers run past 2 tokens: the token tiles of 4 and 8 (full and
# partly empty), every chunk count of columns (one, two, four, eight; sixteen at 4 tokens), every
# rank (the latent in LDS and the narrow weight tiles at 1024), CATS.
BATCHES = [
    ("cats", 264, 520, 3, 0), ("cats", 1032, 264, 8, 0), ("cats", 4096, 200, 5, 0),
    ("cats", 8192, 136, 4, 0), ("mono", 264, 520, 5, 0), ("mono", 520, 136, 8, 0),
    ("mono", 4096, 264, 8, 0), ("mono", 4096, 264, 4, 0), ("mono", 8192, 104, 3, 0),
    ("dual_ideal", 264, 520, 8, 0), ("dual_ideal", 520, 136, 4, 0), ("dual_ideal", 4096, 136, 7, 0),
    ("dual_ideal", 8192, 104, 4, 0), ("dense", 264, 136, 4, 0), ("dense", 4096, 136, 8, 0),
    ("dense", 8192, 104, 3, 0),
    ("dual_pred", 264, 520, 3, 8), ("dual_pred", 264, 520, 8, 16), ("dual_pred", 1032, 264, 5, 32),
    ("dual_pred", 520, 264, 6, 64), ("dual_pred", 2048, 264, 4, 128), ("dual_pred", 4096, 264, 8, 256),
    ("dual_pred", 4096, 264, 3, 512), ("dual_pred", 1032, 264, 8, 512), ("dual_pred", 264, 264, 4, 1024),
    ("dual_pred", 520, 264, 8, 1024), ("dual_pred", 2056, 136, 8, 1024), ("dual_pred", 4096, 136, 5, 1024),
    ("dual_pred", 8192, 136, 3, 8), ("dual_pred", 8192, 136, 4, 1024),
]


@pytest.mark.parametrize("variant,dm,dff,B,rank", BATCHES)
def test_residual_layer_batches(variant, dm, dff, B, rank):
    from workloads.synth import bf16_round

    L = make_layer(960 + rank, dm, dff, 0.03)
    P = make_predictor(960 + rank, dm, rank, dff, 0.05) if rank else None
    layer = Layer(L, P)
    h_in, y_prev = residual_inputs(dm + B + rank, B, dm)
    X = np.stack([oracle.residual_rmsnorm(h_in[b], y_prev[b], eps=EPS)[1] for b in range(B)])
    X = bf16_round(np.array(X, dtype=np.float32))
    plan = plan_for(layer, max_batch=B)
    for k in (0.8, 0.3):  # few active neurons (of a batch) and most
        thld = 0.0 if variant == "dense" else float(np.float32(oracle.calibrate(
            variant, X, k, W_gate=L["W_gate"], W_up=L["W_up"], A_t=None if P is None else P["A_t"],
            B_t=None if P is None else P["B_t"])[0]))
        label = f"residual {variant} {dm}x{dff} B{B} rank {rank} k {k}"
        h_gpu, x_bits, out = run_residual(plan, variant, layer, h_in, y_prev, thld)
        check_norm(h_in, y_prev, h_gpu, x_bits, label)
        check_call(variant, layer, x_bits, thld, out, label)
    plan.close()


def test_residual_rejects_overlap():
    from paper_2505_17701_amd import binding as cd

    layer = Layer(make_layer(977, 264, 520, 0.03))
    plan = plan_for(layer, max_batch=2)
    D = layer.d
    h = torch.zeros((2, 264), dtype=torch.float32, device="cuda")
    x = torch.empty((2, 264), dtype=torch.bfloat16, device="cuda")
    y = torch.empty_like(h)
    with pytest.raises(cd.CountdownError):  # h_out aliasing h_in
        cd.countdown_ffn_residual(plan, 0, h, None, h, x, D["W_gate"], D["W_up"], D["W_down"],
                                  1.0, y=y)
    with pytest.raises(cd.CountdownError):  # eps NaN
        cd.countdown_ffn_residual(plan, 0, h, None, torch.empty_like(h), x, D["W_gate"],
                                  D["W_up"], D["W_down"], 1.0, eps=float("nan"), y=y)
    # y_prev may be y itself
    h2 = torch.empty_like(h)
    y.zero_()
    cd.countdown_ffn_residual(plan, 0, h, y, h2, x, D["W_gate"], D["W_up"], D["W_down"], 1.0,
                              y=y)
    torch.cuda.synchronize()


def test_stack_teacher_forced():
    """All 32 layers of the stack workload (7B-shaped predictor layers, the
    residual stream between them) run back to back on the GPU at batch 1. Every
    layer is checked against the oracle on the inputs the GPU layer received
    (teacher forcing), with its threshold calibrated by the oracle at k = 0.9 on
    8 calibration tokens propagated through the oracle's dense stack. Reported,
    not gated: the end-to-end divergence of the residual stream between the GPU
    stack and the oracle's own sparse stack (free running: a neuron whose score
    lies within rounding of the threshold can be selected by one side only, and
    with random layers such a difference grows from layer to layer), and between
    the oracle's sparse and dense stacks (a random predictor's index set is not
    the one the exact coefficients would pick). The GPU plan reduces y in a fixed
    order, so the report repeats from run to run."""
    from workloads.synth import T_CALIB, bf16_round

    w = WORKLOADS["stack32_llama7b_pred"]
    k, ncal = 0.9, 8

    def norm_bits(h, y):
        """The layer input: residual add, RMSNorm (fp64), rounded to bf16 via fp32."""
        hs, xs = [], []
        for b in range(h.shape[0]):
            ho, r = oracle.residual_rmsnorm(h[b], None if y is None else y[b], eps=EPS)
            hs.append(ho)
            xs.append(r.astype(np.float32))
        return np.stack(hs), bf16_round(np.stack(xs))

    h_cal = stream(9200, T_CALIB, w.d_model).standard_normal((ncal, w.d_model))
    h0 = stream(9100, w.d_model).standard_normal((1, w.d_model)).astype(np.float32)
    y_cal = None
    h, y_prev = h0, None                 # the GPU stack (fp32 residual stream)
    h_os, y_os = h0.astype(np.float64), None  # the oracle's sparse stack, free running
    h_od, y_od = h0.astype(np.float64), None  # the oracle's dense stack
    plan = None
    worst = 0.0
    growth = {}

    def rel_l2(a, b):
        return float(np.linalg.norm(a - b) / np.linalg.norm(b))

    for l in range(w.n_layers):
        L = w.layer(layer=l)
        P = w.predictor(layer=l)
        h_cal, x_cal = norm_bits(h_cal, y_cal)
        y_cal = oracle.dense(x_cal, L["W_gate"], L["W_up"], L["W_down"])
        thld = float(np.float32(oracle.calibrate("dual_pred", x_cal, k, A_t=P["A_t"],
                                                 B_t=P["B_t"])[0]))
        layer = Layer(L, P)
        if plan is None:  # fixed-order y: the reported divergence is reproducible
            from paper_2505_17701_amd import binding as cd

            plan = cd.Plan(w.d_model, w.d_ff, max_batch=1, d_rank=w.d_rank, keep_coef=True,
                           deterministic=True)
        label = f"stack layer {l}"
        h_gpu, x_bits, out = run_residual(plan, "dual_pred", layer, h, y_prev, thld)
        check_norm(h, y_prev, h_gpu, x_bits, label)
        n, flips, rel = check_call("dual_pred", layer, x_bits, thld, out, label)
        worst = max(worst, rel)
        print(f"{label}: thld={thld:.4f} n={n} flips={flips} rel={rel:.2e}", flush=True)
        h, y_prev = h_gpu, out[0].astype(np.float32)
        h_os, x_os = norm_bits(h_os, y_os)
        _, y_os, _ = oracle.ffn_dual_pred(x_os, L["W_gate"], L["W_up"], L["W_down"], P["A_t"],
                                          P["B_t"], thld)
        h_od, x_od = norm_bits(h_od, y_od)
        y_od = oracle.dense(x_od, L["W_gate"], L["W_up"], L["W_down"])
        if l + 1 in (1, 2, 4, 8, 16, 32):
            g_os = rel_l2(h.astype(np.float64) + y_prev, h_os + y_os)
            growth[l + 1] = (g_os, rel_l2(h_os + y_os, h_od + y_od), int(np.sum(
                np.isin(out[1], oracle.ffn_dual_pred(x_os, L["W_gate"], L["W_up"], L["W_down"],
                                                      P["A_t"], P["B_t"], thld)[0],
                        invert=True))))
        del layer
        torch.cuda.empty_cache()
    plan.close()
    fin_gpu = h.astype(np.float64) + y_prev
    fin_os, fin_od = h_os + y_os, h_od + y_od
    assert np.all(np.isfinite(fin_gpu))
    for d, (g_os, g_od, nd) in growth.items():
        print(f"after {d} layers: GPU vs oracle sparse {g_os:.3e} (IDX of that layer: {nd} "
              f"neurons the free-running oracle does not select); oracle sparse vs dense "
              f"{g_od:.3e}", flush=True)
    print(f"stack end to end (final h, relative l2): GPU vs oracle sparse stack "
          f"{rel_l2(fin_gpu, fin_os):.3e}; oracle sparse vs oracle dense stack "
          f"{rel_l2(fin_os, fin_od):.3e}; GPU vs oracle dense stack "
          f"{rel_l2(fin_gpu, fin_od):.3e}; worst per-layer y error {worst:.2e}", flush=True)
