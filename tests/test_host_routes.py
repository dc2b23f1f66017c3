"""Which kernels a call launches, and with how many workgroups, at the edges of the dispatch
rules: read off the library's host code, without a GPU."""
import pytest

import host_hip


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    return host_hip.Host(host_hip.build(str(tmp_path_factory.mktemp("host"))))


def ffn_launches(host, variant, d_model, d_ff, B, rank=0, thld=1.0):
    st, h = host.plan(d_model, d_ff, B, rank)
    assert st == host.cd.CD_OK
    host.launches()
    assert host.ffn(h, variant, B, thld) == host.cd.CD_OK
    out = host.launches()
    host.lib.countdown_plan_destroy(h)
    return out


@pytest.mark.parametrize("variant,d_model,d_ff,B,rank,grid", [
    ("mono", 4096, 8, 3, 0, 2), ("mono", 4096, 1016, 3, 0, 254), ("dense", 4096, 1032, 8, 0, 256),
    # one workgroup per CU up to three quads of neurons, two past that, then whole multiples
    ("mono", 4096, 2048, 8, 0, 256), ("dual_ideal", 4096, 3072, 4, 0, 256),
    ("mono", 4096, 3080, 8, 0, 512), ("dual_pred", 4096, 3080, 8, 512, 512),
    ("dual_tern", 4096, 16384, 3, 0, 512), ("dual_pred", 4096, 16392, 8, 64, 1024),
    # the latents of rank 1024 lie in LDS: one workgroup per CU as far as it reaches
    ("dual_pred", 4096, 2048, 8, 1024, 256), ("dual_pred", 1024, 8192, 4, 1024, 256),
    ("dual_pred", 1024, 8200, 8, 1024, 512),
])
def test_batch_grid(host, variant, d_model, d_ff, B, rank, grid):
    got = [n for k, n in ffn_launches(host, variant, d_model, d_ff, B, rank)
           if k.startswith("k_batch_")]
    assert got == [grid]
    assert grid <= d_ff // 4  # a quad of neurons per workgroup at least
    shares = min(grid, 256)   # and eight at most, as k_batch_* spread them
    for share in range(shares):
        lo, hi = d_ff // 4 * share // shares, d_ff // 4 * (share + 1) // shares
        assert -(-(hi - lo) // (grid // shares)) <= 8


MFMA, ROWS = "batch", "rows"


@pytest.mark.parametrize("variant,d_model,d_ff,B,rank,kind", [
    # few neurons at 3-4 tokens: one row a neuron up to 1024 / 2048 columns, two rows half that
    ("mono", 8, 7168, 3, 0, ROWS), ("mono", 1024, 7168, 4, 0, ROWS), ("mono", 1024, 7176, 3, 0, MFMA),
    ("cats", 1032, 3072, 4, 0, ROWS), ("cats", 2048, 3080, 4, 0, MFMA), ("mono", 2056, 8, 3, 0, MFMA),
    ("mono", 512, 3072, 5, 0, MFMA), ("cats", 8, 8, 8, 0, MFMA),
    ("dense", 512, 7168, 4, 0, ROWS), ("dense", 520, 7168, 3, 0, MFMA), ("dense", 1024, 3072, 4, 0, ROWS),
    ("dense", 1032, 8, 4, 0, MFMA), ("dual_ideal", 1024, 3080, 3, 0, MFMA),
    ("dual_ideal", 512, 7168, 3, 0, ROWS), ("dense", 512, 688, 5, 0, MFMA),
    # one chunk of columns, many neurons, a short rank at 5-8 tokens
    ("dual_pred", 512, 3080, 5, 256, ROWS), ("dual_pred", 512, 3072, 8, 64, MFMA),
    ("dual_pred", 520, 28672, 8, 64, MFMA), ("dual_pred", 512, 28672, 8, 512, MFMA),
    ("dual_pred", 512, 28672, 4, 64, MFMA), ("dual_pred", 8, 28672, 8, 8, ROWS),
    # the ternary predictor: 2 tokens up to 4096 columns, 3 and more always
    ("dual_tern", 4096, 688, 2, 0, MFMA), ("dual_tern", 4104, 688, 2, 0, ROWS),
    ("dual_tern", 64, 688, 3, 0, MFMA), ("dual_tern", 64, 688, 1, 0, ROWS),
    ("mono", 4096, 14336, 2, 0, ROWS),
])
def test_coefficient_kernel(host, variant, d_model, d_ff, B, rank, kind):
    coef = [k for k, _ in ffn_launches(host, variant, d_model, d_ff, B, rank)
            if k.startswith(("k_batch_", "k_coef_"))]
    assert len(coef) == 1
    assert coef[0].startswith("k_batch_" if kind == MFMA else "k_coef_"), coef


@pytest.mark.parametrize("variant,d_model,B,rank,kernel", [
    ("dual_pred", 1024, 1, 8, "k_score_pred<1,0>"), ("dual_pred", 8192, 2, 1024, "k_score_pred<2,7>"),
    ("dual_tern", 256, 1, 0, "k_score_tern<1>"), ("dual_tern", 8192, 1, 0, "k_score_tern<16>"),
])
def test_predictor_scores_alone(host, variant, d_model, B, rank, kernel):
    """A threshold of +inf, and the first pass of per-token thresholds, gather nothing."""
    def coef(launches):
        return [k for k, _ in launches if k.startswith(("k_batch_", "k_coef_", "k_score_"))]

    assert coef(ffn_launches(host, variant, d_model, 1000, B, rank, float("inf"))) == [kernel]
    assert coef(ffn_launches(host, variant, d_model, 1000, B, rank, 3e38))[0].startswith("k_coef_")
    st, h = host.plan(d_model, 1000, B, rank)
    assert st == host.cd.CD_OK
    host.launches()
    assert host.ffn_topk(h, variant, B) == host.cd.CD_OK
    assert coef(host.launches()) == [kernel]
    host.lib.countdown_plan_destroy(h)


@pytest.mark.parametrize("variant,d_model,d_ff,mb,T,rank,batches", [
    ("mono", 4096, 11008, 1, 1, 0, 1), ("dual_pred", 256, 688, 8, 8, 64, 1),
    ("mono", 4096, 688, 1, 2, 0, 0), ("cats", 4104, 2048, 4, 8, 0, 2), ("mono", 8192, 688, 4, 5, 0, 2),
    ("mono", 8192, 2056, 1, 2, 0, 0), ("mono", 8192, 688, 4, 9, 0, 0),
    ("dual_tern", 4104, 28672, 2, 4, 0, 2), ("dual_tern", 8192, 688, 1, 3, 0, 0),
    ("dual_tern", 6144, 11008, 2, 4, 0, 0), ("dual_tern", 6152, 11008, 2, 4, 0, 2),
    ("dual_tern", 6144, 4096, 1, 2, 0, 2), ("dual_tern", 6144, 16392, 1, 2, 0, 2),
    ("dual_pred", 8192, 688, 1, 2, 256, 0), ("dual_pred", 256, 688, 1, 2, 512, 2),
    ("dual_pred", 256, 688, 2, 4, 1024, 2), ("dual_pred", 256, 688, 4, 5, 1024, 0),
])
def test_calibration_route(host, variant, d_model, d_ff, mb, T, rank, batches):
    """Decode-sized batches (their number), or 0: one matrix product."""
    st, h = host.plan(d_model, d_ff, mb, rank)
    assert st == host.cd.CD_OK
    host.launches()
    assert host.calibrate(h, variant, T) == host.cd.CD_OK
    names = [k for k, _ in host.launches()]
    decode = [k for k in names if k.startswith(("k_batch_", "k_coef_", "k_score_"))]
    assert len(decode) == batches
    assert any(k.startswith("k_calib_") for k in names) == (batches == 0)
    assert sum(k.startswith("k_topk_select") for k in names) == max(batches, 1)
    host.lib.countdown_plan_destroy(h)


@pytest.mark.parametrize("variant,B,rank,kernel", [
    ("mono", 4, 0, "k_coef_mono<4,8,false,false>"), ("cats", 8, 0, "k_coef_mono<8,8,false,true>"),
    ("dual_ideal", 3, 0, "k_coef_dual<4,8,false,false>"), ("dual_pred", 4, 256, "k_coef_pred<4,8,false,5,8>"),
    ("dual_pred", 8, 256, "k_coef_pred_mfma<8,8,5>"), ("dense", 8, 0, "k_batch_dual<2,4>"),
])
def test_residual_layers_keep_the_order_of_their_sums(host, variant, B, rank, kernel):
    st, h = host.plan(4096, 14336, B, rank)
    assert st == host.cd.CD_OK
    host.launches()
    assert host.residual(h, variant, B) == host.cd.CD_OK
    assert [k for k, _ in host.launches() if k.startswith(("k_coef_", "k_batch_"))] == [kernel]
    host.lib.countdown_plan_destroy(h)
