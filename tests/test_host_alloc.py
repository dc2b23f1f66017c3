"""Device memory that runs out, a wait that fails: the error is reported by the call that met
it and by no other. HIP keeps a failed call's error until hipGetLastError reads it, and every launch
is checked with hipGetLastError, so an error left behind by another call would be taken for
a failed launch."""
import pytest

import host_hip


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    return host_hip.Host(host_hip.build(str(tmp_path_factory.mktemp("host"))))


def test_calibration_continues_with_a_smaller_chunk(host):
    st, h = host.plan(4096, 11008)
    assert st == host.cd.CD_OK
    host.launches()
    before = host.lib.host_hip_live_allocations()
    # 256 tokens' coefficients take 11 MB; room for 64 tokens' and less than 128 tokens'
    host.limit(4 << 20)
    try:
        assert host.calibrate(h, "mono", 256) == host.cd.CD_OK
    finally:
        host.limit()
    gemms = [k for k, _ in host.launches() if k.startswith("k_calib_gemm")]
    assert len(gemms) == 4  # 64 tokens at a time
    assert host.lib.host_hip_live_allocations() == before + 1  # the workspace, kept
    host.lib.countdown_plan_destroy(h)


@pytest.mark.parametrize("variant,rank", [("mono", 0), ("dual_pred", 64)])
def test_calibration_without_memory_fails_alone(host, variant, rank):
    """No room even for one token's coefficients: CD_ENOMEM, and the plan's next call runs."""
    st, h = host.plan(256, 688, 1, rank)
    assert st == host.cd.CD_OK
    host.launches()
    host.limit(1024)
    try:
        for T in (1, 40):
            assert host.calibrate(h, variant, T) == host.cd.CD_ENOMEM
            assert host.launches() == []
            assert host.ffn(h, variant, 1) == host.cd.CD_OK
            assert len(host.launches()) >= 2
    finally:
        host.limit()
    assert host.calibrate(h, variant, 40) == host.cd.CD_OK
    host.lib.countdown_plan_destroy(h)


def test_plan_without_memory_fails_alone(host):
    st, h = host.plan(256, 688)
    assert st == host.cd.CD_OK
    before = host.lib.host_hip_live_allocations()
    host.limit(4096)  # the flags of 8192 neurons do not fit
    try:
        st, _ = host.plan(256, 8192)
    finally:
        host.limit()
    assert st == host.cd.CD_ENOMEM
    assert host.lib.host_hip_live_allocations() == before
    assert host.ffn(h, "mono", 1) == host.cd.CD_OK
    host.lib.countdown_plan_destroy(h)


def test_calibration_under_capture_fails_alone(host):
    """A calibration waits for its stream, which a capture refuses: CD_EHIP, and the next
    call's launches are not taken for failed ones."""
    st, h = host.plan(256, 688)
    assert st == host.cd.CD_OK
    host.lib.host_hip_set_sync_fails(1)
    try:
        assert host.calibrate(h, "mono", 40) == host.cd.CD_EHIP
    finally:
        host.lib.host_hip_set_sync_fails(0)
    assert host.ffn(h, "mono", 1) == host.cd.CD_OK
    host.lib.countdown_plan_destroy(h)
