"""The rates that bench.py derives from stage times: layers of small tiles, whose dX and weight gradients share a launch, have one
rate for the backward products, the others one for each stage as well."""
import pytest

import bench

UP_DOWN = 6.0e12  # FLOPs of a forward pass, and of either half of a backward pass


class _Run:
    bwd = True

    def flops(self):
        return (4.0e12, 2.0e12), [1]


@pytest.mark.parametrize("dgrad,wgrad", [(6.0, 3.0), (9.0, 0.0)])
def test_backward_rates(dgrad, wgrad):
    st = {"up": 4.0, "down": 2.0, "bwd_dgrad": dgrad, "bwd_wgrad": wgrad}
    out, _ = bench.gemm_summary(_Run(), st, 20.0)
    assert out["bwd_grouped_gemm_tflops"] == pytest.approx(2 * UP_DOWN / 9e-3 / 1e12, rel=1e-4)
    assert out["all_grouped_gemm_tflops"] == pytest.approx(3 * UP_DOWN / 15e-3 / 1e12, rel=1e-4)
    if wgrad:
        assert (out["bwd_dgrad_tflops"], out["bwd_wgrad_tflops"]) == (1000.0, 2000.0)
    else:
        assert out["bwd_dgrad_tflops"] is None and out["bwd_wgrad_tflops"] is None


@pytest.mark.gpu
@pytest.mark.parametrize("T,dtype,joined", [(512, "f32", True), (4096, "bf16", False)])
def test_stages_of_the_backward_pass(T, dtype, joined):
    import paper_2409_12210_amd as m
    from test_gpu_parity import _runner, make
    d, f = (256, 256) if joined else (2048, 2048)
    r = _runner(make("stages", d, (f,) * 8, T, dtype, need_dy=True), need_bwd=True)
    r.fwd()
    m.modse_stage_timing_enable(True)
    r.fwd()
    r.bwd()
    st = m.modse_stage_times()
    m.modse_stage_timing_enable(False)
    assert st["bwd_dgrad"] > 0 and (st["bwd_wgrad"] == 0) == joined
    for other in set(m.STAGES) - {"bwd_wgrad"}:
        assert st[other] > 0, other
