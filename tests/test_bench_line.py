"""The benchmark line stays short enough to be read back whole from the end of a log."""
import json


def test_regimes_are_compact_in_the_benchmark_line():
    import bench
    roof = dict(stage="gate_up", kernel="ffn_mfma_kernel<gate_up> / ffn_stream_kernel<gate_up> (by rows per expert)", bound="hbm",
                achieved=4382.01, peak=8000.0, unit="GB/s", frac=0.5477, traffic=None, avg_launch_ms=0.0397,
                flops_per_launch=738197504.0, bytes_per_launch=173967832.6153846)
    per_k = {"k": 2, "layers": 5, "gate_up": roof, "down": roof}
    rec = dict(workload="c5_dsv2lite L=26 d=2048 E=64 F=1408 Fs=2816 T=256", name="c5_dsv2lite", T=256, regime="decode",
               hip_graph=True, k_vec=[6] * 32, k_sum=104, k_uniform=6, ms_per_step=58.5566, ms_per_step_median_of_events=58.5775,
               tokens_per_s=69949.4, uniform_k_tokens_per_s=53565.8, speedup_vs_uniform_k=1.3059,
               stage_ms_per_step=dict.fromkeys(("routing", "gate_up", "down", "shared", "combine"), 37.1093),
               experts_touched_per_layer=[64] * 32, rooflines=[roof, roof], per_k=[per_k] * 8,
               whole_path=dict(flops_per_step=69277822484480.0), chained_stack=None, stage1_profiling=None, cpu_baseline=None,
               parity_on_sample=dict(tokens=242, layers=[0] * 8, routing_mismatches=0, max_err_over_rms=0.001617,
                                     max_err_over_rms_vs_unrounded_oracle=0.008008))
    line = [bench.compact(rec)] * sum(len(bench_regimes) for bench_regimes in _regimes())
    assert len(json.dumps(line)) < 6000            # the headline's own fields take about 3000 more
    assert line[0]["tokens_per_s"] == rec["tokens_per_s"] and line[0]["parity_on_sample"]["routing_mismatches"] == 0
    assert "parity_on_sample" not in bench.compact(dict(rec, parity_on_sample=None))


def _regimes():
    import bench
    import lexi_synth as S
    return [S.CONFIGS[n].T_regimes for n in bench.DEFAULT_WORKLOADS]
