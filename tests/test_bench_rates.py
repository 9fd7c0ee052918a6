"""The benchmark's roofline entries: FP32 products of the folded layer against
the unit they run on, six bfloat16 products each; everything else against its
own precision's."""
import bench


def test_matrix_peaks():
    assert bench.mfma_peak("lsc_folded_grad", "fp32") == bench.MFMA_PEAK_TFLOPS["bf16"] / 6
    assert bench.mfma_peak("lsc_folded_grad", "bf16") == bench.MFMA_PEAK_TFLOPS["bf16"]
    assert bench.mfma_peak("lsc_resample", "fp32") == bench.MFMA_PEAK_TFLOPS["fp32"]


def test_fractions_stay_below_one():
    # 1M voxels x 1440 x 136 multiply-adds in 2.8 ms, 4.6 GB
    flops, nbytes = 2.0 * 2 ** 20 * 1440 * 136, 2 ** 20 * 1575 * 4.0
    roof = bench.roofline("lsc_folded_grad", 2.8, 1, nbytes, flops, "fp32")
    assert roof["bound"] == "mfma" and 0 < roof["frac"] < 0.5 and roof["peak_of"].startswith("bf16")
    peaks = {"hbm_copy_GBs": 5800.0, "fp32_mfma_TFLOPs": 145.0, "bf16_mfma_TFLOPs": 2330.0}
    bench.with_measured_peak(roof, peaks, "fp32")
    assert roof["measured_peak"] == 388.3 and roof["frac_of_measured_peak"] < 0.5
    roof = bench.roofline("signal2sh_fwd", 0.5, 1, 1.6e9, 2e10, "fp32")
    assert roof["bound"] == "hbm" and bench.with_measured_peak(roof, peaks, "fp32")["measured_peak"] == 5800.0
