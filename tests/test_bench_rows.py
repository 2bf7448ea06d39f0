"""The benchmark's figures per kernel, from launch counts and times as the library reports them."""
import bench


def test_a_reconstruction_in_the_reverse_scans_launch_is_priced_there():
    fl, by = bench.flops_per_tokhd(64, 128, 128), bench.bytes_per_tokhd(64, 128, 128, 2, False)
    tokhd, steps, peak = 16 * 4096, 10, bench.PEAK_BF16_TFLOPS
    apart = bench.kernel_rows({"rebuild": (0.5, 10, 10), "scan_bwd": (1.0, 10, 10)}, fl, by, tokhd, steps, peak)
    shared = bench.kernel_rows({"rebuild": (0.0, 0, 10), "scan_bwd": (1.0, 10, 10)}, fl, by, tokhd, steps, peak)
    kept = bench.kernel_rows({"rebuild": (0.0, 0, 0), "scan_bwd": (1.0, 10, 10)}, fl, by, tokhd, steps, peak)
    assert set(apart) == {"rebuild", "scan_bwd"} and set(shared) == set(kept) == {"scan_bwd"}
    assert kept["scan_bwd"] == apart["scan_bwd"]
    assert shared["scan_bwd"]["with"] == "rebuild"
    for key in ("gflop_per_launch", "mib_per_launch"):
        both = apart["rebuild"][key] + apart["scan_bwd"][key]
        assert abs(shared["scan_bwd"][key] - both) <= 0.1 + 1e-3 * both
    work = (fl["scan_bwd"] + fl["rebuild"]) * tokhd
    assert abs(shared["scan_bwd"]["tflops"] - work / 1e-4 / 1e12) <= 0.01
