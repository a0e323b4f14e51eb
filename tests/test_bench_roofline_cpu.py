"""bench.py's roofline entry: the slowest of the kernels that the timed step
launches, with its own bytes and its own recorded traffic."""
import bench


def test_dominant_kernel_of_the_step():
    x = "k_strided<double, 1024, 8, 2, -1, 32, 0, true, 1, false>"
    z = "k_plane_r2c<double, 1024, 128, 16, 2, true>"
    R, C = 1024 ** 3 * 8, 1024 * 1024 * 513 * 16
    asked = []
    got = bench.roofline({z: 3.1, x: 3.5}, R, C, lambda k: asked.append(k) or 17)
    assert got["kernel"] == x and asked == [x] and got["traffic"] == 17
    assert got["algorithmic_bytes_per_launch"] == 2 * C
    assert got["achieved"] == round(2 * C / 3.5e-3 / 1e9, 1)
    got = bench.roofline({z: 3.6, x: 3.5}, R, C, lambda k: None)
    assert got["kernel"] == z and got["algorithmic_bytes_per_launch"] == R + C


def test_kernel_names():
    full = ("void gfft::k_strided_r<float, 512, 8, 8, 8, 1, false, 2>(gfft::cx<float> const*, "
            "gfft::cx<float>*, gfft::cx<float> const*, int)")
    assert bench.short_kernel(full) == "k_strided_r<float, 512, 8, 8, 8, 1, false, 2>"
    assert bench.kernel_bytes(full, 3, 5) == 10
    assert bench.kernel_bytes("void gfft::k_box_r2c<double, 16>(...)", 3, 5) == 8


def test_traffic_by_kernel(tmp_path):
    path = tmp_path / "t.md"
    path.write_text(f"kernel_source_sha256_16: {bench.kernel_source_hash()}\n\n"
                    "| pass | kernel | HBM bytes (scaled) |\n|---|---|---|\n"
                    "| x_fwd | `gfft::k_strided<double, 1024, 8>` | 123 |\n")
    assert bench.recorded_traffic(str(path), "x_fwd") == 123
    assert bench.recorded_traffic(str(path), "k_strided<double, 1024, 8>") == 123
    assert bench.recorded_traffic(str(path), "k_other") is None
