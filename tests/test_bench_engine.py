"""What bench.py says about the kernels that ran: the engine and types of a split-precision solve, and a roofline
that bounds the whole-side passes (no GPU)."""
import bench


def test_engine_and_types_come_from_the_kernels_that_ran():
    vec = {"bf_side_in_f32": (2, 1.0), "bf_side_out_f32": (2, 1.0), "ulv_up": (4, 0.1)}
    mat = {"bf_struct_leaf_f32": (2, 1.0), "bf_split16": (6, 3.0), "bf_leaf_out_f32": (2, 1.0)}
    assert bench.engine_of(vec) == "valu" and bench.engine_of(mat) == "mfma"
    # an untuned split-precision solve runs the FP32 passes, whatever its tile table says
    assert bench.compute_dtype("split16", vec) == "fp32+fp64"
    assert bench.compute_dtype("split16", mat) == "fp16x2+fp32+fp64"
    assert bench.compute_dtype("mixed", vec) == "fp32+fp64"


def test_roofline_of_whole_side_passes():
    """N = 2^18, q = 9, 64 columns: 6 levels of N/2 groups of two shared real 9 x 9 products per component (2 x 81
    multiply-adds each), a leaf factor of N pairs (8 x 9 multiply-adds), half of M's N pairs of 4 x 9 complex entries."""
    n, q, k = 1 << 18, 9, 64
    flops = 2 * k * (6 * (n // 2) * 2 * 2 * 81 + n * 2 * 36 + n * 36 * 4 // 2)
    for name, e, peak, ms in (("bf_side_in_f64", 16, 78.6, 1.5), ("bf_side_out_f64", 16, 78.6, 2.2),
                              ("bf_side_in_f32", 8, 157.3, 0.8), ("bf_side_out_f32", 8, 157.3, 0.95)):
        b, f, spill, p = bench.kernel_model(name, n, q, k)
        assert f == flops and p == peak and spill == n * q * k * e and b == 16 * n * k + 4 * n * e
        r = bench.roofline_of(name, n, q, k, ms, None)
        # measured times: a bound may not be beaten
        assert r["bound"] == "alu" and 0.05 < r["frac"] < 1.0
    assert bench.kernel_model("bf_side_f64", n, q, k)[0] == 0


def test_counter_labels_of_whole_side_passes(tmp_path, capsys):
    from test_bench_traffic import _write
    import json
    n, k = 1 << 18, 64
    grid, gib = 4096 * 8 * 256, float(1 << 20)
    name = "void fio::k_side_pass<%s>(fio::SideArgs<double>)"
    rows = [(1, "copy", 1, gib), (2, name % "double, true, false, false", grid, 100.0),
            (3, name % "double, false, true, false", grid, 300.0), (4, name % "double, true, true, true", grid // 8, 50.0),
            (5, name % "float, false, false, true", grid // 8, 70.0), (6, name % "double, false, false, false", grid, 9e9),
            (7, name % "double, true, false, false", grid // 2, 9e9)]
    _write(str(tmp_path / "F"), "FETCH_SIZE", rows)
    _write(str(tmp_path / "W"), "WRITE_SIZE", rows)
    bench.traffic_from(str(tmp_path / "F"), str(tmp_path / "W"), n=n, k=k, q=9, out_path=str(tmp_path / "t.json"))
    ks = json.load(open(tmp_path / "t.json"))["kernels"]
    assert {m: (v["dispatches"], v["hbm_bytes_per_launch"]) for m, v in ks.items()} == {
        "bf_side_in_f64": (2, 400 * 1024.0), "bf_side_out_f64": (1, 100 * 1024.0), "bf_side_out_f32": (1, 140 * 1024.0)}
    capsys.readouterr()
