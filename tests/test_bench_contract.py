"""Host-side checks of the benchmark script's contract (no GPU needed)."""
import os
import re
import subprocess
import sys

import paper_2206_10620_amd as pp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr


def test_measured_traffic_belongs_to_the_current_kernel_revision():
    """The HBM traffic bench.py reports was measured with counters on one kernel revision; a stale entry
    must read as null, which bench.py does by comparing revisions.  The committed table and the committed
    profile summaries have to name the revision the library reports."""
    sys.path.insert(0, ROOT)
    import bench
    kernel_of = {2: "k1_tiled", 3: "k3_mfma"}
    for (wl, variant), (rev, nbytes) in bench.MEASURED_TRAFFIC.items():
        assert rev == pp.KERNEL_REVISION, f"{wl}: traffic measured on {rev}, library is {pp.KERNEL_REVISION}"
        assert nbytes > 0
        text = open(os.path.join(ROOT, "profiles", f"{kernel_of[variant]}_{wl}.md")).read()
        assert pp.KERNEL_REVISION in text
        m = re.search(r"= ([0-9.]+) MB, against", text)
        assert m and abs(float(m.group(1)) * 1e6 - nbytes) <= 0.02e6 + 1e-3 * nbytes


def test_binary32_traffic_belongs_to_the_kernel_that_runs():
    sys.path.insert(0, ROOT)
    import bench
    for (wl, kernel), (rev, nbytes) in bench.MEASURED_TRAFFIC_F32.items():
        plan = pp.plan_from_layer(bench.workloads()[wl](), host_only=True)
        chosen = plan.query()["chosen"]
        plan.close()
        assert bench.kernel_of(chosen) == kernel and rev == pp.KERNEL_REVISION
        assert bench.traffic_of(wl, chosen, pp.KERNEL_REVISION) == nbytes and bench.traffic_of(wl, chosen, "another") is None
        text = open(os.path.join(ROOT, "profiles", f"{kernel}_{wl}.md")).read()
        assert pp.KERNEL_REVISION in text
        m = re.search(r"= ([0-9.]+) MB, against", text)
        assert m and abs(float(m.group(1)) * 1e6 - nbytes) <= 0.02e6 + 1e-3 * nbytes
    # a kernel that runs by name only has its own figures, or none
    named = pp.Tuning(variant=2, mfma_kind=5).as_dict()
    assert bench.traffic_of("cfg2_vgg_mid", named, pp.KERNEL_REVISION) is None


def test_a_binary32_kernel_is_held_to_the_rate_of_its_own_instruction():
    sys.path.insert(0, ROOT)
    import bench
    lay = bench.workloads()["cfg3_resnet_c256_n32"]()
    chosen = pp.Tuning(variant=2, mfma_kind=5).as_dict()
    for kernel, us, peak in (("k5_conv_f32", 41.0, 2500.0 / 6), ("k5_whole_f32", 80.0, 157.3), ("k6_f32_3x3", 68.0, 157.3)):
        t = dict(event_ms_per_step=us * 1e-3, wall_ms_per_step=us * 1e-3, chosen=chosen, kernel=kernel)
        roof, line = bench.roofline_of(lay, t, None), bench.summarize(lay, t)
        assert roof["kernel"] == line["kernel"] == kernel and roof["peak"] == peak and 0.1 < roof["frac"] < 1
        assert abs(line["frac_mfma_dense"] - 2 * bench.dense_macs(lay) / us / 1e6 / peak) < 1e-9
    for staging, kernel in ((1, "k5_whole_f32"), (3, "k5_conv_f32")):
        plan = pp.plan_from_layer(lay, host_only=True, tuning=pp.Tuning(variant=2, mfma_kind=5, staging=staging))
        assert plan.kernel == bench.kernel_of(plan.query()["chosen"]) == kernel
        plan.close()


def test_the_json_line_is_last_and_short():
    """A reader that keeps the last 2000 characters of the output has to find the whole line."""
    import json
    sys.path.insert(0, ROOT)
    import bench
    x = 12345.67890123456789
    names = [n for n in bench.workloads()] + ["cfg4_vgg_stack_chained", bench.BLOCK_WORKLOAD, bench.REUSE_WORKLOAD]
    out = {"metric": "effective GMAC/s (nonzero MACs), pattern-pruned 3x3 conv", "value": x, "unit": "GMAC/s", "n_gpus": 1, "steps": 100, "warmup": 20, "ms_per_step": x,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "tuned": False, "dtype": "f16", "data": "synthetic",
           "config": {"workload": "cfg5_enhance_1080p", "n": 1, "c_in": 64, "c_out": 64, "h": 1080, "w": 1920, "patterns": 16, "k_kept": 1638, "keep": x, "fused": "bias+relu",
                      "params": pp.Tuning(variant=3, tile_rows=16, tile_cols=60, tiles_per_wave=2, wg_waves=8, mfma_kind=2, split_k=1).as_dict()},
           "alg_gb_per_s": x, "frac_hbm": x, "frac_fp32_valu": x, "frac_fp32_valu_unpacked": x,
           "roofline": {"bound": "hbm", "achieved": x, "peak": x, "unit": "GB/s", "frac": x, "traffic": x, "kernel": "k3_mfma", "kernel_us": x, "frac_mfma": x, "peak_mfma_tflops": x},
           "copy_reference": {"bytes_moved": 530841600, "us": x, "gb_per_s": x, "layer_us_over_copy_us": x},
           "cpu_baseline": {"value": x, "unit": "GMAC/s", "cores": 16, "kind": "oracle", "sample": "3472222 sampled outputs (2.616% of the layer)", "seconds": x}, "max_rel_err": x}
    lines = bench.output_lines(out, [dict(workload=n, us_per_step=412.34567, note="y" * 500) for n in names])
    assert len(lines) == len(names) + 2 and all(l.startswith("# other {") for l in lines[:-2])
    assert dict(o.split("=") for o in lines[-2].split()[2:]) == {n: "412.3" for n in names}
    assert all("\n" not in l for l in lines) and len(lines[-1]) <= 1600          # (what the runtime prints to stderr comes behind it)
    back = json.loads(lines[-1])
    assert set(out) == set(back) and back["config"]["params"]["wg_waves"] == 8
    assert json.loads(bench.output_lines(out, None)[-1])["value"] == 12345.7


def test_block_product_traffic_belongs_to_the_current_kernel_revision():
    sys.path.insert(0, ROOT)
    import bench
    from paper_2206_10620_amd import pp_block_gemm as pb
    rev, nbytes = bench.MEASURED_TRAFFIC_BLOCK
    assert rev == pb.BLOCK_KERNEL_REVISION and nbytes > 0
    text = open(os.path.join(ROOT, "profiles", "k4_block_gemm_block_ffn_4096.md")).read()
    assert pb.BLOCK_KERNEL_REVISION in text
    m = re.search(r"= ([0-9.]+) MB, against", text)
    assert m and abs(float(m.group(1)) * 1e6 - nbytes) <= 0.02e6 + 1e-3 * nbytes


def test_workload_table_covers_the_benchmark_configurations():
    sys.path.insert(0, ROOT)
    import bench
    names = set(bench.workloads())
    assert bench.DEFAULT_WORKLOAD == "cfg5_enhance_1080p"      # the largest single-GPU configuration
    assert {"cfg2_vgg_mid", "cfg5_enhance_1080p"} <= names
    assert sum(n.startswith("cfg4_vgg_L") for n in names) == 13
    assert sum(n.startswith("cfg3_resnet_") and not n.endswith("_f16") for n in names) == 8
    assert {"cfg2_vgg_mid_f16", "cfg2_shape_foreign_patterns_f32", "cfg2_shape_foreign_patterns_f16"} <= names
