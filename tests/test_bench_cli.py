"""bench.py's command line, host side only (nothing touches a GPU)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    # this build runs on one GPU; the refusal comes before torch or the library is loaded
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=60)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr and "--gpus 1" in r.stderr
    assert r.stdout.strip() == ""            # no JSON line that could be taken for a measurement


def test_help_lists_every_mode():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--help"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0
    for flag in ("--gpus", "--steps", "--warmup", "--workload", "--pipeline", "--all", "--verify", "--draft", "--ragged", "--stream", "--ablations"):
        assert flag in r.stdout


def test_roofline_traffic_is_read_from_the_tracked_counter_summaries():
    """bench.py holds no counter literal: the figure comes from profiles/ (FETCH/WRITE KiB per launch times the
    calibration factors stated there), and a kernel the summary does not list yields no figure."""
    import re
    sys.path.insert(0, ROOT)
    import bench
    text = open(os.path.join(ROOT, "profiles", bench.COUNTER_FILES["reduce5"])).read()
    rows = [ln for ln in text.splitlines() if re.match(r"^\S.*\s{2,}\d+\s+\d+\s+\d+\s", ln)]
    assert len(rows) >= 5
    name = rows[0].split("  ")[0].strip()
    nums = [int(x) for x in re.findall(r"\s(\d+)(?=\s)", rows[0][len(name):])][:3]
    got = bench.counter_traffic("reduce5", [name])
    assert got == nums[1] * 1024 * 2.0 + nums[2] * 1024 * 1.0        # the factors of the summary's calibration line
    assert bench.counter_traffic("reduce5", ["a_kernel_that_does_not_exist"]) is None
    assert bench.counter_traffic("vocab", ["draft_scan_kernel", "draft_merge_kernel"]) > 150e6


def test_gram_work_does_not_depend_on_the_tiles():
    """One image's Gram matrix runs on 32 x 32 tiles, a batch's on 128 x 128 ones: the same work per image is counted."""
    import bench
    assert bench.gram_flops(1, 288, 4096) == 288 * 289 * 4096
    assert bench.gram_flops(64, 288, 4096) == 64 * bench.gram_flops(1, 288, 4096)


def test_roofline_names_the_kernel_that_runs():
    """The kernels of the Gram matrix follow the library's rule: few tiles, many tiles, fp64 products."""
    import bench
    import covspec_inputs as I
    import paper_2605_02218_amd as C

    class Probe:
        probe_launches = staticmethod(lambda p: (0, 0, 0, 0))
    stages = {s: 0.0 for s in C.STAGES}
    stages["gram"] = 1.0
    for kw, modes, kernel in ((dict(batch=1, dtype=I.BF16), (0, 0), "gemm_gram_small_kernel"), (dict(batch=64, dtype=I.BF16), (0, 0), "gemm_dma_kernel"),
                              (dict(batch=1, dtype=I.FP32), (0, 0), "gemm64_small_kernel"), (dict(batch=1, dtype=I.BF16), (1, 1), "gemm64_dma_kernel"),
                              (dict(batch=1, dtype=I.BF16, d_model=4000), (1, 1), "gemm64_kernel")):
        w = I.small_workload(n_tokens=576, n_query=32, n_heads=32, keep_k=144, preselect_m=288, rank_r=72, n_act_layers=4, **dict(dict(d_model=4096), **kw))
        got = bench.roofline_for(w, None, modes, dict(stages, activity=1e-9, gather=1e-9, token_projection=1e-9, lowrank=1e-9), 0.0, Probe)
        assert got["kernel"] == kernel


def test_roofline_names_the_kernel_of_the_greedy_picks():
    """All rows are picks; a small part of the rows with a few images or with many; too many rows for runs of picks."""
    import bench
    for B, M, k, kernel in ((64, 640, 320, "greedy_panel_kernel"), (1, 960, 480, "greedy_panel_kernel"), (1, 961, 480, "greedy_step_kernel"),
                            (4, 2304, 1152, "greedy_step_kernel"), (1, 4096, 100, "greedy_kernel"), (64, 4096, 100, "greedy_single_kernel")):
        assert bench.greedy_kernel_name(B, M, k) == kernel
