"""bench.py argument contract that can be checked without a GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    for extra_env, args in (({}, ["--gpus", "2"]), ({"WORLD_SIZE": "2"}, [])):
        env = dict(os.environ, **extra_env)
        res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py")] + args, capture_output=True, text=True,
                             env=env, timeout=120)
        assert res.returncode != 0
        assert "ONE GPU" in res.stderr and res.stdout.strip() == ""


def test_profiles_name_the_workload_the_bench_times():
    import json
    from paper_2509_26541_amd import workloads as wl
    with open(os.path.join(ROOT, "paper_2509_26541_amd", "hbm_traffic.json")) as f:
        traffic = json.load(f)
    name = wl.CONFIGS[1].name                      # the default workload of bench.py
    assert name in traffic and traffic[name]["attn_bytes_per_launch"] > 0
    path = os.path.join(ROOT, traffic[name]["profile"])
    assert os.path.exists(path)
    text = open(path).read()
    assert "rocprofv3 --kernel-trace --stats" in text and "--pmc FETCH_SIZE" in text and "bench.py --config 2" in text
    # the traffic figure belongs to one version of the kernel source; bench.py reports it only for that one
    assert len(traffic[name]["attn_bf16_hip_sha16"]) == 16


def test_the_traffic_figure_belongs_to_the_kernel_and_its_headers(tmp_path):
    """The hashes that bench.py compares cover every header the kernel's translation unit takes from this repository, as the preprocessor meets them."""
    import json
    import re
    import shutil
    import bench
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with open(os.path.join(ROOT, "paper_2509_26541_amd", "hbm_traffic.json")) as f:
        traffic = json.load(f)
    assert all(set(bench.kernel_hashes()) <= set(rec) for rec in traffic.values())
    if shutil.which(hipcc) is None:
        return
    csrc = os.path.join(ROOT, "paper_2509_26541_amd", "csrc")
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + csrc, "-E", "--cuda-device-only",
                          "-x", "hip", os.path.join(csrc, "attn_bf16.hip"), "-o", str(tmp_path / "attn_bf16.i")], capture_output=True, text=True, check=True)
    marks = re.findall(r'^# \d+ "([^"]+\.hpp)"', (tmp_path / "attn_bf16.i").read_text(), re.M)
    assert {os.path.basename(x) for x in marks if os.path.dirname(x) == csrc} == set(bench.kernel_headers()), res.stderr
