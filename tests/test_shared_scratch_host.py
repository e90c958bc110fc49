"""Who gets the library's scratch buffer: one call at a time on each GPU, in stream order or after the last one
is done, none under graph capture; GPUs do not share a lock.  Runs the host code on a made-up HIP runtime."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_one_call_at_a_time_per_gpu(tmp_path):
    exe, obj = str(tmp_path / "shared_use"), str(tmp_path / "api.o")
    csrc = os.path.join(ROOT, "paper_2301_08984_amd", "csrc")
    flags = ["-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fno-gpu-rdc", "-c"]
    test = os.path.join(ROOT, "tests", "host_runtime", "shared_use.cpp")
    for src, out in ((os.path.join(csrc, "api.hip"), obj), (test, exe + ".o")):
        r = subprocess.run(["hipcc", *flags, src, "-o", out], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
    # kernel launchers are not called here and stay undefined
    r = subprocess.run(["g++", obj, exe + ".o", "-o", exe, "-no-pie", "-pthread", "-Wl,--unresolved-symbols=ignore-all"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all checks passed" in r.stdout, (r.returncode, r.stdout, r.stderr)
