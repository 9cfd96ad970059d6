"""Address- and undefined-behaviour-sanitizer run of the host code that indexes memory by hand:
the oracle's C routines and the library's packing and native tiling (CPU only; the GPU code
cannot run under these sanitizers)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_oracle_and_host_packing_under_asan_and_ubsan(tmp_path):
    exe = str(tmp_path / "sanitize_driver")
    san = ["-fsanitize=address,undefined", "-static-libasan", "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-g", "-O1"]
    obj = str(tmp_path / "rb_oracle.o")
    subprocess.check_call(["gcc", "-std=c11", "-Wall", "-Wextra", *san, "-c",
                           os.path.join(ROOT, "oracle", "rb_oracle.c"), "-o", obj])
    subprocess.check_call(["g++", "-std=c++17", "-Wall", *san,
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2602_05367_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "driver.cpp"),
                           os.path.join(ROOT, "paper_2602_05367_amd", "csrc", "rb_host.cpp"),
                           obj, "-o", exe])
    env = dict(os.environ)
    env["ASAN_OPTIONS"] = "detect_leaks=1:abort_on_error=0"
    res = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, env=env, timeout=120)
    assert res.returncode == 0, res.stdout
    assert "all shapes passed" in res.stdout
    assert "runtime error" not in res.stdout and "AddressSanitizer" not in res.stdout, res.stdout


def test_requests_of_the_few_token_kernel_stay_inside_a_layer(tmp_path):
    """Ops of different widths share a launch: a wavefront that has no columns of the narrower one reads nothing past its end."""
    exe = str(tmp_path / "units_driver")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-fsanitize=address,undefined", "-static-libasan", "-fno-sanitize-recover=all", "-g", "-O1",
                           "-I", os.path.join(ROOT, "paper_2602_05367_amd", "csrc"), os.path.join(ROOT, "tests", "sanitize", "units.cpp"), "-o", exe])
    res = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert res.returncode == 0 and "all in bounds" in res.stdout, res.stdout


def _host_build_of_kernel_headers(tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-fsanitize=address,undefined", "-static-libasan", "-fno-sanitize-recover=all", "-g", "-O1", "-D__host__=", "-D__device__=",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2602_05367_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", name + ".cpp"), "-o", exe])
    return subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)


def test_the_ring_of_sign_tiles_lets_everyone_come_to_the_end(tmp_path):
    """Also a loading wavefront whose readers have given up and run ahead of it: a wait without an end would hang the GPU."""
    res = _host_build_of_kernel_headers(tmp_path, "ring")
    assert res.returncode == 0 and "everyone came to the end" in res.stdout, res.stdout


def test_ops_of_a_plan_hang_together_as_defined(tmp_path):
    """Among them: an addend of the caller's that an op which need not come later stores over is put aside."""
    res = _host_build_of_kernel_headers(tmp_path, "plan")
    assert res.returncode == 0 and "as defined" in res.stdout, res.stdout


def test_passes_of_the_initialisation_are_asked_for_in_measure(tmp_path):
    """A slow update says little of the others: neither many passes with nothing to do nor a look after every few."""
    res = _host_build_of_kernel_headers(tmp_path, "walk")
    assert res.returncode == 0 and "in measure" in res.stdout, res.stdout
