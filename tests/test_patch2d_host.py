"""Native host checks of the 2D patch kernel's plan, against the built library."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plan(cf, tmp_path):
    lib = os.path.join(ROOT, "paper_0906_5170_amd")
    exe = tmp_path / "patch2d_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(lib, "csrc"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "native", "patch2d_check.cpp"), "-o", str(exe),
                    "-L", lib, "-l:libcasimir_fdtd.so", "-L", "/opt/rocm/lib", "-lamdhip64",
                    f"-Wl,-rpath,{lib}:/opt/rocm/lib"], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    assert "patch2d ok" in out.stdout
