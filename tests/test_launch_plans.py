"""Where the launches of a product put their partial tiles, over the sizes, layouts and alignments that the entry points
take.  Runs on the CPU: launch_plans.cpp stands in for the HIP runtime and looks at the arguments."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2508_04355_amd")


def test_partial_tiles_stay_in_their_part_of_the_workspace(tmp_path):
    """Every k-split launch of gemm_tile (also where the kernel with 256 x 256 tiles was planned and refuses the operands)
    writes no more than the workspace has for it."""
    if not os.path.exists(os.path.join(PKG, "libgecc.so")):
        from paper_2508_04355_amd import build
        build.build(verbose=False)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = str(tmp_path / "launch_plans")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"),
                    "-I" + os.path.join(rocm, "include"), os.path.join(ROOT, "tests", "launch_plans.cpp"), "-o", exe, "-rdynamic",
                    "-L" + PKG, "-l:libgecc.so", "-Wl,-rpath," + PKG, "-L" + os.path.join(rocm, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(rocm, "lib")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
