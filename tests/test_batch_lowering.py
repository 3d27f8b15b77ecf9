"""What a batch of copies becomes on the host, in every mode, and that its cost is linear."""

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_batches_are_lowered_to_what_they_mean_in_linear_time(tmp_path):
    rocm = os.path.dirname(os.path.dirname(os.path.abspath(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"))))
    exe = str(tmp_path / "batch_lowering")
    subprocess.run([os.path.join(rocm, "llvm", "bin", "clang++"), "-O3", "-std=c++17", "-Wall", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                    os.path.join(HERE, "models", "batch_lowering.cpp"), "-o", exe,
                    "-L" + os.path.join(rocm, "lib"), "-Wl,-rpath," + os.path.join(rocm, "lib"), "-lamdhip64"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout
