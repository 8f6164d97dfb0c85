"""What the library decides on the host before it launches anything: a small C++ program asks the deciding
functions of the built library themselves.  No GPU is needed and no kernel is launched."""
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parent.parent


def test_host_decisions(tmp_path):
    from paper_2603_09229_amd import binding, build as fk_build
    binding.lib()                                # fails if the library has not been built
    exe = tmp_path / "decisions"
    rocm = Path(fk_build.HIPCC).parent.parent
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", f"-I{rocm / 'include'}", f"-I{ROOT / 'include'}", f"-I{fk_build.CSRC}",
           str(ROOT / "tests" / "host" / "decisions.cpp"), str(fk_build.LIB), f"-L{rocm / 'lib'}", "-lamdhip64",
           f"-Wl,-rpath,{fk_build.LIB.parent}", f"-Wl,-rpath,{rocm / 'lib'}", "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "host decisions ok" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
