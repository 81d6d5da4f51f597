"""The library's launch rules on the host (tests/native/launch_plan.hip), without a GPU."""
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(None)
def _program(q):
    exe = os.path.join(tempfile.mkdtemp(prefix="launch_plan"), "launch_plan")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2605_01774_amd", "csrc"),
                    f"-DELBM_Q={q}", os.path.join(ROOT, "tests", "native", "launch_plan.hip"), "-o", exe], check=True)
    return exe


def ask(lines, q=19):
    """Answers of the program to one question per line, as lists of whole numbers."""
    r = subprocess.run([_program(q)], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
    out = [[int(v) for v in ln.split()] for ln in r.stdout.splitlines()]
    assert len(out) == len(lines)
    return out
