"""Builds small host programs against the library's internal headers and the
built library (test helper; needs hipcc, no GPU)."""
import os
import subprocess

from paper_1909_07717_amd import build as Bd


def host_program(tmp_path, source, name="probe"):
    """Compile `source` (C++, host side only) and link it to the library."""
    src, obj, exe = (str(tmp_path / (name + e)) for e in (".hip", ".o", ""))
    with open(src, "w") as fh:
        fh.write(source)
    subprocess.check_call([Bd.hipcc(), "--cuda-host-only", "-std=c++17", "-O1", "-fPIC",
                           f"-I{Bd.CSRC}", f"-I{os.path.join(Bd.ROOT, 'include')}",
                           "-c", src, "-o", obj])
    subprocess.check_call([Bd.hipcc(), obj, Bd.LIB, f"-Wl,-rpath,{os.path.dirname(Bd.LIB)}",
                           "-o", exe])
    return exe
