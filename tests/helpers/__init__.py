"""Test helpers built with hipcc beside their sources."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
NORMALS_CHECK = os.path.join(HERE, "libnormals_check.so")


def build_normals_check() -> str:
    from paper_1306_3277_amd import build as hipbuild
    tmp = NORMALS_CHECK + ".tmp"
    subprocess.run([hipbuild.hipcc()] + hipbuild.flags() + [
        "-x", "hip", "-shared", os.path.join(HERE, "normals_check.hip"), "-o", tmp],
        check=True, cwd="/tmp")
    os.replace(tmp, NORMALS_CHECK)
    return NORMALS_CHECK
