"""Small host programs of the tests: compiled with hipcc (they include the library's headers) and run on the CPU."""
import os
import subprocess

from paper_1209_5421_amd import build as B

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


def build(source, out_dir, flags=()):
    exe = os.path.join(str(out_dir), os.path.splitext(source)[0])
    cmd = [B.hipcc(), *B.COMMON, "-O1", f"-I{B.CSRC}", os.path.join(HERE, source), "-o", exe, *flags]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def run(exe, *args, env=None):
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    return r.stdout
