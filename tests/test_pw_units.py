"""The grouped widening step's work units for arbitrary group offsets, on the
host: the kernels' own index arithmetic (csrc/pw_units.hpp) compiled into a
small program."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_units_stay_in_their_array_and_their_groups(tmp_path):
    exe = str(tmp_path / "pw_units")
    csrc = os.path.join(os.path.dirname(HERE), "paper_2606_19729_amd", "csrc")
    subprocess.run(["hipcc", "-O1", "-x", "hip", "--offload-arch=gfx950", "-w", "-I", csrc,
                    os.path.join(HERE, "pw_units_host.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
