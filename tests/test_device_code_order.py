"""Orderings that a kernel asks of the compiler, looked up in the assembly it
makes of the sources (no device needed)."""
import os
import re
import subprocess

from paper_2511_21713_amd import build as libbuild


def device_assembly(name, tmp_path):
    out = os.path.join(tmp_path, name + ".asm")
    flags = [f for f in libbuild.FLAGS if f != "-fPIC"]
    subprocess.run(["hipcc", "-S", "--cuda-device-only", *flags, "-o", out, os.path.join(libbuild.SRC, name)],
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_matrix_free_tiles_separate_their_steps(tmp_path):
    """Consecutive steps of a tile update the same LDS sums from different
    lanes: every instantiation has the wavefront barrier between them."""
    text = device_assembly("kernels_mf.hip", str(tmp_path))
    bodies = re.findall(r"^(_ZN4pbfb9k_mf_tile\w+):(.*?)^\.Lfunc_end", text, flags=re.S | re.M)
    assert len(bodies) == 4  # Laplace and Yukawa, FP64 and FP32
    for name, body in bodies:
        assert "; wave barrier" in body, name
