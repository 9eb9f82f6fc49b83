"""What the compiler makes of the kernels' main loops, where a source form that looks the same costs time (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2605_29517_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")


def kernel_bodies(tmp_path, instantiations, flags=()):
    """The gfx950 assembly of kernels of forward_impl.h, in the order given."""
    src = tmp_path / "kernels.hip"
    src.write_text('#include "%s"\nnamespace maxsim { namespace {\n%s\n} }\n' % (
        os.path.join(B.CSRC, "forward_impl.h"),
        "\n".join("template __global__ void %s(FwdParams, OffsetsPtr);" % i for i in instantiations)))
    out = tmp_path / "kernels.s"
    subprocess.run([HIPCC] + B.FLAGS + list(flags) + ["--cuda-device-only", "-S", str(src), "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    bodies = re.findall(r"^_ZN\S*_kernel\S*:(.*?)\.Lfunc_end", out.read_text(), re.S | re.M)
    assert len(bodies) == len(instantiations)
    return bodies


TILE_SHAPES = ["fwd_tile_kernel<fmt(MAXSIM_%s, %d), %s>" % (dt, nu, shape)
               for dt, nu in (("F16", 8), ("BF16", 8), ("F16", 4), ("F32", 8))
               for shape in ("4, 2, false, 4", "8, 2, false, 3", "8, 3, false, 1", "4, 4, false, 1", "8, 4, false, 1")]


def test_tile_walk_stays_in_scalar_registers(tmp_path):
    """The walk over documents is the same in every lane: nothing of it may come back from vector registers per tile."""
    for name, body in zip(TILE_SHAPES, kernel_bodies(tmp_path, TILE_SHAPES)):
        loop = body[body.index("v_mfma"):]
        assert loop.count("v_readfirstlane") == 0, name


def test_argmax_loops_are_aligned(tmp_path):
    """Stretches between the MFMAs of the 16-bit argmax loop begin at fixed places of a cache line, whatever comes before."""
    shapes = ["fwd_tile_kernel<fmt(MAXSIM_%s, 8), 8, %d, true, 1>" % (dt, ncb) for dt in ("F16", "BF16") for ncb in (3, 4)]
    for name, body in zip(shapes, kernel_bodies(tmp_path, shapes, B.FILE_FLAGS.get("forward_argmax.hip", []))):
        first = body.index("v_mfma")
        assert ".p2align\t6" in body[:first] and ".p2align\t6" in body[first:], name
