"""What the compiler makes of the kernels' main loops, where a source form that looks the same costs time (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2605_29517_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")


def kernel_bodies(tmp_path, instantiations, flags=(), header="forward_impl.h", more=""):
    """The gfx950 assembly of kernels of a header, in the order given; `more`: their parameters after the first two."""
    src = tmp_path / "kernels.hip"
    src.write_text('#include "%s"\nnamespace maxsim { namespace {\n%s\n} }\n' % (
        os.path.join(B.CSRC, header),
        "\n".join("template __global__ void %s(FwdParams, OffsetsPtr%s);" % (i, more) for i in instantiations)))
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


def registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$|v(\d+)$", operand)
    return range(0) if not m else range(int(m[3]), int(m[3]) + 1) if m[3] else range(int(m[1]), int(m[2]) + 1)


def test_wide_kernel_waits_for_its_mfmas(tmp_path):
    """The 16x16 MFMAs of the wide kernel are assembly, which the compiler does not see through: an accumulator is read or written by
    other instructions only some cycles after the MFMA that writes it (11 for four passes), an MFMA does not read what a vector
    instruction wrote less than two cycles ago, and nothing spills."""
    shapes = ["fwd_wide_kernel<MAXSIM_%s, WideShape<%s>, false, WD_16%s>" % (dt, shape, half)
              for dt, shape in (("BF16", "2, 4, 4, 2"), ("F16", "4, 2, 2, 3"), ("BF16", "8, 1, 1, 1")) for half in ("", "_HALF")]
    for name, body in zip(shapes, kernel_bodies(tmp_path, shapes, (), "forward_wide_impl.h", ", int, int")):
        assert "scratch_" not in body, name
        now, by_mfma, by_move = 0, {}, {}
        count = 0
        for line in body.split("\n"):
            line = line.split(";")[0].strip()
            if not line or line.startswith("."):
                continue
            op, _, rest = line.partition(" ")
            operands = [x.strip() for x in rest.split(",")]
            now += int(operands[0]) + 1 if op == "s_nop" else 1
            if op.startswith("v_mfma"):
                count += 1
                assert all(now - by_move.get(r, -9) > 2 for o in operands[1:] for r in registers(o)), (name, line)
                by_mfma.update((r, now) for r in registers(operands[0]))
            else:
                assert all(now - by_mfma.get(r, -99) >= 12 for o in operands for r in registers(o)), (name, line)
                if op.startswith("v_"):
                    by_move.update((r, now) for r in registers(operands[0]))
        assert count > 0, name
