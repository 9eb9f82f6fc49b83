"""What the compiler makes of the kernels' main loops, where a source form that looks the same costs time (no GPU needed)."""
import concurrent.futures
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


def blocks(body):
    """The basic blocks of a kernel's assembly, [(instructions, numbers of the blocks that may follow)]."""
    parts, labels = [[]], {}
    for line in body.split("\n"):
        line = line.split(";")[0].strip()
        if re.match(r"\.LBB\w+:$", line):
            parts.append([])
            labels[line[:-1]] = len(parts) - 1
        elif line and not line.startswith("."):
            op, _, rest = line.partition(" ") if " " in line else line.partition("\t")
            parts[-1].append((op, [x.strip() for x in rest.split(",")]))
            if op in ("s_branch", "s_endpgm") or op.startswith("s_cbranch"):
                parts.append([])
    out = []
    for n, part in enumerate(parts):
        op, operands = part[-1] if part else ("", [])
        follow = [labels[operands[0]]] if op == "s_branch" or op.startswith("s_cbranch") else []
        if op not in ("s_branch", "s_endpgm") and n + 1 < len(parts):
            follow.append(n + 1)
        out.append((part, follow))
    return out


def walk(instructions, by_mfma, by_move, broken=None):
    """The state behind a block: cycles since registers were written by an MFMA (while under 12) and by a vector instruction (up to 2).
    An instruction that comes too early goes to `broken`."""
    by_mfma, by_move = dict(by_mfma), dict(by_move)
    for op, operands in instructions:
        step = int(operands[0]) + 1 if op == "s_nop" else 1
        by_mfma = {r: a + step for r, a in by_mfma.items() if a + step < 12}
        by_move = {r: a + step for r, a in by_move.items() if a + step <= 2}
        if op.startswith("v_mfma"):
            if broken is not None and any(r in by_move for o in operands[1:] for r in registers(o)):
                broken.append((op, operands))
            by_mfma.update((r, 0) for r in registers(operands[0]))
        else:
            if broken is not None and any(r in by_mfma for o in operands for r in registers(o)):
                broken.append((op, operands))
            if op.startswith("v_"):
                for o in operands[:2 if "swap" in op else 1]:
                    by_move.update((r, 0) for r in registers(o))
    return by_mfma, by_move


def too_early(body):
    """Instructions that come too early behind an MFMA or a move along any path."""
    graph = blocks(body)
    before = {0: ({}, {})}
    todo = [0]
    while todo:
        n = todo.pop()
        after = walk(graph[n][0], *before[n])
        for f in graph[n][1]:
            merged = tuple({r: min(x.get(r, 99), y.get(r, 99)) for r in x.keys() | y.keys()} for x, y in zip(after, before[f])) if f in before else after
            if f not in before or merged != before[f]:
                before[f] = merged
                todo.append(f)
    broken = []
    for n, state in before.items():
        walk(graph[n][0], *state, broken)
    return broken


def test_too_early_is_seen_along_every_path():
    mfma, end = "v_mfma_f32_16x16x32_f16 v[0:3], v[8:11], v[12:15], v[0:3]\n", "s_endpgm\n"
    assert not too_early(mfma + "s_nop 10\nv_max_f32_e32 v4, v0, v1\n" + end)
    assert too_early(mfma + "s_nop 9\nv_max_f32_e32 v4, v0, v1\n" + end)
    assert too_early("s_branch .LBB0_2\n.LBB0_1:\nv_mov_b32_e32 v3, 0\n" + end + ".LBB0_2:\n" + mfma + "s_cbranch_scc1 .LBB0_1\ns_nop 15\n" + end)  # the branch back
    assert not too_early("s_branch .LBB0_2\n.LBB0_1:\nv_mov_b32_e32 v4, 0\n" + end + ".LBB0_2:\n" + mfma + "s_cbranch_scc1 .LBB0_1\ns_nop 15\n" + end)
    assert too_early("v_permlane16_swap_b32_e32 v7, v8\ns_nop 0\n" + mfma + end) and not too_early("v_permlane16_swap_b32_e32 v7, v8\ns_nop 1\n" + mfma + end)
    assert too_early(".LBB0_1:\n" + mfma + "v_mov_b32_e32 v12, v20\ns_cbranch_scc1 .LBB0_1\n" + end)


WIDE_SHAPES = ("2, 4, 1, 2", "4, 2, 1, 1", "4, 2, 1, 2", "2, 4, 2, 2", "8, 1, 1, 1", "8, 1, 1, 2", "4, 2, 2, 2", "4, 2, 2, 3", "2, 4, 4, 2")


@pytest.fixture(scope="module")
def wide_kernels(tmp_path_factory):
    """Their assembly by element type and kind of results (compiled side by side: half a minute each)."""
    kinds = [(dtype, results) for dtype in ("F16", "BF16") for results in ("WD_16", "WD_16_HALF")]

    def assembly(kind):
        shapes = ["fwd_wide_kernel<MAXSIM_%s, WideShape<%s>, false, %s>" % (kind[0], shape, kind[1]) for shape in WIDE_SHAPES]
        return list(zip(shapes, kernel_bodies(tmp_path_factory.mktemp("_".join(kind)), shapes, (), "forward_wide_impl.h", ", int, int")))
    with concurrent.futures.ThreadPoolExecutor(4) as pool:
        return dict(zip(kinds, pool.map(assembly, kinds)))


@pytest.mark.parametrize("results", ["WD_16", "WD_16_HALF"])
@pytest.mark.parametrize("dtype", ["F16", "BF16"])
def test_wide_kernel_waits_along_every_path(wide_kernels, dtype, results):
    """The 16x16 MFMAs of the wide kernel are assembly, which the compiler does not see through: an accumulator is read or written by
    other instructions only some cycles after the MFMA that writes it (11 for four passes), an MFMA does not read what a vector
    instruction wrote less than two cycles ago, along any path, and nothing spills.  In every shape that with_shape knows."""
    header = open(os.path.join(B.CSRC, "forward_wide_impl.h")).read()
    assert set(re.findall(r"return f\(WideShape<([0-9, ]+)>", header)) == set(WIDE_SHAPES)
    for name, body in wide_kernels[dtype, results]:
        assert "scratch_" not in body, name
        assert body.count("v_mfma_f32_16x16x32") > 0, name
        assert too_early(body) == [], name
