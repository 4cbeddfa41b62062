"""Properties of the compiled kernels that no run can show, read from the gfx950 assembly of this library's sources.

A lane's register read by v_readlane holds what the program put there only if the lane is active: a copy or a spill that
the compiler places under a branch moves the active lanes' values.  The token and small-segment kernels hold one round-key
word per lane, so they may read them only while every lane is on, whatever the compiler did this time.

The out-of-line parts of the tile kernel reach its LDS through pointers that the compiler knows, so that they stay right
wherever it places the array."""
import re
import subprocess

import pytest

from paper_2608_25431_amd import build

KERNELS = ["k_tokensILb0E", "k_tokensILb1E", "k_smallILb0E", "k_smallILb1E"]


def hipcc(*flags):
    cmd = ["/opt/rocm/bin/hipcc", f"--offload-arch={build.ARCH}", *build.HIP_FLAGS, "--cuda-device-only", *flags,
           "-I", f"{build.ROOT}/include", "-I", build.CSRC, build.SOURCES[0]]
    return subprocess.run(cmd, capture_output=True, text=True, timeout=300)


def compiled(out, *flags):
    r = hipcc("-S", *flags, "-o", str(out))
    assert r.returncode == 0, r.stderr
    return out.read_text().splitlines()


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    return compiled(tmp_path_factory.mktemp("asm") / "kernels.s")


def body(lines, kernel):
    start = next(i for i, l in enumerate(lines) if re.match(rf"_ZN4gift\d+{kernel}.*:", l))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    return [l.split(";")[0].strip() for l in lines[start + 1:end] if l.split(";")[0].strip()]


def masked_readlanes(code):
    """Indices of the v_readlane instructions that some path reaches with lanes switched off.  The state is whether exec
    is narrowed and, per scalar register pair, whether the mask saved there is; unknown masks count as narrowed."""
    label = {l[:-1]: i for i, l in enumerate(code) if l.endswith(":")}
    seen, found, work = {}, set(), [(0, False, frozenset())]
    while work:
        i, off, full = work.pop()  # full: registers that hold a whole mask
        while i < len(code):
            old = seen.get(i)
            if old is not None:
                off, full = off or old[0], full & old[1]
                if (off, full) == old:
                    break
            seen[i] = (off, full)
            op, _, args = code[i].partition(" ")
            a = [x.strip() for x in args.split(",")]
            if op == "v_readlane_b32" and off:
                found.add(i)
            elif op == "s_endpgm":
                break
            elif op.endswith("saveexec_b64"):
                full = full - {a[0]} if off else full | {a[0]}
                off = True
            elif a[0] == "exec" and op.startswith("s_"):
                src = a[-1]
                off = not (op in ("s_or_b64", "s_mov_b64") and (src in full or src == "-1"))
            elif op.startswith("s_") and a[0] in full:
                full = full - {a[0]}
            if op == "s_branch":
                i = label[a[0]]
                continue
            if op.startswith("s_cbranch"):
                work.append((label[a[0]], off, full))
            i += 1
    return found


@pytest.mark.parametrize("kernel", KERNELS)
def test_lanes_are_read_while_all_are_on(assembly, kernel):
    code = body(assembly, kernel)
    assert sum(l.startswith("v_readlane_b32") for l in code) >= 12  # the loop over the rounds keeps four of them
    assert not masked_readlanes(code)


def test_tag_mask_gets_lds_pointers(tmp_path):
    calls = [l for l in compiled(tmp_path / "kernels.ll", "-emit-llvm") if re.search(r"call .*@_ZN4gift8tag_mask", l)]
    assert len(calls) >= 8  # four modes, one and two teams
    for l in calls:
        assert len(re.findall(r"ptr addrspace\(3\) noundef", l.split("tag_mask", 1)[1])) == 2, l


@pytest.mark.parametrize("rows,builds", [(63, False), (64, True), (129, False), (160, False)])
def test_rows_per_tile_that_the_expansion_takes(rows, builds):
    """The segment-table expansion keeps the row counts of a tile two per lane of a wave: tiles that it would sort into
    the queue wrongly do not build."""
    r = hipcc("-fsyntax-only", f"-DGIFT_ROWS={rows}")
    assert (r.returncode == 0) == builds, r.stderr
    assert builds or "static assertion failed" in r.stderr
