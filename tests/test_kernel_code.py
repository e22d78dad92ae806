"""The gfx950 code of inner loops whose source form once compiled into something slower with the same results: the
kernels are compiled to assembly here and their loops' instructions counted. (hipcc needs no GPU for this.)"""

import os
import re
import subprocess

import pytest

from paper_2605_14220_amd.build import CSRC, FLAGS, HIPCC, INCLUDE


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    done = {}

    def compile_(name):
        if name not in done:
            out = str(tmp_path_factory.mktemp("asm") / f"{name}.s")
            flags = [f for f in FLAGS if f not in ("-shared", "-fPIC")]
            subprocess.run([HIPCC, *flags, "-I", INCLUDE, "-I", CSRC, "--cuda-device-only", "-S",
                            os.path.join(CSRC, f"{name}.hip"), "-o", out], check=True, capture_output=True)
            done[name] = open(out).read().splitlines()
        return done[name]

    return compile_


def _loops(lines, kernel):
    """The instruction names of every loop (a backward branch and all from its target) of the kernel whose mangled
    name holds `kernel`, the shortest first."""
    start = next(i for i, l in enumerate(lines) if re.match(r"_Z\S*:", l) and kernel in l.split(":")[0])
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    body = lines[start:end]
    label = {m[1]: i for i, l in enumerate(body) if (m := re.match(r"(\.LBB\w+):", l))}
    loops = []
    for i, l in enumerate(body):
        m = re.search(r"s_c?branch\w* (\.LBB\w+)", l)
        if m and label.get(m[1], i) < i:
            loops.append([x.split()[0] for x in body[label[m[1]]:i + 1] if re.match(r"\t[a-z]", x)])
    return sorted(loops, key=len)


@pytest.mark.parametrize("blocks", [1, 4])
def test_ppo_clip_is_no_branch(assembly, blocks):
    """A token's clip decision is arithmetic on the lanes' values: no lane is masked off inside the token loop but
    for the tokens past the response's end (which, with four blocks of threads, the loop tests by itself)."""
    loops = [l for l in _loops(assembly("ppo"), f"ppo_kernelILi{blocks}E") if any("_f64" in x for x in l)]
    assert loops
    masks = sum(x.startswith("s_and_saveexec") for x in loops[0])
    print(f"{blocks} block(s): {len(loops[0])} instructions, {masks} masked regions")
    assert masks == (0 if blocks == 1 else 2)


@pytest.mark.parametrize("shape", ["ILi1ELi2ELb1ELb0E", "ILi1ELi2ELb1ELb1E", "ILi1ELi4ELb1ELb0E", "ILi1ELi4ELb0ELb0E",
                                   "ILi2ELi4ELb0ELb0E"])
def test_k_loop_moves_no_accumulators(assembly, shape):
    """The stage loop of the head's tile pass (row blocks, waves along the rows, split-K4, logits dump) issues its 32
    or 64 MFMAs a wave on accumulators that stay where they are: none is copied between the register files."""
    loop = next(l for l in _loops(assembly("lmhead"), f"lmhead_partials{shape}") if any("mfma" in x for x in l))
    mfma = sum("mfma" in x for x in loop)
    moves = sum(x.startswith("v_accvgpr") for x in loop)
    print(f"{shape}: {mfma} MFMAs, {moves} accumulator moves, {len(loop)} instructions")
    assert mfma in (32, 64) and moves == 0


@pytest.mark.parametrize("kernel,rows", [("rmsnorm_dgamma_partILi16E", 16), ("rmsnorm_dgamma_partILi32E", 32),
                                         ("rmsnorm_bwd_bothILi8E", 32)])
def test_column_sums_issue_few_instructions_a_row(assembly, kernel, rows):
    """grad_gamma's block sums are one chain of rows per workgroup, so a call of few blocks takes its time from the
    row loop's instructions: a column per thread, `rows` rows' loads ahead, at most 11 a row (two columns took 15)."""
    loops = [l for l in _loops(assembly("rmsnorm"), kernel) if sum(x == "global_load_ushort" for x in l) == rows]
    assert loops, "no loop over that many rows' loads"
    print(f"{kernel}: {len(loops[0])} instructions for {rows} rows")
    assert len(loops[0]) <= 11 * rows
